"""Subdomain solves at degrees 1 and 2 where several share a workgroup (from 4096 of them in FP64
and 5632 in FP32, elements times right-hand sides), and just below, where each has its own: both overlaps, a last workgroup that is not full,
several right-hand sides within one, wavefronts whose subdomains differ in their side variants, a periodic wrap,
overwriting and adding, FP64 and FP32, against the FP64 oracle."""
import numpy as np
import pytest

from oracle import solvers as osv
from oracle.gll import gll as oracle_gll
from oracle.mesh import Mesh
from paper_2608_14123_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip('torch')


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2608_14123_amd import binding as b
    return b


# a workgroup holds 16 or 64 subdomains at p = 1 (m = 1, 0) and 10 or 28 at p = 2; 3 x 4199 of them fill
# none of these a whole number of times.  16^3 is the smallest FP64 launch that is packed, 4080 is below it;
# 4 x 1408 is the smallest in FP32, a number that only the right-hand sides bring about.
@pytest.mark.parametrize('ext,bc,periodic,R', [((17, 19, 13), W.DIRICHLET, False, 3), ((16, 16, 16), W.NEUMANN, True, 1),
                                               ((15, 16, 17), W.NEUMANN, False, 1), ((11, 16, 8), W.DIRICHLET, False, 4)])
@pytest.mark.parametrize('p', [1, 2])
@pytest.mark.parametrize('m', [0, 1])
def test_packed_subdomains(binding, p, m, ext, bc, periodic, R):
    print('schwarz pack', p, m, ext, R, flush=True)
    nbr, bcs = W.box_topology(*ext, periodic=(periodic,) * 3, bc_code=bc)
    V = W.box_vertices(*ext)
    mp = lambda X: W.sine_bump_map(X, 0.02)
    mesh = Mesh(p, W.element_coords(V, oracle_gll(p)[0], mp), nbr, bcs, kappa=0.4, mu_star=2.0)
    lv = osv.Level(mesh, m)
    E, n = mesh.E, p + 1
    rng = np.random.default_rng(70 + 10 * p + m)
    r, u0 = rng.uniform(-1, 1, (R, E * n ** 3)), rng.uniform(-1, 1, (R, E * n ** 3))
    X = W.element_coords(V, binding.gll(p)[0], mp)
    dev = lambda a: torch.from_numpy(a.ravel()).cuda()
    for precision in (binding.FP64, binding.FP32):
        lib = binding.Solver(np.full(E, p, np.int32), X, nbr, bcs,
                             binding.default_options(kappa=0.4, mu_star=2.0, n_rhs=R, overlap=m, smoother=binding.WAS,
                                                     precision=precision))
        if precision == binding.FP64:
            z = torch.empty(R * E * n ** 3, dtype=torch.float64, device='cuda')
            lib.schwarz(lib.n_levels, dev(r), z)
        # two steps: in FP32 the first overwrites the correction and the second adds to it, in FP64 both add
        # to the iterate
        u = dev(u0)
        lib.smooth(lib.n_levels, u, dev(r), 2)
        torch.cuda.synchronize()
        for k in range(R):
            f, x = r[k].reshape(E, n, n, n), u0[k].reshape(E, n, n, n)
            if precision == binding.FP64:
                # FP64 sums of the same terms in another order, as on the parity meshes
                ref = lv.B(f).ravel()
                assert np.abs(z.cpu().numpy().reshape(R, -1)[k] - ref).max() < 1e-11 * np.abs(ref).max(), (p, m, ext, k)
            ref = osv.was(lv, x, f, 2).ravel() - u0[k]
            du = u.cpu().numpy().reshape(R, -1)[k] - u0[k]
            # the update's error, in FP32 that of the precision tests
            err = np.linalg.norm(du - ref) / np.linalg.norm(ref)
            assert err < (1e-11 if precision == binding.FP64 else 1e-5), (p, m, ext, k, err)
        lib.close()
