"""The overlap add's tiles of several elements (degrees 5 to 7 on at least 6144 elements) with a last tile that
is not full and two right-hand sides: the sums themselves, and the dot products fused into them through
two SCG steps, in FP64 and FP32, against the C oracle."""
import numpy as np
import pytest

from oracle.gll import gll as oracle_gll
from oracle.o1 import O1
from paper_2608_14123_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip('torch')


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2608_14123_amd import binding as b
    return b


# 6251 elements leave three in the last tile of four (p = 5) and one in the last of two (p = 6, 7); the
# smaller meshes of the other tests take one element a tile
@pytest.mark.parametrize('p', [5, 6, 7])
def test_full_tiles(binding, p):
    ext, R, kappa, mu = (47, 19, 7), 2, 0.4, 3.0
    print('overlap tiles', p, ext, flush=True)
    nbr, bcs = W.box_topology(*ext, bc_code=W.DIRICHLET)
    V = W.box_vertices(*ext)
    mp = lambda X: W.sine_bump_map(X, 0.02)
    ref = O1(p, W.element_coords(V, oracle_gll(p)[0], mp), nbr, bcs, m=1, kappa=kappa, mu_star=mu)
    E, n3 = len(nbr), (p + 1) ** 3
    rng = np.random.default_rng(80 + p)
    r, u0 = rng.uniform(-1, 1, (R, E * n3)), rng.uniform(-1, 1, (R, E * n3))
    top = ref.n_levels
    X = W.element_coords(V, binding.gll(p)[0], mp)
    dev = lambda a: torch.from_numpy(a.ravel()).cuda()
    smoothed = [np.asarray(ref.smooth(top, u0[k], r[k], 2, smoother='scg')).ravel() - u0[k] for k in range(R)]
    for precision, tol in ((binding.FP64, 1e-11), (binding.FP32, 1e-5)):   # as on the parity meshes; the precision tests
        lib = binding.Solver(np.full(E, p, np.int32), X, nbr, bcs,
                             binding.default_options(kappa=kappa, mu_star=mu, n_rhs=R, smoother=binding.SCG,
                                                     precision=precision))
        if precision == binding.FP64:
            z = torch.empty(R * E * n3, dtype=torch.float64, device='cuda')
            lib.schwarz(lib.n_levels, dev(r), z)
            for k in range(R):
                zo = np.asarray(ref.schwarz(top, r[k])).ravel()
                assert np.abs(z.cpu().numpy().reshape(R, -1)[k] - zo).max() < 1e-11 * np.abs(zo).max(), (p, k)
        u = dev(u0)
        lib.smooth(lib.n_levels, u, dev(r), 2)
        torch.cuda.synchronize()
        for k in range(R):
            du = u.cpu().numpy().reshape(R, -1)[k] - u0[k]
            err = np.linalg.norm(du - smoothed[k]) / np.linalg.norm(smoothed[k])
            assert err < tol, (p, precision, k, err)
        lib.close()
    ref.close()
