"""The Schwarz method's tiles for every degree and overlap that has a kernel, on meshes with one-element
directions (no overlap on either side), boundary sides of both kinds and a periodic wrap, for several
right-hand sides, against the FP64 oracle."""
import numpy as np
import pytest

from oracle.gll import gll as oracle_gll
from oracle.mesh import Mesh
from oracle.schwarz import Schwarz
from paper_2608_14123_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip('torch')

PAIRS = [(p, m) for p in range(1, 9) for m in (0, 1)] + [(4, 2), (8, 2), (8, 3)]


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2608_14123_amd import binding as b
    return b


@pytest.mark.parametrize('p,m', PAIRS)
@pytest.mark.parametrize('ext,bc,periodic', [((3, 2, 1), W.DIRICHLET, False), ((2, 3, 2), W.NEUMANN, False),
                                             ((3, 3, 3), W.DIRICHLET, True)])
def test_schwarz_tile(binding, p, m, ext, bc, periodic):
    print('schwarz tile', p, m, ext, flush=True)
    nbr, bcs = W.box_topology(*ext, periodic=(periodic,) * 3, bc_code=bc)
    V = W.box_vertices(*ext)
    mp = lambda X: W.sine_bump_map(X, 0.02)
    mesh = Mesh(p, W.element_coords(V, oracle_gll(p)[0], mp), nbr, bcs, kappa=0.4, mu_star=2.0)
    sz = Schwarz(mesh, m)
    E, n3, R = mesh.E, (p + 1) ** 3, 2
    r = np.random.default_rng(40 + p).uniform(-1, 1, (R, E * n3))
    # coarser degrees of the hierarchy take an overlap that has a kernel at every degree
    kw = dict(overlap=m) if m < 2 else dict(overlap=-1, delta={(4, 2): 0.24, (8, 2): 0.1, (8, 3): 0.24}[p, m])
    lib = binding.Solver(np.full(E, p, np.int32), W.element_coords(V, binding.gll(p)[0], mp), nbr, bcs,
                         binding.default_options(kappa=0.4, mu_star=2.0, n_rhs=R, **kw))
    assert lib.level_overlap(lib.n_levels) == m
    z = torch.empty(R * E * n3, dtype=torch.float64, device='cuda')
    lib.schwarz(lib.n_levels, torch.from_numpy(r.ravel()).cuda(), z)
    torch.cuda.synchronize()
    got = z.cpu().numpy().reshape(R, -1)
    for k in range(R):
        ref = sz.apply(r[k]).ravel()
        # FP64 sums of the same terms in another order, as on the parity meshes
        assert np.abs(got[k] - ref).max() < 1e-11 * np.abs(ref).max(), (p, m, ext, k)
    lib.close()
