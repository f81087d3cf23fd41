"""The operator's tiles at the edges of their element blocks: every degree, element counts that leave
a remainder (or less than one block), a nodal diffusivity and kappa, several right-hand sides and a
permuted element order, against the FP64 oracle."""
import numpy as np
import pytest

from oracle.gll import gll as oracle_gll
from oracle.mesh import Mesh
from oracle import operator as oop
from paper_2608_14123_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip('torch')


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2608_14123_amd import binding as b
    return b


# blocks hold 8, 7, 4, 3 elements at p = 1..4 and one from p = 5 on; (2, 1, 1) is less than one
# block, (5, 2, 1) and (3, 3, 3) leave remainders of every block size
@pytest.mark.parametrize('p', range(1, 9))
@pytest.mark.parametrize('ext,bc,kappa', [((2, 1, 1), W.DIRICHLET, 0.0), ((5, 2, 1), W.NEUMANN, 0.7),
                                          ((3, 3, 3), W.DIRICHLET, 0.3)])
def test_operator_tile_edges(binding, p, ext, bc, kappa):
    print('operator tile', p, ext, flush=True)
    nbr, bcs = W.box_topology(*ext, bc_code=bc)
    V = W.box_vertices(*ext)
    mp = lambda X: W.sine_bump_map(X, 0.02)
    Xo = W.element_coords(V, oracle_gll(p)[0], mp)
    nu = 1.0 + 0.5 * np.cos(np.pi * Xo[:, 0]) * np.cos(np.pi * Xo[:, 1])
    mesh = Mesh(p, Xo, nbr, bcs, kappa=kappa, mu_star=2.0, nu=nu)
    E, n3, R = len(Xo), (p + 1) ** 3, 3
    rng = np.random.default_rng(30 + p)
    u, g = rng.uniform(-1, 1, (R, E * n3)), rng.uniform(-1, 1, (R, E * n3))
    lib = binding.Solver(np.full(E, p, np.int32), W.element_coords(V, binding.gll(p)[0], mp), nbr, bcs,
                         binding.default_options(kappa=kappa, mu_star=2.0, n_rhs=R, order=binding.ORDER_MORTON), nu=nu)
    out = torch.empty(R * E * n3, dtype=torch.float64, device='cuda')
    lib.residual(lib.n_levels, torch.from_numpy(u.ravel()).cuda(), torch.from_numpy(g.ravel()).cuda(), out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(R, -1)
    for k in range(R):
        ref = oop.apply(mesh, u[k]).ravel()
        # FP64 sums of the same terms in another order, as on the parity meshes
        assert np.abs(got[k] - (g[k] - ref)).max() < 1e-12 * np.abs(ref).max(), (p, ext, k)
    lib.close()
