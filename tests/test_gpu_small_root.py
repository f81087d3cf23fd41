"""The one-launch root solve of small hierarchies against the FP64 oracle's SCG: element counts up to its
limit and one beyond (the general path), every kind of boundary, the semidefinite operator, several
right-hand sides, both stopping rules."""
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


CASES = [((1, 1, 1), W.DIRICHLET, False, 0.0), ((3, 2, 1), W.DIRICHLET, False, 0.0), ((4, 4, 4), W.DIRICHLET, False, 0.0),
         ((5, 4, 3), W.NEUMANN, False, 0.7), ((3, 3, 3), W.DIRICHLET, True, 0.5), ((4, 4, 4), W.DIRICHLET, True, 0.0),
         ((3, 4, 4), W.NEUMANN, False, 0.0), ((13, 5, 1), W.DIRICHLET, False, 0.2)]


@pytest.mark.parametrize('ext,bc,periodic,kappa', CASES)
@pytest.mark.parametrize('weighting', ['quintic', 'plain'])
def test_root_solve(binding, ext, bc, periodic, kappa, weighting):
    print('small root', ext, bc, periodic, kappa, weighting, flush=True)
    nbr, bcs = W.box_topology(*ext, periodic=(periodic,) * 3, bc_code=bc)
    V = W.box_vertices(*ext)
    mp = lambda X: W.sine_bump_map(X, 0.02)
    # p = 1 maps of a bump that vanishes at the vertices of coarse grids are still the grid's own
    mesh = Mesh(1, W.element_coords(V, oracle_gll(1)[0], mp), nbr, bcs, kappa=kappa, mu_star=4.0)
    lv = osv.Level(mesh, 1, weighting)
    null = kappa == 0.0 and not (bcs == W.DIRICHLET).any()
    project = osv.project_range if null else None
    E, R = mesh.E, 3
    rng = np.random.default_rng(50)
    g = rng.uniform(-1, 1, (R, 8 * E))
    if null:
        g -= g.mean(axis=1, keepdims=True)
    u0 = rng.uniform(-1, 1, (R, 8 * E))
    for rtol, cap in ((1e-9, 200), (0.0, 6)):
        lib = binding.Solver(np.full(E, 1, np.int32), W.element_coords(V, binding.gll(1)[0], mp), nbr, bcs,
                             binding.default_options(kappa=kappa, mu_star=4.0, n_rhs=R, root_rtol=rtol, root_max_iter=cap,
                                                     null_space=int(null),
                                                     weighting=binding.WEIGHT_PLAIN if weighting == 'plain'
                                                     else binding.WEIGHT_QUINTIC))
        u = torch.from_numpy(u0.ravel()).cuda()
        it = lib.root_solve(u, torch.from_numpy(g.ravel()).cuda())
        torch.cuda.synchronize()
        got = u.cpu().numpy().reshape(R, -1)
        its = []
        for k in range(R):
            x, f = u0[k].reshape(E, 2, 2, 2), g[k].reshape(E, 2, 2, 2)
            r = f - lv.A(x)
            if null:
                r = osv.project_range(r)
            stats = {}
            ref = osv.scg(lv, x, f, cap, r_max=rtol * osv.norm(r), stats=stats, project=project).ravel()
            # the iterates of an FP64 CG agree to rounding times the conditioning of the recurrence
            assert np.abs(got[k] - ref).max() < 1e-7 * np.abs(ref).max(), (ext, rtol, k)
            its.append(stats.get('iters'))
        if rtol > 0 and None not in its:
            assert it == max(its), (it, its)
        lib.close()
