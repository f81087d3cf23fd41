"""What a root solve reports when right-hand sides are not finite: the same from the one-launch solve (64
elements) as from the general one (65)."""
import numpy as np
import pytest

from paper_2608_14123_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip('torch')


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2608_14123_amd import binding as b
    return b


@pytest.mark.parametrize('ext', [(4, 4, 4), (13, 5, 1)])
@pytest.mark.parametrize('value', [np.nan, np.inf])
def test_non_finite_right_hand_sides(binding, ext, value):
    print('small root status', ext, value, flush=True)
    nbr, bcs = W.box_topology(*ext, bc_code=W.DIRICHLET)
    E, R = int(np.prod(ext)), 3
    X = W.element_coords(W.box_vertices(*ext), binding.gll(1)[0], None)
    lib = binding.Solver(np.full(E, 1, np.int32), X, nbr, bcs,
                         binding.default_options(mu_star=2.0, n_rhs=R, root_rtol=1e-9, root_max_iter=200))
    g = np.random.default_rng(8).uniform(-1, 1, (R, 8 * E))

    def solve(g):
        u = torch.zeros(R * 8 * E, dtype=torch.float64, device='cuda')
        return lib.root_solve(u, torch.from_numpy(np.ascontiguousarray(g).ravel()).cuda())

    assert solve(g) > 4
    for k in range(R):   # one of several: a breakdown
        bad = g.copy()
        bad[k, 3] = value
        with pytest.raises(binding.DgfasError) as e:
            solve(bad)
        assert e.value.code == binding.DGFAS_EBREAKDOWN
    assert solve(g) > 4
    # nothing to iterate on: no right-hand side has a residual to reduce
    assert solve(np.full_like(g, np.nan)) == 0
    assert solve(np.zeros_like(g)) == 0
    lib.close()
