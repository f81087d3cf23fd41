"""The degree transfers at the edges of their element blocks: every degree pair of the hierarchy,
element counts that leave a remainder of a block or fill less than one, two right-hand sides, against
the FP64 oracle."""
import numpy as np
import pytest

from oracle import transfer as otr
from paper_2608_14123_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip('torch')


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2608_14123_amd import binding as b
    return b


# blocks hold 28, 16, 10, 7, 5, 4 and 3 elements at fine degrees 2 to 8; two right-hand sides follow
# each other element by element, so 2, 22 and 58 elements are transferred
@pytest.mark.parametrize('p', range(2, 9))
@pytest.mark.parametrize('ext', [(1, 1, 1), (11, 1, 1), (29, 1, 1)])
def test_transfer_tile_edges(binding, p, ext):
    print('transfer', p, ext, flush=True)
    nbr, bcs = W.box_topology(*ext, bc_code=W.DIRICHLET)
    X = W.element_coords(W.box_vertices(*ext), binding.gll(p)[0], None)
    E, R, pc = len(X), 2, max(1, p // 2)
    lib = binding.Solver(np.full(E, p, np.int32), X, nbr, bcs,
                         binding.default_options(n_rhs=R, order=binding.ORDER_NATURAL))
    l = lib.n_levels
    rng = np.random.default_rng(60 + p)
    sf, sc = (R * E,) + (p + 1,) * 3, (R * E,) + (pc + 1,) * 3
    uf, uc, ub = rng.uniform(-1, 1, sf), rng.uniform(-1, 1, sc), rng.uniform(-1, 1, sc)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x.ravel())).cuda()
    out = torch.full((uc.size,), np.nan, dtype=torch.float64, device='cuda')
    fine, bare = dev(uf), dev(uf)
    # sums of at most 3 (p + 1) products of entries of order one, as on the parity meshes
    def close(got, ref):
        assert np.abs(got.cpu().numpy() - ref.ravel()).max() <= 1e-13 * np.abs(ref).max(), (p, ext)
    lib.project(l, dev(uf), out)
    close(out, otr.project(pc, p, uf))
    lib.restrict(l, dev(uf), out)
    close(out, otr.restrict(pc, p, uf))
    lib.prolong_add(l, dev(uc), fine, ubar=dev(ub))
    close(fine, uf + otr.prolong(pc, p, uc - ub))
    lib.prolong_add(l, dev(uc), bare)
    close(bare, uf + otr.prolong(pc, p, uc))
    lib.close()
