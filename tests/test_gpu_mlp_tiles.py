"""The MLP's matrix products at the edges of their tiles and K-slices.  Inputs, weights and targets are
small whole numbers (times powers of two behind the loss), sparse enough that every BF16 operand and
every FP32 sum is exact: the results equal the FP64 oracle's, whatever the order of the sums."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip('torch')


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2608_14123_amd import binding as b
    return b


def sparse(rng, rows, cols, per_row):
    """Each row has up to per_row entries of +-1."""
    W = np.zeros((rows, cols))
    for _ in range(per_row):
        W[np.arange(rows), rng.integers(0, cols, rows)] = rng.choice([-1.0, 1.0], rows)
    return W


# rows n_out is a power of two, so that the loss's scale is exact.  One value of every size; tiles of 64
# met exactly, by one more and by one less; operands no four of which are aligned (odd n_in, h); K-slices
# that end within a step of 64 (n_in = 700: 352 + 348); slices of the rows (512, 2048)
@pytest.mark.parametrize('n_in,h,n_out,rows', [(1, 1, 1, 1), (37, 63, 8, 32), (64, 64, 64, 64), (65, 68, 2, 128),
                                               (700, 65, 16, 256), (700, 128, 1, 2048), (9, 130, 64, 512)])
def test_products_are_exact(binding, n_in, h, n_out, rows):
    print('mlp tiles', n_in, h, n_out, rows, flush=True)
    rng = np.random.default_rng(n_in + h)
    W1 = sparse(rng, h, n_in, 3).T
    W2, W3 = sparse(rng, h, h, 3), sparse(rng, h, n_out, 3)
    theta = np.concatenate([W1.ravel(), rng.integers(-1, 2, h), W2.ravel(), rng.integers(-1, 2, h), W3.ravel(),
                            rng.integers(-1, 2, n_out)]).astype(np.float64)
    X = rng.integers(-2, 3, (rows, n_in)).astype(np.float64)
    Yo, _ = omlp.forward(theta, X, n_in, h, n_out)
    T = Yo - rng.integers(-3, 4, Yo.shape)
    lo, go = omlp.loss_and_grad(theta, X, T, n_in, h, n_out)
    net = binding.Mlp(n_in, h, n_out, seed=5)
    net.set_params(theta.astype(np.float32))
    # the second input starts four bytes past a 16-byte boundary
    for off in (0, 1):
        Xd = torch.zeros(rows * n_in + 1, dtype=torch.float32, device='cuda')[off:off + rows * n_in]
        Xd.copy_(torch.from_numpy(X.ravel().astype(np.float32)))
        Xd = Xd.view(rows, n_in)
        Y = torch.full((rows, n_out), np.nan, dtype=torch.float32, device='cuda')
        net.forward(Xd, Y)
        grad = torch.full((net.n_params,), np.nan, dtype=torch.float32, device='cuda')
        loss = net.gradient(Xd, torch.from_numpy(T.astype(np.float32)).cuda(), grad)
        torch.cuda.synchronize()
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), Yo)
        assert np.array_equal(grad.cpu().numpy().astype(np.float64), go)
        assert abs(loss - lo) <= 1e-15 * max(1.0, lo)
    net.close()
