"""Fully connected products in 128 x 128 tiles (csrc/fc_split.hip), which a batch reaches with 72 tiles: reductions of one,
four and eight parts, even and uneven, of whole and ragged steps.  A row gives the bits it gives in a small
batch, which runs in blocks of 16 x 32, and both are the FP64 product to FP32 accuracy."""
import numpy as np
import pytest

from test_gpu_split_conv import _P, _fc_net, _run

pytestmark = pytest.mark.gpu

# (terms K, outputs N): steps of 32 terms, parts
DIMS = [
    (100, 300),    # 4 steps, one part
    (250, 100),    # 8 steps in four parts of two; no 16-byte rows
    (784, 100),    # 25 steps in four parts of 6, 6, 6 and 7
    (1000, 257),   # 32 steps in four parts, the last step of 8 terms; outputs one past two tiles
    (2048, 128),   # 64 steps in eight parts of eight
    (2050, 130),   # 65 steps in eight parts of 8, the last of 9, the last step of two terms
    (2100, 100),   # 66 steps in eight parts of 8 and 9
]


@pytest.mark.parametrize("forward", [True, False])
@pytest.mark.parametrize("dims", DIMS)
def test_tiles(dims, forward):
    P = _P()
    K, N = dims
    nodes, rng = _fc_net(*((K, N) if forward else (N, K)), K + N)
    net = P.Net(nodes)
    w = nodes[1]["W"].astype(np.float64)
    w = w.T if forward else w
    add = nodes[1]["b"].astype(np.float64) if forward else 0.0
    name = "fc_forward" if forward else "fc_backsub"
    tiles_n = -(-N // 128)
    M = (-(-72 // tiles_n) - 1) * 128 + 1     # the fewest rows of 72 tiles, one row in the last
    assert -(-M // 128) * tiles_n >= 72
    x = (rng.normal(size=(M, K)) * 10.0 ** rng.uniform(-12, 3, size=(M, K))).astype(np.float32)
    # infinities, NaN and values that round up to an infinity, in the first, a middle and the last term
    for r, (k, v) in enumerate(((0, np.inf), (K - 1, -np.inf), (K // 2, np.nan), (K // 2, 3.4028e38), (K - 1, -3.3961e38))):
        x[200 + r, k] = v
    big = _run(net, name, x, N)
    few = 500                                 # rows of 100 to 130 outputs: 4 to 8 tiles, 12 of 300
    assert -(-few // 128) * tiles_n < 72
    for r0 in (0, M - few):
        assert np.array_equal(_run(net, name, x[r0:r0 + few], N), big[r0:r0 + few], equal_nan=True)
    assert np.array_equal(big[200] == np.inf, w[0] > 0) and np.array_equal(big[200] == -np.inf, w[0] < 0)
    assert np.array_equal(big[201] == np.inf, w[K - 1] < 0) and np.array_equal(big[201] == -np.inf, w[K - 1] > 0)
    assert np.all(np.isnan(big[202]))
    plain = np.r_[0:200, 205:M]
    ref = x[plain] @ w + add
    mag = np.abs(x[plain]).astype(np.float64) @ np.abs(w) + np.abs(add)
    # six part products a term, each FP32 addition within 2^-24 of the magnitudes, and the products left out
    assert np.all(np.abs(big[plain] - ref) <= (6 * K + 21) * 2.0 ** -24 * mag + 1e-37)
    assert np.linalg.norm(big[plain] - ref) <= 2.0 ** -22 * np.linalg.norm(mag)
