"""Output grids of one to sixteen positions on the split-operand convolutions (csrc/conv_split.hip): a lane
stores four consecutive positions of a tile that holds many rows, so on the smallest grids they belong to up
to four rows.  Every output is written, once, in both directions, against the FP64 convolution."""
import numpy as np
import pytest

from oracle import net as onet
from test_gpu_split_conv import _P, _run

pytestmark = pytest.mark.gpu

ONE = [  # (Ci, H, W, Co, k, s, p) whose output is 1x1: every forward pattern; the first one's planes back too
    (16, 1, 1, 32, 3, 1, 1), (16, 3, 3, 32, 3, 1, 0), (8, 3, 3, 16, 3, 1, 0), (64, 3, 3, 64, 3, 1, 0),
    (16, 2, 2, 16, 2, 1, 0), (16, 2, 2, 32, 4, 2, 1), (32, 4, 4, 64, 4, 2, 0), (16, 1, 1, 32, 3, 2, 1),
    (16, 2, 2, 48, 3, 2, 1), (32, 3, 3, 32, 3, 2, 0), (16, 1, 1, 32, 1, 2, 0), (32, 2, 2, 64, 1, 2, 0),
]
# 3x3 / 1 with padding 1: output and input grid of 1 x W and 2 x W positions
SMALL = [(16, 1, w, 32, 3, 1, 1) for w in range(2, 17)] + [(32, 2, w, 64, 3, 1, 1) for w in range(1, 9)]


@pytest.mark.parametrize("geom", ONE + SMALL)
def test_small_grids(geom):
    P = _P()
    ci, h, w, co, k, s, p = geom
    ho, wo = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
    rng = np.random.default_rng(3 + sum(geom))
    nodes = [{"kind": "input", "shape": (ci, h, w)},
             {"kind": "conv", "src": 0, "W": rng.normal(size=(co, ci, k, k)).astype(np.float32),
              "b": rng.normal(size=co).astype(np.float32), "stride": s, "pad": p},
             {"kind": "relu", "src": 1},
             {"kind": "fc", "src": 2, "W": np.ones((2, co * ho * wo), np.float32), "b": np.zeros(2, np.float32)}]
    net, on = P.Net(nodes), onet.Net(nodes)
    W64, bias = nodes[1]["W"].astype(np.float64), onet.bias_vector(on, 1)
    din, dout = on.sizes[0], on.sizes[1]
    for M in (1, 3, 5, 67, 300):
        G = rng.normal(size=(M, din)).astype(np.float32)
        A = rng.normal(size=(M, dout)).astype(np.float32)
        conv = lambda f, W, x: f(W, x.astype(np.float64), on.shapes[0], on.shapes[1], s, p)
        ref = conv(onet.conv_apply, W64, G) + bias
        mag = conv(onet.conv_apply, np.abs(W64), np.abs(G)) + np.abs(bias)
        refb, magb = conv(onet.conv_adjoint, W64, A), conv(onet.conv_adjoint, np.abs(W64), np.abs(A))
        # FP32 accumulation of six part products a term in any order, and the part products left out
        tol, tolb = (6 * ci * k * k + 5) * 2.0 ** -24 * mag, (6 * co * k * k + 5) * 2.0 ** -24 * magb
        for offset in (0, 1):
            out, back = _run(net, "conv_forward", G, dout, offset), _run(net, "conv_backsub", A, din, offset)
            assert np.all(np.abs(out - ref) <= tol), (geom, M, offset, np.argwhere(np.abs(out - ref) > tol)[:4])
            assert np.all(np.abs(back - refb) <= tolb), (geom, M, offset, np.argwhere(np.abs(back - refb) > tolb)[:4])


@pytest.mark.parametrize("geom", [(16, 1, 1, 32, 3, 1, 1), (32, 1, 2, 16, 3, 1, 1), (16, 2, 2, 16, 2, 1, 1)])
def test_small_grids_accumulate(geom):
    """The transposed product added to what the buffer holds."""
    import torch
    P = _P()
    ci, h, w, co, k, s, p = geom
    ho, wo = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
    rng = np.random.default_rng(9)
    nodes = [{"kind": "input", "shape": (ci, h, w)},
             {"kind": "conv", "src": 0, "W": rng.normal(size=(co, ci, k, k)).astype(np.float32),
              "b": np.zeros(co, np.float32), "stride": s, "pad": p},
             {"kind": "relu", "src": 1},
             {"kind": "fc", "src": 2, "W": np.ones((2, co * ho * wo), np.float32), "b": np.zeros(2, np.float32)}]
    net, on = P.Net(nodes), onet.Net(nodes)
    W64 = nodes[1]["W"].astype(np.float64)
    for M in (1, 3, 67):
        A = rng.normal(size=(M, on.sizes[1])).astype(np.float32)
        C = rng.normal(size=(M, on.sizes[0])).astype(np.float32)
        a_d, c_d = torch.tensor(A, device="cuda"), torch.tensor(C, device="cuda")
        torch.cuda.synchronize()
        net.conv_backsub(1, a_d.data_ptr(), c_d.data_ptr(), M, accumulate=True)
        net.sync()
        ref = C + onet.conv_adjoint(W64, A.astype(np.float64), on.shapes[0], on.shapes[1], s, p)
        mag = np.abs(C) + onet.conv_adjoint(np.abs(W64), np.abs(A).astype(np.float64), on.shapes[0], on.shapes[1], s, p)
        assert np.all(np.abs(c_d.cpu().numpy() - ref) <= (6 * co * k * k + 5) * 2.0 ** -24 * mag)
