"""Convolutions on the bf16 matrix instructions with FP32 operands cut into three exact parts
(csrc/conv_split.hip): every access pattern at the sizes where tiles, rows per workgroup, channel
groups and stores change, against the FP64 convolution, element by element."""
import numpy as np
import pytest
import torch

from oracle import net as onet

pytestmark = pytest.mark.gpu


def _P():
    import paper_2205_00263_amd as P
    return P


def _net(geom, seed, bf16_weights=False):
    ci, h, co, k, s, p = geom
    rng = np.random.default_rng(seed)
    ho = (h + 2 * p - k) // s + 1
    w = rng.normal(size=(co, ci, k, k)).astype(np.float32)
    if bf16_weights:   # one significant part, the other two zero
        w = (w.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32).copy()
    return [{"kind": "input", "shape": (ci, h, h)},
            {"kind": "conv", "src": 0, "W": w, "b": rng.normal(size=co).astype(np.float32), "stride": s, "pad": p},
            {"kind": "relu", "src": 1},
            {"kind": "fc", "src": 2, "W": np.ones((2, co * ho * ho), np.float32), "b": np.zeros(2, np.float32)}], rng


def _run(net, name, x, width, offset=0):
    """One product into a buffer that starts `offset` floats past a 16-byte boundary."""
    M = len(x)
    x_d = torch.tensor(x, device="cuda")
    buf = torch.full((offset + M * width + 8,), 7.0, device="cuda")
    torch.cuda.synchronize()
    getattr(net, name)(1, x_d.data_ptr(), buf.data_ptr() + 4 * offset, M)
    net.sync()
    out = buf.cpu().numpy()
    assert np.all(out[:offset] == 7.0) and np.all(out[offset + M * width:] == 7.0)   # nothing written beside it
    return out[offset:offset + M * width].reshape(M, width)


GEOMS = [  # (Ci, H, Co, k, s, p)
    # 3x3 / 1: one, two and four channel groups a stage, several stages, one to many rows a workgroup
    (8, 5, 16, 3, 1, 1), (16, 9, 32, 3, 1, 0), (24, 7, 48, 3, 1, 2), (40, 6, 64, 3, 1, 1), (64, 3, 64, 3, 1, 1),
    (32, 12, 64, 3, 1, 1), (32, 33, 32, 3, 1, 1),
    # 2x2 / 1, 1x1 / 2
    (16, 7, 32, 2, 1, 0), (32, 6, 16, 2, 1, 1), (32, 9, 64, 1, 2, 0), (16, 8, 16, 1, 2, 0),
    # 4x4 / 2: phases with different and equal padding, odd planes, an input column no filter reaches
    (16, 8, 32, 4, 2, 1), (16, 9, 48, 4, 2, 2), (32, 13, 32, 4, 2, 0), (64, 10, 64, 4, 2, 0), (16, 30, 16, 4, 2, 1),
    # 3x3 / 2
    (16, 9, 32, 3, 2, 1), (32, 8, 64, 3, 2, 0), (48, 7, 16, 3, 2, 1), (16, 17, 32, 3, 2, 1),
]


@pytest.mark.parametrize("geom", GEOMS)
def test_split_convolution(geom):
    P = _P()
    ci, h, co, k, s, p = geom
    nodes, rng = _net(geom, 11 + sum(geom))
    net, on = P.Net(nodes), onet.Net(nodes)
    din, dout = on.sizes[0], on.sizes[1]
    W64 = nodes[1]["W"].astype(np.float64)
    bias = onet.bias_vector(on, 1)
    for M in (1, 5, 67):
        # magnitudes from 1e-12 to 1e3 side by side
        G = (rng.normal(size=(M, din)) * 10.0 ** rng.uniform(-12, 3, size=(M, din))).astype(np.float32)
        A = (rng.normal(size=(M, dout)) * 10.0 ** rng.uniform(-12, 3, size=(M, dout))).astype(np.float32)
        ref = onet.conv_apply(nodes[1]["W"], G.astype(np.float64), on.shapes[0], on.shapes[1], s, p) + bias
        mag = onet.conv_apply(np.abs(W64), np.abs(G).astype(np.float64), on.shapes[0], on.shapes[1], s, p) + np.abs(bias)
        refb = onet.conv_adjoint(nodes[1]["W"], A.astype(np.float64), on.shapes[0], on.shapes[1], s, p)
        magb = onet.conv_adjoint(np.abs(W64), np.abs(A).astype(np.float64), on.shapes[0], on.shapes[1], s, p)
        # FP32 accumulation of n terms in any order: (n + 1) 2^-24 of the sum of magnitudes at most, six part
        # products per term, and 2^-22 for the part products left out
        tol, tolb = (6 * ci * k * k + 5) * 2.0 ** -24 * mag, (6 * co * k * k + 5) * 2.0 ** -24 * magb
        for offset in (0, 1, 2):
            out, back = _run(net, "conv_forward", G, dout, offset), _run(net, "conv_backsub", A, din, offset)
            assert np.all(np.abs(out - ref) <= tol + 1e-37), (geom, M, offset)
            assert np.all(np.abs(back - refb) <= tolb + 1e-37), (geom, M, offset)
            # and the error is that of a short FP32 sum, not the worst case: 2^-21 in the 2-norm
            assert np.linalg.norm(out - ref) <= 2.0 ** -21 * np.linalg.norm(mag)
            assert np.linalg.norm(back - refb) <= 2.0 ** -21 * np.linalg.norm(magb)


@pytest.mark.parametrize("geom", [(32, 12, 64, 3, 1, 1), (16, 7, 32, 2, 1, 0), (16, 8, 32, 4, 2, 1), (16, 9, 32, 3, 2, 1),
                                  (24, 7, 48, 3, 1, 2), (32, 9, 64, 1, 2, 0)])
@pytest.mark.parametrize("bf16_weights", [False, True])
def test_split_convolution_of_infinities(geom, bf16_weights):
    """An infinite operand gives what an FP32 product gives: infinities of the weight's sign at the outputs
    it reaches, finite values at the others; NaN stays NaN."""
    P = _P()
    ci, h, co, k, s, p = geom
    nodes, rng = _net(geom, 5, bf16_weights)
    net, on = P.Net(nodes), onet.Net(nodes)
    din, dout = on.sizes[0], on.sizes[1]
    for name, n_in, n_out in (("conv_forward", din, dout), ("conv_backsub", dout, din)):
        x = rng.normal(size=(6, n_in)).astype(np.float32)
        at = [int(v) for v in rng.integers(0, n_in, size=5)]
        for r in range(4):
            x[r, at[r]] = np.inf if r % 2 == 0 else -np.inf
        x[4, at[4]] = np.nan
        out = _run(net, name, x, n_out)
        for r in range(5):
            e = np.zeros((1, n_in))
            e[0, at[r]] = -1.0 if r % 2 else 1.0
            if name == "conv_forward":
                hit = onet.conv_apply(nodes[1]["W"], e, on.shapes[0], on.shapes[1], s, p)[0]
            else:
                hit = onet.conv_adjoint(nodes[1]["W"], e, on.shapes[0], on.shapes[1], s, p)[0]
            if r == 4:
                assert np.array_equal(np.isnan(out[r]), hit != 0)
                continue
            assert np.array_equal(out[r] == np.inf, hit > 0) and np.array_equal(out[r] == -np.inf, hit < 0)
            assert np.all(np.isfinite(out[r][hit == 0]))
        assert np.all(np.isfinite(out[5]))


def _fc_net(din, dout, seed):
    rng = np.random.default_rng(seed)
    return [{"kind": "input", "shape": (din, 1, 1)},
            {"kind": "fc", "src": 0, "W": rng.normal(size=(dout, din)).astype(np.float32),
             "b": rng.normal(size=dout).astype(np.float32)},
            {"kind": "relu", "src": 1},
            {"kind": "fc", "src": 2, "W": np.ones((2, dout), np.float32), "b": np.zeros(2, np.float32)}], rng


FC_DIMS = [  # (din, dout): one, four and eight reduction parts, ragged steps, octets and output tiles
    (7, 3), (32, 16), (33, 17), (100, 10), (255, 31), (256, 100), (784, 100), (2050, 130), (100, 2100),
]


@pytest.mark.parametrize("dims", FC_DIMS)
def test_split_fully_connected(dims):
    """Both kernels (a wavefront per reduction part for few rows, 128 x 128 tiles for many) against FP64,
    element by element; a row alone, in a small and in a large batch gives the same bits."""
    P = _P()
    din, dout = dims
    nodes, rng = _fc_net(din, dout, din + dout)
    net = P.Net(nodes)
    W64, b = nodes[1]["W"].astype(np.float64), nodes[1]["b"].astype(np.float64)
    big = 257 * 128 if max(din, dout) <= 256 else 33 * 128 + 1   # 256 tiles or more on one side at least
    for name, n_in, n_out in (("fc_forward", din, dout), ("fc_backsub", dout, din)):
        x = (rng.normal(size=(big, n_in)) * 10.0 ** rng.uniform(-12, 3, size=(big, n_in))).astype(np.float32)
        w = W64.T if name == "fc_forward" else W64
        add = b if name == "fc_forward" else 0.0
        outs = {}
        for M in (1, 17, 130, big):
            outs[M] = _run(net, name, x[:M], n_out)
            assert np.array_equal(outs[M][:1], outs[1])
        assert np.array_equal(outs[big][:130], outs[130])
        ref, mag = x[:130] @ w + add, np.abs(x[:130]).astype(np.float64) @ np.abs(w) + np.abs(add)
        assert np.all(np.abs(outs[130] - ref) <= (6 * n_in + 21) * 2.0 ** -24 * mag + 1e-37)
        assert np.linalg.norm(outs[130] - ref) <= 2.0 ** -22 * np.linalg.norm(mag)
        last = slice(big - 5, big)
        assert np.all(np.abs(outs[big][last] - (x[last] @ w + add)) <=
                      (6 * n_in + 21) * 2.0 ** -24 * (np.abs(x[last]).astype(np.float64) @ np.abs(w) + np.abs(add)) + 1e-37)
        for offset in (1, 2):
            assert np.array_equal(_run(net, name, x[:17], n_out, offset), outs[17])
        y = x[:4].copy()
        y[0, 0], y[1, n_in - 1], y[2, n_in // 2] = np.inf, -np.inf, np.nan
        out = _run(net, name, y, n_out)
        assert np.array_equal(out[0] == np.inf, w[0] > 0) and np.array_equal(out[0] == -np.inf, w[0] < 0)
        assert np.array_equal(out[1] == np.inf, w[n_in - 1] < 0) and np.array_equal(out[1] == -np.inf, w[n_in - 1] > 0)
        assert np.all(np.isnan(out[2])) and np.all(np.isfinite(out[3]))
