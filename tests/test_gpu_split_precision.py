"""Products of the split-operand kernels (csrc/split.h) in the shortest sums: one nonzero term per row, where
nothing averages out, against FP64 and against what one FP32 rounding leaves."""
import numpy as np
import pytest

from oracle import net as onet
from test_gpu_split_conv import _P, _run

pytestmark = pytest.mark.gpu

# (Ci, H, Co, k, s, p): every kind of access pattern
CONVS = [(16, 9, 32, 3, 1, 1), (32, 12, 64, 3, 1, 1), (16, 7, 32, 2, 1, 0), (16, 8, 32, 4, 2, 1), (32, 13, 32, 4, 2, 0),
         (16, 9, 32, 3, 2, 1), (32, 9, 64, 1, 2, 0)]
# (din, dout, rows): one, four and eight reduction parts of the blocks for few rows; 128 x 128 tiles (72 of them)
FCS = [(100, 40, 100), (784, 100, 60), (2050, 130, 40), (300, 256, 36 * 128)]


def _mantissas(rng, shape, e=0):
    return (rng.choice([-1.0, 1.0], size=shape) * rng.uniform(1, 2, size=shape) * 2.0 ** e).astype(np.float32)


def _layer(kind, dims, rng, w_exp=0):
    """A net whose node 1 is the layer, without bias, and the layer's weights."""
    if kind == "conv":
        ci, h, co, k, s, p = dims
        ho = (h + 2 * p - k) // s + 1
        w, shape, width = _mantissas(rng, (co, ci, k, k), w_exp), (ci, h, h), co * ho * ho
        node = {"kind": "conv", "src": 0, "W": w, "b": np.zeros(co, np.float32), "stride": s, "pad": p}
    else:
        din, dout = dims[:2]
        w, shape, width = _mantissas(rng, (dout, din), w_exp), (din, 1, 1), dout
        node = {"kind": "fc", "src": 0, "W": w, "b": np.zeros(dout, np.float32)}
    return [{"kind": "input", "shape": shape}, node, {"kind": "relu", "src": 1},
            {"kind": "fc", "src": 2, "W": np.ones((2, width), np.float32), "b": np.zeros(2, np.float32)}]


def _products(kind, dims, rng, x_exp=0, w_exp=0):
    """Per direction: the kernel's outputs and the exact ones (FP64: one product of 24-bit numbers each)."""
    P = _P()
    nodes = _layer(kind, dims, rng, w_exp)
    net, on = P.Net(nodes), onet.Net(nodes)
    W = nodes[1]["W"].astype(np.float64)
    M = dims[2] if kind == "fc" else 48
    for fwd in (True, False):
        n_in, n_out = (on.sizes[0], on.sizes[1]) if fwd else (on.sizes[1], on.sizes[0])
        x = np.zeros((M, n_in), np.float32)
        x[np.arange(M), rng.integers(0, n_in, size=M)] = _mantissas(rng, M, x_exp)
        out = _run(net, kind + ("_forward" if fwd else "_backsub"), x, n_out).astype(np.float64)
        if kind == "fc":
            ref = x.astype(np.float64) @ (W.T if fwd else W)
        else:
            f = onet.conv_apply if fwd else onet.conv_adjoint
            ref = f(W, x.astype(np.float64), on.shapes[0], on.shapes[1], dims[4], dims[5])
        yield out, ref


@pytest.mark.parametrize("kind,dims", [("conv", d) for d in CONVS] + [("fc", d) for d in FCS])
def test_one_term(kind, dims):
    """With parts rounded to nearest, x = x0 + x1 + x2 and w = w0 + w1 + w2 have |x1|, |w1| <= 2^-8 and
    |x2|, |w2| <= 2^-17 of their leading power of two: the products left out, x1 w2 + x2 w1 + x2 w2, stay
    below 2^-24 + 2^-34 of the product, the sum's one rounding adds 2^-24, the small products' own less than
    2^-28.  Uniform residuals leave out 2^-25 sqrt(2) / 3 in the mean square, against 5.8e-8 of an FP32
    rounding of products of mantissas in [1, 2): 3 % more than that at most."""
    rng = np.random.default_rng(sum(dims))
    err, f32 = [], []
    for out, ref in _products(kind, dims, rng):
        assert np.array_equal(out != 0, ref != 0)
        assert np.all(np.abs(out - ref) <= 2.0 ** -23 * (1 + 2.0 ** -4) * np.abs(ref))
        err.append((out - ref)[ref != 0])
        f32.append((ref.astype(np.float32) - ref)[ref != 0])
    err, f32 = np.concatenate(err), np.concatenate(f32)
    assert len(err) > 2000
    # 3 % by the above, 3.5 % more for the scatter of a norm of 2000 values
    assert np.linalg.norm(err) <= 1.065 * np.linalg.norm(f32), np.linalg.norm(err) / np.linalg.norm(f32)


@pytest.mark.parametrize("kind,dims", [("conv", (16, 9, 32, 3, 1, 1)), ("conv", (16, 8, 32, 4, 2, 1)), ("fc", FCS[0]),
                                       ("fc", FCS[3])])
@pytest.mark.parametrize("w_exp", [-100, -110, -120])
def test_tiny_weights(kind, dims, w_exp):
    """Weights whose lower parts end below FP32's smallest normal number, against operands that bring the products
    back: a part is a multiple of 2^-133 (the smallest bf16 number), so the weight is right to half of that."""
    rng = np.random.default_rng(sum(dims) - w_exp)
    for out, ref in _products(kind, dims, rng, x_exp=100, w_exp=w_exp):
        assert np.all(np.abs(out - ref) <= (2.0 ** -23 * (1 + 2.0 ** -4) + 2.0 ** (-134 - w_exp)) * np.abs(ref))


@pytest.mark.parametrize("dims", [FCS[0], FCS[3]])
def test_infinite_terms_large_weights(dims):
    """An infinite term of a fully connected product meets weights whose lower parts have the other sign, and
    leave FP32's range in a product with its largest number: still the infinity an FP32 product gives."""
    P = _P()
    din, dout, M = dims
    rng = np.random.default_rng(5)
    nodes = _layer("fc", dims, rng, 10)
    net = P.Net(nodes)
    w = nodes[1]["W"].astype(np.float64)
    for name, n_in, n_out, wt in (("fc_forward", din, dout, w.T), ("fc_backsub", dout, din, w)):
        x = rng.normal(size=(M, n_in)).astype(np.float32)
        at = rng.integers(0, n_in, size=M)
        sign = rng.choice([-1.0, 1.0], size=M)
        x[np.arange(M), at] = sign * np.inf
        out = _run(net, name, x, n_out)
        assert np.array_equal(out, np.where(wt[at] * sign[:, None] > 0, np.inf, -np.inf))


@pytest.mark.parametrize("dims", [CONVS[0], CONVS[3], CONVS[5], CONVS[6]])
def test_infinite_terms_large_weights_convolutions(dims):
    """The same for convolutions, with a finite value next to FP32's largest number elsewhere in the row: it is
    cut off, not rounded to an infinity, and its products with 2^-120 are exact to FP32 accuracy."""
    P = _P()
    ci, h, co, k, s, p = dims
    for w_exp in (10, -120):
        rng = np.random.default_rng(7)
        nodes = _layer("conv", dims, rng, w_exp)
        net, on = P.Net(nodes), onet.Net(nodes)
        W = nodes[1]["W"].astype(np.float64)
        for name, f, n_in, n_out in (("conv_forward", onet.conv_apply, on.sizes[0], on.sizes[1]),
                                     ("conv_backsub", onet.conv_adjoint, on.sizes[1], on.sizes[0])):
            M = 12
            e = np.zeros((M, n_in))
            e[np.arange(M), rng.integers(0, n_in, size=M)] = rng.choice([-1.0, 1.0], size=M)
            hit = f(W, e, on.shapes[0], on.shapes[1], s, p)
            if w_exp > 0:
                x = rng.normal(size=(M, n_in)).astype(np.float32)
                x[e != 0] = (e[e != 0] * np.inf).astype(np.float32)
                out = _run(net, name, x, n_out)
                assert np.array_equal(out == np.inf, hit > 0) and np.array_equal(out == -np.inf, hit < 0)
                assert np.all(np.isfinite(out[hit == 0]))
            else:
                big = np.float32(3.4028e38)
                out = _run(net, name, (e * big).astype(np.float32), n_out)
                # cut off, the first part leaves up to 2^-7: twice the bound of rounded parts on each product left
                # out; the weights (2^-120) are right to 2^-14
                assert np.all(np.abs(out - hit * float(big)) <= (2.0 ** -22 + 2.0 ** -14) * np.abs(hit * float(big)))
