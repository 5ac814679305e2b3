"""The peak that bench.py prices a kernel class at: split-operand products against the six-fold bf16 rate, everything
else against the FP32 matrix rate (no GPU)."""
import pytest

import bench
import workloads as W


def _peak(cfg, kind, node, variants=0):
    nodes = W.make_workload(cfg).nodes
    stats = {"name": f"{kind}@node{node}", "count": 10, "ms": 10.0, "flops": 1e12, "bytes": 1e9}
    return bench.roofline_of(stats, None, bench.split_products(nodes, kind, node, variants))["peak"]


@pytest.mark.parametrize("cfg,kind,node,split", [
    # ConvBig: first layer of three input channels on the FP32 kernels, the others and the FC layers split
    (3, "conv_forward", 1, False), (3, "conv_backsub", 1, False), (3, "conv_forward", 3, True), (3, "conv_backsub", 3, True),
    (3, "conv_forward", 5, True), (3, "conv_backsub", 7, True), (3, "fc_forward", 9, True), (3, "fc_backsub", 13, True),
    (3, "conv_forward", -1, True), (3, "fold", -1, False), (3, "bottom", -1, False),
    # ConvSmall: the transposed second convolution on the tap form
    (2, "conv_forward", 3, True), (2, "conv_backsub", 3, False), (2, "conv_forward", 1, False),
])
def test_peak(cfg, kind, node, split):
    assert _peak(cfg, kind, node) == (419.4 if split else 157.3)


def test_peak_with_the_split_kernel_off():
    import paper_2205_00263_amd as P
    off = P.VARIANTS["no_win_conv"]
    assert _peak(3, "conv_forward", 3, off) == 157.3 and _peak(3, "fc_forward", 9, off) == 419.4
