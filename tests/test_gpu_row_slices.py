"""ReLU folds and relaxations whose rows are cut into slices, a' kept for unstable neurons only, and
objective rows read from the filters (csrc/relu.hip): layer widths around the 256 neurons of a
workgroup and row counts around the slices of 32 and 64 rows, against the FP64 oracle's bounds and
analytic gradients."""
import numpy as np
import pytest

from oracle import backsub as ob
from oracle import bab as obab
from oracle import net as onet
from oracle import optimize as oo

from _common import assert_parity, root_unstable

pytestmark = pytest.mark.gpu


def _fc(rng, src, din, dout):
    return {"kind": "fc", "src": src, "W": (rng.normal(size=(dout, din)) / np.sqrt(din)).astype(np.float32),
            "b": (0.1 * rng.normal(size=dout)).astype(np.float32)}


def _conv(rng, src, ci, co, k, s, p):
    return {"kind": "conv", "src": src, "W": (rng.normal(size=(co, ci, k, k)) / np.sqrt(ci * k * k)).astype(np.float32),
            "b": (0.1 * rng.normal(size=co)).astype(np.float32), "stride": s, "pad": p}


def _check(nodes, d0, seed, radius):
    """Bounds and gradients of every set of a split subproblem with random parameters."""
    import paper_2205_00263_amd as P
    rng = np.random.default_rng(seed)
    x = rng.normal(size=d0)
    lo, hi = (x - radius).astype(np.float32), (x + radius).astype(np.float32)
    C, c0 = rng.normal(size=(2, nodes[-1]["W"].shape[0])).astype(np.float32), np.zeros(2, np.float32)
    net_o = onet.Net(nodes)
    q = oo.Query(net_o, lo, hi, C, c0, None, 0.0)
    root, _ = oo.root_pass(q)
    pb = P.Problem(P.Net(nodes), n_spec=2, capacity=8)
    rid, _, _ = pb.bound_init(lo, hi, C, c0)
    j0 = int(root_unstable(net_o, root)[0][0])
    gid = int(pb.branch_split([rid], [0], [j0])[0])
    osub = obab.branch_split(net_o, root, 0, j0)[0]
    offs = np.cumsum([0] + [net_o.sizes[i] for i in net_o.relus])
    for key in oo.set_keys(net_o):
        alpha = rng.uniform(0, 1, offs[-1]).astype(np.float32)
        beta = rng.uniform(0, 0.5, offs[-1]).astype(np.float32)
        pb.set_params(gid, P.set_index(key), alpha=alpha, beta=beta)
        for t, i in enumerate(net_o.relus):
            if i in osub.sets[key]:
                osub.sets[key][i]["alpha"] = alpha[offs[t]:offs[t + 1]].astype(np.float64)
                osub.sets[key][i]["beta"] = beta[offs[t]:offs[t + 1]].astype(np.float64)
    pb.bound_optimize([gid], steps=0)
    oo.bound_optimize(q, osub, steps=0)
    rows = []
    for key in oo.set_keys(net_o):
        lbr, ga, gb, _ = pb.bound_grad(gid, P.set_index(key))
        if key == "final":
            start, const = ob.spec_start(net_o, q.C), q.c0
        else:
            m, s = key
            st = osub.states[net_o.relus[m]]
            js = np.nonzero((st.l < 0) & (st.u > 0))[0]
            start, const = ob.neuron_start(net_o, net_o.relus[m], js, s), np.zeros(len(js))
            rows.append(len(js))
        if len(const) == 0:
            assert len(lbr) == 0
            continue
        out = ob.backsub(net_o, start, const, osub.states, osub.sets[key], None, lo, hi)
        assert_parity(lbr, out["lb"], f"{key} rows")
        g = oo.bound_grads(net_o, out)
        for name, got in (("alpha", ga), ("beta", gb)):
            ref = np.concatenate([g[i][name] if i in g else np.zeros(net_o.sizes[i]) for i in net_o.relus])
            assert np.linalg.norm(got - ref) <= 1e-3 * max(np.linalg.norm(ref), 1e-6), (key, name)
    return rows


@pytest.mark.parametrize("width,rows", [(5, 33), (255, 31), (256, 32), (257, 64), (511, 65), (513, 129), (300, 700)])
def test_row_slices_of_fully_connected_layers(width, rows):
    rng = np.random.default_rng(width + rows)
    nodes = [{"kind": "input", "shape": (12, 1, 1)}, _fc(rng, 0, 12, width), {"kind": "relu", "src": 1},
             _fc(rng, 2, width, rows), {"kind": "relu", "src": 3}, _fc(rng, 4, rows, 3)]
    nodes[3]["b"][:] = 0
    used = _check(nodes, 12, 5, 0.6)
    assert max(used) > rows // 2   # most rows of the second layer take part


@pytest.mark.parametrize("rows", [63, 64, 65, 1023, 1024, 1025, 2049])
def test_rows_of_wide_layers(rows):
    """Row lists built by sixteen wavefronts, 64 neurons at a time."""
    rng = np.random.default_rng(rows)
    nodes = [{"kind": "input", "shape": (8, 1, 1)}, _fc(rng, 0, 8, 30), {"kind": "relu", "src": 1},
             _fc(rng, 2, 30, rows), {"kind": "relu", "src": 3}, _fc(rng, 4, rows, 3)]
    _check(nodes, 8, 5, 0.6)


@pytest.mark.parametrize("k,s,p", [(3, 1, 1), (4, 2, 1), (3, 2, 0), (2, 1, 0), (1, 2, 0)])
def test_objective_rows_from_filters(k, s, p):
    rng = np.random.default_rng(10 * k + s)
    ho = (7 + 2 * p - k) // s + 1
    nodes = [{"kind": "input", "shape": (1, 7, 7)}, _conv(rng, 0, 1, 6, 3, 1, 1), {"kind": "relu", "src": 1},
             _conv(rng, 2, 6, 5, k, s, p), {"kind": "relu", "src": 3}, _fc(rng, 4, 5 * ho * ho, 3)]
    _check(nodes, 49, 6, 0.4)


@pytest.mark.parametrize("filter_first", [True, False])
def test_objective_rows_from_filters_of_a_sum(filter_first):
    """A block whose one branch starts at the first ReLU of the pass and whose other one does not."""
    rng = np.random.default_rng(21)
    nodes = [{"kind": "input", "shape": (1, 6, 6)}, _conv(rng, 0, 1, 4, 3, 1, 1), {"kind": "relu", "src": 1},
             _conv(rng, 2, 4, 4, 3, 1, 1), {"kind": "relu", "src": 3}, _conv(rng, 4, 4, 5, 3, 2, 1), _conv(rng, 2, 4, 5, 1, 2, 0),
             {"kind": "add", "src": 5 if filter_first else 6, "src2": 6 if filter_first else 5},
             {"kind": "relu", "src": 7}, _fc(rng, 8, 45, 3)]
    _check(nodes, 36, 7, 0.3)


@pytest.mark.parametrize("n", [1, 223, 224, 225, 448, 449, 897, 1793])
def test_uploads_of_every_length(n):
    """Lists of n splits and 2 n subproblems around the lengths that travel in one kernel's arguments
    (896 words), in several (3584) and by a copy: equal splits of one parent have equal bounds."""
    import paper_2205_00263_amd as P
    rng = np.random.default_rng(3)
    nodes = [{"kind": "input", "shape": (6, 1, 1)}, _fc(rng, 0, 6, 24), {"kind": "relu", "src": 1},
             _fc(rng, 2, 24, 9), {"kind": "relu", "src": 3}, _fc(rng, 4, 9, 3)]
    x = rng.normal(size=6)
    pb = P.Problem(P.Net(nodes), n_spec=2, capacity=2 * n + 24)
    rid, _, _ = pb.bound_init(x - 0.5, x + 0.5, rng.normal(size=(2, 3)), np.zeros(2))
    W1 = nodes[1]["W"].astype(np.float64)
    few = np.nonzero(np.abs(W1 @ x + nodes[1]["b"]) < 0.4 * np.abs(W1).sum(1))[0][:4]   # unstable
    alone = np.array([pb.bound_optimize(pb.branch_split([rid], [0], [int(j)]), steps=0)[0] for j in few])
    lb, _ = pb.bound_optimize(pb.branch_split([rid] * n, [0] * n, few[np.arange(n) % len(few)]), steps=0)
    assert np.array_equal(lb.reshape(n, 2, -1), alone[np.arange(n) % len(few)])
