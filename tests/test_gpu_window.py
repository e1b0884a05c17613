"""The level walk with the recent node values in LDS (the default schedule of
small and middle-sized batches), against the oracle: the three workgroup
shapes (mean level width up to 160, up to 400, above), levels of more than one
chunk, SCC blocks solved by a dense inverse and by their series, receivers
that interpolate (several on one node), both precisions, one right-hand side
up to more pairs than one round of workgroups, and replays of a captured pass.

The bars are those of the other schedules: 1e-11 in FP64, 1e-4 in FP32.
"""
import numpy as np
import pytest

import workloads as W
from helpers import gpu_run, oracle_J, oracle_JT, oracle_ops, rel_l2, rel_l2_pairs, seeded_ds, states_for

torch = pytest.importorskip("torch")
fm = pytest.importorskip("paper_2609_14982_amd")

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-11, "fp32": 1e-4}
CASES = ["narrow", "blocks", "series", "wide"]


@pytest.fixture(scope="module", params=CASES)
def case(request):
    if request.param == "narrow":
        wl = W.grids.deformed_2d(81, 41, 5100, 0.4, 3, S=3, B=3, R=12, name="window 81x41")
        W.eikonal(wl)
    elif request.param == "wide":
        wl = W.grids.deformed_3d(61, 59, 31, 5200, 1, 1, 3, 1, 1, name="window 61x59x31")
        W.eikonal(wl)
    else:
        wl = W.curved_state(41, 41, 25, A=500.0, eps_T=0.05)
    nodes, w, _ = W.interpolating_receivers(wl, 23, 5300)
    nodes[1], w[1] = nodes[0], w[0]          # two receivers at one place
    wl.rcv, wl.rcv_w = nodes, w
    fm.set_iterative_block_min(2 if request.param == "series" else 0)
    try:
        states = states_for(fm, wl)
    finally:
        fm.set_iterative_block_min(0)
    # the oracle's answers for five right-hand sides, of which a test takes the first B
    ops, n = oracle_ops(wl), wl.T.reshape(wl.S, -1).shape[1]
    rng = np.random.default_rng(5500)
    ref = {"ds": seeded_ds(wl, 5, 5400)}
    ref["x"] = oracle_J(ops, ref["ds"], True)
    ref["y"] = oracle_J(ops, ref["ds"][0], False, out="receivers")
    for name, k in (("nodes", n), ("receivers", nodes.shape[0])):
        ref["w_" + name] = rng.standard_normal((wl.S, k, 5))
        ref["g_" + name] = oracle_JT(ops, ref["w_" + name], name)
    return wl, states, ref


@pytest.mark.parametrize("prec,B", [("fp64", 1), ("fp64", 5), ("fp32", 3)])
def test_window_walk_all_modes(case, prec, B):
    wl, states, ref = case
    p = fm.FM_FP64 if prec == "fp64" else fm.FM_FP32
    tol = TOL[prec]
    print(f"case window {wl.name} S={wl.S} B={B} {prec}", flush=True)
    ds = ref["ds"][..., :B]
    x = gpu_run(fm, torch, states, B, p, "J", ds, fm.FM_DS_PER_PAIR, fm.FM_OUT_NODES)
    assert rel_l2_pairs(x, ref["x"][..., :B]) <= tol
    y = gpu_run(fm, torch, states, B, p, "J", ds[0], fm.FM_DS_BROADCAST, fm.FM_OUT_RECEIVERS)
    assert rel_l2_pairs(y, ref["y"][..., :B]) <= tol
    for mode, name in ((fm.FM_W_NODES, "nodes"), (fm.FM_W_RECEIVERS, "receivers")):
        w, g = ref["w_" + name][..., :B], ref["g_" + name][..., :B]
        each = gpu_run(fm, torch, states, B, p, "JT", w, mode, fm.FM_JT_PER_SOURCE)
        assert rel_l2_pairs(each, g) <= tol
        total = gpu_run(fm, torch, states, B, p, "JT", w, mode, fm.FM_JT_SUMMED)
        assert rel_l2(total, g.sum(axis=0)) <= tol


def test_window_walk_two_rounds(case):
    """Pairs past one round of workgroups: every column is one of three."""
    wl, states, ref = case
    B = {"window 81x41": 640, "window 61x59x31": 320}.get(wl.name, 640)
    print(f"case window rounds {wl.name} S={wl.S} B={B}", flush=True)
    ds = np.tile(ref["ds"][0][:, :3], (1, B // 3 + 1))[:, :B]
    y = gpu_run(fm, torch, states, B, fm.FM_FP64, "J", ds, fm.FM_DS_BROADCAST, fm.FM_OUT_RECEIVERS)
    assert rel_l2_pairs(y[..., :3], ref["y"][..., :3]) <= TOL["fp64"]
    for b in range(3, B):
        assert np.array_equal(y[..., b], y[..., b % 3])


def test_window_walk_replays(case):
    """A captured J then J^T, replayed on changed inputs between eager passes."""
    wl, states, _ = case
    B = 2
    st = torch.cuda.Stream()
    rng = np.random.default_rng(5700)
    with torch.cuda.stream(st):
        b = fm.Batch(states, B, fm.FM_FP64, stream=st)
        ds = torch.zeros(b.N, B, dtype=torch.float64, device="cuda")
        y = torch.empty(b.S, b.R, B, dtype=torch.float64, device="cuda")
        g = torch.empty(b.N, B, dtype=torch.float64, device="cuda")

        def both():
            b.apply_J(ds, fm.FM_DS_BROADCAST, y, fm.FM_OUT_RECEIVERS)
            b.apply_JT(y, fm.FM_W_RECEIVERS, g, fm.FM_JT_SUMMED)

        both()
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            both()
        for _ in range(3):
            ds.copy_(torch.from_numpy(rng.standard_normal((b.N, B))))
            both()
            ref = [y.clone(), g.clone()]
            y.fill_(float("nan"))
            g.fill_(float("nan"))
            graph.replay()
            st.synchronize()
            assert torch.equal(y, ref[0]) and torch.equal(g, ref[1])
        b.status()
        b.free()
