"""Which kernel each direction of a batch runs (fm_batch_walk): the cases of the
window walk's tests do run it, in the workgroup of their level width, schedules
that are asked for run as asked, and a node split in the mode that other tests
leave to the default is checked against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import gpu_run, oracle_J, oracle_ops, rel_l2, rel_l2_pairs, seeded_ds, states_for
from test_gpu_window import case  # noqa: F401

torch = pytest.importorskip("torch")
fm = pytest.importorskip("paper_2609_14982_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,B", [("fp64", 1), ("fp64", 5), ("fp32", 3), ("fp64", 2), ("fp64", "rounds")])
def test_window_cases_run_the_window_walk(case, prec, B):  # noqa: F811
    wl, states, _ = case
    if B == "rounds":
        B = {"window 81x41": 640, "window 61x59x31": 320}.get(wl.name, 640)
    width = wl.N // min(st.stats()[k] for st in states for k in ("levels_fwd", "levels_rev"))
    print(f"case route {wl.name} B={B} {prec} width {width}", flush=True)
    b = fm.Batch(states, B, fm.FM_FP64 if prec == "fp64" else fm.FM_FP32)
    for transpose in (False, True):
        w = b.walk(transpose)
        assert w["kernel"] == "window" and w["window"] > 0 and w["side"] > 0
        assert w["threads"] == (256 if width <= 160 else 512 if width <= 400 else 768)
    b.free()


def test_asked_schedules_run_as_asked(case):  # noqa: F811
    wl, states, _ = case
    for tuning, kernel, threads, unroll in (({"split": 4, "threads": 256, "unroll": 3}, "split", 256, 3),
                                            ({"split": 2, "unroll": 4}, "split", 512, 4),
                                            ({"split": 1}, "groups", 1024, 2),
                                            ({"rhs_per_group": 2, "split": 1, "unroll": 1}, "groups", 1024, 1)):
        b = fm.Batch(states, 16, fm.FM_FP64, tuning=tuning)
        for transpose in (False, True):
            w = b.walk(transpose)
            assert (w["kernel"], w["threads"], w["unroll"]) == (kernel, threads, unroll)
            assert w["window"] == 0 and w["side"] == 0
        b.free()
    # the node split's own default with 16 columns: fewer nodes per thread in the transpose
    b = fm.Batch(states, 16, fm.FM_FP64, tuning={"xcd_aware": 1})
    assert [b.walk(t)["unroll"] for t in (False, True)] == [4, 2]
    assert b.tuning()["unroll"] == 4
    b.free()


def test_multisource_2d_summed_in_the_node_split():
    wl = W.grids.deformed_2d(161, 81, 2024, 0.4, 5, S=6, B=16, R=40, name="c2-family 161x81")
    W.eikonal(wl)
    states, ops, B = states_for(fm, wl), oracle_ops(wl), 16
    print("case node split 161x81 S=6 B=16", flush=True)
    p = seeded_ds(wl, B, 901, per_pair=False)
    y = np.random.default_rng(902).standard_normal((wl.S, wl.rcv.shape[0], B))
    xr, gr = oracle_J(ops, p, False, out="receivers"), O.apply_JT_summed(ops, list(y), "receivers")
    for tun in ({"split": 8}, {"xcd_aware": 1}):
        b = fm.Batch(states, B, fm.FM_FP64, tuning=tun)
        assert b.walk(False)["kernel"] == b.walk(True)["kernel"] == "split"
        b.free()
        x = gpu_run(fm, torch, states, B, fm.FM_FP64, "J", p, fm.FM_DS_BROADCAST, fm.FM_OUT_RECEIVERS, tun)
        assert rel_l2_pairs(x, xr) <= 1e-11
        g = gpu_run(fm, torch, states, B, fm.FM_FP64, "JT", y, fm.FM_W_RECEIVERS, fm.FM_JT_SUMMED, tun)
        assert rel_l2(g, gr) <= 1e-11
