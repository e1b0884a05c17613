"""SCC blocks in FP32 batches: c ds of a member enters the block's FP64
right-hand side unrounded, as in the other schedules.  One column per block
with ds on that block's members only, so that nothing upstream is nonzero and
the members' values are A_C^{-1} (c ds) rounded once, to FP32: half a unit in
the last place of each value, and 1e-11 of the block's largest for the FP64
solve."""
import numpy as np
import pytest

import workloads as W
from helpers import gpu_run, oracle_ops, states_for
from oracle import diag

torch = pytest.importorskip("torch")
fm = pytest.importorskip("paper_2609_14982_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_pair", [False, True])
@pytest.mark.parametrize("series", [False, True])
@pytest.mark.parametrize("tuning", [None, {"split": 1}])
def test_block_members_fp32(series, per_pair, tuning):
    wl = W.curved_state(41, 41, 25, A=500.0, eps_T=0.05)
    wl.rcv = np.array([wl.node(5, 7, 0)], dtype=np.int64)
    fm.set_iterative_block_min(2 if series else 0)
    try:
        states = states_for(fm, wl)
    finally:
        fm.set_iterative_block_min(0)
    op = oracle_ops(wl)[0]
    ncomp, lab = diag.scc_labels(op.W)
    size = np.bincount(lab)
    blocks = [np.flatnonzero(lab == c) for c in np.flatnonzero(size > 1)]
    print(f"case fp32 blocks {[len(b) for b in blocks]} series={series} per_pair={per_pair} {tuning}", flush=True)
    assert blocks
    rng = np.random.default_rng(71)
    ds = np.zeros((wl.N, len(blocks)))
    c = op.c.astype(np.float32).astype(np.float64)
    ref = []
    for k, m in enumerate(blocks):
        ds[m, k] = rng.standard_normal(len(m)).astype(np.float32)
        A = np.eye(len(m)) - op.W[m][:, m].toarray()
        ref.append(np.linalg.solve(A, c[m] * ds[m, k]))
    mode = fm.FM_DS_PER_PAIR if per_pair else fm.FM_DS_BROADCAST
    x = gpu_run(fm, torch, states, len(blocks), fm.FM_FP32, "J", ds[None] if per_pair else ds, mode, fm.FM_OUT_NODES,
                tuning)[0]
    for k, m in enumerate(blocks):
        err = np.abs(x[m, k] - ref[k])
        assert np.all(err <= 2.0 ** -24 * np.abs(ref[k]) + 1e-11 * np.abs(ref[k]).max()), float(np.max(err / np.abs(ref[k])))
