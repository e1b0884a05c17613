"""The schedule a batch takes by itself: its workgroups are resident at once,
and so are those of a second batch on another stream."""
import numpy as np
import pytest

import workloads as W
from helpers import states_for

torch = pytest.importorskip("torch")
fm = pytest.importorskip("paper_2609_14982_amd")

pytestmark = pytest.mark.gpu

CARD = 256     # resident 512-thread workgroups of the node split, one per CU


@pytest.fixture(scope="module")
def wide():
    """A source amid 65^3 nodes: 97 levels of 2800 nodes on average."""
    wl = W.flat_radial(65, 65, 65, src_ijk=(32, 32, 32))
    wl.rcv = np.arange(0, wl.N, wl.N // 40, dtype=np.int64)
    state = states_for(fm, wl)[0]
    assert state.stats()["levels_fwd"] * 2400 <= wl.N
    return wl, state


@pytest.mark.parametrize("S,B", [(12, 8), (16, 16), (5, 16)])
def test_two_default_batches_fit_on_two_streams(wide, S, B):
    wl, state = wide
    print(f"case two default batches 65^3 S={S} B={B}", flush=True)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    batches = [fm.Batch([state] * S, B, fm.FM_FP64, tuning={"xcd_aware": 1}, stream=s) for s in streams]
    for b in batches:
        t = b.tuning()
        assert t["split"] > 1 and t["threads"] == 512
        assert 2 * 8 * ((S + 7) // 8) * t["split"] <= CARD
    rng = np.random.default_rng(61)
    w = torch.from_numpy(rng.standard_normal((S, b.R, B))).cuda()
    ds = torch.from_numpy(rng.standard_normal((b.N, B))).cuda()
    y = [torch.empty(S, b.R, B, dtype=torch.float64, device="cuda") for _ in range(3)]
    g = [torch.empty(b.N, B, dtype=torch.float64, device="cuda") for _ in range(3)]

    def both(b, i):
        b.apply_J(ds, fm.FM_DS_BROADCAST, y[i], fm.FM_OUT_RECEIVERS)
        b.apply_JT(w, fm.FM_W_RECEIVERS, g[i], fm.FM_JT_SUMMED)

    torch.cuda.synchronize()
    both(batches[0], 2)                  # alone
    batches[0].status()
    for _ in range(3):
        for b, i in zip(batches, (0, 1)):
            both(b, i)
    for b in batches:
        b.status()
    for i in (0, 1):
        assert torch.equal(y[i], y[2]) and torch.equal(g[i], g[2])
    for b in batches:
        b.free()


@pytest.mark.parametrize("S", [16, 24, 40])
def test_receiver_inputs_count_in_the_choice(S):
    """256-thread workgroups, two per CU until the receiver inputs (124 of four
    entries, 16 columns, 64 KB) leave LDS for one: the default takes fewer."""
    wl = W.flat_radial(21, 21, 11)
    wl.rcv, wl.rcv_w, _ = W.interpolating_receivers(wl, 124, 62)
    state = states_for(fm, wl)[0]
    print(f"case receiver inputs 21x21x11 S={S}", flush=True)
    B = 16
    b = fm.Batch([state] * S, B, fm.FM_FP64, tuning={"threads": 256})
    assert b.tuning()["split"] > 1 and 8 * ((S + 7) // 8) * b.tuning()["split"] <= CARD
    one = fm.Batch([state], B, fm.FM_FP64, tuning={"split": 1})
    rng = np.random.default_rng(63)
    w = torch.from_numpy(rng.standard_normal((1, b.R, B))).cuda()
    got = torch.empty(S, b.N, B, dtype=torch.float64, device="cuda")
    ref = torch.empty(1, b.N, B, dtype=torch.float64, device="cuda")
    b.apply_JT(w.expand(S, -1, -1).contiguous(), fm.FM_W_RECEIVERS, got, fm.FM_JT_PER_SOURCE)
    one.apply_JT(w, fm.FM_W_RECEIVERS, ref, fm.FM_JT_PER_SOURCE)
    b.status()
    one.status()
    assert torch.linalg.norm(got - ref) <= 1e-13 * torch.linalg.norm(ref.expand_as(got))
    b.free()
    one.free()
