"""What bench.py says ran: the kernel of each direction as the batch reports it,
and a schedule that creates the batch again (zeros where only the library's
default does)."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


class Reported:
    def __init__(self, J, JT):
        self.kernels = [J, JT]

    def tuning(self):
        return {"rhs_per_group": 4, "threads": 512, "unroll": 4, "split": 8, "balance": 0}

    def walk(self, transpose=False):
        kernel, unroll = self.kernels[transpose]
        return {"kernel": kernel, "threads": 512, "unroll": unroll, "window": 0, "side": 0}


@pytest.mark.parametrize("J,JT,name,zeros", [
    (("window", 0), ("window", 0), "k_ring", True),
    (("window", 0), ("split", 2), "k_ring", True),
    (("split", 4), ("window", 0), "k_split", True),
    (("split", 4), ("split", 2), "k_split", True),
    (("split", 4), ("split", 4), "k_split", False),
    (("groups", 2), ("groups", 2), "k_sweep", False)])
def test_schedule_names_what_ran(J, JT, name, zeros):
    batch = Reported(J, JT)
    kernel, sched = bench.schedule_report(batch)
    assert kernel == name
    assert (sched["J"]["kernel"], sched["JT"]["kernel"]) == (J[0], JT[0])
    for k, v in batch.tuning().items():
        assert sched[k] == (0 if zeros else v)


def test_window_bytes_of_a_small_state():
    # 10 nodes, 4 rhs, FP64: 24 bytes of rows and 36 of records per node and
    # rhs, 16 per node once, a 3-node block per rhs
    st = {"N": 10, "sum_k2": 9}
    assert bench.window_bytes([st, st], 4, 8) == 2 * (4 * 10 * 60 + 160 + 4 * 72)
    assert bench.window_bytes([st], 4, 4) == 4 * 10 * 40 + 120 + 4 * 72
