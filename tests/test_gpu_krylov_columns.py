"""The column reductions of LSQR and CGLS at the row widths where their lanes
split differently: one right-hand side, odd counts, more columns than a wave,
the most (256).  Every column is one of five, and a column's solve does not
depend on the others: the sums are grouped differently for each width, which
moves a result by rounding times the condition of three steps, so 1e-10
against the same columns solved five at a time."""
import numpy as np
import pytest

import workloads as W
from helpers import rel_l2, states_for

torch = pytest.importorskip("torch")
fm = pytest.importorskip("paper_2609_14982_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    wl = W.grids.deformed_2d(61, 31, 5800, 0.3, 3, S=3, B=5, R=17, name="columns 61x31")
    W.eikonal(wl)
    states = states_for(fm, wl)
    d = np.random.default_rng(5801).standard_normal((3, 17, 5))
    return states, d, _solve(states, d)


def _solve(states, d):
    B = d.shape[2]
    b = fm.Batch(states, B, fm.FM_FP64)
    rhs = torch.from_numpy(np.ascontiguousarray(d)).cuda()
    out = []
    for solver in (fm.Lsqr(b), fm.Cgls(b, 3)):
        solver.start(rhs)
        solver.iterate(3)
        b.status()
        out.append(solver.x().cpu().numpy())
        out.append((solver.scalars()[3:4] if len(out) == 1 else solver.history()).cpu().numpy())
        solver.free()
    b.free()
    return out


@pytest.mark.parametrize("B", [1, 3, 64, 129, 256])
def test_columns_do_not_depend_on_the_width(case, B):
    states, d, ref = case
    print(f"case krylov columns B={B}", flush=True)
    pick = np.arange(B) % 5
    for got, want in zip(_solve(states, d[:, :, pick]), ref):
        assert rel_l2(got, want[..., pick]) <= 1e-10
