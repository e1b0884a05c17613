"""The first-arrival solver's lists of recomputed nodes at their edges: grids
of one list tile (4096 nodes), one node less or a row more, grids that end
inside a 64-node word, a grid that is all seeds, and convergence at exactly
max_iter iterations; one source (an iteration in one launch) and forty equal
ones (listed).  Against the Jacobi oracle: 1e-14 relative (the bar of
test_gpu_eikonal.py), the same number of iterations."""
import numpy as np
import pytest

import workloads as W
from oracle import eikonal as E

torch = pytest.importorskip("torch")
fm = pytest.importorskip("paper_2609_14982_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(16, 16, 16), (15, 21, 13), (17, 16, 16), (3, 3, 3), (9, 9, 9)])
@pytest.mark.parametrize("S", [1, 40])
def test_lists_match_oracle(n, S):
    wl = W.smooth_3d(*n, topo_amp=0.1, with_T=False)
    s = wl.s * (1.0 + 0.2 * np.sin(wl.X[:, 0]))
    xi = np.array([[1.0, 1.0, 0.5]])
    rho = 20.0 if n == (9, 9, 9) else 1.0
    print(f"case eikonal lists {n} S={S} rho={rho}", flush=True)
    ref, rit = E.solve_point(3, *n, wl.X, s, xi[0], rho)
    solver = fm.Eikonal(3, *n, wl.X, S)
    T = torch.empty((S, wl.N), dtype=torch.float64, device="cuda")
    sd = torch.from_numpy(s).cuda()
    for limit in (100000, rit):
        T.fill_(float("nan"))
        assert solver.solve(sd, np.tile(xi, (S, 1)), rho, T, limit) == rit
        assert np.max(np.abs(T.cpu().numpy() - ref)) <= 1e-14 * ref.max()
    if rit > 1:
        with pytest.raises(fm.FmError):
            solver.solve(sd, np.tile(xi, (S, 1)), rho, T, rit - 1)
    solver.free()
