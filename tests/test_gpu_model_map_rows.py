"""The model map's row widths: 16-byte parts of a row, and single values where
the row or an address does not allow them (odd counts, arrays one value past a
16-byte boundary); columns of one plane up to several of 16; the smallest
grids.  Against the oracle's matrix with the bars of test_gpu_model_map.py:
1e-14 in FP64, 1e-6 in FP32."""
import numpy as np
import pytest

from helpers import rel_l2
from oracle.model_map import cell_count, model_map_matrix

torch = pytest.importorskip("torch")
fm = pytest.importorskip("paper_2609_14982_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g", [(3, 2, 2, 2), (3, 5, 3, 33), (3, 23, 17, 18), (2, 2, 1, 2), (2, 37, 1, 40)])
@pytest.mark.parametrize("B,off", [(1, 0), (2, 0), (3, 0), (4, 1), (16, 0)])
def test_rows_against_oracle(g, B, off):
    dim, n1, n2, n3 = g
    print(f"case model map rows {g} B={B} offset={off}", flush=True)
    Nc = cell_count(dim, n1, n2, n3)
    rng = np.random.default_rng(5300 + B)
    v = rng.uniform(1.6, 3.2, Nc)
    Mo = model_map_matrix(dim, n1, n2, n3, v)
    N = Mo.shape[0]
    m = fm.ModelMap(dim, n1, n2, n3, v)
    dv, gn = rng.standard_normal((Nc, B)), rng.standard_normal((N, B))
    for dt, tol in ((torch.float64, 1e-14), (torch.float32, 1e-6)):
        def device(a, rows):
            flat = torch.full((rows * B + off,), float("nan"), device="cuda", dtype=dt)[off:]
            t = flat.view(rows, B)
            if a is not None:
                t.copy_(torch.from_numpy(a))
            return t

        ds, mt = device(None, N), device(None, Nc)
        m.apply(device(dv, Nc), ds)
        m.apply_T(device(gn, N), mt)
        torch.cuda.synchronize()
        assert rel_l2(ds.double().cpu().numpy(), Mo @ dv) <= tol
        assert rel_l2(mt.double().cpu().numpy(), Mo.T @ gn) <= tol
    m.free()
