"""The one-pass friction report at the edges of its row widths: every number
of waves and loads per row filled exactly, one column over, and one short of
a whole 4-column group, with row counts that leave workgroups and wave
groups partly empty, and tensors that start at any 4-byte boundary.  Against
the fp64 oracle, with the bounds of test_gpu_diag.py (fp64 sums in another
order; an SVD for sigma_1)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_30342_amd import rikfad as R

from parity import log

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# Widths below 4 take one column per lane (workgroups of 16 rows and of
# more), widths above 16384 the two-pass iteration.
SHAPES = [(9, 3), (1000, 3), (5000, 2), (33000, 1), (40000, 3), (1, 1), (40, 4), (33, 5), (300, 255),
          (17, 256), (16, 257), (5000, 513), (15, 769), (4099, 1023), (1, 1024), (3, 2047),
          (9, 2049), (1030, 4096), (5, 4097), (21, 8193), (6, 12289), (13, 16383), (7, 16384),
          (3, 16385), (2049, 16390)]


@pytest.mark.parametrize("m,n", SHAPES, ids=[f"{m}x{n}" for m, n in SHAPES])
def test_report_at_row_width_edges(m, n):
    off = (m + n) % 4                   # elements before the tensor
    log(f"[case] friction report {m}x{n} offset {off}")
    rng = np.random.default_rng(m * 20000 + n)
    xi = sum(np.outer(rng.random(m), rng.random(n)) for _ in range(3))
    xi = (xi + 0.05 * rng.random((m, n))).astype(np.float32)
    buf = torch.full((m * n + off + 4,), float("nan"), device="cuda")   # neighbours poison sums
    buf[off:off + m * n] = torch.from_numpy(xi).view(-1)
    got = R.rikfad_friction_report(buf.data_ptr() + 4 * off, m, n, 1e-8, 60,
                                   torch.cuda.current_stream().cuda_stream)
    want = O.friction_report(xi.astype(np.float64), 1e-8)
    for k in ("xi_fro2", "sum_r", "sigma1", "stable_rank"):
        assert got[k] == pytest.approx(want[k], rel=1e-9), k
    assert got["err_fro2"] == pytest.approx(want["err_fro2"], rel=1e-9,
                                            abs=1e-12 * want["xi_fro2"])
    assert got["eckart_young_floor"] == pytest.approx(want["eckart_young_floor"], abs=1e-6)


def test_report_of_zero_and_nonfinite_tensors():
    """A zero tensor has no direction (sigma_1 = 0, no division by 0); a
    non-finite entry reaches every sum over it."""
    s = torch.cuda.current_stream().cuda_stream
    z = torch.zeros(50, 300, device="cuda")
    got = R.rikfad_friction_report(z.data_ptr(), 50, 300, 0.0, 5, s)
    assert (got["xi_fro2"], got["err_fro2"], got["sum_r"], got["sigma1"]) == (0.0, 0.0, 0.0, 0.0)
    z[49, 299] = float("inf")
    got = R.rikfad_friction_report(z.data_ptr(), 50, 300, 0.0, 5, s)
    assert got["sum_r"] == float("inf") and got["xi_fro2"] == float("inf")
