"""FP64 diagnostics over every strip height (GPU) against the oracle on the decoded state.

The strips of the diagnostics pass are 1 to 64 rows tall, by the number of 256-column tiles
times rows.  The sizes take one-row strips (up to a single tile of 1024 rows), the first taller
ones with a ragged last strip, and several tiles with a ragged last tile.  The oracle gets the
library's own decoded populations, so only FP64 rounding is left: both sides sum n terms of
like sign to within 1e-10 of the sum (n eps for n below 10^6 terms of size one), and the sums
whose terms cancel to within 1e-13 n (terms below 0.1, partial sums below sqrt(n) of them).
"""
import pytest
import torch

from lbmhd_inputs import random_fields

pytestmark = pytest.mark.gpu

SIZES = [(2, 2), (5, 3), (64, 64), (300, 7), (256, 1024), (257, 1023), (200, 2050), (700, 1025)]


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_diagnostics_at_every_strip_height(nx, ny, storage):
    from oracle import oracle as orc
    from paper_1607_08675_amd.lattice import Lattice, LBMHDConfig
    L = Lattice(LBMHDConfig(nx=nx, ny=ny, nu=0.01, eta=0.01, les=1, cs=0.1, storage=storage))
    L.init_fields(*random_fields(nx, ny, seed=nx + ny)).step(2)
    got = L.diag()
    want = orc.diag(orc.Params(nx, ny, nu=0.01, eta=0.01, les=True, cs=0.1),
                    L.populations().cpu().numpy())
    n = nx * ny
    for k in ("mass", "e_kin", "e_mag", "enstrophy", "current_sq", "max_abs_divB", "max_u"):
        assert abs(got[k] - want[k]) <= 1e-10 * abs(want[k]), (k, got[k], want[k])
    for k in ("mom_x", "mom_y", "flux_x", "flux_y", "cross_helicity"):
        assert abs(got[k] - want[k]) <= 1e-13 * n, (k, got[k], want[k])
    assert got["nonfinite"] == 0
    assert got == L.diag() == L.diag_noalloc()
    torch.cuda.synchronize()
