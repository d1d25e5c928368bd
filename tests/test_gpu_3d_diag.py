"""One-pass FP64 diagnostics of the 3D lattice (GPU) against the oracle on the decoded state.

A block takes a column of 64 x 4 sites through several planes; the sizes have ragged tiles in x
and y, lattices of one plane, one row or one column (every neighbour a periodic image), one
plane per block and several, and more units than blocks.  The oracle gets the library's own
decoded populations, so only FP64 rounding is left (bounds as for the 2D diagnostics: sums of
like sign within 1e-10 of the sum, cancelling sums within 1e-13 per site).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (1, 5, 3), (7, 1, 4), (65, 5, 1), (2, 2, 2), (64, 4, 9), (130, 9, 33),
         (40, 37, 70), (33, 130, 260)]


def lattice(nx, ny, nz, storage):
    from oracle import oracle3 as o3
    from paper_1607_08675_amd.lattice3 import Lattice3, LBMHD3Config
    L = Lattice3(LBMHD3Config(nx=nx, ny=ny, nz=nz, nu=0.01, eta=0.01, les=1, storage=storage))
    rng = np.random.default_rng(nx + 10 * ny + 100 * nz)
    f = [1 + 0.01 * rng.standard_normal((nz, ny, nx))]
    f += [0.05 * rng.standard_normal((nz, ny, nx)) for _ in range(6)]
    L.init_fields(*f).step(1)
    return o3, L, o3.Params(nx, ny, nz, nu=0.01, eta=0.01, les=1, cs=0.1)


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("nx,ny,nz", SIZES)
def test_diagnostics_match_the_oracle(nx, ny, nz, storage):
    o3, L, p = lattice(nx, ny, nz, storage)
    got, want = L.diag(), o3.diag(p, L.populations().cpu().numpy())
    for k in ("mass", "e_kin", "e_mag", "max_u"):
        assert abs(got[k] - want[k]) <= 1e-10 * abs(want[k]), (k, got[k], want[k])
    assert abs(got["max_abs_divB"] - want["max_abs_divB"]) <= 1e-13
    for k in ("mom_x", "mom_y", "mom_z", "flux_x", "flux_y", "flux_z"):
        assert abs(got[k] - want[k]) <= 1e-13 * nx * ny * nz, (k, got[k], want[k])
    assert got["nonfinite"] == 0


def test_nonfinite_sites_are_counted():
    _, L, _ = lattice(66, 5, 7, "fp32")
    x = L.populations()
    x[3, 6, 4, 65] = float("nan")
    x[26, 0, 0, 64] = float("inf")
    L.set_populations(x)
    assert L.diag()["nonfinite"] == 2
    torch.cuda.synchronize()
