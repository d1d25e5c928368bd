"""The 3D step's linear site order (GPU) on flows that vary in all three directions.

A small lattice repeated py times along y and pz times along z takes the order under test (the
small one goes by rows): every site's operands are those of the small lattice's site, so the
populations are its own repeated, bit for bit.  The periods along y and z differ, so sites
whose y and z were mixed up would not fit.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(mrt=0), dict(mrt=1, s5=1.3, s7=0.7, s8=1.6, sg=1.1, szz=0.9)])
@pytest.mark.parametrize("nx,ny,nz,py,pz,storage", [
    (96, 12, 10, 5, 5, "fp32"),    # plain stores
    (96, 13, 16, 10, 5, "fp32"),   # non-temporal
    (90, 7, 12, 10, 5, "fp16"),    # ragged rows, several rows a block
    (33, 13, 7, 10, 10, "fp16"),   # an uneven last block
    (64, 14, 15, 10, 10, "fp16"),  # non-temporal
    (90, 8, 9, 5, 5, "fp32"),      # row order, plain stores
])
def test_repeated_lattice(nx, ny, nz, py, pz, storage, kw):
    from paper_1607_08675_amd.lattice3 import Lattice3, LBMHD3Config
    rng = np.random.default_rng(nx + ny)
    f = [1.0 + 0.02 * rng.standard_normal((nz, ny, nx))]
    f += [0.02 * rng.standard_normal((nz, ny, nx)) for _ in range(6)]
    out = []
    for a, b in ((1, 1), (pz, py)):
        L = Lattice3(LBMHD3Config(nx=nx, ny=b * ny, nz=a * nz, nu=1e-3, eta=2e-3, les=1,
                                  storage=storage, **kw))
        out.append(L.init_fields(*(np.tile(x, (a, b, 1)) for x in f)).step(3).populations())
    assert torch.equal(out[0].repeat(1, pz, py, 1), out[1])
