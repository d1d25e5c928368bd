"""The 3D step's site orders and stores (GPU) against the row order of a lattice that takes it.

Sites in linear order, plain stores, both or neither are chosen by the lattice's size.  A flow
that does not vary along z or y steps every (y, z) column alike, so a lattice of a size that
takes another order must reproduce the small lattice's populations bit for bit in each of them.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def run(nx, ny, nz, n, **kw):
    from paper_1607_08675_amd.lattice3 import Lattice3, LBMHD3Config
    L = Lattice3(LBMHD3Config(nx=nx, ny=ny, nz=nz, nu=1e-3, eta=2e-3, les=1, **kw))
    rng = np.random.default_rng(nx)
    f = [(1.0 if q == 0 else 0.0) + 0.02 * rng.standard_normal(nx) for q in range(7)]
    L.init_fields(*(np.broadcast_to(a, (nz, ny, nx)) for a in f)).step(n)
    return L.populations()


# the bytes of two lattices (45 populations a site): FP32 x 360, FP16 x 180
@pytest.mark.parametrize("nx,ny,nz,storage", [
    (96, 60, 50, "fp32"),    # 104 MB, rows of whole lines: linear, plain
    (90, 40, 45, "fp32"),    # 58 MB, ragged rows: row order, plain
    (96, 130, 80, "fp32"),   # 359 MB: linear, non-temporal
    (256, 30, 40, "fp32"),   # 111 MB, one block a row: row order, plain
    (90, 70, 60, "fp16"),    # 68 MB, ragged rows: linear, plain
    (33, 130, 70, "fp16"),   # 54 MB, several rows a block, an uneven last block
    (64, 140, 150, "fp16"),  # 242 MB: linear, non-temporal
])
@pytest.mark.parametrize("kw", [dict(mrt=0), dict(mrt=1, s5=1.3, s7=0.7, s8=1.6, sg=1.1, szz=0.9)])
def test_orders_agree_with_the_small_lattice(nx, ny, nz, storage, kw):
    want = run(nx, 2, 2, 3, storage=storage, **kw)[:, :1, :1]
    got = run(nx, ny, nz, 3, storage=storage, **kw)
    assert torch.equal(got, want.expand_as(got))
