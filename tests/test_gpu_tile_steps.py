"""Several steps of a lattice per launch (GPU), the automatic mode's tile kernel: equal
to single steps bit for bit.

A launch takes up to nine steps (three with neighbour terms) of a tile in LDS from a region of
16 x 16, 32 x 32, 32 x 28 or 64 x 32 sites.  The sizes take both regions and both sides of the line
between them, one tile and several with ragged ends, lattices smaller than the region (whose
sites are periodic images of each other) and the step counts every split (one launch, even and
uneven launches, a lone last step), then larger lattices where only whole launches are taken
and the remainder goes by rows.  The reference is the same library with steps_per_pass = 1.
"""
import pytest
import torch

from lbmhd_inputs import random_fields
from state_words import stored_words

pytestmark = pytest.mark.gpu

SIZES = [(2, 2), (3, 5), (8, 8), (9, 40), (64, 64), (200, 200), (201, 200), (24, 1700), (97, 501)]
# the cross-helicity closure's rates at the transport coefficients its other tests use
CLOSURES = {0: {}, 1: {}, 2: dict(delta=1.3), 3: dict(delta=1.3), 4: dict(cs=0.05), 6: {}}


def lattices(nx, ny, les, storage):
    from paper_1607_08675_amd.lattice import Lattice, LBMHDConfig
    kw = dict(nx=nx, ny=ny, nu=2e-3, eta=3e-3, les=les, storage=storage, s5=1.2, s7=1.4, s8=0.9)
    kw.update(CLOSURES[les])
    f = random_fields(nx, ny, seed=nx + 7 * ny, rho_amp=0.004, u_amp=0.02, b_amp=0.02)
    out = []
    for spp in (1, 0):
        L = Lattice(LBMHDConfig(**kw, steps_per_pass=spp))
        L.init_fields(*f)
        out.append(L)
    return out


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("les", sorted(CLOSURES))
@pytest.mark.parametrize("nx,ny", SIZES)
def test_tiles_equal_single_steps(nx, ny, les, storage):
    one, tile = lattices(nx, ny, les, storage)
    for n in (1, 2, 3, 4, 5, 6, 9, 11, 16):
        one.step(n)
        tile.step(n)
        assert one.step_count == tile.step_count
        assert torch.equal(stored_words(one), stored_words(tile)), n


@pytest.mark.parametrize("nx,ny,les,storage", [
    (1000, 1100, 1, "fp32"), (2100, 1900, 1, "fp32"), (1400, 1300, 0, "fp16"),
    (2100, 2000, 1, "fp16"), (1300, 1301, 0, "fp32"), (2300, 2200, 0, "fp16"),
    (2300, 2201, 1, "fp16"), (170000, 20, 1, "fp32"), (900, 1000, 2, "fp32"), (2050, 1100, 2, "fp16"),
    (1100, 1200, 4, "fp16")])
def test_tiles_equal_single_steps_mid_sizes(nx, ny, les, storage):
    one, tile = lattices(nx, ny, les, storage)
    for n in (1, 2, 3, 4, 6, 7, 13):
        one.step(n)
        tile.step(n)
        assert torch.equal(stored_words(one), stored_words(tile)), n


@pytest.mark.parametrize("nx,ny,les,storage,n,every", [
    (64, 64, 1, "fp32", 43, 10), (64, 64, 1, "fp16", 23, 5), (300, 70, 2, "fp32", 13, 4),
    (130, 90, 0, "fp32", 7, 1)])
def test_run_on_tiles_equals_the_plain_sequence(nx, ny, les, storage, n, every):
    one, tile = lattices(nx, ny, les, storage)
    want = []
    for _ in range(n // every):
        one.step(every)
        want.append(one.diag())
    one.step(n % every)
    assert tile.run(n, every) == want
    assert torch.equal(stored_words(one), stored_words(tile))


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("nx,ny", [(5, 3), (64, 64), (333, 250)])
def test_stored_pairs_equal_single_steps(nx, ny, storage):
    one, tile = lattices(nx, ny, 1, storage)
    m = 3
    store = torch.zeros(m, tile.lattice_bytes, dtype=torch.uint8, device="cuda")
    tile.step_store_pairs(tile.save_state(), store, m)
    for k in range(m):
        one.step(2)
        assert torch.equal(stored_words(one), stored_words(tile, store[k])), k
