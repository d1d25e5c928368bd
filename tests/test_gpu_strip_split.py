"""Row-walking kernels on lattices that do not split evenly (GPU): equal to single steps bit for bit.

The strips of the two- and three-step kernels and of the paired reverse step come from the block
count rounded to whole strips per XCD; the launch then holds strips past the lattice (whose
blocks return at once), or takes plain block order where too many would.  The sizes take both,
with ragged tiles and ragged last strips, and strips of the least and of intermediate heights.
"""
import pytest
import torch

from lbmhd_inputs import random_fields
from state_words import stored_words

pytestmark = pytest.mark.gpu

# strips (triples): 300 x 70 nine of 8 rows, too few to fill up (plain order);
# 600 x 500 63 + 1 past the lattice; 1448 x 700 78 of 9 rows + 2; 2500 x 333
# 42 + 6; 700 x 2900 162 of 18 rows + 6
SIZES = [(300, 70), (600, 500), (1448, 700), (2500, 333), (700, 2900)]


def lattice(nx, ny, spp, **kw):
    from paper_1607_08675_amd.lattice import Lattice, LBMHDConfig
    L = Lattice(LBMHDConfig(nx=nx, ny=ny, nu=2e-3, eta=3e-3, steps_per_pass=spp, **kw))
    L.init_fields(*random_fields(nx, ny, seed=nx + ny, rho_amp=0.004, u_amp=0.02, b_amp=0.02))
    return L


@pytest.mark.parametrize("kw,spp", [
    (dict(les=1), 3), (dict(les=1), 2), (dict(les=1, storage="fp16"), 2), (dict(les=2), 2),
    (dict(les=4, storage="fp16"), 2)])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_uneven_strips_equal_single_steps(nx, ny, kw, spp):
    one, many = lattice(nx, ny, 1, **kw), lattice(nx, ny, spp, **kw)
    assert many.steps_per_pass == spp
    one.step(6)
    many.step(6)
    assert torch.equal(stored_words(one), stored_words(many))


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_uneven_strips_of_the_paired_reverse_step(nx, ny, storage):
    """lambda bit for bit; the closure-constant derivatives to the rounding of
    FP64 sums of the same FP32 contributions (2e6 terms, eps n / 2 of their
    magnitudes' sum; the magnitudes sum to within 1e4 of the derivative)."""
    L = lattice(nx, ny, 1, les=1, storage=storage)
    x0 = L.save_state()
    x1 = L.new_state_buffer()
    L.step_between(x0, x1)
    lam2 = L.new_adj_buffer()
    L.step(2)
    L.adj_seed_energy(L.save_state(), lam2)
    a1, a0, b0 = (torch.zeros_like(lam2) for _ in range(3))
    acc_a, acc_b = L.new_adj_acc(), L.new_adj_acc()
    L.adj_step(x1, lam2, a1, acc_a)
    L.adj_step(x0, a1, a0, acc_a)
    L.adj_step2(x0, lam2, b0, acc_b)
    assert torch.equal(L.adj_view(a0), L.adj_view(b0))
    for a, b in zip(L.adj_acc_total(acc_a), L.adj_acc_total(acc_b)):
        assert abs(a - b) <= 1e-6 * abs(a) + 1e-12, (a, b)
