"""Reverse steps by tiles (GPU), at the lattices where the kernel changes.

Pairs (les = 0, 1): 12 x 12 and 28 x 12 tiles on small and middling lattices,
rows where the tiles would outnumber the accumulator's slots (low, wide
lattices) and on large ones.  Each pair equals two single reverse steps bit for
bit.  Kinetic closure (les = 2, 3): 28 x 8 and 60 x 8 tiles where the strips
are 8 rows high, rows elsewhere.  A lattice repeated along y takes the other
kernel, and its reverse step is the first one's repeated: the same operations
on the same values at every site, so bit for bit; the derivatives, summed over
each column in FP32, keep the same 8-row strips only where both are tiled, and
are compared there (FP64 sums of the strips, 1e-12 relative to the sum of n
such terms of one sign or the other: 1e-10 of the value).
"""
import numpy as np
import pytest
import torch

from lbmhd_inputs import random_planes

pytestmark = pytest.mark.gpu

W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
W19 = np.concatenate([W9, np.zeros(10)])


@pytest.fixture(scope="module")
def lb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1607_08675_amd import lattice
    return lattice


def make(lb, nx, ny, les, storage):
    return lb.Lattice(lb.LBMHDConfig(nx=nx, ny=ny, nu=0.01, eta=0.02, les=les, cs=0.12,
                                     cs_b=0.07, delta=1.3, storage=storage))


def planes(nx, ny, seed):
    scale = np.concatenate([W9 * 0.02, np.full(10, 0.01)])
    return random_planes(19, nx, ny, seed, W19, scale)


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("les", [0, 1])
@pytest.mark.parametrize("nx,ny", [(12, 12), (64, 64), (61, 50), (200, 200), (29, 13),
                                   (1030, 3), (1000, 701), (2050, 1710)])
def test_pair_equals_two_single_steps(lb, nx, ny, les, storage):
    print(f"\nadj pair tiles les={les} {storage} {nx}x{ny}", flush=True)
    L = make(lb, nx, ny, les, storage)
    L.set_populations(planes(nx, ny, nx + ny + les))
    x0, x1 = L.save_state(), L.new_state_buffer().zero_()
    L.step_between(x0, x1)
    g = torch.Generator(device="cuda").manual_seed(nx * ny)
    lam = L.new_adj_buffer()
    lam.copy_(torch.randn(lam.shape, generator=g, device="cuda", dtype=torch.float32))
    mid, one, acc1 = L.new_adj_buffer(), L.new_adj_buffer(), L.new_adj_acc()
    L.adj_step(x1, lam, mid, acc1)
    L.adj_step(x0, mid, one, acc1)
    two, acc2 = L.new_adj_buffer(), L.new_adj_acc()
    L.adj_step2(x0, lam, two, acc2)
    assert torch.equal(L.adj_view(one), L.adj_view(two))
    for a, b in zip(L.adj_acc_total(acc2), L.adj_acc_total(acc1)):
        assert abs(a - b) <= 1e-10 * abs(b), (a, b)


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("les", [2, 3])
@pytest.mark.parametrize("nx,ny,times", [(64, 64, 65), (61, 16, 3), (28, 8, 1200), (300, 200, 21),
                                         (1000, 128, 9), (257, 3, 5), (3, 5, 1000)])
def test_kinetic_step_of_a_repeated_lattice(lb, nx, ny, times, les, storage):
    print(f"\nadj kin tiles les={les} {storage} {nx}x{ny} x{times}", flush=True)
    p = planes(nx, ny, 3 * nx + ny + les)
    g = torch.Generator().manual_seed(nx * ny)
    lam0 = torch.randn(19, ny, nx, generator=g)
    out, tot, rows = [], [], []
    for k in (1, times):
        L = make(lb, nx, k * ny, les, storage)
        L.set_populations(np.tile(p, (1, k, 1)))
        lam, prev, acc = L.new_adj_buffer(), L.new_adj_buffer(), L.new_adj_acc()
        L.adj_view(lam).copy_(lam0.repeat(1, k, 1))
        L.adj_step(L.save_state(), lam, prev, acc)
        out.append(L.adj_view(prev).clone())
        tot.append(L.adj_acc_total(acc))
        rows.append(-(-nx // 256) * k * ny <= 4096)
    assert torch.equal(out[0].repeat(1, times, 1), out[1])
    if all(rows) and ny % 8 == 0:
        for a, b in zip(*tot):
            assert abs(times * a - b) <= 1e-10 * abs(b), (a, b)


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("nsteps", [2, 3, 4, 5, 6, 7])
def test_kept_states_and_segments_give_one_gradient(lb, nsteps, storage):
    """All even states kept (an odd and an even number of reverse launches, a
    last single step or none) against segments of two steps: the same steps and
    reverse steps in the same order, so energy and field gradients bit for bit."""
    from lbmhd_inputs import perturbed_orszag_tang
    from paper_1607_08675_amd.adjoint import Checkpointed
    fields = perturbed_orszag_tang(36, 28, u0=0.08, b0=0.08)
    out = []
    for every in (1, 2):
        L = make(lb, 36, 28, 1, storage)
        run = Checkpointed(L, every)
        J = run.forward(fields, nsteps)
        assert L.step_count == nsteps
        out.append((J, L.populations(), run.backward()))
    (J0, p0, g0), (J1, p1, g1) = out
    assert J0 == J1 and torch.equal(p0, p1)
    for a, b in zip(g0[:4], g1[:4]):
        assert torch.equal(a, b)
    for a, b in zip(g0[4:], g1[4:]):
        assert abs(a - b) <= 1e-10 * abs(b)
