"""The paired reverse step by strips of rows (GPU) equals two single reverse steps.

The sizes are ones that go by rows: strips past the lattice (63 of 64, 125 of 128, 47 of 48),
whole strips, plain block order (one and two strips), four strips of wide lattices, and with
FP16 storage large lattices and a low one.  lambda bit for bit.  The closure-constant
derivatives add the same FP32 contributions in FP64 in another order: n terms of random sign
sum to about sqrt(n) of them, partial sums of at most 1e5 terms round to 1e5 eps of that, so
1e-10 of the sum, as for the tiles, leaves two digits for a sum that happens to be small; a
strip lost or counted twice moves it by more than 1e-3.
"""
import pytest
import torch

from test_gpu_adjoint_tiles import make, planes
from test_dispatch_rules import rules  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

CASES = [(2000, 1500, "fp32"), (1000, 3000, "fp32"), (2500, 1880, "fp32"), (4096, 512, "fp32"),
         (50000, 80, "fp32"), (70000, 60, "fp32"), (107142, 28, "fp32"), (1030, 3, "fp32"),
         (2048, 3969, "fp16"), (5000, 1650, "fp16"), (107142, 28, "fp16"), (1030, 3, "fp16")]


@pytest.mark.parametrize("les,cs", [(0, 0.12), (1, 0.12), (1, 0.0)])
@pytest.mark.parametrize("nx,ny,storage", CASES)
def test_pair_by_rows_equals_two_single_steps(rules, nx, ny, storage, les, cs):  # noqa: F811
    from paper_1607_08675_amd import lattice as lb
    assert not rules.rule_adj_tile(nx, ny, storage == "fp16")
    print(f"\nadj pair rows les={les} cs={cs} {storage} {nx}x{ny}", flush=True)
    L = make(lb, nx, ny, les, storage)
    if cs == 0.0:
        L = lb.Lattice(lb.LBMHDConfig(**{**L.cfg.__dict__, "cs": 0.0, "cs_b": 0.0}))
    L.set_populations(planes(nx, ny, nx + ny + les))
    x0, x1 = L.save_state(), L.new_state_buffer()
    L.step_between(x0, x1)
    g = torch.Generator(device="cuda").manual_seed(nx * ny)
    lam = torch.randn(L.adj_lattice_bytes // 4, generator=g, device="cuda", dtype=torch.float32)
    mid, one, acc1 = L.new_adj_buffer(), L.new_adj_buffer(), L.new_adj_acc()
    L.adj_step(x1, lam, mid, acc1)
    L.adj_step(x0, mid, one, acc1)
    two, acc2 = mid, L.new_adj_acc()
    L.adj_step2(x0, lam, two, acc2)
    assert torch.equal(L.adj_view(one), L.adj_view(two))
    for a, b in zip(L.adj_acc_total(acc2), L.adj_acc_total(acc1)):
        assert abs(a - b) <= 1e-10 * abs(b), (a, b)
        assert (b != 0.0) == (les == 1)
