"""Launches that keep states on their way (GPU): lbmhd_step_store and
lbmhd_step_store_pairs, tile by tile in automatic mode, against single steps
(lbmhd_step_between on a handle with steps_per_pass = 1) bit for bit.

Sizes: both tile regions, lattices smaller than a region, ragged tiles, and
lattices beyond the lines where rows take over; counts below, at and beyond one
launch.  The rows between two kept states (a stride larger than a lattice)
and the states behind the last one stay as they were.
"""
import pytest
import torch

from lbmhd_inputs import random_fields

pytestmark = pytest.mark.gpu

SIZES = [(2, 2), (3, 5), (40, 64), (200, 200), (201, 200), (97, 501), (1030, 900), (1300, 1200)]


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("les", [0, 1, 2, 3, 4, 6])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_kept_states_equal_single_steps(nx, ny, les, storage):
    from paper_1607_08675_amd.lattice import Lattice, LBMHDConfig
    print(f"\nkept states les={les} {storage} {nx}x{ny}", flush=True)
    kw = dict(nx=nx, ny=ny, nu=2e-3, eta=3e-3, les=les, storage=storage,
              cs=0.05 if les == 4 else 0.1)
    one, auto = (Lattice(LBMHDConfig(**kw, steps_per_pass=k)) for k in (1, 0))
    one.init_fields(*random_fields(nx, ny, seed=nx + ny, rho_amp=0.004, u_amp=0.02, b_amp=0.02))
    x0 = one.save_state()
    n = 9
    ref = [x0]
    for _ in range(n):
        ref.append(one.new_state_buffer().zero_())
        one.step_between(ref[-2], ref[-1])
    size = one.lattice_bytes
    for pairs in (False, True):
        if pairs and les >= 2:
            continue
        for count in ((1, 2, 4) if pairs else (1, 2, 3, 7, 9)):
            store = torch.full((count + 1, size + 512), 7, dtype=torch.uint8, device="cuda")
            (auto.step_store_pairs if pairs else auto.step_store)(x0, store[:count], count)
            for k in range(count):
                want = ref[2 * k + 2 if pairs else k + 1]
                got = store[k, :size].clone()
                assert torch.equal(auto.state_view(got), auto.state_view(want)), (pairs, count, k)
            assert bool((store[:count, size:] == 7).all()) and bool((store[count] == 7).all())
