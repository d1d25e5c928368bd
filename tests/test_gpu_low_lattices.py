"""Lattices on both sides of the rule that keeps low, wide ones off the tiles, and narrow ones
off the wide tiles (GPU): automatic steps and kept states equal single steps bit for bit."""
import pytest
import torch

from test_gpu_strip_split import lattice
from state_words import stored_words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("les", [1, 2, 4])
@pytest.mark.parametrize("nx,ny", [(25000, 4), (50000, 6), (16666, 6), (31250, 32), (60, 40000)])
def test_automatic_steps_equal_single_steps(nx, ny, les, storage):
    kw = dict(les=les, storage=storage, cs=0.05)
    one, auto = lattice(nx, ny, 1, **kw), lattice(nx, ny, 0, **kw)
    x0 = one.save_state()
    for n in (5, 2, 6):
        one.step(n)
        auto.step(n)
        assert torch.equal(stored_words(one), stored_words(auto)), n
    ref = [x0]
    for _ in range(8):
        ref.append(one.new_state_buffer())
        one.step_between(ref[-2], ref[-1])
    store = torch.empty(8, one.lattice_bytes, dtype=torch.uint8, device="cuda")
    auto.step_store(x0, store, 8)
    for k in range(8):
        assert torch.equal(stored_words(auto, store[k]), stored_words(one, ref[k + 1])), k
    if les == 1:
        auto.step_store_pairs(x0, store, 4)
        for k in range(4):
            assert torch.equal(stored_words(auto, store[k]), stored_words(one, ref[2 * k + 2])), k
