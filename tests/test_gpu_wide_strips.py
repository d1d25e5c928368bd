"""Row-walking kernels on lattices of 257 to 341 tiles of columns (GPU), whose rows go in four
strips where one would leave a third of the card idle: equal to single steps bit for bit.
Strips of 9, of 9 with a last one of 6, and of the least height with a last one of 4 rows."""
import pytest
import torch

from test_gpu_strip_split import lattice
from state_words import stored_words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,spp", [(dict(les=1), 3), (dict(les=0), 2), (dict(les=2), 2),
                                    (dict(les=2, storage="fp16"), 2)])
@pytest.mark.parametrize("nx,ny", [(66000, 36), (87000, 33), (65537, 20)])
def test_four_strips_equal_single_steps(nx, ny, kw, spp):
    one, many = lattice(nx, ny, 1, **kw), lattice(nx, ny, spp, **kw)
    one.step(6)
    many.step(6)
    assert torch.equal(stored_words(one), stored_words(many))
