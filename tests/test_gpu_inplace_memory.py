"""In-place lattices without room for copies, and with one workspace for two handles (GPU)."""
import ctypes

import pytest
import torch

from lbmhd_inputs import random_fields
from state_words import stored_words

pytestmark = pytest.mark.gpu

KW = dict(nx=2048, ny=1500, nu=2e-3, eta=3e-3, les=1)


def lattice(seed, **kw):
    from paper_1607_08675_amd.lattice import Lattice, LBMHDConfig
    L = Lattice(LBMHDConfig(**KW, **kw))
    return L.init_fields(*random_fields(2048, 1500, seed=seed, rho_amp=0.004, u_amp=0.02,
                                        b_amp=0.02))


def test_steps_without_the_room_and_with_it_again():
    two, one = lattice(5, steps_per_pass=1), lattice(5, inplace=True)
    give = (ctypes.c_void_p(one._halos.data_ptr()), one._halos.numel())
    for room, n in (((None, 0), 5), (give, 4), ((None, 0), 2), (give, 7)):
        assert one._L.lbmhd_bind_halos(one._h, *room) == 0
        one.step(n)
        two.step(n)
    assert torch.equal(stored_words(two), stored_words(one))


def test_two_handles_share_one_workspace():
    from paper_1607_08675_amd._capi import check
    ref = [lattice(s, steps_per_pass=1) for s in (7, 8)]
    a, b = lattice(7, inplace=True), lattice(8, inplace=True)
    # b again with a's workspace and on a stream of its own
    other = torch.cuda.Stream()
    state = b.save_state()
    torch.cuda.synchronize()
    check(b._L.lbmhd_bind(b._h, b._a.data_ptr(), b.lattice_bytes, None, 0, a._ws.data_ptr(),
                          a._ws.numel(), other.cuda_stream), "lbmhd_bind", b._h)
    check(b._L.lbmhd_bind_halos(b._h, b._halos.data_ptr(), b._halos.numel()),
          "lbmhd_bind_halos", b._h)
    b.load_state(state, 0)
    for _ in range(6):
        a.step(3)
        b.step(3)
    torch.cuda.synchronize()
    for r, L in zip(ref, (a, b)):
        r.step(18)
        assert r.diag() == L.diag()
        torch.cuda.synchronize()
        got = stored_words(L)
        torch.cuda.synchronize()
        assert torch.equal(stored_words(r), got)


# strips of 28 rows, a last strip of one row, two strips of uneven heights; six rows, which the
# copies would outgrow
@pytest.mark.parametrize("nx,ny,rows", [(110000, 28, True), (15600, 193, True),
                                        (50000, 97, True), (500000, 6, False)])
def test_low_wide_lattices_in_place(nx, ny, rows):
    from paper_1607_08675_amd.lattice import Lattice, LBMHDConfig
    f = random_fields(nx, ny, seed=nx + ny, rho_amp=0.004, u_amp=0.02, b_amp=0.02)
    two = Lattice(LBMHDConfig(**{**KW, "nx": nx, "ny": ny}, steps_per_pass=1)).init_fields(*f)
    one = Lattice(LBMHDConfig(**{**KW, "nx": nx, "ny": ny}, inplace=True)).init_fields(*f)
    assert (one._halos is not None) == rows
    for n in (5, 4, 1, 3):
        two.step(n)
        one.step(n)
    assert torch.equal(stored_words(two), stored_words(one))


def test_a_lattice_steps_where_the_copies_find_no_memory(monkeypatch):
    from paper_1607_08675_amd import lattice as lb
    empty = torch.empty

    def full(*size, **kw):
        if size == (room,):
            raise torch.OutOfMemoryError("planted")
        return empty(*size, **kw)

    room = lattice(5, inplace=True)._halos.numel()
    monkeypatch.setattr(lb.torch, "empty", full)
    two, one = lattice(5, steps_per_pass=1), lattice(5, inplace=True)
    monkeypatch.undo()
    assert one._halos is None
    two.step(5)
    one.step(5)
    assert torch.equal(stored_words(two), stored_words(one))
    assert two.diag() == one.diag()
