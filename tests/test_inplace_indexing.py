"""Index arithmetic of the in-place row-walking kernels, enumerated on the CPU.

A block of the in-place two- or three-step kernel reads its own tile and strip from the lattice
and everything around it from the copies that k_halo_save makes before the pass.  The model
follows the kernels' formulas for every block, pass, column and plane and checks that each read
lies in its buffer and gives the site x - c of the state before the pass, that a block never
reads a lattice element outside its own tile and strip, and that inside it a row is stored only
after the last pass that reads it.
"""
import pytest

PLANES = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]


def saved(nx, ny, D, strip_h, strips, tile_w, tiles):
    """What k_halo_save leaves: (boundary, k) -> row and (boundary, y, j) -> site."""
    rows = {(s, k): (s * strip_h - D + k) % ny for s in range(strips) for k in range(2 * D)}
    cols = {(t, y, j): ((t * tile_w - D + j) % nx, y)
            for t in range(tiles) for y in range(ny) for j in range(2 * D)}
    return rows, cols


@pytest.mark.parametrize("D", [2, 3])
@pytest.mark.parametrize("nx,ny,strip_h,tile_w", [
    (24, 32, 8, 8), (21, 37, 8, 8), (9, 33, 32, 8), (8, 16, 8, 8), (17, 9, 8, 16), (16, 41, 40, 8)])
def test_every_read_is_the_old_state(nx, ny, strip_h, tile_w, D):
    strips, tiles = -(-ny // strip_h), -(-nx // tile_w)
    rows, cols = saved(nx, ny, D, strip_h, strips, tile_w, tiles)
    halo = D - 1                      # halo rows and columns of the first update
    for strip in range(strips):
        for tile in range(tiles):
            x0, y0 = tile * tile_w, strip * strip_h
            wt, h = min(tile_w, nx - x0), min(strip_h, ny - y0)
            last_read, stored = {}, {}
            for t in range(h + 2 * halo):
                r = y0 - halo + t
                if r - halo >= y0:
                    stored[r - halo] = t
                for cx, cy in PLANES:
                    y = r - cy
                    k = y - y0
                    inside = 0 <= k < h
                    b = strip if k < 0 else (strip + 1) % strips
                    idx = D + k if k < 0 else D + k - h
                    if not inside:
                        assert 0 <= idx < 2 * D
                        assert rows[(b, idx)] == y % ny
                        continue          # whole rows: any column, wrapped
                    last_read[y] = t
                    for lc in range(-halo, wt + halo):
                        x = (x0 + lc) % nx
                        want = ((x - cx) % nx, y)
                        if 0 <= lc < wt:
                            if lc == 0 and cx == 1:
                                got = cols[(tile, y, D - 1)]
                            elif lc == wt - 1 and cx == -1:
                                got = cols[((tile + 1) % tiles, y, D)]
                            else:
                                assert x0 <= x - cx < x0 + wt   # its own tile
                                got = (x - cx, y)
                        else:
                            e = tile if lc < 0 else (tile + 1) % tiles
                            j = D + (lc if lc < 0 else lc - wt) - cx
                            assert 0 <= j < 2 * D
                            got = cols[(e, y, j)]
                        assert got == want
            assert sorted(stored) == list(range(y0, y0 + h))
            # two steps: a row is stored in the pass of its last read, after that
            # pass's barrier; three: one pass later
            assert all(stored[y] >= last_read[y] + (D - 2) for y in stored)
