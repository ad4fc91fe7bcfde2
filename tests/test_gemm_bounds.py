"""Host-side model of the bf16 GEMM's operand loads and LDS layout
(csrc/gemm.hip), for every tile shape: each byte a load touches lies inside the
operand, for ragged and exact tiles; LDS accesses stay in their slots; a ring
slot is refilled only when it is free.

The kernel forms each 16-byte load from a buffer descriptor (base = first
row of the tile, range = bytes up to the end of the operand's last row), a
lane offset (the row inside the tile, 8 q + i / 8 for piece q and lane i,
and a swizzled 16-byte chunk) and a scalar offset (the K step).  The
hardware zero-fills a load whose lane offset is past the range and does not
range-check the scalar offset, so the rows past a ragged tile's end must be
caught by the lane offset and the K step must stay inside a row.  This model
recomputes those offsets the same way for every tile row, wave, piece, lane
and K step (0 .. K / 64 - 1; past the last tile the descriptors are empty)."""
import os
import re

import numpy as np
import pytest

BK, WAVES = 64, 4

# The tile shapes of the bf16 GEMM: 16 x 16 blocks per wave (rows, columns),
# ring slots of the X operand (the other has one more), X is A
SHAPES = [(8, 8, 2, False), (8, 6, 2, False), (4, 8, 2, True), (4, 6, 3, False), (4, 4, 4, False)]


def test_shapes_are_those_of_the_kernel():
    src = open(os.path.join(os.path.dirname(__file__), "..", "paper_2606_13501_amd", "csrc", "gemm.hip")).read()
    found = re.findall(r"typedef Shape<(\d+), (\d+), (\d+), (true|false)> Tile", src)
    assert [(int(a), int(b), int(c), d == "true") for a, b, c, d in found] == SHAPES


def shape_loads(M, K, ld, blocks, row_in_lane=True):
    """(lowest, highest) byte touched by an operand's loads over all tiles of
    32 * blocks rows, and the rows of the first tile each lane fills, as
    {(LDS row, physical chunk): (row, chunk)}.  row_in_lane=False: with the
    piece's row in the scalar offset, outside the range check."""
    rows, kt = 32 * blocks, K // BK
    lane = np.arange(64)
    lo, hi, home = np.inf, -np.inf, {}
    for t in range((M + rows - 1) // rows):
        m0 = t * rows
        n_rec = ((M - m0 - 1) * ld + K) * 2
        for wave in range(WAVES):
            for u in range(blocks):
                c = (lane & 7) ^ (4 * (u & 1) + (lane >> 4))
                piece = (blocks * wave * 8 + 8 * u) * ld * 2
                vo = (lane >> 3) * ld * 2 + c * 16 + piece
                if t == 0:
                    lds = (blocks * wave + u) * 1024 + 16 * lane
                    for v, a, ch in zip(vo, lds, c):
                        home[(int(a) // 128, int(a) % 128 // 16)] = (int(v) // (ld * 2), int(ch))
                live = (vo if row_in_lane else vo - piece) < n_rec   # otherwise zero-filled, nothing read
                if live.any():
                    lo = min(lo, m0 * ld * 2 + vo[live].min())
                    hi = max(hi, m0 * ld * 2 + vo[live].max() + (kt - 1) * BK * 2 + 15)
    return lo, hi, home


@pytest.mark.parametrize("blocks", [8, 6, 4])
@pytest.mark.parametrize("M,K,ld", [
    (1, 64, 64), (300, 192, 200), (257, 128, 128), (512, 64, 72),
    (5, 128, 136), (8, 128, 128),            # fewer rows than one load piece, or one piece
    (64, 5120, 5120),                        # the step's output projection weight
    (3072, 3072, 3072), (2880, 768, 768),    # image block weights; a ragged one
    (75600, 13824, 13824),                   # 720p activations of the MLP down projection
])
def test_tile_shape_loads_stay_inside_and_fill_the_tile(M, K, ld, blocks):
    lo, hi, home = shape_loads(M, K, ld, blocks)
    assert lo >= 0 and hi <= ((M - 1) * ld + K) * 2 - 1
    rows = 32 * blocks
    assert len(home) == rows * 8      # every chunk of the slot is filled, each from its own row
    for (row, phys), (src, chunk) in home.items():
        assert src == row and phys == chunk ^ ((row >> 1) & 7)


@pytest.mark.parametrize("blocks", [8, 6, 4])
def test_scalar_piece_offset_would_leave_the_operand(blocks):
    """What the lane offset prevents at the ragged last tile."""
    M, K, ld = 75600, 5120, 5120
    assert shape_loads(M, K, ld, blocks, row_in_lane=False)[1] > ((M - 1) * ld + K) * 2 - 1


@pytest.mark.parametrize("mb,nb,r,xa", SHAPES)
def test_tile_shape_lds_regions(mb, nb, r, xa):
    """Fragment reads stay in their operand's slot, and the epilogue window of a
    wave in the wave's own part of a Y slot, with every chunk at its own place."""
    slot_a, slot_w = 32 * mb * 128, 32 * nb * 128
    ra, rw = (r, r + 1) if xa else (r + 1, r)
    assert ra * slot_a + rw * slot_w <= 160 * 1024
    lane = np.arange(64)
    fr, fh = lane & 15, lane >> 4
    for b, slot in ((mb, slot_a), (nb, slot_w)):
        seen = set()
        for half_wave in range(2):
            for kk in range(2):
                for j in range(b):
                    row = half_wave * 16 * b + 16 * j + fr
                    off = row * 128 + (((4 * kk + fh) ^ ((fr >> 1) & 7)) << 4)
                    assert off.max() + 15 < slot
                    # physical chunk = logical chunk ^ swizzle of the row in the tile
                    assert (((off >> 4) & 7) == ((4 * kk + fh) ^ ((row >> 1) & 7))).all()
                    seen.update(off.tolist())
        assert len(seen) == slot // 16
    ly = nb if xa else mb
    cw = 64 if nb % 4 == 0 and ly >= 8 else 32
    places = set()
    for row in range(32):
        for c in range(cw // 4):
            if cw == 64:
                places.add(row * 256 + ((((c >> 1) | ((c & 1) << 3)) ^ (((row & 1) << 3) | ((row >> 1) & 7))) << 4))
            else:
                places.add(row * 128 + ((((c >> 1) | ((c & 1) << 2)) ^ ((((row >> 1) & 1) << 2) | ((row >> 2) & 3))) << 4))
    assert len(places) == 32 * cw // 4 and max(places) + 16 <= ly * 1024


@pytest.mark.parametrize("mb,nb,r,xa", SHAPES)
@pytest.mark.parametrize("kt", [1, 2, 3, 7])
def test_ring_slots_are_free_and_landed(mb, nb, r, xa, kt):
    """A replay of the loads over three tiles of kt steps: a slot is refilled
    only after the barrier that ends its step, never while it serves as the
    epilogue window, and the loads a barrier waits for (all but the newest
    (R - 2) LX + (R - 1) LY) include the next step's."""
    lx, ly = (mb, nb) if xa else (nb, mb)
    ry, steps = r + 1, 3 * kt
    x, y, issued = {}, {}, []           # slot -> step; loads in issue order
    done_x, done_y = set(), set()       # steps whose slot may be overwritten

    def issue(what, step):
        ring, slots, done, n = (x, r, done_x, lx) if what == "x" else (y, ry, done_y, ly)
        old = ring.get(step % slots)
        assert old is None or old in done, (what, step, old)
        ring[step % slots] = step
        issued.extend([(what, step)] * n)

    for s in range(r):
        issue("x", s)
        issue("y", s)
    for s in range(steps):
        assert x[s % r] == s and y[s % ry] == s
        if s > 0:
            done_y.add(s - 1)           # read before the last barrier; the window of a finished tile is drained
        issue("y", s + r)
        pending = (r - 2) * lx + (r - 1) * ly
        landed = issued[:len(issued) - pending] if pending else issued
        for what, n in (("x", lx), ("y", ly)):
            assert landed.count((what, s + 1)) == n, (what, s)
        done_x.add(s)
        issue("x", s + r)
        if (s + 1) % kt == 0:           # the epilogue's window: Y's slot of step s
            assert y[s % ry] == s
