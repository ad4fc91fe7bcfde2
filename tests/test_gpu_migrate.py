"""dit_migration_execute on the GPU: device buffers stand in for the ranks'
slices; applying a plan rebuilds every destination slice bit for bit as
direct slicing of the global tensor does (SP row layouts of the 720p token
matrix, box layouts of a channel-major latent, odd sizes that force narrow
copy units, a replicated field)."""
import numpy as np
import pytest
import torch

from gpu_util import log, require_gpu
from oracle import migrate as M

pytestmark = pytest.mark.gpu


def _run(kind, global_t, src, dst):
    B = require_gpu()
    shape = tuple(global_t.shape)
    eb = global_t.element_size()
    f = B.MigField(kind, shape, eb, src, dst)
    entries, n = B.migration_plan(f)
    sb = [global_t[tuple(slice(a, b) for a, b in zip(s, e))].contiguous().clone() for _, s, e in src]
    db = [torch.full([b - a for a, b in zip(s, e)], 7, dtype=global_t.dtype, device="cuda") for _, s, e in dst]
    B.migration_execute(f, entries, n, sb, db)
    torch.cuda.synchronize()
    for (r, s, e), got in zip(dst, db):
        want = global_t[tuple(slice(a, b) for a, b in zip(s, e))]
        assert torch.equal(got, want), (r, s, e)
    return n


@pytest.mark.parametrize("d1,d2", [(1, 8), (8, 2), (4, 3), (2, 4), (8, 8), (5, 7)])
def test_sp_token_layouts(d1, d2):
    log(f"case migrate tokens 75600x64 bf16 SP{d1} -> SP{d2}")
    g = torch.randn(75600, 64, device="cuda").to(torch.bfloat16)
    n = _run(M.SHARDED, g, M.row_layout(75600, list(range(d1)), [64]), M.row_layout(75600, list(range(8, 8 + d2)), [64]))
    log(f"  {n} entries")


def test_latent_boxes_fp32():
    log("case migrate latent 16x21x90x160 fp32, (f, h) boxes -> h bands")
    g = torch.randn(16, 21, 90, 160, device="cuda")
    src = [(3 * i + j, [0, fa, ha, 0], [16, fb, hb, 160]) for i, (fa, fb) in enumerate([(0, 7), (7, 21)])
           for j, (ha, hb) in enumerate([(0, 30), (30, 61), (61, 90)])]
    dst = [(10 + k, [0, 0, a, 0], [16, 21, b, 160]) for k, (a, b) in enumerate([(0, 23), (23, 45), (45, 68), (68, 90)])]
    _run(M.SHARDED, g, src, dst)


def test_odd_sizes_narrow_units():
    log("case migrate 7x13x5 bf16 and 3x3 int8-sized")
    g = torch.randn(7, 13, 5, device="cuda").to(torch.bfloat16)
    src = M.row_layout(7, [0, 1, 2], [13, 5])
    dst = [(5, [0, 3, 1], [7, 11, 4]), (6, [2, 0, 0], [5, 13, 5])]
    _run(M.SHARDED, g, src, dst)
    g8 = torch.randint(0, 255, (9, 3), device="cuda", dtype=torch.uint8)
    _run(M.SHARDED, g8, M.row_layout(9, [0, 1], [3]), M.row_layout(9, [2, 3, 4, 5], [3]))


def test_replicated():
    log("case migrate replicated 33x65 fp32 to 4 ranks")
    g = torch.randn(33, 65, device="cuda")
    whole = ([0, 0], [33, 65])
    _run(M.REPLICATED, g, [(0,) + whole, (1,) + whole], [(r,) + whole for r in (1, 2, 3, 4)])


def test_many_boxes_mixed_units_and_order():
    """Twenty boxes in one launch (4-, 8- and 16-byte units); then entries whose
    destinations meet, and a chain that reads what an earlier entry wrote:
    entries take effect in order."""
    log("case migrate 5 -> 16 shards of 67 x 37 x 4 (4- to 16-byte units)")
    for dtype in (torch.uint8, torch.bfloat16, torch.float32):
        g = torch.randn(67, 37, 4, device="cuda").mul(50).to(dtype)
        src = M.row_layout(67, list(range(5)), [37, 4])
        dst = [(k, [a, c, 0], [b, d, 4]) for k, ((a, b), (c, d)) in enumerate(
            ((x, x + 9 if x < 58 else 67), (y, y + 19 if y < 18 else 37)) for x in range(0, 67, 9) for y in (0, 19))]
        n = _run(M.SHARDED, g, src, [(k, s, [min(e[0], 67), min(e[1], 37), 4]) for k, s, e in dst])
        assert n > 16
    B = require_gpu()
    log("case migrate overlapping destinations and a chain")
    f = B.MigField(M.SHARDED, (8, 16), 4, [(0, [0, 0], [8, 16]), (1, [0, 0], [8, 16]), (2, [0, 0], [8, 16])],
                   [(3, [0, 0], [8, 16]), (4, [0, 0], [8, 16])])
    a, b = (torch.randn(8, 16, device="cuda") for _ in range(2))
    d0, d1 = (torch.zeros(8, 16, device="cuda") for _ in range(2))
    entries = (B.CMigEntry * 3)()

    def entry(e, src, dst, off, ext):
        e.src_index, e.dst_index = src, dst
        for d in range(2):
            e.src_off[d] = e.dst_off[d] = off[d]
            e.extent[d] = ext[d]
        e.bytes = 4 * ext[0] * ext[1]

    entry(entries[0], 0, 0, (0, 0), (8, 16))     # d0 = a
    entry(entries[1], 1, 0, (2, 4), (3, 8))      # part of d0 = b
    entry(entries[2], 2, 1, (0, 0), (8, 16))     # d1 = d0, which is source slice 2
    for _ in range(20):
        d0.zero_()
        d1.zero_()
        B.migration_execute(f, entries, 3, [a, b, d0], [d0, d1])
        torch.cuda.synchronize()
        want = a.clone()
        want[2:5, 4:12] = b[2:5, 4:12]
        assert torch.equal(d0, want) and torch.equal(d1, want)


def test_boxes_whose_workgroups_exceed_one_launch():
    """Nine boxes of just under 2 GiB in 1-byte units: together more work-items
    than a launch may have (2^32)."""
    B = require_gpu()
    log("case migrate 9 boxes of 2 GiB, 7-byte rows")
    n, rows = 9, (2**31 - 1) // 7
    free, _ = torch.cuda.mem_get_info()
    if free < 60 << 30:
        pytest.skip("needs 60 GiB of GPU memory")
    shape = (n * rows, 7)
    src = [(0, [0, 0], [n * rows, 7])]
    dst = [(1 + k, [k * rows, 0], [(k + 1) * rows, 7]) for k in range(n)]
    f = B.MigField(M.SHARDED, shape, 1, src, dst)
    entries, count = B.migration_plan(f)
    assert count == n
    g = torch.randint(0, 255, (n * rows * 7 // 8 + 1,), device="cuda", dtype=torch.int64)
    g = (g * 0x0101010101010101 + torch.arange(len(g), device="cuda") * 0x9E3779B97F4A7C1).view(torch.uint8)
    out = [torch.full((rows, 7), 7, dtype=torch.uint8, device="cuda") for _ in range(n)]
    B.migration_execute(f, entries, count, [g], out)
    torch.cuda.synchronize()
    for k in range(n):
        assert torch.equal(out[k].view(-1), g[k * rows * 7:(k + 1) * rows * 7]), k


def _bands(n, shape, axis):
    cut = [shape[axis] * k // n for k in range(n + 1)]
    return [(k, [a if d == axis else 0 for d in range(len(shape))], [b if d == axis else shape[d] for d in range(len(shape))])
            for k, (a, b) in enumerate(zip(cut, cut[1:]))]


@pytest.mark.parametrize("dtype,shape,src,dst,entries", [
    # 9 x 8 boxes: three launches; 1-, 2-, 4- and 16-byte units in one launch (rows of 52 to 112 bytes)
    (torch.uint8, (90, 640), (9, 0), [0, 112, 164, 222, 225, 230, 400, 528, 640], 72),
    (torch.bfloat16, (45, 9, 333), (7, 0), (11, 2), 77),
    # few units and many (about 2^20), in 8 boxes (searched one by one) and 9 or more (at once)
    (torch.float32, (1 << 15, 31), (1, 0), (8, 0), 8), (torch.float32, (1 << 15, 33), (1, 0), (8, 0), 8),
    (torch.float32, (1 << 15, 33), (1, 0), (9, 0), 9), (torch.uint8, (1100, 1001), (2, 0), (5, 1), 10),
    # 16-byte units: rows of 63, 64 and 65 units, following each other or not
    (torch.float32, (20000, 252), (1, 0), (1, 0), 1), (torch.float32, (20000, 256), (2, 0), (3, 0), 4),
    (torch.float32, (20000, 260), (8, 0), (7, 0), 14),
    (torch.float32, (20000, 504), (2, 0), (2, 1), 4), (torch.float32, (20000, 512), (1, 1), (2, 1), 2),
])
def test_launch_forms(dtype, shape, src, dst, entries):
    """Units per thread and the search for a workgroup's box, at their lines;
    plans of more boxes than two launches take."""
    log(f"case migrate {dtype} {shape} {src} -> {dst}")
    g = torch.randint(0, 255, shape, device="cuda", dtype=torch.int32).to(dtype)
    if isinstance(dst, list):
        to = [(k, [0, a], [shape[0], b]) for k, (a, b) in enumerate(zip(dst, dst[1:]))]
    else:
        to = _bands(dst[0], shape, dst[1])
    assert _run(M.SHARDED, g, _bands(src[0], shape, src[1]), to) == entries


def test_a_box_beyond_32_bit_indices_between_small_ones():
    """2^31 units and more in one box (1-byte units): a launch of its own, after
    the boxes before it."""
    log("case migrate 2 GiB box of 7-byte rows between two small ones")
    if torch.cuda.mem_get_info()[0] < 20 << 30:
        pytest.skip("needs 20 GiB of GPU memory")
    cut = [0, 100, 100 + 2**31 // 7 + 10, 2**31 // 7 + 213]
    g = torch.randint(0, 255, (cut[-1], 7), device="cuda", dtype=torch.uint8)
    dst = [(1 + k, [a, 0], [b, 7]) for k, (a, b) in enumerate(zip(cut, cut[1:]))]
    assert _run(M.SHARDED, g, [(0, [0, 0], [cut[-1], 7])], dst) == 3
