"""Every tile shape of the bf16 GEMM, with ragged last tiles in both
directions, one K step up to more than a ring holds, one and several tiles per
workgroup, all epilogues: against float64 (the oracle, or the same on the GPU)
on sampled rows (the edges of every 32-row block pair near tile ends), and bit
for bit against the two shapes that can be forced.  test_each_tile_shape asserts
which shape a case takes; test_linear_tile_shapes does not."""
import numpy as np
import pytest
import torch

import synth
from oracle import dit_block as O
from gpu_util import require_gpu, dev, host, empty, check, log

pytestmark = pytest.mark.gpu

# M, N, K on 256 compute units (the shape that the choice takes there)
CASES = [
    (1, 8, 64),              # 128 x 128, one row and one block of columns
    (130, 264, 64),          # 128 x 128, a second tile row of 2 rows, one K step
    (1000, 3072 + 72, 320),  # 128 x 128, five K steps: one more than the ring of X
    (1400, 3080, 192),       # 128 x 192
    (2650, 3080, 448),       # 256 x 192, seven K steps
    (4090, 3072, 128),       # 256 x 192
    (4090, 4096, 192),       # 256 x 256
    (9300, 3080, 64),        # many tiles of one K step each: the load cursor runs over tiles
]


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K", CASES)
def test_linear_tile_shapes(M, N, K, epi):
    B = require_gpu()
    log(f"case tile shapes M={M} N={N} K={K} epi={epi}")
    lengths = [M // 3, 0, M - M // 3]
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    a = synth.draw((M, K), (60, M, N, K), "bf16")
    w = synth.draw((N, K), (61, M, N, K), "bf16", std=0.05)
    b = synth.draw((N,), (62, M, N, K), "bf16", std=0.05)
    res = synth.draw((M, N), (63, M, N, K), "bf16")
    gate = synth.draw((3, N), (64, M, N, K), "f32", std=0.7)
    at, wt, bt, rt, gt = dev(a), dev(w), dev(b), dev(res), dev(gate)

    def run(tile_n):
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.debug_gemm_tile_n(tile_n)
        try:
            B.linear(at, wt, bt, out, epi=epi, res=rt if epi >= 2 else None, gate=gt if epi == 3 else None,
                     gate_stride=N, cu_seqlens=cu if epi == 3 else None)
            torch.cuda.synchronize()
        finally:
            B.debug_gemm_tile_n(0)
        return out

    out = run(0)
    for tile_n in (256, 192):
        assert torch.equal(out, run(tile_n)), f"differs from {tile_n}-wide tiles"
    rows = np.unique(np.clip(np.concatenate([np.arange(0, M, 128), np.arange(127, M, 128), np.arange(31, M, 512),
                                             [cu[1] - 1, cu[1], M - 1]]), 0, M - 1))
    z = O.linear(O.decode(a[rows]), O.decode(w), O.decode(b))
    req = np.searchsorted(cu[1:], rows, side="right")
    if epi == 1:
        z = O.gelu_tanh(z)
    elif epi == 2:
        z = O.decode(res[rows]) + z
    elif epi == 3:
        z = O.decode(res[rows]) + gate[req].astype(np.float64) * z
    check(host(out)[rows], z, "bf16", f"linear epi={epi}")


# tile: (M, N) of at most one tile per workgroup on 256 compute units, and of several
SHAPES = {
    (128, 128): [(130, 264), (4689, 1544)],
    (128, 192): [(906, 4104), (1876, 6152)],
    (128, 256): [(5465, 1000), (4883, 3080)],
    (256, 192): [(5077, 1544), (5853, 3080)],
    (256, 256): [(3331, 3592), (5950, 4104)],
}


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("K", [64, 448])   # fewer steps than any ring holds, and more
@pytest.mark.parametrize("tile,M,N", [(t, *mn) for t, sizes in SHAPES.items() for mn in sizes])
def test_each_tile_shape(tile, M, N, K, epi):
    B = require_gpu()
    log(f"case tile {tile[0]} x {tile[1]} M={M} N={N} K={K} epi={epi}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus != 256:
        pytest.skip(f"the sizes are for 256 compute units, not {cus}")
    assert B.debug_gemm_plan(M, N, K, cus) == tile
    assert (-(-M // tile[0]) * -(-N // tile[1]) > cus) == ((M, N) == SHAPES[tile][1])
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)

    def rn(*shape, std=1.0, dtype=torch.bfloat16):
        return torch.empty(shape, device="cuda").normal_(0, std, generator=g).to(dtype)

    a, w, b, res = rn(M, K), rn(N, K, std=0.05), rn(N, std=0.05), rn(M, N)
    gate = rn(3, N, std=0.7, dtype=torch.float32)
    cu = np.array([0, M // 3, M // 3, M], dtype=np.int32)

    def run(tile_n):
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.debug_gemm_tile_n(tile_n)
        try:
            B.linear(a, w, b, out, epi=epi, res=res if epi >= 2 else None, gate=gate if epi == 3 else None,
                     gate_stride=N, cu_seqlens=cu if epi == 3 else None)
            torch.cuda.synchronize()
        finally:
            B.debug_gemm_tile_n(0)
        return out

    out = run(0)
    for tile_n in (256, 192):
        assert torch.equal(out, run(tile_n)), f"differs from 256 x {tile_n} tiles"
    rows = np.unique(np.clip(np.concatenate([np.arange(0, M, 128), np.arange(127, M, 128), np.arange(31, M, 512),
                                             [cu[1] - 1, cu[1], M - 1]]), 0, M - 1))
    at = torch.from_numpy(rows).cuda()
    z = a[at].double() @ w.double().T + b.double()
    if epi == 1:
        z = 0.5 * z * (1 + torch.tanh(np.sqrt(2 / np.pi) * (z + 0.044715 * z ** 3)))
    elif epi == 2:
        z = res[at].double() + z
    elif epi == 3:
        z = res[at].double() + gate.double()[(at >= int(cu[1])).long() * 2] * z
    check(host(out[at]), z.cpu().numpy(), "bf16", f"tile {tile} epi={epi}")
