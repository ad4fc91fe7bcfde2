"""Every tile shape of the bf16 GEMM where the per-shape choice takes it, with
ragged last tiles in both directions, one K step up to more than a ring holds,
one and several tiles per workgroup: against the oracle on sampled rows (the
edges of every 32-row block pair near tile ends), and bit for bit against the
two shapes that can be forced."""
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
    (2650, 3080, 448),       # 128 x 256
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
