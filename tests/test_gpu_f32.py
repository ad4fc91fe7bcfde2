"""The fp32 kernels at the edges of their tiles and at the line between the two
GEMM kernels, against float64; rows alone have the bits they have in a larger
call.  Bounds: a sum of K products of N(0, 1) and N(0, 0.05^2) values is off by
at most about sqrt(K) 2^-24 of its terms' size; 1e-5 is over ten times that."""
import numpy as np
import pytest
import torch

from gpu_util import require_gpu, log

pytestmark = pytest.mark.gpu


def _rand(*shape, seed, std=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.empty(shape, device="cuda").normal_(0, std, generator=g)


def _gelu(z):
    return 0.5 * z * (1 + torch.tanh(np.sqrt(2 / np.pi) * (z + 0.044715 * z ** 3)))


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K,pad", [
    (1, 4, 1, 3), (17, 20, 37, 3), (64, 384, 384, 0), (65, 68, 130, 2), (77, 768, 1536, 0), (15, 12, 64, 4),
    (400, 1060, 52, 0),      # 7 x 17 tiles of 64 x 64: near the end of the small kernel's side
    (449, 1020, 84, 0),      # 8 x 16: the large kernel's first shape
    (1000, 1004, 200, 0), (777, 2048, 21, 3),     # the large kernel
])
def test_linear_f32(M, N, K, pad, epi):
    B = require_gpu()
    log(f"case linear f32 M={M} N={N} K={K} epi={epi}")
    ld = K + pad
    a, w = _rand(M, ld, seed=1)[:, :K], _rand(N, ld, seed=2, std=0.05)[:, :K]
    b, res = _rand(N, seed=3), _rand(M, N, seed=4)
    gate = _rand(2, N, seed=5)
    cu = [0, M // 2, M]
    kw = dict(epi=epi, res=res if epi >= 2 else None, gate=gate if epi == 3 else None, gate_stride=N)

    def run(a, res, cu):
        out = torch.full((a.shape[0], N), float("nan"), device="cuda")
        B.linear(a, w, b, out, **dict(kw, res=res if epi >= 2 else None), cu_seqlens=cu if epi == 3 else None)
        torch.cuda.synchronize()
        return out

    out = run(a, res, cu)
    z = a.double() @ w.double().T + b.double()
    g = gate.double()[torch.arange(M, device="cuda").ge(cu[1]).long()]
    want = [z, _gelu(z), res.double() + z, res.double() + g * z][epi]
    assert (out.double() - want).abs().max().item() <= 1e-5 * max(1.0, want.abs().max().item())
    n = min(M, 33)   # the first rows alone
    assert torch.equal(run(a[:n], res[:n], [0, min(cu[1], n), n]), out[:n])


@pytest.mark.parametrize("H,d", [(3, 64), (2, 128)])
def test_attention_f32(H, d):
    B = require_gpu()
    log(f"case attention f32 H={H} d={d}")
    lq = [1, 15, 16, 17, 33, 5, 0, 40, 3]
    lk = [1, 16, 15, 63, 64, 65, 9, 130, 0]
    cu_q, cu_k = np.concatenate([[0], np.cumsum(lq)]), np.concatenate([[0], np.cumsum(lk)])
    W = H * d
    q, kv = _rand(int(cu_q[-1]), W, seed=6), _rand(int(cu_k[-1]), 2 * W, seed=7)
    k, v = kv[:, :W], kv[:, W:]

    def run(q, k, v, cu_q, cu_k):
        out = torch.full((q.shape[0], W), 7.0, device="cuda")
        B.attention_varlen(q, k, v, out, cu_q, cu_k, H, d)
        torch.cuda.synchronize()
        return out

    out = run(q, k, v, cu_q, cu_k)
    for r in range(len(lq)):
        a, b, e, f = int(cu_q[r]), int(cu_q[r + 1]), int(cu_k[r]), int(cu_k[r + 1])
        if a == b:
            continue
        if e == f:
            assert (out[a:b] == 0).all()
            continue
        for h in range(H):
            c = slice(h * d, (h + 1) * d)
            p = torch.softmax(q[a:b, c].double() @ k[e:f, c].double().T / d ** 0.5, -1)
            assert (out[a:b, c].double() - p @ v[e:f, c].double()).abs().max().item() <= 5e-6
        assert torch.equal(run(q[a:b], k[e:f], v[e:f], [0, b - a], [0, f - e]), out[a:b])


def test_attention_f32_minus_infinity():
    """Keys whose score is -inf count nothing, also where a whole tile of 16 has no other."""
    B = require_gpu()
    log("case attention f32 -inf")
    d, n = 64, 100
    q, k, v = _rand(20, d, seed=8).abs(), _rand(n, d, seed=9), _rand(n, d, seed=10)
    dead = torch.zeros(n, dtype=torch.bool, device="cuda")
    dead[16:48] = True
    dead[70] = True
    k[dead, 0] = float("-inf")
    out = torch.empty(20, d, device="cuda")
    B.attention_varlen(q, k, v, out, [0, 20], [0, n], 1, d)
    torch.cuda.synchronize()
    p = torch.softmax(q.double() @ k[~dead].double().T / 8.0, -1)
    assert (out.double() - p @ v[~dead].double()).abs().max().item() <= 5e-6


@pytest.mark.parametrize("times", [1, 9])   # 7 and 63 requests (the search for a tile's request)
@pytest.mark.parametrize("H,d", [(5, 64), (3, 128)])
def test_attention_f32_few_keys(H, d, times):
    """Up to 16 keys per request (one wave per tile): against float64, and the
    bits of the same requests beside one of 17 keys (four waves)."""
    B = require_gpu()
    log(f"case attention f32 few keys H={H} d={d}")
    lq, lk = [1, 17, 3, 0, 16, 40, 2] * times, [1, 16, 0, 3, 15, 2, 9] * times
    W = H * d
    q, k, v = _rand(sum(lq) + 5, W, seed=13), _rand(sum(lk) + 17, W, seed=14), _rand(sum(lk) + 17, W, seed=15)

    def run(lq, lk):
        out = torch.full((sum(lq), W), 7.0, device="cuda")
        B.attention_varlen(q[:sum(lq)], k[:sum(lk)], v[:sum(lk)], out, [0] + list(np.cumsum(lq)),
                           [0] + list(np.cumsum(lk)), H, d)
        torch.cuda.synchronize()
        return out

    out = run(lq, lk)
    assert torch.equal(out.view(torch.int32), run(lq + [5], lk + [17])[:sum(lq)].view(torch.int32))
    a = e = 0
    for nq, nk in zip(lq, lk):
        for h in range(H):
            c = slice(h * d, (h + 1) * d)
            p = torch.softmax(q[a:a + nq, c].double() @ k[e:e + nk, c].double().T / d ** 0.5, -1)
            assert (out[a:a + nq, c].double() - p @ v[e:e + nk, c].double()).abs().le(5e-6).all()
        a, e = a + nq, e + nk


def test_attention_f32_work_items_beyond_one_grid_dimension():
    """2^24 + 64 workgroups of 256: 2^32 work-items and more do not fit one grid
    dimension.  With one key every output row is its value row, exactly."""
    B = require_gpu()
    H, d, n = 64, 64, (1 << 22) + 16
    log(f"case attention f32 {n} queries x {H} heads")
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GiB of GPU memory")
    q = torch.zeros(n, H * d, device="cuda")
    k, v = _rand(1, H * d, seed=11), _rand(1, H * d, seed=12)
    out = torch.full((n, H * d), 7.0, device="cuda")
    B.attention_varlen(q, k, v, out, [0, n], [0, 1], H, d)
    torch.cuda.synchronize()
    for part in out.split(1 << 18):
        assert torch.equal(part, v.expand(len(part), -1))
