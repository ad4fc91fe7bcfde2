"""The conditioning Linears at the edges of their dispatch: every rows-per-wave
and requests-per-pass form, widths with whole groups of inputs (512 bf16
values), a ragged last group, and none.  Against float64 (sums of up to 2,560
fp32 products, error a few times 2^-24; the bound is ten times what was seen),
and bit for bit against each request alone."""
import numpy as np
import pytest
import torch

from gpu_util import require_gpu, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,F", [
    (torch.bfloat16, 128, 64), (torch.bfloat16, 640, 576), (torch.bfloat16, 1536, 512), (torch.bfloat16, 4224, 1088),
    (torch.float32, 384, 20), (torch.float32, 512, 768)])
@pytest.mark.parametrize("n_req", [1, 2, 3, 5, 8, 9, 64])
def test_modulation_forms(dtype, D, F, n_req):
    B = require_gpu()
    log(f"case modulation {dtype} D={D} F={F} n_req={n_req}")
    g = torch.Generator(device="cuda")
    g.manual_seed(D + n_req)

    def rn(*shape, std):
        return torch.empty(shape, device="cuda").normal_(0, std, generator=g).to(dtype)

    w = dict(w_t1=rn(D, F, std=0.05), b_t1=rn(D, std=0.02), w_t2=rn(D, D, std=0.05), b_t2=rn(D, std=0.02),
             w_ada=rn(6 * D, D, std=0.05), b_ada=rn(6 * D, std=0.02))
    cfg = B.BlockConfig(D, D // 128, 128, 4 * D, F, (0, 64, 64), dtype)
    cw = B.make_weights(w)
    t = torch.empty(n_req, device="cuda").uniform_(0, 1000, generator=g)
    ws = torch.empty(4 * (F + 2 * D) * n_req + 1024, dtype=torch.uint8, device="cuda")

    def run(t):
        mod = torch.full((len(t), 6, D), float("nan"), device="cuda")
        B.timestep_modulation(cfg, cw, t, mod, ws)
        torch.cuda.synchronize()
        return mod

    mod = run(t)
    d = {k: v.double() for k, v in w.items()}
    f = torch.exp(-np.log(10000.0) * torch.arange(F // 2, device="cuda", dtype=torch.float64) / (F // 2))
    a = t.double()[:, None] * f
    e = torch.cat([torch.cos(a), torch.sin(a)], 1)
    silu = torch.nn.functional.silu
    want = silu(silu(e @ d["w_t1"].T + d["b_t1"]) @ d["w_t2"].T + d["b_t2"]) @ d["w_ada"].T + d["b_ada"]
    err = (mod.double().view(n_req, -1) - want).norm() / want.norm()
    assert err.item() <= 4e-6
    for r in {0, n_req // 2, n_req - 1}:
        assert torch.equal(run(t[r:r + 1].clone()), mod[r:r + 1])


@pytest.mark.parametrize("dtype,D,F,n_req", [
    # one row per wave: rows of 1 to 16 vectors a lane, whole and ragged, and one too long for it (a request
    # alone, which every case compares with, takes it at these widths)
    (torch.bfloat16, 512, 4096, 1), (torch.bfloat16, 1920, 8192, 1), (torch.bfloat16, 256, 16384, 1),
    (torch.float32, 2048, 2048, 2), (torch.float32, 1920, 4100, 3), (torch.float32, 384, 384, 3),
    # 2 rows per wave, and a last group of 1, 2 and 4 requests after a full one
    (torch.bfloat16, 1920, 640, 12), (torch.bfloat16, 1536, 1536, 10), (torch.bfloat16, 2048, 2048, 9),
    (torch.float32, 1024, 1028, 9), (torch.float32, 768, 256, 12), (torch.float32, 2048, 4, 13),
    # 4 rows per wave with and without such a group; 8 rows from 28,672 outputs on
    (torch.float32, 1920, 2044, 9), (torch.bfloat16, 4736, 128, 6), (torch.bfloat16, 4864, 128, 6)])
def test_modulation_rows_and_last_groups(dtype, D, F, n_req):
    test_modulation_forms(dtype, D, F, n_req)
