"""The bf16 GEMM issues its MFMAs as inline assembly on the accumulation
registers, which the compiler does not see as MFMAs.  This test compiles the
kernel for gfx950 with the library's own flags and checks every instance: no
instruction but the next MFMA touches an accumulator within the wait states
after an MFMA that writes it, no MFMA reads a register that a vector
instruction wrote in the 2 wait states before it, and the K loop neither
copies accumulators nor waits for all loads in flight."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_13501_amd import build as B
from test_attention_asm import _blocks, scan

SHAPES = ["ILi8ELi8ELi2E", "ILi8ELi6ELi2E", "ILi4ELi8ELi2E", "ILi4ELi6ELi3E", "ILi4ELi4ELi4E"]


def _flat(line):
    """Accumulation register n as vector register 1000 + n."""
    line = re.sub(r"\ba\[(\d+):(\d+)\]", lambda m: f"v[{1000 + int(m.group(1))}:{1000 + int(m.group(2))}]", line)
    return re.sub(r"\ba(\d+)\b", lambda m: f"v{1000 + int(m.group(1))}", line)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(B.HIPCC) and shutil.which(B.HIPCC) is None:
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("asm") / "gemm.s"
    flags = [f for f in B.FLAGS if f != "-fPIC"] + B.EXTRA.get("gemm.hip", [])
    cmd = [B.HIPCC] + flags + ["-x", "hip", "--cuda-device-only", "-S", os.path.join(B.CSRC, "gemm.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = out.read_text().split("\n")
    found = {}
    for h in [i for i, l in enumerate(lines) if re.match(r"^_Z\S*gemm_bf16_nt\S*:", l)]:
        end = next(i for i in range(h, len(lines)) if lines[i].startswith(".Lfunc_end"))
        found[lines[h].split(":")[0]] = lines[h:end]
    return found


def test_every_shape_and_epilogue_is_compiled(kernels):
    for shape in SHAPES:
        assert sum(shape in name for name in kernels) == 4, shape


def test_accumulators_keep_their_distance(kernels):
    for name, body in kernels.items():
        problems = scan([_flat(l) for l in body])
        assert not problems, f"{name}:\n" + "\n".join(f"line {i}: {m}" for i, m in problems[:10])


def test_k_loop_has_no_copies_and_no_full_waits(kernels):
    for name, body in kernels.items():
        loops = [b for b in _blocks(body) if sum("v_mfma" in l for _, l, _ in b["ins"]) >= 32]
        assert len(loops) == 1, name
        ins = [l for _, l, _ in loops[0]["ins"]]
        assert not [l for l in ins if l.startswith(("v_accvgpr", "scratch_", "v_readlane", "v_writelane"))], name
        waits = [int(m.group(1)) for l in ins for m in re.finditer(r"vmcnt\((\d+)\)", l)]
        assert len(waits) == 1 and waits[0] >= 6, f"{name}: vmcnt waits {waits}"
