"""The few-rows GEMM is bound by its loads, so its loop must not wait for more than the chunk it is about to multiply: in the
compiled loop the strictest wait leaves one whole chunk in flight. CPU only: compiled to assembly, nothing runs."""
import os
import re
import shutil

import pytest

from paper_2406_00023_amd import build


def matrix_loops(asm: str, kernel: str):
    """[(mfma, loads, smallest vmcnt)] of the innermost loops with matrix instructions in the kernels of that name."""
    found = []
    for body in re.findall(r"^_Z\S*%s\S*:(.*?)^\.Lfunc_end" % kernel, asm, flags=re.S | re.M):
        lines = body.split("\n")
        label = {m.group(1): n for n, l in enumerate(lines) if (m := re.match(r"(\.LBB\w+):", l))}
        for n, line in enumerate(lines):
            m = re.search(r"s_cbranch_\w+ (\.LBB\w+)", line)
            if not m or label.get(m.group(1), n) >= n:
                continue
            loop = lines[label[m.group(1)]:n]
            if any("_cbranch" in l for l in loop) or not any("v_mfma" in l for l in loop):
                continue
            waits = [int(w) for l in loop for w in re.findall(r"vmcnt\((\d+)\)", l)]
            found.append((sum("v_mfma" in l for l in loop), sum("global_load" in l for l in loop), min(waits, default=0)))
    return found


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_loop_keeps_one_chunk_in_flight():
    loops = matrix_loops(build.device_assembly("ffn.hip"), "gemm_bf16_rows_kernel")
    assert {m for m, _, _ in loops} == {12, 24, 48}              # three chunks of four k-steps, one, two and four row blocks
    for mfma, loads, vmcnt in loops:
        blocks = mfma // 12
        assert loads == 3 * (4 + blocks)                         # weight pieces and copies of token rows
        assert vmcnt >= loads // 3, (mfma, loads, vmcnt)
