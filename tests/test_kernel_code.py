"""What the compiler makes of the GEMM's K loops (gfx950 assembly; no GPU)."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2606_18502_amd import build

pytestmark = pytest.mark.slow


def k_loops(asm):
    """(kernel, lines of its innermost loop that loads operands into LDS)."""
    lines = asm.split("\n")
    starts = [i for i, l in enumerate(lines) if re.match(r"_ZN\w*gemm_fp8_kernel\w*:", l)]
    for i, e in zip(starts, starts[1:] + [len(lines)]):
        body, labels, loop = lines[i:e], {}, None
        for n, l in enumerate(body):
            m = re.match(r"(\.LBB\w+):", l)
            if m:
                labels[m.group(1)] = n
            m = re.search(r"s_c?branch\w* (\.LBB\w+)", l)
            if m and m.group(1) in labels:
                part = body[labels[m.group(1)]:n + 1]
                if any("global_load_lds" in x for x in part) and (loop is None or len(part) < len(loop)):
                    loop = part
        yield body[0].split(":")[0], loop


def test_small_tiles_copy_no_accumulators_in_the_k_loop(tmp_path):
    """A register copy between two MFMAs of a step waits for the first: in the
    loops of the small tiles every accumulator stays in its registers."""
    if shutil.which(build.hipcc()) is None and not os.path.exists(build.hipcc()):
        pytest.skip("no hipcc")
    out = str(tmp_path / "k.s")
    res = subprocess.run([build.hipcc(), *build._hip_flags(), "-S", "--offload-device-only",
                          os.path.join(build.CSRC, "gemm_k7_12.hip"), "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    seen = 0
    for name, loop in k_loops(open(out).read()):
        assert loop is not None, name
        copies = [x.strip() for x in loop if "v_accvgpr" in x]
        assert not copies, (name, copies[:4])
        assert any("v_mfma" in x for x in loop), name
        seen += 1
    assert seen >= 15
