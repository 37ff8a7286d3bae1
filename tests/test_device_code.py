"""CPU: the gfx950 code of the library as compiled.

The written-out direct loads (sdp_gemm_mfma.hip: direct_load) are out of the compiler's sight, which therefore adds no wait states
for them.  Two hazards apply: a scalar register that the vector unit wrote may be read by a memory instruction only five wait
states later, M0 by a load to LDS one instruction after a scalar move.  Each such load from a scalar base must stand behind
    s_mov_b32 m0, ..
    s_mov_b64 <its scalar base>, ..
and the move's source may come from wherever it likes (the scalar unit waits for the vector unit by itself)."""
import os
import re
import subprocess

import pytest

from paper_2507_09029_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
KERNEL = re.compile(r"[0-9a-f]+ <.*sdp_gemm_kernelI(?:Li\d+E){6}Li(\d)EEE.*>:")  # the last argument: which operands are depth-major
LOAD = re.compile(r"global_load_lds_dwordx4 v\d+, (s\[\d+:\d+\])")


def unsafe_loads(lines):
    """(scalar-base loads to LDS in the kernels that write them out, those that are not preceded by the two moves)"""
    n, bad, written_out = 0, [], False
    for i, line in enumerate(lines):
        if line.endswith(">:"):
            k = KERNEL.match(line)
            written_out = bool(k) and k[1] != "0"
        m = LOAD.match(line)
        if m and written_out:
            n += 1
            if not lines[i - 1].startswith(f"s_mov_b64 {m[1]}, ") or not lines[i - 2].startswith("s_mov_b32 m0, "):
                bad.append(lines[max(0, i - 6): i + 1])
    return n, bad


def test_written_out_loads_meet_their_hazards(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = build.LIB if os.path.exists(build.LIB) else build.build_library()
    local = tmp_path / "lib.so"
    os.symlink(lib, local)
    subprocess.run([OBJDUMP, "--offloading", str(local)], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    total, bad = 0, []
    for obj in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True, text=True).stdout
        n, b = unsafe_loads([line.split("//")[0].strip() for line in text.splitlines()])
        total, bad = total + n, bad + b
    assert total > 0
    assert not bad, "\n\n".join("\n".join(b) for b in bad[:3]) + f"\n{len(bad)} of {total} loads"
