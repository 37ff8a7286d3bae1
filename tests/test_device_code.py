"""CPU: the gfx950 code of the library as compiled.

The written-out direct loads (sdp_gemm_mfma.hip: direct_load) are out of the compiler's sight, which therefore adds no wait states
for them.  Two hazards apply: a scalar register that the vector unit wrote may be read by a memory instruction only five wait
states later, M0 by a load to LDS one instruction after a scalar move.  Each such load from a scalar base must stand behind
    s_mov_b32 m0, ..
    s_mov_b64 <its scalar base>, ..
and the move's source may come from wherever it likes (the scalar unit waits for the vector unit by itself).

The attention core's matrix instructions that read LDS rows which the whole workgroup has put there stand behind a barrier on every
path from the kernel's entry."""
import os
import re
import subprocess

import pytest

from paper_2507_09029_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
# the last argument: which operands are depth-major; two contractions in one launch always have some
KERNEL = re.compile(r"[0-9a-f]+ <.*sdp_gemm_(?:kernelI(?:Li\d+E){6}Li(\d)E|(pair)_kernelI(?:Li\d+E){5})EE.*>:")
LOAD = re.compile(r"global_load_lds_dwordx4 v\d+, (s\[\d+:\d+\])")


def unsafe_loads(lines):
    """({in a pair's kernel: scalar-base loads to LDS where they are written out}, those that are not preceded by the two moves)"""
    n, bad, written_out, pair = {False: 0, True: 0}, [], False, False
    for i, line in enumerate(lines):
        if line.endswith(">:"):
            k = KERNEL.match(line)
            written_out, pair = bool(k) and k[1] != "0", bool(k) and bool(k[2])
        m = LOAD.match(line)
        if m and written_out:
            n[pair] += 1
            if not lines[i - 1].startswith(f"s_mov_b64 {m[1]}, ") or not lines[i - 2].startswith("s_mov_b32 m0, "):
                bad.append(lines[max(0, i - 6): i + 1])
    return n, bad


def gfx950_code(folder):
    """the disassembly of each of the library's device objects, as lines"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = build.LIB if os.path.exists(build.LIB) else build.build_library()
    local = folder / "lib.so"
    os.symlink(lib, local)
    subprocess.run([OBJDUMP, "--offloading", str(local)], cwd=folder, check=True, stdout=subprocess.DEVNULL)
    for obj in sorted(folder.glob("lib.so.*gfx950")):
        yield subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True, text=True).stdout.splitlines()


def test_written_out_loads_meet_their_hazards(tmp_path):
    single, pairs, bad = 0, 0, []
    for lines in gfx950_code(tmp_path):
        n, b = unsafe_loads([line.split("//")[0].strip() for line in lines])
        single, pairs, bad = single + n[False], pairs + n[True], bad + b
    assert single > 0 and pairs > 0
    assert not bad, "\n\n".join("\n".join(b) for b in bad[:3]) + f"\n{len(bad)} of {single + pairs} loads"


def kernels(lines):
    """{symbol: [(offset, instruction, offset of the branch target or None)]}"""
    out, code, base = {}, None, 0
    for line in lines:
        m = re.match(r"([0-9a-f]+) <(.*)>:", line)
        if m:
            base, code = int(m[1], 16), out.setdefault(m[2], [])
        elif code is not None and "//" in line:
            ins, note = line.split("//", 1)
            target = re.search(r"\+0x([0-9a-f]+)>\s*$", note)
            code.append((int(note.split(":")[0], 16) - base, ins.strip(), int(target[1], 16) if target else None))
    return out


def mfmas_before_a_barrier(code):
    """matrix instructions that some path from the entry reaches without a barrier"""
    at = {offset: i for i, (offset, _, _) in enumerate(code)}
    seen, todo, n = set(), [0], 0
    while todo:
        i = todo.pop()
        while i is not None and i not in seen:
            seen.add(i)
            _, ins, target = code[i]
            assert not ins.startswith(("s_setpc", "s_swappc")), "the paths cannot be followed"
            if ins.startswith(("s_barrier", "s_endpgm")):
                break
            n += ins.startswith("v_mfma")
            if ins.startswith("s_cbranch"):
                todo.append(at[target])
            i = at[target] if ins.startswith("s_branch") else i + 1
    return n


def test_rows_that_a_workgroup_shares_are_read_behind_a_barrier(tmp_path):
    counts = {}
    for lines in gfx950_code(tmp_path):
        for symbol, code in kernels(lines).items():
            k = re.search(r"(attn_(?:fwd|bwd|bwd_dq|bwd_dkv)_kernel)ILi(\d+)ELi(\d)EE", symbol)
            if k:
                counts[k[1], int(k[2]), int(k[3])] = mfmas_before_a_barrier(code)
    # one wave along the walked axis: the workgroup's tiles; eight: dK/dV's rows of V (heads above 64), of K (above 96)
    shared = {(name, hw, 1): 0 for name in ("attn_fwd_kernel", "attn_bwd_dq_kernel", "attn_bwd_dkv_kernel") for hw in (64, 96, 128)}
    shared |= {("attn_bwd_dkv_kernel", hw, 8): 0 for hw in (96, 128)}
    # dK/dV and dQ in one launch: dQ's waves have tiles of their own, and no more than these come without a barrier
    shared |= {("attn_bwd_kernel", hw, 8): counts["attn_bwd_dq_kernel", hw, 8] for hw in (96, 128)}
    assert {k: counts[k] for k in shared} == shared


def test_attention_kernels_know_where_delta_comes_from(tmp_path):
    """dK/dV takes delta from memory or from O's rows by its kind: a choice at run time between the two pointers, one of them null, costs
    registers and shows as an access of no known address space"""
    seen = 0
    for lines in gfx950_code(tmp_path):
        for symbol, code in kernels(lines).items():
            if re.search(r"attn_(?:f32_)?(?:fwd|bwd|dq|dkv|bwd_dq|bwd_dkv)_kernelI", symbol):
                seen += 1
                assert not [ins for _, ins, _ in code if ins.startswith("flat_")], symbol
    assert seen > 0
