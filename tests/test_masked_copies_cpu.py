"""The built kernels hold no register copy under a mask that has not been lifted.

At the end of a divergent block the compiler once moved values that every lane
needs to other registers before the masked lanes were back: those lanes then
loaded tables at an undefined index.  Such a copy stands between a branch target
(the end of the block) and the `s_or_b64 exec` that follows it, and its
destination is written nowhere else in the kernel.  Nothing in the source rules
it out, so every build is searched for it."""
import re
import shutil
import subprocess
from concurrent.futures import ProcessPoolExecutor

import pytest

from built_code import code_objects, llvm_tool

OBJDUMP = llvm_tool("llvm-objdump")
# instructions whose first operand is not a vector register that they write
NO_DST = ("global_store", "ds_write", "scratch_store", "flat_store", "buffer_store", "s_", "v_cmp", "v_readlane",
          "v_readfirstlane")
LINE = re.compile(r"\t(\S+)\s*([^/]*?)\s*//\s*([0-9A-F]+):")
REG = re.compile(r"([va])(?:(\d+)|\[(\d+):(\d+)\])$")


def registers(operand):
    m = REG.match(operand)
    if not m:
        return []
    lo, hi = (m[2], m[2]) if m[2] else (m[3], m[4])
    return [(m[1], r) for r in range(int(lo), int(hi) + 1)]


def masked_copies(listing):
    """(kernels, copies): copies as (kernel, instruction) in llvm-objdump's listing."""
    kernels, hits = 0, []
    for body in re.split(r"\n(?=[0-9a-f]{16} <)", listing)[1:]:
        name = body[body.index("<") + 1:body.index(">")]
        code, targets, writes = [], set(), {}
        for m in LINE.finditer(body):
            op, args, addr = m[1], m[2], int(m[3], 16)
            if op.startswith(("s_cbranch", "s_branch")):
                off = int(args.split()[0])
                targets.add(addr + 4 + 4 * (off - 65536 if off > 32767 else off))
            elif not op.startswith(NO_DST):
                for r in registers(args.split(",")[0]):
                    writes.setdefault(r, []).append(addr)
            code.append((addr, op, args))
        kernels += bool(code)
        copies, mask_end = [], False
        for addr, op, args in code:
            if addr in targets:
                copies, mask_end = [], True
            if not mask_end:
                continue
            if op == "s_or_b64" and args.startswith("exec, exec"):
                own = {a for a, _ in copies}
                hits += [(name, text) for a, text in copies
                         if any(set(writes[r]) <= own for r in registers(text.split(None, 1)[1].split(",")[0]))]
                mask_end = False
            elif op.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_and_saveexec", "s_mov_b64 exec")):
                mask_end = False
            elif op.startswith("v_") and not op.startswith(NO_DST) and registers(args.split(",")[0]):
                copies.append((addr, f"{op} {args}"))
    return kernels, hits


def _scan(obj, tmp):
    path = tmp / f"{hash(obj)}.co"
    path.write_bytes(obj)
    r = subprocess.run([OBJDUMP, "-d", str(path)], capture_output=True, text=True, check=True)
    return masked_copies(r.stdout)


FAULTY = """
x:	file format elf64-amdgpu

0000000000001000 <kernel>:
	v_mov_b32_e32 v95, 1                                       // 000000001000: 7E
	s_and_saveexec_b64 s[4:5], vcc                             // 000000001004: BE
	s_cbranch_execz 2                                          // 000000001008: BF
	v_add_f64 v[2:3], v[2:3], v[4:5]                           // 00000000100C: D2 00
	v_mov_b32_e32 v7, v8                                       // 000000001010: 7E
	v_accvgpr_write_b32 a129, v95                              // 000000001014: D3 00
	s_or_b64 exec, exec, s[4:5]                                // 00000000101C: 87
	v_accvgpr_read_b32 v1, a129                                // 000000001020: D3 00
	s_endpgm                                                   // 000000001028: BF
"""


def test_search_finds_a_masked_copy():
    assert masked_copies(FAULTY) == (1, [("kernel", "v_accvgpr_write_b32 a129, v95")])
    lines = FAULTY.splitlines(True)
    restore = next(i for i, l in enumerate(lines) if "s_or_b64" in l)
    lines[restore - 1], lines[restore] = (lines[restore].replace("00000000101C", "000000001014"),
                                          lines[restore - 1].replace("000000001014", "000000001018"))
    assert masked_copies("".join(lines)) == (1, [])


@pytest.mark.skipif(not shutil.which(OBJDUMP), reason="needs llvm-objdump")
def test_no_masked_copy_in_the_built_library(tmp_path):
    from paper_2506_09743_amd import build
    objs = code_objects(build.LIB)
    assert objs
    with ProcessPoolExecutor(4) as pool:
        found = list(pool.map(_scan, objs, [tmp_path] * len(objs)))
    assert sum(k for k, _ in found) > 100
    assert [h for _, hs in found for h in hs] == []
