"""The built library's device code keeps the wait that the result of a matrix
instruction needs before any other instruction reads or overwrites it.  The
hardware does not hold such an access back; the compiler inserts the wait, but
has left it out where a branch with an empty side lies between the last product
and the first read of its result (wrong energies, no error).  In straight code
it keeps 8 wait states after the BF16 instructions and 10 after the FP32 one:
fewer on any path through any kernel fails (a load may name the registers of a
dead result at once: what it loads comes long after the product has ended).

A later matrix instruction that takes the result as its accumulator waits for
it in hardware, and everything after that one is later still."""
import os
import re
import shutil
import struct
import subprocess

import pytest

STATES = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_16x16x16_bf16": 8, "v_mfma_f32_16x16x4_f32": 10}
REG = re.compile(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+)\b)")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def regs(text):
    return [(t, k) for t, a, b, c in REG.findall(text) for k in (range(int(a), int(b) + 1) if a else (int(c),))]


def kernels(listing):
    """(name, instructions and labels) of each function of a listing."""
    name, body = None, []
    for line in listing.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m and re.match(r"L\d+$", m.group(1)):
            body.append(m.group(1) + ":")
        elif m:
            if name:
                yield name, body
            name, body = m.group(1), []
        elif name and line.startswith("\t"):
            body.append(line.split("//")[0].strip())
    if name:
        yield name, body


def early_uses(body):
    """(position, instruction, states kept, states needed) of uses that come too early on some path."""
    at_label, bad = {}, {}
    for _ in range(3):   # loops carry an age around once
        age = {}         # register -> (states since its matrix instruction issued, states needed)
        for n, line in enumerate(body):
            if line.endswith(":"):
                for r, (a, w) in at_label.get(line[:-1], {}).items():
                    if r not in age or age[r][0] - age[r][1] > a - w:
                        age[r] = (a, w)
                continue
            op, _, rest = line.partition(" ")
            args = [regs(t) for t in rest.split(",")] if rest else []
            if op.startswith("v_mfma"):
                for r in args[1] + args[2]:
                    if r in age:
                        bad[n] = (line, *age[r])
                for r in (args[3] if len(args) > 3 else []):
                    age.pop(r, None)
            else:
                loads = op.startswith(("ds_read", "global_load", "buffer_load", "scratch_load"))
                for r in (r for g in args[loads:] for r in g):
                    if r in age:
                        bad[n] = (line, *age[r])
                for r in (args[0] if loads and args else []):   # arrives far later than the product ends
                    age.pop(r, None)
            step = int(rest, 0) + 1 if op == "s_nop" else 1
            age = {r: (a + step, w) for r, (a, w) in age.items() if a + step < w}
            if op.startswith("v_mfma"):
                for r in args[0]:
                    age[r] = (0, STATES[op])
            if op.startswith(("s_cbranch", "s_branch")):
                d = at_label.setdefault(rest.split()[0], {})
                for r, (a, w) in age.items():
                    if r not in d or d[r][0] - d[r][1] > a - w:
                        d[r] = (a, w)
            if op in ("s_branch", "s_endpgm"):
                age = {}
    return [(n, *v) for n, v in sorted(bad.items())]


def code_objects(path):
    """The gfx950 code objects bundled in a library."""
    data, at = open(path, "rb").read(), 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        count, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in target and size:
                yield data[at + offset:at + offset + size]
        at += 24


PRODUCT = """
0000000000000100 <k>:
\tv_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], 0
{between}
\tv_add_f32_e32 v4, v0, v5
\ts_endpgm
"""


@pytest.mark.parametrize("between,early", [
    ("\ts_nop 7", 0), ("\ts_nop 6", 1), ("\ts_nop 6\n\tv_mov_b32_e32 v20, 0", 0),
    # the wait on one side of a branch only
    ("\ts_cbranch_scc1 L1\n\ts_nop 7\n0000000000000200 <L1>:", 1),
    ("\ts_nop 3\n\ts_cbranch_scc1 L1\n\ts_nop 7\n0000000000000200 <L1>:\n\ts_nop 2", 0),
    # overwritten too early; taken as an accumulator, whose own wait then counts
    ("\tv_mov_b32_e32 v1, 0\n\ts_nop 7", 1),
    ("\tv_mfma_f32_16x16x32_bf16 v[16:19], v[8:11], v[12:15], v[0:3]\n\tv_mov_b32_e32 v1, 0", 0),
    ("\tv_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]\n\ts_nop 4", 1),
])
def test_scanner(between, early):
    found = [early_uses(body) for _, body in kernels(PRODUCT.format(between=between))]
    assert [len(f) for f in found] == [early]


def test_library_waits(tmp_path):
    import paper_2509_21694_amd as M
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    seen = 0
    for k, obj in enumerate(code_objects(M.LIB_PATH)):
        path = tmp_path / f"{k}.o"
        path.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", "--mcpu=gfx950", str(path)],
                              capture_output=True, text=True, check=True).stdout
        assert set(re.findall(r"v_mfma_\w+", text)) <= set(STATES)
        for name, body in kernels(text):
            if any("v_mfma" in x for x in body):
                seen += 1
                assert early_uses(body) == [], name
    assert seen > 100
