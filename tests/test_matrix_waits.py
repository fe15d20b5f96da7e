"""The waits around the matrix products and the direct-to-LDS loads that are written as inline assembly (csrc/mq_linear.h), in the
compiled library.

The compiler does not see those products and places no waits for them.  The rules it keeps for its own: an operand that a vector
instruction has written is read two wait states later at the earliest, a result of the 16x16x32 product is read or written by
anything but the next product into it eight wait states later at the earliest.  A scalar register that a vector instruction has
written is read by a load or store five wait states later at the earliest, m0 by a direct-to-LDS load one.  Every path through the kernels is followed for that
long, over branches and the ends of loops."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_06786_amd import build as mq_build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
KERNELS = re.compile(r"_ZN2mq\d+(fwd_kernel|fwd_split_kernel|fwd_wide_kernel|dx_kernel|dw_kernel)I")
OPERAND_WAIT, RESULT_WAIT, DESCRIPTOR_WAIT, M0_WAIT = 2, 8, 5, 1
PRODUCT = "v_mfma_f32_16x16x32_bf16"


def _registers(text, kinds="va"):
    out = set()
    for kind, one, lo, hi in re.findall(rf"(?<![\w.])([{kinds}])(?:(\d+)|\[(\d+):(\d+)\])(?!\w)", text):
        out.update((kind, i) for i in (range(int(lo), int(hi) + 1) if lo else [int(one)]))
    return out


def parse(lines):
    """Instructions of one kernel: (text, wait states, registers read, registers written, product, successors)."""
    code, at = [], {}
    for line in lines:
        m = re.match(r"\s+([a-z]\w*)(.*?)//\s*([0-9A-F]+):[^<]*(?:<[^>+]*\+?(0x[0-9a-f]+)?>)?", line)
        if m:
            at[int(m.group(3), 16)] = len(code)
            code.append((m.group(1), m.group(2).strip(), m.group(4)))
    start = min(at) if at else 0
    out = []
    for i, (op, args, target) in enumerate(code):
        parts = [p.strip() for p in args.split(",")]
        product = op.startswith("v_mfma")
        read, written = set(), set()
        if op.startswith("v_"):
            first = 2 if "swap" in op else 1   # a swap writes both of its operands
            for p in parts[:first]:
                written |= _registers(p)
            for p in parts[first - 1 if "swap" in op else 1:]:
                read |= _registers(p)
            if "swap" in op:
                read |= written
        else:
            read = _registers(args)            # memory and LDS: a load's destination counts, a late arrival is waited for elsewhere
        steps = int(parts[0], 0) + 1 if op == "s_nop" else 1
        following = [] if op in ("s_endpgm", "s_branch") else [i + 1]
        if op.startswith(("s_branch", "s_cbranch")):
            following.append(at[start + int(target or "0", 16)])
        out.append((op + " " + args, steps, read, written, product, [f for f in following if f < len(code)]))
    return out


def violations(code):
    found = []

    def memory(other):
        return other[0].startswith(("buffer_", "global_", "flat_", "scratch_"))

    def follow(i, regs, wait, bad):
        seen, stack = {}, [(f, wait) for f in code[i][5]]
        while stack:
            j, left = stack.pop()
            if left <= 0 or seen.get(j, 0) >= left:
                continue
            seen[j] = left
            if bad(code[j], regs):
                found.append((code[i][0], code[j][0], wait - left))
                continue
            stack += [(f, left - code[j][1]) for f in code[j][5]]

    for i, (text, _, read, written, product, _) in enumerate(code):
        if product:
            # the next product into the same accumulator is exempt, as an operand of another one the result is not
            def bad(other, regs):
                if not other[4]:
                    return bool(regs & (other[2] | other[3]))
                return bool(regs & other[2]) and other[3] != regs or bool(regs & _registers(",".join(other[0].split(",")[1:3])))
            follow(i, written, RESULT_WAIT, bad)
        elif text.startswith("v_") and written:
            follow(i, written, OPERAND_WAIT, lambda other, regs: other[4] and bool(regs & other[2]))
        op, _, args = text.partition(" ")
        scalars = _registers(args.split(",")[0], "s") if op.startswith("v_") else set()
        if scalars:
            follow(i, scalars, DESCRIPTOR_WAIT, lambda other, regs: memory(other) and bool(regs & _registers(other[0], "s")))
        if op.startswith("s_") and args.split(",")[0].strip() == "m0":
            follow(i, {"m0"}, M0_WAIT, lambda other, regs: memory(other) and other[0].endswith(" lds"))
    return found


def test_the_scan_sees_what_it_looks_for():
    def code(*lines):
        return parse(["\t%s // %012X: 00000000%s" % (t, 4 * i, " <k+%s>" % t.split("@")[1] if "@" in t else "") for i, t in enumerate(lines)])

    p = PRODUCT + " a[0:3], v[0:3], v[4:7], a[0:3]"
    q = PRODUCT + " a[4:7], v[8:11], v[4:7], a[4:7]"
    assert not violations(code("v_add_u32 v20, v1, v2", p, p, q, "s_nop 7", "v_accvgpr_read_b32 v9, a0", "s_endpgm"))
    assert len(violations(code("v_add_u32 v1, v1, v2", p, "s_endpgm"))) == 1
    assert len(violations(code("v_add_u32 v1, v1, v2", "s_nop 0", p, "s_endpgm"))) == 1
    assert not violations(code("v_add_u32 v1, v1, v2", "s_nop 1", p, "s_endpgm"))
    assert len(violations(code("v_permlane16_swap_b32 v20, v5", q, "s_endpgm"))) == 1
    assert len(violations(code("v_accvgpr_write_b32 a2, v1", p, "s_endpgm"))) == 1
    assert len(violations(code(p, "s_nop 6", "v_accvgpr_read_b32 v9, a3", "s_endpgm"))) == 1
    assert not violations(code(p, "s_nop 7", "global_store_dwordx4 v[12:13], a[0:3], off", "s_endpgm"))
    assert len(violations(code(p, "s_nop 6", "global_store_dwordx4 v[12:13], a[0:3], off", "s_endpgm"))) == 1
    # descriptors and m0
    load = "buffer_load_dwordx4 v5, s[8:11], 0 offen lds"
    assert len(violations(code("v_readfirstlane_b32 s9, v1", "s_nop 3", load, "s_endpgm"))) == 1
    assert not violations(code("v_readfirstlane_b32 s9, v1", "s_nop 4", load, "s_endpgm"))
    assert not violations(code("v_readfirstlane_b32 s12, v1", load, "s_endpgm"))
    assert len(violations(code("v_readfirstlane_b32 s8, v1", p, "s_mov_b32 s3, s4", q, "s_nop 0", load, "s_endpgm"))) == 1
    assert len(violations(code("s_add_u32 m0, s4, 0x1000", load, "s_endpgm"))) == 1
    assert not violations(code("s_add_u32 m0, s4, 0x1000", p, load, "s_endpgm"))
    # around the end of a loop: the write is the last instruction but one, the product the first
    assert len(violations(code("s_nop 7", p, "s_nop 7", "v_add_u32 v1, v1, v2", "s_cbranch_scc1 65532 @0x4", "s_endpgm"))) == 1
    assert not violations(code("s_nop 7", p, "s_nop 7", "v_add_u32 v1, v1, v2", "s_cbranch_scc1 65531 @0x0", "s_endpgm"))


def test_products_of_the_library(tmp_path):
    if not os.path.exists(mq_build.LIB):
        pytest.fail(f"{mq_build.LIB} is not built (python -c 'import __graft_entry__ as g; g.build()')")
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    shutil.copy(mq_build.LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    kernels = products = loads = 0
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", name], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]{16} <)", text):
            m = re.match(r"[0-9a-f]{16} <([^>]+)>:", part)
            if not m or not KERNELS.match(m.group(1)):
                continue
            code = parse(part.split("\n")[1:])
            kernels += 1
            products += sum(c[4] for c in code)
            loads += sum(c[0].endswith(" lds") for c in code)
            assert not violations(code), (m.group(1), violations(code)[:3])
    assert kernels > 100 and products > 5000 and loads > 500
