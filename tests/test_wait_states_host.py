"""Distances between dependent vector instructions in the compiled kernels.

gfx950 needs two wait states (other instructions, or s_nop) between
  * a vector instruction that writes a vector register and a matrix instruction that reads it,
  * a vector instruction that writes a scalar register or vcc and a vector instruction that reads it,
  * a vector instruction that writes a vector register and a lane-exchange (permlane*_swap, DPP) that reads it.
The compiler keeps them for its own instructions, not around or inside written-out assembly.  The kernels are
compiled here as the library compiles them and every such pair is measured.  CPU only."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_1911_04477_amd import build

NEED = 2


def regs(op):
    """'v[4:7]' -> {('v', 4) ..}; 's3', 'vcc', 'a[0:15]', '-v3', '|v3|'; anything else: empty."""
    op = op.strip().strip("-|")
    if op.startswith("abs("):
        op = op[4:-1]
    if op.startswith("vcc"):
        return {("s", "vcc")}
    m = re.fullmatch(r"([vsa])\[(\d+):(\d+)\]", op) or re.fullmatch(r"([vsa])(\d+)", op)
    if not m:
        return set()
    lo = int(m.group(2))
    hi = int(m.group(3)) if m.lastindex == 3 else lo
    return {(m.group(1), r) for r in range(lo, hi + 1)}


def operands(text):
    out = []
    for t in re.split(r",\s*(?![^\[]*\])", text):
        out.append(t.strip().split(" ")[0] if t.strip() else "")
    return out


TWO_RESULTS = re.compile(r"v_(add_co|sub_co|subrev_co|addc_co|subb_co|subbrev_co|mad_u64_u32|mad_i64_i32|div_scale)")


def accesses(name, ops):
    """Registers written and read by one vector instruction."""
    if name.startswith(("v_permlane", "v_swap")):
        both = regs(ops[0]) | regs(ops[1])
        return both, both
    nd = 2 if TWO_RESULTS.match(name) else 1
    w = set().union(*[regs(o) for o in ops[:nd]])
    r = set().union(set(), *[regs(o) for o in ops[nd:]])
    if re.match(r"v_(fmac|mac|dot\w*c)_", name) or "dpp" in name:
        r |= regs(ops[0])  # read-modify-write, or lanes that keep their old value
    return w, r


def violations(asm):
    """(line number, line, wait states) of every reader that follows its writer too closely."""
    found, pending, at_label, want = [], [], {}, []
    lines = asm.splitlines()

    def step(line, no, pending, report):
        """One instruction: checks it against the pending writes [(age, register)], returns the new pending list."""
        code = line.split(";")[0].split("//")[0].strip()
        if not code or code.startswith(".") or code.endswith(":"):
            return pending, None
        name, _, rest = code.partition(" ")
        name = name.strip()
        if "\t" in name:
            name, _, rest = code.partition("\t")
        waits = 1
        if name == "s_nop":
            waits = int(rest.strip(), 0) + 1
        new = []
        if name.startswith("v_") and name != "v_nop":
            w, r = accesses(name, operands(rest))
            matrix = name.startswith("v_mfma")
            exchange = name.startswith("v_permlane") or "dpp" in name
            for age, reg in pending:
                if age < NEED and reg in r and (reg[0] == "s" or matrix or exchange):
                    report(no, line.strip(), age)
            if not matrix:
                new = [(0, reg) for reg in w]
        pending = [(age + waits, reg) for age, reg in pending if age + waits < NEED] + new
        target = None
        if name.startswith(("s_cbranch", "s_branch")):
            target = rest.strip()
        if name in ("s_branch", "s_endpgm", "s_setpc_b64"):
            return ([], (target, pending)) if target else ([], None)
        return pending, ((target, pending) if target else None)

    for no, line in enumerate(lines, 1):
        code = line.split(";")[0].strip()
        if re.fullmatch(r"[\w.$]+:", code):
            at_label[code[:-1]] = no
            continue
        pending, jump = step(line, no, pending, lambda *f: found.append(f))
        if jump and jump[1]:
            want.append(jump)
    for target, pend in want:  # along the taken branch
        no = at_label.get(target)
        while no is not None and no < len(lines) and pend:
            pend, _ = step(lines[no], no + 1, pend, lambda *f: found.append(f))
            pend = [(a, r) for a, r in pend if a > 0]  # only what was pending at the branch
            no += 1
    return found


def test_the_checker_itself():
    bad = violations("v_bfi_b32 v1, s0, v2, v3\nv_mov_b32 v9, v8\nv_mfma_scale_f32_32x32x64_f8f6f4 a[0:15], v[0:3], v[4:7], a[0:15]")
    assert [(n, a) for n, _, a in bad] == [(3, 1)]
    assert not violations("v_bfi_b32 v1, s0, v2, v3\ns_nop 1\nv_mfma_f32_32x32x1_2b_f32 v[64:95], v1, v4, v[64:95]")
    assert [a for _, _, a in violations("v_cmp_le_f32 vcc, 0, v1\nv_addc_co_u32 v0, vcc, v0, v0, vcc")] == [0]
    assert not violations("v_cmp_le_f32 s[0:1], 0, v1\nv_cmp_le_f32 vcc, 0, v2\ns_nop 0\nv_addc_co_u32 v0, s[0:1], v0, v0, s[0:1]")
    assert [a for _, _, a in violations("v_mov_b32 v1, 0\ns_cbranch_scc1 L\ns_nop 7\nL:\nv_permlane32_swap_b32 v0, v1")] == [1]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if shutil.which(build.HIPCC) is None:
        pytest.skip("needs hipcc")
    out = tmp_path_factory.mktemp("asm")

    def compile_one(source):
        path = str(out / (source + ".s"))
        subprocess.run([build.HIPCC, *build.FLAGS, *build.EXTRA_FLAGS.get(source, []), "-S", "--cuda-device-only",
                        os.path.join(build.CSRC, source), "-o", path], check=True, stderr=subprocess.DEVNULL)
        with open(path) as f:
            return f.read()

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        return dict(zip(build.SOURCES, ex.map(compile_one, build.SOURCES)))


@pytest.mark.parametrize("source", build.SOURCES)
def test_wait_states(source, assembly):
    bad = violations(assembly[source])
    assert not bad, f"{len(bad)} readers too close: " + "; ".join(f"{n}: {t} ({a})" for n, t, a in bad[:4])
