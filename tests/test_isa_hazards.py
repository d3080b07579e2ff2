"""Wait states around the inline assembly of the built library.

The compiler fills the gaps that gfx950 asks for between dependent vector instructions, but it
does not look inside inline assembly.  This test disassembles the library's own code object and
checks every pair of dependent instructions against the wait states that the compiler itself
leaves (an instruction counts 1, `s_nop N` counts N + 1), along fall-through and every branch:

    VALU write of VCC or a scalar register -> VALU read of it (carry-in, mask)      2
    VALU write of a vector or accumulation register -> MFMA read of it              2
    VALU write of a vector register -> row swap (v_permlane*_swap) of it            2
    MFMA write -> any other instruction that reads or overwrites the result         7
"""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2608_22883_amd", "lib", "libfovea.so")
LLVM = "/opt/rocm/llvm/bin"
WINDOW = 8  # the longest gap checked, and one more


def registers(op):
    """The 32-bit registers of an operand (VCC as one)."""
    op = op.strip().lstrip("-").strip("|")
    if op in ("vcc", "vcc_lo", "vcc_hi"):
        return ["vcc"]
    m = re.fullmatch(r"([vas])(\d+)", op)
    if m:
        return [op]
    m = re.fullmatch(r"([vas])\[(\d+):(\d+)\]", op)
    if m:
        return [m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)]
    return []


class Inst:
    __slots__ = ("addr", "text", "name", "wait", "reads", "writes", "kind", "target")

    def __init__(self, addr, text, target):
        self.addr, self.text, self.target = addr, text, target
        name, _, rest = text.partition(" ")
        ops = [o.split()[0] if o.split() else "" for o in rest.split(",")] if rest else []
        self.name = name
        self.wait = int(ops[0], 0) + 1 if name == "s_nop" else 1
        self.kind = "mfma" if name.startswith("v_mfma") else "valu" if name.startswith("v_") else ""
        self.reads, self.writes = [], []
        if self.kind:
            n = 0 if name == "v_nop" else 1
            if "_co_" in name or name.startswith("v_div_scale") or "swap" in name:
                n = 2
            for o in ops[:n]:
                self.writes += registers(o)
            for o in ops[n:]:
                self.reads += registers(o)
            if "swap" in name or name.startswith(("v_fmac", "v_mac", "v_dot2c")):
                self.reads += self.writes
            if name.startswith("v_div_fmas"):
                self.reads.append("vcc")
        elif name.startswith(("ds_", "global_", "buffer_", "flat_", "scratch_")):
            load = not any(s in name for s in ("store", "write", "lds", "atomic"))
            for o in ops[1:] if load else ops:
                self.reads += registers(o)


def check(inst, last, now):
    """The broken gap of one instruction, or None; `last`: register -> (time, kind) of its write."""
    if not (inst.kind or inst.reads):
        return None
    for r in inst.reads:
        if r not in last:
            continue
        t, kind = last[r]
        gap = now - t - 1
        if kind == "valu" and inst.kind == "valu" and (r == "vcc" or r[0] == "s"):
            need = 2
        elif kind == "valu" and r[0] in "va" and (inst.kind == "mfma" or "permlane" in inst.name):
            need = 2
        elif kind == "mfma" and inst.kind != "mfma":
            need = 7
        else:
            continue
        if gap < need:
            return f"{r}: {gap} of {need} wait states before {inst.text}"
    if inst.kind == "valu":
        for r in inst.writes:
            if r in last and last[r][1] == "mfma" and now - last[r][0] - 1 < 7:
                return f"{r}: overwritten {now - last[r][0] - 1} wait states after an MFMA by {inst.text}"
    return None


def kernels(text):
    """(name, instructions) of every function of an llvm-objdump listing."""
    name, out = None, []
    for line in text.splitlines():
        m = re.match(r"^(?:[0-9a-f]+ )?<(.*)>:$", line)
        if m:
            if out:
                yield name, out
            name, out = m.group(1), []
        elif line.startswith("\t") and "//" in line:
            body, note = line.strip().split("//", 1)
            addr = int(note.split(":")[0], 16)
            m = re.search(r"<[^+>]*(?:\+0x([0-9a-f]+))?>", note) if "branch" in body else None
            out.append(Inst(addr, " ".join(body.split()), int(m.group(1) or "0", 16) if m else None))
    if out:
        yield name, out


def broken_gaps(insts):
    """Every broken gap of a function, along fall-through and (one branch deep) every branch."""
    at = {i.addr - insts[0].addr: n for n, i in enumerate(insts)}
    found = []

    def step(n, last, now):
        i = insts[n]
        bad = check(i, last, now)
        if bad:
            found.append(f"{i.addr:#x} {bad}")
        for r in i.writes:
            last[r] = (now, i.kind)
        return now + i.wait

    last, now = {}, 0
    for n, i in enumerate(insts):
        now = step(n, last, now)
        if i.target is not None:
            side = {r: w for r, w in last.items() if now - w[0] <= WINDOW}
            m, t = at[i.target], now
            while side and t - now < WINDOW and m < len(insts):
                t = step(m, side, t)
                if insts[m].name in ("s_branch", "s_endpgm"):
                    break
                m += 1
        if i.name in ("s_branch", "s_endpgm", "s_setpc_b64"):
            last = {}
    return sorted(set(found))


def listing(tmp):
    objcopy, bundler, objdump = (os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump"))
    if not all(shutil.which(t) for t in (objcopy, bundler, objdump)):
        pytest.skip("no LLVM tools to list the code object with")
    fat, co = str(tmp / "fat.bin"), str(tmp / "gfx950.co")
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout  # noqa: E731
    run(objcopy, "--dump-section", f".hip_fatbin={fat}", LIB, os.devnull)
    run(bundler, "--unbundle", "--type=o", f"--input={fat}", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
        f"--output={co}")
    return run(objdump, "-d", "--no-show-raw-insn", co)


@pytest.mark.parametrize("code,broken", [
    (["v_cmp_ge_f32_e32 vcc, v1, v2", "v_addc_co_u32_e32 v0, vcc, v0, v0, vcc"], 1),
    (["v_cmp_ge_f32_e32 vcc, v1, v2", "s_nop 1", "v_addc_co_u32_e32 v0, vcc, v0, v0, vcc"], 0),
    (["v_cmp_ge_f32_e64 s[2:3], v1, v2", "v_mov_b32_e32 v5, v6", "v_addc_co_u32_e64 v0, vcc, v0, v0, s[2:3]"], 1),
    (["v_accvgpr_write_b32 a2, v1", "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"], 1),
    (["v_mov_b32_e32 v3, v1", "s_nop 0", "v_permlane32_swap_b32_e32 v2, v3"], 1),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", "s_nop 5", "v_accvgpr_read_b32 v1, a3"], 1),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", "s_nop 6", "v_accvgpr_read_b32 v1, a3"], 0),
])
def test_scan_finds_short_gaps(code, broken):
    text = "<f>:\n" + "".join(f"\t{c} // {8 * n:012X}: 0\n" for n, c in enumerate(code))
    (_, insts), = kernels(text)
    assert len(broken_gaps(insts)) == broken


def test_library_keeps_the_wait_states(tmp_path):
    seen, bad = 0, []
    for name, insts in kernels(listing(tmp_path)):
        seen += sum(i.kind == "mfma" for i in insts)
        gaps = broken_gaps(insts)
        if gaps:
            bad.append(f"{name[:70]}: {len(gaps)}, first {gaps[0]}")
    assert seen > 1000, "no matrix instructions found: the listing was not read"
    assert not bad, "\n".join(bad)
