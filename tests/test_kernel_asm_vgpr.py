"""MFMA results kept in VGPRs, in the gfx950 code of the built library (CPU
only: the library's own code objects are disassembled).

A matrix instruction's result may be read by another instruction only when
its passes are over; the compiler puts waits (s_nop or other work) in
between.  tests/test_kernel_asm.py looks for a misplaced wait behind a read of
an accumulator register (AGPR); the wave-row kernels keep their accumulators
in VGPRs, which any instruction may read.  So: along every straight run of
code (a branch not taken goes on), no instruction other than an MFMA reads a
result register fewer wait states after its MFMA than the MFMA has passes:
16 for the FP64 16x16x4 form, 8 for FP32 16x16x4, 4 for FP64 4x4x4."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2109_05451_amd", "libh2gemv.so")
OBJDUMP = os.environ.get("LLVM_OBJDUMP", "/opt/rocm/llvm/bin/llvm-objdump")
PASSES = {"v_mfma_f64_16x16x4_f64": 16, "v_mfma_f32_16x16x4_f32": 8, "v_mfma_f64_4x4x4_4b_f64": 4}


def registers(operand):
    m = re.fullmatch(r"-?\|?([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand)
    if not m:
        return []
    lo, hi = (m[2], m[2]) if m[2] else (m[3], m[4])
    return [(m[1], i) for i in range(int(lo), int(hi) + 1)]


def early_reads(lines):
    """(function, instruction, wait states) of each read that comes too soon,
    and the number of MFMAs by form."""
    out, count, live, fn = [], {}, {}, None
    for line in lines:
        s = line.split("//")[0].strip()
        if s.endswith(">:"):
            fn, live = s[1:-2], {}
            continue
        if not line.startswith(("\t", " ")) or not s:
            continue
        name, _, rest = s.partition(" ")
        if name in ("s_branch", "s_endpgm", "s_setpc_b64"):
            live = {}
            continue
        ops = [o.split()[0] for o in rest.split(",") if o.strip()]
        mfma = name.startswith("v_mfma")
        store = "store" in name or "write" in name.split("_")[1:2]
        if not mfma:
            for r in (r for o in (ops if store else ops[1:]) for r in registers(o)):
                if r in live and live[r][0] < live[r][1]:
                    out.append((fn, s, live[r][0]))
        step = int(ops[0], 0) + 1 if name == "s_nop" else 1
        live = {r: (d + step, p) for r, (d, p) in live.items() if d + step < p}
        if mfma:
            base = name.split("_e64")[0]
            count[base] = count.get(base, 0) + 1
            if base in PASSES:
                live.update({r: (0, PASSES[base]) for r in registers(ops[0])})
        elif ops and not store:
            for r in registers(ops[0]):
                live.pop(r, None)
    return out, count


def test_scanner_finds_the_pattern():
    head = ["<_Zk>:", "\tv_mfma_f64_16x16x4_f64 v[0:7], v[8:9], v[10:11], v[0:7]"]
    assert len(early_reads(head + ["\tv_add_f64 v[12:13], v[6:7], v[14:15]", "\ts_nop 15"])[0]) == 2
    assert len(early_reads(head + ["\ts_nop 7", "\tglobal_store_dwordx2 v[20:21], v[0:1], off"])[0]) == 2
    assert early_reads(head + ["\ts_nop 15", "\tv_add_f64 v[12:13], v[6:7], v[14:15]"])[0] == []
    assert early_reads(head + ["\ts_branch 12", "\tv_add_f64 v[12:13], v[6:7], v[14:15]"])[0] == []


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not available")
def test_no_early_read_of_a_result(tmp_path):
    shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    objects = sorted(glob.glob(str(tmp_path / "lib.so.*gfx950")))
    assert objects
    total = {}
    for obj in objects:
        p = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", obj], check=True,
                           capture_output=True, text=True)
        hits, count = early_reads(p.stdout.splitlines())
        assert hits == [], hits[:3]
        for k, v in count.items():
            total[k] = total.get(k, 0) + v
    # the forms that the test knows, and no other of these types
    assert total.get("v_mfma_f64_16x16x4_f64", 0) > 1000
    assert all(k in PASSES for k in total if "f64" in k or "f32_16x16x4_f32" in k), total
