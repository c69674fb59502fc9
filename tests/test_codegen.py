"""The compiled kernels (gfx950 code of the built library), read on the CPU.

A kernel whose registers do not reach keeps values in accumulation registers
or scratch.  The compiler once put such copies, of values every lane needs,
at the top of a block where two sides of a branch join, ahead of the
instruction that switches the other side's lanes on again: those lanes kept
garbage, and loaded from it later.  The kernels are written without branches
between the reaction passes and the factorisation, where nearly every register
is live; that no copy stands in such a place anywhere is checked here, on what
was built."""
import os
import re
import shutil
import subprocess

import paper_2311_14941_amd as sc
from paper_2311_14941_amd import build

COPY = ("v_accvgpr_write", "scratch_store", "buffer_store")


def masked_copies(lines):
    """(kernel, instruction) of the copies that stand between a block's first
    instruction and the first in it that restores lanes of the execution mask.
    A block begins at a label or behind a branch."""
    found, kernel, block = [], None, []
    for s in lines:
        m = re.match(r"^(?:[0-9a-f]+ )?<(\w+)>:", s)
        if m:
            if not re.match(r"L\d+$", m.group(1)):
                kernel = m.group(1)
            block = []
            continue
        s = s.split("//")[0].strip()
        if not s:
            continue
        op, _, args = s.partition(" ")
        if op.startswith(("s_cbranch", "s_branch", "s_setpc", "s_endpgm")):
            block = []
        elif block is not None and (op == "s_or_saveexec_b64" or op == "s_or_b64" and args.strip().startswith("exec")):
            found += [(kernel, t) for t in block if t.startswith(COPY)]
            block = None
        elif args.split(",")[0].strip().startswith("exec") or "saveexec" in op:
            block = None  # lanes chosen by this block itself
        elif block is not None:
            block.append(s)
    return found


def test_a_copy_ahead_of_the_mask_is_found():
    join = ["<kernel>:", "\ts_and_saveexec_b64 s[0:1], vcc", "\ts_cbranch_execz L0", "\tv_accvgpr_write_b32 a1, v1", "",
            "<L0>:", "\tv_add_f64 v[0:1], v[0:1], v[2:3]", "{}", "\ts_or_b64 exec, exec, s[0:1]", "{}", "\ts_endpgm"]
    for copy in ("\tv_accvgpr_write_b32 a43, v0  // 00: D3", "\tscratch_store_dwordx2 off, v[0:1], off offset:4"):
        assert masked_copies([s.format(copy) if k == 7 else s.format("\ts_nop 0") for k, s in enumerate(join)]) == [
            ("kernel", copy.split("//")[0].strip())]
        assert masked_copies([s.format(copy) if k == 9 else s.format("\ts_nop 0") for k, s in enumerate(join)]) == []


def test_no_kernel_copies_under_part_of_the_mask(tmp_path):
    sc.ensure_built()
    objdump = os.path.join(os.path.dirname(os.path.realpath(build.HIPCC)), "..", "lib", "llvm", "bin", "llvm-objdump")
    if not os.path.exists(objdump):
        objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    lib = str(tmp_path / "lib.so")
    shutil.copy(sc.LIBPATH, lib)
    subprocess.run([objdump, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    kernels, found = set(), []
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" not in f:
            continue
        p = subprocess.Popen([objdump, "-d", "--symbolize-operands", "--no-show-raw-insn", "--no-leading-addr",
                              str(tmp_path / f)], stdout=subprocess.PIPE, text=True)
        lines = []
        for s in p.stdout:
            m = re.match(r"^(?:[0-9a-f]+ )?<(\w+)>:", s)
            if m and not re.match(r"L\d+$", m.group(1)):
                found += masked_copies(lines)
                lines = []
                kernels.add(m.group(1))
            lines.append(s)
        found += masked_copies(lines)
        assert p.wait() == 0
    assert sum("integrate" in k for k in kernels) > 40, len(kernels)
    assert not found, found[:10]
