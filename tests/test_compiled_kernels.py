"""Properties of the compiled kernels that no run shows reliably, read from the assembly of the library built here (no
GPU)."""
import os
import re
import subprocess
import sys

import pytest

from paper_2602_08426_amd import binding as pb
from paper_2602_08426_amd import build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> instructions of every kernel of the built library."""
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(pb.library_path()):
        build.build_library()
    tmp = tmp_path_factory.mktemp("code")
    os.symlink(pb.library_path(), tmp / "lib.so")
    objdump = os.path.join(LLVM, "llvm-objdump")
    subprocess.run([objdump, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    out, name = {}, None
    for part in sorted(p for p in os.listdir(tmp) if p.endswith("gfx950")):
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", part], cwd=tmp, check=True, capture_output=True,
                              text=True).stdout
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(_Z\w+)>:", line)
            if m:
                name = m.group(1)
                out[name] = []
            elif name is not None and line.startswith("\t"):
                out[name].append(line.split("//")[0].strip())
    return out


def _lds_address(ins, constants):
    """Byte address of a one-word LDS access, or None if its base register holds no known constant."""
    m = re.match(r"ds_read_b32 v\d+, v(\d+)|ds_write_b32 v(\d+),", ins)
    base = constants.get(m.group(1) or m.group(2))
    off = re.search(r"offset:(\d+)", ins)
    return None if base is None else base + (int(off.group(1)) if off else 0)


def test_verdict_word_is_not_written_while_waves_may_still_read_it(kernels):
    """The general attention kernel asks first whether the call is its own.  Behind the last barrier of that question
    every wave reads the verdict; until the next barrier no wave may store to the same word, or a late wave takes
    something else for the verdict and leaves (or stays) alone."""
    names = [n for n in kernels if "sparse_attn_kernel" in n]
    assert len(names) >= 9
    for name in names:
        constants, barriers, word = {}, 0, None
        for ins in kernels[name]:
            m = re.match(r"v_mov_b32_e32 v(\d+), (0x[0-9a-f]+|\d+)$", ins)
            if m:
                constants[m.group(1)] = int(m.group(2), 0)
            elif ins.startswith("s_barrier"):
                barriers += 1
                if barriers == 3:
                    break
            elif barriers == 2 and word is None and ins.startswith("ds_read_b32"):
                word = _lds_address(ins, constants)
                assert word is not None, (name, ins)
            elif word is not None and ins.startswith("ds_write_b32"):
                assert _lds_address(ins, constants) != word, (name, ins)
        assert barriers == 3 and word is not None, name


REMARKS = """
remark: Function Name: _ZN5prism22sparse_attn_w64_kernelILi32EEEvPKt
remark:     VGPRs: {v} [-Rpass-analysis=kernel-resource-usage]
remark:     AGPRs: {a}
remark:     ScratchSize [bytes/lane]: {scratch}
remark:     VGPRs Spill: {spill}
remark:     LDS Size [bytes/block]: 65548
"""


@pytest.mark.parametrize("v,a,scratch,spill,good", [
    (156, 100, 0, 0, True), (156, 96, 0, 0, True),
    (152, 100, 0, 0, False),                               # the loop's last VGPRs would be the first AGPRs
    (156, 92, 0, 0, False),
    (158, 97, 0, 0, False),                                # counted as 160 and 97: one workgroup per CU
    (156, 100, 16, 0, False), (156, 100, 0, 3, False),
])
def test_build_refuses_a_kernel_without_the_registers_of_its_row_loop(v, a, scratch, spill, good):
    check_registers = build.check_registers
    text = REMARKS.format(v=v, a=a, scratch=scratch, spill=spill)
    if good:
        check_registers(text, {32: (156, 96)})
    else:
        with pytest.raises(RuntimeError):
            check_registers(text, {32: (156, 96)})
    with pytest.raises(RuntimeError):
        check_registers(text, {64: (256, 256)})            # no such kernel in the report


def test_asm_blocks_list_every_scalar_register_they_write(tmp_path):
    """s40 and up, vcc and M0 in the generated row loops, and whatever the blocks of prism_attn.hip set."""
    subprocess.run([sys.executable, os.path.join(build.CSRC, "gen_attn_w64.py"), str(tmp_path / "x_w64_body.inc")],
                   check=True, capture_output=True)
    blocks = [(tmp_path / n).read_text() for n in ("x_w64_body.inc", "x_w32_body.inc")]
    with open(os.path.join(build.CSRC, "prism_attn.hip")) as f:
        blocks += [b for b in re.findall(r"asm volatile\(.*?\);", f.read(), re.S)]
    seen = 0
    for text in blocks:
        code, clobbers = text, set(re.findall(r'"(\w+)"', text.rsplit(":", 1)[1]))
        written = set()
        for ins in re.findall(r'(?:"|\\n\\t)([a-z]\w+ [^"\\]+)', code):
            m = re.match(r"(s_(?!cmp|cbranch|branch|waitcnt|nop|barrier|endpgm|setprio)\w+|v_cmp\w+|v_readfirstlane_b32)"
                         r" (m0|vcc|exec|s\d+|s\[\d+:\d+\])", ins)
            if m is None or m.group(2) == "exec":          # saved and restored inside the block
                continue
            regs = re.match(r"s\[(\d+):(\d+)\]", m.group(2))
            written |= ({f"s{i}" for i in range(int(regs.group(1)), int(regs.group(2)) + 1)} if regs else {m.group(2)})
        seen += "m0" in written
        assert written <= clobbers, sorted(written - clobbers)
    assert seen >= 2
