"""What the compiler made of the device code built here.

The additions of 16-bit floats are written in asm, about which the
scheduler knows nothing: it may move them between the loads of a step, and the step then takes a trip to memory for each
row instead of one for all.  In every kernel no basic block may load a row behind its first such addition.

The update kernel that sums long runs itself keeps more rows in flight where a row takes the whole wavefront: every table of
a call pays for the registers, in wavefronts, unless they are those that the kernel has without it.  Its wavefronts count their pieces when
the stores of their sums have arrived, which only an instruction between them says."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2104_05158_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    """The code objects of the built library."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(build.LIB):
        build.build_library(verbose=False)
    d = tmp_path_factory.mktemp("device_code")
    shutil.copy(build.LIB, d / "libtbe.so")
    subprocess.run([OBJDUMP, "--offloading", "libtbe.so"], cwd=d, check=True, capture_output=True)
    return [str(p) for p in sorted(d.glob("libtbe.so.*gfx950"))]


@pytest.fixture(scope="module")
def kernels(parts):
    """{demangled name: [basic block: its loads ('L') and mixed additions ('a'), stores of 8 bytes past the L2s ('S'), counts ('C')
    and waits for all of memory ('W') in order]}"""
    found = {}
    for part in parts:
        text = subprocess.run([OBJDUMP, "-d", "-C", "--no-show-raw-insn", "--no-leading-addr", "--symbolize-operands", part],
                              check=True, capture_output=True, text=True).stdout
        blocks = None
        for line in text.splitlines():
            head = re.match(r"<(.*)>:$", line)
            if head:
                if not re.match(r"L\d+$", head[1]):
                    blocks = found.setdefault(head[1], [])
                blocks.append("")
            elif blocks is not None and re.match(r"\s*(global|buffer)_load", line):
                blocks[-1] += "L"
            elif blocks is not None and re.match(r"\s*global_store_dwordx2.* sc1", line):
                blocks[-1] += "S"
            elif blocks is not None and "s_waitcnt vmcnt(0)" in line:
                blocks[-1] += "W"
            elif blocks is not None and re.match(r"\s*global_atomic_add v.* sc0", line):
                blocks[-1] += "C"
            elif blocks is not None and "v_fma_mix_f32" in line:
                blocks[-1] += "a"
            elif blocks is not None and re.match(r"\s*s_(cbranch|branch)", line):
                blocks.append("")
    return found


def test_rows_of_a_step_are_requested_before_the_first_is_added(kernels):
    mixed = {k: b for k, b in kernels.items() if any("a" in x for x in b)}
    for name in ("forward_kernel", "forward_bag_kernel", "reduce_update_kernel", "window_runs_kernel", "long_run_fixup_kernel"):
        assert any(name in k for k in mixed), name
    late = [k for k, blocks in mixed.items() if any(re.search("a.*L", b) for b in blocks)]
    assert not late, late


def test_update_that_sums_long_runs_keeps_its_wavefronts(parts):
    registers = {}
    for part in parts:
        text = subprocess.run([OBJDUMP.replace("objdump", "readelf"), "--notes", part], check=True, capture_output=True, text=True).stdout
        for kernel in text.split(".agpr_count:")[1:]:
            value = lambda key: int(re.search(key + r":\s+(\d+)", kernel)[1])
            registers[re.search(r"\.symbol:\s+'?([\w.]+)\.kd", kernel)[1]] = value(r"\.vgpr_count"), value(r"\.private_segment_fixed_size")
    names = subprocess.run(["c++filt"], input="\n".join(registers), capture_output=True, text=True, check=True).stdout.split("\n")
    seen = 0
    for (vgprs, scratch), name in zip(registers.values(), names):
        row = re.search(r"reduce_update_kernel<(.*), (.*), 0, 16, [2-9]>", name)     # row-wise AdaGrad; 0 and 1 leave long runs to others
        if row:
            # 512 registers a lane in steps of eight: five wavefronts a SIMD with rows of fp32, six with 16-bit ones
            assert scratch == 0 and vgprs <= (96 if row[2] == "float" else 80), (name, vgprs, scratch)
            seen += 1
    assert seen == 6, seen


def test_a_piece_is_counted_after_its_stores_have_arrived(kernels):
    counting = [k for k in kernels if re.search(r"reduce_update_kernel<.*, .*, [012], 16, 2>", k)]
    assert len(counting) == 18
    for k in counting:
        order = "".join(kernels[k])
        assert re.search("S[^SWC]*W[^SWC]*C", order) and not re.search("S[^W]*C", order), k
