"""What the compiler made of the device code built here.  The additions of 16-bit floats are written in asm, about which the
scheduler knows nothing: it may move them between the loads of a step, and the step then takes a trip to memory for each
row instead of one for all.  In every kernel no basic block may load a row behind its first such addition."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2104_05158_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name: [basic block: its loads ('L') and mixed additions ('a') in order]} of the built library."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(build.LIB):
        build.build_library(verbose=False)
    d = tmp_path_factory.mktemp("device_code")
    shutil.copy(build.LIB, d / "libtbe.so")
    subprocess.run([OBJDUMP, "--offloading", "libtbe.so"], cwd=d, check=True, capture_output=True)
    found = {}
    for part in sorted(d.glob("libtbe.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "-C", "--no-show-raw-insn", "--no-leading-addr", "--symbolize-operands", str(part)],
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
