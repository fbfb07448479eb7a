"""The compiled kernels' buffer accesses (CPU): every one carries its whole offset
in the vector offset and the instruction's constant.

The range check that drops the stores of a ragged last tile covers these two; the
scalar offset of the raw buffer builtins is excluded from it, so an access that
moves along the tile by its scalar offset would rely on a check it is not promised.
"""
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"
TOOLS = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")]


def test_scalar_offsets_are_zero(tmp_path):
    if not all(os.path.exists(t) for t in TOOLS):
        pytest.skip("no LLVM tools")
    from paper_2605_15547_amd import build, crmath
    if not os.path.exists(crmath.LIB_PATH):
        build.build()
    fat, dev = str(tmp_path / "fat.bin"), str(tmp_path / "dev.co")
    subprocess.check_call([TOOLS[0], "--dump-section", ".hip_fatbin=" + fat, crmath.LIB_PATH,
                           os.devnull])
    subprocess.check_call([TOOLS[1], "--type=o", "--unbundle", "--input=" + fat, "--output=" + dev,
                           "--targets=hipv4-amdgcn-amd-amdhsa--" + build.ARCH])
    text = subprocess.run([TOOLS[2], "-d", "--no-show-raw-insn", dev], capture_output=True, text=True,
                          check=True).stdout
    # data, vector offset, descriptor, scalar offset, modifiers
    scalar = re.findall(r"\bbuffer_(?:load|store)\w*\s+\S+,\s*\S+,\s*s\[\d+:\d+\],\s*(\S+)", text)
    assert len(scalar) > 1000
    assert set(scalar) == {"0"}
