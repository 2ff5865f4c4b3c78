"""No kernel of the library needs scratch memory: one that does pays for it at every launch when several
streams are in use.  Read from the metadata of the objects that the build leaves next to the package.
CPU only."""
import glob
import os
import re
import subprocess

import pytest

import paper_2510_00636_amd as ea

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-readelf")), reason="no ROCm toolchain")
def test_no_kernel_needs_scratch_memory(tmp_path):
    pattern = os.path.join(os.path.dirname(os.path.abspath(ea.__file__)), "_build", "*.hip.o")
    if not glob.glob(pattern):
        import __graft_entry__
        __graft_entry__.build()
    kernels = {}
    for obj in sorted(glob.glob(pattern)):
        fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
        subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, obj, os.devnull],
                       check=True, timeout=60)
        subprocess.run([os.path.join(LLVM, "clang-offload-bundler"), "--type=o", "--unbundle", "--input=" + fat,
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--output=" + code], check=True, timeout=60)
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", code], check=True, timeout=60,
                               capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            kernels[name] = int(size)
    assert len(kernels) > 50
    assert not {k: v for k, v in kernels.items() if v}
