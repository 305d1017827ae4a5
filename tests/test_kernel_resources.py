"""Registers of the built kernels, from the metadata of the library's own code object: kernels whose speed rests on eight waves
per SIMD have at most 64 vector registers and spill none."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1908_06077_amd as nuq

LLVM = "/opt/rocm/llvm/bin"
pytestmark = pytest.mark.skipif(not shutil.which("llvm-readelf", path=LLVM), reason="no LLVM tools")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("code")
    library = os.path.join(os.path.dirname(nuq.__file__), "libnuq.so")
    bundle, code = str(tmp / "bundle"), str(tmp / "code")
    subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + bundle, library, os.devnull], check=True)
    subprocess.run([LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--input=" + bundle, "--output=" + code,
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    found = re.findall(r"\.name: +(\S+)\n(?:(?! *\.name:).*\n)*? *\.vgpr_count: +(\d+)\n *\.vgpr_spill_count: +(\d+)", notes)
    return {name: (int(vgprs), int(spilled)) for name, vgprs, spilled in found}


@pytest.mark.parametrize("pattern,count", [(r"k_finishI", 6), (r"k_encodeILi(16|32|64)ELi\dELi0E", 5)])
def test_eight_waves_per_simd(kernels, pattern, count):
    of = {n: r for n, r in kernels.items() if re.search(pattern, n)}
    assert len(of) == count, sorted(of)
    assert not {n: r for n, r in of.items() if r[0] > 64 or r[1]}
