"""What the compiler reports of the built kernels, where a launch rule counts on it.  Read from the build's objects."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_19157_amd import build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """demangled name without its arguments -> (vector registers with the accumulators, bytes of scratch per lane)"""
    tools = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")] + [shutil.which("c++filt")]
    objs = [os.path.join(build.HERE, "_build", os.path.basename(src) + ".o") for src in build.sources()]
    if not all(t and os.path.exists(t) for t in tools + objs):
        pytest.skip("needs the objects of a build and the tools of ROCm's llvm")
    objcopy, bundler, readelf, cxxfilt = tools
    d = tmp_path_factory.mktemp("co")
    got = {}
    for obj in objs:
        fat, co = str(d / "fat"), str(d / "co")
        subprocess.run([objcopy, f"--dump-section=.hip_fatbin={fat}", obj, os.devnull], check=True)
        subprocess.run([bundler, "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}",
                        f"--output={co}"], check=True)
        notes = subprocess.run([readelf, "--notes", co], check=True, capture_output=True, text=True).stdout
        for k in re.split(r"\n  - ", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", k)
            if name and ".vgpr_count" in k:
                f = {n: int(re.search(rf"\.{n}:\s+(\d+)", k).group(1)) for n in ("vgpr_count", "private_segment_fixed_size")}
                got[name.group(1)] = (f["vgpr_count"], f["private_segment_fixed_size"])
    names = subprocess.run([cxxfilt], input="\n".join(got), check=True, capture_output=True, text=True).stdout.split("\n")
    return {re.sub(r"\(.*|void saw::", "", n): v for n, v in zip(names, got.values())}


def test_pair_blocks_of_the_16_bit_kernel_fit_twice_on_a_simd(kernels):
    """The pair rule takes up to 2048 items as resident at once: eight wavefronts on a compute unit, two on a SIMD, 256 registers
    each."""
    pair = {n: v for n, v in kernels.items() if n.startswith("decode_kv16_mfma_kernel<") and ", true, false>" in n}
    assert len(pair) == 16
    assert {n: v for n, v in pair.items() if v[0] > 256 or v[1]} == {}
