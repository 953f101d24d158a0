"""The kernels' register bounds ask for as many wavefronts per SIMD as do without a spill: no kernel of the built library keeps vector registers
in scratch memory, in either format.  Read from the notes that the compiler wrote into the library's code objects."""
import os
import re
import subprocess

import pytest

import paper_2508_00806_amd as adacc

LLVM = "/opt/rocm/llvm/bin/"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """{kernel: vector registers spilled} of the library"""
    if not os.path.exists(adacc.LIB_PATH) or not os.path.exists(LLVM + "llvm-objcopy"):
        pytest.skip("needs the built library and the compiler's tools")
    d = tmp_path_factory.mktemp("notes")
    whole = d / "bundles"
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", f".hip_fatbin={whole}", adacc.LIB_PATH, os.devnull], check=True)
    data = whole.read_bytes()
    starts = [m.start() for m in re.finditer(BUNDLE, data)] + [len(data)]
    found = {}
    for i, (a, b) in enumerate(zip(starts, starts[1:])):
        part, code = d / f"{i}.bundle", d / f"{i}.co"
        part.write_bytes(data[a:b])
        subprocess.run([LLVM + "clang-offload-bundler", "--type=o", "--unbundle", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                        f"--input={part}", f"--output={code}"], check=True)
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(code)], check=True, capture_output=True, text=True).stdout
        for kernel in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            found[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    return found


@pytest.mark.parametrize("kernels", ["compress_long_kernel", "compress_kernel", "compress_batch_kernel"])
def test_no_vector_register_is_spilled(spills, kernels):
    ours = {n: s for n, s in spills.items() if re.search(r"\d" + kernels + "I", n)}
    assert any("bf16" in n for n in ours) and any("3f16" in n for n in ours)
    assert {n: s for n, s in ours.items() if s} == {}


# those that bound their registers for reasons of their own: short tensors (four wavefronts a SIMD), the placement (four; sixteen to a workgroup)
@pytest.mark.parametrize("kernels", ["compress_short_kernelI", "place_kernelE", "place_many_kernelE", "place_batch_kernelE", "decompress_kernelI"])
def test_no_vector_register_is_spilled_either(spills, kernels):
    ours = {n: s for n, s in spills.items() if re.search(r"\d" + kernels, n)}
    assert any("bf16" in n for n in ours) and any("3f16" in n for n in ours)
    assert {n: s for n, s in ours.items() if s} == {}
