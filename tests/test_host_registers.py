"""What the built kernels need per lane, as the compiler recorded it: kernels whose loops would wait for spilled registers have none."""
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def resources(tmp_path_factory):
    """source -> {kernel's mangled name: (registers, bytes of scratch)}"""
    if shutil.which("hipcc") is None:
        pytest.skip("needs hipcc")
    from paper_2210_15748_amd import build as hip_build
    where = tmp_path_factory.mktemp("resources")

    def of(source):
        obj = hip_build.OBJ / (source + ".o")
        if not obj.exists() or hip_build.stale():
            hip_build.build(force=True)
        subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={where}/fatbin", str(obj), f"{where}/host.o"], check=True)
        subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={where}/fatbin",
                        f"--output={where}/device.co"], check=True)
        notes = subprocess.run([f"{LLVM}/llvm-readobj", "--notes", f"{where}/device.co"], check=True, capture_output=True, text=True).stdout
        out = {}
        for block in notes.split("- .agpr_count")[1:]:
            value = {k: re.search(rf"\.{k}:\s+(\S+)", block).group(1) for k in ("name", "vgpr_count", "private_segment_fixed_size")}
            out[value["name"]] = (int(value["vgpr_count"]), int(value["private_segment_fixed_size"]))
        return out
    return of


def test_comparing_with_every_centroid_spills_nothing(resources):
    kernels = {k: v for k, v in resources("filter_kernels").items() if re.search(r"filter_gemm_kernelILi\dELi4ELi0ELb", k)}
    assert len(kernels) == 6                                   # three widths, all vectors or those of a list
    assert {k: v for k, v in kernels.items() if v[1]} == {}


def test_riders_leave_the_hashing_its_registers(resources):
    """A launch that carries a grouping of candidate lists along keeps as many waves to a CU as the hashing alone."""
    kernels = resources("hash_kernels")
    shape = re.compile(r"hash_mfma_i8_kernelILi(\d)ELi(\d+)ELi2ELb([01])ELi(\d)EE")
    table = {m.groups(): v[0] for k, v in kernels.items() if (m := shape.search(k))}
    assert table
    for (ks, lt, wide, riders), registers in table.items():
        if riders == "1":
            assert registers <= table[ks, lt, wide, "0"], (ks, lt, wide)
