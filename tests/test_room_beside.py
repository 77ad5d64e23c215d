"""What runs beside the expert GEMMs fits beside them.  A block of theirs on tiles of 256 columns holds a compute unit
for a share of the launch's tiles, so another kernel's wavefront gets in meanwhile only if each SIMD's 512 registers (allocated by
eight) hold both and it asks for no LDS.  Read from the library as built (no GPU needed)."""
import re
import shutil
import subprocess

import pytest

import paper_2210_17223_amd as moe

OBJDUMP, READELF = "/opt/rocm/llvm/bin/llvm-objdump", "/opt/rocm/llvm/bin/llvm-readelf"
REGISTERS = 512


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: (registers as allocated, bytes of static LDS)}"""
    moe.lib()                                       # (built if it is not there)
    if shutil.which(OBJDUMP) is None or shutil.which(READELF) is None:
        pytest.skip("no llvm tools")
    where = tmp_path_factory.mktemp("code")
    shutil.copy(moe.lib_path(), where / "libmoe.so")
    subprocess.run([OBJDUMP, "--offloading", "libmoe.so"], cwd=where, check=True, capture_output=True)
    out = {}
    for f in sorted(where.glob("*gfx950")):
        notes = subprocess.run([READELF, "--notes", str(f)], check=True, capture_output=True, text=True).stdout
        for entry in re.split(r"\n  - (?=\.)", notes)[1:]:
            field = lambda key: re.search(rf"\.{key}: +(\S+)", entry)[1]
            out[field("symbol")] = (-(-int(field("vgpr_count")) // 8) * 8, int(field("group_segment_fixed_size")))
    return out


@pytest.mark.parametrize("guest,hosts,least", [
    # the pack, beside every forward GEMM, pre-activations kept or not
    ("scatter_rows_kernel", r"grouped_gemm_(w4|mfma)_kernelILb0E", 16),
    # the stand-in link's copy, beside the padded layer's GEMMs (which keep nothing)
    ("link_copy_kernel", r"grouped_gemm_(w4|mfma)_kernelILb[01]ELi\dELb0E", 16),
])
def test_a_wavefront_fits_beside_the_expert_gemms(kernels, guest, hosts, least):
    guests = [v for n, v in kernels.items() if guest in n]
    beside = {n: v[0] for n, v in kernels.items() if re.search(hosts, n)}
    assert guests and len(beside) >= least
    for registers, lds in guests:
        assert lds == 0
        over = {n: r for n, r in beside.items() if r + registers > REGISTERS}
        assert not over, (registers, over)
