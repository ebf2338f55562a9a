"""What the code objects of the built library say of their kernels: registers and LDS decide how many wavefronts a SIMD holds.

Kernels of whole tiles do not pay for the quarter form, whose registers and rows of dealer words would take wavefronts from
every long launch, and no kernel keeps anything in scratch memory except the one that is known to."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2309_04875_amd import build

LLVM = "/opt/rocm/llvm/bin/"
DRELU, RELU, SIGN, DRELU_SHARED, RELU_SHARED = range(5)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(name, template arguments) -> (vector registers, bytes of scratch per lane)."""
    if not os.path.exists(LLVM + "llvm-readobj") or not os.path.exists(build.LIBRARY):
        pytest.skip("needs the ROCm toolchain and a built library")
    where = tmp_path_factory.mktemp("code")
    library = shutil.copy(build.LIBRARY, where)
    subprocess.run([LLVM + "llvm-objdump", "--offloading", library], check=True, stdout=subprocess.DEVNULL)
    out = {}
    for path in where.iterdir():
        if not path.name.endswith("gfx950"):
            continue
        notes = subprocess.run([LLVM + "llvm-readobj", "--notes", str(path)], check=True, stdout=subprocess.PIPE, text=True).stdout
        for block in notes.split("- .agpr_count:")[1:]:
            def field(key):
                return re.search(r"\.%s:\s+(\S+)" % key, block).group(1)
            name = re.match(r"_ZN2hb\d+([a-z_0-9]+kernel)(?:I((?:L[ib]\d+E)+)E)?", field("name"))
            if name:
                args = tuple(int(a) for a in re.findall(r"L[ib](\d+)E", name.group(2) or ""))
                out[name.group(1), args] = (int(field("vgpr_count")), int(field("private_segment_fixed_size")))
    assert len(out) > 500
    return out


def _wavefronts(registers):
    return min(8, 512 // (-(-registers // 8) * 8))


# Wavefronts per SIMD of the whole-tile kernels before they shared a kernel with the quarter form.
TWO_PARTIES = [((22, 32), (DRELU, RELU, SIGN, DRELU_SHARED, RELU_SHARED), 8), ((17, 21), (RELU, RELU_SHARED), 7),
               ((13, 16), (RELU, RELU_SHARED), 7), ((9, 10), (RELU, RELU_SHARED), 5), ((4, 4), (RELU, RELU_SHARED), 4),
               ((4, 21), (DRELU,), 7), ((12, 21), (DRELU, SIGN, DRELU_SHARED), 8)]


@pytest.mark.parametrize("widths,modes,wavefronts", TWO_PARTIES)
@pytest.mark.parametrize("kernel", ["tile_kernel", "tile_batch_kernel"])
def test_whole_tiles_of_two_parties(kernels, kernel, widths, modes, wavefronts):
    for w in range(widths[0], widths[1] + 1):
        for mode in modes:
            registers, _ = kernels[kernel, (w, mode, 0)]
            assert _wavefronts(registers) >= wavefronts, (w, mode, registers)


@pytest.mark.parametrize("parties,w,mode,wavefronts", [(3, 4, DRELU, 6), (3, 5, DRELU, 6), (4, 4, DRELU, 5), (4, 5, DRELU, 5)]
                         + [(4, w, DRELU, 5) for w in (11, 12, 17, 18, 19, 20, 21)])
def test_whole_tiles_of_more_parties(kernels, parties, w, mode, wavefronts):
    registers, _ = kernels["mp_tile_kernel", (w, parties, mode, 0)]
    assert _wavefronts(registers) >= wavefronts, registers


def test_scratch(kernels):
    # Four-party ReLU at w = 4 keeps its shares there (its loop over eight pairs is not unrolled).
    known = {("mp_tile_kernel", (4, 4, RELU, 0)), ("mp_tile_kernel", (4, 4, RELU, 1))}
    assert {k for k, (_, scratch) in kernels.items() if scratch} <= known


# Forms that are slower, or that nothing launches, are not in the library.
@pytest.mark.parametrize("kernel,arguments", [("mp_tile_kernel", (1, 4, RELU, 2))] + [("tile_batch_kernel", (w, SIGN, form)) for w in (13, 32) for form in (2, 3)])
def test_forms_left_out(kernels, kernel, arguments):
    assert (kernel, arguments[:-1] + (arguments[-1] & 1,)) in kernels and (kernel, arguments) not in kernels
