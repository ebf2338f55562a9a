"""What the code objects of the built library say of their kernels: registers and LDS decide how many wavefronts a SIMD holds.

Kernels of whole tiles do not pay for the quarter form, whose registers and rows of dealer words would take wavefronts from
every long launch, those that draw dealer words in step hold what they were measured with, and no kernel keeps anything in scratch
memory."""
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


# Wavefronts per SIMD of the kernels that draw dealer words in step, whole tiles and with quarters (forms 2 and 3): what long
# launches run.  Template arguments before the form; widths and wavefronts.
IN_STEP = [
    ("tile_kernel", (RELU,), 2, ((1, 7, 4), (8, 9, 5), (10, 12, 6), (13, 21, 7), (22, 32, 8))),
    ("tile_kernel", (RELU_SHARED,), 2, ((1, 7, 4), (8, 9, 5), (10, 12, 6), (13, 21, 7), (22, 32, 8))),
    ("tile_kernel", (RELU,), 3, ((4, 7, 4), (8, 12, 5), (13, 16, 7), (17, 21, 5), (22, 32, 7))),
    ("tile_kernel", (RELU_SHARED,), 3, ((4, 7, 4), (8, 12, 5), (13, 16, 7), (17, 21, 5), (22, 32, 7))),
    ("tile_kernel", (DRELU,), 2, ((10, 32, 8),)),
    ("tile_kernel", (DRELU_SHARED,), 2, ((10, 32, 8),)),
    ("tile_kernel", (DRELU,), 3, ((10, 31, 8), (32, 32, 7))),
    ("tile_kernel", (DRELU_SHARED,), 3, ((10, 32, 8),)),
    ("tile_kernel", (SIGN,), 2, ((13, 32, 8),)),
    ("tile_kernel", (SIGN,), 3, ((13, 32, 8),)),
    ("tile_sim_kernel", (), 2, ((1, 2, 4), (3, 3, 6), (4, 4, 4), (5, 5, 6), (6, 9, 7), (10, 32, 8))),
    ("tile_sim_kernel", (), 3, ((4, 4, 4), (5, 7, 5), (8, 8, 8), (9, 12, 5), (13, 16, 7), (17, 21, 5), (22, 32, 6))),
    ("mp_tile_kernel", (3, RELU), 2, ((1, 1, 4), (2, 5, 3), (6, 9, 4), (10, 12, 5), (13, 21, 6), (22, 32, 7))),
    ("mp_tile_kernel", (3, RELU), 3, ((4, 5, 3), (6, 9, 4), (10, 21, 5), (22, 32, 7))),
    ("mp_tile_kernel", (3, DRELU), 2, ((5, 5, 7), (6, 32, 8))),
    ("mp_tile_kernel", (3, DRELU), 3, ((5, 21, 7), (22, 32, 8))),
    ("mp_tile_kernel", (4, RELU), 2, ((1, 4, 4), (5, 7, 3), (8, 12, 4), (13, 21, 5), (22, 32, 6))),
    ("mp_tile_kernel", (4, RELU), 3, ((4, 4, 4), (5, 6, 3), (7, 7, 2), (8, 12, 3), (13, 16, 4), (17, 21, 3), (22, 32, 4))),
    ("mp_tile_kernel", (4, DRELU), 2, ((5, 8, 6), (9, 32, 8))),
    ("mp_tile_kernel", (4, DRELU), 3, ((5, 6, 5), (7, 21, 3), (22, 32, 5))),
]
BATCHED = [("tile_batch_kernel",) + row[1:] for row in IN_STEP if row[0] == "tile_kernel" and row[1] != (SIGN,)]


@pytest.mark.parametrize("kernel,arguments,form,least", IN_STEP + BATCHED)
def test_words_in_step(kernels, kernel, arguments, form, least):
    seen = {a[0] for name, a in kernels if name == kernel and a[1:] == arguments + (form,)}
    assert seen == {w for lo, hi, _ in least for w in range(lo, hi + 1)}
    for lo, hi, wavefronts in least:
        for w in range(lo, hi + 1):
            registers, _ = kernels[kernel, (w,) + arguments + (form,)]
            assert _wavefronts(registers) >= wavefronts, (w, registers)


# The same of one thread per group (w > 32), without words in step and with.
@pytest.mark.parametrize("kernel,arguments,wavefronts", [("group_kernel", (mode,), (8, 7)) for mode in range(5)]
                         + [("wide_sim_kernel", (), (8, 8)), ("mp_group_kernel", (3, DRELU), (8, 8)), ("mp_group_kernel", (3, RELU), (6, 8)),
                            ("mp_group_kernel", (4, DRELU), (5, 6)), ("mp_group_kernel", (4, RELU), (4, 7))])
def test_one_thread_per_group(kernels, kernel, arguments, wavefronts):
    for w in range(33, 65):
        for runs in (0, 1):
            registers, _ = kernels[kernel, (w,) + arguments + (runs,)]
            assert _wavefronts(registers) >= wavefronts[runs], (w, runs, registers)


def test_scratch(kernels):
    assert {k for k, (_, scratch) in kernels.items() if scratch} == set()


# Forms that are slower, or that nothing launches, are not in the library.
@pytest.mark.parametrize("kernel,arguments", [("tile_batch_kernel", (w, SIGN, form)) for w in (13, 32) for form in (2, 3)]
                         + [("mp_tile_kernel", (4, p, DRELU, form)) for p in (3, 4) for form in (2, 3)])
def test_forms_left_out(kernels, kernel, arguments):
    assert (kernel, arguments[:-1] + (arguments[-1] & 1,)) in kernels and (kernel, arguments) not in kernels
