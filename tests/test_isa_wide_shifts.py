"""The device code of the built library has no 64-bit vector shift whose amount is in a vector register (hb_protocol.hpp,
word_at): with the amount in the last register of a wavefront's allocation such shifts have given wrong shares now and then,
and where the amount lands is the register allocator's choice."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2309_04875_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WIDE_SHIFT = re.compile(r"\bv_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\S*\s+v\[\d+:\d+\], v\d")


def _matches(code_object):
    """Kernel symbol -> number of such shifts."""
    proc = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", code_object], stdout=subprocess.PIPE, text=True)
    found, symbol, shifts = {}, None, 0
    for line in proc.stdout:
        if line.endswith(">:\n"):
            symbol = line.strip()
        elif "rev_" in line and "64" in line:
            shifts += "v_lshlrev_b64" in line or "v_lshrrev_b64" in line
            if WIDE_SHIFT.search(line):
                found[symbol] = found.get(symbol, 0) + 1
    assert proc.wait() == 0
    return found, shifts


def test_pattern():
    assert WIDE_SHIFT.search("\tv_lshrrev_b64 v[2:3], v63, v[4:5]")
    assert WIDE_SHIFT.search("\tv_ashrrev_i64 v[2:3], v1, 3")
    assert not WIDE_SHIFT.search("\tv_lshrrev_b64 v[2:3], s4, v[4:5]")
    assert not WIDE_SHIFT.search("\tv_lshlrev_b64 v[2:3], 9, v[4:5]")


def test_no_64_bit_shift_by_a_vector_register(tmp_path):
    if not os.path.exists(OBJDUMP) or not os.path.exists(build.LIBRARY):
        pytest.skip("needs the ROCm toolchain and a built library")
    library = shutil.copy(build.LIBRARY, tmp_path)                     # the code objects are unpacked beside it
    subprocess.run([OBJDUMP, "--offloading", library], check=True, stdout=subprocess.DEVNULL)
    objects = sorted(str(p) for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    assert len(objects) > 30
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        results = list(pool.map(_matches, objects))
    assert sum(shifts for _, shifts in results) > 10000                # the kernels were found: SplitMix64 is full of them
    found = {symbol: count for per_object, _ in results for symbol, count in per_object.items()}
    assert not found, "%d shifts in %d kernels, first %s" % (sum(found.values()), len(found), sorted(found.items())[:3])
