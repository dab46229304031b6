"""Registers of the compiled kernels whose speed rests on several waves per
SIMD, read from the metadata of the built library (no GPU needed)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2607_26566_amd.build import LIB

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """symbol -> {vgpr_count, vgpr_spill_count} of every gfx950 kernel."""
    d = tmp_path_factory.mktemp("code")
    fat = str(d / "fatbin")
    subprocess.run(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", LIB, fat], check=True)
    data, out = open(fat, "rb").read(), {}
    for at in (m.start() for m in re.finditer(re.escape(MAGIC), data)):
        entry = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, entry - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + n]:
                co = str(d / "object")
                with open(co, "wb") as f:
                    f.write(data[at + off:at + off + size])
                notes = subprocess.run([READELF, "--notes", co], check=True, capture_output=True,
                                       text=True).stdout
                for block in re.split(r"\n  - ", notes):
                    sym = re.search(r"\.symbol:\s+(\S+)\.kd", block)
                    if sym:
                        out[sym[1]] = {k: int(re.search(rf"\.{k}:\s+(\d+)", block)[1])
                                       for k in ("vgpr_count", "vgpr_spill_count",
                                                 "private_segment_fixed_size")}
            entry += 24 + n
    assert os.path.getsize(fat) and out
    return out


def find(kernels, name):
    got = {k: v for k, v in kernels.items() if name in k}
    assert got, name
    return got


# the conditioning table streams every adaLN weight: it needs 5 waves per SIMD
# (512 registers, allotted in eights) in flight, as much as 8 rows x 4 columns allow
def test_conditioning_rows_keep_five_waves_per_simd(kernels):
    for k, v in {**find(kernels, "linear_rows_group_kernel"), **find(kernels, "linear_rows_kernel")}.items():
        assert (v["vgpr_count"] + 7) // 8 * 8 * 5 <= 512, (k, v)
        assert v["vgpr_spill_count"] == 0, (k, v)


def test_cache_signal_does_not_spill(kernels):
    for k, v in find(kernels, "cache_signal_kernel").items():
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (k, v)
