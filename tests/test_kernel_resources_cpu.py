"""The device code built into libgx.so: no kernel spills registers or keeps
private arrays in memory (read from the metadata of the code objects)."""
import os
import re
import struct
import subprocess

import pytest

import paper_1801_05857_amd as gx

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 code objects of every offload bundle in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24: p + 24 + ln].decode()
            p += 24 + ln
            if "gfx950" in triple and size:
                yield blob[at + off: at + off + size]
        at = blob.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(gx.LIB_PATH):
        from paper_1801_05857_amd import build

        build.build(force=False)
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    tmp = tmp_path_factory.mktemp("co")
    out = {}
    for k, co in enumerate(_code_objects(open(gx.LIB_PATH, "rb").read())):
        path = tmp / f"{k}.co"
        path.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                               check=True).stdout
        for entry in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
            f = dict(re.findall(r"\n\s*\.(\w+):\s+(\S+)", entry))
            out[f["name"]] = f
    return out


def test_every_kernel_family_is_there(kernels):
    for name in ("fop_kernel", "level_kernel", "lds_levels_kernel", "serve_step_kernel",
                 "batch_explore_kernel", "move_kernel"):
        assert any(name in k for k in kernels), name


def test_no_kernel_spills(kernels):
    bad = {k: (f["vgpr_spill_count"], f["private_segment_fixed_size"]) for k, f in kernels.items()
           if int(f["vgpr_spill_count"]) or int(f["private_segment_fixed_size"])}
    assert not bad


def test_find_or_put_of_one_key_fits_eight_wavefronts(kernels):
    """One key in flight, or 4-lane subgroups, and at most 64 vector registers:
    eight wavefronts a SIMD need at most 80 scalar registers as well."""
    seen = 0
    for name, f in kernels.items():
        m = re.search(r"fop_kernelILi\d+ELi\d+ELi\d+ELi1E", name)
        if m and int(f["vgpr_count"]) <= 64:
            seen += 1
            assert int(f["sgpr_count"]) <= 80, name
    assert seen > 60
