"""What the built kernels use, from the notes of libhive.so's gfx950 code object
(no GPU needed).  A kernel that keeps its registers' arrays in scratch memory
still gives the right results, only slower, so nothing else shows it."""
import os
import re
import struct
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_15095_amd", "libhive.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(data: bytes):
    """gfx950 code objects of the offload bundles in a host library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + n].decode()
            p += 24 + n
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Bytes of scratch memory per lane, by kernel symbol."""
    if not os.path.exists(LIB) or not os.path.exists(READELF):
        pytest.skip("no built library, or no llvm-readelf")
    got = {}
    for i, obj in enumerate(code_objects(open(LIB, "rb").read())):
        f = tmp_path_factory.mktemp("co") / f"{i}.elf"
        f.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\S+)\s+\.private_segment_fixed_size:\s+(\d+)", notes):
            got[name] = int(size)
    return got


@pytest.mark.parametrize("kernel", ["evict_lanes_kernel", "evict_kernel", "set_evict_kernel", "ops_kernel",
                                    "set_ops_kernel", "small_batch_kernel", "ddr_", "dds_kernel", "resize_kernel",
                                    "merge_kernel"])
def test_launched_kernels_use_no_scratch(scratch, kernel):
    mine = {k: v for k, v in scratch.items() if kernel in k}
    assert mine, f"no kernel named {kernel} among {len(scratch)}"
    assert not any(mine.values()), {k: v for k, v in mine.items() if v}


@pytest.mark.parametrize("mode", [0, 1, 2, 3])  # insert, delete, lookup, mixed
@pytest.mark.parametrize("waves,loads", [(4, 16), (8, 4)])
def test_probe_variants_of_filter_tables_are_built(scratch, mode, waves, loads):
    """Variant 0 (4 waves per SIMD, 16 loads) can be asked for on tables with a
    spill filter, for every kind of batch, beside the library's own choice."""
    assert any(f"10ops_kernelILi16ELj{mode}ELb0ELi0ELi{waves}ELi{loads}ELi1EE" in k for k in scratch)


def test_tuner_measures_every_variant_by_name():
    """The tuner's candidates are the library's choice and each variant by its
    own number, 4 waves and 16 loads among them."""
    from paper_2510_15095_amd import autotune
    from paper_2510_15095_amd import hive as H
    got = autotune.probe_candidates()
    assert got == [0, 1, 2, 3, 4, H.PROBE_4X16] and H.PROBE_VARIANTS[0] == ("library",)
    assert len(H.PROBE_VARIANTS) == 5
