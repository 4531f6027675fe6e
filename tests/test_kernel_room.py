"""A resident executor leaves one block's room per compute unit free for the
process's other kernels.  A kernel whose blocks need more than that waits until
the executor stops, and a program that waits for it first never goes on; the
registers and the shared memory of the built kernels say which (no GPU needed).
"""
import os
import re
import subprocess

import pytest

from test_kernel_resources import LIB, READELF, code_objects

WAVES, VGPRS = 8, 512  # per SIMD of a compute unit
LDS = 80 * 1024  # a block of more waits beside another one, whatever is free of the 160 KiB


def _up(x, to):
    return -(-x // to) * to


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(threads, registers, shared bytes), by kernel symbol."""
    if not os.path.exists(LIB) or not os.path.exists(READELF):
        pytest.skip("no built library, or no llvm-readelf")
    got = {}
    for i, obj in enumerate(code_objects(open(LIB, "rb").read())):
        f = tmp_path_factory.mktemp("co") / f"{i}.elf"
        f.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("  - .agpr_count:")[1:]:
            def num(key):
                return int(re.search(rf"\.{key}:\s+(\d+)", entry)[1])
            got[re.search(r"\.name:\s+(_Z\S+)", entry)[1]] = (num("max_flat_workgroup_size"), num("vgpr_count"),
                                                              num("group_segment_fixed_size"))
    return got


def _fits(kernel, worker, blocks):
    """One block of `kernel` on a compute unit with `blocks` of `worker`."""
    (t, v, lds), (wt, wv, _) = kernel, worker
    per, wper = _up(t, 256) // 256, _up(wt, 256) // 256  # waves per SIMD
    return (per * _up(v, 8) + blocks * wper * _up(wv, 8) <= VGPRS and per + blocks * wper <= WAVES and
            lds <= LDS)


@pytest.mark.parametrize("S", [16, 32, 64])
@pytest.mark.parametrize("blocks", [1, 2])  # asked for; and the default, one less than fit
def test_other_kernels_fit_beside_a_resident_executor(kernels, S, blocks):
    (worker,) = [v for k, v in kernels.items() if f"drain_worker_kernelILi{S}E" in k]
    assert _fits(worker, worker, 2) and not _fits(worker, worker, 3), "three blocks fit, two are the default"
    bad = [k for k, v in kernels.items()
           if "drain_worker" not in k and not _fits(v, worker, blocks)]
    assert len(kernels) > 100 and not bad, {k: kernels[k] for k in bad}
