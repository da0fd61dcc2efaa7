"""bench.py's map from kernels to the sources whose hash decides whether a recorded
profile is of the present code (no GPU needed)."""
import os
import re

import pytest

import bench

CSRC = os.path.join(bench.HERE, bench.KERNEL_DIR)


def _file(kernel):
    return bench.KERNEL_FILES[max((p for p in bench.KERNEL_FILES if kernel.startswith(p)), key=len)]


def test_every_kernel_maps_to_its_file():
    found = 0
    for f in sorted(os.listdir(CSRC)):
        if not f.endswith(".hip"):
            continue
        text = open(os.path.join(CSRC, f)).read()
        for name in re.findall(r"__global__[^;{]*?void\s+(?:__launch_bounds__\([^{;]*?\)\s+)?(\w+)\(", text):
            found += 1
            assert _file(name) == f, name
    assert found > 30


def test_hash_follows_the_kernels_file(monkeypatch, tmp_path):
    before = {k: bench.kernel_source_hash(k) for k in ("conv3x3_tile<1,2,4,1,4,4,dg>", "conv_gen<2,2,1>", None)}
    for f in os.listdir(CSRC):
        if f.endswith((".hip", ".h")):
            (tmp_path / f).write_bytes(open(os.path.join(CSRC, f), "rb").read())
    monkeypatch.setattr(bench, "KERNEL_DIR", str(tmp_path) + os.sep)
    assert {k: bench.kernel_source_hash(k) for k in before} == before
    with open(tmp_path / "conv_tile.hip", "a") as fh:
        fh.write("//")
    after = {k: bench.kernel_source_hash(k) for k in before}
    assert [after[k] != before[k] for k in before] == [True, False, True]


@pytest.mark.parametrize("full,short", [
    ("void tgpk::(anonymous namespace)::conv3x3_tile<1, 2, 4, 1, 4, 4, true, true, false>(int)",
     "conv3x3_tile<1,2,4,1,4,4,dg,split>"),
    ("void tgpk::(anonymous namespace)::conv3x3_tile<1, 1, 4, 1, 5, 3, false, false, true>(int)",
     "conv3x3_tile<1,1,4,1,5,3,tall>"),
    ("void tgpk::(anonymous namespace)::conv1x1_tile<2, 2, 4, 1, 2, false>(int)", "conv1x1_tile<2,2,4,1>"),
    ("void tgpk::(anonymous namespace)::conv3x3_rows32<192, 2, 3, 3, 1, 1>(int)",
     "conv3x3_rows32<192,2,3,3,8w,rk>"),
])
def test_kernels_are_named_as_their_launchers_name_them(full, short):
    assert bench.short_kernel_name(full) == short
