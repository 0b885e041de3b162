"""Sizes and layouts that the host code decides, against what the device code
does with them (no GPU): host_layout.hip, linked to libpanda.so, prints them."""
import os
import subprocess

import pytest

from paper_1507_07039_amd import panda

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1507_07039_amd")


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    """layout(mode): the lines host_layout prints, as lists of integers."""
    if not os.path.exists(panda.LIB_PATH):
        pytest.fail("libpanda.so is not built (run __graft_entry__.build())")
    exe = str(tmp_path_factory.mktemp("host_layout") / "host_layout")
    r = subprocess.run(
        ["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
         "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
         os.path.join(ROOT, "tests", "host_layout.hip"), "-o", exe, "-L", PKG, "-lpanda",
         "-Wl,-rpath," + PKG], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def lines(mode):
        r = subprocess.run([exe, mode], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        return [[int(x) for x in line.split()] for line in r.stdout.splitlines()]
    return lines


def test_folding_scratch_wherever_the_product_folds(layout):
    """The three-plane product on packed C sums a range of k in one run up to
    some length and folds longer ones through memory; the host must have given
    it that memory for every k at which it does."""
    for k, run, scratch in layout("fold"):
        assert 0 < run <= k
        assert run == k or scratch > 0, (k, run, scratch)


def test_loads_clear_only_the_h_partials(layout):
    """A load clears every h partial of its network, and no more than the room
    carved for them (in a batch that is the grouped kernels' count, not the
    single network's)."""
    lines = layout("hpart")
    assert {(prec, batched) for _, _, prec, batched, _, _ in lines} == {(0, 0), (0, 1), (1, 0), (1, 1)}
    for line in lines:
        cleared, room = line[4:]
        assert 0 < cleared <= room, line
