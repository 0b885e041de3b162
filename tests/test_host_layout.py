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

    def lines(mode, *args):
        r = subprocess.run([exe, mode] + [str(a) for a in args], capture_output=True, text=True, timeout=60)
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


# us an iteration measured in the small and in the grouped kernels, FP32 and
# split form, where they differ by more than an eighth
@pytest.mark.parametrize("n,Ne,Na,small,fp32,split", [
    (20, 125, 125, 37, 150, 139), (400, 125, 125, 311, 416, 471), (16, 250, 250, 81, 212, 171),
    (8, 354, 354, 104, 239, 173), (100, 354, 354, 927, 667, 730), (2, 500, 500, 64, 240, 172),
    (8, 500, 500, 171, 291, 200), (32, 500, 500, 609, 419, 443), (100, 500, 500, 1953, 1153, 1293),
    (2, 700, 700, 119, 303, 194), (16, 700, 700, 737, 557, 503), (16, 40, 400, 57, 172, 128),
    (200, 40, 400, 478, 367, 365), (400, 40, 400, 974, 628, 656), (2, 100, 2000, 133, 285, 184),
    (8, 100, 2000, 469, 376, 239), (32, 100, 2000, 1890, 616, 629), (8, 30, 1000, 94, 200, 155),
    (64, 30, 1000, 635, 334, 332), (64, 64, 1024, 823, 374, 362), (300, 65, 130, 234, 339, 368),
    (8, 2000, 100, 409, 663, 680), (4, 1000, 300, 148, 322, 233)])
def test_batches_take_the_faster_kernels(layout, n, Ne, Na, small, fp32, split):
    for precision, grouped in ((0, fp32), (1, split)):
        assert layout("batch", n, Ne, Na, precision) == [[int(small < grouped)]], (precision, grouped)


# the same for one network, the tiled kernels of either form beside the small
# ones; a choice within 3 % of the better is not told apart
@pytest.mark.parametrize("Ne,Na,small,fp32,split", [
    (40, 400, 25, 72, 77), (500, 500, 39, 93, 102), (750, 750, 82, 112, 97), (500, 1000, 66, 100, 88),
    (500, 1100, 89, 102, 88), (300, 1500, 81, 97, 84), (256, 1600, 85, 95, 84), (288, 1600, 87, 98, 86),
    (128, 1700, 64, 91, 80), (129, 1700, 82, 94, 81), (256, 1700, 91, 97, 82), (224, 1800, 92, 95, 85),
    (128, 1900, 71, 91, 82), (129, 1900, 92, 93, 83), (128, 2048, 75, 92, 79), (129, 2000, 94, 93, 83),
    (192, 2048, 97, 93, 81), (64, 2048, 73, 87, 79), (1200, 420, 97, 138, 137), (2000, 150, 98, 211, 166),
    (2048, 190, 101, 233, 195), (2000, 40, 75, 189, 157)])
def test_networks_take_the_faster_kernels(layout, Ne, Na, small, fp32, split):
    for precision, tiled in ((0, fp32), (1, split)):
        took = small if layout("run", Ne, Na, precision) == [[1]] else tiled
        assert took <= 1.03 * min(small, tiled), precision


@pytest.mark.parametrize("n", [1, 4000, 65536, 65537, 300000])
def test_partial_gradients_sum_few_edges(n):
    """The warm start's partial gradients (FP32 sums over the edges of a wave,
    added in FP64) number up to 2048, so that each sums no more edges than that
    many share; the workspace has a slot of 5313 floats for each."""
    chunks = -(-n // 32)
    slots = min(-(-chunks // 4), 512) * 4
    assert panda.load_library().panda_mlp_grad_workspace_bytes(n) >= slots * panda.MLP_PARAMS * 4


@pytest.mark.parametrize("Ne,Na", [(40, 400), (3, 11), (500, 500), (200, 4000), (700, 18000)])
def test_features_need_little_scratch(layout, Ne, Na):
    """The features' workspace: one padded N_e x N_a matrix, the vectors, and for
    networks past the small kernels (whose contexts are far larger) 64 MiB of
    split tiles."""
    up = lambda n, m: -(-n // m) * m  # noqa: E731
    need = up(Ne, 64) * up(Na, 128) * 4 + 8 * 40 * (Ne + Na) + (1 << 18)
    if not layout("small", Ne, Na)[0][0]:
        need += 64 << 20
    assert 0 < panda.load_library().panda_ws_features_workspace_bytes(Ne, Na) <= need
