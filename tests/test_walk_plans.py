"""The tile shapes of the column-walk kernels, as walkplan.h chooses them from a problem's size: that
header is plain C++, compiled here with the host's compiler. Kinds: f32 the 32-channel block forward,
b32 / b16 the block backward by walks, t16 the 16-channel one in the form that its launch takes (R = 0: tile
by tile), c64 the 64-channel conv backward."""
from __future__ import annotations

import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CUS = 256
KINDS = {"f32": (7, 80), "b32": (7, 160), "b16": (8, 160), "t16": (8, 160), "c64": (7, 160)}   # most rows per walk, KB of LDS


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = os.environ.get("CXX") or shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    so = str(tmp_path_factory.mktemp("walkplan") / "walkplan.so")
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "walkplan_driver.cpp")], check=True)
    lib = C.CDLL(so)
    fn = lib.walk_plan
    fn.argtypes = [C.c_char_p, C.c_int64, C.c_int, C.c_int, C.c_int, C.POINTER(C.c_int64)]

    def choose(kind, n, H, W):
        out = (C.c_int64 * 6)()
        if not fn(kind.encode(), n, H, W, CUS, out):
            return None
        return dict(zip(("F", "TH", "bands", "tiles", "R", "lds"), out))

    choose.pend_helpers = lib.walk_pend_helpers
    return choose


@pytest.mark.parametrize("kind", KINDS)
def test_a_shape_covers_the_frames_and_fits(plan, kind):
    """Bands cover a frame, several of them hold one frame each, walks are no longer than a band, and
    the windows fit; every width that a network's stage can have is taken."""
    rng = random.Random(3)
    max_rows, kb = KINDS[kind]
    for _ in range(1500):
        n, H, W = round(8192 ** rng.random()), rng.randint(1, 64), rng.randint(1, 64)
        p = plan(kind, n, H, W)
        assert p is not None, (n, H, W)
        assert p["bands"] * p["TH"] >= H and (p["bands"] - 1) * p["TH"] < H, (n, H, W, p)
        assert 1 <= p["F"] <= max(1, n) and (p["F"] == 1 or p["bands"] == 1), (n, H, W, p)
        assert p["tiles"] == -(-n // p["F"]) * p["bands"], (n, H, W, p)
        assert (kind == "t16" and p["R"] == 0 and p["F"] == 1) or 1 <= p["R"] <= min(p["TH"], max_rows), (n, H, W, p)
        assert 0 < p["lds"] <= kb * 1024, (n, H, W, p)


@pytest.mark.parametrize("n,H,W,rows", [(2048, 21, 21, 5), (8192, 21, 21, 5), (640, 21, 21, 2), (2048, 11, 11, 2),
                                        (8192, 42, 42, 2), (2048, 30, 45, 2), (128, 21, 21, 2)])
def test_the_block_forward_walks_several_rows(plan, n, H, W, rows):
    """A walk of one row reuses no input fragment: wherever the launch has rows to walk, R is above 1
    (2048 frames of 21x21: 38 us at R = 7, 47 at R = 1)."""
    assert plan("f32", n, H, W)["R"] >= rows


@pytest.mark.parametrize("n,H,W,most", [(40, 11, 11, 80), (56, 10, 10, 112), (8, 24, 24, 64), (8, 21, 21, 64), (5, 11, 11, 32)])
def test_few_frames_leave_few_partials(plan, n, H, W, most):
    """Each workgroup of the 64-channel conv backward leaves 152 KB of partial sums: a launch on few
    frames is not cut into single rows to reach every CU (40 frames of 11x11: 19 us in 40 workgroups, 29 in
    240)."""
    assert plan("c64", n, H, W)["tiles"] <= most


@pytest.mark.parametrize("kind,n,H,W,most", [("b32", 40, 21, 21, 120), ("b32", 128, 11, 11, 128), ("b32", 40, 8, 12, 40),
                                             ("b16", 40, 11, 11, 80), ("b16", 40, 16, 16, 80)])
def test_block_backwards_on_few_frames_are_not_cut_into_single_rows(plan, kind, n, H, W, most):
    """128 frames of 11x11 with 32 channels: 18 us in 64 or 128 workgroups, 24 in 256."""
    assert plan(kind, n, H, W)["tiles"] <= most


@pytest.mark.parametrize("n,H,W,tiles", [(8192, 30, 45, True), (8192, 32, 32, True), (8192, 38, 33, True), (8192, 48, 40, True),
                                         (2048, 84, 84, True), (2048, 100, 60, True), (2048, 42, 42, False),
                                         (640, 42, 42, False), (8192, 21, 21, False), (8192, 11, 11, False),
                                         (300, 200, 200, False), (128, 42, 42, False), (8, 84, 84, False)])
def test_the_16_channel_block_backward_takes_the_faster_form(plan, n, H, W, tiles):
    """Where both forms were timed in turn and one is more than 3% faster."""
    p = plan("t16", n, H, W)
    assert (p["R"] == 0) == tiles, p
    assert p["tiles"] == -(-n // p["F"]) * p["bands"] and p["bands"] * p["TH"] >= H


@pytest.mark.parametrize("n", [1, 2048])
def test_the_block_forward_takes_every_frame_of_the_layer_calls(plan, n):
    """Sides up to 256, from 140 wide on in one workgroup per CU."""
    for W in range(1, 257):
        for H in (1, 2, 3, 7, 40, 256):
            p = plan("f32", n, H, W)
            assert p is not None, (n, H, W)
            assert p["lds"] <= (80 if W < 140 else 160) * 1024, (n, H, W, p)


def test_every_kernel_instance_is_compared_on_the_gpu(plan):
    """R is a constant of the kernels: the shapes of the bit-equality tests reach every compiled one."""
    pytest.importorskip("torch")
    from test_gpu_walks import SHAPES, TILES16, WIDE32, WIDE64

    def rows(kind, shapes):
        return {plan(kind, *c)["R"] for c in shapes}

    wide = [c for c in WIDE32 if c[2] >= 140 and c[1] > 2]   # (two rows fit whole)
    assert rows("f32", SHAPES) == set(range(1, 8))
    assert rows("f32", wide) == {1, 2}
    assert rows("b32", SHAPES) == set(range(1, 8))
    assert rows("t16", SHAPES) >= set(range(1, 9)) and rows("t16", TILES16) == {0}
    assert rows("c64", SHAPES) == set(range(1, 8))
    assert all(plan("c64", *c) is None for c in WIDE64)
    assert plan("t16", 1700, 29, 34)["R"] == 0 and plan("t16", 850, 29, 34)["R"] > 0   # (the network's backward)


@pytest.mark.parametrize("blocks,kind,n,H,W,helped", [(304, "b32", 8, 9, 9, True), (304, "b32", 114, 21, 21, True), (304, "b32", 301, 11, 11, True),
                                                      (304, "b32", 304, 21, 21, False), (592, "c64", 2, 11, 11, True), (592, "c64", 87, 12, 9, True),
                                                      (592, "c64", 105, 22, 18, False), (80, "b16", 94, 42, 42, True), (80, "b16", 119, 42, 42, False),
                                                      (0, "b32", 8, 9, 9, False)])
def test_idle_units_take_the_pending_sums(plan, blocks, kind, n, H, W, helped):
    """The partial sums of the launches before (152 blocks of 64 entries per 32-channel weight, 592 of 64, 40 of 16) are added up beside
    the tiles where enough compute units have none: 8 frames of 9x9 waited 23 us for them. No launch grows past the units."""
    parts = min(CUS, plan(kind, n, H, W)["tiles"])
    k = plan.pend_helpers(blocks, parts, CUS)
    assert (k > 0) == helped, (parts, k)
    for parts in range(1, CUS + 1):
        k = plan.pend_helpers(blocks, parts, CUS)
        assert 0 <= k <= min(blocks, CUS - parts)
        assert k == 0 or -(-blocks // k) <= 2 * -(-blocks // parts)


def test_tiles_are_taken_one_by_one_only_where_they_are_many(plan):
    """The tile-by-tile kernel sums the launches before it in its own workgroups only: its launches leave no unit idle."""
    for n in range(1, 512, 3):
        for H, W in ((1, 64), (2, 3), (21, 21), (29, 34), (42, 42), (48, 40), (64, 64), (64, 17)):
            p = plan("t16", n, H, W)
            assert p["R"] or p["tiles"] >= 2 * CUS, (n, H, W, p)
