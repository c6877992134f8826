"""The library's kernel choice and KV-cache plan (host code, asked through the
probe library; no GPU needed), on 256 compute units unless said otherwise."""
import itertools

import pytest

from tests.gpu_helpers import plan_of
from tests.probes import route
from tests.test_gpu_kv_shapes import INSTANCES


def test_instances_take_the_plan_they_name():
    # the GPU test of the kernel's instantiations runs each with and without counts
    for mode, d, bc, rows, plan, shape in INSTANCES:
        B, Hq, Hkv, nq, nk = shape
        assert nk % bc != 0 and (Hq // Hkv * nq) % rows != 0 and nq < 128
        for causal, count in itertools.product((True, False), (True, False)):
            assert plan_of(mode, d, bc, shape, causal, count) == (rows, plan), (mode, d, bc, shape)


def test_instances_are_all_there_are():
    # per mode, d and block: 16-row tiles unsplit on eight and four waves, or split;
    # the same for 32-row ones; and the column pairs that are built
    want = {(m, d, bc, rows, plan) for m, d, bc in itertools.product(("fast", "fp8qk"), (64, 128), (64, 128))
            for rows, plan in itertools.product((16, 32), ("c1w8", "c1w4", "split"))}
    want |= {("fast", 64, 64, 16, "c2w8"), ("fast", 64, 128, 16, "c2w8"), ("fast", 128, 64, 16, "c2w8"),
             ("fast", 128, 64, 16, "c2w4"), ("fast", 128, 128, 16, "c2w8"), ("fast", 128, 128, 16, "c2w4"),
             ("fp8qk", 64, 128, 16, "c2w8"), ("fp8qk", 128, 64, 16, "c2w8"), ("fp8qk", 128, 128, 16, "c2w8"),
             ("fp8qk", 128, 128, 16, "c2w4")}
    assert {i[:5] for i in INSTANCES} == want and len(INSTANCES) == len(want)


@pytest.mark.parametrize("mode", ["fast", "fp8qk"])
def test_a_split_is_one_generation_of_workgroups(mode):
    # A split is planned as one workgroup per compute unit: no XCD (32 of them) may
    # get more, also where the tiles do not divide by 8
    seen = set()
    for heads in range(1, 130):
        for nk in (2100, 9000, 60000, 131001):
            for G, nq in ((4, 1), (1, 32), (1, 48)):
                r = route(heads, G, 1, nq, nk, 128, 128, mode=mode)
                if r["C"] > 1:
                    assert r["slots"] <= 32 and r["slots"] * 8 >= r["units"] * r["C"], (heads, nk, G, nq, r)
                    seen.add(r["units"])
    assert {1, 2, 3, 5, 9, 11, 12, 21, 33} <= seen


@pytest.mark.parametrize("shape,mode,rows", [
    # a cache in HBM, tiles on less than half of the compute units: by ranges of the
    # keys (us: that, two workgroups per tile that share its columns, and the kernel
    # of one 32-row tile per query head, which split too)
    ((61, 1, 1, 1, 16384, 128, 128), "fast", 16),       # 104, 124, 112
    ((64, 1, 1, 4, 16384, 128, 128), "fp8qk", 16),      # 73, 87, 78
    ((64, 1, 1, 16, 65193, 128, 64), "fp8qk", 16),      # 274, 337, 289
    ((61, 1, 1, 4, 65193, 64, 128), "fast", 16),        # 216, 255, 233
    ((20, 2, 2, 1, 7503, 128, 128), "fast", 16),        # 43, 59, 47
    ((6, 8, 8, 2, 34693, 64, 128), "fast", 16),         # 85, 130, 91
    ((13, 4, 1, 64, 58454, 64, 64), "fp8qk", 32),       # 144, 16 rows unsplit 186, 125
    # two 16-row tiles of a head or one of 32 rows: the smaller ones read a range twice
    ((5, 8, 8, 32, 95011, 128, 128), "fp8qk", 32),      # 250, 16 rows split 300, 267
])
def test_long_caches_are_split_where_that_is_faster(shape, mode, rows):
    r = route(*shape, mode=mode)
    assert r["kernel"] == 0 and r["rows"] == rows and r["C"] > 1, r


def test_short_caches_share_the_columns():
    # 24 x 16/2 heads x 2757 keys: 20 us by columns, 24 by ranges; 64 x 32 queries x
    # 4096 keys, two tiles of a head on one L2: 33 us, 36 with one workgroup per tile
    for shape in ((64, 1, 1, 32, 4096, 128, 128), (24, 16, 2, 1, 2757, 128, 64), (5, 32, 8, 1, 3799, 128, 128), (3, 8, 1, 1, 4096, 128, 128)):
        r = route(*shape)
        assert r["kernel"] == 0 and r["cols"] == 2 and r["C"] == 1, r
        assert r["slots"] % 2 == 0, r      # a pair reads the same K: one XCD


@pytest.mark.parametrize("shape,causal", [
    # (us, with counts: this plan, 32-row tiles, the kernels before)
    ((1, 4, 4, 4096, 4096), False),      # 61, 71, 61
    ((1, 8, 8, 2048, 2048), False),      # 38, 43, 38
    ((1, 32, 32, 512, 512), True),       # 21, 24, 21
    ((2, 16, 2, 286, 286), True),        # 16 or 17, 20, 17
    ((2, 8, 8, 686, 25902), True),       # 303, 346, 303
])
def test_counts_avoid_the_kernel_that_spills(shape, causal):
    r = route(*shape, 128, 128, causal=causal, count=True)
    assert r["kernel"] == 128 or (r["kernel"] == 0 and r["rows"] == 16), r
    # without counts, and with E4M3 scores, it is the fastest
    assert route(*shape, 128, 128, causal=causal)["rows"] == 32
    assert route(*shape, 128, 128, causal=causal, mode="fp8qk", count=True)["rows"] == 32


def test_one_workspace_size_with_and_without_counts():
    # the size query does not know which of the two calls follows
    for nq in (1, 24, 48, 100):
        for h in (1, 3, 7, 20):
            for nk in (3000, 20000, 90000):
                shape = (h, 4, 1, nq, nk, 128, 128)
                a, b = route(*shape), route(*shape, count=True)
                assert a["ws"] == b["ws"]
                for r in (a, b):                       # enough for the plan either call would like most
                    full = route(*shape, count=r is b, ws_bytes=1 << 40)
                    assert {k: full[k] for k in full} == r, shape


def test_long_chunk_that_starts_inside_a_block():
    # (37 us on the KV-cache kernel, 63 on the fast kernel; 51 before)
    r = route(1, 16, 4, 1995, 3914, 64, 64, mode="fp8qk")
    assert r["kernel"] == 0 and r["rows"] == 32, r
