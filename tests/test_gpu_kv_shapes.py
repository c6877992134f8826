"""The KV-cache kernel's plans (16- or 32-row tiles of a group's query rows, four
or eight waves, unsplit, by columns, or over ranges of the keys) at lengths that leave
partial tiles, partial last blocks, rounds with idle waves and tiles that hold
rows of several query heads, against the oracle on every row; and workspaces
between the least and the reported size."""
import numpy as np
import pytest
import torch

from paper_2606_06521_amd.inputs import last_queries, make_inputs
from tests.gpu_helpers import compare, device_cus, log, plan_of, run_gpu, to_device

pytestmark = pytest.mark.gpu

# (B, Hq, Hkv, Nq, Nk, d, block_kv)
SHAPES = [
    (1, 8, 2, 1, 20000, 128, 128),
    (1, 8, 8, 3, 515, 64, 64),
    (2, 16, 4, 8, 1501, 128, 64),      # rows of two heads per tile
    (1, 8, 4, 8, 200, 128, 64),
    (60, 8, 4, 4, 333, 64, 128),
    (40, 8, 8, 37, 261, 64, 64),
    (16, 8, 8, 33, 1300, 128, 128),
    (16, 8, 8, 60, 2600, 128, 128),
    (1, 16, 1, 120, 12001, 128, 128),  # rows of up to two heads per tile
]

# Every instantiation of the kernel: mode, d, block_kv, rows per tile, plan on 256
# compute units ("c2w4": unsplit, two workgroups per tile, four waves each; "split":
# ranges of the keys), and a shape (B, Hq, Hkv, Nq, Nk) that takes it with and
# without counts (tests/test_kv_plan.py checks that), with a partial last tile, a
# partial last block and more than one round of the waves.
INSTANCES = [
    ("fast", 128, 128, 16, "c1w4", (2, 1, 1, 17, 517)),
    ("fast", 128, 128, 16, "c1w8", (3, 9, 3, 77, 2566)),
    ("fast", 128, 128, 16, "c2w4", (2, 1, 1, 1, 538)),
    ("fast", 128, 128, 16, "c2w8", (2, 1, 1, 1, 1560)),
    ("fast", 128, 128, 16, "split", (2, 1, 1, 2, 5059)),
    ("fast", 128, 128, 32, "c1w4", (12, 16, 1, 45, 515)),
    ("fast", 128, 128, 32, "c1w8", (8, 16, 1, 33, 2628)),
    ("fast", 128, 128, 32, "split", (1, 32, 2, 33, 7082)),
    ("fast", 128, 64, 16, "c1w4", (1, 2, 2, 1, 263)),
    ("fast", 128, 64, 16, "c1w8", (2, 24, 3, 45, 784)),
    ("fast", 128, 64, 16, "c2w4", (2, 1, 1, 1, 329)),
    ("fast", 128, 64, 16, "c2w8", (1, 2, 2, 1, 772)),
    ("fast", 128, 64, 16, "split", (1, 2, 2, 1, 3549)),
    ("fast", 128, 64, 32, "c1w4", (3, 32, 2, 45, 263)),
    ("fast", 128, 64, 32, "c1w8", (2, 48, 3, 45, 801)),
    ("fast", 128, 64, 32, "split", (1, 16, 2, 45, 3009)),
    ("fast", 64, 128, 16, "c1w4", (3, 12, 4, 120, 531)),
    ("fast", 64, 128, 16, "c1w8", (3, 16, 2, 45, 1033)),
    ("fast", 64, 128, 16, "c2w8", (2, 1, 1, 1, 1031)),
    ("fast", 64, 128, 16, "split", (1, 2, 2, 1, 6195)),
    ("fast", 64, 128, 32, "c1w4", (12, 16, 1, 45, 525)),
    ("fast", 64, 128, 32, "c1w8", (2, 48, 3, 45, 4659)),
    ("fast", 64, 128, 32, "split", (1, 8, 2, 45, 11198)),
    ("fast", 64, 64, 16, "c1w4", (3, 12, 4, 120, 258)),
    ("fast", 64, 64, 16, "c1w8", (1, 2, 2, 1, 532)),
    ("fast", 64, 64, 16, "c2w8", (1, 2, 2, 1, 833)),
    ("fast", 64, 64, 16, "split", (2, 1, 1, 1, 3686)),
    ("fast", 64, 64, 32, "c1w4", (3, 64, 4, 45, 259)),
    ("fast", 64, 64, 32, "c1w8", (8, 16, 1, 33, 776)),
    ("fast", 64, 64, 32, "split", (3, 3, 1, 77, 3061)),
    ("fp8qk", 128, 128, 16, "c1w4", (40, 4, 4, 2, 525)),
    ("fp8qk", 128, 128, 16, "c1w8", (3, 16, 2, 45, 1058)),
    ("fp8qk", 128, 128, 16, "c2w4", (40, 3, 3, 1, 775)),
    ("fp8qk", 128, 128, 16, "c2w8", (2, 1, 1, 1, 1039)),
    ("fp8qk", 128, 128, 16, "split", (2, 1, 1, 2, 6024)),
    ("fp8qk", 128, 128, 32, "c1w4", (40, 16, 1, 13, 513)),
    ("fp8qk", 128, 128, 32, "c1w8", (2, 64, 4, 33, 1573)),
    ("fp8qk", 128, 128, 32, "split", (2, 4, 1, 45, 11203)),
    ("fp8qk", 128, 64, 16, "c1w4", (8, 16, 2, 33, 258)),
    ("fp8qk", 128, 64, 16, "c1w8", (1, 2, 2, 1, 530)),
    ("fp8qk", 128, 64, 16, "c2w8", (2, 1, 1, 1, 596)),
    ("fp8qk", 128, 64, 16, "split", (2, 1, 1, 3, 3527)),
    ("fp8qk", 128, 64, 32, "c1w4", (3, 64, 4, 45, 261)),
    ("fp8qk", 128, 64, 32, "c1w8", (2, 64, 4, 33, 771)),
    ("fp8qk", 128, 64, 32, "split", (1, 6, 2, 100, 3521)),
    ("fp8qk", 64, 128, 16, "c1w4", (12, 8, 1, 45, 515)),
    ("fp8qk", 64, 128, 16, "c1w8", (2, 1, 1, 1, 1037)),
    ("fp8qk", 64, 128, 16, "c2w8", (2, 3, 1, 1, 1573)),
    ("fp8qk", 64, 128, 16, "split", (2, 1, 1, 1, 5086)),
    ("fp8qk", 64, 128, 32, "c1w4", (20, 4, 2, 100, 518)),
    ("fp8qk", 64, 128, 32, "c1w8", (3, 32, 2, 45, 5735)),
    ("fp8qk", 64, 128, 32, "split", (1, 6, 2, 60, 11141)),
    ("fp8qk", 64, 64, 16, "c1w4", (3, 32, 4, 45, 258)),
    ("fp8qk", 64, 64, 16, "c1w8", (2, 2, 1, 1, 521)),
    ("fp8qk", 64, 64, 16, "split", (1, 2, 2, 2, 3041)),
    ("fp8qk", 64, 64, 32, "c1w4", (5, 16, 4, 100, 267)),
    ("fp8qk", 64, 64, 32, "c1w8", (8, 16, 1, 33, 797)),
    ("fp8qk", 64, 64, 32, "split", (2, 3, 1, 100, 3521)),
]


@pytest.mark.parametrize("mode", ["fast", "fp8qk"])
@pytest.mark.parametrize("B,Hq,Hkv,nq,nk,d,bc", SHAPES)
def test_shapes_against_oracle(B, Hq, Hkv, nq, nk, d, bc, mode):
    fmt = "e4m3" if mode == "fp8qk" else "bf16_e4m3"
    inp = last_queries(make_inputs(B, Hq, Hkv, nk, d, fmt=fmt, delta=8.0, seed=2300 + nk), nq)
    dev = to_device(inp)
    for S, order, causal, scale in [(256.0, "reverse", True, "static"), (16.0, "forward", False, "dynamic"),
                                    (3.0, "forward", True, "static")]:
        label = f"kv plan {mode} B={B} Hq={Hq} Hkv={Hkv} nq={nq} nk={nk} d={d} bc={bc} S={S} {order} {causal}"
        log(label)
        gpu = run_gpu(dev, mode, S, order, causal, bc, scale=scale)
        compare(inp, gpu, mode, S, order, causal, bc, label=label, scale=scale)


@pytest.mark.parametrize("mode,d,bc,rows,plan,shape", INSTANCES, ids=lambda x: str(x).replace(" ", ""))
def test_instances_against_oracle(mode, d, bc, rows, plan, shape):
    B, Hq, Hkv, nq, nk = shape
    assert plan_of(mode, d, bc, shape, n_cu=device_cus()) == (rows, plan)
    fmt = "e4m3" if mode == "fp8qk" else "bf16_e4m3"
    inp = last_queries(make_inputs(B, Hq, Hkv, nk, d, fmt=fmt, delta=8.0, seed=2700 + nk), nq)
    dev = to_device(inp)
    for S, order, causal, scale in [(256.0, "reverse", True, "static"), (16.0, "forward", False, "dynamic"),
                                    (3.0, "reverse", True, "static")]:
        label = f"kv {rows} rows {plan} {mode} d={d} bc={bc} {shape} S={S} {order} {causal}"
        log(label)
        gpu = run_gpu(dev, mode, S, order, causal, bc, scale=scale)
        compare(inp, gpu, mode, S, order, causal, bc, label=label, scale=scale)


@pytest.mark.parametrize("mode", ["faithful", "fast", "fp8qk"])
@pytest.mark.parametrize("nq,nk,d,bc", [(1, 130, 64, 64), (40, 333, 128, 128), (3, 20001, 128, 64), (60, 259, 64, 128)])
def test_rows_after_the_cache_are_not_used(nq, nk, d, bc, mode):
    # K and V are the head of an allocation that goes on with NaN: a last block
    # that read them (its V rows meet P = 0) would give NaN
    fmt = {"faithful": "f32", "fast": "bf16_e4m3", "fp8qk": "e4m3"}[mode]
    inp = last_queries(make_inputs(1, 1, 1, nk, d, fmt=fmt, delta=8.0, seed=2350 + nk), nq)
    q, k, v = to_device(inp)

    def head_of_nan(t):
        raw = torch.full((1, 1, nk + 256, d * t.element_size()), 0x7F, dtype=torch.uint8, device="cuda")
        if t.element_size() > 1:
            raw = raw.view(t.dtype)
            raw[:] = float("nan")
        else:
            raw = raw.view(t.dtype)
        raw[:, :, :nk] = t
        head = raw[:, :, :nk]
        assert head.is_contiguous()
        return head

    dev = (q, head_of_nan(k), head_of_nan(v))
    for S, order, causal, scale in [(256.0, "reverse", True, "static"), (16.0, "forward", False, "dynamic")]:
        label = f"NaN after the cache {mode} nq={nq} nk={nk} d={d} bc={bc} {order} {causal}"
        log(label)
        gpu = run_gpu(dev, mode, S, order, causal, bc, scale=scale)
        compare(inp, gpu, mode, S, order, causal, bc, label=label, scale=scale)


@pytest.mark.parametrize("mode", ["fast", "fp8qk"])
@pytest.mark.parametrize("order", ["forward", "reverse"])
@pytest.mark.parametrize("Hq,Hkv,nq,nk,d", [(4, 1, 200, 200, 64), (6, 2, 200, 200, 128), (4, 1, 150, 350, 128)])
def test_nan_in_v_stays_in_its_block(Hq, Hkv, nq, nk, d, order, mode):
    # A NaN in the last key's V reaches (as 0 times NaN) rows that visit that key's
    # block, and no row of an earlier block of positions, whichever kernel runs
    from paper_2606_06521_amd import attn_fp8 as A
    fmt = "e4m3" if mode == "fp8qk" else "bf16_e4m3"
    inp = make_inputs(1, Hq, Hkv, nk, d, fmt=fmt, delta=8.0, seed=2360 + d)
    q, k, v = to_device(last_queries(inp, nq) if nq < nk else inp)
    bad = v.clone()
    bad.view(torch.uint8)[:, :, nk - 1, 5] = 0x7F
    clean = (nk - 1) // 64 * 64 - (nk - nq)            # rows before the last block of 64 positions
    clean -= clean % 32                                # (a tile's rows lie together)
    for tile in (None, 128, 256):
        label = f"NaN in V {mode} Hq={Hq} nq={nq} nk={nk} d={d} {order} tile={tile}"
        log(label)
        kw = dict(S=256.0, order=order, causal=True, block_kv=64, mode=mode, tile=tile)
        want = A.fwd(q, k, v, **kw)[0][:, :, :clean]
        got = A.fwd(q, k, bad, **kw)[0][:, :, :clean]
        assert clean >= 96 and torch.equal(got, want), label


def test_workspace_sizes():
    # Reported: room for 32 ranges per tile.  The least a call accepts is what
    # a split of 32-row tiles per query head over 8 workgroups takes, 64 x (8 x 32 + 32 d + 32)
    # floats here; anything from there on runs with fewer ranges.
    from paper_2606_06521_amd import attn_fp8 as A
    B, Hq, Hkv, nq, nk, d = 1, 8, 8, 1, 40000, 64
    inp = last_queries(make_inputs(B, Hq, Hkv, nk, d, fmt="bf16_e4m3", delta=8.0, seed=2400), nq)
    q, k, v = to_device(inp)
    st, full = A.attn_fp8_kv_workspace_bytes(B, Hq, Hkv, nq, nk, d, 1, 128, A.ATTN_MODE_FAST)
    least = 4 * 64 * (8 * 32) + 4 * 64 * (32 * d + 32)
    assert st == 0 and full > least
    ws = torch.full((full,), 0xFF, dtype=torch.uint8, device="cuda")
    sptr = torch.cuda.current_stream().cuda_stream

    def call(ptr, nbytes):
        o = torch.full((B, Hq, nq, d), float("nan"), device="cuda")
        lse = torch.full((B, Hq, nq), float("nan"), device="cuda")
        st = A.attn_fp8_fwd_kv(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(), B, Hq,
                               Hkv, nq, nk, d, 1, 128, 1, 256.0, 1, 1.0, 1.0, 1.0, ptr, nbytes, sptr)
        torch.cuda.synchronize()
        return st, o.cpu().numpy(), lse.cpu().numpy()

    for nbytes in (full, (full + least) // 2, least, 0):
        st, o, lse = call(ws.data_ptr() if nbytes else None, nbytes)
        assert st == 0
        log(f"kv workspace {nbytes} of {full}")
        compare(inp, (o, lse, None), "fast", 256.0, "reverse", True, 128, label=f"workspace {nbytes}")
    assert call(ws.data_ptr(), least - 1)[0] == A.ATTN_ERR_INVALID_ARG


# (B, Hq, Hkv, Nq, Nk, d, block_kv): the first query lies inside a KV block, in
# the block's first or last row, or in an earlier block than the wave's other rows
CHUNKS = [(2, 4, 2, 130, 257, 128, 128), (1, 4, 4, 257, 515, 64, 64), (1, 2, 1, 640, 705, 128, 64),
          (1, 2, 2, 300, 1003, 64, 128)]


@pytest.mark.parametrize("tile", [None, 128, 256])
@pytest.mark.parametrize("B,Hq,Hkv,nq,nk,d,bc", CHUNKS)
def test_chunk_that_starts_inside_a_block(B, Hq, Hkv, nq, nk, d, bc, tile):
    # both schedules of the fast kernel (rows before the chunk are empty) and
    # whichever kernel the library picks
    assert (nk - nq) % bc != 0
    for mode, fmt in (("fast", "bf16_e4m3"), ("fp8qk", "e4m3")):
        inp = last_queries(make_inputs(B, Hq, Hkv, nk, d, fmt=fmt, delta=8.0, seed=2500 + nk), nq)
        dev = to_device(inp)
        for S, order, causal, scale in [(256.0, "reverse", True, "static"), (1.0, "forward", True, "dynamic"),
                                        (16.0, "reverse", False, "static")]:
            label = f"chunk {mode} tile={tile} nq={nq} nk={nk} d={d} bc={bc} S={S} {order} {causal}"
            log(label)
            gpu = run_gpu(dev, mode, S, order, causal, bc, scale=scale, tile=tile)
            compare(inp, gpu, mode, S, order, causal, bc, label=label, scale=scale)


@pytest.mark.parametrize("H,Hkv,n,d,bc", [(2, 1, 700, 128, 128), (4, 4, 515, 64, 64), (1, 1, 1024, 128, 64)])
def test_small_square_problems_on_either_kernel(H, Hkv, n, d, bc):
    # few heads: the library's choice is the KV-cache kernel; its codes are those
    # of the fast kernel, so the counts are equal on every row
    for mode, fmt in (("fast", "bf16_e4m3"), ("fp8qk", "e4m3")):
        inp = make_inputs(1, H, Hkv, n, d, fmt=fmt, delta=8.0, seed=2600 + n)
        dev = to_device(inp)
        for order, causal in (("reverse", True), ("forward", False)):
            label = f"square {mode} n={n} d={d} bc={bc} {order} {causal}"
            log(label)
            gpu = run_gpu(dev, mode, 256.0, order, causal, bc)
            compare(inp, gpu, mode, 256.0, order, causal, bc, label=label)
            other = run_gpu(dev, mode, 256.0, order, causal, bc, tile=128)
            assert np.array_equal(gpu[2], other[2]), label
            assert np.allclose(gpu[0], other[0], rtol=1e-5, atol=1e-6), label
