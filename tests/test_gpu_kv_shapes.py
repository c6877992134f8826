"""The KV-cache kernel's plans (16- or 32-row tiles of a group's query rows, four
or eight waves, unsplit, by columns, or over ranges of the keys), each at lengths that leave
partial tiles, partial last blocks, rounds with idle waves and tiles that hold
rows of several query heads, against the oracle on every row; and workspaces
between the least and the reported size."""
import numpy as np
import pytest
import torch

from paper_2606_06521_amd.inputs import last_queries, make_inputs
from tests.gpu_helpers import compare, log, run_gpu, to_device

pytestmark = pytest.mark.gpu

# (B, Hq, Hkv, Nq, Nk, d, block_kv): the plan on 256 compute units
SHAPES = [
    (1, 8, 2, 1, 20000, 128, 128),     # 16 rows, 19 ranges of the keys
    (1, 8, 8, 3, 515, 64, 64),         # 16 rows, eight waves
    (2, 16, 4, 8, 1501, 128, 64),      # 16 rows, two workgroups by columns, rows of two heads per tile
    (1, 8, 4, 8, 200, 128, 64),        # 16 rows, four waves, by columns
    (60, 8, 4, 4, 333, 64, 128),       # 16 rows, four waves
    (40, 8, 8, 37, 261, 64, 64),       # the same in two generations
    (16, 8, 8, 33, 1300, 128, 128),    # 32 rows, four waves
    (16, 8, 8, 60, 2600, 128, 128),    # 32 rows, eight waves
    (1, 16, 1, 120, 12001, 128, 128),  # 32 rows, 4 ranges, rows of up to two heads per tile
]


@pytest.mark.parametrize("mode", ["fast", "fp8qk"])
@pytest.mark.parametrize("B,Hq,Hkv,nq,nk,d,bc", SHAPES)
def test_plans_against_oracle(B, Hq, Hkv, nq, nk, d, bc, mode):
    fmt = "e4m3" if mode == "fp8qk" else "bf16_e4m3"
    inp = last_queries(make_inputs(B, Hq, Hkv, nk, d, fmt=fmt, delta=8.0, seed=2300 + nk), nq)
    dev = to_device(inp)
    for S, order, causal, scale in [(256.0, "reverse", True, "static"), (16.0, "forward", False, "dynamic"),
                                    (3.0, "forward", True, "static")]:
        label = f"kv plan {mode} B={B} Hq={Hq} Hkv={Hkv} nq={nq} nk={nk} d={d} bc={bc} S={S} {order} {causal}"
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
