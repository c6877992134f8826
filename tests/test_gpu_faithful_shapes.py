"""The FP32 kernel's tile and workgroup shapes (16- or 32-row tiles, four or
eight waves, one or two workgroups per tile), chosen by how far the tiles fill
the chip, each at lengths that leave partial tiles, partial last blocks and
rounds with idle waves, against the oracle on every row; and its exp2."""
import numpy as np
import pytest
import torch

from paper_2606_06521_amd.inputs import last_queries, make_inputs
from tests.gpu_helpers import compare, log, run_gpu, to_device

pytestmark = pytest.mark.gpu

# (heads, query rows, keys): with 256 compute units, 32-row tiles on four waves
# (512 tiles or more), on eight (256 or more), 16-row tiles (more than 128), and two
# workgroups per 16-row tile
SHAPES = [(172, 65, 65), (104, 79, 129), (40, 50, 50), (33, 49, 700), (3, 17, 1025), (1, 1, 130)]


@pytest.mark.parametrize("d,block_kv", [(64, 64), (128, 128), (128, 64), (64, 128)])
@pytest.mark.parametrize("H,nq,nk", SHAPES)
def test_shapes_against_oracle(H, nq, nk, d, block_kv):
    inp = make_inputs(1, H, H, nk, d, fmt="f32", delta=8.0, seed=1700 + H)
    if nq < nk:
        inp = last_queries(inp, nq)
    dev = to_device(inp)
    for i, (mode, S, order, causal, scale) in enumerate([
            ("faithful", 256.0, "reverse", True, "static"), ("faithful", 3.0, "forward", False, "static"),
            ("faithful", 16.0, "forward", True, "dynamic"), ("nocast", 448.0, "reverse", False, "static")]):
        label = f"faithful shape H={H} nq={nq} nk={nk} d={d} bk={block_kv} #{i}"
        log(label)
        gpu = run_gpu(dev, mode, S, order, causal, block_kv, scale=scale)
        compare(inp, gpu, mode, S, order, causal, block_kv, label=label, scale=scale)


@pytest.mark.parametrize("order", ["forward", "reverse"])
def test_dynamic_scale_of_subnormal_probabilities(order):
    # Blocks 88 to 95 nats below the running maximum: their P are FP32 subnormals
    # (below 2^-126), cast through the convert with scales down to 2^-126; codes
    # and counts are those of the exact product P * 2^kj.  (With the sinks last,
    # the same blocks come before the maximum rises.)
    for d, bkv in ((64, 64), (128, 128)):
        inp = make_inputs(1, 2, 2, 700, d, fmt="f32", delta=91.0, seed=1790 + d)
        dev = to_device(inp)
        label = f"faithful dynamic delta=91 d={d} bk={bkv} {order}"
        log(label)
        gpu = run_gpu(dev, "faithful", 16.0, order, False, bkv, scale="dynamic")
        compare(inp, gpu, "faithful", 16.0, order, False, bkv, label=label, scale="dynamic")
        if order == "forward":       # neither none nor all of the other blocks' codes are zero
            z = int(gpu[2][..., 2].sum())
            assert 0 < z < 2 * 700 * (700 - bkv), z


def test_scales_whose_reciprocal_overflows():
    # S = 2^-127 is the last power of two with a finite FP32 reciprocal; below it
    # every code is 0 too (P S < 2^-10), so the output is 0 and every key counts
    inp = make_inputs(1, 2, 1, 150, 64, fmt="f32", delta=5.0, seed=1795)
    dev = to_device(inp)
    for e in (-127, -128, -149):
        label = f"faithful S=2^{e}"
        log(label)
        gpu = run_gpu(dev, "faithful", 2.0 ** e, "reverse", True, 64)
        compare(inp, gpu, "faithful", 2.0 ** e, "reverse", True, 64, label=label)


def test_exp2_is_correctly_rounded():
    # against FP64 exp2 rounded once: equal, but for values whose FP64 result lies
    # within its own error (2^-51 relative, both sides) of a rounding midpoint:
    # one value in 2^27, so at most a handful of 2^22
    from tests import probes as pr
    rng = np.random.default_rng(3)
    edge = np.arange(-160, 1).astype(np.float32)
    x = np.concatenate([edge, np.nextafter(edge, np.float32(-np.inf)), np.nextafter(edge, np.float32(1)),
                        edge + np.float32(0.5), np.float32([-np.inf, -1e30, -0.0]),
                        rng.uniform(-40, 0, 1 << 21).astype(np.float32),
                        (-np.exp2(rng.uniform(-30, 8, 1 << 21))).astype(np.float32)])
    xt = torch.from_numpy(x).cuda()
    out = torch.empty_like(xt)
    assert pr.lib().probe_exp2_f64(xt.data_ptr(), x.size, out.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream) == 0
    got = out.cpu().numpy()
    want = np.exp2(x.astype(np.float64)).astype(np.float32)
    bad = np.nonzero(got != want)[0]
    assert bad.size <= 4, [(float(x[i]), float(got[i]), float(want[i])) for i in bad[:8]]
    nan = torch.full((64,), float("nan"), device="cuda")
    assert pr.lib().probe_exp2_f64(nan.data_ptr(), 64, nan.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream) == 0
    assert torch.isnan(nan).all()
