"""The layer forward's two kernels on both sides of the rule that chooses
between them (bf16: 512 workgroups of 256 queries; float32 always takes the
128-query one), at lengths around their query blocks and key tiles, against
the fp64 oracle; scores that grow along the row, so that the running maximum
is raised again and again; and the grouped-query forward with the same.

Then the float32 backward at the edges of its blocks.  Bars as for the layer
(gpu_helpers): the kernels differ in summation order only.
"""

import numpy as np
import pytest

from gpu_helpers import announce, check_close, compare_layer, run_gpu, to_device, torch_cuda

pytestmark = pytest.mark.gpu


def _case(B, H, N, dtype, grow=False):
    from paper_2609_34650_amd import inputs
    fixed = [h for h in range(H) if h % 4 == 3]
    inp = inputs.make_inputs(B, H, N, 64, fixed, dtype, stream_id=51, backward=False)
    if grow:  # queries shifted by 4, keys growing along the row
        ramp = np.linspace(0.0, 1.5, N, dtype=np.float32)[:, None]
        rnd = inputs.round_to_bf16 if dtype == "bf16" else (lambda x: x)
        inp["Q"], inp["K"] = rnd(inp["Q"] + 4.0), rnd(inp["K"] + ramp)
    return inp


@pytest.mark.parametrize("B,H,N", [(8, 64, 1), (8, 64, 33), (8, 64, 64), (8, 64, 65), (8, 64, 129), (8, 64, 255),
                                   (8, 64, 256), (4, 64, 257), (3, 64, 700),                    # 256-query kernel
                                   (8, 63, 256), (7, 64, 65), (4, 63, 257), (1, 8, 129), (1, 5, 1000)])
def test_bf16_forward_both_sides_of_the_rule(B, H, N):
    announce(f"forward dispatch bf16 B={B} H={H} N={N}")
    inp = _case(B, H, N, "bf16")
    heads = [(0, 0), (B - 1, H - 1), (B // 2, 3)]
    compare_layer(run_gpu(inp, "bf16", backward=False), inp, "bf16", backward=False, heads=heads)


@pytest.mark.parametrize("dtype,B,H,N", [("bf16", 4, 64, 300), ("bf16", 1, 6, 300), ("f32", 2, 6, 300)])
def test_growing_scores_raise_the_maximum(dtype, B, H, N):
    announce(f"forward growing scores {dtype} B={B} H={H} N={N}")
    inp = _case(B, H, N, dtype, grow=True)
    heads = [(0, 0), (B - 1, H - 2)]
    compare_layer(run_gpu(inp, dtype, backward=False), inp, dtype, backward=False, heads=heads)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [96, 128])
def test_gqa_growing_scores_raise_the_maximum(dtype, d):
    torch = torch_cuda()
    from oracle import saf_oracle as orc
    from paper_2609_34650_amd import binding, inputs
    announce(f"gqa forward growing scores {dtype} d={d}")
    B, Hq, Hkv, N = 1, 4, 2, 300
    rnd = inputs.round_to_bf16 if dtype == "bf16" else (lambda x: x)
    q = inputs.make_inputs(B, Hq, N, d, [3], dtype, stream_id=52, backward=False)
    kv = inputs.make_inputs(B, Hkv, N, d, [], dtype, stream_id=53, backward=False)
    inp = dict(q, Q=rnd(q["Q"] + 4.0), K=rnd(kv["K"] + np.linspace(0.0, 1.5, N, dtype=np.float32)[:, None]),
               V=kv["V"])
    t = to_device(inp, dtype)
    O, L = binding.saf_hybrid_attn_fwd_gqa(t["Q"], t["K"], t["V"], inp["is_fixed"], t["a"], t["r"])
    torch.cuda.synchronize()
    oO, oL = orc.layer_forward_gqa(inp["Q"], inp["K"], inp["V"], inp["is_fixed"], inp["a"], inp["r"])
    check_close("O", O.double().cpu().numpy(), oO, dtype)
    check_close("LSE", L.double().cpu().numpy(), oL, dtype)


@pytest.mark.parametrize("B,H,N", [(1, 4, 15), (1, 4, 16), (3, 4, 17), (1, 4, 48), (2, 4, 49), (1, 4, 64), (3, 5, 80),
                                   (1, 4, 112), (2, 8, 321)])
def test_f32_backward_at_its_tile_edges(B, H, N):
    """16 queries and 16 keys a wavefront, blocks of 64 (fixed heads 128)."""
    from paper_2609_34650_amd import inputs
    announce(f"float32 layer B={B} H={H} N={N}")
    inp = inputs.make_inputs(B, H, N, 64, [1, H - 1], "f32", stream_id=54)
    compare_layer(run_gpu(inp, "f32"), inp, "f32")


@pytest.mark.parametrize("B,H,N,n_fixed", [(1, 64, 1024, 64), (1, 63, 1024, 63),     # all fixed: 256 workgroups, 252
                                           (1, 50, 2048, 17), (1, 49, 2048, 17),     # over a third: 400, 392
                                           (5, 64, 257, 21), (5, 64, 384, 21),       # to a third, short: 128 queries
                                           (5, 64, 257, 22), (4, 64, 513, 21), (4, 64, 640, 22)])
def test_bf16_forward_rule_by_fixed_share(B, H, N, n_fixed):
    """Both kernels on the lines that depend on the share of fixed heads."""
    from paper_2609_34650_amd import inputs
    announce(f"forward dispatch by share B={B} H={H} N={N} fixed={n_fixed}")
    inp = inputs.make_inputs(B, H, N, 64, list(range(H - n_fixed, H)), "bf16", stream_id=55, backward=False)
    heads = [(0, 0), (B - 1, H - 1), (B // 2, H - n_fixed)]
    compare_layer(run_gpu(inp, "bf16", backward=False), inp, "bf16", backward=False, heads=heads)


def test_growing_scores_raise_the_maximum_of_256_queries():
    announce("forward growing scores, 256-query kernel, ragged")
    inp = _case(3, 64, 700, "bf16", grow=True)
    compare_layer(run_gpu(inp, "bf16", backward=False), inp, "bf16", backward=False, heads=[(0, 0), (2, 62)])
