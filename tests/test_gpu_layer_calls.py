"""The whole-layer calls against the single calls they stand for: same bits in every output, at the edges of what shares
a launch (8, 16 and more experts, short rows whose staged gradients fill the LDS, tables and none, slices, capacity)."""
import pytest

from paper_2504_03871_amd import binding as B
from tests import gpu_util as U
from tests.test_gpu_gemm_paths import filled_layer

pytestmark = pytest.mark.gpu

OUTS = ("logits", "topk_idx", "topk_w", "counts", "kept", "offsets", "row_of", "src_of", "x_perm", "saved", "y_perm", "out",
        "dy_perm", "d_topk_w", "dx_perm", "dW1", "dW1b", "dW2", "dWr", "d_logits", "dx")


def bits(t):
    import torch
    return t.contiguous().view(torch.uint8)


@pytest.mark.parametrize("T, d, f, E, k, dtype, act, cap, part, light", [
    (1, 64, 64, 1, 1, "bf16", B.ACT_GELU, 0, False, False),          # one token, one expert
    (700, 192, 320, 8, 2, "bf16", B.ACT_GELU, 0, False, True),       # a table, the weight gradient of up to eight experts
    (700, 64, 128, 12, 3, "f16", B.ACT_SWIGLU, 60, True, False),     # up to sixteen: the staged rows are too many for a shared launch
    (333, 2112, 128, 16, 4, "bf16", B.ACT_SWIGLU, 0, False, True),   # long rows, three slots of four and a last column unit
    (300, 128, 192, 17, 8, "f16", B.ACT_GELU, 40, False, False),     # more than sixteen: matrix-core weight gradient
    (257, 132, 68, 33, 2, "f32", B.ACT_SWIGLU, 0, True, False),      # fp32, groups of sixteen
    (512, 128, 256, 8, 2, "f32", B.ACT_GELU, 0, False, True),
    (5000, 36, 68, 5, 3, "f32", B.ACT_GELU, 0, False, False),        # histogram and ranks in two launches
    (900, 256, 128, 256, 2, "bf16", B.ACT_GELU, 0, False, False),    # one thread per expert in the map
])
def test_layer_calls_equal_the_single_calls(T, d, f, E, k, dtype, act, cap, part, light):
    import torch
    L = filled_layer(T, d, f, E, k, dtype, act)
    L.cfg.capacity = cap
    if part:
        L.set_slices([i % 7 for i in range(E)], [3 + 5 * (i % 9) for i in range(E)])
    L.bias = torch.linspace(0.5, -0.5, E, device="cuda")

    def reset(acc):
        U.fill_sentinels(L)
        for t in (L.ws, L.saved):
            t.fill_(7)
        if acc:
            for t in (L.dW1, L.dW1b, L.dW2, L.dWr):
                if t is not None:
                    t.fill_(0.125)

    for acc in (0, 1):
        reset(acc)
        L.route(); L.dispatch()
        if light:
            L.ffn_fwd_light(); L.combine(); L.route(); L.dispatch(); L.ffn_recompute()
        else:
            L.ffn_fwd(); L.combine()
        L.combine_bwd(); L.ffn_bwd(acc); L.dispatch_bwd(); L.route_bwd(acc)
        torch.cuda.synchronize()
        want = {n: getattr(L, n).clone() for n in OUTS if getattr(L, n) is not None}
        reset(acc)
        if light:
            B.moe_layer_fwd(L.cfg, L.bufs(), B.FWD_LIGHT)
            B.moe_layer_fwd(L.cfg, L.bufs(), B.FWD_RECOMPUTE)
        else:
            B.moe_layer_fwd(L.cfg, L.bufs())
        B.moe_layer_bwd(L.cfg, L.bufs(), acc)
        torch.cuda.synchronize()
        for n, t in want.items():
            assert torch.equal(bits(getattr(L, n)), bits(t)), (n, acc)


def test_layer_calls_of_no_tokens():
    import torch
    L = filled_layer(16, 64, 64, 4, 2, "bf16")
    L.cfg.T = 0
    U.fill_sentinels(L)
    B.moe_layer_fwd(L.cfg, L.bufs())
    B.moe_layer_bwd(L.cfg, L.bufs())
    torch.cuda.synchronize()
    assert L.counts.tolist() == [0] * 4 and L.kept.tolist() == [0] * 4 and L.offsets.tolist() == [0] * 5
    assert not L.dWr.any() and bool((L.dx.float() == U.SENTINEL).all()) and bool((L.dW1 == U.SENTINEL).all())
    L.dWr.fill_(3.0)
    B.moe_layer_bwd(L.cfg, L.bufs(), 1)
    torch.cuda.synchronize()
    assert bool((L.dWr == 3.0).all())
