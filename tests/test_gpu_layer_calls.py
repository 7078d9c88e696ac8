"""The whole-layer calls against the single calls they stand for: same bits in every output, at the edges of what shares
a launch (8, 16 and more experts, short rows whose staged gradients fill the LDS, tables and none, slices, capacity)."""
import pytest

from paper_2504_03871_amd import binding as B
from tests import gpu_util as U
from tests.test_gpu_gemm_paths import filled_layer, last_round_parts, tile_rows

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


@pytest.mark.parametrize("T, d, f, E, k, dtype, act, n", [
    (40, 64, 192, 6, 1, "bf16", B.ACT_GELU, 9),        # nine calls: eight in one pass and one added; experts without rows in some
    (300, 320, 576, 3, 2, "f16", B.ACT_SWIGLU, 3),     # whole and ragged stages, tiles past both widths
    (130, 128, 64, 2, 2, "bf16", B.ACT_SWIGLU, 1),     # every expert has all the rows: two stages and a remainder of two
    (50, 36, 68, 3, 1, "f32", B.ACT_SWIGLU, 3),
])
@pytest.mark.parametrize("acc", [0, 1])
def test_weight_gradients_over_several_calls(T, d, f, E, k, dtype, act, n, acc):
    """The sum over the calls of H^T dy and x^T dA, multiplied in fp64 from the stored tensors."""
    import torch
    from paper_2504_03871_amd.layer import MoELayer
    first = filled_layer(T, d, f, E, k, dtype, act, seed=1)
    calls = [first]
    for j in range(1, n):
        m = MoELayer(T, d, f, E, k, dtype=first.cfg.dtype, act=act, params=first, defer_dw=True)
        gen = torch.Generator(device="cuda:0").manual_seed(j + 5)
        for t in (m.x, m.d_out):
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
        calls.append(m)
    if n == 9:
        calls[4].set_slices([0] * E, [0] * E)                                # a call without any rows
        first.bias = calls[1].bias = torch.arange(E, device="cuda").float() * 3   # most rows on the last experts
    old = 0.25 if acc else 0.0
    grads = [g for g in (first.dW1, first.dW1b, first.dW2) if g is not None]
    for g in grads:
        g.fill_(0.25 if acc else U.SENTINEL)
    for j, m in enumerate(calls):
        m.forward()
        m.backward_inputs(1 if j > 0 else 0)
    MoELayer.expert_dw(calls, acc)
    torch.cuda.synchronize()
    planes = 2 if act == B.ACT_SWIGLU else 1
    el = first.x.element_size()
    want = [torch.full(g.shape, old, dtype=torch.float64, device="cuda") for g in grads]
    for m in calls:
        at = B.moe_workspace_bytes(m.cfg) - planes * T * k * f * el          # the standard workspace's last region
        at = at if planes * T * k * f * el % 256 == 0 else at // 256 * 256
        da = m.ws[at:at + planes * T * k * f * el].view(m.tdtype).view(planes, T * k, f).double()
        hid, dy, x = m.saved_plane(planes).double(), m.dy_perm.double(), m.x_perm.double()
        for e in range(E):
            o, c = int(m.offsets[e]), int(m.kept[e])
            lo, hi = (0, c) if m.slice_lo is None else (0, 0)
            r = slice(o + lo, o + hi)
            for i in range(planes):
                want[i][e] += x[r].t() @ da[i][r]
            want[planes][e] += hid[r].t() @ dy[r]
    for g, w in zip(grads, want):
        assert (g.double() - w).norm() <= 1e-5 * w.norm()      # fp32 sums


@pytest.mark.parametrize("T, d, f, E, k, dtype, act, n", [
    (40, 64, 192, 6, 1, "bf16", B.ACT_GELU, 9),        # a second pass of one call
    (300, 320, 576, 3, 2, "f16", B.ACT_SWIGLU, 3),
    (1100, 192, 320, 2, 1, "bf16", B.ACT_SWIGLU, 2),
    (50, 36, 68, 3, 1, "f32", B.ACT_SWIGLU, 3),
])
def test_weight_gradients_over_several_calls_are_those_of_call_after_call(T, d, f, E, k, dtype, act, n):
    """One pass over all calls has the very sums of a backward after the other that accumulates: no longer chains."""
    import torch
    from paper_2504_03871_amd.layer import MoELayer
    first = filled_layer(T, d, f, E, k, dtype, act, seed=1)
    calls = [first] + [MoELayer(T, d, f, E, k, dtype=first.cfg.dtype, act=act, params=first) for _ in range(n - 1)]
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    for m in calls:
        for t in (m.x, m.d_out):
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
        m.forward()
    if n > 2:
        calls[1].set_slices([0] * E, [0] * E)                                # a call without any rows
        calls[-1].set_slices([0] * E, [T * k if e == 1 else 0 for e in range(E)])
    grads = [g for g in (first.dW1, first.dW1b, first.dW2) if g is not None]
    for j, m in enumerate(calls):
        m.backward(1 if j > 0 else 0)
    want = [g.clone() for g in grads]
    for g in grads:
        g.fill_(U.SENTINEL)
    for m in calls:
        m.backward_inputs()
    MoELayer.expert_dw(calls)
    torch.cuda.synchronize()
    for g, w in zip(grads, want):
        assert torch.equal(g, w)


@pytest.mark.parametrize("T, d, f, E, k, dtype, act", [
    (700, 192, 2112, 4, 2, "bf16", B.ACT_GELU),        # 160-row tiles, 33 stages in seven parts or so
    (700, 192, 1088, 4, 2, "f16", B.ACT_SWIGLU),       # 17 and 17 stages of two products, a part across the seam
    (450, 320, 2048, 3, 1, "bf16", B.ACT_SWIGLU),
    (450, 320, 4096, 3, 1, "f16", B.ACT_GELU),
    (1100, 192, 1088, 2, 1, "bf16", B.ACT_SWIGLU),     # the same of 256-row tiles
    (1100, 192, 2112, 2, 1, "f16", B.ACT_GELU),
    (1100, 320, 4096, 2, 1, "bf16", B.ACT_GELU),       # with remainders of up to 64 rows, which a whole last round would split on their own
    (9356, 1024, 4096, 4, 1, "f16", B.ACT_GELU),       # and as it does: too many tiles behind the last whole round for two parts each
])
def test_input_gradient_split_along_k(T, d, f, E, k, dtype, act):
    """dx_perm of the backward that leaves the weight gradients out, its tiles split along K, against the unsplit one; the
    partial sums behind the workspace and in a room of the caller's."""
    import torch
    from paper_2504_03871_amd.layer import MoELayer
    src = filled_layer(T, d, f, E, k, dtype, act)
    L = MoELayer(T, d, f, E, k, dtype=src.cfg.dtype, act=act, params=src, defer_dw=True)
    L.x.copy_(src.x)
    L.d_out.copy_(src.d_out)
    L.forward()
    L.backward()
    whole = L.dx_perm.double()
    tiles, parts = last_round_parts(L.kept, (2 if act == B.ACT_SWIGLU else 1) * f, d, tile_rows(L))
    small = any(0 < int(c) % 256 <= 64 for c in L.kept)
    assert tile_rows(L) == (256 if T > 1000 else 160) and (parts > 1) == (T < 9000) and (small or f != 4096 or T < 1000), (tiles, parts)
    room = torch.empty(B.moe_layer_bwd_inputs_room_bytes(L.cfg), dtype=torch.uint8, device="cuda")
    assert room.numel() > 0 and L.ws.numel() >= B.moe_workspace_bytes(L.cfg) + room.numel()
    n = int(L.offsets[E])
    split = []
    for r in (None, room):
        L.dx_perm.fill_(U.SENTINEL)
        L.backward_inputs(room=r)
        torch.cuda.synchronize()
        err = (L.dx_perm.double()[:n] - whole[:n]).norm() / whole[:n].norm()
        # two results rounded to the storage type once each
        assert err < {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype], float(err)
        split.append(bits(L.dx_perm).clone())
    assert torch.equal(*split)
