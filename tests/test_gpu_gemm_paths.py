"""GPU tests of single paths of the grouped GEMMs at the sizes where they can go wrong: edges of tiles, remainders,
empty experts."""
import pytest

from paper_2504_03871_amd import binding as B

pytestmark = pytest.mark.gpu

DT = {"f32": B.DTYPE_F32, "bf16": B.DTYPE_BF16, "f16": B.DTYPE_F16}


def filled_layer(T, d, f, E, k, dtype, act=B.ACT_GELU, seed=0):
    import torch
    from paper_2504_03871_amd.layer import MoELayer
    L = MoELayer(T, d, f, E, k, dtype=DT[dtype], act=act)
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    for t, std in ((L.x, 1.0), (L.d_out, 1.0), (L.Wr, d ** -0.5), (L.W1, d ** -0.5), (L.W2, f ** -0.5), (L.W1b, d ** -0.5)):
        if t is not None:
            t.copy_(torch.randn(t.shape, generator=gen, device=t.device) * std)
    return L


@pytest.mark.parametrize("T, d, f, E, k, dtype, act", [
    (700, 192, 320, 4, 2, "bf16", B.ACT_GELU),        # neither width a multiple of the tile, several K stages
    (300, 64, 576, 3, 1, "f16", B.ACT_SWIGLU),
    (3, 320, 256, 8, 1, "bf16", B.ACT_SWIGLU),        # experts without rows keep what they had
    (40, 36, 68, 3, 1, "f32", B.ACT_GELU),            # fp32: tiles of 32 rows
    (65, 388, 4100, 2, 1, "f32", B.ACT_SWIGLU),       # and of 64
])
def test_accumulated_weight_gradients_are_old_plus_new(T, d, f, E, k, dtype, act):
    """accumulate = 1 adds, in fp32 and with one rounding, the very sums that accumulate = 0 stores."""
    import torch
    L = filled_layer(T, d, f, E, k, dtype, act)
    L.forward()
    L.combine_bwd()
    L.ffn_bwd(0)
    grads = [g for g in (L.dW1, L.dW1b, L.dW2) if g is not None]
    new = [g.clone() for g in grads]
    old = [torch.randn_like(g) for g in grads]
    for g, o in zip(grads, old):
        g.copy_(o)
    L.ffn_bwd(1)
    torch.cuda.synchronize()
    for g, o, n in zip(grads, old, new):
        assert torch.equal(g, o + n)


@pytest.mark.parametrize("T, d, f, E, k, act", [
    (5, 4, 4, 2, 1, B.ACT_GELU),            # far below one tile and one K stage in every dimension
    (65, 36, 64, 1, 1, B.ACT_SWIGLU),       # one row past a row tile, four K values past a stage
    (200, 132, 260, 3, 2, B.ACT_SWIGLU),    # four columns past a column tile
    (129, 64, 128, 4, 1, B.ACT_GELU),       # whole tiles and stages
    (33, 36, 68, 1, 1, B.ACT_SWIGLU),       # one row past a tile of 32
    (1100, 36, 3076, 2, 1, B.ACT_GELU),     # tiles of 64 rows in the row-tile GEMMs, of 32 in the weight gradients
    (1100, 36, 3076, 2, 1, B.ACT_SWIGLU),
    (65, 388, 4100, 2, 1, B.ACT_SWIGLU),    # and the other way round
    (7000, 36, 4100, 2, 1, B.ACT_GELU),     # too many tiles to share a launch: dH and dW2 in their own
    (7000, 3588, 36, 2, 1, B.ACT_SWIGLU),   # dx in its own, dW1 and dW1b in one
])
def test_fp32_gemms_at_tile_and_stage_edges(T, d, f, E, k, act):
    from paper_2504_03871_amd import synth as S
    from tests.test_gpu_parity import run_case
    run_case(S.WORKLOADS["cfg0"].scaled(T=T, d=d, f=f, E=E, k=k, act=act))


@pytest.mark.parametrize("T, d, f, dtype, act, per_rounding, chains", [
    (1920, 256, 1024, "f32", B.ACT_SWIGLU, 1, 2),    # 512 tiles of 64 rows per gradient: 32-row tiles, two chains per sum
    (512, 256, 1024, "f32", B.ACT_SWIGLU, 1, 2),
    (1920, 256, 1024, "f32", B.ACT_GELU, 1, 2),
    (2000, 516, 1540, "f32", B.ACT_SWIGLU, 1, 1),    # 64-row tiles
    (1920, 256, 1024, "bf16", B.ACT_SWIGLU, 8, 1),
    (8192, 256, 1024, "f16", B.ACT_GELU, 8, 1),
])
def test_weight_gradient_sums_round_as_seldom_as_their_chains_say(T, d, f, dtype, act, per_rounding, chains):
    """Weight gradients against fp64 products of the stored tensors.  A rounding is off by 0.425 u of the partial sum
    (u = 2^-24; uniform within half a unit, evenly spread logarithms), and like-sized products in random order make partial
    sums whose squares grow evenly: a chain of L roundings is off by 0.425 u sqrt(L / 2) = 0.30 u sqrt(L).  fp32 instructions
    round after every product, 16-bit ones after eight.  Bound: a tenth more."""
    import torch
    E, k = 8, 2
    L = filled_layer(T, d, f, E, k, dtype, act)
    L.forward()
    L.combine_bwd()
    L.ffn_bwd()
    torch.cuda.synchronize()
    planes, n = 2 if act == B.ACT_SWIGLU else 1, T * k * f * L.x.element_size()
    dact = L.ws[L.ws.numel() - planes * n:].view(L.tdtype).view(planes, T * k, f).double()    # the workspace's last region
    pairs = [(L.x_perm.double(), dact[i], g) for i, g in enumerate([L.dW1, L.dW1b][:planes])] + [(L.saved_plane(planes).double(), L.dy_perm.double(), L.dW2)]
    for a, b, g in pairs:
        err = size = roundings = 0.0
        for e in range(E):
            r = slice(int(L.offsets[e]), int(L.offsets[e + 1]))
            want = a[r].t() @ b[r]
            err += float((g[e].double() - want).norm() ** 2)
            size += float(want.norm() ** 2)
            roundings += float(want.norm() ** 2) * (r.stop - r.start) / per_rounding / chains
        print(f"{dtype} {T} {d} {f}: {(err / size) ** 0.5 * 2 ** 24:.2f} u, {0.3 * (roundings / size) ** 0.5:.2f} u expected")
        assert (err / size) ** 0.5 <= 1.1 * 0.3 * (roundings / size) ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("dtype, d, f", [("f32", 36, 68), ("bf16", 64, 64)])
def test_a_row_with_nan_stays_in_its_row(dtype, d, f):
    """What lies behind the last K value of a row (the next row) takes no part in its sums."""
    import torch
    L = filled_layer(90, d, f, 2, 1, dtype)
    L.route()
    L.dispatch()
    L.x_perm[7] = float("nan")
    L.ffn_fwd()
    torch.cuda.synchronize()
    bad = torch.isnan(L.y_perm.float()).any(dim=1).nonzero().flatten().tolist()
    assert bad == [7]


@pytest.mark.parametrize("T, d, f, E, k, dtype, act, zipf", [
    (1, 64, 64, 2, 1, "DT_BF16", "ACT_GELU", 0.0),        # one row, one K stage, half a column tile
    (32, 128, 192, 2, 2, "DT_F16", "ACT_SWIGLU", 0.0),    # 32 rows per expert: the most that still goes this way
    (33, 128, 192, 2, 2, "DT_F16", "ACT_SWIGLU", 0.0),    # 160-row tiles
    (48, 128, 192, 2, 2, "DT_F16", "ACT_SWIGLU", 0.0),
    (96, 192, 320, 4, 2, "DT_BF16", "ACT_SWIGLU", 1.5),   # skewed: an expert with two row tiles, one with next to none
    (190, 64, 4096, 8, 2, "DT_BF16", "ACT_GELU", 1.5),    # split along K, full 64-row tiles beside the split ones
    (60, 192, 2112, 5, 2, "DT_BF16", "ACT_SWIGLU", 0.0),  # 33 K stages in eight parts, every expert one row tile
    (100, 192, 2112, 5, 2, "DT_F16", "ACT_GELU", 2.5),    # and in four, an expert with two; one (almost) without rows
    (450, 128, 192, 40, 4, "DT_BF16", "ACT_SWIGLU", 1.2), # more than 32 experts, some with several row tiles
])
def test_few_rows_per_expert(T, d, f, E, k, dtype, act, zipf):
    from paper_2504_03871_amd import synth as S
    from tests.test_gpu_parity import run_case
    run_case(S.WORKLOADS["cfg1"].scaled(T=T, d=d, f=f, E=E, k=k, dtype=getattr(S, dtype), act=getattr(S, act), zipf_s=zipf))


@pytest.mark.parametrize("T, f", [(3, 9 << 20), (3, 15 << 20), (33, 15 << 20)])
@pytest.mark.parametrize("act", [B.ACT_GELU, B.ACT_SWIGLU])
def test_rows_past_a_tile_whose_offsets_wrap_32_bits_are_not_stored(act, T, f):
    """A few rows of millions of elements.  With f = 15 << 20 row 159 of a 160-row tile, which the backward runs and, above 32
    rows, the forward, lies beyond 4 GiB from the tile's start, and the rows in between fall back into the valid ones.  The
    64-row tiles of the forward of three rows cannot wrap (64 rows of d f < 2^30 elements, d = 64, are at most 2 GiB), nor can
    256-row ones, which more than 512 rows or 128 per expert of at most 4 GiB in all get."""
    import torch
    d = 64
    L = filled_layer(T, d, f, 1, 1, "bf16", act)
    L.forward()
    L.combine_bwd()
    L.ffn_bwd()
    torch.cuda.synchronize()
    assert 255 * f * 2 > 1 << 32 and tile_rows(L) == 160
    assert any(m * f * 2 % (1 << 32) < T * f * 2 for m in range(T, 160)) == (f == 15 << 20)   # rows past the tile's that wrap into it
    # the last region of the workspace: dA, or dG and dU
    planes = 2 if act == B.ACT_SWIGLU else 1
    dact = L.ws[L.ws.numel() - planes * T * f * 2:].view(L.tdtype).view(planes, T, f).float()
    x, dy, saved = L.x_perm.float(), L.dy_perm.float(), [L.saved_plane(i).float() for i in range(planes + 1)]
    step = 1 << 20
    for c in range(0, f, step):
        s = slice(c, min(c + step, f))
        dh = dy @ L.W2[0, s].float().t()
        pre = [x @ w[0, :, s].float() for w in (L.W1, L.W1b) if w is not None]
        if act == B.ACT_SWIGLU:
            sg = torch.sigmoid(saved[0][:, s])
            want = pre + [torch.nn.functional.silu(pre[0]) * pre[1], dh * saved[1][:, s] * sg * (1 + saved[0][:, s] * (1 - sg)), dh * saved[0][:, s] * sg]
        else:
            a = saved[0][:, s].double()
            grad = 0.5 * torch.erfc(-a / 2 ** 0.5) + a * torch.exp(-a * a / 2) / (2 * torch.pi) ** 0.5
            want = pre + [torch.nn.functional.gelu(pre[0]), dh * grad.float()]
        for got, ref in zip([t[:, s] for t in saved] + [t[:, s] for t in dact], want):
            # two roundings to bf16 (2^-9 each) at most, the pre-activation's and the result's
            assert (got - ref).norm() <= 2.0 ** -7 * ref.norm()


def routes(L):
    """Rows of a 16-bit layer's forward tiles, how many of them there are when weights are streamed, the same of the backward's."""
    return B.moe_gemm_block_tile(7, L.T * L.k, L.E, L.act == B.ACT_SWIGLU, 0, L.d, L.f)[:4]


def tile_rows(L):
    """Rows of a 16-bit layer's row tiles (more than 32 rows per expert)."""
    return routes(L)[2]


def last_round_parts(kept, f, N, rows=256):
    """(tiles, K parts) of a row-tile GEMM over these rows, as the kernels compute them."""
    n_rt, ntn = sum(-(-int(n) // rows) for n in kept), -(-N // 256)
    return n_rt * ntn, B.moe_gemm_block_tile(4, 0, n_rt, 0, 0, f // 64, ntn)[2]


@pytest.mark.parametrize("T, d, f, E, k, dtype, act", [
    (700, 192, 2112, 4, 2, "bf16", B.ACT_GELU),        # 160-row tiles: 33 stages of 64 in 7 parts or so, full and partly filled tiles
    (450, 320, 2048, 3, 1, "f16", B.ACT_SWIGLU),       # a last column tile of 64
    (1090, 320, 2112, 2, 1, "bf16", B.ACT_SWIGLU),     # and of 256 rows
    (4096, 128, 2048, 40, 2, "bf16", B.ACT_SWIGLU),    # expert-major tile list
    (8200, 1088, 4096, 4, 2, "f16", B.ACT_GELU),       # a whole round before the split tiles
])
def test_last_round_split_along_k(T, d, f, E, k, dtype, act):
    """y = hidden W2 with the tiles of the last round split along K, against the same rows multiplied in fp64."""
    import torch
    L = filled_layer(T, d, f, E, k, dtype, act)
    L.forward()
    torch.cuda.synchronize()
    tiles, parts = last_round_parts(L.kept, f, d, tile_rows(L))
    assert parts > 1 and (tiles > 256) == (T == 8200)
    hid = L.saved_plane(2 if act == B.ACT_SWIGLU else 1)
    tol = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}[dtype]   # one rounding of the result: 2^-9 (2^-12) relative at most
    for e in range(E):
        o, n = int(L.offsets[e]), int(L.kept[e])
        ref = hid[o:o + n].double() @ L.W2[e].double()
        err = (L.y_perm[o:o + n].double() - ref).norm() / ref.norm()
        assert err < tol, (e, float(err))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_small_remainders_split_along_k_in_the_gelu_input_gradient(dtype):
    """dx = dA W1^T of 256-row tiles in a launch shared with dW1: remainders of at most 64 rows are split along K on their own."""
    import torch
    T, d, f, E, k = 1100, 128, 2560, 4, 2
    L = filled_layer(T, d, f, E, k, dtype)
    L.forward()
    L.combine_bwd()
    L.ffn_bwd()
    torch.cuda.synchronize()
    assert tile_rows(L) == 256 and any(0 < int(n) % 256 <= 64 for n in L.kept) and any(int(n) % 256 > 64 or int(n) > 256 for n in L.kept)
    dact = L.ws[L.ws.numel() - T * k * f * 2:].view(L.tdtype).view(T * k, f)   # the workspace's last region
    tol = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}[dtype]                        # one rounding of the result
    for e in range(E):
        r = slice(int(L.offsets[e]), int(L.offsets[e + 1]))
        ref = dact[r].double() @ L.W1[e].double().t()
        assert (L.dx_perm[r].double() - ref).norm() < tol * ref.norm(), e


@pytest.mark.parametrize("dtype, cap", [("bf16", 2000), ("f16", 1100)])
def test_last_round_split_along_k_in_the_gelu_input_gradient(dtype, cap):
    """dx = dA W1^T in a launch of its own (more than 2048 tiles possible, few there because of the capacity) with 34
    stages of 64 in parts of unequal length, against the stored dA multiplied in fp64."""
    import torch
    from paper_2504_03871_amd.layer import MoELayer
    T, d, f, E = 131072, 1024, 2176, 2
    L = MoELayer(T, d, f, E, 1, dtype=DT[dtype], act=B.ACT_GELU, capacity=cap)
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    for t, std in ((L.x, 1.0), (L.d_out, 1.0), (L.Wr, d ** -0.5), (L.W1, d ** -0.5), (L.W2, f ** -0.5)):
        t.normal_(0.0, std, generator=gen)
    L.forward()
    L.combine_bwd()
    L.ffn_bwd()
    torch.cuda.synchronize()
    tiles, parts = last_round_parts(L.kept, f, d)
    assert -(-d // 256) * (-(-T // 256) + E) > 2048 and parts > 1 and f // 64 % parts != 0, (tiles, parts)
    dact = L.ws[L.ws.numel() - T * f * 2:].view(L.tdtype).view(T, f)     # the workspace's last region
    tol = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}[dtype]                  # one rounding of the result
    for e in range(E):
        o, n = int(L.offsets[e]), int(L.kept[e])
        assert n == cap
        ref = dact[o:o + n].double() @ L.W1[e].double().t()
        err = (L.dx_perm[o:o + n].double() - ref).norm() / ref.norm()
        assert err < tol, (e, float(err))


@pytest.mark.parametrize("T, d, f, E, k, dtype, act, zipf", [
    (159, 64, 64, 1, 1, "bf16", "gelu", 0.0),         # one row short of a tile; one K stage of the three
    (160, 128, 128, 1, 1, "bf16", "swiglu", 0.0),     # two stages
    (161, 192, 192, 1, 1, "bf16", "gelu", 0.0),       # a tile of one row; three stages
    (512, 256, 576, 1, 1, "f16", "gelu", 0.0),        # the most rows that go this way; four stages and nine
    (513, 256, 576, 1, 1, "bf16", "gelu", 0.0),       # 256-row tiles
    (130, 320, 256, 2, 1, "bf16", "swiglu", 0.0),     # bands of 32 rows at both wave rows' ends
    (700, 64, 2112, 4, 2, "bf16", "gelu", 1.5),       # GEMM2 split along K; experts with several tiles and with a part of one
    (512, 128, 192, 33, 8, "f16", "swiglu", 0.0),     # more than 32 experts, below their line
    (529, 128, 192, 33, 8, "bf16", "gelu", 1.2),      # and above it
])
def test_experts_of_few_row_tiles(T, d, f, E, k, dtype, act, zipf):
    from paper_2504_03871_amd import synth as S
    from tests.test_gpu_parity import run_case
    run_case(S.WORKLOADS["cfg1"].scaled(T=T, d=d, f=f, E=E, k=k, dtype=getattr(S, "DT_" + dtype.upper()), act=getattr(S, "ACT_" + act.upper()), zipf_s=zipf))


@pytest.mark.parametrize("T, d, f, E, k, dtype, act", [
    (513, 64, 64, 1, 1, "bf16", "swiglu"),       # SwiGLU in 256-row tiles: a tile of one row, half a column tile
    (545, 128, 192, 1, 1, "f16", "swiglu"),      # two bands of 32 rows for four wave rows
    (1400, 192, 320, 2, 1, "bf16", "swiglu"),    # six bands or so, three column tiles
    (1100, 64, 4096, 2, 1, "bf16", "gelu"),      # GELU, hidden plane stored plainly (9 MB)
    (16400, 64, 2112, 2, 1, "f16", "gelu"),      # and streamed (69 MB)
])
def test_forward_stores_of_high_tiles(T, d, f, E, k, dtype, act):
    from paper_2504_03871_amd import synth as S
    from tests.test_gpu_parity import run_case
    run_case(S.WORKLOADS["cfg1"].scaled(T=T, d=d, f=f, E=E, k=k, dtype=getattr(S, "DT_" + dtype.upper()), act=getattr(S, "ACT_" + act.upper())))


@pytest.mark.parametrize("T, d, f, dtype, act", [
    (600, 64, 64, "bf16", "gelu"),        # one K stage in every row-tile GEMM (SwiGLU's dx: two)
    (600, 64, 64, "bf16", "swiglu"),
    (600, 128, 192, "f16", "gelu"),       # two and three, as many as the operand with more LDS has
    (600, 192, 128, "f16", "swiglu"),
    (600, 256, 192, "bf16", "gelu"),      # four: the first that meets the loop's steady state
    (600, 192, 256, "bf16", "swiglu"),
    (600, 192, 192, "bf16", "gelu"),      # three with a GELU table, which takes the place of the first; and in a longer loop, six
    (600, 384, 384, "bf16", "gelu"),
])
def test_short_k_in_high_tiles(T, d, f, dtype, act):
    """256-row tiles whose operands have two and three LDS stages, with fewer K stages than these, as many, and one more."""
    from paper_2504_03871_amd import synth as S
    from tests.test_gpu_parity import run_case
    run_case(S.WORKLOADS["cfg1"].scaled(T=T, d=d, f=f, E=1, k=1, dtype=getattr(S, "DT_" + dtype.upper()), act=getattr(S, "ACT_" + act.upper())))


@pytest.mark.parametrize("T, d, f, E, k, dtype, act", [
    (1440, 1024, 2624, 32, 2, "bf16", B.ACT_GELU),     # 160-row tiles; dH and dx share launches with the weight gradients
    (700, 1088, 1792, 32, 2, "f16", B.ACT_SWIGLU),     # a last column tile of 64 columns
    (1200, 1088, 832, 64, 8, "bf16", B.ACT_SWIGLU),    # 256-row tiles
    (1600, 576, 2432, 64, 6, "f16", B.ACT_GELU),
    (2000, 2048, 2048, 160, 8, "f16", B.ACT_GELU),     # 160-row tiles, too many of them to share a launch
    (2625, 2304, 2304, 160, 8, "bf16", B.ACT_SWIGLU),  # and 256-row ones
    (250, 2048, 2048, 32, 2, "bf16", B.ACT_GELU),      # 16 rows per expert, still in 160-row tiles
    (9, 4096, 8192, 4, 1, "f16", B.ACT_SWIGLU),        # 2 rows; y split along K
])
def test_weights_requested_as_streaming_data(T, d, f, E, k, dtype, act):
    """Layers of more than 320 MB of weights and at most a row tile per expert on average, one expert with several tiles:
    every row-tile GEMM against the same rows multiplied in fp64, those of the backward with the weight gradients (in one
    launch up to 2048 tiles) and without them (always in launches of their own)."""
    import torch
    swiglu = act == B.ACT_SWIGLU
    rows = 160 if T * k <= 128 * E or (E <= 32 and T * k <= 512 * E) else 256
    assert T * k <= rows * E and E * d * f * (3 if swiglu else 2) * 2 > 320 << 20
    L = filled_layer(T, d, f, E, k, dtype, act)
    least = (320 << 20) // (d * f * (3 if swiglu else 2) * 2) + 1
    assert routes(L) == [rows, least, rows, least]
    assert all((-(-n // 256) * (T * k // rows + E) > 2048) == (E == 160) for n in (d, f))
    L.bias = torch.tensor([2.5] + [0.0] * (E - 1), device=L.device)
    L.forward()
    L.combine_bwd()
    one = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}[dtype]   # one rounding of the result
    planes = 2 if swiglu else 1
    dact = L.ws[L.ws.numel() - planes * T * k * f * 2:].view(L.tdtype).view(planes, T * k, f)   # the workspace's last region
    grads = []
    for backward in (L.ffn_bwd, L.ffn_bwd_inputs):
        dact.fill_(float("nan"))
        L.dx_perm.fill_(float("nan"))
        backward()
        grads.append(torch.cat([t.view(T * k, -1) for t in (*dact, L.dx_perm)], 1))
    torch.cuda.synchronize()
    assert T < 10 or int(L.kept.max()) > rows >= int(L.kept.median())
    assert int((L.kept > 0).sum()) >= least
    for e in range(E):
        o, n = int(L.offsets[e]), int(L.kept[e])
        at = lambda t: t[o:o + n].double()
        pre = [at(L.x_perm) @ w[e].double() for w in (L.W1, L.W1b) if w is not None]
        dh = at(L.dy_perm) @ L.W2[e].double().t()
        v = [at(L.saved_plane(i)) for i in range(planes)]
        if swiglu:
            sg = torch.sigmoid(v[0])
            da = [dh * v[1] * sg * (1 + v[0] * (1 - sg)), dh * v[0] * sg]
        else:
            da = [dh * (0.5 * torch.erfc(-v[0] / 2 ** 0.5) + v[0] * torch.exp(-v[0] * v[0] / 2) / (2 * torch.pi) ** 0.5)]
        checks = [*((a, b, one) for a, b in zip(v, pre)), (at(L.y_perm), at(L.saved_plane(planes)) @ L.W2[e].double(), one)]
        for got in (at(g) for g in grads):
            parts = [got[:, i * f:(i + 1) * f] for i in range(planes)]
            dx = sum(p @ w[e].double().t() for p, w in zip(parts, (L.W1, L.W1b)))
            # (dA: its rounding, and fp16's polynomial derivative or the fast sigmoid, well below another one)
            checks += [*((p, r, 2 * one) for p, r in zip(parts, da)), (got[:, planes * f:], dx, one)]
        for got, ref, tol in checks:
            assert (got - ref).norm() <= tol * ref.norm(), e


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_last_round_split_along_k_in_the_input_gradient_of_low_tiles(dtype):
    """dx = dA W1^T of 160-row tiles, which are too many to share a launch where 256-row ones would not be, with the last
    round split: partial sums and the rows they come from each in their own part of the workspace."""
    import torch
    from paper_2504_03871_amd.layer import MoELayer
    T, d, f, E, k, cap = 8192, 4160, 2112, 32, 2, 150
    L = MoELayer(T, d, f, E, k, dtype=DT[dtype], act=B.ACT_GELU, capacity=cap)
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    for t, std in ((L.x, 1.0), (L.d_out, 1.0), (L.Wr, d ** -0.5), (L.W1, d ** -0.5), (L.W2, f ** -0.5)):
        t.normal_(0.0, std, generator=gen)
    L.forward()
    L.combine_bwd()
    L.ffn_bwd()
    torch.cuda.synchronize()
    ntn = -(-d // 256)
    tiles, parts = last_round_parts(L.kept, f, d, 160)
    assert ntn * (-(-T * k // 160) + E) > 2048 >= ntn * (-(-T * k // 256) + E) and tiles % 256 and parts > 1, (tiles, parts)
    dact = L.ws[L.ws.numel() - T * k * f * 2:].view(L.tdtype).view(T * k, f)   # the workspace's last region
    tol = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}[dtype]                        # one rounding of the result
    dh = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]                         # two: the pre-activation's and the result's
    for e in range(E):
        o, n = int(L.offsets[e]), int(L.kept[e])
        ref = dact[o:o + n].double() @ L.W1[e].double().t()
        assert (L.dx_perm[o:o + n].double() - ref).norm() < tol * ref.norm(), e
        a = L.saved_plane(0)[o:o + n].double()
        grad = 0.5 * torch.erfc(-a / 2 ** 0.5) + a * torch.exp(-a * a / 2) / (2 * torch.pi) ** 0.5
        ref = (L.dy_perm[o:o + n].double() @ L.W2[e].double().t()) * grad
        assert (dact[o:o + n].double() - ref).norm() < dh * ref.norm(), e


@pytest.mark.parametrize("A", [1, 1023, 1024, 1025, 4096, 4097])
@pytest.mark.parametrize("E, cap", [(1, 0), (8, 0), (17, 60), (256, 5)])
def test_dispatch_of_short_lists(A, E, cap):
    """One block, whole and ragged blocks, and both sides of the line up to which a block counts the other blocks'
    ids itself; few and many experts, with and without capacity, ids outside [0, E) among them.  Exact."""
    import numpy as np
    import torch
    from tests import gpu_util as U
    idx = np.random.default_rng(A * E).integers(-1, E + 1, size=(A, 1)).astype(np.int32)
    cfg = B.make_cfg(A, 64, 64, E, 1, capacity=cap)
    out = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (E, E, E + 1, A, A)]
    ws = torch.empty(B.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    B.moe_dispatch(cfg, None, torch.from_numpy(idx).cuda(), None, None, *out, None, ws)
    torch.cuda.synchronize()
    for name, got, want in zip(("counts", "kept", "offsets", "row_of", "src_of"), out, U.O.dispatch_plan(idx, E, cap)):
        assert (got.cpu().numpy() == want).all(), name


@pytest.mark.parametrize("T, d, E, k, dtype", [
    (2049, 128, 3, 2, "DT_BF16"), (2048, 128, 3, 2, "DT_BF16"),     # both sides of the line for few, short rows
    (37, 36, 5, 3, "DT_F32"), (100, 1024, 32, 2, "DT_F16"), (100, 512, 33, 4, "DT_F16"),
])
def test_gate_backward_of_short_inputs(T, d, E, k, dtype):
    from paper_2504_03871_amd import synth as S
    from tests.test_gpu_parity import run_case
    base = S.WORKLOADS["cfg0" if dtype == "DT_F32" else "cfg1"]
    run_case(base.scaled(T=T, d=d, f=128, E=E, k=k, dtype=getattr(S, dtype)))


@pytest.mark.parametrize("T, d, E, k, dtype", [
    (1, 64, 1, 1, "DT_BF16"), (17, 192, 16, 3, "DT_F16"),           # one token; one past a block, half a K block at the end
    (48, 2112, 17, 2, "DT_BF16"), (31, 1088, 32, 4, "DT_F16"),      # two expert tiles; one wave with a second K block
    (15, 1152, 9, 2, "DT_BF16"),                                    # sixteen waves, nine of them busy
    (33, 36, 5, 3, "DT_F32"), (16, 516, 32, 2, "DT_F32"),           # fp32: a row that ends inside a quarter
    (100, 4, 16, 2, "DT_F32"), (40, 1100, 20, 2, "DT_F32"),
    (4096, 64, 8, 2, "DT_BF16"), (4097, 64, 8, 2, "DT_BF16"),       # both sides of the line
    (64, 128, 33, 2, "DT_F32"),                                     # more than 32 experts
])
def test_gate_of_few_tokens(T, d, E, k, dtype):
    from paper_2504_03871_amd import synth as S
    from tests.test_gpu_parity import run_case
    base = S.WORKLOADS["cfg0" if dtype == "DT_F32" else "cfg1"]
    run_case(base.scaled(T=T, d=d, f=64, E=E, k=k, dtype=getattr(S, dtype)))


@pytest.mark.parametrize("T, d, E, bound", [(2048, 64, 8, 2), (2048, 128, 8, 2), (1000, 260, 13, 2), (1000, 512, 32, 2), (2000, 516, 8, 2),
                                            (1000, 516, 32, 3), (1000, 1024, 20, 3)])
def test_fp32_gate_sums_in_short_chains(T, d, E, bound):
    """Logits against 64 bits.  A chain of n like-sized sums is off by about 0.3 u sqrt(n) (u = 2^-24; a rounding is off by 0.425 u
    of a partial sum, and those grow like a random walk).  Four chains of 16 products per lane, then at most 16 waves' sums:
    0.3 u sqrt(16 + 4 + 16) = 1.8 u, bound 2 u.  Two expert tiles of rows longer than 512 have one chain of 64 products:
    0.3 u sqrt(64 + 16) = 2.7 u, bound 3 u."""
    import numpy as np
    import torch
    rng = np.random.default_rng(d)
    x, Wr = rng.standard_normal((T, d)).astype(np.float32), (rng.standard_normal((d, E)) * d ** -0.5).astype(np.float32)
    cfg = B.make_cfg(T, d, 64, E, 2, dtype=B.DTYPE_F32)
    e = lambda n, t: torch.empty(T, n, dtype=t, device="cuda")
    logits, idx, w = e(E, torch.float32), e(2, torch.int32), e(2, torch.float32)
    ws = torch.empty(B.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    B.moe_route(cfg, torch.from_numpy(x).cuda(), torch.from_numpy(Wr).cuda(), None, None, logits, idx, w, ws)
    torch.cuda.synchronize()
    want = x.astype(np.float64) @ Wr.astype(np.float64)
    err = np.linalg.norm(logits.cpu().numpy() - want) / np.linalg.norm(want)
    print(f"T {T} d {d} E {E}: {err:.3e}")
    assert err <= bound * 2.0 ** -24


@pytest.mark.parametrize("T, d, E, dtype", [
    (1, 64, 1, "bf16"), (4096, 1088, 6, "bf16"), (100, 1984, 16, "f16"),   # four waves along K: one K block, two and three, four
    (33, 2048, 8, "bf16"), (17, 4160, 16, "f16"), (5, 9280, 3, "bf16"),     # eight waves: two K blocks each, five, nine and ten
    (48, 704, 17, "f16"), (1000, 2112, 32, "bf16"),                         # two expert tiles
])
def test_a_token_has_the_same_logits_in_a_batch_of_any_size(T, d, E, dtype):
    """The gate of few tokens adds K up in the order of the one for many: bit-equal logits, ids and weights."""
    import torch
    k, many = min(E, 2), 4097
    gen = torch.Generator(device="cuda:0").manual_seed(d)
    x = torch.randn(many, d, generator=gen, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float16)
    Wr, bias = torch.randn(d, E, generator=gen, device="cuda"), torch.randn(E, generator=gen, device="cuda")
    got = []
    for n in (T, many):
        cfg = B.make_cfg(n, d, 64, E, k, dtype=DT[dtype])
        out = [torch.empty(n, c, dtype=t, device="cuda") for c, t in ((E, torch.float32), (k, torch.int32), (k, torch.float32))]
        ws = torch.empty(B.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
        B.moe_route(cfg, x[:n], Wr, bias, None, *out, ws)
        got.append([t[:T] for t in out])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("A, E", [(65 * 1024, 5), (97 * 1024 + 3, 256), (200000, 100)])
def test_dispatch_with_scanned_prefixes(A, E):
    """More than 64 blocks: whole and ragged batches of the scan, more experts than one of its blocks has threads.  Exact."""
    import numpy as np
    import torch
    from tests import gpu_util as U
    idx = np.random.default_rng(E).integers(-1, E + 1, size=(A, 1)).astype(np.int32)
    cfg = B.make_cfg(A, 64, 64, E, 1, capacity=A // E)
    out = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (E, E, E + 1, A, A)]
    ws = torch.empty(B.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    B.moe_dispatch(cfg, None, torch.from_numpy(idx).cuda(), None, None, *out, None, ws)
    torch.cuda.synchronize()
    for name, got, want in zip(("counts", "kept", "offsets", "row_of", "src_of"), out, U.O.dispatch_plan(idx, E, A // E)):
        assert (got.cpu().numpy() == want).all(), name
