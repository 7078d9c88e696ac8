"""Host-side enumeration of the block -> tile numbering of the grouped GEMMs (the code the kernels run, called
through the C ABI): every tile of a ragged map is computed exactly once, every K part of a split tile exactly
once, nothing is out of range, surplus blocks exit, and the fp32 partial sums of the split tiles stay inside
their workspace region.  Also the byte-offset bound of the weight-gradient GEMM's operand walk."""
import itertools

import pytest

from paper_2504_03871_amd import binding as B

SPLIT_K, SPLIT_ROWS, NUM_XCD = 8, 64, 8


def test_row_tile_numbering_covers_every_tile_once():
    cases = itertools.product((0, 1, 5, 61, 64, 67), (0, 1, 3, 8), (1, 4, 16, 56))   # full tiles, partial tiles, column tiles
    for n_full, n_part, ntn in cases:
        for n_split in sorted({0, min(n_part, 1), n_part}):
            n_rt = n_full + n_part
            E = max(n_part, 1)
            grid = ntn * (n_rt + E) + E * ntn * (SPLIT_K - 1)        # the launch's worst-case block count
            seen, parts = {}, {}
            for vb in range(grid):
                ok, rt, _, nt, st, ks = B.moe_gemm_block_tile(0, vb, n_rt, n_full, n_split, 1, ntn)
                if not ok:
                    continue
                assert 0 <= rt < n_rt and 0 <= nt < ntn
                if st < 0:
                    assert rt < n_rt - n_split and (rt, nt) not in seen
                    seen[(rt, nt)] = vb
                else:
                    assert 0 <= st < n_split and rt == n_rt - n_split + st and 0 <= ks < SPLIT_K
                    assert (st, nt, ks) not in parts
                    parts[(st, nt, ks)] = vb
                    # fp32 partial sums: index of the last element this block may write, against the region
                    N = ntn * 256
                    last = ((st * SPLIT_K + ks) * SPLIT_ROWS + (SPLIT_ROWS - 1)) * N + (N - 1)
                    assert last * 4 < E * SPLIT_K * SPLIT_ROWS * N * 4
            assert len(seen) == (n_rt - n_split) * ntn and len(parts) == n_split * ntn * SPLIT_K
            # blocks of the full region that share an XCD (block % 8) get a contiguous run of tiles: walking an
            # XCD's blocks in dispatch order moves through row-tile groups of four, column by column
            per = (n_full * ntn) // NUM_XCD
            if per >= 8 and ntn >= 2 and n_full >= 4:
                x0 = [B.moe_gemm_block_tile(0, b, n_rt, n_full, n_split, 1, ntn) for b in range(0, 8 * NUM_XCD, NUM_XCD)]
                assert len({(t[1] // 4) for t in x0}) <= 2          # eight consecutive tiles of XCD 0: at most two groups


def test_weight_gradient_numbering_covers_every_tile_once_and_balances_xcds():
    for ntm, ntn, E in ((1, 1, 3), (4, 16, 2), (16, 56, 2), (56, 16, 1), (7, 5, 4), (3, 3, 5)):
        P = ntm * ntn
        P8 = (P + NUM_XCD - 1) // NUM_XCD * NUM_XCD
        seen = set()
        per_xcd = [[0] * NUM_XCD for _ in range(E)]
        for vb in range(P8 * E):
            ok, slot, mt, nt, _, _ = B.moe_gemm_block_tile(1, vb, ntm=ntm, ntn=ntn)
            if not ok:
                continue
            assert 0 <= slot < E and 0 <= mt < ntm and 0 <= nt < ntn and (slot, mt, nt) not in seen
            seen.add((slot, mt, nt))
            per_xcd[slot][vb % NUM_XCD] += 1
        assert len(seen) == P * E
        for e in range(E):      # an expert's tiles are spread evenly over the XCDs (skewed experts stay balanced)
            assert max(per_xcd[e]) - min(per_xcd[e]) <= 1
        if ntm >= 4 and ntn >= 8 and P8 // NUM_XCD >= 32:     # 32 tiles running together on XCD 0: a 4 x 8 patch
            t = [B.moe_gemm_block_tile(1, b, ntm=ntm, ntn=ntn) for b in range(0, 32 * NUM_XCD, NUM_XCD)]
            assert len({x[2] for x in t}) + len({x[3] for x in t}) <= 12 + 1


def test_rejects_bad_arguments():
    lib = B.lib()
    import ctypes
    out = (ctypes.c_int32 * 6)()
    assert lib.moe_gemm_block_tile(0, 0, 4, 5, 0, 1, 1, out) == -2        # more full tiles than tiles
    assert lib.moe_gemm_block_tile(0, 0, 4, 2, 3, 1, 1, out) == -2        # more split tiles than partial ones
    assert lib.moe_gemm_block_tile(2, 0, 4, 2, 0, 1, 1, out) == -3
    assert lib.moe_gemm_block_tile(0, 0, 4, 2, 0, 1, 1, None) == -1


@pytest.mark.parametrize("n_full, n_part, ntn", [(0, 3, 5), (1, 0, 1), (7, 2, 9), (8, 0, 32), (13, 1, 23), (67, 8, 16), (40, 3, 56)])
def test_chunked_row_tile_numbering_covers_every_tile_once(n_full, n_part, ntn):
    """Full and ragged bands of eight row tiles, strips of eight columns, several chunks of 256 and a ragged last one."""
    n_rt = n_full + n_part
    t = [B.moe_gemm_block_tile(3, vb, n_rt, n_full, 0, 1, ntn) for vb in range(n_rt * ntn + 8)]
    assert sorted((x[1], x[3]) for x in t if x[0]) == list(itertools.product(range(n_rt), range(ntn)))
    assert not any(x[0] for x in t[n_rt * ntn:])
    assert all(x[1] >= n_full for x in t[n_full * ntn:n_rt * ntn])      # partly filled row tiles last


@pytest.mark.parametrize("n_full, n_part, ntn, stages", [(0, 3, 5, 33), (1, 0, 1, 32), (61, 8, 4, 64), (16, 0, 8, 128), (30, 1, 9, 224), (64, 0, 4, 64), (40, 3, 5, 31)])
def test_tail_split_numbering_covers_every_tile_and_k_part_once(n_full, n_part, ntn, stages):
    """Fewer tiles than one round, one round and a few, exactly one round, K too short; stages that parts do not divide."""
    n_rt = n_full + n_part
    t = [x for x in (B.moe_gemm_block_tile(4, vb, n_rt, n_full, 0, stages, ntn) for vb in range(n_rt * ntn + 256)) if x[0]]
    parts, tail = t[0][2], n_rt * ntn % 256
    whole = [(x[1], x[3]) for x in t if x[4] < 0]
    split = [(x[1], x[3], x[5]) for x in t if x[4] >= 0]
    tiles = {(r, c) for r, c, _ in split}
    assert sorted(whole + list(tiles)) == list(itertools.product(range(n_rt), range(ntn)))
    assert len(set(split)) == len(split) == len(tiles) * parts
    assert len(split) <= 256 and len(tiles) in (0, tail)
    assert (parts > 1) == bool(split)
    if stages * 64 < 2048 or tail == 0:
        assert not split
    # slot (index among the split tiles, part) of every block: 0 .. 255, each once
    assert sorted(x[4] * parts + x[5] for x in t if x[4] >= 0) == list(range(len(split)))
    assert parts <= 8 <= stages


@pytest.mark.parametrize("n_rt, E, mates, split, ntn", [
    (1, 1, 0, 1, 1), (8, 8, 0, 1, 32), (16, 16, 0, 0, 64), (200, 256, 0, 0, 16), (3, 5, 0, 1, 9),   # one row tile per expert
    (2, 1, 1, 1, 1), (11, 8, 1, 1, 32), (14, 8, 1, 0, 112), (9, 6, 1, 1, 9), (225, 128, 1, 0, 16), (70, 40, 1, 0, 5),
])
def test_few_row_numbering_covers_every_tile_and_part_once_and_keeps_row_tiles_together(n_rt, E, mates, split, ntn):
    t = [x for x in (B.moe_gemm_block_tile(5, vb, n_rt, mates, split, E, ntn) for vb in range(n_rt * ntn * 8 + 8)) if x[0]]
    parts = t[0][2]
    assert parts == (1 if not split else 4 if mates else 8)
    assert sorted((x[1], x[3], x[5]) for x in t) == list(itertools.product(range(n_rt), range(ntn), range(parts)))
    assert all(x[4] == (x[1] if split else -1) for x in t)
    if split:                                               # fp32 partial sums: tile slots of the workspace region
        assert max(x[4] * parts + x[5] for x in t) < E * 8
    if mates and len(t) >= 1024:
        # row tiles that share weights are neighbours in the list: the 64 blocks an XCD runs at a time are 8 x 8 patches
        x0 = t[0:64 * NUM_XCD:NUM_XCD]
        assert len({x[1] for x in x0}) <= 8 and len({(x[3], x[5]) for x in x0}) <= 9
        # and the chip as a whole reads whole weight rows: XCDs beside each other take neighbouring columns
        assert len({(x[3], x[5]) for x in t[:64 * NUM_XCD]}) >= min(64, ntn * parts)


@pytest.mark.parametrize("rows, E, ntn, stages", [
    (16384, 8, 4, 64), (6000, 2, 5, 45), (2000, 3, 9, 33), (9003, 6, 5, 45), (16384, 8, 16, 224), (1000, 1, 36, 32), (16384, 8, 4, 31), (1, 4, 1, 32)])
def test_the_reduction_is_launched_where_a_tile_count_can_split_and_only_there(rows, E, ntn, stages):
    """Every tile count that rows spread over E experts can have, against the split the kernels themselves compute."""
    counts = range((rows + 255) // 256, min(rows, rows // 256 + E) + 1)
    splits = [B.moe_gemm_block_tile(4, 0, n, 0, 0, stages, ntn)[2] > 1 for n in counts]
    assert B.moe_gemm_block_tile(6, rows, E, 0, 0, stages, ntn)[0] == any(splits)
    assert B.moe_gemm_block_tile(6, rows, E, 0, 1, stages, ntn)[0] == (stages >= 32)     # some rows left out: any count


@pytest.mark.parametrize("rows, E, ntn, stages", [
    (4096, 8, 4, 64), (700, 2, 5, 45), (1280, 8, 32, 64), (159, 1, 9, 33), (320, 2, 256, 32), (16000, 32, 8, 128), (4096, 8, 4, 31), (1, 4, 1, 32)])
def test_the_same_of_160_row_tiles(rows, E, ntn, stages):
    counts = range((rows + 159) // 160, min(rows, rows // 160 + E) + 1)
    splits = [B.moe_gemm_block_tile(4, 0, n, 0, 0, stages, ntn)[2] > 1 for n in counts]
    assert B.moe_gemm_block_tile(6, rows, E, 1, 0, stages, ntn)[0] == any(splits)
    if E > 1:
        assert B.moe_gemm_block_tile(6, rows, E, 1, 1, stages, ntn)[0] == (stages >= 32)


@pytest.mark.parametrize("kind, n_rt, n_split, ntm, ntn", [
    (4, 4, 0, 1 << 26, 1), (6, 4, 0, 1 << 26, 1), (6, 1 << 16, 0, 32, 1 << 16),                # K = 64 ntm beyond 32 bits
    (0, 1 << 16, 0, 1, 1 << 16), (3, 1 << 16, 0, 1, 1 << 16), (4, 1 << 16, 0, 32, 1 << 16),  # tiles beyond 32 bits
    (0, 1 << 12, 1 << 12, 1, 1 << 17), (5, 1 << 16, 1, 8, 1 << 13),                          # with their K parts
    (1, 0, 0, 1 << 16, 1 << 16),                                                             # tiles of an expert
])
def test_sizes_beyond_32_bits_are_refused(kind, n_rt, n_split, ntm, ntn):
    import ctypes
    out = (ctypes.c_int32 * 6)()
    assert B.lib().moe_gemm_block_tile(kind, 0, n_rt, 0, n_split, ntm, ntn, out) == -2


def forward_rows(rows, E, d, f, swiglu):
    return B.moe_gemm_block_tile(7, rows, E, int(swiglu), 0, d, f)[0]


@pytest.mark.parametrize("E, d, f, swiglu, rows", [
    (32, 2048, 8192, True, 8), (32, 2048, 8192, False, 8),   # from eight rows per expert and d 2048 on
    (64, 1024, 2048, True, 16), (64, 960, 2048, False, 16),  # more than 32 experts: from 16 rows on, SwiGLU from d 1024 on
    (8, 4096, 8192, True, 2), (4, 4096, 8192, True, 2),      # SwiGLU's matrices of 64 MB: from two rows on
])
def test_few_rows_in_160_row_tiles_from_a_width_and_a_row_count_on(E, d, f, swiglu, rows):
    assert forward_rows(rows * E, E, d, f, swiglu) == 160 and forward_rows(rows * E - 1, E, d, f, swiglu) == 64
    most = 24 if E <= 32 else 32
    assert forward_rows(most * E, E, d, f, swiglu) == 160
    assert forward_rows(24 * E + 1, E, d, f, swiglu) == (64 if E <= 32 else 160) and forward_rows(32 * E + 1, E, d, f, swiglu) == 160


@pytest.mark.parametrize("E, d, f, swiglu, rows", [
    (32, 1984, 8192, True, 16), (32, 1984, 8192, False, 16), (64, 960, 2048, True, 24), (7, 1344, 7552, True, 16),   # narrower
    (8, 4096, 7936, True, 2), (8, 4096, 14336, False, 2),    # matrices of 62 MB; GELU
    (8, 4096, 2560, False, 16),                              # 320 MB of weights in all
    (12, 3200, 5120, True, 8),                               # y: 156 tiles, neither most of a round nor split
])
def test_few_rows_in_their_own_kernel(E, d, f, swiglu, rows):
    assert forward_rows(rows * E, E, d, f, swiglu) == 64


@pytest.mark.parametrize("E, d, f, swiglu, least", [
    (26, 512, 4352, True, 26), (8, 4096, 14336, True, 1), (8, 4096, 2560, False, 0), (8, 4096, 2624, False, 8), (256, 2048, 1024, False, 41),
])
def test_weights_are_streamed_from_320_mb_of_experts_with_rows_on(E, d, f, swiglu, least):
    """A launch has at least one row tile per expert with rows."""
    bytes_of = lambda tiles: tiles * d * f * (3 if swiglu else 2) * 2
    for rows in (E, 100 * E):
        assert B.moe_gemm_block_tile(7, rows, E, int(swiglu), 0, d, f)[3] == least
    assert (bytes_of(least) > 320 << 20 >= bytes_of(least - 1)) if least else bytes_of(E) <= 320 << 20
    assert B.moe_gemm_block_tile(7, 513 * E, E, int(swiglu), 0, d, f)[3] == 0     # several tiles per expert


@pytest.mark.parametrize("T, E, d, f", [(8, 8, 4096, 8192), (7, 8, 4096, 8192), (64, 16, 2048, 14336), (64, 16, 1984, 14336), (192, 16, 4096, 2048)])
def test_workspace_of_few_rows_is_the_routes(T, E, d, f):
    """Room for y's partial sums: eight parts of 64 rows per expert in the few-row kernel, up to 256 tiles of 256 x 256 else;
    what does not fit the region of dA adds to the workspace."""
    need = lambda f: B.moe_workspace_bytes(B.make_cfg(T, d, f, E, 2, B.DTYPE_BF16, B.ACT_SWIGLU))
    dact = lambda f: 2 * (2 * T) * f * 2
    tiles = (2 * T // 160 + E) * -(-d // 256)
    sums = E * 8 * 64 * d * 4 if forward_rows(2 * T, E, d, f, True) == 64 else min(8 * tiles, 256) * 256 * 256 * 4
    assert need(f) - need(1984) == max(dact(f), sums) - dact(1984)     # 1984 columns: no split
