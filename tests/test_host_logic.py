"""Host logic of the library, without a GPU: the weight re-layout against the documented tile order written
out independently in numpy, and invariants of the GEMM launch shapes over the shapes of every configuration."""
import numpy as np
import pytest

import bild_inputs as bi
from paper_2302_07863_amd import binding as b


def _bf16_bits(x):
    u = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) & 0xFFFF).astype(np.uint16)


def _expected_tiles(w_n_by_k, dtype):
    """Tile order from its description: tiles of 16 features x KT inputs, 1 KiB each, feature blocks outermost and
    tiles of a block contiguous along the inputs; lane l of a tile owns feature l % 16 and KT/4 consecutive inputs
    starting at (l // 16) * KT/4."""
    n, k = w_n_by_k.shape
    kt = 32 if dtype == bi.DT_BF16 else 16
    per = kt // 4
    tn = (n + 15) // 16
    padded = np.zeros((tn * 16, k), dtype=np.float32)
    padded[:n] = w_n_by_k
    t = padded.reshape(tn, 16, k // kt, 4, per)          # [block, feature, k tile, lane group, j]
    t = t.transpose(0, 2, 3, 1, 4)                          # [block, k tile, lane group, feature, j] = lanes in order
    flat = np.ascontiguousarray(t).reshape(-1)
    return _bf16_bits(flat).view(np.uint8) if dtype == bi.DT_BF16 else flat.view(np.uint8)


@pytest.mark.parametrize("dtype", [bi.DT_F32, bi.DT_BF16])
@pytest.mark.parametrize("n,k", [(16, 32), (40, 96), (200, 64), (33, 160)])
def test_tile_matrix_matches_the_documented_order(dtype, n, k):
    rng = np.random.default_rng(n * 1000 + k)
    w = rng.normal(size=(n, k)).astype(np.float32)
    want = _expected_tiles(w, dtype)
    assert np.array_equal(b.tile_matrix(w, False, dtype), want)
    assert np.array_equal(b.tile_matrix(np.ascontiguousarray(w.T), True, dtype), want)      # math layout [k][n]
    assert len(want) == ((n + 15) // 16) * (k // (32 if dtype == bi.DT_BF16 else 16)) * 1024


def _projections(shape):
    d, i, f = shape.d, shape.inner, shape.d_ff
    out = [(3 * i, d, False, False), (i, d, False, False), (d, i, False, False), (f, d, shape.gated, False),
           (d, f, False, False), (shape.vocab, d, False, True)]
    if shape.cross:
        out.append((2 * i, d, False, False))
    return out


@pytest.mark.parametrize("pair", sorted(bi.PAIRS))
def test_gemm_launch_shapes_are_consistent(pair):
    """Every projection of every configuration, for 1..32 rows and for row-block launches: the waves of a workgroup
    factor into input slices x feature groups, the feature-group workgroups cover every feature tile exactly once,
    the LDS request fits, and the staged chunk is a whole number of input tiles."""
    cfg = bi.PAIRS[pair]()
    for shape in (cfg.small, cfg.large):
        kt = 32 if shape.dtype == bi.DT_BF16 else 16
        for n, k, gated, head in _projections(shape):
            for rows in (1, 2, 3, 4, 7, 11, 16, 17, 32) + (() if head else (33, 512, 1000)):
                s = b.gemm_shape(n, k, rows, gated, head, shape.dtype)
                tiles = ((2 * n if gated else n) + 15) // 16
                if rows > 512:
                    # the dense-tile kernel: 64 rows x (4 waves x 4 feature tiles) per workgroup, chunks of 128 inputs
                    assert (s["wk"], s["nwv"], s["rw"], s["kc"]) == (1, 4, 4, 128)
                    assert (s["blocks"] - 1) * 16 < tiles <= s["blocks"] * 16 and s["row_blocks"] == (rows + 63) // 64
                    assert 2 * s["lds"] <= s["lds_limit"]          # two workgroups share a compute unit (registers)
                    continue
                assert s["nwv"] in (1, 2, 4, 8) and s["nwv"] % s["wk"] == 0, (n, k, rows, s)
                assert s["wk"] in (1, 2, 4, 8), (n, k, rows, s)   # the kernels cut the wave index by shifts
                # feature tiles per wave: 2 = gate and linear branch; 4 only for a very wide LM head at up to 16 rows
                assert s["rw"] == (2 if gated else (4 if head and rows <= 16 and tiles >= 8192 else 1))
                per_wg = (s["nwv"] // s["wk"]) * s["rw"]
                assert (s["blocks"] - 1) * per_wg < tiles <= s["blocks"] * per_wg, (n, k, rows, s)
                assert s["row_blocks"] == (rows + 31) // 32
                assert 0 < s["lds"] <= s["lds_limit"], (n, k, rows, s)
                assert s["kc"] % kt == 0 and s["kc"] >= kt
                assert s["wk"] <= max(1, min(s["kc"], k) // kt)


@pytest.mark.parametrize("pair", sorted(bi.PAIRS))
def test_attention_launch_shapes_are_consistent(pair):
    """Key splits stay within the partial buffers and the grid the kernels assume; partials are left to the consumer
    projection only in the range it merges (at most 8 splits and 16 rows, one (row, head) pair per thread of a 256-thread
    workgroup, a weight table of at most 4 KiB); the LDS request fits; a workgroup
    that is not split further streams at most about 160 KiB unless the split limits are exhausted."""
    cfg = bi.PAIRS[pair]()
    for shape in (cfg.small, cfg.large):
        esz = 2 if shape.dtype == bi.DT_BF16 else 4
        for nkeys in (1, 31, 64, 128, 512, 1024, 2048, 4096):
            for rows in (1, 2, 4, 5, 8, 9, 11, 16, 32, 33, 700):
                for max_splits in (8, 16, 64):
                    s = b.attn_shape(shape.heads, shape.d_head, rows, nkeys, max_splits, shape.dtype)
                    assert 1 <= s["splits"] <= max_splits and shape.heads * s["splits"] <= max(512, shape.heads)
                    assert s["splits"] & (s["splits"] - 1) == 0
                    if rows > 32:
                        assert s["splits"] == 1
                    if s["defer"]:
                        assert 1 < s["splits"] <= 8 and rows <= 16 and rows * shape.heads <= 256
                        assert rows * shape.heads * s["splits"] * 4 <= 4096
                    assert s["waves"] in (1, 2, 4, 8) and 0 < s["lds"] <= 128 * 1024
                    if min(rows, 32) <= 16 and shape.d_head <= 64:
                        assert s["waves"] >= 4      # q is staged in one piece per thread from 256 threads on
                    per_wg = nkeys * shape.d_head * 2 * esz / s["splits"]
                    if per_wg > 160 * 1024 and rows <= 32 and not s["defer"]:
                        assert s["splits"] * 2 > max_splits or shape.heads * s["splits"] * 2 > 512


def test_launch_shape_rules_at_their_boundaries():
    """The measured thresholds of the GEMM launch shapes: eight-wave workgroups once a thread of a four-wave workgroup
    would stage more than eight pieces (rows x inputs > 8192); single-row launches never field between one and two
    workgroups per compute unit; a very wide LM head takes four feature tiles per wave up to 16 rows."""
    assert b.gemm_shape(1024, 1024, 8)["nwv"] == 4 and b.gemm_shape(1024, 1024, 9)["nwv"] == 8
    assert b.gemm_shape(512, 512, 16)["nwv"] == 4 and b.gemm_shape(512, 512, 17)["nwv"] == 8
    one, two = b.gemm_shape(12288, 4096, 1), b.gemm_shape(12288, 4096, 2)
    assert one["blocks"] == 768 and one["nwv"] == 2 and two["blocks"] == 384 and two["nwv"] == 4
    for n, k in ((1024, 1024), (3072, 1024), (4096, 1024), (1024, 4096), (12288, 4096), (22016, 4096), (4096, 11008)):
        blocks = b.gemm_shape(n, k, 1)["blocks"]
        assert not 256 < blocks < 512, (n, k, blocks)
    wide = b.gemm_shape(250112, 512, 1, False, True)
    assert wide["rw"] == 4 and wide["blocks"] * wide["nwv"] * 4 >= 250112 // 16
    assert b.gemm_shape(250112, 512, 17, False, True)["rw"] == 1
    assert b.gemm_shape(32128, 1024, 1, False, True)["rw"] == 1


def test_debug_calls_reject_bad_arguments():
    lib = b.lib()
    assert lib.bild_debug_tiled_bytes(0, 32, 0) == b.EINVAL
    assert lib.bild_debug_tiled_bytes(16, 40, 1) == b.EINVAL
    assert lib.bild_debug_gemm_shape(16, 32, 0, 0, 0, 0, None) == b.EINVAL


def test_launch_shapes_of_ragged_widths_keep_a_power_of_two_of_input_slices():
    """Widths whose tile count is not a power of two (96 inputs = 6 fp32 tiles, 160 = 10) in row-block launches: the
    kernels split the wave index into (input slice, feature group) by shifts, so the slices must be a power of two."""
    for dtype, kt in ((bi.DT_F32, 16), (bi.DT_BF16, 32)):
        for k in (96, 160, 192, 320, 6 * kt, 10 * kt, 12 * kt):
            for n in (48, 96, 288, 1000, 4096):
                for rows in (1, 3, 16, 33, 40, 300):
                    s = b.gemm_shape(n, k, rows, False, False, dtype)
                    assert s["wk"] in (1, 2, 4, 8) and s["nwv"] in (1, 2, 4, 8) and s["nwv"] % s["wk"] == 0, (n, k, rows, s)
                    assert s["wk"] <= max(1, min(s["kc"], k) // kt), (n, k, rows, s)


@pytest.mark.parametrize("heads,d_head", [(32, 128), (16, 64), (16, 128)])
def test_caches_past_32_bit_offsets_stay_with_64_bit_addresses(heads, d_head):
    """Keys of a layer lie [position][heads * d_head] in bf16: the kernels with 32-bit offsets take a cache below 2 GiB only."""
    last = (1 << 31) // (heads * d_head * 2) - 1
    if heads * d_head == 4096:
        assert last == 262143
    for positions in (32, 8192, last):
        for nkeys in (64, positions):
            s = b.cache_rule(heads, d_head, positions, nkeys)
            assert s["one_kernel"] == 1 and 1 <= s["splits"] <= 16 and s["waves"] in (4, 8), (positions, s)
    for positions in (last + 1, last + 33, 2 * (last + 1), 4 * (last + 1)):
        for nkeys in (64, positions):
            assert b.cache_rule(heads, d_head, positions, nkeys) == dict(one_kernel=0, splits=0, waves=0), positions


@pytest.mark.parametrize("units", [64, 96, 128, 144, 160, 191, 192, 256, 304])
def test_every_tile_of_a_wide_pass_has_a_workgroup(units):
    """Passes of wide models in one kernel, for whole and partitioned cards: where such a pass is taken at all, the workgroups from the
    first with a part of q, k, v (the FFN's input, a head) on hold all of it, at every length around the lines of the rule."""
    taken = 0
    for d, heads in ((1280, 10), (1536, 12), (1536, 6), (2048, 16), (2048, 8), (2560, 20), (3072, 24), (4096, 32)):
        for d_ff, gated in ((96, False), (d, True), (4096, True), (5632, True), (4 * d, False), (11008, True)):
            for keys in (1, 256, 257, 1024, 1280, 1281, 2000, 2048, 2304, 2305, 8192):
                s = b.wide_split(d, heads, d_ff, gated, units, keys)
                if not s["qkv_tiles"]:
                    assert not any(s.values())
                    continue
                taken += 1
                case = (d, heads, d_ff, gated, keys, s)
                assert s["qkv_first"] >= 0 and (units - s["qkv_first"]) * s["qkv_tiles"] >= 3 * heads * 128 // 16, case
                assert s["ffn_first"] >= 0 and (units - s["ffn_first"]) * s["ffn_tiles"] >= (d_ff // 8 if gated else d_ff // 16), case
                assert s["heads_first"] >= 0 and s["heads_first"] + heads * s["ranges"] <= units and s["ranges"] in (1, 2, 4, 8), case
                assert d // 16 <= units
    assert taken > 0 or units < 96


def test_tiles_of_a_wide_pass_at_the_lines_of_the_rule():
    """Three tiles of q, k, v a workgroup up to 1280 keys, then two where all of them have a workgroup, above 2304 keys only if none of those has a
    head as well."""
    tiles = lambda d, heads, units: [b.wide_split(d, heads, 5632, True, units, keys)["qkv_tiles"] for keys in (1280, 1281, 2304, 2305, 8192)]
    assert tiles(2048, 16, 256) == [3, 2, 2, 3, 3] and tiles(2048, 16, 191) == [3, 3, 3, 3, 3]
    assert tiles(1280, 10, 256) == [3, 2, 2, 2, 2] and tiles(4096, 32, 256) == [3] * 5 and tiles(2560, 20, 256) == [3] * 5


ONE_ROUND = {(96, 256): (768, 4096), (96, 192): (32, 1024), (48, 128): (32, 32)}  # least inputs, and with rotary positions


@pytest.mark.parametrize("n,k,gated,rotary", [(768, 3072, 0, 0), (5632, 1024, 1, 0), (3072, 1024, 0, 0), (4096, 1024, 0, 0), (1024, 4096, 0, 0), (4096, 4096, 0, 0), (6144, 2048, 0, 1),
                                              (12288, 4096, 0, 1), (22016, 4096, 1, 0), (4096, 11008, 0, 0), (3072, 640, 0, 1), (4608, 384, 0, 0), (3072, 768, 0, 0)])
def test_tile_shapes_of_one_round_make_one_on_every_die(n, k, gated, rotary):
    """Launch shapes that pay where each compute unit has one workgroup: no die has more than its 32, and enough inputs for their epilogue."""
    seen = set()
    for rows in range(33, 2049):
        s = b.tile_shape(n, k, rows, bool(gated), bool(rotary))
        shape = (s["rows"], s["features"])
        if shape in ONE_ROUND:
            seen.add(shape)
            assert s["busiest"] <= 32, (rows, s)
            assert k >= ONE_ROUND[shape][rotary], (rows, s)
    want = {(768, 3072): {(48, 128)}, (3072, 1024): {(96, 256), (96, 192)}, (12288, 4096): set(ONE_ROUND), (22016, 4096): {(48, 128)}, (6144, 2048): {(96, 192)},
            (3072, 640): set(), (4608, 384): {(96, 192)}, (4096, 4096): {(96, 256), (48, 128)}}
    if (n, k) in want:
        assert seen == want[n, k]


@pytest.mark.parametrize("d,heads,d_ff,gated,most", [
    # where one kernel took 0.7 to 0.95 times as long as the separate ones
    (1536, 12, 6912, 0, 16), (1792, 13, 9248, 0, 16), (1536, 6, 8192, 1, 16), (2048, 16, 8192, 1, 16), (2048, 8, 7968, 1, 16), (2304, 18, 6912, 0, 16), (2560, 20, 6016, 1, 16), (3328, 26, 4384, 1, 16),
    (3328, 13, 9824, 0, 16), (3584, 14, 8544, 1, 16), (3840, 30, 4896, 1, 16), (4096, 32, 5120, 0, 24), (4096, 32, 6016, 1, 24), (4096, 32, 8224, 1, 32), (4096, 16, 8704, 0, 32), (4096, 32, 11008, 1, 32),
    # and 1.03 to 1.25 times
    (2048, 16, 5632, 1, 8), (2048, 16, 8224, 1, 8), (2048, 16, 8192, 0, 8), (2304, 18, 2304, 0, 8), (2304, 9, 4608, 0, 8), (2560, 10, 3328, 0, 8), (2560, 20, 3648, 0, 8), (3072, 24, 3008, 1, 8), (3328, 13, 2176, 1, 8),
    (4096, 32, 4096, 0, 8), (4096, 16, 2048, 1, 8)])
def test_rows_of_wide_passes_in_one_kernel(d, heads, d_ff, gated, most):
    """Passes of nine rows and more are one kernel only where the hidden state and the heads are wide enough for the model, and up to a number of keys that depends on the rows."""
    one = lambda rows, keys: b.wide_split(d, heads, d_ff, bool(gated), 256, keys, rows)["qkv_tiles"] > 0
    nine = 9 if d >= 2048 or gated or d_ff >= 7680 else 10
    assert [r for r in range(1, 33) if one(r, 100)] == [r for r in range(1, most + 1) if r != 9 or nine == 9]
    wide = 8192 if d >= 2048 else 6656
    limits = {8: 8192, nine: wide if nine == 9 else 6656, 16: 8192 if d_ff >= 8192 else wide, 17: 4096 if d_ff > 8192 else 1280 if gated else 2048, 25: 2048}
    for rows, keys in limits.items():
        assert one(rows, keys) == (rows <= most), rows
        assert not one(rows, keys + 1) or rows == 8


@pytest.mark.parametrize("dtype,d,vocab,rows,want", [
    # fp32: wider than 2048 only against short workgroups that do not fit twice, of matrices above the last-level cache's half
    (bi.DT_F32, 2112, 60000, (1, 4, 9, 16), "short"), (bi.DT_F32, 3072, 32000, (9, 10, 12, 16), "short"), (bi.DT_F32, 3456, 60000, (1, 8, 9), "short"), (bi.DT_F32, 3840, 46000, (1, 8, 10, 16), "short"),
    (bi.DT_F32, 3840, 12000, (10, 16), "sweep"), (bi.DT_F32, 4096, 16000, (1, 8, 9), "short"), (bi.DT_F32, 4096, 32000, (1, 4, 9), "short"), (bi.DT_F32, 4096, 32000, (10, 16), "sweep"), (bi.DT_F32, 4096, 50000, (5, 8), "sweep"),
    (bi.DT_F32, 1280, 60000, (1, 9), "short"), (bi.DT_F32, 1280, 90000, (17, 32), "short"), (bi.DT_F32, 1536, 128000, (17, 24), "short"), (bi.DT_F32, 2048, 32000, (2, 4), "short"), (bi.DT_F32, 2048, 50000, (1, 9, 32), "sweep"),
    (bi.DT_F32, 1024, 50000, (1, 32), "sweep"), (bi.DT_F32, 256, 50000, (1,), "short"), (bi.DT_F32, 256, 50000, (2, 32), "sweep"), (bi.DT_F32, 2112, 4000, (17, 32), "short"),
    # bf16: wider than 2048 from five rows on as tile planes, but for nine rows of 4096 inputs of which the short workgroups fit twice
    (bi.DT_BF16, 4096, 32000, (9,), "short"), (bi.DT_BF16, 4096, 32000, (5, 8, 10, 32), "planes"), (bi.DT_BF16, 4096, 64000, (9,), "short"), (bi.DT_BF16, 4096, 24000, (9,), "planes"), (bi.DT_BF16, 4096, 1000, (5, 8), "short"), (bi.DT_BF16, 4096, 1000, (9,), "planes"),
    (bi.DT_BF16, 7424, 24000, (5,), "short"), (bi.DT_BF16, 5312, 24000, (7,), "planes"), (bi.DT_BF16, 3072, 32000, (12,), "planes"), (bi.DT_BF16, 2048, 32000, (9, 32), "sweep"), (bi.DT_BF16, 512, 32128, (1,), "short")])
def test_kernels_of_the_head(dtype, d, vocab, rows, want):
    """Which kernels have the head of bild_head_stats, at sizes where one of them is clearly the slower one."""
    assert {r: b.head_route(d, vocab, r, dtype) for r in rows} == dict.fromkeys(rows, want)


@pytest.mark.parametrize("units", [144, 256, 304])
def test_every_tile_of_a_wide_pass_of_many_rows_has_a_workgroup(units):
    """The same above eight rows; above sixteen a head is twice as many workgroups'."""
    taken = {}
    for d, heads in ((1536, 12), (1536, 6), (2560, 20), (3072, 24), (4096, 32), (4096, 16)):
        for d_ff, gated in ((4096, True), (5632, True), (8192, False), (4 * d, False), (11008, True)):
            for keys, rows in [(k, r) for k in (1, 256, 257, 1024, 1280, 1281, 2000, 2048, 2304, 2305, 4096, 8192) for r in (9, 16, 17, 32)]:
                s = b.wide_split(d, heads, d_ff, gated, units, keys, rows)
                if not s["qkv_tiles"]:
                    assert not any(s.values())
                    continue
                taken[rows] = taken.get(rows, 0) + 1
                case = (d, heads, d_ff, gated, keys, rows, s)
                assert s["qkv_first"] >= 0 and (units - s["qkv_first"]) * s["qkv_tiles"] >= 3 * heads * 128 // 16, case
                assert s["ffn_first"] >= 0 and (units - s["ffn_first"]) * s["ffn_tiles"] >= (d_ff // 8 if gated else d_ff // 16), case
                assert s["heads_first"] >= 0 and s["heads_first"] + heads * (2 if rows > 16 else 1) * s["ranges"] <= units and s["ranges"] in (1, 2, 4, 8), case
    assert set(taken) == ({9, 16, 17, 32} if units >= 256 else {9, 16}), taken
