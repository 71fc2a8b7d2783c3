"""Edges of kernels and of the rules that pick them, against the CPU oracle: sizes around tiles, remainders and
the smallest and largest of a kernel's range."""
import numpy as np
import pytest

import oracle
import paper_2506_17255_amd as skl
import workloads as wk
from skl_harness import STAGED_ROUTES, GpuLayer, build_states_on_gpu, matmul_f64, rel_fro, staged_routes, worst_tile_rel_fro

pytestmark = pytest.mark.gpu


def hash_params(rng, d):
    return (2 * rng.integers(0, 1 << 23, size=d) + 1).astype(np.uint32), rng.integers(0, 1 << 24, size=d).astype(np.uint32)


@pytest.mark.parametrize("in_f,out_f,d,widths", [
    (2051, 264, 4, (8, 33)),         # eight channels per workgroup, the last one with three; whole 16-byte pieces
    (2048, 333, 3, (10,)),           # rows not aligned to 16 bytes
    (70, 1030, 2, (16, 64)),         # few channels: one per workgroup
    (515, 96, 8, (250, 3)),          # tables that leave room for fewer channels per workgroup
    (3, 65536, 2, (500,)),           # the most outputs a 32-bit key can number
    (3, 65544, 2, (500,)),           # one step beyond: 64-bit keys
    (2048, 96, 4, (512, 100)),       # the most LDS: eight channels' keys fill 64 KiB
    (5, 96, 4, (4096, 100)),         # the same with one channel per workgroup
    (16385, 256, 2, (8, 33)),        # many short rows: workgroups of 256 threads, offsets from the host
    (24577, 264, 3, (8, 33)),        # many rows
])
def test_row_sketch_construction(in_f, out_f, d, widths):
    """Bit-identical to the oracle's sequential update (integers: no tolerance)."""
    rng = np.random.default_rng(in_f + out_f)
    W = (rng.standard_normal((in_f, out_f)) * 0.02).astype(np.float16)
    W[:, ::3] = np.float16(0.0078125) * rng.choice(np.array([-1, 1], dtype=np.float16), size=W[:, ::3].shape)     # ties of both signs
    K = np.array([widths[j % len(widths)] for j in range(in_f)], dtype=np.uint32)
    A, C = hash_params(rng, d)
    got = build_states_on_gpu(W, 1, out_f, d, A, C, K)
    assert np.array_equal(got, oracle.update(W, 1, out_f, d, A, C, K).states)


def test_row_sketch_construction_of_more_channels_than_a_grid_holds_workgroups():
    """2^22 + 3 channels, one of them so wide that a workgroup has room for a single channel."""
    in_f, out_f = (1 << 22) + 3, 8
    rng = np.random.default_rng(22)
    W = rng.integers(0, 0x7C00, size=(in_f, out_f), dtype=np.uint16).view(np.float16)
    K = np.ones(in_f, dtype=np.uint32)
    K[7] = 16384
    A, C = hash_params(rng, 1)
    got = build_states_on_gpu(W, 1, out_f, 1, A, C, K)
    assert np.array_equal(got, oracle.update(W, 1, out_f, 1, A, C, K).states)


def row_layer(seed, in_f, out_f, d, widths):
    rng = np.random.default_rng(seed)
    W = (rng.standard_normal((in_f, out_f)) * 0.02).astype(np.float16)
    A, C = hash_params(rng, d)
    return oracle.update(W, 1, out_f, d, A, C, np.asarray(widths, dtype=np.uint32))


# float32 result of float32 sums of at most 2048 exact products: relative error below sqrt(2048) * 2^-24 = 2.7e-6
SUM_TOL = 2048**0.5 * 2.0**-24


@pytest.mark.parametrize("wide_share", [0.01, 0.3, 1.0])
@pytest.mark.parametrize("in_f,tokens,ldx_pad", [(1030, 17, 2), (1030, 300, 0), (264, 1, 0), (520, 257, 3)])
def test_activation_packing_of_the_staged_prefill(in_f, tokens, ldx_pad, wide_share):
    """Channels near each other (windows of X in LDS), scattered (fetched one by one) and in their own order; rows of
    X on 16-byte boundaries and not; token counts around the 16-token blocks and 256-token tiles."""
    rng = np.random.default_rng(in_f + tokens)
    sk = row_layer(5, in_f, 264, 3, np.where(rng.random(in_f) < wide_share, 20, 9))
    X = wk.f32_to_bf16_bits(rng.standard_normal((tokens, in_f)).astype(np.float32))
    ref = oracle.linear(oracle.query(sk), X, x_kind="bf16")
    with GpuLayer(sk, skl.FLAG_STAGED_PREFILL) as g:
        y = g.gemm(X, "bf16", "f32", ldx=in_f + ldx_pad)
    assert rel_fro(y, ref) <= SUM_TOL, rel_fro(y, ref)


@pytest.mark.parametrize("flags", [0, skl.FLAG_STAGED_PREFILL])
@pytest.mark.parametrize("in_f,tokens,ldx_pad", [(5, 33, 0), (7, 20, 2), (8, 17, 1), (513, 40, 0), (1029, 100, 6), (391, 16, 1)])
def test_activation_packing_of_odd_rows(in_f, tokens, ldx_pad, flags):
    """Rows of fewer than eight channels, and rows that end inside a 16-byte piece, on any 2-byte boundary; the last row of X
    ends where its buffer does."""
    rng = np.random.default_rng(in_f + tokens)
    sk = row_layer(6, in_f, 264, 3, np.where(rng.random(in_f) < 0.02, 20, 9))
    X = wk.f32_to_bf16_bits(rng.standard_normal((tokens, in_f)).astype(np.float32))
    ref = oracle.linear(oracle.query(sk), X, x_kind="bf16")
    with GpuLayer(sk, flags) as g:
        y = g.gemm(X, "bf16", "f32", ldx=in_f + ldx_pad)
    assert np.isfinite(y).all() and rel_fro(y, ref) <= SUM_TOL, rel_fro(y, ref)


@pytest.mark.parametrize("tokens", [1, 16, 17, 64, 65, 100, 128, 129])
@pytest.mark.parametrize("in_f,out_f,ldy_pad,y_dt", [
    # (staged) shares of fewer than eight blocks: one per tile, stored without partials; ragged outputs
    (256, 300, 0, "f32"),
    (1030, 264, 3, "bf16"),     # four shares per tile, rows of Y not on 16-byte boundaries, ragged last block
    (2048, 1024, 0, "f16"),     # eight shares per tile
    (520, 520, 8, "f32"),       # two shares of four and five blocks
])
def test_short_prompts(in_f, out_f, ldy_pad, y_dt, tokens):
    """Calls of at most 128 tokens, the way the library chooses (mostly one pass) and staged (tiles of 64 and of 128 tokens),
    against the fused kernel, which other calls of these layers may take, and the oracle; 129 tokens: the first call of the
    other rules."""
    rng = np.random.default_rng(in_f + out_f + tokens)
    sk = row_layer(6, in_f, out_f, 4, np.where(rng.random(in_f) < 0.02, 20, 9))
    X = wk.f32_to_bf16_bits(rng.standard_normal((tokens, in_f)).astype(np.float32))
    ref = oracle.linear(oracle.query(sk), X, x_kind="bf16")
    # one rounding of the result: half a unit of the last place, at most 2^-8 (bf16) and 2^-11 (f16) relative
    tol = {"f32": SUM_TOL, "f16": 2.0**-11, "bf16": 2.0**-8}[y_dt]
    with GpuLayer(sk) as g, GpuLayer(sk, skl.FLAG_FUSED_PREFILL) as f, GpuLayer(sk, skl.FLAG_STAGED_PREFILL) as st:
        assert g.info["prefill_kernel"] == skl.SKL_PREFILL_FUSED
        need, fused = (skl.sketch_linear_workspace_bytes(h.handle, 1, tokens) for h in (g, f))
        assert (need != fused) == (tokens <= 128)       # the way the call goes, told by the workspace it asks for
        y, other, staged = (h.gemm(X, "bf16", y_dt, ldy=out_f + ldy_pad) for h in (g, f, st))
        for h, v in ((g, y), (st, staged)):
            assert np.array_equal(v, h.gemm(X, "bf16", y_dt, ldy=out_f + ldy_pad))
    assert y.shape == ref.shape
    for v in (y, other, staged):
        assert rel_fro(v, ref) <= tol, rel_fro(v, ref)


@pytest.mark.parametrize("in_f,out_f,d,staged", [
    (15360, 8192, 2, True),     # 240 MiB of dense weights
    (15424, 8192, 2, False),    # 64 channels more
    (15424, 8192, 7, True),     # blocks of four words (seven rows leave no room for eight)
])
def test_short_prompts_of_layers_around_the_cache_size(in_f, out_f, d, staged):
    """Which way a short prompt goes, told by the workspace it asks for; the fused way is the fused kernel's bit for bit."""
    rng = np.random.default_rng(in_f + d)
    A, C = hash_params(rng, d)
    K = np.full(in_f, 4, dtype=np.uint32)
    states = (rng.standard_normal(in_f * d * 4) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, 1, out_f, d, A, C, K, states)
    X = wk.f32_to_bf16_bits(rng.standard_normal((20, in_f)).astype(np.float32))
    with GpuLayer(sk) as g, GpuLayer(sk, skl.FLAG_FUSED_PREFILL) as f:
        assert g.info["prefill_kernel"] == skl.SKL_PREFILL_FUSED
        need, fused = (skl.sketch_linear_workspace_bytes(h.handle, 1, 20) for h in (g, f))
        assert (need > in_f * out_f * 2) == staged and (need == fused) != staged
        y, other = (h.gemm(X, "bf16", "f32") for h in (g, f))
    assert rel_fro(y, other) <= (2 * in_f) ** 0.5 * 2.0**-24        # two float32 sums of in_f exact products each
    assert staged or np.array_equal(y, other)


@pytest.mark.parametrize("bits", [16, 4])
@pytest.mark.parametrize("tokens", [1, 64, 100, 128])
def test_short_prompts_in_a_workspace_of_the_fused_kernel(tokens, bits):
    """A workspace that holds the fused kernel's need but not the dense weights: the call is accepted, and is the fused
    kernel's bit for bit; one byte less is refused; the full need gives the staged result."""
    rng = np.random.default_rng(tokens + bits)
    sk = row_layer(8, 264, 776, 3, np.where(rng.random(264) < 0.02, 20, 9))
    if bits < 16:
        sk = oracle.quantize(sk, bits)
    X = wk.f32_to_bf16_bits(rng.standard_normal((tokens, 264)).astype(np.float32))
    with GpuLayer(sk) as g, GpuLayer(sk, skl.FLAG_FUSED_PREFILL) as f:
        need, fused = (skl.sketch_linear_workspace_bytes(h.handle, 1, tokens) for h in (g, f))
        assert fused < need
        want = f.gemm(X, "bf16", "f32")
        for n in (fused, need - 1):
            assert np.array_equal(g.gemm(X, "bf16", "f32", ws_bytes=n), want)
        assert np.array_equal(g.gemm(X, "bf16", "f32", ws_bytes=need), g.gemm(X, "bf16", "f32"))
        with pytest.raises(skl.SketchLinearError) as e:
            g.gemm(X, "bf16", "f32", ws_bytes=fused - 1)
        assert e.value.status == skl.SKL_ERR_BUFFER_TOO_SMALL


@pytest.mark.parametrize("in_f,out_f,d,widths,bits,tokens,x_dt,y_dt,ldy_pad", [
    (777, 3001, 4, (9, 24), 16, 1, "bf16", "f32", 0),               # ragged rows of Y, a last tile of few outputs
    (777, 3001, 4, (9, 24), 16, 16, "f16", "f16", 3),               # tiles of 32 tokens
    (777, 3001, 4, (9, 200, 330, 1000), 16, 17, "bf16", "bf16", 0),     # wide channels in blocks of four, two and one words
    (1030, 4000, 3, (9, 250), 16, 33, "bf16", "f32", 0),            # tiles of 64 tokens
    (777, 3001, 2, (9, 2000), 16, 64, "f16", "f32", 4),
    (777, 3001, 1, (9, 500), 16, 65, "bf16", "f32", 0),             # one row; tiles of 96 tokens
    (900, 3001, 5, (60, 90), 16, 96, "bf16", "bf16", 3),            # five rows: fewer gathers in flight
    (2048, 5001, 6, (40, 70), 16, 97, "f16", "f16", 0),             # tiles of 128 tokens
    (1500, 6000, 8, (30, 100), 16, 20, "bf16", "f32", 0),           # eight rows: blocks of four words
    (1500, 9000, 7, (1, 2), 16, 20, "bf16", "f32", 0),              # tables shorter than a copy
    (2048, 6050, 4, (33, 113), 16, 113, "bf16", "f32", 0),          # the largest eight-word table (65088 bytes)
    (900, 3001, 4, (9, 24), 8, 40, "bf16", "f32", 0),               # low-bit states: tables in the workspace
    (900, 1100, 3, (9, 24), 16, 129, "bf16", "f32", 0),             # two token tiles
    (900, 1100, 2, (9, 24), 4, 300, "bf16", "f16", 4),              # three
    (520, 777, 4, (9, 24), 16, 512, "f16", "f32", 0),               # four, all full
    (1100, 777, 4, (9, 24), 16, 500, "f16", "f32", 0),              # four, the last one ragged
])
def test_prompts_in_one_pass(in_f, out_f, d, widths, bits, tokens, x_dt, y_dt, ldy_pad):
    """Against the oracle and the staged kernel, twice bit for bit.  The way the call goes shows in the workspace (the weight
    words that the staged kernel would leave at its end are not written) or, where the workspace is the fused kernel's or ends
    in expanded tables, in sums that are neither that kernel's nor the staged one's to the last bit."""
    rng = np.random.default_rng(in_f + out_f + tokens)
    A, C = hash_params(rng, d)
    K = np.where(rng.random(in_f) < 0.03, rng.choice(widths[1:], in_f), widths[0]).astype(np.uint32)
    states = (rng.standard_normal(int(K.sum()) * d) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, 1, out_f, d, A, C, K, states)
    if bits < 16:
        sk = oracle.quantize(sk, bits)
    x = rng.standard_normal((tokens, in_f)).astype(np.float32)
    X = wk.f32_to_bf16_bits(x) if x_dt == "bf16" else x.astype(np.float16).view(np.uint16)
    W_hat = oracle.query(sk)
    ref = matmul_f64(W_hat, X if x_dt == "bf16" else X.view(np.float16), x_dt)
    # float32 sums of in_f exact products, then one rounding to the output type
    tol = SUM_TOL + {"f32": 0.0, "f16": 2.0**-11, "bf16": 2.0**-8}[y_dt]
    with GpuLayer(sk) as g, GpuLayer(sk, skl.FLAG_STAGED_PREFILL) as st, GpuLayer(sk, skl.FLAG_FUSED_PREFILL) as fu:
        ws, need = g.workspace(1, tokens)
        ws.fill_(0xA5)
        y = g.gemm(X, x_dt, y_dt, ldy=out_f + ldy_pad)
        if tokens <= 128 and bits == 16:
            assert bool((ws[need - 4096:need] == 0xA5).all())
        else:
            exact = g.gemm(X, x_dt, "f32")
            assert not np.array_equal(exact, st.gemm(X, x_dt, "f32"))
            # (512 tokens: two groups of blocks, as the fused kernel has two shares per tile, and the same sums)
            assert tokens == 512 or not np.array_equal(exact, fu.gemm(X, x_dt, "f32"))
        assert np.array_equal(y, g.gemm(X, x_dt, y_dt, ldy=out_f + ldy_pad))
        other = st.gemm(X, x_dt, y_dt, ldy=out_f + ldy_pad)
    for v in (y, other):
        assert np.isfinite(v.astype(np.float32)).all() and rel_fro(v, ref) <= tol, rel_fro(v, ref)


@pytest.mark.parametrize("query_mode", [0, 1])
@pytest.mark.parametrize("in_f,out_f,d,widths,tokens", [
    (777, 3001, 4, (9, 200, 330, 1000), 30),    # all widths of blocks, a group with one block of each: what a run of blocks
    (777, 3001, 3, (9, 250, 500, 1300), 60),    # begins with (products of nothing) and ends with, in every tile of tokens
    (777, 3001, 2, (9, 400, 800, 2000), 90),
    (777, 3001, 1, (9, 800, 1700, 4000), 120),
    (1500, 6000, 8, (30, 60, 100, 450), 20),
    (777, 3001, 4, (9, 200, 330, 1000), 40),    # tiles of three, five and seven 16-token blocks
    (777, 3001, 3, (9, 250, 500, 1300), 70),
    (777, 3001, 1, (9, 800, 1700, 4000), 105),
    (777, 3001, 8, (9, 100, 165, 500), 80),
    (777, 3001, 6, (9, 130, 220, 660), 97),
])
def test_one_pass_runs_of_blocks(in_f, out_f, d, widths, tokens, query_mode):
    """Runs of blocks of one width class begin with an empty pipeline and carry their last products over a barrier."""
    rng = np.random.default_rng(d + tokens)
    A, C = hash_params(rng, d)
    K = np.where(rng.random(in_f) < 0.06, rng.choice(widths[1:], in_f), widths[0]).astype(np.uint32)
    states = (rng.standard_normal(int(K.sum()) * d) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, 1, out_f, d, A, C, K, states)
    x = rng.standard_normal((tokens, in_f)).astype(np.float16).view(np.uint16)
    ref = matmul_f64(oracle.query(sk, query_mode), x.view(np.float16), "f16")
    with GpuLayer(sk, query_mode=query_mode) as g:
        ws, need = g.workspace(1, tokens)
        ws.fill_(0xA5)
        y = g.gemm(x, "f16", "f32")
        assert bool((ws[need - 4096:need] == 0xA5).all())       # (the staged kernel would leave weight words there)
    assert np.isfinite(y).all() and rel_fro(y, ref) <= SUM_TOL, rel_fro(y, ref)


@pytest.mark.parametrize("in_f,out_f,d,widths,tokens", [
    (688, 6104, 2, (95, 381), 465),         # whole tiles are faster than a pass over the tables per token tile
])
def test_prompts_that_stay_staged(in_f, out_f, d, widths, tokens):
    """Layers whose tables the fused kernel cannot hold, where one pass fits the workspace but is slower: the staged kernel's
    result bit for bit."""
    rng = np.random.default_rng(in_f + tokens)
    A, C = hash_params(rng, d)
    K = np.where(np.arange(in_f) % 100 == 7, widths[1], widths[0]).astype(np.uint32)
    sk = oracle.Sketch(in_f, out_f, 1, out_f, d, A, C, K, (rng.standard_normal(d * int(K.sum())) * 0.02).astype(np.float16).view(np.uint16))
    X = wk.f32_to_bf16_bits(rng.standard_normal((tokens, in_f)).astype(np.float32))
    with GpuLayer(sk) as g, GpuLayer(sk, skl.FLAG_STAGED_PREFILL) as st:
        assert np.array_equal(g.gemm(X, "bf16", "f32"), st.gemm(X, "bf16", "f32"))


@pytest.mark.parametrize("in_f,out_f,tokens,x_dt,y_dt,ldy_pad", [
    (64, 600, 300, "bf16", "f32", 0),           # fewer stages than the pipeline holds
    (264, 3001, 600, "bf16", "bf16", 0),        # rows of Y not on 16-byte boundaries, ragged last tile and token tile
    (200, 5700, 2000, "f16", "f16", 4),
    (128, 28672, 300, "bf16", "bf16", 0),
    (100, 20000, 520, "bf16", "f32", 0),
    (200, 8200, 2000, "bf16", "bf16", 0),
    (200, 11008, 2048, "bf16", "f32", 0),
    (200, 12000, 2048, "f16", "bf16", 8),
])
def test_whole_tiles_of_staged_prompts(in_f, out_f, tokens, x_dt, y_dt, ldy_pad):
    """Staged products of few channels and all element types, twice bit for bit, all outputs against a product in 64 bits.
    (Which way such calls go: test_ways_of_staged_prompts.)"""
    rng = np.random.default_rng(in_f + out_f + tokens)
    A, C = hash_params(rng, 3)
    K = np.where(rng.random(in_f) < 0.03, 24, 9).astype(np.uint32)
    sk = oracle.Sketch(in_f, out_f, 1, out_f, 3, A, C, K, (rng.standard_normal(3 * int(K.sum())) * 0.02).astype(np.float16).view(np.uint16))
    x = rng.standard_normal((tokens, in_f)).astype(np.float32)
    X = wk.f32_to_bf16_bits(x) if x_dt == "bf16" else x.astype(np.float16).view(np.uint16)
    ref = matmul_f64(oracle.query(sk), X if x_dt == "bf16" else X.view(np.float16), x_dt)
    tol = SUM_TOL + {"f32": 0.0, "f16": 2.0**-11, "bf16": 2.0**-8}[y_dt]
    with GpuLayer(sk, skl.FLAG_STAGED_PREFILL) as g:
        y = g.gemm(X, x_dt, y_dt, ldy=out_f + ldy_pad)
        assert np.array_equal(y, g.gemm(X, x_dt, y_dt, ldy=out_f + ldy_pad))
    assert np.isfinite(y).all() and worst_tile_rel_fro(y, ref) <= 2 * tol, worst_tile_rel_fro(y, ref)
    assert rel_fro(y, ref) <= tol, rel_fro(y, ref)


@pytest.mark.parametrize("in_f,out_f,tokens,n_wide,y_dt,ldy_pad,way", STAGED_ROUTES)
def test_ways_of_staged_prompts(in_f, out_f, tokens, n_wide, y_dt, ldy_pad, way, tmp_path):
    """Every way of a staged call over a dirty workspace: all outputs against a product in 64 bits, rounded no more than
    the sums of shared tiles are, whatever the way."""
    t = __import__("torch")
    rng = np.random.default_rng(in_f + out_f + tokens)
    A, C = hash_params(rng, 2)
    K = np.full(in_f, 9, dtype=np.uint32)
    K[in_f - n_wide:] = 36
    scale = np.where(np.arange(in_f) < in_f - n_wide, 0.02, 0.4).repeat(2 * K)
    order = rng.permutation(in_f)
    states = np.split((rng.standard_normal(scale.size) * scale).astype(np.float16).view(np.uint16), np.cumsum(2 * K)[:-1])
    sk = oracle.Sketch(in_f, out_f, 1, out_f, 2, A, C, K[order], np.concatenate([states[j] for j in order]))
    X = wk.f32_to_bf16_bits(rng.standard_normal((tokens, in_f)).astype(np.float32))
    (kind, cb, chains, measure), = staged_routes([(in_f, out_f, tokens, n_wide)], tmp_path)
    assert (kind, cb, chains) == way
    with GpuLayer(sk, skl.FLAG_STAGED_PREFILL) as g:
        ws, _ = g.workspace(1, tokens)
        ws.fill_(0xFF)
        y = t.from_numpy(g.gemm(X, "bf16", y_dt, ldy=out_f + ldy_pad)).cuda().double()
        ws.fill_(0xFF)
        again = t.from_numpy(g.gemm(X, "bf16", y_dt, ldy=out_f + ldy_pad)).cuda().double()
        ref = t.from_numpy(wk.bf16_bits_to_f32(X)).cuda().double() @ t.from_numpy(oracle.query(sk).view(np.float16)).cuda().double()
    assert bool((y == again).all()) and bool(t.isfinite(y).all())
    # the measure counts four roundings of the result, of up to 2^-25 each in root mean square; one more for the result itself,
    # then that to a shorter type
    tol = 2.0**-24 * (measure + 1) ** 0.5 + {"f32": 0.0, "f16": 2.0**-11, "bf16": 2.0**-8}[y_dt]
    err = float((y - ref).norm() / ref.norm())
    assert err <= tol, (err, tol)
    for t0 in range(0, tokens, 128):                            # no wrong tile hides in the norm of the whole
        d, r = (y - ref)[t0:t0 + 128], ref[t0:t0 + 128]
        pad = -out_f % 32
        d, r = (t.nn.functional.pad(v, (0, pad)).reshape(len(v), -1, 32).square().sum((0, 2)) for v in (d, r))
        assert float((d / r).max()) <= (2 * tol) ** 2, (t0, int((d / r).argmax()))


@pytest.mark.parametrize("batch", [1, 2, 4, 5, 16])
@pytest.mark.parametrize("in_f,out_f,tile_in,tile_out,d,one_launch_to", [
    (64, 24, 64, 24, 2, 16),         # the smallest rows of a group; the last 16 outputs of a group are eight
    (300, 70, 100, 35, 3, 16),       # rows and outputs of a group that fill no step; tables off 16-byte boundaries
    (63, 32, 63, 32, 2, 0),          # one row less than the one-launch kernel's lane groups: split
    (1024, 64, 128, 16, 4, 16),      # the most input rows
    (1088, 64, 64, 32, 4, 0),        # beyond: split
    (64, 2048, 64, 16, 2, 16),       # 512 workgroups at batch 16: one round
    (64, 2064, 64, 16, 2, 5),        # 516: split there
    (64, 8208, 64, 16, 2, 0),        # 513 workgroups and more: split at batch 1, too
    (1024, 32, 128, 16, 4, 1),       # (with the widths below) the most LDS at batch 1: tables, rows and sums fill 64 KiB
])
def test_small_group_decode(in_f, out_f, tile_in, tile_out, d, one_launch_to, batch):
    """2-D groups on both sides of the line between one launch (up to a batch of one_launch_to) and a split reduction,
    which alone writes to the workspace; groups of unequal width."""
    rng = np.random.default_rng(in_f + out_f + batch)
    W = (rng.standard_normal((in_f, out_f)) * 0.02).astype(np.float16)
    A, C = hash_params(rng, d)
    K = rng.integers(9, 200, size=(in_f // tile_in) * (out_f // tile_out)).astype(np.uint32)
    if (in_f, out_f, tile_in) == (1024, 32, 128):
        K[0] = (65536 - 4 * (1024 + 1024)) // 8 // (2 * d)
    sk = oracle.update(W, tile_in, tile_out, d, A, C, K)
    x = rng.standard_normal((batch, in_f)).astype(np.float16)
    ref = oracle.linear(oracle.query(sk), x)
    with GpuLayer(sk) as g:
        ws, _ = g.workspace(0, batch)
        ws.fill_(0xA5)
        y = g.gemv(x, "f32")
        assert bool((ws == 0xA5).all()) == (batch <= one_launch_to)
    assert rel_fro(y, ref) <= SUM_TOL, rel_fro(y, ref)


@pytest.mark.parametrize("d,widths", [
    (1, (255, 257, 256, 4095, 4096, 4097, 8191, 8192, 9003, 1, 8, 300)),        # lengths around the batches, any alignment
    (2, (128, 129, 2048, 2049, 4096, 4100, 5, 4, 2047, 700, 1024, 4095)),
    (3, (85, 86, 683, 1366, 2731, 1365, 2730, 3, 2733, 99, 682, 101)),
])
def test_table_staging_of_2d_groups(d, widths):
    """Tables that start on boundaries of 16, 4 and 2 bytes and end inside a piece: weights bit for bit, then the
    other kernels that stage them."""
    for n_in, n_out in ((192, 256), (768, 64)):
        rng = np.random.default_rng(d + n_in)
        W = (rng.standard_normal((n_in, n_out)) * 0.02).astype(np.float16)
        A, C = hash_params(rng, d)
        sk = oracle.update(W, 64, 64, d, A, C, np.asarray(widths, dtype=np.uint32))
        W_hat = oracle.query(sk)
        x = rng.standard_normal((70, n_in)).astype(np.float16)
        ref = oracle.linear(W_hat, x)
        with GpuLayer(sk) as g:
            assert np.array_equal(g.reconstruct(), W_hat)
            for batch in (1, 5):
                assert rel_fro(g.gemv(x[:batch], "f32"), ref[:batch]) <= SUM_TOL
            assert rel_fro(g.gemm(x.view(np.uint16), "f16", "f32"), ref) <= SUM_TOL


@pytest.mark.parametrize("batch", [2, 5, 16])
@pytest.mark.parametrize("in_f,out_f", [(520, 260), (520, 261), (520, 262), (520, 1027),
                                         (520, 12287), (520, 12288), (520, 12289),      # batch 16: 7.1 MB past the caches, but for the last
                                         (2048, 4098), (2048, 4100)])                   # batch 16: 6.3 MB, past them only where rows are not aligned
def test_batched_decode_stores(in_f, out_f, batch):
    """Rows of partial sums on 16-byte boundaries and not, a last unit of a few outputs; stores through the caches and,
    where a call leaves megabytes of them, past."""
    rng = np.random.default_rng(out_f + batch)
    sk = row_layer(7, in_f, out_f, 4, np.where(rng.random(in_f) < 0.02, 40, 17))
    x = rng.standard_normal((batch, in_f)).astype(np.float16)
    ref = oracle.linear(oracle.query(sk), x)
    with GpuLayer(sk) as g:
        y = g.gemv(x, "f32")
    assert rel_fro(y, ref) <= SUM_TOL, rel_fro(y, ref)


@pytest.mark.parametrize("query_mode", [0, 1])
@pytest.mark.parametrize("in_f,out_f,tile_in,tile_out,d,widths,tokens,x_dt,y_dt,ldx_pad", [
    (256, 256, 128, 128, 2, (200, 333), 17, "f16", "f16", 0),       # two tables, tiles of 32 tokens
    (8, 16, 8, 16, 1, (3, 3), 1, "bf16", "f32", 0),                 # one lane group of one step
    (72, 96, 24, 48, 3, (7, 20), 33, "f16", "f32", 3),              # steps that span groups and end short; odd rows of X
    (1032, 160, 8, 16, 4, (1, 5), 65, "bf16", "bf16", 1),           # a table per eight rows, more than fit the wavefronts
    (640, 512, 128, 128, 3, (170, 171), 129, "bf16", "f32", 0),     # two tiles of tokens, sixteen wavefronts
    (512, 4096, 256, 256, 3, (682, 683), 130, "f16", "f32", 0),     # 32 outputs per tile, tables on odd addresses
    (2048, 64, 256, 64, 8, (1500, 1600), 40, "f16", "f16", 0),      # tables that do not all fit at once
    (160, 4096, 32, 32, 2, (20, 21), 520, "f16", "f32", 0),         # 640 workgroups of four wavefronts
    (136, 8192, 8, 32, 1, (2, 3), 1040, "bf16", "f32", 0),          # 2304 of one
    (64, 2048, 64, 64, 3, (90, 91), 300, "f16", "f32", 0),          # few rows, many outputs: tiles of 64 x 64
])
def test_group_prompts(in_f, out_f, tile_in, tile_out, d, widths, tokens, x_dt, y_dt, ldx_pad, query_mode):
    """The kernel for groups of whole lanes and output blocks, at its edges, against the oracle in 64 bits."""
    rng = np.random.default_rng(in_f + out_f + tokens)
    A, C = hash_params(rng, d)
    K = rng.choice(widths, (in_f // tile_in) * (out_f // tile_out)).astype(np.uint32)
    states = (rng.standard_normal(int(K.sum()) * d) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, tile_in, tile_out, d, A, C, K, states)
    x = rng.standard_normal((tokens, in_f)).astype(np.float32)
    X = wk.f32_to_bf16_bits(x) if x_dt == "bf16" else x.astype(np.float16).view(np.uint16)
    ref = matmul_f64(oracle.query(sk, query_mode), X if x_dt == "bf16" else X.view(np.float16), x_dt)
    with GpuLayer(sk, query_mode=query_mode) as g:
        y = g.gemm(X, x_dt, y_dt, ldx=in_f + ldx_pad, ldy=out_f + 3)
        assert np.array_equal(y, g.gemm(X, x_dt, y_dt, ldx=in_f + ldx_pad, ldy=out_f + 3))
    tol = SUM_TOL + {"f32": 0.0, "f16": 2.0**-11, "bf16": 2.0**-8}[y_dt]
    assert np.isfinite(y.astype(np.float32)).all() and rel_fro(y, ref) <= tol, rel_fro(y, ref)


@pytest.mark.parametrize("in_f,out_f,tile_in,tile_out,d,widths,tokens", [
    (1024, 2048, 8, 16, 1, (155, 160), 1040),       # 40 KB of tables to a workgroup: four of them on a compute unit, two wavefronts each
    (16, 512, 16, 512, 2, (250, 256), 8200),        # few rows, few sketch rows and many results: tiles of 64 x 64
    (64, 1088, 32, 64, 4, (40, 41), 4100),          # more sketch rows: 64 x 1088 of them no longer
])
def test_group_prompts_of_many_results(in_f, out_f, tile_in, tile_out, d, widths, tokens):
    rng = np.random.default_rng(in_f + tokens)
    A, C = hash_params(rng, d)
    K = rng.choice(widths, (in_f // tile_in) * (out_f // tile_out)).astype(np.uint32)
    states = (rng.standard_normal(int(K.sum()) * d) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, tile_in, tile_out, d, A, C, K, states)
    X = wk.f32_to_bf16_bits(rng.standard_normal((tokens, in_f)).astype(np.float32))
    ref = matmul_f64(oracle.query(sk), X, "bf16")
    with GpuLayer(sk) as g:
        y = g.gemm(X, "bf16", "f32")
    assert np.isfinite(y).all() and worst_tile_rel_fro(y, ref) <= SUM_TOL, worst_tile_rel_fro(y, ref)


@pytest.mark.parametrize("query_mode", [0, 1])
@pytest.mark.parametrize("in_f,out_f,tile_in,tile_out,d,widths,batch,one_launch", [
    (512, 128, 32, 16, 3, (9, 20), 2, True),        # the fewest rows, input rows and outputs that take the prompt kernel
    (512, 112, 32, 16, 3, (9, 20), 2, False),       # fewer outputs: partial sums
    (520, 16384, 8, 16, 2, (2, 3), 16, True),       # 32 outputs per tile do not fit the groups
    (1024, 512, 256, 256, 4, (300, 301), 5, True),
    (504, 144, 72, 16, 3, (9, 20), 16, True),       # fewer rows: the small kernel, which takes groups of at least 64
    (1100, 520, 20, 40, 2, (9, 20), 3, False),      # groups that are no whole lanes: partial sums
    (2048, 512, 256, 256, 2, (99, 300), 2, True),   # more rows than 1024: by estimate
    (2048, 512, 64, 64, 4, (30, 31), 2, False),
])
def test_group_decode_of_several_rows(in_f, out_f, tile_in, tile_out, d, widths, batch, one_launch, query_mode):
    rng = np.random.default_rng(in_f + out_f)
    A, C = hash_params(rng, d)
    K = rng.choice(widths, (in_f // tile_in) * (out_f // tile_out)).astype(np.uint32)
    states = (rng.standard_normal(int(K.sum()) * d) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, tile_in, tile_out, d, A, C, K, states)
    x = rng.standard_normal((batch, in_f)).astype(np.float16)
    ref = matmul_f64(oracle.query(sk, query_mode), x, "f16")
    with GpuLayer(sk, query_mode=query_mode) as g:
        ws, need = g.workspace(0, batch)
        ws.fill_(0xA5)
        y = g.gemv(x, "f32", ldy=out_f + 1)
        assert bool((ws[:need] == 0xA5).all()) == one_launch
        assert np.array_equal(y, g.gemv(x, "f32", ldx=in_f + 8))
    assert np.isfinite(y).all() and rel_fro(y, ref) <= SUM_TOL, rel_fro(y, ref)


@pytest.mark.parametrize("in_f,out_f,tile_in,tile_out,d,K,batch,one_launch", [
    (1024, 512, 256, 512, 5, 3276, 4, False),       # tables of 32 KB, one at a time by one wavefront: partial sums
    (944, 256, 16, 256, 8, 16, 3, False),           # 59 tables above an output and eight sketch rows
    (2048, 256, 16, 64, 1, 8, 2, True),             # 128 tables, but 256 partial sums per output in the split form
    (640, 512, 64, 128, 2, 128, 16, True),          # ten small ones
    (1024, 1024, 128, 128, 3, 170, 9, True),
])
def test_group_decode_of_several_rows_by_tables(in_f, out_f, tile_in, tile_out, d, K, batch, one_launch):
    """Both sides of the rule that prices the tables above an output; only the split form writes to the workspace."""
    rng = np.random.default_rng(in_f + out_f)
    A, C = hash_params(rng, d)
    n = (in_f // tile_in) * (out_f // tile_out)
    states = (rng.standard_normal(n * K * d) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, tile_in, tile_out, d, A, C, np.full(n, K, dtype=np.uint32), states)
    x = rng.standard_normal((batch, in_f)).astype(np.float16)
    ref = matmul_f64(oracle.query(sk), x, "f16")
    with GpuLayer(sk) as g:
        ws, need = g.workspace(0, batch)
        ws.fill_(0xA5)
        y = g.gemv(x, "f32")
        assert bool((ws[:need] == 0xA5).all()) == one_launch
    assert np.isfinite(y).all() and rel_fro(y, ref) <= SUM_TOL, rel_fro(y, ref)


@pytest.mark.parametrize("query_mode", [0, 1])
@pytest.mark.parametrize("in_f,out_f,d,widths,batch", [
    (777, 1500, 4, (9, 200, 330, 1300), 1),     # blocks of all widths, some groups with one table buffer, some of one block
    (2000, 333, 3, (9, 250, 500, 1800), 1),
    (300, 1200, 1, (3, 1200, 1700, 4060), 1),
    (520, 14300, 2, (9, 400, 900, 2500), 1),    # segments of more than 12 wavefronts
    (150, 9000, 4, (500, 700, 1100), 1),        # two units per wavefront, the last one without outputs
    (900, 1100, 5, (9, 200), 1),
    (900, 1100, 8, (9, 120, 450), 1),
    (777, 1500, 4, (9, 200, 330, 1300), 2),
    (777, 1500, 4, (9, 200, 330, 1300), 9),     # the second eight rows: one of them
    (2000, 333, 3, (9, 250, 500, 1800), 5),
    (520, 2100, 2, (9, 400, 900, 2500), 16),
    (300, 1200, 1, (3, 1200, 1700, 4060), 8),
    (900, 1100, 5, (9, 200), 7),                # more than four rows: nothing in flight across the blocks
    (900, 1100, 8, (9, 120, 450), 12),
])
def test_decode_runs_of_blocks(in_f, out_f, d, widths, batch, query_mode):
    """Runs of blocks of one width class begin with an empty pipeline and carry their last products over a barrier; rows past
    the batch hold whatever LDS held."""
    rng = np.random.default_rng(in_f + d + batch)
    A, C = hash_params(rng, d)
    K = np.where(rng.random(in_f) < 0.06, rng.choice(widths[1:], in_f), widths[0]).astype(np.uint32)
    states = (rng.standard_normal(int(K.sum()) * d) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, 1, out_f, d, A, C, K, states)
    x = rng.standard_normal((batch, in_f)).astype(np.float16)
    ref = matmul_f64(oracle.query(sk, query_mode), x, "f16")
    with GpuLayer(sk, query_mode=query_mode) as g:
        y = g.gemv(x, "f32")
        assert np.array_equal(y, g.gemv(x, "f32", ldx=in_f + 8))
    assert np.isfinite(y).all() and rel_fro(y, ref) <= SUM_TOL, rel_fro(y, ref)


@pytest.mark.parametrize("query_mode", [0, 1])
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("in_f,out_f,d,widths", [
    (777, 1500, 4, (9, 200, 330, 1300)),        # blocks of all widths
    (300, 700, 1, (3, 1200, 1700, 4060)),
    (900, 600, 8, (9, 120, 450)),
    (50, 900, 4, (700, 1500)),                  # eight blocks with a large table among them: 8-bit codes are expanded by a launch of their own
    (90, 900, 4, (700, 1500)),                  # more blocks
])
def test_staged_prompts_expand_codes_in_either_query_mode(in_f, out_f, d, widths, bits, query_mode):
    """The rebuild launch expands codes while it stages a table: zeros of either sign included (a negative code with scale 0 stands
    for -0, which the signed maximum ranks below +0)."""
    rng = np.random.default_rng(in_f + bits)
    A, C = hash_params(rng, d)
    K = np.where(rng.random(in_f) < 0.1, rng.choice(widths[1:], in_f), widths[0]).astype(np.uint32)
    qmax = 127 if bits == 8 else 7
    codes = rng.integers(-qmax, qmax + 1, size=int(K.sum()) * d).astype(np.int8)
    scales = (rng.random(in_f * d) * 0.1).astype(np.float16)
    scales[rng.random(in_f * d) < 0.2] = 0
    scales = scales.view(np.uint16)
    states = oracle.dequantize_states(in_f, out_f, 1, out_f, d, K, bits, codes, scales)
    q = oracle.QuantSketch(in_f, out_f, 1, out_f, d, A, C, K, states, bits=bits, codes=codes, scales=scales)
    X = wk.f32_to_bf16_bits(rng.standard_normal((600, in_f)).astype(np.float32))
    ref = matmul_f64(oracle.query(q, query_mode), X, "bf16")
    with GpuLayer(q, skl.FLAG_STAGED_PREFILL, query_mode) as g:
        for tokens in (40, 200, 600):
            y = g.gemm(X[:tokens], "bf16", "f32")
            assert np.isfinite(y).all() and worst_tile_rel_fro(y, ref[:tokens]) <= SUM_TOL, tokens
        # a call that multiplies by one puts the rebuilt weights out: bit for bit, but for the sign of a zero
        ones = np.zeros((64, in_f), dtype=np.uint16)
        rows = rng.choice(in_f, 64, replace=in_f < 64)
        ones[np.arange(64), rows] = 0x3F80
        w = oracle.query(q, query_mode).view(np.float16).astype(np.float32)[rows]
        assert np.array_equal(g.gemm(ones, "bf16", "f32"), w)


@pytest.mark.parametrize("in_f,out_f,d,K", [
    (32768, 4096, 1, 2),        # tables of 288 bytes in the only buffer, groups of 1024 channels
    (65536, 2048, 4, 1),        # 576 bytes
])
def test_batched_decode_through_tables_smaller_than_a_chunk(in_f, out_f, d, K):
    """A table is copied in whole chunks of 1 KiB; the activations behind the table area stay what they are."""
    rng = np.random.default_rng(in_f)
    A, C = hash_params(rng, d)
    states = (rng.standard_normal(in_f * d * K) * 0.02).astype(np.float16).view(np.uint16)
    sk = oracle.Sketch(in_f, out_f, 1, out_f, d, A, C, np.full(in_f, K, dtype=np.uint32), states)
    x = rng.standard_normal((16, in_f)).astype(np.float16)
    W_hat = oracle.query(sk)
    ref = np.vstack([matmul_f64(W_hat[j:j + 4096], x[:, j:j + 4096], "f16")[None] for j in range(0, in_f, 4096)]).sum(axis=0)
    with GpuLayer(sk) as g:
        for batch in (2, 9, 16):
            y = g.gemv(x[:batch], "f32")
            # (a row at a time: one wrong row of sixteen must not hide among the others)
            assert max(rel_fro(y[b], ref[b]) for b in range(batch)) <= SUM_TOL, batch


@pytest.mark.parametrize("out_f,batch,ldh_pad,h_dt", [
    (4096, 15, 0, "f32"),       # 240 wavefronts of the row reduction: the other one
    (4096, 16, 0, "f16"),       # 256: the first
    (4097, 16, 3, "f32"),       # partial sums and rows of h on 4-byte boundaries, one output in the last piece
    (4098, 16, 2, "f16"),
    (16390, 4, 2, "f32"),       # 65 x 4; rows of h on 16-byte boundaries, a last piece of two outputs
])
def test_gate_up_reductions(out_f, batch, ldh_pad, h_dt):
    """Both reductions of the gate/up pair around the line between them; layers with unlike numbers of block groups."""
    t = __import__("torch")
    rng = np.random.default_rng(out_f + batch)
    x = rng.standard_normal((batch, 200)).astype(np.float16)
    A, C = hash_params(rng, 2)
    skg, sku = (oracle.Sketch(200, out_f, 1, out_f, 2, A, C, K, (rng.standard_normal(2 * int(K.sum())) * 0.02).astype(np.float16).view(np.uint16))
                for K in (np.full(200, 9, dtype=np.uint32), rng.integers(2, 40, size=200).astype(np.uint32)))
    ref = oracle.gate_up(oracle.linear(oracle.query(skg), x), oracle.linear(oracle.query(sku), x))
    with GpuLayer(skg) as g, GpuLayer(sku) as u:
        xd = t.from_numpy(x.view(np.int16)).cuda()
        h = t.full((batch, out_f + ldh_pad), float("nan"), dtype={"f32": t.float32, "f16": t.float16}[h_dt], device="cuda")
        ws = t.empty(skl.sketch_linear_gemv_group_workspace_bytes([g.handle, u.handle], batch), dtype=t.uint8, device="cuda")
        skl.sketch_linear_gemv_gate_up(g.handle, u.handle, xd.data_ptr(), skl.SKL_F16, 200, h.data_ptr(),
                                       {"f32": skl.SKL_F32, "f16": skl.SKL_F16}[h_dt], out_f + ldh_pad, batch, ws.data_ptr(), ws.numel(), g.stream())
        got = h.float().cpu().numpy()
    assert np.isnan(got[:, out_f:]).all()
    # SiLU and the product pass the sums' relative errors on at most doubled, expf adds a few units of the last place
    tol = 4 * SUM_TOL + (2.0**-11 if h_dt == "f16" else 0.0)
    assert rel_fro(got[:, :out_f], ref) <= tol, rel_fro(got[:, :out_f], ref)
