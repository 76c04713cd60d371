"""Branches of the launch rules (how many rows, keys or columns a workgroup takes, by the size of the problem): each at the
sizes where it can go wrong, against the oracle.  The forms that a rule chooses by cost are asked of the library and asserted,
so that a size that a changed rule sends elsewhere fails instead of testing another form.  Tolerances: REL_TOL for bf16 outputs; 1e-4 for 32-bit sums of
exponentials, whose argument, below 32 in magnitude, is rounded to 2^-19 at most twice (2 * 2^-19 * ln 2 = 2.6e-6 of a
weight) before a sum of up to 192 positive terms (192 * 2^-24 = 1.1e-5)."""
import ctypes
import math

import numpy as np
import pytest
import torch

import synth_inputs as si
import parity as recipes
from parity import REL_TOL, rel_err

pytestmark = pytest.mark.gpu

DEV = "cuda"
SUM_TOL = 1e-4


@pytest.fixture(scope="module")
def cm():
    import paper_2506_03275_amd as cm
    cm.load()
    return cm


def _attn_form(cm, H, N, E, c, with_list):
    """(rows of a whole chunk's workgroup, chunks taken whole, chunks in parts), pieces of the column-sum pass"""
    out = (ctypes.c_int32 * 4)()
    cm.load().chipmunk_internal_attn_form(1, H, N, E, c, int(with_list), out)
    return tuple(out[:3]), out[3]


def _attn_part_form(cm, H, N, E, c, k):
    """how the chunks in parts are walked: 0 a workgroup per 64 rows, 1 the same with two waves to a row, 2 those per 32 rows,
    -1 there are none; k: a list's columns, 0 without one"""
    return cm.load().chipmunk_internal_attn_part_form(1, H, N, E, c, k, int(k > 0))


def _mlp_form(cm, B, N, D, F, c, k=1, a_ld=None):
    """first and second dense GEMM on 256 x 256 tiles, delta with 256 neurons per workgroup; scores: pieces, sums, or (0, 0):
    the kernel for few chunks"""
    out = (ctypes.c_int32 * 5)()
    cm.load().chipmunk_internal_mlp_form(B, N, D, F, c, k, a_ld or -(-N // 8) * 8, out)
    return [bool(v) for v in out[:3]], tuple(out[3:])


def _mlp_tiles(cm, B, N, D, F, c, k, a_ld=None):
    """dense: form of the first GEMM (0 a chunk's tiles, 1 large, 2 of 64 x 64), of the second (the same) and tiles per XCD taken
    whole; then the delta's"""
    out = (ctypes.c_int64 * 6)()
    cm.load().chipmunk_internal_mlp_tiles(B, N, D, F, c, k, a_ld or -(-N // 8) * 8, out)
    return list(out)


def _u8(nbytes):
    return torch.empty(max(int(nbytes), 16), dtype=torch.uint8, device=DEV)


@pytest.mark.parametrize("E", [64, 128])
@pytest.mark.parametrize("B,H,N,c,apart", [(1, 20, 700, 192, True), (2, 8, 640, 128, True), (1, 27, 640, 192, False),
                                           (1, 20, 639, 192, False), (2, 7, 1031, 128, False), (1, 15, 1536, 192, True),
                                           (1, 15, 1535, 192, False), (1, 11, 2101, 192, False)])
def test_refresh_in_one_kernel_and_apart(cm, oracle, B, H, N, E, c, apart):
    """Both sides of the rule, statistics updated in place.  Apart, the sums and the output are those of the two entry points
    that make them alone, bit by bit; the one kernel's are rounded differently."""
    assert bool(cm.load().chipmunk_internal_attn_refresh_apart(B, H, N, c)) == apart
    (q1, k1, _), (q2, k2, v), _ = si.attn_steps(B, H, N, E, 38, DEV)
    scale, NB, ld = 1 / math.sqrt(E), -(-N // c), -(-N // 4) * 4 + 4
    m_ref, l_ref = oracle.attn_row_stats(si.np_f32(q1), si.np_f32(k1), scale)
    m, l = (torch.from_numpy(t.astype(np.float32)).to(DEV) for t in (m_ref, l_ref))
    m0, l0 = m.clone(), l.clone()
    out, D = torch.empty_like(q2), torch.full((B, H, NB, ld), -1.0, dtype=torch.float32, device=DEV)
    cm.attn_dense_colsum_stale(q2, k2, v, out, m, l, D, c, scale, m, l)
    qn, kn, vn = si.np_f32(q2), si.np_f32(k2), si.np_f32(v)
    ref = oracle.attn_colsum_stale(qn, kn, m0.cpu().numpy().astype(np.float64), l0.cpu().numpy().astype(np.float64), c, scale)
    assert rel_err(D[..., :N].cpu().numpy().astype(np.float64), ref) <= SUM_TOL
    assert bool((D[..., N:] == -1.0).all())
    assert rel_err(si.np_f32(out), oracle.attn_dense(qn, kn, vn, c, scale)) <= REL_TOL
    m_ref, l_ref = oracle.attn_row_stats(qn, kn, scale)
    lse = m.cpu().numpy().astype(np.float64) + np.log(l.cpu().numpy().astype(np.float64))
    assert np.abs(lse - (m_ref + np.log(l_ref))).max() <= 2e-3
    D_alone, out_alone = torch.full_like(D, -1.0), torch.empty_like(out)
    cm.attn_colsum_stale(q2, k2, m0, l0, D_alone, c, scale)
    cm.attn_dense(q2, k2, v, out_alone, None, c, scale, None)
    assert torch.equal(D, D_alone) == apart
    if apart:
        assert torch.equal(out, out_alone)


@pytest.mark.parametrize("N,E,c,pieces", [(1, 128, 192, 1), (64, 64, 128, 1), (130, 128, 192, 1), (511, 64, 192, 2),
                                          (513, 128, 128, 2), (1100, 128, 192, 4), (2113, 64, 128, 8), (2113, 128, 192, 8)])
def test_column_sums_in_pieces_of_the_keys(cm, oracle, N, E, c, pieces):
    """The column-sum pass cuts a chunk's keys into 1 to 8 runs of 64-key tiles, the last tile ragged or not."""
    assert _attn_form(cm, 1, N, E, c, False)[1] == pieces
    (q, k, _), _, _ = si.attn_steps(1, 1, N, E, 21, DEV)
    scale, NB, ld = 1 / math.sqrt(E), -(-N // c), -(-N // 4) * 4 + 4
    m_ref, l_ref = oracle.attn_row_stats(si.np_f32(q), si.np_f32(k), scale)
    m = torch.from_numpy(m_ref.astype(np.float32) - 0.25).to(DEV)
    l = torch.from_numpy(l_ref.astype(np.float32) * 1.5).to(DEV)
    D = torch.full((1, 1, NB, ld), -1.0, dtype=torch.float32, device=DEV)
    cm.attn_colsum_stale(q, k, m, l, D, c, scale)
    ref = oracle.attn_colsum_stale(si.np_f32(q), si.np_f32(k), m.cpu().numpy().astype(np.float64),
                                   l.cpu().numpy().astype(np.float64), c, scale)
    got = D.cpu().numpy()
    assert rel_err(got[..., :N].astype(np.float64), ref) <= SUM_TOL
    assert (got[..., N:] == -1.0).all()


@pytest.mark.parametrize("E", [64, 128])
@pytest.mark.parametrize("H,N,form,part", [
    (2, 1, (192, 0, 2), 0), (50, 130, (192, 0, 50), 0), (3, 130, (192, 0, 3), 2),    # all in parts of 64 rows, or of 32
    (200, 256, (128, 400, 0), -1), (400, 65, (128, 400, 0), -1), (400, 192, (192, 400, 0), -1),   # all whole
    (520, 190, (192, 512, 8), 2), (530, 129, (192, 512, 18), 2), (560, 190, (192, 512, 48), 0),   # the last round in parts
    (200, 190, None, -1)])                                                           # another form for each E
def test_dense_attention_in_workgroups_of_64_128_and_192_rows(cm, oracle, E, H, N, form, part):
    """Without a list a workgroup takes one, two or three blocks of 64 rows, by the number of workgroups, those of the last
    round one (or two waves half of one each) where that is cheaper; c is 128 here and 192 there, which no longer decides
    it.  The ends of the sequence leave waves and whole blocks without rows."""
    assert _attn_form(cm, H, N, E, 128 if N % 2 else 192, False)[0] == (form or {64: (128, 400, 0), 128: (192, 200, 0)}[E])
    assert _attn_part_form(cm, H, N, E, 128 if N % 2 else 192, 0) == part
    q, k, v = recipes.attn_inputs(1, H, N, E, 22, DEV)
    scale = 1 / math.sqrt(E)
    c = 128 if N % 2 else 192
    out, base = torch.full_like(q, 7.0), recipes.attn_base(tuple(q.shape), N, "unit", 22, DEV)
    cm.attn_sparse_delta(q, k, v, None, None, base, out, c, scale, -1.0)
    basen = si.np_f32(base).astype(np.float64)
    dense = oracle.attn_dense(si.np_f32(q), si.np_f32(k), si.np_f32(v), c, scale)
    assert rel_err(si.np_f32(out), basen - dense, dense) <= REL_TOL


@pytest.mark.parametrize("H,N,E,c,k,form,part", [
    (1, 193, 128, 192, 70, (0, 2), 0), (2, 650, 64, 192, 33, (0, 8), 0), (2, 300, 128, 128, 129, (0, 6), 2),   # all in parts
    (22, 300, 128, 128, 129, (0, 66), 0),
    (110, 320, 64, 128, 20, (330, 0), -1), (200, 384, 128, 192, 9, (400, 0), -1),                              # all whole
    (200, 500, 128, 192, 70, (512, 88), 0), (260, 300, 128, 192, 40, (512, 8), 0), (520, 129, 64, 128, 65, (1024, 16), 0)])
def test_column_lists_walked_by_parts_of_a_chunk(cm, oracle, H, N, E, c, k, form, part):
    """Few chunks: a workgroup per 64 rows or per 32, all of a chunk walking its one list; the last chunk ends before its last
    part.  Then cases with enough chunks to be walked whole, and cases whose last round alone is in parts."""
    assert _attn_form(cm, H, N, E, c, True)[0] == (c, *form) and _attn_part_form(cm, H, N, E, c, k) == part
    q, kk, v = recipes.attn_inputs(1, H, N, E, 23, DEV)
    scale, NB = 1 / math.sqrt(E), -(-N // c)
    base = recipes.attn_base(tuple(q.shape), k, "delta", 23, DEV)
    idx, counts = recipes.attn_indices(H * NB, N, k, 23, DEV, ragged=True)
    idx, counts = idx.view(1, H, NB, k), counts.view(1, H, NB)
    out = torch.full_like(q, 7.0)
    cm.attn_sparse_delta(q, kk, v, idx, counts, base, out, c, scale, 1.0)
    basen = si.np_f32(base).astype(np.float64)
    ref = oracle.attn_sparse_delta(si.np_f32(q), si.np_f32(kk), si.np_f32(v), idx.cpu().numpy(), counts.cpu().numpy(),
                                   basen, c, scale, 1.0)
    assert rel_err(si.np_f32(out), ref, ref - basen) <= REL_TOL
    cm.attn_sparse_delta(q, kk, v, idx, counts, base, base, c, scale, 1.0)      # in place
    assert torch.equal(base, out)


@pytest.mark.parametrize("B,N,D,F,c,act,bias,large", [
    (1, 977, 128, 31808, 192, 1, True, (True, False)),   # first GEMM on 256 x 256 tiles: two steps, neurons and tokens ragged
    (2, 509, 256, 16320, 192, 0, False, (True, False)),   # two batches, no bias
    (1, 4090, 3968, 640, 192, 0, True, (False, True)),    # second GEMM: ten steps, half a tile of columns missing, tokens ragged
    (1, 28660, 4096, 64, 192, 1, False, (False, True)),   # one step
    (2, 2041, 3968, 384, 192, 1, True, (False, True)),
])
def test_dense_mlp_on_large_tiles(cm, oracle, B, N, D, F, c, act, bias, large):
    """The dense GEMMs whose problem is large enough for 256 x 256 tiles; the cache cells past N stay as they are."""
    assert tuple(_mlp_form(cm, B, N, D, F, c, a_ld=-(-N // 8) * 8 + 8)[0][:2]) == large
    x, _, w1, b1, w2, b2 = recipes.mlp_inputs(B, N, D, F, 24, DEV)
    if not bias:
        b1, b2 = torch.zeros_like(b1), torch.zeros_like(b2)
    a_ld = -(-N // 8) * 8 + 8
    out = torch.empty_like(x)
    a_cache = torch.full((B, F, a_ld), 3.0, dtype=torch.bfloat16, device=DEV)
    cm.mlp_dense(x, w1, b1 if bias else None, w2, b2 if bias else None, out, a_cache, c, act)
    ref, a_ref, _ = oracle.mlp_dense(si.np_f32(x), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), si.np_f32(b2), c, act, a_ld=a_ld)
    assert rel_err(si.np_f32(a_cache)[..., :N], a_ref[..., :N]) <= REL_TOL
    assert torch.all(a_cache[..., N:] == 3.0)
    assert rel_err(si.np_f32(out), ref) <= REL_TOL


@pytest.mark.parametrize("C", [1, 3, 255, 257, 1024, 1025, 2049, 3073, 4096, 5121, 7168, 7169, 8192, 8193, 10241, 12288, 12289, 14336, 14337])
@pytest.mark.parametrize("kind", ["normal", "constant", "two_values", "few_ulps", "spikes", "wide"])
def test_topk_of_rows_kept_in_registers(cm, oracle, C, kind):
    """Both sides of every limit between the instances, on scores that halving the range of keys
    finds easy and on scores that it does not: one value, two, a range of a few ulps around a power of two, a few spikes
    over zeros of both signs, scores of both signs and all exponents with infinities.  Bit-exact, ties to the lower column."""
    rng = np.random.default_rng([25, C])
    R, ld = 3, -(-C // 4) * 4
    if kind == "normal": a = rng.standard_normal((R, C))
    elif kind == "constant": a = np.full((R, C), -3.25)
    elif kind == "two_values": a = rng.choice([1.0, 2.0], size=(R, C))
    elif kind == "few_ulps": a = 1.0 + 2.0 ** -23 * rng.integers(-3, 4, size=(R, C))
    elif kind == "spikes":
        a = rng.choice([0.0, -0.0], size=(R, C))
        a[:, rng.integers(0, C, 5)] = rng.random(5)
    else:
        a = rng.standard_normal((R, C)) * 2.0 ** rng.integers(-140, 120, size=(R, C))
        a[:, ::97], a[:, 5::131] = np.inf, -np.inf
    a = a.astype(np.float32)
    b = rng.standard_normal((R, C)).astype(np.float32)
    cur, prev = (torch.full((R, ld), float("inf"), dtype=torch.float32, device=DEV) for _ in range(2))   # padding is never picked
    cur[:, :C], prev[:, :C] = torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV)
    for k in sorted({1, -(-C // 14), C // 2, C} - {0}):
        for p in (None, b) if kind != "wide" else (None,):
            idx = torch.full((R, k + 1), -7, dtype=torch.int32, device=DEV)
            counts = torch.full((R,), -7, dtype=torch.int32, device=DEV)
            cm.topk_cols(cur[:, :C], None if p is None else prev[:, :C], k, idx, counts)
            ref_idx, ref_counts = oracle.topk_cols(a, p, k, k_stride=k + 1, idx_fill=-7)
            assert np.array_equal(idx.cpu().numpy(), ref_idx), k
            assert np.array_equal(counts.cpu().numpy(), ref_counts)


@pytest.mark.parametrize("C", [14592, 14593, 16383, 16384, 16385, 20480, 20481, 24575, 24576, 24577])
@pytest.mark.parametrize("kind", ["normal", "constant", "two_values", "few_ulps", "wide"])
def test_topk_of_rows_kept_in_more_registers(cm, oracle, C, kind):
    """Eight units of a wave, and sixteen waves, which take a row only where a third of it is kept."""
    test_topk_of_rows_kept_in_registers(cm, oracle, C, kind)


@pytest.mark.parametrize("C", [1024, 4000, 12288, 16384])
@pytest.mark.parametrize("equal", [2, 300])
def test_topk_of_ties_on_the_threshold(cm, oracle, C, equal):
    """A few and many columns that equal the threshold, of which none but one, all but one and all are taken."""
    rng = np.random.default_rng([27, C])
    a = np.stack([rng.permutation(C) for _ in range(3)]).astype(np.float32)
    above = C // 3                                          # columns above the shared score
    a[(a >= C - above - equal) & (a < C - above)] = C - above - 1
    cur = torch.from_numpy(a).to(DEV)
    for k in (above, above + 1, above + equal - 1, above + equal, above + equal + 1):
        idx = torch.full((3, k), -7, dtype=torch.int32, device=DEV)
        counts = torch.full((3,), -7, dtype=torch.int32, device=DEV)
        cm.topk_cols(cur, None, k, idx, counts)
        ref_idx, _ = oracle.topk_cols(a, None, k, k_stride=k, idx_fill=-7)
        assert np.array_equal(idx.cpu().numpy(), ref_idx), k


@pytest.mark.parametrize("B,N,D,F,c,plan", [
    (1, 1, 4864, 64, 128, (16, 2)),          # one token, one neuron tile half full, 76 steps in sixteen pieces
    (1, 49 * 128 - 60, 512, 64, 128, (8, 2)),   # eight pieces of one step
    (1, 9500, 640, 7680, 192, (4, 2)),       # ten steps in four pieces
    (1, 9500, 640, 12224, 192, (5, 1)),      # in five, one sum each, the last of 256 neurons' tiles three quarters full
    (1, 129 * 128 - 1, 512, 8576, 128, (3, 1)),   # 129 chunks, eight steps in three pieces, one sum each, the last tile half full
    (1, 127 * 128, 128, 320, 128, (1, 2)),   # 127, 128 and 129 chunks: both sides of a tile
    (2, 64 * 192, 256, 576, 192, (1, 2)),
    (1, 128 * 128 + 5, 384, 64, 128, (1, 2)),
    (1, 128 * 128 + 5, 512, 16960, 128, (1, 2)),   # eight steps, one piece in two sums, many neuron tiles
    (2, 1400, 3968, 10304, 192, (4, 2)),     # 62 steps in four pieces, two sums each, the last neuron tile half full
])
def test_neuron_scores_in_pieces_of_the_contraction(cm, oracle, B, N, D, F, c, plan):
    """Chunk means of full, ragged and one-row chunks, and the scores GEMM's pieces and sums.  Tolerance: the mean enters as two
    bf16 numbers (2^-16 of it is lost at most), the 32-bit sums of D products add less: 1e-4 of the scores' RMS."""
    assert _mlp_form(cm, B, N, D, F, c)[1] == plan
    g = si.generator(26, DEV)
    x, w1 = si.randn_bf16((B, N, D), g), si.randn_bf16((F, D), g, 1 / math.sqrt(D))
    T = torch.full((B, -(-N // c), F), float("nan"), dtype=torch.float32, device=DEV)
    cm.mlp_tile_mean_preact(x, w1, T, c, _u8(cm.mlp_tile_mean_workspace_bytes(B, N, D, F, c)))
    ref = oracle.mlp_tile_scores(si.np_f32(x), si.np_f32(w1), c)
    assert rel_err(T.cpu().numpy(), ref) <= SUM_TOL
    again = torch.empty_like(T)
    cm.mlp_tile_mean_preact_static(x, w1, again, c)
    assert rel_err(again.cpu().numpy(), ref) <= SUM_TOL


@pytest.mark.parametrize("E", [64, 128])
@pytest.mark.parametrize("H,N,c,form,part", [(2, 900, 192, (0, 10), 2), (2, 600, 128, (0, 10), 2), (9, 900, 192, (0, 45), 0),
                                             (14, 600, 128, (0, 70), 0), (100, 700, 192, (400, 0), -1), (80, 600, 128, (400, 0), -1)])
def test_last_step_of_column_lists(cm, oracle, E, H, N, c, form, part):
    """Lists that end at, before and behind the edges of tiles (32 columns) and steps (64), one step to three, in either half
    of the buffers: the last step leaves out an empty second tile and brings the base rows (ragged last chunk: some do
    not exist).  Chunks in parts of 32 rows and of 64, and chunks walked whole: two or three blocks of rows per wave."""
    NB, k = -(-N // c), 193
    assert _attn_form(cm, H, N, E, c, True)[0] == (c, *form) and _attn_part_form(cm, H, N, E, c, k) == part
    q, kk, v = recipes.attn_inputs(1, H, N, E, 27, DEV)
    base = recipes.attn_base(tuple(q.shape), 64, "delta", 27, DEV)
    idx, counts = recipes.attn_indices(H * NB, N, k, 27, DEV)
    edges = torch.tensor([1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 192, 193], dtype=torch.int32)
    counts = edges[torch.arange(H * NB) % len(edges)].to(DEV)
    idx, counts = idx.view(1, H, NB, k), counts.view(1, H, NB)
    out = torch.full_like(q, 7.0)
    scale = 1 / math.sqrt(E)
    cm.attn_sparse_delta(q, kk, v, idx, counts, base, out, c, scale, 1.0)
    basen = si.np_f32(base).astype(np.float64)
    ref = oracle.attn_sparse_delta(si.np_f32(q), si.np_f32(kk), si.np_f32(v), idx.cpu().numpy(), counts.cpu().numpy(),
                                   basen, c, scale, 1.0)
    assert rel_err(si.np_f32(out), ref, ref - basen) <= REL_TOL


@pytest.mark.parametrize("B,N,D,F,c,k,act,bias", [
    (1, 700, 1536, 8256, 192, 8194, 1, True), (1, 900, 512, 8192, 128, 8130, 0, False), (1, 192, 640, 42560, 192, 42560, 1, True),
    (2, 700, 1536, 8192, 192, 8130, 0, False), (2, 440, 512, 8192, 128, 8130, 1, True)])
def test_mlp_delta_with_256_neurons_per_workgroup(cm, oracle, B, N, D, F, c, k, act, bias):
    """The first GEMM of the MLP delta on its wide tiles (few chunks, many neurons): counts that end in a tile's first half, in
    its second, at its edge, at nothing; a ragged last chunk, one batch and two; both forms of the cache write-back, bit for
    bit alike.  The caches hold noise, which the delta takes as it takes activations."""
    assert _mlp_form(cm, B, N, D, F, c, k)[0][2]
    _, x2, w1, b1, w2, _ = recipes.mlp_inputs(B, N, D, F, 28, DEV)
    if not bias:
        b1 = torch.zeros_like(b1)
    NB, a_ld = -(-N // c), -(-N // 8) * 8 + 8
    g = si.generator(28, DEV)
    a_cache, o_cache = si.randn_bf16((B, F, a_ld), g, 0.5), si.randn_bf16((B, N, D), g)
    o_ref, a_ref = (si.np_f32(t).astype(np.float64) for t in (o_cache, a_cache))
    o_before, a_before = o_ref.copy(), a_cache.clone()
    idx, _ = recipes.mlp_indices(B * NB, F, k, 28, DEV)
    counts = torch.tensor([k, 0, 256, 300, 129, 1, 512, k - 1][:B * NB], dtype=torch.int32, device=DEV)
    idx, counts = idx.view(B, NB, k), counts.view(B, NB)
    o2, a2 = o_cache.clone(), a_cache.clone()
    bias1 = b1 if bias else None
    cm.mlp_sparse_delta(x2, w1, bias1, w2, idx, counts, a_cache, o_cache, c, act, _u8(cm.mlp_workspace_bytes(B, N, D, F, c, k)))
    cm.mlp_sparse_delta_overlapped(x2, w1, bias1, w2, idx, counts, a2, o2, c, act, _u8(cm.mlp_overlapped_workspace_bytes(B, N, D, F, c, k)))
    assert torch.equal(a_cache, a2) and torch.equal(o_cache, o2)
    oracle.mlp_sparse_delta(si.np_f32(x2), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), idx.cpu().numpy(), counts.cpu().numpy(),
                            a_ref, o_ref, c, act)
    assert rel_err(si.np_f32(a_cache)[..., :N], a_ref[..., :N]) <= REL_TOL
    assert rel_err(si.np_f32(o_cache), o_ref, o_ref - o_before) <= REL_TOL
    assert torch.equal(a_cache[..., N:], a_before[..., N:])


@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("B,N,D,F,c,k,large,wide", [
    (1, 1021, 256, 16320, 128, 16300, True, True), (1, 1021, 256, 16320, 128, 1000, True, False),
    (1, 841, 512, 12928, 192, 12886, True, True), (2, 2000, 1536, 4096, 192, 500, True, False),
    (2, 440, 512, 8192, 128, 8130, False, True), (1, 300, 768, 2048, 192, 300, False, False),
    (2, 440, 512, 1024, 128, 1024, False, False)])
def test_unchanged_input_leaves_the_caches_alone(cm, B, N, D, F, c, k, large, wide, act):
    """The delta of an input that has not changed is nothing, bit for bit, whichever tiles filled the cache (256 x 256 or 192 or
    128 x 128) and whichever the delta takes (256 neurons or 128): their products (16x16x32 and 32x32x16) add in the same
    order.  So a chunk's results do not hang on how many chunks a call has."""
    form = _mlp_form(cm, B, N, D, F, c, k)[0]
    assert (form[0], form[2]) == (large, wide)
    x, _, w1, b1, w2, b2 = recipes.mlp_inputs(B, N, D, F, 30, DEV)
    out = torch.empty_like(x)
    a_cache = torch.zeros((B, F, -(-N // 8) * 8), dtype=torch.bfloat16, device=DEV)
    cm.mlp_dense(x, w1, b1, w2, b2, out, a_cache, c, act)
    o_before, a_before = out.clone(), a_cache.clone()
    NB = -(-N // c)
    idx, _ = recipes.mlp_indices(B * NB, F, k, 30, DEV)
    counts = torch.full((B, NB), k, dtype=torch.int32, device=DEV)
    cm.mlp_sparse_delta(x, w1, b1, w2, idx.view(B, NB, k), counts, a_cache, out, c, act, _u8(cm.mlp_workspace_bytes(B, N, D, F, c, k)))
    assert torch.equal(a_cache, a_before) and torch.equal(out, o_before)


@pytest.mark.parametrize("B,N,D,F,c,k,tiles", [
    (1, 100, 384, 320, 128, 200, [2, 2, 0, 0, 2, 0]), (1, 7 * 128 - 5, 256, 512, 128, 140, [2, 2, 0, 2, 2, 0]),
    (1, 9 * 192, 128, 640, 192, 300, [2, 2, 0, 2, 2, 0]), (3, 5 * 128 - 60, 640, 256, 128, 256, [2, 2, 0, 0, 2, 0]),
    (1, 17 * 192 - 1, 256, 448, 192, 65, [2, 2, 0, 2, 2, 0]),
    # and on the chunk's tiles, in the second GEMMs those beyond one per CU 64 rows at a time
    (1, 7 * 192 - 5, 3328, 2560, 192, 1372, [0, 0, 23, 0, 0, 23]), (1, 14 * 128 - 5, 2432, 1344, 128, 785, [0, 0, 32, 0, 0, 32]),
    (1, 11 * 192 - 100, 3328, 1280, 192, 700, [2, 0, 32, 0, 0, 32]), (1, 47 * 128 - 70, 1024, 448, 128, 300, [0, 0, 32, 0, 0, 32]),
    (1, 15 * 192 - 5, 1664, 1152, 192, 642, [0, 0, 25, 0, 0, 25]), (1, 55 * 192 - 5, 512, 512, 192, 348, [0, 0, 28, 0, 0, 28]),
    (3, 53 * 128 - 5, 384, 128, 128, 89, [0, 0, 60, 0, 0, 60])])
def test_mlp_of_any_number_of_chunks(cm, oracle, B, N, D, F, c, k, tiles):
    """1 to 159 chunks, none a multiple of eight: the tiles of the chunks beyond one are dealt out over the XCDs one by one, in the
    sparse and in the dense form, each exactly once."""
    assert _mlp_tiles(cm, B, N, D, F, c, k) == tiles
    x1, x2, w1, b1, w2, b2 = recipes.mlp_inputs(B, N, D, F, 31, DEV)
    NB, a_ld = -(-N // c), -(-N // 8) * 8
    out = torch.empty_like(x1)
    a_cache = torch.zeros((B, F, a_ld), dtype=torch.bfloat16, device=DEV)
    cm.mlp_dense(x1, w1, b1, w2, b2, out, a_cache, c, 1)
    ref, a_ref, _ = oracle.mlp_dense(si.np_f32(x1), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), si.np_f32(b2), c, 1, a_ld=a_ld)
    assert rel_err(si.np_f32(a_cache)[..., :N], a_ref[..., :N]) <= REL_TOL
    assert rel_err(si.np_f32(out), ref) <= REL_TOL
    o_ref, a_ref = (si.np_f32(t).astype(np.float64) for t in (out, a_cache))
    o_before = o_ref.copy()
    idx, counts = recipes.mlp_indices(B * NB, F, k, 31, DEV, ragged=True)
    idx, counts = idx.view(B, NB, k), counts.view(B, NB)
    cm.mlp_sparse_delta(x2, w1, b1, w2, idx, counts, a_cache, out, c, 1, _u8(cm.mlp_workspace_bytes(B, N, D, F, c, k)))
    oracle.mlp_sparse_delta(si.np_f32(x2), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), idx.cpu().numpy(), counts.cpu().numpy(),
                            a_ref, o_ref, c, 1)
    assert rel_err(si.np_f32(a_cache)[..., :N], a_ref[..., :N]) <= REL_TOL
    assert rel_err(si.np_f32(out), o_ref, o_ref - o_before) <= REL_TOL


@pytest.mark.parametrize("c,chunks,tiles", [(128, 22, [2, 0]), (192, 22, [2, 0]),      # of 64 x 64
                                            (128, 200, [0, 50]), (192, 90, [0, 23])])   # whole chunks: four stages, three
def test_mlp_second_gemm_at_the_ends_of_its_ring(cm, oracle, c, chunks, tiles):
    """Lists of 0 to 14 steps of 32 neurons, on both sides of a step's edge: fewer steps than the ring has stages, as many, more, odd
    and even."""
    counts_of = [0, 1, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 257, 288, 320, 400, 417, 448]
    B, N, D, F, k = 1, chunks * c - 37, 256, 512, 448
    assert _mlp_tiles(cm, B, N, D, F, c, k)[4:] == tiles
    _, x2, w1, b1, w2, _ = recipes.mlp_inputs(B, N, D, F, 32, DEV)
    NB, a_ld = -(-N // c), -(-N // 8) * 8
    g = si.generator(32, DEV)
    a_cache, o_cache = si.randn_bf16((B, F, a_ld), g, 0.5), si.randn_bf16((B, N, D), g)
    o_ref, a_ref = (si.np_f32(t).astype(np.float64) for t in (o_cache, a_cache))
    o_before = o_ref.copy()
    idx, _ = recipes.mlp_indices(NB, F, k, 32, DEV)
    counts = torch.tensor([counts_of[i % len(counts_of)] for i in range(NB)], dtype=torch.int32, device=DEV)
    idx, counts = idx.view(B, NB, k), counts.view(B, NB)
    ws = torch.full((cm.mlp_workspace_bytes(B, N, D, F, c, k),), 255, dtype=torch.uint8, device=DEV)   # NaN wherever nothing is written
    cm.mlp_sparse_delta(x2, w1, b1, w2, idx, counts, a_cache, o_cache, c, 1, ws)
    oracle.mlp_sparse_delta(si.np_f32(x2), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), idx.cpu().numpy(), counts.cpu().numpy(),
                            a_ref, o_ref, c, 1)
    assert rel_err(si.np_f32(a_cache)[..., :N], a_ref[..., :N]) <= REL_TOL
    assert rel_err(si.np_f32(o_cache), o_ref, o_ref - o_before) <= REL_TOL


@pytest.mark.parametrize("F", [64, 128, 192, 320])
@pytest.mark.parametrize("c,N,tiles", [(128, 333, [2, 0]), (192, 333, [2, 0]),                       # of 64 x 64
                                       (128, 386 * 128 - 37, [0, 49]), (192, 337 * 192 - 37, [0, 43])])   # whole chunks
def test_mlp_dense_second_gemm_at_the_ends_of_its_ring(cm, oracle, c, N, tiles, F):
    """Dense contractions of 2, 4, 6 and 10 steps of 32; the first and the last rows against the oracle."""
    assert _mlp_tiles(cm, 1, N, 128, F, c, 1)[1:3] == tiles
    x, _, w1, b1, w2, b2 = recipes.mlp_inputs(1, N, 128, F, 33, DEV)
    a_ld = -(-N // 8) * 8
    out, a = torch.empty_like(x), torch.zeros((1, F, a_ld), dtype=torch.bfloat16, device=DEV)
    cm.mlp_dense(x, w1, b1, w2, b2, out, a, c, 1)
    for rows in (slice(0, min(N, 300)), slice(max(N - 700, 0), N)):
        ref, _, _ = oracle.mlp_dense(si.np_f32(x[:, rows].contiguous()), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), si.np_f32(b2), c, 1,
                                     a_ld=-(-x[:, rows].shape[1] // 8) * 8)
        assert rel_err(si.np_f32(out[:, rows].contiguous()), ref) <= REL_TOL


@pytest.mark.parametrize("B,N,D,F,c,k,act,bias,tiles", [
    (1, 1, 128, 64, 128, 32, 1, True, [2, 2, 0, 2, 2, 0]),             # one token: two steps of 64, one
    (2, 613, 128, 1024, 128, 512, 0, False, [2, 2, 0, 2, 2, 0]),       # tiles of 64 x 64, two batches, no bias
    (1, 777, 1152, 1984, 192, 700, 1, True, [2, 2, 0, 2, 2, 0]),
    (2, 200, 640, 704, 192, 352, 1, True, [2, 2, 0, 2, 2, 0]),         # the last chunk ends in its first 64 rows
    (1, 1500, 640, 1024, 128, 330, 0, True, [2, 2, 0, 2, 2, 0]),
    (1, 1000, 2560, 512, 192, 200, 0, True, [2, 0, 0, 2, 0, 0]),       # second GEMM in parts of 64 rows
    (1, 500, 128, 12288, 192, 5000, 1, True, [2, 2, 0, 2, 0, 0]),      # a list too long for the tiles of 64 x 64
    (1, 4500, 3072, 256, 192, 77, 1, False, [2, 1, 0, 2, 0, 64]),      # its last round in parts
    (1, 3603, 4992, 512, 128, 50, 0, True, [2, 0, 128, 2, 0, 128]),     # of both second GEMMs
])
def test_mlp_on_small_tiles(cm, oracle, B, N, D, F, c, k, act, bias, tiles):
    """Few tiles: 64 x 64 in both GEMMs, chunks in parts of 64 rows, the last round in parts.  Lists that end at and beside the
    edges of tiles and steps, an empty one; the workspace holds NaN wherever nothing is written; both forms of the cache
    write-back alike; the cells past N stay as they are."""
    assert _mlp_tiles(cm, B, N, D, F, c, k, -(-N // 8) * 8 + 8) == tiles
    x1, x2, w1, b1, w2, b2 = recipes.mlp_inputs(B, N, D, F, 34, DEV)
    if not bias:
        b1, b2 = torch.zeros_like(b1), torch.zeros_like(b2)
    bias1, bias2 = (b1, b2) if bias else (None, None)
    NB, a_ld = -(-N // c), -(-N // 8) * 8 + 8
    out = torch.full_like(x1, 7.0)
    a_cache = torch.full((B, F, a_ld), 3.0, dtype=torch.bfloat16, device=DEV)
    cm.mlp_dense(x1, w1, bias1, w2, bias2, out, a_cache, c, act)
    ref, a_ref, _ = oracle.mlp_dense(si.np_f32(x1), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), si.np_f32(b2), c, act, a_ld=a_ld)
    assert rel_err(si.np_f32(a_cache)[..., :N], a_ref[..., :N]) <= REL_TOL
    assert torch.all(a_cache[..., N:] == 3.0)
    assert rel_err(si.np_f32(out), ref) <= REL_TOL
    o_ref, a_ref = (si.np_f32(t).astype(np.float64) for t in (out, a_cache))
    o_before = o_ref.copy()
    idx, _ = recipes.mlp_indices(B * NB, F, k, 34, DEV)
    edges = torch.tensor([k, 0, 1, 63, 64, 65, 127, 128, 129, k - 1, 31, 32, 33, 96, 257], dtype=torch.int32).clamp(0, k)
    counts = edges[torch.arange(B * NB) % len(edges)].to(DEV)
    idx, counts = idx.view(B, NB, k), counts.view(B, NB)
    nan = lambda n: torch.full((max(n, 16),), 255, dtype=torch.uint8, device=DEV)  # noqa: E731
    o2, a2 = out.clone(), a_cache.clone()
    cm.mlp_sparse_delta(x2, w1, bias1, w2, idx, counts, a_cache, out, c, act, nan(cm.mlp_workspace_bytes(B, N, D, F, c, k)))
    cm.mlp_sparse_delta_overlapped(x2, w1, bias1, w2, idx, counts, a2, o2, c, act, nan(cm.mlp_overlapped_workspace_bytes(B, N, D, F, c, k)))
    assert torch.equal(a_cache, a2) and torch.equal(out, o2)
    oracle.mlp_sparse_delta(si.np_f32(x2), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), idx.cpu().numpy(), counts.cpu().numpy(),
                            a_ref, o_ref, c, act)
    assert rel_err(si.np_f32(a_cache)[..., :N], a_ref[..., :N]) <= REL_TOL
    assert torch.all(a_cache[..., N:] == 3.0)
    assert rel_err(si.np_f32(out), o_ref, o_ref - o_before) <= REL_TOL


@pytest.mark.parametrize("B,N,D,F,c,k,first_dense,first_delta", [(1, 500, 256, 640, 192, 320, 2, 2), (1, 1021, 256, 16320, 128, 1000, 1, 2),
                                                                (1, 700, 1024, 8000, 192, 1000, 0, 2), (1, 900, 1024, 10240, 128, 5000, 1, 1),
                                                                (1, 1000, 2560, 512, 192, 500, 2, 0)])
def test_unchanged_input_on_small_tiles(cm, B, N, D, F, c, k, first_dense, first_delta):
    """Tiles of 64 x 64 add their products in the order of the larger ones: the delta of an input that has not changed is nothing,
    bit for bit, whichever filled the cache."""
    tiles = _mlp_tiles(cm, B, N, D, F, c, k)
    assert (tiles[0], tiles[3]) == (first_dense, first_delta)
    x, _, w1, b1, w2, b2 = recipes.mlp_inputs(B, N, D, F, 35, DEV)
    out = torch.empty_like(x)
    a_cache = torch.zeros((B, F, -(-N // 8) * 8), dtype=torch.bfloat16, device=DEV)
    cm.mlp_dense(x, w1, b1, w2, b2, out, a_cache, c, 1)
    o_before, a_before = out.clone(), a_cache.clone()
    NB = -(-N // c)
    idx, _ = recipes.mlp_indices(B * NB, F, k, 35, DEV)
    counts = torch.full((B, NB), k, dtype=torch.int32, device=DEV)
    cm.mlp_sparse_delta(x, w1, b1, w2, idx.view(B, NB, k), counts, a_cache, out, c, 1, _u8(cm.mlp_workspace_bytes(B, N, D, F, c, k)))
    assert torch.equal(a_cache, a_before) and torch.equal(out, o_before)


@pytest.mark.parametrize("B,N,D,c,F,k,whole,streams", [
    (1, 88 * 192 - 37, 2048, 192, 256, 70, 176, True), (2, 33 * 192 - 5, 3072, 192, 256, 70, 192, True),
    (1, 70 * 128 - 100, 4096, 128, 256, 70, 280, True), (2, 44 * 128 - 1, 3072, 128, 256, 70, 256, True),
    (1, 88 * 192 - 37, 2048, 192, 512, 448, 176, True), (1, 65 * 192 - 5, 3072, 192, 512, 448, 192, True),
    (1, 70 * 128 - 100, 4096, 128, 512, 448, 280, True), (2, 44 * 128 - 1, 3072, 128, 512, 448, 256, True),
    (1, 63 * 128 - 5, 4096, 128, 512, 448, 252, False), (1, 42 * 192 - 1, 4096, 192, 512, 448, 168, False)])
def test_mlp_delta_of_an_output_past_the_caches(cm, oracle, B, N, D, c, F, k, whole, streams):
    """Outputs of over 67 MB, which pass the caches by, and just below, with and without a last round in parts of 64 rows; the first
    two and the last two chunks of each batch against the oracle, the longer lists with 14, 5, 6 and 9 steps."""
    assert _mlp_tiles(cm, B, N, D, F, c, k)[4:] == [0, whole]
    assert bool(cm.load().chipmunk_internal_mlp_streams(B, N, D, c)) == streams
    g = si.generator(35, DEV)
    x, w1, w2 = si.randn_bf16((B, N, D), g), si.randn_bf16((F, D), g, D ** -0.5), si.randn_bf16((F, D), g, F ** -0.5)
    b1, NB, a_ld = si.randn_bf16((F,), g), -(-N // c), -(-N // 8) * 8
    a_cache, o_cache = si.randn_bf16((B, F, a_ld), g, 0.5), si.randn_bf16((B, N, D), g)
    idx, counts = recipes.mlp_indices(B * NB, F, k, 35, DEV, ragged=True)
    idx, counts = idx.view(B, NB, k), counts.view(B, NB)
    if k == 448:
        counts[:, [0, 1, -2, -1]] = torch.tensor([448, 129, 161, 288], dtype=torch.int32, device=DEV)
    a_new, o_new = a_cache.clone(), o_cache.clone()
    cm.mlp_sparse_delta(x, w1, b1, w2, idx, counts, a_new, o_new, c, 1, _u8(cm.mlp_workspace_bytes(B, N, D, F, c, k)))
    for first in (0, NB - 2):
        rows, n = slice(first * c, min((first + 2) * c, N)), min((first + 2) * c, N) - first * c
        o_ref = si.np_f32(o_cache[:, rows].contiguous()).astype(np.float64)
        a_ref = np.zeros((B, F, -(-n // 8) * 8))
        a_ref[..., :n] = si.np_f32(a_cache[..., rows].contiguous())
        o_before = o_ref.copy()
        oracle.mlp_sparse_delta(si.np_f32(x[:, rows].contiguous()), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2),
                                idx[:, first:first + 2].contiguous().cpu().numpy(),
                                counts[:, first:first + 2].contiguous().cpu().numpy(), a_ref, o_ref, c, 1)
        assert rel_err(si.np_f32(a_new[..., rows].contiguous()), a_ref[..., :n]) <= REL_TOL
        assert rel_err(si.np_f32(o_new[:, rows].contiguous()), o_ref, o_ref - o_before) <= REL_TOL


@pytest.mark.parametrize("B,N,D,c", [(1, 27001, 5120, 192), (2, 16500, 4096, 128)])
def test_neuron_scores_of_an_input_past_the_caches(cm, oracle, B, N, D, c):
    """An x of over 256 MB; the first two and the last two chunks of each batch against the oracle."""
    F, NB = 64, -(-N // c)
    assert B * N * D * 2 > 256 << 20
    g = si.generator(36, DEV)
    x, w1 = si.randn_bf16((B, N, D), g), si.randn_bf16((F, D), g, D ** -0.5)
    T = torch.full((B, NB, F), float("nan"), dtype=torch.float32, device=DEV)
    cm.mlp_tile_mean_preact(x, w1, T, c, _u8(cm.mlp_tile_mean_workspace_bytes(B, N, D, F, c)))
    for first in (0, NB - 2):
        ref = oracle.mlp_tile_scores(si.np_f32(x[:, first * c:(first + 2) * c].contiguous()), si.np_f32(w1), c)
        assert rel_err(T[:, first:first + 2].cpu().numpy(), ref) <= SUM_TOL


@pytest.mark.parametrize("geom,batch,words,dtype", [
    ((3, 5, 9, 13, 2, 2, 4, 3), 3, 2560, torch.bfloat16),       # rows of 320 16-byte words: one sweep of five per lane
    ((0, 4, 6, 7, 5, 4, 6, 8), 2, 2568, torch.bfloat16),        # 321 words; the voxel is wider than the grid
    ((1, 3, 50, 1, 0, 1, 7, 1), 1, 701, torch.int32),           # 4-byte words, more than one sweep, remainder rows
    ((7, 1, 1, 1, 0, 3, 3, 3), 4, 1, torch.int32),              # no full voxel at all
    ((0, 7, 64, 67, 1, 4, 6, 8), 1, 2304, torch.bfloat16),      # 138 MB: streamed
    ((2, 7, 64, 67, 0, 2, 5, 8), 1, 1201, torch.int32),         # 144 MB in 4-byte words
    ((3, 5, 50, 61, 2, 2, 4, 3), 5, 64, torch.bfloat16),        # 76 275 short rows, several a wave
    ((1, 5, 50, 61, 0, 2, 4, 8), 9, 63, torch.int32),           # 137 259 in 4-byte words
    ((0, 9, 50, 61, 3, 4, 6, 8), 20, 504, torch.bfloat16),      # 554 MB of them, just short
])
def test_voxel_rows_and_permutation_in_one_launch(cm, oracle, geom, batch, words, dtype):
    """The copy's launch also writes the permutation and its inverse; rows of one and more sweeps, several rows a wave, small and
    streamed copies."""
    npre, T, H, W, nsuf, vt, vh, vw = geom
    N = npre + T * H * W + nsuf
    perm_ref, inv_ref = oracle.voxel_perm(*geom)
    src = torch.randint(-2 ** 15, 2 ** 15 - 1, (batch, N, words), device=DEV, dtype=torch.int32)
    src = src.to(torch.int16).view(torch.bfloat16) if dtype == torch.bfloat16 else src
    dst = torch.zeros_like(src)
    perm, inv = (torch.full((N,), -1, dtype=torch.int32, device=DEV) for _ in range(2))
    cm.voxel_reorder(src, dst, perm, inv, npre, T, H, W, nsuf, vt, vh, vw)
    assert np.array_equal(perm.cpu().numpy(), perm_ref) and np.array_equal(inv.cpu().numpy(), inv_ref)
    bits = torch.int16 if dtype == torch.bfloat16 else torch.int32
    assert torch.equal(dst.view(bits), src.view(bits)[:, torch.from_numpy(perm_ref).long().to(DEV)])
    back = torch.zeros_like(src)
    perm.fill_(-1)
    cm.voxel_reorder(dst, back, perm, None, npre, T, H, W, nsuf, vt, vh, vw, inverse=True)
    assert torch.equal(back.view(bits), src.view(bits)) and np.array_equal(perm.cpu().numpy(), perm_ref)


def test_mlp_delta_of_more_neurons_than_32_bits_of_bytes(cm, oracle):
    """A chunk's rows in the second GEMM take k c 2 bytes: here 32 768 more than 2^32.  Only the last 256 neurons reach the output."""
    N, D, c, last = 8, 128, 192, 256
    F = k = (2 ** 32 // (2 * c) // 128 + 1) * 128
    assert k * c * 2 > 2 ** 32
    g = si.generator(42, DEV)
    w1, w2 = (torch.empty((F, D), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    for r in range(0, F, 1 << 21):
        w1[r:r + (1 << 21)].copy_(si.randn_bf16((min(1 << 21, F - r), D), g, D ** -0.5))
    w2.zero_()
    w2[-last:] = si.randn_bf16((last, D), g, last ** -0.5)
    x, o_cache = si.randn_bf16((1, N, D), g), si.randn_bf16((1, N, D), g)
    a_cache = torch.zeros((1, F, 8), dtype=torch.bfloat16, device=DEV)
    idx = torch.arange(F, dtype=torch.int32, device=DEV).view(1, 1, F)
    counts = torch.full((1, 1), k, dtype=torch.int32, device=DEV)
    o_ref, a_ref = si.np_f32(o_cache).astype(np.float64), np.zeros((1, last, 8))
    o_before = o_ref.copy()
    cm.mlp_sparse_delta(x, w1, None, w2, idx, counts, a_cache, o_cache, c, 1, _u8(cm.mlp_workspace_bytes(1, N, D, F, c, k)))
    oracle.mlp_sparse_delta(si.np_f32(x), si.np_f32(w1[-last:]), np.zeros(last, dtype=np.float32), si.np_f32(w2[-last:]),
                            np.arange(last, dtype=np.int32).reshape(1, 1, last), np.array([[last]], dtype=np.int32), a_ref, o_ref, c, 1)
    assert rel_err(si.np_f32(a_cache[:, -last:].contiguous()), a_ref) <= REL_TOL
    assert rel_err(si.np_f32(o_cache), o_ref, o_ref - o_before) <= REL_TOL


@pytest.mark.parametrize("H,N,E,c,k,form", [
    (1, 193, 128, 192, 96, 0), (1, 193, 128, 192, 97, 2), (2, 650, 64, 192, 300, 2),            # up to 128 parts
    (11, 1000, 128, 192, 768, 1), (10, 1250, 128, 128, 800, 1), (11, 1000, 64, 192, 767, 0), (11, 1000, 64, 192, 768, 2),
    (10, 2100, 128, 192, 2048, 1), (260, 300, 128, 192, 150, 2), (260, 300, 64, 192, 150, 2)])   # over 256 parts; behind whole chunks
@pytest.mark.parametrize("masked", [False, True])
def test_column_lists_walked_by_pairs_of_waves(cm, oracle, H, N, E, c, k, form, masked):
    """Two waves share their rows and take every second tile: lists of one tile (the second wave has none), of an odd and an even
    number, ending inside one.  masked: the first step's second tile holds columns whose scores are -inf (products beyond the largest
    32-bit number): nothing of what the second wave multiplies there counts.  Judged chunk by chunk, each on the scale
    of its own update: a weight is rounded to bf16 (2^-9 of it), and beside lists of hundreds of columns, whose updates are small,
    one of 33 is off by more than 2 % of the whole tensor's RMS (0.023 at 768 columns)."""
    assert _attn_part_form(cm, H, N, E, c, k) == form
    q, kk, v = recipes.attn_inputs(1, H, N, E, 41, DEV)
    scale, NB = 1 / math.sqrt(E), -(-N // c)
    idx, _ = recipes.attn_indices(H * NB, N, k, 41, DEV)
    edges = torch.tensor([n for n in (k, 0, 1, 32, 33, 63, 64, 65, 95, 97, 128, 129) if n <= k], dtype=torch.int32)
    counts = edges[torch.arange(H * NB) % len(edges)].to(DEV)
    if masked:   # column 0 in those places (only one list has them all), every query's first column large
        q[..., 0], kk[..., 0, :], kk[..., 0, 0] = 2.0 ** 100, 0.0, -(2.0 ** 100)
        kk[..., 1:, 0] = 0.0
        place = torch.arange(64, device=DEV)
        second = place // (E // 64) % 2 == 1
        idx = torch.where(idx == 0, 1, idx)
        idx[:, :64][:, second[:min(64, k)]] = 0
        counts = torch.where(counts < 65, torch.where(counts == 0, 0, k), counts).to(torch.int32)   # no list may be masked whole
    idx, counts = idx.view(1, H, NB, k).contiguous(), counts.view(1, H, NB)
    base = recipes.attn_base(tuple(q.shape), k, "delta", 41, DEV)
    out = torch.full_like(q, 7.0)
    cm.attn_sparse_delta(q, kk, v, idx, counts, base, out, c, scale, 1.0)
    basen = si.np_f32(base).astype(np.float64)
    ref = oracle.attn_sparse_delta(si.np_f32(q), si.np_f32(kk), si.np_f32(v), idx.cpu().numpy(), counts.cpu().numpy(),
                                   basen, c, scale, 1.0)
    got = si.np_f32(out)
    for rows in (slice(i * c, min(N, (i + 1) * c)) for i in range(NB)):
        for h in range(H):
            assert rel_err(got[0, h, rows], ref[0, h, rows], ref[0, h, rows] - basen[0, h, rows]) <= REL_TOL
    cm.attn_sparse_delta(q, kk, v, idx, counts, base, base, c, scale, 1.0)      # in place
    assert torch.equal(base, out)


@pytest.mark.parametrize("H,N,E,form", [(2, 2, 128, 0), (3, 96, 128, 0), (3, 97, 64, 2), (20, 384, 128, 2), (20, 700, 128, 1),
                                        (22, 400, 64, 2), (10, 2050, 64, 1)])
def test_dense_attention_walked_by_pairs_of_waves(cm, oracle, H, N, E, form):
    """The same without a list, and the statistics that the column sums are made with: a reference within 2^8 of the row's maximum
    and the sum against it."""
    c, scale = 192, 1 / math.sqrt(E)
    assert _attn_part_form(cm, H, N, E, c, 0) == form
    q, k, v = recipes.attn_inputs(1, H, N, E, 42, DEV)
    out, NB, ld = torch.full_like(q, 7.0), -(-N // c), -(-N // 4) * 4
    D = torch.zeros((1, H, NB, ld), dtype=torch.float32, device=DEV)
    ws = _u8(cm.attn_dense_workspace_bytes(1, H, N))
    cm.attn_dense(q, k, v, out, D, c, scale, ws)
    ref, D_ref = oracle.attn_dense(si.np_f32(q), si.np_f32(k), si.np_f32(v), c, scale, want_colsum=True)
    assert rel_err(si.np_f32(out), ref) <= REL_TOL
    assert rel_err(D.cpu().numpy()[..., :N].astype(np.float64), D_ref) <= REL_TOL
    m, l = (t.cpu().numpy().astype(np.float64) for t in cm.attn_dense_row_stats(ws, 1, H, N))
    m_ref, l_ref = oracle.attn_row_stats(si.np_f32(q), si.np_f32(k), scale)
    assert np.abs(m + np.log(l) - (m_ref + np.log(l_ref))).max() <= 2e-3
    assert (m <= m_ref + 1e-3).all() and (m >= m_ref - 8 * math.log(2.0) - 1e-3).all()


@pytest.mark.parametrize("B,N,D,F,c,form", [
    (1, 1, 128, 64, 192, (1, 1)), (1, 15 * 128 + 7, 128, 4096, 128, (1, 1)), (2, 8 * 192, 1152, 4160, 192, (2, 1)),
    (1, 16 * 128 + 1, 640, 8192, 128, (2, 1)), (2, 15 * 128 + 1, 1280, 320, 128, (1, 1)), (1, 32 * 128 - 1, 384, 8256, 128, (4, 1)),
    (1, 32 * 128 + 1, 256, 576, 128, (1, 1)), (3, 16 * 192, 1152, 4224, 192, (2, 0)), (1, 47 * 128 + 3, 512, 11328, 128, (4, 1)),
    (1, 48 * 128 + 1, 512, 64, 128, (0, 1)), (1, 128 * 128, 640, 64, 128, (0, 0)), (2, 50 * 128 - 3, 640, 2048, 128, (0, 0)),
    (1, 64 * 128, 1024, 5120, 128, (0, 0)), (2, 15 * 128 + 1, 1408, 320, 128, (0, 1)), (1, 6 * 192, 4736, 1984, 192, (0, 1)),
    (1, 8 * 128, 3200, 192, 128, (0, 1)), (1, 16 * 192, 256, 16448, 192, (4, 1)), (1, 16 * 192 + 1, 256, 16448, 192, (0, 1)),
    (1, 17 * 128, 256, 16384, 128, (4, 1))])
def test_neuron_scores_of_few_chunks(cm, oracle, B, N, D, F, c, form):
    """Up to 48 chunks: one to three blocks of 16 of them, the last ragged; workgroups of 16, 32 and 64 neurons; contractions of fewer
    lines than a workgroup has waves, and of a number that its waves do not divide; both sides of the limits (of chunks
    by entries, of entries with few neurons, of chunks with many), beyond which the contraction is cut into pieces or not.
    Means in workgroups of 128 and of 512 columns.  Tolerance as for the pieces."""
    out = (ctypes.c_int32 * 2)()
    cm.load().chipmunk_internal_scores_form(B, N, D, F, c, out)
    assert tuple(out) == form
    g = si.generator(43, DEV)
    x, w1 = si.randn_bf16((B, N, D), g), si.randn_bf16((F, D), g, 1 / math.sqrt(D))
    NB = -(-N // c)
    T = torch.full((B * NB + 1, F), float("nan"), dtype=torch.float32, device=DEV)
    cm.mlp_tile_mean_preact(x, w1, T[:-1].view(B, NB, F), c, _u8(cm.mlp_tile_mean_workspace_bytes(B, N, D, F, c)))
    assert rel_err(T[:-1].view(B, NB, F).cpu().numpy(), oracle.mlp_tile_scores(si.np_f32(x), si.np_f32(w1), c)) <= SUM_TOL
    assert bool(T[-1].isnan().all())
    again = torch.empty((B, NB, F), dtype=torch.float32, device=DEV)
    cm.mlp_tile_mean_preact_static(x, w1, again, c)
    assert torch.equal(again.view(-1, F), T[:-1])


@pytest.mark.parametrize("B,N,D,F,c,act,bias,rows", [
    (1, 3174, 640, 1024, 192, 1, True, (128, 128)), (2, 1175, 768, 1344, 192, 0, False, (128, 128)), (1, 965, 512, 3200, 192, 1, True, (128, 192)),
    (2, 620, 512, 2560, 192, 0, True, (128, 192)), (1, 2116, 512, 576, 192, 1, False, (192, 128)), (2, 1036, 512, 576, 192, 1, True, (192, 128)),
    (2, 388, 1024, 4864, 128, 1, True, (192, 128)), (2, 534, 1664, 1728, 128, 0, True, (128, 192)),
    (1, 2376, 896, 512, 192, 1, True, (192, 192)), (2, 465, 512, 2176, 192, 0, True, (192, 192))])   # 7 % less than tiles of 64 x 64, by price
def test_dense_mlp_on_the_other_chunk_sizes_rows(cm, oracle, B, N, D, F, c, act, bias, rows):
    """The tiles of a dense MLP need not follow the chunks: both GEMMs, the first, the second on 128 rows for chunks of 192 and the other
    way round, the last tile ragged; the cells past N stay as they are, and the delta of the same input, on the chunk's own rows, is
    nothing, bit for bit."""
    out = (ctypes.c_int32 * 2)()
    cm.load().chipmunk_internal_mlp_dense_rows(B, N, D, F, c, -(-N // 8) * 8 + 8, out)
    assert tuple(out) == rows
    tiles = _mlp_tiles(cm, B, N, D, F, c, 1, -(-N // 8) * 8 + 8)
    assert (rows[0] == c or tiles[0] == 0) and (rows[1] == c or tiles[1] == 0)
    x, _, w1, b1, w2, b2 = recipes.mlp_inputs(B, N, D, F, 44, DEV)
    if not bias:
        b1, b2 = torch.zeros_like(b1), torch.zeros_like(b2)
    NB, a_ld = -(-N // c), -(-N // 8) * 8 + 8
    o = torch.full_like(x, 7.0)
    a_cache = torch.full((B, F, a_ld), 3.0, dtype=torch.bfloat16, device=DEV)
    cm.mlp_dense(x, w1, b1 if bias else None, w2, b2 if bias else None, o, a_cache, c, act)
    ref, a_ref, _ = oracle.mlp_dense(si.np_f32(x), si.np_f32(w1), si.np_f32(b1), si.np_f32(w2), si.np_f32(b2), c, act, a_ld=a_ld)
    assert rel_err(si.np_f32(a_cache)[..., :N], a_ref[..., :N]) <= REL_TOL
    assert torch.all(a_cache[..., N:] == 3.0)
    assert rel_err(si.np_f32(o), ref) <= REL_TOL
    o_before, a_before, k = o.clone(), a_cache.clone(), 200
    idx, _ = recipes.mlp_indices(B * NB, F, k, 44, DEV)
    counts = torch.full((B, NB), k, dtype=torch.int32, device=DEV)
    cm.mlp_sparse_delta(x, w1, b1 if bias else None, w2, idx.view(B, NB, k), counts, a_cache, o, c, act,
                        _u8(cm.mlp_workspace_bytes(B, N, D, F, c, k)))
    assert torch.equal(a_cache, a_before) and torch.equal(o, o_before)


@pytest.mark.parametrize("H,N,E,c,fused", [(43, 2304, 128, 192, 512), (43, 2304, 64, 192, 512), (43, 2303, 128, 192, 512),
                                           (31, 2305, 128, 128, 512), (28, 3501, 64, 128, 768), (37, 3000, 64, 192, 512),
                                           (28, 3499, 64, 128, 784), (10, 3072, 64, 192, 0), (10, 3072, 128, 192, 160),
                                           (12, 2500, 64, 192, 0), (6, 5376, 128, 192, 0), (7, 2304, 128, 128, 0),
                                           (43, 2299, 64, 192, 516), (43, 2700, 64, 192, 645)])
def test_refresh_with_its_last_chunks_apart(cm, oracle, H, N, E, c, fused):
    """The first chunks in the one kernel, those of a short last round apart, statistics updated in place: the heads at both
    ends and the one in which the launches meet against the oracle; the sums made apart are those of the entry point that makes
    them alone, bit by bit, and the one kernel's are not."""
    assert cm.load().chipmunk_internal_attn_refresh_fused(1, H, N, E, c) == fused
    (q1, k1, _), (q2, k2, v), _ = si.attn_steps(1, H, N, E, 41, DEV)
    scale, NB, ld = 1 / math.sqrt(E), -(-N // c), -(-N // 4) * 4 + 4
    s1 = torch.matmul(q1.float(), k1.float().transpose(-1, -2).contiguous()) * scale
    m = s1.amax(-1)
    l = torch.exp(s1 - m[..., None]).sum(-1)
    del s1
    m0, l0 = m.clone(), l.clone()
    out, D = torch.full_like(q2, float("nan")), torch.full((1, H, NB, ld), -1.0, dtype=torch.float32, device=DEV)
    cm.attn_dense_colsum_stale(q2, k2, v, out, m, l, D, c, scale, m, l)
    D_alone = torch.full_like(D, -1.0)
    cm.attn_colsum_stale(q2, k2, m0, l0, D_alone, c, scale)
    assert torch.equal(D.view(-1, ld)[fused:], D_alone.view(-1, ld)[fused:])
    assert fused == 0 or not torch.equal(D.view(-1, ld)[:fused], D_alone.view(-1, ld)[:fused])
    assert bool((D[..., N:] == -1.0).all())
    heads = sorted({0, min(fused // NB, H - 1), H - 1})
    qn, kn, vn = (si.np_f32(t[:, heads]) for t in (q2, k2, v))
    f64 = lambda t: t[:, heads].cpu().numpy().astype(np.float64)
    assert rel_err(f64(D[..., :N]), oracle.attn_colsum_stale(qn, kn, f64(m0), f64(l0), c, scale)) <= SUM_TOL
    assert rel_err(si.np_f32(out[:, heads]), oracle.attn_dense(qn, kn, vn, c, scale)) <= REL_TOL
    m_ref, l_ref = oracle.attn_row_stats(qn, kn, scale)
    assert np.abs(f64(m) + np.log(f64(l)) - (m_ref + np.log(l_ref))).max() <= 2e-3
    assert bool(torch.isfinite(out).all()) and bool(torch.isfinite(m).all()) and bool((l > 0).all())


def test_refresh_with_its_last_chunks_apart_and_far_normalisers(cm):
    """Normalisers 60 below the current scores: every weight is inside 32 bits and the two ways agree.  200 below: the one kernel caps
    its factors, the pass that makes the last chunks' sums overflows like the formula; neither gives a NaN."""
    H, N, E, c, fused = 43, 2304, 128, 192, 512
    assert cm.load().chipmunk_internal_attn_refresh_fused(1, H, N, E, c) == fused
    q, k, v = recipes.attn_inputs(1, H, N, E, 45, DEV)
    scale, NB = 1 / math.sqrt(E), -(-N // c)
    out, D, alone = torch.empty_like(q), *(torch.empty((1, H, NB, N), dtype=torch.float32, device=DEV) for _ in range(2))
    m, l = torch.full((1, H, N), -60.0, device=DEV), torch.full((1, H, N), float(N), device=DEV)
    cm.attn_dense_colsum_stale(q, k, v, out, m, l, D, c, scale)
    cm.attn_colsum_stale(q, k, m, l, alone, c, scale)
    assert bool(torch.isfinite(D).all()) and float(((D - alone).abs() / alone).max()) <= 1e-3
    cm.attn_dense_colsum_stale(q, k, v, out, m - 140, l, D, c, scale)
    one, apart = D.view(-1, N)[:fused], D.view(-1, N)[fused:]
    assert not bool(D.isnan().any()) and bool((one >= 2.0 ** 100).all()) and bool(torch.isinf(apart).all())
    assert bool(torch.isfinite(out).all())
