"""GPU parity at the sizes where a kernel's tiles, remainders or dispatch rules change, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from parity_util import assert_close, dev, host, prep

pytestmark = pytest.mark.gpu


def attention_inputs(seed, B, q_len, H, Hkv, d, ctx, dtype):
    r = np.random.default_rng(seed)
    q = prep(r.standard_normal((B, q_len, H, d)) * 2.5, dtype)
    k, v = (prep(r.standard_normal((B, Hkv, ctx + q_len, d)), dtype) for _ in range(2))
    return q, k, v


def pages(tensors, seed, size=16):
    """caches [B, Hkv, N, d] -> their page pools [B * n, size, Hkv, d] and the page table [B, n] they share"""
    B, Hkv, N, d = tensors[0].shape
    n = (N + size - 1) // size
    table = torch.from_numpy(np.random.default_rng(seed).permutation(B * n).astype(np.int32)).cuda().view(B, n)
    pools = []
    for x in tensors:
        rows = torch.zeros((B, n * size, Hkv, d), dtype=x.dtype, device="cuda")
        rows[:, :N] = x.transpose(1, 2)
        pool = torch.empty((B * n, size, Hkv, d), dtype=x.dtype, device="cuda")
        pool[table.view(-1).long()] = rows.view(B * n, size, Hkv, d)
        pools.append(pool)
    return pools, table


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", [
    # q_len, G, ctx, slices, with two sequences of two KV heads: 65 rows (one past the 64-row block), 96 | 97, 128 (two
    # whole blocks), 130 (a third); caches of just under and over a 32-token tile per compute unit; slices of a tile,
    # of some, and of 24 and more
    (13, 5, 2100, 0), (12, 8, 2300, 3), (97, 1, 2048, 2), (16, 8, 2400, 2), (13, 10, 2100, 0), (8, 10, 2039, 0),
    (8, 10, 2041, 0),
])
def test_more_than_64_rows(hippo, shape, d):
    q_len, G, ctx, S = shape
    q, k, v = attention_inputs(q_len + d, 2, q_len, 2 * G, 2, d, ctx, "bf16")
    ref, _ = oracle.attention(q, k, v, ctx, None)
    qd, kd, vd = dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16")
    what = "%s d=%d" % (shape, d)
    plain = hippo.hippo_verify_attention(qd, kd, vd, ctx, num_splits=S)
    assert_close(host(plain), ref, "bf16", what)
    k2, v2 = kd.clone(), vd.clone()
    k2[:, :, ctx:] = 7.0
    v2[:, :, ctx:] = 7.0
    new = [x[:, :, ctx:].transpose(1, 2).contiguous() for x in (kd, vd)]
    out = hippo.hippo_verify_attention(qd, k2, v2, ctx, num_splits=S, k_new=new[0], v_new=new[1])
    assert torch.equal(out, plain) and torch.equal(k2, kd) and torch.equal(v2, vd), what   # the same arithmetic
    pools, table = pages([kd, vd], 3)
    assert torch.equal(hippo.hippo_verify_attention_paged(qd, *pools, table, ctx, num_splits=S), plain), what


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G, S", [(7, 3), (8, 2), (5, 1)])
def test_a_row_does_not_depend_on_the_rows_beside_it(hippo, G, S, d):
    # slices of 24 32-token tiles and more of a cache that a last-level cache holds: the tiles are the same for 16, 48, 64 and
    # more rows, so a call's first rows are bit for bit those of a call over fewer (the last tile masks what they do not see)
    ctx = 2305
    q, k, v = (dev(x, "bf16") for x in attention_inputs(G + d, 2, 13, 2 * G, 2, d, ctx, "bf16"))
    whole = hippo.hippo_verify_attention(q, k, v, ctx, num_splits=S)
    for n in (2, 6, 64 // G, 12):
        few = hippo.hippo_verify_attention(q[:, :n].contiguous(), k[:, :, :ctx + n], v[:, :, :ctx + n], ctx, num_splits=S)
        assert torch.equal(few, whole[:, :n]), n


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("shape", [
    # q_len, G, ctx: up to 16 query rows and 128 (fp32) or 256 rows of cache by the library's choice, and just beyond; one
    # slice asked for up to 736 rows and beyond; an empty context
    (2, 8, 0), (1, 7, 127), (1, 7, 128), (4, 4, 252), (4, 4, 253), (2, 9, 126), (1, 16, 735), (1, 16, 736), (13, 7, 115),
])
def test_one_slice_writes_the_output(hippo, shape, dtype):
    q_len, G, ctx = shape
    for d in (64, 128):
        q, k, v = attention_inputs(ctx + d, 3, q_len, 2 * G, 2, d, ctx, "fp32" if dtype == "fp32" else "bf16")
        if dtype == "fp8":
            kd, vd = dev(k, "bf16"), dev(v, "bf16")
            codes = hippo.hippo_quantize_kv_e4m3(kd, vd)
            k, v = (host(c.view(torch.float8_e4m3fn).float()) * host(m)[..., None, None] for c, m in
                    ((codes[0], codes[2]), (codes[1], codes[3])))
            call = lambda S: hippo.hippo_verify_attention_fp8kv(dev(q, "bf16"), *codes, ctx, num_splits=S, want_lse=True)
        else:
            kd, vd = dev(k, dtype), dev(v, dtype)
            call = lambda S: hippo.hippo_verify_attention(dev(q, dtype), kd, vd, ctx, num_splits=S, want_lse=True)
        ref, ref_lse = oracle.attention(q, k, v, ctx, None)
        tol = "fp32" if dtype == "fp32" else "bf16"
        for S in (0, 1, 2):
            out, lse = call(S)
            assert_close(host(out), ref, tol, "%s d=%d S=%d" % (shape, d, S))
            # lse inherits the denominator's rounding: 1e-5, or 2^-9 where the probabilities are rounded to bf16
            np.testing.assert_allclose(host(lse), ref_lse, rtol=0, atol=2e-5 if dtype == "fp32" else 2.0 ** -8)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", [
    # q_len, G, ctx, slices of 72 to 73 32-token tiles: three row blocks over 14, 18 and 24 tiles a slice; four over 24; two
    # equal chunks of three blocks over 18 and 24, the second with a row less; four chunks of four; two of three over 12 and 14
    (6, 7, 2300, 5), (6, 7, 2300, 4), (6, 7, 2311, 3), (7, 8, 2300, 3), (13, 7, 2290, 4), (11, 7, 2300, 3), (31, 8, 2300, 3), (13, 7, 2290, 6), (13, 7, 2290, 5),
])
def test_tile_shapes_by_slice_length_and_rows(hippo, shape, d):
    test_more_than_64_rows(hippo, shape, d)


@pytest.mark.parametrize("shape", [
    # B, q_len, G, KV heads, head dim, ctx, dtype: a slice per compute unit whose partials fit the static array, ones
    # that would exceed it in fp32 (by a little, by half), and more heads than compute units
    (1, 16, 8, 4, 128, 9000, "bf16"), (1, 16, 8, 1, 64, 20000, "fp32"), (1, 8, 8, 1, 128, 9000, "fp32"),
    (1, 16, 4, 2, 128, 9000, "fp32"), (1, 13, 7, 4, 128, 2100, "fp32"), (1, 16, 8, 4, 64, 2100, "fp32"),
    (33, 4, 8, 8, 64, 40, "fp32"),
])
def test_static_scratch_call_takes_the_workspace_calls_slices(hippo, shape):
    B, q_len, G, Hkv, d, ctx, dtype = shape
    q, k, v = attention_inputs(5, B, q_len, Hkv * G, Hkv, d, ctx, dtype)
    ref, _ = oracle.attention(q, k, v, ctx, None)
    q, k, v = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    need = hippo.workspace_bytes(hippo.CALL_VERIFY_ATTENTION, hippo.kv_desc(k, Hkv * G), None, q_len, ctx + q_len)
    assert need <= hippo.load().hippo_static_scratch_bytes()
    out = hippo.hippo_verify_attention_static(q, k, v, ctx)
    assert torch.equal(out, hippo.hippo_verify_attention(q, k, v, ctx))
    assert_close(host(out), ref, dtype, "static %s" % (shape,))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", [
    # q_len, G, ctx, slices, with two sequences of two KV heads: one row to 128 in every row-block size and just past
    # it (65 to 128 in one block where the slice count is given, or their partials fit the static array: 120 rows of 64
    # channels; otherwise in two), and more than one chunk; slices of part of a tile, a tile, and of more super-tiles
    # than the ring has stages
    (1, 1, 0, 0), (1, 16, 16, 0), (17, 1, 300, 0), (3, 11, 1000, 1), (7, 7, 1200, 2), (8, 8, 2500, 0), (13, 5, 4200, 0),
    (12, 8, 2100, 2), (97, 1, 4096, 3), (15, 8, 2100, 0), (16, 8, 4100, 0), (16, 8, 2100, 40), (13, 10, 900, 2),
])
def test_fp32_attention_row_blocks(hippo, shape, d):
    q_len, G, ctx, S = shape
    q, k, v = attention_inputs(q_len + d, 2, q_len, 2 * G, 2, d, ctx, "fp32")
    ref, ref_lse = oracle.attention(q, k, v, ctx, None)
    qd, kd, vd = dev(q, "fp32"), dev(k, "fp32"), dev(v, "fp32")
    what = "%s d=%d" % (shape, d)
    plain, lse = hippo.hippo_verify_attention(qd, kd, vd, ctx, num_splits=S, want_lse=True)
    # A logit z that is a sum of d products in fp32 is off by some |z| sqrt(d/3) 2^-24 / sqrt(3) / sqrt(2) (random walk
    # in two chains of growing partial sums): 1.9e-6 for the largest here, z = 12 at d = 128, and so is the weight of the
    # token it may leave alone to decide a row.  Twice that of sum_n p_n |v_n| is allowed where it is more than the fp32
    # bound, which a row of cancelling values can miss (the largest seen: 2.0e-6 of that sum).
    spread, _ = oracle.attention(q, k, np.abs(v), ctx, None)
    err = np.abs(host(plain) - ref)
    assert (err <= np.maximum(1e-5 * np.maximum(np.abs(ref), np.sqrt(np.mean(ref ** 2))), 2.0 ** -18 * spread)).all(), what
    np.testing.assert_allclose(host(lse), ref_lse, rtol=2e-5, atol=2e-5, err_msg=what)
    k2, v2 = kd.clone(), vd.clone()
    k2[:, :, ctx:] = 7.0
    v2[:, :, ctx:] = 7.0
    new = [x[:, :, ctx:].transpose(1, 2).contiguous() for x in (kd, vd)]
    out = hippo.hippo_verify_attention(qd, k2, v2, ctx, num_splits=S, k_new=new[0], v_new=new[1])
    assert torch.equal(out, plain) and torch.equal(k2, kd) and torch.equal(v2, vd), what   # the same arithmetic
    pools, table = pages([kd, vd], 3)
    assert torch.equal(hippo.hippo_verify_attention_paged(qd, *pools, table, ctx, num_splits=S), plain), what
    # rows of a wider buffer: any 16-byte-aligned row stride
    wide = [torch.zeros((2, 2, ctx + q_len, d + 12), device="cuda") for _ in range(2)]
    views = [w[..., :d].copy_(x) for w, x in zip(wide, (kd, vd))]
    assert torch.equal(hippo.hippo_verify_attention(qd, *views, ctx, num_splits=S), plain), what


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("ctx", [0, 15, 16, 700])
def test_fp32_infinity_in_the_last_value_row(hippo, ctx, d):
    # the one row that sees it gets the infinity, not a NaN from rows past the cache's end
    q, k, v = attention_inputs(d, 2, 1, 14, 2, d, ctx, "fp32")
    ref, _ = oracle.attention(q, k, v, ctx, None)
    v[:, :, ctx, 5] = np.inf
    v[:, :, ctx, 6] = -np.inf
    got = host(hippo.hippo_verify_attention(dev(q, "fp32"), dev(k, "fp32"), dev(v, "fp32"), ctx))
    assert (got[..., 5] == np.inf).all() and (got[..., 6] == -np.inf).all()
    rest = [c for c in range(d) if c not in (5, 6)]
    assert_close(got[..., rest], ref[..., rest], "fp32", "ctx %d d=%d" % (ctx, d))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("size", [1e9, 1e20, 3e37])
def test_fp32_logits_of_any_finite_size(hippo, size, d):
    # one token's key decides every row, for it or against it; then all tokens' logits are huge and alike (the attention
    # mass, whose normaliser is one fp32 number of that size, cannot hold their count beside it)
    q, k, v = attention_inputs(d, 2, 5, 14, 2, d, 700, "fp32")
    q[..., 3] = np.where(np.abs(q[..., 3]) < 0.5, 0.5, q[..., 3]).clip(-3, 3)
    k[:, :, 300, 3] = size
    ref, _ = oracle.attention(q, k, v, 700, None)
    assert_close(host(hippo.hippo_verify_attention(dev(q, "fp32"), dev(k, "fp32"), dev(v, "fp32"), 700)), ref, "fp32",
                 "attention")
    got = attention_mass(hippo, q, k, "fp32", 4, 12, 14, 10)
    assert_close(got, oracle.s_attn(q, k, 10, 4 * 12 * 14), "fp32", "attention mass")
    q[..., 4:] = 0.0
    k[:, :, :, 3] = size
    q[..., :3] = 0.0                                                   # exactly alike: uniform weights
    ref, _ = oracle.attention(q, k, v, 700, None)
    assert_close(host(hippo.hippo_verify_attention(dev(q, "fp32"), dev(k, "fp32"), dev(v, "fp32"), 700)), ref, "fp32",
                 "attention, uniform")


def score_inputs(seed, B, L, H, Hkv, d, n, dtype, scale=2.0):
    r = np.random.default_rng(seed)
    return prep(r.standard_normal((B, L, H, d)) * scale, dtype), prep(r.standard_normal((B, Hkv, n, d)), dtype)


def attention_mass(hippo, q, k, dtype, frames, gh, gw, prefix):
    """the raw s_attn term of a call that scores by attention alone"""
    _, comps = hippo.hippo_score_tokens(dev(q, dtype), dev(k, dtype), hippo.video_desc(frames, gh, gw, prefix),
                                        flags=1, want_components=True)
    return host(comps)[0]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", [
    # B, text rows, G, frames, grid: 1 token and 1 row; 127, 128, 129 tokens; 32 and 33 rows; row runs of unequal
    # lengths; runs that come out empty (6 runs of 3 chunks over 14)
    (1, 1, 1, 1, 1, 1), (1, 32, 1, 1, 1, 127), (2, 33, 1, 1, 8, 16), (1, 5, 7, 1, 3, 43), (1, 64, 7, 5, 9, 11),
    (1, 31, 14, 3, 13, 17), (3, 17, 3, 2, 15, 16),
])
def test_fp32_attention_mass(hippo, shape, d):
    B, L, G, frames, gh, gw = shape
    n_vis = frames * gh * gw
    q, k = score_inputs(L + d, B, L, 2 * G, 2, d, n_vis + 9, "fp32")
    got = attention_mass(hippo, q, k, "fp32", frames, gh, gw, 4)
    assert_close(got, oracle.s_attn(q, k, 4, n_vis), "fp32", "%s d=%d" % (shape, d))


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", [
    # B, frames, grid, channels, crop: a pass is 512 channels; one pass and one piece more, short last passes, a
    # single piece; one frame, two, runs of several with a short last one; crops cut at the edges, of one token, of 32
    (1, 1, 5, 5, 512, 5, 5), (1, 2, 5, 7, 8, 5, 5), (2, 9, 11, 13, 520, 5, 5), (1, 3, 6, 5, 1024, 5, 5),
    (1, 40, 16, 16, 768, 5, 5), (1, 37, 11, 12, 504, 4, 8), (1, 5, 3, 3, 1544, 1, 1),
    # bf16 keeps the frame before in registers for two passes: three, over runs of several frames
    (1, 60, 16, 16, 1032, 5, 5),
])
def test_embedding_terms_over_passes_of_channels(hippo, shape, dtype):
    B, F, gh, gw, ch, cy, cx = shape
    r = np.random.default_rng(F * ch)
    n = F * gh * gw
    emb = r.standard_normal((B, F, gh, gw, ch))
    emb = prep((emb + 0.7 * np.roll(emb, 1, 1) + 0.7 * np.roll(emb, 1, 3)).reshape(B, n, ch), dtype)
    emb[:, n // 2] = 0.0                                              # a zero-norm row
    q, k = score_inputs(1, B, 3, 2, 1, 64, n, dtype)
    vid = hippo.video_desc(F, gh, gw, 0, cy, cx)
    st, ss = oracle.s_temp(emb, F), oracle.s_spa(emb, F, gh, gw, cy, cx)
    for flags in (7, 6):                                              # beside the attention term, and alone
        _, comps = hippo.hippo_score_tokens(dev(q, dtype), dev(k, dtype), vid, emb=dev(emb, dtype), flags=flags,
                                            want_components=True)
        assert_close(host(comps)[1], st, dtype, "s_temp %s %d" % (shape, flags))
        # a crop's variance is a difference of cosines: its error is measured against the largest one
        np.testing.assert_allclose(host(comps)[2], ss, rtol=0, atol=(2e-6 if dtype == "fp32" else 2e-3) * ss.max() + 1e-9)


@pytest.mark.parametrize("shape", [
    # an fp32 block of four waves takes 256 channels a pass, one of eight 512: a pass, less a piece and one more; two passes
    # and a piece more; four; batch elements and frame runs of several with a short last one; 0: the keys of both KV heads
    (2, 3, 6, 7, 252, 5, 5), (1, 4, 5, 5, 256, 5, 5), (1, 2, 11, 6, 260, 4, 8), (1, 21, 16, 16, 512, 5, 5),
    (3, 19, 11, 11, 516, 5, 5), (1, 5, 7, 11, 384, 5, 5), (1, 40, 16, 16, 768, 5, 5), (2, 7, 6, 6, 1024, 5, 5),
    (1, 70, 11, 11, 1020, 5, 5), (2, 9, 7, 6, 0, 5, 5),
    # crops for two four-wave blocks a compute unit in runs of eight frames
    (1, 240, 11, 11, 516, 5, 5),
])
def test_fp32_embedding_terms_beside_the_sweep(hippo, shape):
    B, F, gh, gw, ch, cy, cx = shape
    if ch:
        test_embedding_terms_over_passes_of_channels(hippo, shape, "fp32")
    n = F * gh * gw
    q, k = score_inputs(ch, B, 37, 6, 2, 128, n + 11, "fp32")
    emb = dev(prep(np.random.default_rng(n + ch).standard_normal((B, n, ch)), "fp32"), "fp32") if ch else None
    vid = hippo.video_desc(F, gh, gw, 5, cy, cx)
    comps = [hippo.hippo_score_tokens(dev(q, "fp32"), dev(k, "fp32"), vid, emb=emb, flags=flags, want_components=True)[1]
             for flags in (7, 1, 6)]
    assert torch.equal(comps[0][0], comps[1][0])                      # the sweep's blocks, with and without riders
    assert torch.equal(comps[0][1:], comps[2][1:])                    # the crops' sums, beside a sweep and alone


@pytest.mark.parametrize("L, frames", [(16, 24), (64, 64)])     # the riders lead; the sweep's blocks of 512 query rows do
def test_wide_embedding_terms_beside_the_sweep(hippo, L, frames):
    n = frames * 256
    q, k = score_inputs(L, 1, L, 64, 8, 128, n + 3, "bf16", 0.5)
    q, k, vid = dev(q, "bf16"), dev(k, "bf16"), hippo.video_desc(frames, 16, 16, 3)
    comps = [hippo.hippo_score_tokens(q, k, vid, flags=flags, want_components=True)[1] for flags in (7, 1, 6)]
    assert torch.equal(comps[0][0], comps[1][0]) and torch.equal(comps[0][1:], comps[2][1:])
    emb = oracle.keys_as_embedding(host(k)[:, :, :3 + 3 * 256], 3, 3 * 256)
    st, ss = oracle.s_temp(emb, 3), oracle.s_spa(emb, 3, 16, 16)      # the first two frames, whose neighbours are among three
    assert_close(host(comps[0])[1][:, :512], st[:, :512], "bf16", "s_temp")
    np.testing.assert_allclose(host(comps[0])[2][:, :512], ss[:, :512], rtol=0, atol=2e-3 * ss.max())


@pytest.mark.parametrize("ch, L, frames", [
    # two passes beside a sweep of many times their work; three: before a short sweep that fills the chip, beside one that does
    # not, behind a long one, and in few blocks
    (768, 1024, 4), (1536, 16, 33), (1536, 16, 12), (1536, 256, 33), (1544, 16, 3),
])
def test_wide_embeddings_of_their_own_beside_the_sweep(hippo, ch, L, frames):
    n = frames * 256
    q, k = score_inputs(L, 1, L, 64, 8, 128, n, "bf16", 0.5)
    emb = np.random.default_rng(ch).standard_normal((1, frames, 256, ch))
    emb = prep((emb + 0.7 * np.roll(emb, 1, 1)).reshape(1, n, ch), "bf16")
    q, k, vid, e = dev(q, "bf16"), dev(k, "bf16"), hippo.video_desc(frames, 16, 16, 0), dev(emb, "bf16")
    comps = [hippo.hippo_score_tokens(q, k, vid, emb=e, flags=flags, want_components=True)[1] for flags in (7, 1, 6)]
    assert torch.equal(comps[0][0], comps[1][0]) and torch.equal(comps[0][1:], comps[2][1:])
    st, ss = oracle.s_temp(emb, frames), oracle.s_spa(emb, frames, 16, 16)
    assert_close(host(comps[0])[1], st, "bf16", "s_temp")
    np.testing.assert_allclose(host(comps[0])[2], ss, rtol=0, atol=2e-3 * ss.max())


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("ch", [64, 520])
def test_rows_of_denormal_squared_norm(hippo, ch, dtype):
    # entries of 0 and +-2^-70: squared norms are denormal and, like all dot products of such rows, exact
    r = np.random.default_rng(ch)
    emb = r.standard_normal((1, 4, 6, 7, ch))
    emb[0, 0, 1, 2] = r.integers(-1, 2, ch) * 2.0 ** -70              # alone in its crop
    for at in ((2, 1, 2), (2, 1, 3), (3, 1, 2)):                      # two in a crop, and one a frame on
        emb[(0,) + at] = r.integers(-1, 2, ch) * 2.0 ** -70
    emb = prep(emb.reshape(1, 4 * 42, ch), dtype)
    q, k = score_inputs(1, 1, 3, 2, 1, 64, 4 * 42, dtype)
    st, ss = oracle.s_temp(emb, 4), oracle.s_spa(emb, 4, 6, 7)
    for flags in (7, 6):
        scores, comps = hippo.hippo_score_tokens(dev(q, dtype), dev(k, dtype), hippo.video_desc(4, 6, 7, 0),
                                                 emb=dev(emb, dtype), flags=flags, want_components=True)
        assert_close(host(comps)[1], st, dtype, "s_temp")
        np.testing.assert_allclose(host(comps)[2], ss, rtol=0, atol=(2e-6 if dtype == "fp32" else 2e-3) * ss.max())
        assert np.isfinite(host(scores)).all()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("ch, crop", [(64, 5), (520, 5), (64, 6), (64, 8)])      # one pass, two; crops above 32 tokens
def test_rows_with_a_nan_have_cosine_zero(hippo, ch, crop, dtype):
    emb = prep(np.random.default_rng(ch).standard_normal((1, 4 * 63, ch)), dtype)
    rows = [2 * 63 + 9 + 2, 3 * 63 + 62]                              # inside a crop; the last token of the last frame
    zeroed = emb.copy()
    zeroed[0, rows] = 0.0
    emb[0, rows[0], 3] = np.nan
    emb[0, rows[1], ch - 1] = np.nan
    q, k = score_inputs(1, 1, 3, 2, 1, 64, 4 * 63, dtype)
    st, ss = oracle.s_temp(zeroed, 4), oracle.s_spa(zeroed, 4, 7, 9, crop, crop)
    for flags in (7, 6):
        scores, comps = hippo.hippo_score_tokens(dev(q, dtype), dev(k, dtype), hippo.video_desc(4, 7, 9, 0, crop, crop),
                                                 emb=dev(emb, dtype), flags=flags, want_components=True)
        assert_close(host(comps)[1], st, dtype, "s_temp")
        np.testing.assert_allclose(host(comps)[2], ss, rtol=0, atol=(2e-6 if dtype == "fp32" else 2e-3) * ss.max())
        assert np.isfinite(host(scores)).all()


def test_wide_keys_as_embedding(hippo):
    # 8 KV heads x 128 channels: the keys of all heads side by side, 1024 channels in two passes; 4 heads: one, fp32 two
    for dtype, heads in (("fp32", 8), ("bf16", 8), ("fp32", 4), ("bf16", 4)):
        q, k = score_inputs(9, 1, 3, heads, heads, 128, 4 * 6 * 11 + 3, dtype)
        emb = oracle.keys_as_embedding(k, 2, 4 * 6 * 11)
        ss = oracle.s_spa(emb, 4, 6, 11)
        for flags in (7, 6):
            _, comps = hippo.hippo_score_tokens(dev(q, dtype), dev(k, dtype), hippo.video_desc(4, 6, 11, 2), flags=flags,
                                                want_components=True)
            assert_close(host(comps)[1], oracle.s_temp(emb, 4), dtype, "s_temp")
            np.testing.assert_allclose(host(comps)[2], ss, rtol=0, atol=(2e-6 if dtype == "fp32" else 2e-3) * ss.max())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale, shift", [
    # logits that fit fp32's exponent range as they are; rows whose exponentials overflow, underflow to denormals or
    # to zero without a reference; both kinds of rows and of 32-token tiles in one call
    (0.5, 0.0), (3.0, 0.0), (40.0, 0.0), (1.0, 150.0), (1.0, -80.0), (1.0, -150.0), (120.0, 0.0),
])
def test_attention_mass_over_the_exponent_range(hippo, scale, shift, d):
    q, k = score_inputs(7, 2, 21, 14, 2, d, 3 * 11 * 13 + 5, "bf16", scale)
    if shift:                                       # a shared component that moves every logit by about `shift`
        q[..., 0] = np.sqrt(d) * np.log(2.0)
        k[..., 0] = shift
        q[:, ::3, :, 0] = 0.0                       # every third text row stays where it was
        q, k = prep(q, "bf16"), prep(k, "bf16")
    got = attention_mass(hippo, q, k, "bf16", 3, 11, 13, 2)
    assert_close(got, oracle.s_attn(q, k, 2, 3 * 11 * 13), "bf16", "scale %g shift %g d=%d" % (scale, shift, d))


@pytest.mark.parametrize("shift", [0.0, 6.0, 24.0, 64.0, -24.0])
def test_attention_mass_keeps_its_precision_at_large_logits(hippo, shift):
    # Logits around `shift`.  A row's normaliser is rounded to fp32 at its own magnitude, at 64..128 powers of two by up
    # to 2^-18, 2.6e-6 of the row's weights, to either side: over 448 rows that averages out to less than a tenth.  A
    # logarithm with a bias would show whole in the column sums (2.6e-6 here), as the bound of 2^-20 must not allow.
    q, k = score_inputs(11, 1, 64, 14, 2, 128, 2048, "bf16", 1.0)
    q[..., 0] = np.sqrt(128)
    k[..., 0] = shift
    q, k = prep(q, "bf16"), prep(k, "bf16")
    ref = oracle.s_attn(q, k, 0, 2048)
    got = attention_mass(hippo, q, k, "bf16", 8, 16, 16, 0)
    assert np.linalg.norm(got - ref) <= 2.0 ** -20 * np.linalg.norm(ref)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("first, last", [(0, 1), (8, 12), (14, 15), (39, 40)])
def test_attention_mass_where_some_rows_leave_the_exponent_range(hippo, first, last, d):
    # 560 query rows in blocks of three 64-row chunks: large logits in a block's first chunk, a later one or its last, and
    # in no chunk of the other blocks; a video whose last wave has one token
    q, k = score_inputs(8, 1, 40, 28, 2, d, 257 + 5, "bf16", 0.5)
    q[..., 0] = 0.0
    q[:, first:last, :, 0] = np.sqrt(d)
    k[..., 0] = 120.0 + np.arange(k.shape[2]) % 7
    q, k = prep(q, "bf16"), prep(k, "bf16")
    got = attention_mass(hippo, q, k, "bf16", 1, 1, 257, 2)
    assert_close(got, oracle.s_attn(q, k, 2, 257), "bf16", "rows %d to %d d=%d" % (first, last, d))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n, L, H, Hkv", [
    # tiles of 128 tokens: one with idle waves, whole ones, one token more; chunks of 32 query rows: one row, one chunk, as many
    # as stay in registers (5), one more, several runs; the most tiles that take one sweep, and one token more, of few rows
    # (two sweeps) and of as many as take one
    (97, 1, 1, 1), (128, 8, 4, 1), (129, 23, 14, 2), (1408, 40, 4, 1), (257, 41, 4, 1), (3000, 91, 14, 2),
    (65536, 3, 2, 1), (65537, 3, 2, 1), (65536, 98, 1, 1), (65537, 98, 1, 1),
])
@pytest.mark.parametrize("rows_out", [None, (0, 1, 60.0), (-1, None, 60.0), (0, 1, -30.0), (0, None, 60.0)])
def test_fp32_attention_mass_in_one_sweep(hippo, n, L, H, Hkv, d, rows_out):
    # logits of a few units, and text rows (the first, the last, all) whose tiles' sums leave the words that the blocks
    # exchange for the bins, upwards or downwards
    if rows_out is not None and n > 4000:
        rows_out = rows_out[:2] + (rows_out[2] / 2,)
    q, k = score_inputs(n + L, 2 if n < 200 else 1, L, H, Hkv, d, n + 5, "fp32", 0.7)
    q[..., 0] = 0.0
    if rows_out is not None:
        first, last, shift = rows_out
        q[:, first:last, :, 0] = np.sqrt(d)
        k[..., 0] = shift
    ref = oracle.s_attn(q, k, 2, n)
    got = attention_mass(hippo, q, k, "fp32", 1, 1, n, 2)
    # 1e-5, and of a logit of `shift`: the channel that makes it comes first, so each of d additions, the product with the
    # scale and the one with log2(e) round by up to 2^-24 of it, and an exponential moves by as much
    shift = 0.0 if rows_out is None else abs(rows_out[2])
    bound = (1e-5 + shift * (d + 2) * 2.0 ** -24) * np.maximum(np.abs(ref), np.sqrt((ref ** 2).mean()))
    assert (np.abs(got - ref) <= bound).all(), np.abs((got - ref) / bound).max()


def logits_by_token(z, rows, d):
    """fp32 queries [1, rows, 1, d] and keys [1, 1, n, d] of one channel: row r's logit of token t is rows[r] * z[t]"""
    q, k = np.zeros((1, len(rows), 1, d), np.float32), np.zeros((1, 1, len(z), d), np.float32)
    q[0, :, 0, 0], k[0, 0, :, 0] = np.sqrt(d) * np.asarray(rows), z
    return q, k


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [131, 3136, 16384, 65536])
def test_fp32_attention_mass_of_rows_that_one_token_decides(hippo, n, d):
    # the other tiles' sums, each a few millionths of a unit of the row's, count all the same
    z = np.full(n, np.log(0.49 / 65536 / 128))
    z[n // 3] = 5.5
    q, k = logits_by_token(z, [1.0] * 98, d)           # (four chunks of rows: one sweep at all these sizes)
    got, ref = attention_mass(hippo, q, k, "fp32", 1, 1, n, 0), oracle.s_attn(q, k, 0, n)
    # a logit is rounded three times (one product, two factors), its exponential and the row's sum a few times more, the sum
    # over the rows, all alike, once a row, by half a unit of what is there so far
    assert (np.abs(got / ref - 1) <= (3 * np.abs(z) + 8 + 98 / 2) * 2.0 ** -24).all(), np.abs(got / ref - 1).max()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n, L", [(128, 3), (1290, 33), (9000, 70), (9000, 333)])
def test_fp32_attention_mass_of_sums_of_any_size(hippo, n, L, d):
    # whole tiles of logits from -55 to 76, in an order that has neighbours far apart; rows that see all of it, parts of it
    # and the reverse: sums in the words, in every bin, in several at once
    z = np.linspace(-55.0, 76.0, -(-n // 128))
    z = np.repeat(np.random.default_rng(n).permutation(z), 128)[:n]
    rows = np.random.default_rng(L).choice([1.0, 0.9, 0.5, 0.25, 0.1, 0.02, 0.0, -0.1, -0.6], L)
    rows[0] = 1.0
    q, k = logits_by_token(z, rows, d)
    got, ref = attention_mass(hippo, q, k, "fp32", 1, 1, n, 0), oracle.s_attn(q, k, 0, n)
    # a logit is rounded three times (one product, two factors), its exponential and the row's sum a few times more, the
    # sum over rows once a row
    bound = (3 * 2 * 76 + 8 + L) * 2.0 ** -24
    np.testing.assert_allclose(got, ref, rtol=bound, atol=1e-30)


@pytest.mark.parametrize("n, rows", [(88 * 128, 32), (88 * 128 + 1, 32), (176 * 128, 33), (176 * 128 + 1, 64), (264 * 128 + 1, 96),
                                     (264 * 128 + 1, 97)])
def test_fp32_attention_mass_of_few_rows_over_many_tokens(hippo, n, rows):
    # one sweep up to 88 tiles of tokens a chunk of 32 rows, and from four chunks on; two sweeps else
    q, k = score_inputs(rows, 1, rows, 1, 1, 64, n + 1, "fp32", 0.7)
    assert_close(attention_mass(hippo, q, k, "fp32", 1, 1, n, 1), oracle.s_attn(q, k, 1, n), "fp32", "s_attn")


@pytest.mark.parametrize("shift", [110.0, -110.0])
@pytest.mark.parametrize("chunk", [0, 3, 4, 5, 8, 9])
def test_fp32_attention_mass_where_a_long_run_meets_a_row_out_of_range(hippo, chunk, shift):
    # one run of ten chunks a KV head: the row is met while its block's waves still sweep (steps of both parities), at the
    # last step that they share and at those behind it; all must leave the sweep together
    L, H, Hkv, d, n = 80, 16, 4, 64, 8192
    q, k = score_inputs(chunk + 70, 1, L, H, Hkv, d, n, "fp32", 0.7)
    q[..., 0] = 0.0
    q[:, chunk * 32 // (H // Hkv), :, 0] = np.sqrt(d)
    k[..., 0] = shift
    ref = oracle.s_attn(q, k, 0, n)
    got = [attention_mass(hippo, q, k, "fp32", 1, 1, n, 0) for _ in range(3)]
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
    # 1e-5, and of a logit of `shift`: each of d additions and two products round by up to 2^-24 of it
    bound = (1e-5 + abs(shift) * (d + 2) * 2.0 ** -24) * np.maximum(np.abs(ref), np.sqrt((ref ** 2).mean()))
    assert (np.abs(got[0] - ref) <= bound).all(), np.abs((got[0] - ref) / bound).max()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("rows, d", [(1, 64), (2047, 128), (2049, 128), (70001, 64)])
def test_codes_over_the_exponent_range(hippo, dtype, rows, d):
    # codes are the rounded quotients' whatever the multiplier: ordinary, tiny and huge heads, and one of zeros
    r = np.random.default_rng(rows)
    x = r.standard_normal((1, 4, rows, d)) * np.exp2(r.integers(-12, 1, (1, 4, rows, 1)))
    x *= np.array([1.0, 2.0 ** -90, 2.0 ** 100, 0.0]).reshape(1, 4, 1, 1)
    x = prep(x, dtype)
    k, v, ks, vs = hippo.hippo_quantize_kv_e4m3(dev(x, dtype), dev(-x, dtype))
    codes, scale = oracle.quantize_e4m3(x)
    np.testing.assert_array_equal(ks.cpu().numpy(), scale)
    np.testing.assert_array_equal(vs.cpu().numpy(), scale)
    np.testing.assert_array_equal(k.cpu().numpy(), codes)
    np.testing.assert_array_equal(v.cpu().numpy() & 0x7f, codes & 0x7f)


@pytest.mark.parametrize("n", [40960, 40961, 57344, 57345, 70657, 73728, 73729])
@pytest.mark.parametrize("ties", [False, True])
def test_topk_of_long_sequences(hippo, n, ties):
    r = np.random.default_rng(n)
    s = r.standard_normal((2, n)).astype(np.float32)
    if ties:
        s = np.round(s * 2) / 2                      # some ten values: the k-th largest is one of thousands of ties
        s[1] = 0.25                                  # and a sequence of nothing but ties
    cache = torch.zeros((2, 1, n, 64), dtype=torch.bfloat16, device="cuda")
    vid = hippo.video_desc(1, 1, n, 0)
    for k in (1, n // 4, n - 3, n):
        idx, _, _ = hippo.hippo_select_gather_kv(torch.from_numpy(s).cuda(), k, cache, cache, vid, gather=False)
        want = np.sort(np.argsort(-s, axis=1, kind="stable")[:, :k], axis=1)
        np.testing.assert_array_equal(idx.cpu().numpy(), want)


@pytest.mark.parametrize("shape", [
    # B, heads, d, tokens, k: one block a head and several; more heads than compute units share, heads that do not divide
    # them; the last indices that fit LDS and one more; the last tokens of the one launch and one more; all kept; more than
    # 128 MiB to copy, and in 8 bits less
    (1, 1, 64, 1, 1), (2, 3, 128, 1025, 600), (1, 300, 64, 70, 33), (3, 7, 64, 4097, 1000), (1, 2, 64, 9000, 8580),
    (1, 2, 64, 9000, 8581), (1, 1, 128, 24576, 4000), (1, 1, 128, 24577, 4000), (40, 8, 64, 97, 97), (20, 8, 128, 1000, 900),
    # a head per compute unit and one more; two of up to 4096 tokens and one more, of 4096 tokens and one more
    (1, 256, 64, 4097, 30), (1, 257, 64, 4097, 30), (1, 512, 64, 4096, 30), (1, 513, 64, 4096, 30), (2, 256, 64, 4097, 30),
])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32, torch.uint8])
def test_draft_cache_in_one_launch(hippo, shape, dtype):
    B, Hkv, d, n, k = shape
    g = torch.Generator(device="cuda").manual_seed(n + k)
    scores = torch.randint(0, 50, (B, n), generator=g, device="cuda").float()         # ties at the threshold
    N = n + 11
    kc, vc = (torch.randint(0, 250, (B, N, Hkv, d), generator=g, device="cuda").to(dtype).transpose(1, 2) for _ in range(2))
    vid = hippo.video_desc(1, 1, n, 4)
    idx, ref_idx = [hippo.hippo_select_gather_kv(scores, k, kc, vc, vid, gather=flag)[0] for flag in (True, False)]
    assert torch.equal(idx, ref_idx)                                                  # with the gather, and without
    order = torch.sort(scores, dim=1, descending=True, stable=True).indices[:, :k].sort(1).values
    assert torch.equal(idx.long(), order)
    dst = [torch.full((B, Hkv, 11 + k, d + 16), 7, device="cuda").to(dtype) for _ in range(2)]
    out = [x[..., :d] for x in dst]                                                   # rows with a gap behind them
    hippo.hippo_select_gather_kv(scores, k, kc, vc, vid, k_dst=out[0], v_dst=out[1])
    rows = torch.cat([torch.arange(4, device="cuda").expand(B, 4), 4 + order,
                      torch.arange(4 + n, N, device="cuda").expand(B, 7)], 1)
    for src, got, whole in zip((kc, vc), out, dst):
        assert torch.equal(got, torch.stack([src[b][:, rows[b]] for b in range(B)]))
        assert bool((whole[..., d:].float() == 7).all())


@pytest.mark.parametrize("n", [16384, 16385, 24576])
def test_draft_cache_in_a_graph(hippo, n):
    # the same rows and indices from a replayed graph, whichever number of launches it holds, over new scores each time
    g = torch.Generator(device="cuda").manual_seed(n)
    scores = torch.empty((2, n), device="cuda")
    kc, vc = (torch.randn((2, 2, n + 9, 64), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    vid = hippo.video_desc(1, 1, n, 3)
    scores.normal_(generator=g)
    outs = hippo.hippo_select_gather_kv(scores, 700, kc, vc, vid)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        held = hippo.hippo_select_gather_kv(scores, 700, kc, vc, vid)
    for _ in range(4):
        scores.normal_(generator=g)
        graph.replay()
        outs = hippo.hippo_select_gather_kv(scores, 700, kc, vc, vid)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(held, outs))


@pytest.mark.parametrize("dtype, d, G, layers, F, gh, gw, L", [
    ("fp32", 64, 2, 2, 85, 13, 24, 26), ("fp32", 64, 2, 1, 128, 24, 24, 20),     # two sweeps of two chunks of rows
    ("fp32", 128, 7, 1, 128, 12, 20, 12), ("fp32", 64, 7, 1, 16, 14, 14, 64),    # the same of 128 channels; one sweep
    ("bf16", 64, 7, 1, 16, 16, 16, 64), ("bf16", 128, 7, 1, 64, 16, 16, 32),
])
def test_scores_are_the_same_bits_call_after_call(hippo, dtype, d, G, layers, F, gh, gw, L):
    # what one wave leaves in LDS for another is there at the barrier between them: 300 calls, from memory and from the caches
    g = torch.Generator(device="cuda").manual_seed(d + L)
    n, tdt = F * gh * gw, torch.bfloat16 if dtype == "bf16" else torch.float32
    q = [torch.randn((1, L, 2 * G, d), generator=g, device="cuda").to(tdt) for _ in range(layers)]
    k = [torch.randn((1, 2, n, d), generator=g, device="cuda").to(tdt) for _ in range(layers)]
    vid, away = hippo.video_desc(F, gh, gw, 0), torch.empty(600 << 20, dtype=torch.uint8, device="cuda")
    ref = hippo.hippo_score_tokens_layers(q, k, vid, want_components=True)[1]
    different = torch.zeros((), dtype=torch.int64, device="cuda")
    for i in range(300):
        if i % 3 == 0:
            away.zero_()
        different += (hippo.hippo_score_tokens_layers(q, k, vid, want_components=True)[1] != ref).any()
    assert int(different) == 0


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n, L", [
    # a tile and less; eight tiles and a token more; 16 (the most whose statistics pass 2 merges itself) and 17; 8, 9 chunks
    # of rows a KV head; one row
    (256, 1), (1, 9), (2048, 13), (2049, 64), (4095, 37), (4096, 128), (4097, 128), (300, 147), (700, 293),
])
def test_bf16_attention_mass_of_short_videos(hippo, n, L, d):
    q, k = score_inputs(n + L, 2, L, 14, 2, d, n + 5, "bf16")
    q[:, L // 2] *= 30.0                                              # a text row of large logits
    q = prep(q, "bf16")
    got = attention_mass(hippo, q, k, "bf16", 1, 1, n, 3)
    assert_close(got, oracle.s_attn(q, k, 3, n), "bf16", "%d tokens, %d rows, d=%d" % (n, L, d))


@pytest.mark.parametrize("n, Hkv, parts", [(2500, 8, (12, 13)), (2500, 16, (6, 7, 25)), (1000, 32, (32, 33))])
def test_bf16_attention_mass_of_many_short_videos(hippo, n, Hkv, parts):
    # up to 1024 blocks of 10 tiles, 4096 of 4, pass 2 merges the statistics; one batch element more: the same bits, a launch
    q, k = score_inputs(n, max(parts), 9, 2 * Hkv, Hkv, 64, n, "bf16")
    whole = attention_mass(hippo, q, k, "bf16", 1, 1, n, 0)
    assert_close(whole[:1], oracle.s_attn(q[:1], k[:1], 0, n), "bf16", "%d tokens" % n)
    for some in parts:
        assert np.array_equal(attention_mass(hippo, q[:some], k[:some], "bf16", 1, 1, n, 0), whole[:some])


@pytest.mark.parametrize("n, Hkv, layers, B, merged", [
    # ten tiles of 256 tokens or four: pass 2 merges the row statistics of up to 1024 blocks, or 4096, and a launch those of more
    (2500, 8, 1, 12, True), (2500, 8, 1, 13, False), (3724, 16, 4, 1, True), (3724, 16, 4, 6, False),
    (1000, 32, 1, 32, True), (1000, 32, 1, 33, False), (4096, 2, 1, 1, True), (4097, 2, 1, 1, False),
])
def test_where_pass_2_of_bf16_scoring_merges_the_row_statistics(hippo, kernels, n, Hkv, layers, B, merged):
    q = torch.zeros((layers, B, 9, 2 * Hkv, 64), dtype=torch.bfloat16, device="cuda")
    k = torch.zeros((layers, B, Hkv, n, 64), dtype=torch.bfloat16, device="cuda")
    names = kernels(lambda: hippo.hippo_score_tokens_layers(q, k, hippo.video_desc(1, 1, n, 0), flags=hippo.SCORE_ATTN))
    assert [x for x in names if "sattn_mfmaILi64ELi2E" in x]
    assert any("sattn_row_lse" in x for x in names) != merged


def test_bf16_attention_mass_of_long_runs_of_rows(hippo):
    # a block's threads cover a run of 512 rows; longer ones have a launch for their statistics
    for L in (256, 257, 320):
        q, k = score_inputs(L, 1, L, 32, 8, 64, 2000, "bf16")
        got = attention_mass(hippo, q, k, "bf16", 4, 20, 25, 0)
        assert_close(got, oracle.s_attn(q, k, 0, 2000), "bf16", "%d text rows" % L)


@pytest.mark.parametrize("dtype, channels", [("bf16", (8, 64, 72, 256, 384, 392, 448, 456)), ("fp32", (4, 64, 68, 128, 192, 196))])
def test_embedding_terms_of_few_channels(hippo, dtype, channels):
    # channels for one wave of the block, a piece more, for all waves but one, a piece more
    for ch in channels:
        test_embedding_terms_over_passes_of_channels(hippo, (1, 7, 6, 11, ch, 5, 5), dtype)


@pytest.mark.parametrize("dtype, Hkv, d, few", [
    ("fp32", 4, 64, False), ("fp32", 2, 128, False), ("fp32", 3, 64, True), ("fp32", 1, 128, True),
    ("bf16", 8, 64, False), ("bf16", 7, 64, False), ("bf16", 4, 128, False), ("bf16", 6, 64, True), ("bf16", 3, 128, True),
])
def test_which_embedding_blocks_ask_for_waves_without_channels(hippo, kernels, dtype, Hkv, d, few):
    # those of 192 fp32 channels or 384 bf16 ones and fewer; beside the sweep (one or two of fp32) and in a launch of their own
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k = torch.ones((1, 23, Hkv, d), dtype=tdt, device="cuda"), torch.ones((1, Hkv, 655 * 45, d), dtype=tdt, device="cuda")
    for frames in (400, 40):
        vid = hippo.video_desc(frames, 15, 3, 0, 3, 3)
        beside = kernels(lambda: hippo.hippo_score_tokens(q, k[:, :, :frames * 45], vid))
        assert [x for x in beside if "with_embILi%dELi%dE" % (d, few) in x], beside
    alone = kernels(lambda: hippo.hippo_score_tokens(q, k, hippo.video_desc(655, 15, 3, 0, 3, 3), flags=hippo.SCORE_TEMP | hippo.SCORE_SPA))
    assert [x for x in alone if "emb_scores_run32" in x and "ELi%dEEE" % few in x], alone


@pytest.mark.parametrize("B, Hkv, d, L, video, channels, few", [
    # one sweep: 504 blocks, and 516, of which 512 run at once; two sweeps: 1341, of which 1024 do
    (4, 3, 128, 4, (46, 6, 12, 0, 5, 5), 192, True), (4, 3, 128, 4, (47, 6, 12, 0, 5, 5), 192, False),
    (4, 3, 128, 4, (47, 6, 12, 0, 5, 5), 64, True),
    (3, 3, 64, 16, (50, 14, 17, 0, 4, 3), 192, False), (3, 3, 64, 16, (50, 14, 17, 0, 4, 3), 128, True),
])
def test_fp32_embedding_blocks_beyond_what_runs_at_once(hippo, kernels, B, Hkv, d, L, video, channels, few):
    n = video[0] * video[1] * video[2]
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, emb = (torch.randn(shape, generator=g, device="cuda") for shape in ((B, L, 2 * Hkv, d), (B, Hkv, n, d), (B, n, channels)))
    vid = hippo.video_desc(*video)
    names = kernels(lambda: hippo.hippo_score_tokens(q, k, vid, emb=emb))
    assert [x for x in names if "with_embILi%dELi%dE" % (d, few) in x], names
    # the terms of a launch of their own, whose blocks are all of few channels: the same bits
    both, alone = (hippo.hippo_score_tokens(q, k, vid, emb=emb, flags=flags, want_components=True)[1]
                   for flags in (hippo.SCORE_ALL, hippo.SCORE_TEMP | hippo.SCORE_SPA))
    assert torch.equal(both[1:], alone[1:])


@pytest.mark.parametrize("d, B, Hkv, q_len, G, ctx", [
    # more than 256 MiB of K and V; 65, 72, 91 and 96 rows in one block, 97 in two; one slice a head, slices of a tile more or less
    (128, 8, 8, 13, 5, 8200), (128, 4, 16, 9, 8, 8190), (64, 8, 8, 13, 7, 16390), (128, 2, 32, 12, 8, 8201), (128, 8, 8, 97, 1, 8200),
    (64, 16, 32, 13, 7, 2100), (64, 66, 4, 13, 7, 4000),               # 512 heads in two chunks, 264 in one block a head
])
def test_65_to_96_rows_of_a_large_cache(hippo, d, B, Hkv, q_len, G, ctx):
    g = torch.Generator(device="cuda").manual_seed(ctx + G)
    shape = (B, Hkv, ctx + q_len, d)
    k, v = (torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    assert 4 * k.numel() > 256 << 20
    q = torch.randn((B, q_len, Hkv * G, d), generator=g, device="cuda").to(torch.bfloat16)
    unit = np.ones((B, Hkv, d))                                       # the slices' outputs keep their scale: of the values'
    unit[0, 0], unit[0, 1, ::2] = 2.0 ** 100, 2.0 ** -20              # unit, which the bound below holds in
    v *= torch.from_numpy(unit).cuda().unsqueeze(2)
    v[-1, -1, :, 3] = float("inf")                                    # and what is not finite to its channel
    q[1, :, :G] *= 8.0
    out, lse = hippo.hippo_verify_attention(q, k, v, ctx, want_lse=True)
    for b, hk in ((0, 0), (0, 1), (1, 0), (B - 1, Hkv - 1)):
        heads = slice(hk * G, hk * G + G)
        at = [c for c in range(d) if (b, hk, c) != (B - 1, Hkv - 1, 3)]
        rows = [host(x[b:b + 1, hk:hk + 1].contiguous()) for x in (k, v[..., at])]
        ref, ref_lse = oracle.attention(host(q[b:b + 1, :, heads].contiguous()), rows[0],
                                        np.pad(rows[1], ((0, 0),) * 3 + ((0, d - len(at)),)), ctx)
        got = host(out[b:b + 1, :, heads][..., at].contiguous())
        assert_close(got / unit[b, hk, at], ref[..., :len(at)] / unit[b, hk, at], "bf16", "head %d of %d" % (hk, b))
        np.testing.assert_allclose(host(lse[b:b + 1, heads].contiguous()), ref_lse, rtol=0, atol=2.0 ** -8)
    assert not torch.isfinite(out[-1, :, -G:, 3]).any()
    k2, v2 = k.clone(), v.clone()
    k2[:, :, ctx:], v2[:, :, ctx:] = 7.0, 7.0
    new = [x[:, :, ctx:].transpose(1, 2).contiguous() for x in (k, v)]
    bits = lambda x: x.view(torch.int16)
    assert torch.equal(bits(hippo.hippo_verify_attention(q, k2, v2, ctx, k_new=new[0], v_new=new[1])), bits(out))
    assert torch.equal(k2, k) and torch.equal(v2, v)
    del k2, v2
    pools, table = pages([k, v], 3)
    assert torch.equal(bits(hippo.hippo_verify_attention_paged(q, *pools, table, ctx)), bits(out))
    static = torch.empty_like(out)
    hippo.hippo_verify_attention_static(q, k, v, ctx, out=static)
    assert torch.equal(bits(static), bits(out))


@pytest.mark.parametrize("d, ctx, first_len, first_rows", [(64, 16500, 9000, 13), (64, 16500, 16516, 16), (128, 8300, 4000, 13)])
def test_65_to_96_rows_in_a_workspace_of_before_the_cache_grew(hippo, d, ctx, first_len, first_rows):
    # sized for a shorter cache, or for more rows: two chunks, the same bits as with their slices asked for
    B, Hkv, q_len, G = 8, 8, 13, 7
    g = torch.Generator(device="cuda").manual_seed(ctx)
    k, v = (torch.randn((B, Hkv, ctx + q_len, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    assert 4 * k.numel() > 256 << 20
    q = torch.randn((B, q_len, Hkv * G, d), generator=g, device="cuda").to(torch.bfloat16)
    kvd = hippo.kv_desc(k, Hkv * G)
    first, asked = (hippo.workspace_bytes(hippo.CALL_VERIFY_ATTENTION, kvd, None, rows, n)
                    for rows, n in ((first_rows, first_len), (q_len, ctx + q_len)))
    assert first < asked
    room = torch.full((first + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    out = hippo.hippo_verify_attention(q, k, v, ctx, workspace=room[:first])
    assert torch.all(room[first:] == 0x5A)
    assert torch.equal(out, hippo.hippo_verify_attention(q, k, v, ctx, num_splits=2))
    pools, table = pages([k, v], 3)
    assert torch.equal(hippo.hippo_verify_attention_paged(q, *pools, table, ctx, workspace=room[:first]), out)
    with pytest.raises(hippo.HippoError) as e:
        hippo.hippo_verify_attention(q, k, v, ctx, workspace=room[:first // 2])
    assert e.value.status == hippo.ERR_WORKSPACE_TOO_SMALL


@pytest.mark.parametrize("H, Hkv, d, F, gh, gw, L", [(32, 8, 128, 27, 13, 8, 46), (14, 2, 64, 16, 16, 16, 64)])
def test_short_videos_in_a_workspace_without_room_for_finer_cuts(hippo, H, Hkv, d, F, gh, gw, L):
    n, vid = F * gh * gw, hippo.video_desc(F, gh, gw, 0)
    q, k = score_inputs(L, 1, L, H, Hkv, d, n, "bf16")
    qd, kd = dev(q, "bf16"), dev(k, "bf16")
    need = hippo.workspace_bytes(hippo.CALL_SCORE_TOKENS, hippo.kv_desc(kd, H), vid, L, n)
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    for short in (0, 256):                                  # all it asks for; a little less
        mass = torch.zeros((1, n), device="cuda")
        hippo.hippo_score_tokens(qd, kd, vid, flags=hippo.SCORE_ACCUMULATE_ONLY, attn_mass_inout=mass, workspace=ws[:need - short])
        assert torch.all(ws[need - short:] == 0x5A)
        assert_close(host(mass), oracle.s_attn(q, k, 0, n), "bf16", "%d bytes short" % short)


@pytest.mark.parametrize("d, B, Hkv, q_len, G, ctx", [(128, 8, 8, 13, 5, 8200), (64, 8, 8, 13, 7, 16390), (128, 2, 32, 12, 8, 8201)])
def test_65_to_96_rows_keep_channels_of_any_unit(hippo, d, B, Hkv, q_len, G, ctx):
    """Channels far below their neighbours keep the bits that bf16 slices give them: each is compared in its own unit."""
    g = torch.Generator(device="cuda").manual_seed(ctx + d)
    k, v = (torch.randn((B, Hkv, ctx + q_len, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    assert 4 * k.numel() > 256 << 20
    q = torch.randn((B, q_len, Hkv * G, d), generator=g, device="cuda").to(torch.bfloat16)
    unit = np.ones((B, Hkv, d))
    unit[0, 0, ::2], unit[0, 1, 1::4], unit[1, 0, :d // 2], unit[1, 1, 5] = 2.0 ** -33, 2.0 ** -45, 2.0 ** -90, 2.0 ** 60
    unit[0, 2], unit[0, 2, 9] = 2.0 ** -105, 0.0
    v *= torch.from_numpy(unit).cuda().unsqueeze(2)
    out = hippo.hippo_verify_attention(q, k, v, ctx)
    for b, hk in ((0, 0), (0, 1), (1, 0), (1, 1), (0, 2)):
        heads, at = slice(hk * G, hk * G + G), np.flatnonzero(unit[b, hk])
        own = unit[b, hk, at]
        ref, _ = oracle.attention(host(q[b:b + 1, :, heads].contiguous()), host(k[b:b + 1, hk:hk + 1].contiguous()),
                                  np.pad(host(v[b:b + 1, hk:hk + 1][..., at].contiguous()) / own, ((0, 0),) * 3 + ((0, d - len(at)),)),
                                  ctx)
        got = host(out[b:b + 1, :, heads].contiguous())
        assert_close(got[..., at] / own, ref[..., :len(at)], "bf16", "head %d of %d" % (hk, b))
        assert not got[..., unit[b, hk] == 0].any()
