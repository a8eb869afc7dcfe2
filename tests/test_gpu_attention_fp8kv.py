"""GPU parity: hippo_verify_attention_fp8kv / hippo_draft_attention_fp8kv (through the C ABI) vs the
CPU oracle's attention over the dequantised cache.  The arithmetic is the bf16 path's (codes convert
to bf16 exactly, the multipliers are fp32 factors), so the bf16 tolerances apply unchanged."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from parity_util import assert_close, dev, host, prep

pytestmark = pytest.mark.gpu


def codes_dev(c: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(c)).cuda()


def run_case(hippo, q, k, v, ctx, num_splits=0, scale=0.0, fn="verify", what=""):
    q = prep(q, "bf16")
    kc, km = si.quantize_e4m3(k)
    vc, vm = si.quantize_e4m3(v)
    f = hippo.hippo_verify_attention_fp8kv if fn == "verify" else hippo.hippo_draft_attention_fp8kv
    out, lse = f(dev(q, "bf16"), codes_dev(kc), codes_dev(vc), torch.from_numpy(km).cuda(),
                 torch.from_numpy(vm).cuda(), ctx, softmax_scale=scale, num_splits=num_splits, want_lse=True)
    torch.cuda.synchronize()
    ro, rl = oracle.attention_fp8kv(q, kc, vc, km, vm, ctx, scale if scale > 0 else None)
    assert_close(host(out), ro, "bf16", what + " out")
    np.testing.assert_allclose(host(lse), rl, rtol=2.0 ** -9, atol=2.0 ** -9, err_msg=what + " lse")
    return host(out)


def rand_case(seed, B, ql, H, Hkv, d, ctx, qscale=1.0):
    r = np.random.default_rng(seed)
    q = r.standard_normal((B, ql, H, d)) * qscale
    k = r.standard_normal((B, Hkv, ctx + ql, d))
    # unequal magnitudes per (batch element, KV head), so the multipliers differ
    v = r.standard_normal((B, Hkv, ctx + ql, d)) * r.uniform(0.3, 3.0, (B, Hkv, 1, 1))
    return q, k, v


@pytest.mark.parametrize("shape", [
    # B, q_len, H, Hkv, d, ctx
    (1, 1, 4, 4, 64, 1),          # single context row, MHA
    (2, 3, 8, 2, 64, 37),         # ragged, barely more than one tile
    (1, 9, 7, 1, 128, 333),       # R = 63, one KV head
    (2, 5, 16, 2, 128, 1000),     # R = 40
    (1, 6, 28, 4, 128, 2049),     # headline head geometry, tile-boundary tail
    (1, 2, 6, 2, 64, 0),          # empty context: rows see only the new tokens
    (1, 12, 16, 2, 64, 515),      # R = 96 > 64: more than one row chunk
    (1, 1, 28, 4, 128, 832),      # the draft call's shape
])
def test_random_shapes_sharp_softmax(hippo, shape):
    B, ql, H, Hkv, d, ctx = shape
    q, k, v = rand_case(hash(shape) % 1000, B, ql, H, Hkv, d, ctx, qscale=3.0)
    # library-chosen slices, one slice (long slices: the four-group variant), and a few
    for s in (0, 1, 3):
        run_case(hippo, q, k, v, ctx, s, what="%s S=%d" % (shape, s))
    run_case(hippo, q, k, v, ctx, 0, fn="draft", what="%s draft" % (shape,))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("shape", [
    # q_len, G, ctx, forced slices: slices of at least 24 32-token tiles (four token groups, two stages)
    (1, 7, 4096, 1),              # R = 7: one 16-row block
    (1, 7, 4096, 2),
    (5, 4, 2048, 1),              # R = 20: two row blocks
    (9, 7, 3072, 2),              # R = 63: four row blocks
    (3, 14, 1700, 1),             # R = 42: three row blocks, ragged last tile
])
def test_long_slices_every_row_block_count(hippo, shape, d):
    ql, G, ctx, S = shape
    q, k, v = rand_case(ql * 1000 + G + d, 1, ql, 2 * G, 2, d, ctx, qscale=3.0 if d == 64 else 2.5)
    run_case(hippo, q, k, v, ctx, S, what="fp8 long slices %s d=%d" % (shape, d))


def test_causal_mask_probe_with_one_hot_values(hippo):
    # V = identity (code 0x38 = 1.0): the output IS the probability row; mass beyond ctx+i must be 0
    B, ql, H, Hkv, d, ctx = 1, 6, 4, 2, 128, 100
    n = ctx + ql
    q, k, _ = rand_case(5, B, ql, H, Hkv, d, ctx)
    v = np.zeros((B, Hkv, n, d), np.float32)
    v[:, :, np.arange(n), np.arange(n)] = 1.0
    out = run_case(hippo, q, k, v, ctx, what="probe")
    for i in range(ql):
        assert np.all(out[0, i, :, ctx + i + 1:] == 0.0)
        np.testing.assert_allclose(out[0, i].sum(-1), 1.0, atol=2e-2)
    ones = run_case(hippo, q, k, np.ones_like(v), ctx, what="rows sum to 1")
    np.testing.assert_allclose(ones, 1.0, atol=8e-3)


def test_token_order_probe(hippo):
    # the fp8 path permutes tile rows between the K operand and the V read: give every token its own
    # value vector and a query that picks exactly one token, for every token of two tiles and a tail
    B, H, Hkv, d, n = 1, 2, 1, 64, 75
    r = np.random.default_rng(3)
    k = r.standard_normal((B, Hkv, n, d)).astype(np.float32)
    k /= np.linalg.norm(k, axis=-1, keepdims=True)
    v = r.standard_normal((B, Hkv, n, d)).astype(np.float32)
    kc, km = si.quantize_e4m3(k)
    vc, vm = si.quantize_e4m3(v)
    kdec = oracle.e4m3_decode(kc) * km[:, :, None, None]
    vdec = oracle.e4m3_decode(vc) * vm[:, :, None, None]
    for t in range(n - 1):
        q = np.zeros((B, 1, H, d), np.float32)
        q[0, 0, :, :] = 200.0 * kdec[0, 0, t] / np.linalg.norm(kdec[0, 0, t])
        q = prep(q, "bf16")
        out = hippo.hippo_verify_attention_fp8kv(dev(q, "bf16"), codes_dev(kc), codes_dev(vc),
                                                 torch.from_numpy(km).cuda(), torch.from_numpy(vm).cuda(), n - 1)
        ro, _ = oracle.attention_fp8kv(q, kc, vc, km, vm, n - 1)
        assert_close(host(out), ro, "bf16", "token %d" % t)
    assert np.abs(ro[0, 0, 0] - vdec[0, 0, n - 2]).max() < 0.2     # the probe does isolate one token


def test_strided_caches_and_custom_scale(hippo):
    # K and V interleaved in one allocation ([B,Hkv,N_alloc,2,d]): stride_n = 2d, oversized stride_h
    B, ql, H, Hkv, d, ctx = 2, 4, 6, 3, 64, 150
    q, k, v = rand_case(11, B, ql, H, Hkv, d, ctx)
    q = prep(q, "bf16")
    kc, km = si.quantize_e4m3(k)
    vc, vm = si.quantize_e4m3(v)
    n, n_alloc = ctx + ql, ctx + ql + 13
    buf = torch.zeros((B, Hkv, n_alloc, 2, d), dtype=torch.uint8, device="cuda")
    buf[:, :, :n, 0] = codes_dev(kc)
    buf[:, :, :n, 1] = codes_dev(vc)
    kd, vd = buf[:, :, :, 0], buf[:, :, :, 1]
    assert kd.stride(2) == 2 * d
    out = hippo.hippo_verify_attention_fp8kv(dev(q, "bf16"), kd, vd, torch.from_numpy(km).cuda(),
                                             torch.from_numpy(vm).cuda(), ctx, softmax_scale=0.21)
    torch.cuda.synchronize()
    ro, _ = oracle.attention_fp8kv(q, kc, vc, km, vm, ctx, 0.21)
    assert_close(host(out), ro, "bf16", "strided")


def test_split_count_does_not_change_the_result(hippo):
    q, k, v = rand_case(12, 1, 5, 28, 4, 128, 3000)
    outs = [run_case(hippo, q, k, v, 3000, s, what="S=%d" % s) for s in (1, 2, 5, 33)]
    for o in outs[1:]:
        assert np.max(np.abs(o - outs[0])) <= 2 ** -7 * np.max(np.abs(outs[0])) + 1e-6


@pytest.mark.parametrize("name", ["c3_16k", "c4_long"])
def test_full_size(hippo, name):
    """The benchmark shapes with their caches quantised, in the launch configuration bench.py times."""
    cfg = si.CONFIGS[name]
    x = si.make_inputs(cfg, 0)
    run_case(hippo, x["q_new"], x["k"], x["v"], cfg.ctx_len, 0, what=name)


def test_prune_then_draft_attention_on_an_fp8_cache(hippo):
    """The draft path with an 8-bit cache end to end: the gather copies the kept rows' codes (bit
    exact, the per-head multipliers stay valid), and the draft attention over the pruned codes equals
    the oracle's attention over the same rows of the dequantised cache."""
    cfg = si.CONFIGS["draft"]
    x = si.make_inputs(cfg, 4)
    n = cfg.ctx_len + 1                                   # context + the draft token's own row
    kc, km = si.quantize_e4m3(x["k"][:, :, :n])
    vc, vm = si.quantize_e4m3(x["v"][:, :, :n])
    r = np.random.default_rng(0)
    scores = r.standard_normal((cfg.batch, cfg.n_visual)).astype(np.float32)
    k_keep = (cfg.n_visual * cfg.keep_pct + 99) // 100
    vid = hippo.video_desc(cfg.n_frames, cfg.grid_h, cfg.grid_w, cfg.n_prefix)
    idx, kp, vp = hippo.hippo_select_gather_kv(torch.from_numpy(scores).cuda(), k_keep, codes_dev(kc), codes_dev(vc),
                                               vid, cfg.n_q_heads)
    torch.cuda.synchronize()
    ridx = oracle.topk(scores, k_keep)
    np.testing.assert_array_equal(idx.cpu().numpy(), ridx)
    rows = np.concatenate([np.arange(cfg.n_prefix), cfg.n_prefix + ridx[0],
                           np.arange(cfg.n_prefix + cfg.n_visual, n)])
    assert cfg.batch == 1
    np.testing.assert_array_equal(kp.cpu().numpy(), kc[:, :, rows])
    np.testing.assert_array_equal(vp.cpu().numpy(), vc[:, :, rows])
    q = prep(x["q_new"][:, :1], "bf16")
    ctx = len(rows) - 1
    out = hippo.hippo_draft_attention_fp8kv(dev(q, "bf16"), kp, vp, torch.from_numpy(km).cuda(),
                                            torch.from_numpy(vm).cuda(), ctx)
    torch.cuda.synchronize()
    ro, _ = oracle.attention_fp8kv(q, kc[:, :, rows], vc[:, :, rows], km, vm, ctx)
    assert_close(host(out), ro, "bf16", "draft attention over the pruned fp8 cache")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("shape", [(1, 1, 1, 64), (2, 3, 77, 64), (1, 4, 1670, 128), (2, 2, 5000, 128)])
def test_quantize_kv_bit_exact(hippo, dtype, shape):
    """The library's writer of the 8-bit format against the oracle's: codes and multipliers bit for bit
    (values spread over eight octaves per head, planted zeros, ties and the subnormal range)."""
    B, Hkv, N, d = shape
    r = np.random.default_rng(N)
    mag = np.exp2(r.uniform(-9, 8, (B, Hkv, N, d)))
    k = prep(r.standard_normal(shape) * mag, dtype)
    v = prep(r.standard_normal(shape) * r.uniform(0.05, 20, (B, Hkv, 1, 1)), dtype)
    k[:, :, ::7, ::5] = 0.0
    v[0, 0] = 0.0                                           # an all-zero head: multiplier 1, codes 0
    if N > 8:
        # one head whose maximum is exactly 448: the values themselves are encoded, ties included
        k[0, -1] = np.clip(k[0, -1], -400, 400)
        k[0, -1, 0, :8] = [448.0, 1.0625, 1.1875, -1.0625, 2.0 ** -10, 1.5 * 2.0 ** -9, 2.5 * 2.0 ** -9, -0.0]
    kd, vd = dev(k, dtype), dev(v, dtype)
    kc, vc, ks, vs = hippo.hippo_quantize_kv_e4m3(kd, vd)
    torch.cuda.synchronize()
    rk, rkm = oracle.quantize_e4m3(k)
    rv, rvm = oracle.quantize_e4m3(v)
    np.testing.assert_array_equal(ks.cpu().numpy(), rkm)
    np.testing.assert_array_equal(vs.cpu().numpy(), rvm)
    np.testing.assert_array_equal(kc.cpu().numpy(), rk)
    np.testing.assert_array_equal(vc.cpu().numpy(), rv)


def test_quantize_strided_prefix_then_attend(hippo):
    """Quantise the first n rows of caches that sit interleaved in one allocation, into a larger code
    buffer, then attend over the codes: equals the oracle's attention over its own quantisation."""
    B, ql, H, Hkv, d, ctx = 2, 3, 8, 2, 128, 300
    q, k, v = rand_case(21, B, ql, H, Hkv, d, ctx)
    q, k, v = prep(q, "bf16"), prep(k, "bf16"), prep(v, "bf16")
    n = ctx + ql
    buf = torch.zeros((B, Hkv, n + 9, 2, d), dtype=torch.bfloat16, device="cuda")
    buf[:, :, :n, 0] = dev(k, "bf16")
    buf[:, :, :n, 1] = dev(v, "bf16")
    buf[:, :, n:] = 1000.0                                   # rows beyond n must not reach the maximum
    codes = torch.full((B, Hkv, n + 20, 2, d), 0x7F, dtype=torch.uint8, device="cuda")
    kc, vc, ks, vs = hippo.hippo_quantize_kv_e4m3(buf[:, :, :, 0], buf[:, :, :, 1], n_rows=n,
                                                  k_codes=codes[:, :, :, 0], v_codes=codes[:, :, :, 1])
    out = hippo.hippo_verify_attention_fp8kv(dev(q, "bf16"), kc, vc, ks, vs, ctx)
    torch.cuda.synchronize()
    rk, rkm = oracle.quantize_e4m3(k)
    rv, rvm = oracle.quantize_e4m3(v)
    np.testing.assert_array_equal(kc[:, :, :n].cpu().numpy(), rk)
    np.testing.assert_array_equal(ks.cpu().numpy(), rkm)
    assert torch.all(codes[:, :, n:] == 0x7F)                # nothing written past n_rows
    ro, _ = oracle.attention_fp8kv(q, rk, rv, rkm, rvm, ctx)
    assert_close(host(out), ro, "bf16", "attention over the library's own quantisation")


def quantize(hippo, k, v, n, polls):
    """hippo_quantize_kv_e4m3 whose blocks look `polls` times for each other's maxima, into code rows with a gap"""
    lib = hippo.load()
    fn = lib.hippo_quantize_kv_e4m3_polls
    fn.argtypes, fn.restype = lib.hippo_quantize_kv_e4m3.argtypes + [C.c_int32], C.c_int
    B, Hkv, _, d = k.shape
    codes = torch.full((2, B, Hkv, n + 1, d + 16), 0x7F, dtype=torch.uint8, device="cuda")[..., :d]
    scale = torch.full((2, B, Hkv), -1.0, device="cuda")
    src, dst = hippo.kv_desc(k, Hkv), hippo.kv_desc(codes[0], Hkv)
    ws = torch.full((lib.hippo_quantize_kv_workspace_bytes(C.byref(src), n),), 1, dtype=torch.uint8, device="cuda")
    hippo._check(fn(k.data_ptr(), v.data_ptr(), C.byref(src), n, codes[0].data_ptr(), codes[1].data_ptr(), C.byref(dst),
                    scale[0].data_ptr(), scale[1].data_ptr(), ws.data_ptr(), ws.numel(), hippo._stream(None), polls),
                 "hippo_quantize_kv_e4m3_polls")
    return codes, scale


@pytest.mark.parametrize("B, Hkv, n, d, dtype", [
    # one slice a head: registers full, the first vectors in LDS, both full; two; two
    (24, 12, 512, 128, "bf16"), (24, 12, 513, 128, "bf16"), (16, 12, 768, 128, "bf16"), (16, 12, 769, 128, "bf16"),
    (40, 6, 640, 128, "fp32"),
    (2, 3, 53001, 64, "bf16"), (1, 3, 25001, 128, "fp32"), (1, 2, 131072, 128, "bf16"),  # 35, 66 and 171, the last ones short
    (2, 4, 68001, 128, "bf16"), (3, 4, 45003, 64, "fp32"),                               # fetched past the caches
    (1, 1, 73729, 128, "bf16"), (1, 8, 9217, 128, "bf16"),                               # just above 36 MiB
])
def test_large_sources_are_quantised_as_their_heads_are(hippo, B, Hkv, n, d, dtype):
    """A source of many megabytes, whose slices stay on the chip, against its heads one by one, which take two launches:
    the same codes and multipliers, whatever the blocks' waits come to."""
    g = torch.Generator(device="cuda").manual_seed(n)
    rows = torch.randn((2, B, Hkv, n + 2, d + 8), generator=g, device="cuda")[..., :d]
    rows *= torch.exp2(torch.randint(-9, 9, (2, B, Hkv, 1, 1), generator=g, device="cuda").float())
    # every head's largest value in a row of its own, another sign in V; a head of zeros, a tiny one; rows beyond n larger
    at = torch.randint(0, n, (B, Hkv), generator=g, device="cuda")
    at.view(-1)[-1] = n - 1
    b, hk = torch.meshgrid(torch.arange(B, device="cuda"), torch.arange(Hkv, device="cuda"), indexing="ij")
    rows[0, b, hk, at, d - 1], rows[1, b, hk, at, 0] = 5000.0, -7000.0
    rows[:, :, :, n:] = 1e6
    rows[1, 0, 0, :n] = 0.0
    rows[0, -1, 0, :n] *= 2.0 ** -100
    k, v = rows.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    want = []
    for i in range(B):
        for j in range(Hkv):          # pieces of less than 36 MiB, each with the row of its head's largest values
            parts, top = [], at[i, j].view(1)
            for lo in range(0, n, 65536):
                index = torch.cat([torch.arange(lo, min(n, lo + 65536), device="cuda"), top])
                parts.append(hippo.hippo_quantize_kv_e4m3(*(x[i:i + 1, j:j + 1, index] for x in (k, v))))
            assert all(torch.equal(part[2 + t], parts[0][2 + t]) for part in parts for t in (0, 1))
            want.append([torch.cat([part[t][:, :, :-1] for part in parts], 2) for t in (0, 1)] + list(parts[0][2:]))
    for polls in (-1, 0, 1):
        codes, scale = quantize(hippo, k, v, n, polls)
        assert torch.equal(scale, torch.stack([torch.cat([w[2 + t] for w in want]).view(B, Hkv) for t in (0, 1)]))
        for t in (0, 1):
            assert torch.equal(codes[t, :, :, :n], torch.cat([w[t] for w in want], 1).view(B, Hkv, n, d)), "%d looks" % polls
        assert torch.all(codes[:, :, :, n:] == 0x7F)


@pytest.mark.parametrize("B, Hkv, n, d, dtype, once", [
    # 26 KB a head from 36 MiB on, 50 KB from 256 MiB on; just below 36 MiB, and there
    (64, 32, 207, 64, "bf16", False), (64, 32, 208, 64, "bf16", True), (32, 32, 51, 128, "fp32", False), (32, 32, 52, 128, "fp32", True),
    (94, 32, 199, 128, "bf16", False), (94, 32, 200, 128, "bf16", True), (260, 32, 108, 128, "bf16", False),
    (1, 8, 9215, 128, "bf16", False), (1, 8, 9216, 128, "bf16", True),
])
def test_which_heads_are_quantised_in_one_sweep(hippo, kernels, B, Hkv, n, d, dtype, once):
    g = torch.Generator(device="cuda").manual_seed(n)
    k, v = (torch.randn((B, Hkv, n, d), generator=g, device="cuda").to(torch.float32 if dtype == "fp32" else torch.bfloat16)
            for _ in range(2))
    names = kernels(lambda: hippo.hippo_quantize_kv_e4m3(k, v))
    assert any("kv_quantize_once" in x for x in names) == once
    assert any("kv_absmax" in x for x in names) != once
    whole = hippo.hippo_quantize_kv_e4m3(k, v)
    few = slice(0, None, 9)                                 # in two launches, unless they are many heads too
    assert all(torch.equal(x[few], y) for x, y in zip(whole, hippo.hippo_quantize_kv_e4m3(k[few], v[few])))


def test_quantised_heads_of_the_most_slices(hippo):
    # 256 slices of 192 KB; a row of zeros more, which changes no maximum, takes two launches
    g = torch.Generator(device="cuda").manual_seed(5)
    n = 256 * 192 * 1024 // 256
    x = torch.zeros((2, 1, 1, n + 1, 128), dtype=torch.bfloat16, device="cuda")
    x[..., :n, :] = torch.randn((2, 1, 1, n, 128), generator=g, device="cuda")
    want = hippo.hippo_quantize_kv_e4m3(*x)
    for polls in (-1, 2):
        codes, scale = quantize(hippo, x[0], x[1], n, polls)
        assert torch.equal(scale, torch.stack(want[2:]))
        assert all(torch.equal(codes[t, :, :, :n], want[t][:, :, :n]) for t in (0, 1))


def test_two_large_quantisations_share_the_gpu(hippo):
    g = torch.Generator(device="cuda").manual_seed(3)
    data = [torch.randn((2, 1, 4, 90001, 128), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
    alone = [hippo.hippo_quantize_kv_e4m3(k, v) for k, v in data]
    torch.cuda.synchronize()
    streams, together = [torch.cuda.Stream() for _ in data], [[], []]
    for _ in range(3):
        for i, s in enumerate(streams):
            together[i].append(hippo.hippo_quantize_kv_e4m3(*data[i], stream=s))
    torch.cuda.synchronize()
    for ref, got in zip(alone, together):
        for x in got:
            assert all(torch.equal(a, b) for a, b in zip(ref, x))


def test_large_quantisations_at_once_do_not_take_each_others_work(hippo):
    """Three calls whose heads do not fit the chip together: blocks wait for maxima of slices that have no place yet, and share
    those between them.  (Each taking all of them took 30 times as long as one call after the other; here 1.5 times.)"""
    g = torch.Generator(device="cuda").manual_seed(8)
    data = [torch.randn((2, 1, 8, 196000, 128), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3)]
    alone = [hippo.hippo_quantize_kv_e4m3(k, v) for k, v in data]
    streams = [torch.cuda.Stream() for _ in data]
    out = [[torch.empty_like(x) for x in a[:2]] for a in alone]

    def run(streams):
        got, begin, ends = [], torch.cuda.Event(enable_timing=True), []
        torch.cuda.synchronize()
        begin.record()
        for s in set(streams):
            s.wait_event(begin)
        for _ in range(4):
            for (k, v), (kc, vc), s in zip(data, out, streams):
                got.append(hippo.hippo_quantize_kv_e4m3(k, v, k_codes=kc, v_codes=vc, stream=s))
        for s in set(streams):
            ends.append(torch.cuda.Event(enable_timing=True))
            ends[-1].record(s)
        torch.cuda.synchronize()
        return max(begin.elapsed_time(e) for e in ends), got[-3:]

    run(streams)
    in_turn = min(run(streams[:1] * 3)[0] for _ in range(3))
    for _ in range(3):
        time, got = run(streams)
        assert time < 5 * in_turn
        for ref, x in zip(alone, got):
            assert all(torch.equal(a, b) for a, b in zip(ref, x))
