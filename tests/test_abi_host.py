"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments with the documented status before launching anything.
Pointers handed over here are fake, aligned, non-null addresses -- they are never dereferenced
because validation fails first."""
import ctypes as C
import itertools
import os
import re

import pytest

import paper_2601_08273_amd as h

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x10000          # 256-byte aligned, never touched


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(h.LIB_PATH):
        from paper_2601_08273_amd import build
        build.build(verbose=False)
    return h.load()


def test_exports_match_header(lib):
    text = open(os.path.join(ROOT, "include", "hippo.h")).read()
    declared = set(re.findall(r"\b(hippo_[a-z0-9_]+)\s*\(", text))
    assert declared == set(h.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name


def test_header_is_plain_c(tmp_path):
    """The boundary is a C ABI: the header must compile as C99 on its own, without warnings."""
    import subprocess
    src = tmp_path / "use_header.c"
    src.write_text('#include "hippo.h"\nint main(void) { return (int)sizeof(hippo_kv_desc) == 0; }\n')
    r = subprocess.run(["gcc", "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-fsyntax-only",
                        "-I", os.path.join(ROOT, "include"), str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_struct_layout_matches_header():
    assert C.sizeof(h.KvDesc) == 48 and h.KvDesc.stride_b.offset == 24
    assert C.sizeof(h.VideoDesc) == 24


def test_status_strings(lib):
    seen = {h.status_string(s) for s in range(8)}
    assert len(seen) == 8 and h.status_string(0) == "ok"
    assert "unknown" in h.status_string(99)


def _kv(**kw):
    d = dict(batch=1, n_q_heads=28, n_kv_heads=4, head_dim=128, dtype=h.DTYPE_BF16)
    d.update(kw)
    n = 20000
    d.setdefault("stride_n", d["head_dim"])
    d.setdefault("stride_h", n * d["head_dim"])
    d.setdefault("stride_b", d["n_kv_heads"] * n * d["head_dim"])
    return h.KvDesc(**d)


def _verify(lib, kv, q_len=6, ctx=16640, ws_bytes=1 << 30, q=FAKE, k=FAKE, v=FAKE, out=FAKE, ws=FAKE, splits=0,
            fn="hippo_verify_attention"):
    return getattr(lib, fn)(q, q_len, k, v, C.byref(kv), ctx, 0.0, splits, out, None, ws, ws_bytes, None)


def test_attention_argument_errors(lib):
    kv = _kv()
    for fn in ("hippo_verify_attention", "hippo_draft_attention"):
        assert _verify(lib, kv, q=None, fn=fn) == h.ERR_NULL_ARG
        assert _verify(lib, kv, out=None, fn=fn) == h.ERR_NULL_ARG
        assert _verify(lib, kv, ws=None, fn=fn) == h.ERR_NULL_ARG
        assert _verify(lib, kv, q_len=0, fn=fn) == h.ERR_BAD_SHAPE
        assert _verify(lib, kv, ctx=-1, fn=fn) == h.ERR_BAD_SHAPE
        assert _verify(lib, kv, splits=-2, fn=fn) == h.ERR_BAD_SHAPE
        assert _verify(lib, kv, k=FAKE + 8, fn=fn) == h.ERR_BAD_ALIGN
        assert _verify(lib, kv, ws=FAKE + 16, fn=fn) == h.ERR_BAD_ALIGN
        assert _verify(lib, kv, ws_bytes=1024, fn=fn) == h.ERR_WORKSPACE_TOO_SMALL
    assert _verify(lib, _kv(dtype=7)) == h.ERR_BAD_DTYPE
    assert _verify(lib, _kv(head_dim=96)) == h.ERR_BAD_SHAPE
    assert _verify(lib, _kv(n_q_heads=30)) == h.ERR_BAD_SHAPE          # not a multiple of n_kv_heads
    assert _verify(lib, _kv(stride_n=64)) == h.ERR_BAD_SHAPE           # rows overlap
    assert _verify(lib, _kv(stride_n=132)) == h.ERR_BAD_ALIGN          # 264-byte rows
    assert lib.hippo_verify_attention(FAKE, 6, FAKE, FAKE, None, 10, 0.0, 0, FAKE, None, FAKE, 1 << 20, None) \
        == h.ERR_NULL_ARG


def test_static_scratch_argument_errors(lib):
    """The entry point without a workspace: every refusal below happens before the device is touched."""
    def call(kv, q_len=6, ctx=16640, q=FAKE, k=FAKE, v=FAKE, out=FAKE, splits=0):
        return lib.hippo_verify_attention_static(q, q_len, k, v, C.byref(kv), ctx, 0.0, splits, out, None, None)
    kv = _kv()
    limit = lib.hippo_static_scratch_bytes()
    assert limit == 8 << 20
    assert call(kv, q=None) == h.ERR_NULL_ARG
    assert call(kv, out=None) == h.ERR_NULL_ARG
    assert call(kv, q_len=0) == h.ERR_BAD_SHAPE
    assert call(kv, ctx=-1) == h.ERR_BAD_SHAPE
    assert call(_kv(dtype=7)) == h.ERR_BAD_DTYPE
    assert call(_kv(head_dim=96)) == h.ERR_BAD_SHAPE
    # the headline shape fits; four sequences of eight KV heads with 64 forced slices do not
    assert h.workspace_bytes(h.CALL_VERIFY_ATTENTION, kv, None, 6, 16646) <= limit
    big = _kv(batch=4, n_q_heads=64, n_kv_heads=8)
    assert h.workspace_bytes(h.CALL_VERIFY_ATTENTION, big, None, 6, 37126, 0, 64) > limit
    assert call(big, ctx=37120, splits=64) == h.ERR_STATIC_SCRATCH_LIMIT
    assert "static" in h.status_string(h.ERR_STATIC_SCRATCH_LIMIT)


def test_static_scratch_holds_the_librarys_choice_of_slices(lib):
    """What the library plans by itself fits the static array wherever one slice per KV head does: the static call and
    the workspace call then take the same slices, and only what cannot be served at all is refused."""
    limit = lib.hippo_static_scratch_bytes()
    for dtype in (h.DTYPE_F32, h.DTYPE_BF16):
        for batch, heads, group, d, q_len, ctx in itertools.product((1, 2, 5, 16, 70), (1, 2, 4, 8), (1, 5, 8), (64, 128),
                                                                    (1, 8, 13, 16, 25, 64), (0, 500, 9000, 33280)):
            kv = _kv(batch=batch, n_q_heads=heads * group, n_kv_heads=heads, head_dim=d, dtype=dtype)
            need, one = (h.workspace_bytes(h.CALL_VERIFY_ATTENTION, kv, None, q_len, ctx + q_len, 0, s) for s in (0, 1))
            assert 0 < need <= max(limit, one), (dtype, batch, heads, group, d, q_len, ctx)


def test_workspace_query(lib):
    kv = _kv()
    need = h.workspace_bytes(h.CALL_VERIFY_ATTENTION, kv, None, 6, 16646)
    assert need > 0 and need % 256 == 0
    assert _verify(lib, kv, ws_bytes=need - 1) == h.ERR_WORKSPACE_TOO_SMALL
    # more splits need more room; explicit split count is honoured by the query
    assert h.workspace_bytes(h.CALL_VERIFY_ATTENTION, kv, None, 6, 16646, 0, 128) > \
        h.workspace_bytes(h.CALL_VERIFY_ATTENTION, kv, None, 6, 16646, 0, 8)
    assert h.workspace_bytes(h.CALL_VERIFY_ATTENTION, _kv(dtype=9), None, 6, 16646) == 0
    assert h.workspace_bytes(42, kv, None, 6, 16646) == 0
    vid = h.video_desc(64, 16, 16, 128)
    assert h.workspace_bytes(h.CALL_SCORE_TOKENS, kv, vid, 128, 16646) > 0
    assert h.workspace_bytes(h.CALL_SCORE_TOKENS, kv, None, 128, 16646) == 0
    assert h.workspace_bytes(h.CALL_SELECT_GATHER_KV, kv, vid, 0, 16646, 1639) >= 256


@pytest.mark.parametrize("batch, heads, d, rows, one", [
    (32, 8, 64, 80, True), (33, 8, 64, 80, False), (33, 8, 64, 64, False), (12, 32, 64, 96, False), (80, 8, 64, 68, False),
    (2, 160, 64, 80, False), (2, 192, 64, 80, True), (66, 4, 64, 80, True), (22, 12, 64, 80, True), (300, 1, 64, 80, True),
    (32, 8, 128, 80, True), (33, 8, 128, 80, False), (12, 32, 128, 80, False), (8, 40, 128, 80, True), (50, 8, 128, 68, True),
    (321, 1, 128, 96, True), (322, 1, 128, 96, False), (606, 1, 64, 96, True), (607, 1, 64, 96, False),
])
def test_which_heads_take_65_to_96_rows_in_one_block(lib, batch, heads, d, rows, one):
    """The workspace says it: one block for all rows also stores two factors a row and slice."""
    al = lambda x: (x + 255) // 256 * 256
    kv = _kv(batch=batch, n_q_heads=heads * rows, n_kv_heads=heads, head_dim=d)
    slots = batch * heads * rows                            # rounds of one slice a head
    two = al(slots * d * 2) + 2 * al(slots * 4)
    need = h.workspace_bytes(h.CALL_VERIFY_ATTENTION, kv, None, 1, (300 << 20) // (4 * batch * heads * d))
    assert need == two + (al(slots * 8) if one else 0)


def test_a_workspace_outlives_the_growth_of_its_cache(lib):
    """What a decoding loop asked for at its first length, or for more query rows, is enough at every later one: 65 to 96 rows
    of a bf16 cache beyond 256 MiB need twice as much in one block, and take two chunks where there is less."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("what passes the checks is launched")
    for heads, group, d, q_len in itertools.product((1, 4, 8), (1, 5, 8), (64, 128), (9, 13, 16, 72, 91)):
        kv = _kv(batch=4, n_q_heads=heads * group, n_kv_heads=heads, head_dim=d)
        ask = lambda rows, n: h.workspace_bytes(h.CALL_VERIFY_ATTENTION, kv, None, rows, n)
        for n in (4000, 30000, 60000, 150000, 300000, 600000):
            for first in (ask(q_len, 4000), ask(2 * q_len, n) if 64 < q_len * group <= 96 else ask(q_len, n)):
                assert _verify(lib, kv, q_len=q_len, ctx=n - q_len, ws_bytes=first) == h.ERR_HIP     # no GPU: the launch fails
                assert _verify(lib, kv, q_len=q_len, ctx=n - q_len, ws_bytes=min(first, ask(q_len, 4000)) - 1) \
                    == h.ERR_WORKSPACE_TOO_SMALL


def _score(lib, kv, vid, l_txt=128, seq_len=16646, flags=h.SCORE_ALL, q=FAKE, k=FAKE, emb=None, emb_dim=0,
           emb_stride=0, mass=None, scores=FAKE, ws=FAKE, ws_bytes=1 << 32):
    return lib.hippo_score_tokens(q, l_txt, k, C.byref(kv), seq_len, C.byref(vid), emb, emb_dim, emb_stride,
                                  flags, mass, scores, None, ws, ws_bytes, None)


def test_score_argument_errors(lib):
    kv, vid = _kv(), h.video_desc(64, 16, 16, 128)
    assert _score(lib, kv, vid, q=None) == h.ERR_NULL_ARG
    assert _score(lib, kv, vid, scores=None) == h.ERR_NULL_ARG
    assert _score(lib, kv, vid, flags=h.SCORE_ACCUMULATE_ONLY, mass=None) == h.ERR_NULL_ARG
    assert _score(lib, kv, vid, flags=0) == h.ERR_BAD_SHAPE
    assert _score(lib, kv, vid, flags=64) == h.ERR_BAD_SHAPE
    assert _score(lib, kv, vid, l_txt=0) == h.ERR_BAD_SHAPE
    assert _score(lib, kv, vid, seq_len=16000) == h.ERR_BAD_SHAPE               # video runs past the cache
    assert _score(lib, kv, h.video_desc(64, 16, 16, 128, 9, 9)) == h.ERR_BAD_SHAPE   # 81-token crops
    assert _score(lib, kv, h.video_desc(0, 16, 16, 128)) == h.ERR_BAD_SHAPE
    assert _score(lib, kv, vid, emb=FAKE, emb_dim=100, emb_stride=104) == h.ERR_BAD_SHAPE   # dim % 8
    assert _score(lib, kv, vid, emb=FAKE, emb_dim=512, emb_stride=516) == h.ERR_BAD_ALIGN
    assert _score(lib, kv, vid, emb=FAKE + 2, emb_dim=512, emb_stride=512) == h.ERR_BAD_ALIGN
    assert _score(lib, kv, vid, ws_bytes=4096) == h.ERR_WORKSPACE_TOO_SMALL
    # shapes no kernel grid can hold are refused before the first launch: frames are a y dimension
    assert _score(lib, kv, h.video_desc(65536, 2, 2, 128), seq_len=1 << 20) == h.ERR_BAD_SHAPE
    assert _score(lib, kv, h.video_desc(65535, 2, 2, 128), seq_len=1 << 20, ws_bytes=4096) == h.ERR_WORKSPACE_TOO_SMALL
    # ... and the key tiles of the bf16 sweeps (256 tokens each): 65535 of them at most
    assert _score(lib, kv, h.video_desc(65535, 16, 17, 128), seq_len=1 << 25) == h.ERR_BAD_SHAPE
    assert _score(lib, kv, h.video_desc(65535, 16, 16, 0), seq_len=65535 * 256, ws_bytes=4096) == h.ERR_WORKSPACE_TOO_SMALL


@pytest.mark.parametrize("H, Hkv, d, n, L, layers, runs", [
    # one chunk of three on three quarters of the compute units and more; of fewer
    (64, 8, 128, 1836, 17, 2, 1), (28, 4, 128, 7680, 21, 1, 1), (28, 4, 128, 6825, 26, 1, 1), (28, 4, 128, 5120, 26, 1, 2),
    (14, 2, 64, 4600, 128, 1, 4), (14, 2, 64, 4600, 184, 1, 6), (4, 2, 64, 3360, 161, 1, 6),  # a chunk of four; two of six; one of two
    (14, 2, 64, 4096, 64, 1, 7), (28, 4, 128, 1400, 121, 1, 7), (28, 4, 128, 7000, 40, 1, 2),
    # 64 partials a token more for two chunks of three, 32 and 16 for one of two; 40 and 24 for one of three
    (8, 8, 64, 396, 154, 4, 1), (16, 8, 64, 462, 35, 4, 1), (16, 4, 128, 374, 30, 4, 2), (80, 10, 64, 768, 55, 1, 4), (64, 8, 64, 816, 55, 1, 7),
])
def test_runs_of_rows_of_short_videos(lib, H, Hkv, d, n, L, layers, runs):
    """Finer cuts where they save a third of a run's chunks and more: the column partials that are asked for say how many runs
    there are."""
    al = lambda x: (x + 255) // 256 * 256
    rows, tiles = H * L * layers, (n + 255) // 256
    rest = 2 * al(rows * tiles * 4) + al(rows * 4) + 3 * al(n * 4)
    need = lib.hippo_score_layers_workspace_bytes(C.byref(_kv(n_q_heads=H, n_kv_heads=Hkv, head_dim=d)),
                                                  C.byref(h.video_desc(1, 1, n, 0)), L, layers)
    assert need - rest == al(layers * Hkv * runs * n * 4)


def test_a_workspace_for_a_longer_video_serves_a_shorter_one(lib):
    """The finer cuts of short videos take more column partials than some longer ones need: less is enough without them."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("what passes the checks is launched")
    for (q_heads, heads, d), larger, smaller, least in (
            ((16, 2, 64), (492, 3, 4, 26, 1), (492, 3, 4, 18, 1), 175360),
            ((8, 1, 128), (10, 11, 21, 29, 4), (10, 11, 21, 29, 3), 142592),
            ((1, 1, 64), (506, 3, 9, 139, 2), (331, 3, 9, 139, 2), 258816),
            ((32, 8, 128), (28, 13, 8, 46, 1), (27, 13, 8, 46, 1), 259072)):
        kv = _kv(n_q_heads=q_heads, n_kv_heads=heads, head_dim=d)
        ask = lambda f, gh, gw, l, n: lib.hippo_score_layers_workspace_bytes(C.byref(kv), C.byref(h.video_desc(f, gh, gw, 0)), l, n)
        f, gh, gw, l, n = smaller
        layers = (C.c_void_p * n)(*[FAKE] * n)
        call = lambda bytes: lib.hippo_score_tokens_layers(n, layers, l, layers, 0, C.byref(kv), f * gh * gw,
                                                           C.byref(h.video_desc(f, gh, gw, 0)), None, 0, 0, h.SCORE_ALL, None,
                                                           FAKE, None, FAKE, bytes, None)
        assert least < ask(*larger) < ask(*smaller)
        assert call(ask(*larger)) == call(least) == h.ERR_HIP                  # no GPU: the launch fails
        assert call(least - 1) == h.ERR_WORKSPACE_TOO_SMALL


def test_select_argument_errors(lib):
    kv, vid = _kv(), h.video_desc(64, 16, 16, 128)

    def call(k=1639, scores=FAKE, idx=FAKE, ksrc=FAKE, vsrc=FAKE, kdst=FAKE, vdst=FAKE, src=kv, dst=kv,
             src_len=16646, ws_bytes=256):
        return lib.hippo_select_gather_kv(scores, k, ksrc, vsrc, C.byref(src) if src else None, src_len,
                                          C.byref(vid), kdst, vdst, C.byref(dst) if dst else None, idx, FAKE,
                                          ws_bytes, None)
    assert call(scores=None) == h.ERR_NULL_ARG
    assert call(idx=None) == h.ERR_NULL_ARG
    assert call(vdst=None) == h.ERR_NULL_ARG                    # K without V
    assert call(src=None) == h.ERR_NULL_ARG
    assert call(dst=None) == h.ERR_NULL_ARG
    assert call(k=0) == h.ERR_BAD_SHAPE
    assert call(k=16385) == h.ERR_BAD_SHAPE
    assert call(src_len=16000) == h.ERR_BAD_SHAPE
    assert call(dst=_kv(head_dim=64)) == h.ERR_BAD_SHAPE
    assert call(dst=_kv(dtype=h.DTYPE_F32)) == h.ERR_BAD_SHAPE
    assert call(kdst=FAKE + 4) == h.ERR_BAD_ALIGN
    assert call(ws_bytes=16) == h.ERR_WORKSPACE_TOO_SMALL


def test_binding_refuses_missing_library(monkeypatch, tmp_path):
    monkeypatch.setattr(h, "_lib", None)
    monkeypatch.setattr(h, "LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(RuntimeError, match="no fallback"):
        h.load()


def test_spec_verify_argument_errors(lib):
    V, g = 151936, 5
    need = lib.hippo_spec_verify_workspace_bytes(1, g, V, h.DTYPE_BF16)
    assert need > 0 and need % 256 == 0
    assert lib.hippo_spec_verify_workspace_bytes(1, g, V, 5) == 0
    assert lib.hippo_spec_verify_workspace_bytes(1, 65, V, h.DTYPE_F32) == 0
    assert lib.hippo_spec_verify_workspace_bytes(1, g, (1 << 20) + 1, h.DTYPE_F32) == 0

    def call(p=FAKE, q=FAKE, dtype=h.DTYPE_BF16, ps=V, qs=V, tok=FAKE, ua=FAKE, us=FAKE, B=1, gamma=g, vocab=V,
             T=1.0, nacc=FAKE, nxt=FAKE, ws=FAKE, ws_bytes=need):
        return lib.hippo_spec_verify(p, q, dtype, ps, qs, tok, ua, us, B, gamma, vocab, T, nacc, nxt, None, ws,
                                     ws_bytes, None)
    assert call(p=None) == h.ERR_NULL_ARG
    assert call(q=None) == h.ERR_NULL_ARG                       # sampling needs the draft's logits
    assert call(tok=None) == h.ERR_NULL_ARG
    assert call(us=None) == h.ERR_NULL_ARG
    assert call(nxt=None) == h.ERR_NULL_ARG
    assert call(ws=None) == h.ERR_NULL_ARG
    assert call(dtype=2) == h.ERR_BAD_DTYPE
    assert call(gamma=-1) == h.ERR_BAD_SHAPE
    assert call(gamma=65) == h.ERR_BAD_SHAPE
    assert call(vocab=0) == h.ERR_BAD_SHAPE
    assert call(B=0) == h.ERR_BAD_SHAPE
    assert call(T=-1.0) == h.ERR_BAD_SHAPE
    assert call(T=float("nan")) == h.ERR_BAD_SHAPE
    assert call(ps=V - 8) == h.ERR_BAD_SHAPE                    # rows overlap
    assert call(ps=V + 4) == h.ERR_BAD_ALIGN                    # bf16 rows must stay 16-byte aligned
    assert call(q=FAKE + 2) == h.ERR_BAD_ALIGN
    assert call(ws=FAKE + 64) == h.ERR_BAD_ALIGN
    assert call(ws_bytes=need - 1) == h.ERR_WORKSPACE_TOO_SMALL


def test_attention_append_argument_errors(lib):
    kv = _kv()
    for fn in (lib.hippo_verify_attention_append, lib.hippo_draft_attention_append):
        def call(q=FAKE, kn=FAKE, vn=FAKE, k=FAKE, v=FAKE, out=FAKE, ws=FAKE, ws_bytes=1 << 30, q_len=6, ctx=16640):
            return fn(q, q_len, kn, vn, k, v, C.byref(kv), ctx, 0.0, 0, out, None, ws, ws_bytes, None)
        assert call(kn=None) == h.ERR_NULL_ARG
        assert call(vn=None) == h.ERR_NULL_ARG
        assert call(k=None) == h.ERR_NULL_ARG
        assert call(kn=FAKE + 4) == h.ERR_BAD_ALIGN
        assert call(q_len=0) == h.ERR_BAD_SHAPE
        assert call(ws_bytes=64) == h.ERR_WORKSPACE_TOO_SMALL


def test_attention_fp8kv_argument_errors(lib):
    fp8 = dict(dtype=h.DTYPE_FP8_E4M3)
    for fn in (lib.hippo_verify_attention_fp8kv, lib.hippo_draft_attention_fp8kv):
        def call(kv=None, q=FAKE, k=FAKE, v=FAKE, ks=FAKE, vs=FAKE, out=FAKE, ws=FAKE, ws_bytes=1 << 30, q_len=6,
                 ctx=16640):
            kv = kv or _kv(**fp8)
            return fn(q, q_len, k, v, ks, vs, C.byref(kv), ctx, 0.0, 0, out, None, ws, ws_bytes, None)
        assert call(ks=None) == h.ERR_NULL_ARG
        assert call(vs=None) == h.ERR_NULL_ARG
        assert call(k=None) == h.ERR_NULL_ARG
        assert call(_kv(dtype=h.DTYPE_F32)) == h.ERR_BAD_DTYPE              # the descriptor names the cache type
        assert call(_kv(dtype=h.DTYPE_BF16)) == h.ERR_BAD_DTYPE
        assert call(_kv(stride_n=128 + 8, **fp8)) == h.ERR_BAD_ALIGN        # fine for bf16, not for bytes
        assert call(k=FAKE + 8) == h.ERR_BAD_ALIGN
        assert call(q_len=0) == h.ERR_BAD_SHAPE
        assert call(ws_bytes=64) == h.ERR_WORKSPACE_TOO_SMALL
    # 8-bit caches exist for the fp8 attention calls and the gather only
    kv8, vid = _kv(**fp8), h.video_desc(64, 16, 16, 128)
    assert _verify(lib, kv8) == h.ERR_BAD_DTYPE
    assert _verify(lib, kv8, fn="hippo_draft_attention") == h.ERR_BAD_DTYPE
    assert lib.hippo_verify_attention_append(FAKE, 6, FAKE, FAKE, FAKE, FAKE, C.byref(kv8), 16640, 0.0, 0, FAKE, None,
                                             FAKE, 1 << 30, None) == h.ERR_BAD_DTYPE
    assert h.workspace_bytes(h.CALL_SCORE_TOKENS, kv8, vid, 128, 16646) == 0
    need = h.workspace_bytes(h.CALL_VERIFY_ATTENTION, kv8, None, 6, 16646)
    assert need > 0 and need == h.workspace_bytes(h.CALL_VERIFY_ATTENTION, _kv(), None, 6, 16646)
    assert h.workspace_bytes(h.CALL_SELECT_GATHER_KV, kv8, vid, 0, 16646, 1639) == 256
    # gather of an 8-bit cache: descriptors must agree, rows must stay 16-byte aligned
    sel = lambda src, dst: lib.hippo_select_gather_kv(FAKE, 1639, FAKE, FAKE, C.byref(src), 16646, C.byref(vid), FAKE,
                                                       FAKE, C.byref(dst), FAKE, FAKE, 256, None)
    assert sel(kv8, _kv()) == h.ERR_BAD_SHAPE                                 # 8-bit source, bf16 destination
    assert sel(kv8, _kv(stride_n=128 + 8, **fp8)) == h.ERR_BAD_ALIGN


def test_quantize_argument_errors(lib):
    src, dst = _kv(), _kv(dtype=h.DTYPE_FP8_E4M3)
    need = lib.hippo_quantize_kv_workspace_bytes(C.byref(src), 16646)
    assert need > 0 and need % 256 == 0
    assert lib.hippo_quantize_kv_workspace_bytes(C.byref(src), 0) == 0
    assert lib.hippo_quantize_kv_workspace_bytes(C.byref(dst), 100) == 0        # the source is bf16 or fp32

    def call(k=FAKE, v=FAKE, s=src, n=16646, kc=FAKE, vc=FAKE, d=dst, ks=FAKE, vs=FAKE, ws=FAKE, ws_bytes=need):
        return lib.hippo_quantize_kv_e4m3(k, v, C.byref(s), n, kc, vc, C.byref(d), ks, vs, ws, ws_bytes, None)
    assert call(k=None) == h.ERR_NULL_ARG
    assert call(vc=None) == h.ERR_NULL_ARG
    assert call(ks=None) == h.ERR_NULL_ARG
    assert call(ws=None) == h.ERR_NULL_ARG
    assert call(s=dst) == h.ERR_BAD_DTYPE
    assert call(d=src) == h.ERR_BAD_DTYPE
    assert call(d=_kv(dtype=h.DTYPE_FP8_E4M3, n_kv_heads=2, n_q_heads=28)) == h.ERR_BAD_SHAPE
    assert call(n=0) == h.ERR_BAD_SHAPE
    assert call(kc=FAKE + 4) == h.ERR_BAD_ALIGN
    assert call(d=_kv(dtype=h.DTYPE_FP8_E4M3, stride_n=128 + 8)) == h.ERR_BAD_ALIGN
    assert call(ws_bytes=need - 1) == h.ERR_WORKSPACE_TOO_SMALL
    # (KV head, K or V) pairs are a y dimension of the launch: more than 32767 KV heads cannot be launched
    many = dict(n_kv_heads=32768, n_q_heads=32768)
    assert call(s=_kv(**many), d=_kv(dtype=h.DTYPE_FP8_E4M3, **many), ws_bytes=1 << 40) == h.ERR_BAD_SHAPE


def test_attention_paged_argument_errors(lib):
    def desc(**kw):
        d = dict(batch=1, n_q_heads=28, n_kv_heads=4, head_dim=128, dtype=h.DTYPE_BF16, page_size=16, max_pages=1100,
                 n_pool_pages=2000, stride_page=16 * 4 * 128, stride_n=4 * 128, stride_h=128)
        d.update(kw)
        return h.PagedKvDesc(**d)

    def call(pd=None, q=FAKE, k=FAKE, v=FAKE, table=FAKE, ctx=16640, q_len=6, splits=0, ws_bytes=1 << 30,
             fn=lib.hippo_verify_attention_paged):
        pd = pd or desc()
        return fn(q, q_len, k, v, table, C.byref(pd), ctx, 0.0, splits, FAKE, None, FAKE, ws_bytes, None)
    for fn in (lib.hippo_verify_attention_paged, lib.hippo_draft_attention_paged):
        assert call(table=None, fn=fn) == h.ERR_NULL_ARG
        assert call(k=None, fn=fn) == h.ERR_NULL_ARG
        assert call(desc(page_size=24), fn=fn) == h.ERR_BAD_SHAPE          # not a power of two
        assert call(desc(page_size=8), fn=fn) == h.ERR_BAD_SHAPE
        assert call(desc(max_pages=100), fn=fn) == h.ERR_BAD_SHAPE         # table too narrow for the cache
        assert call(desc(stride_page=1000), fn=fn) == h.ERR_BAD_SHAPE      # pages overlap
        assert call(desc(stride_page=16 * 4 * 128 + 4), fn=fn) == h.ERR_BAD_ALIGN
        assert call(desc(dtype=9), fn=fn) == h.ERR_BAD_DTYPE
        assert call(table=FAKE + 2, fn=fn) == h.ERR_BAD_ALIGN
        assert call(ws_bytes=64, fn=fn) == h.ERR_WORKSPACE_TOO_SMALL
    # one slice over 16.6K tokens of 16-token pages does not fit the page staging area
    assert call(splits=1) == h.ERR_BAD_SHAPE
    assert lib.hippo_verify_attention_paged(FAKE, 6, FAKE, FAKE, FAKE, None, 10, 0.0, 0, FAKE, None, FAKE, 1 << 20,
                                            None) == h.ERR_NULL_ARG


def test_score_layers_argument_errors(lib):
    kv, vid = _kv(), h.video_desc(64, 16, 16, 128)
    need1 = lib.hippo_score_layers_workspace_bytes(C.byref(kv), C.byref(vid), 128, 1)
    need4 = lib.hippo_score_layers_workspace_bytes(C.byref(kv), C.byref(vid), 128, 4)
    assert need1 == h.workspace_bytes(h.CALL_SCORE_TOKENS, kv, vid, 128, 16646) and need4 > 2 * need1
    assert lib.hippo_score_layers_workspace_bytes(C.byref(kv), C.byref(vid), 128, 65) == 0

    def call(n=4, qs=None, ks=None, emb_layer=0, ws_bytes=need4, scores=FAKE):
        qa = (C.c_void_p * 4)(*(qs or [FAKE] * 4))
        ka = (C.c_void_p * 4)(*(ks or [FAKE] * 4))
        return lib.hippo_score_tokens_layers(n, C.cast(qa, C.c_void_p), 128, C.cast(ka, C.c_void_p), emb_layer,
                                             C.byref(kv), 16646, C.byref(vid), None, 0, 0, h.SCORE_ALL, None, scores,
                                             None, FAKE, ws_bytes, None)
    assert call(n=0) == h.ERR_BAD_SHAPE
    assert call(n=65) == h.ERR_BAD_SHAPE
    assert call(emb_layer=4) == h.ERR_BAD_SHAPE
    assert call(qs=[FAKE, None, FAKE, FAKE]) == h.ERR_NULL_ARG
    assert call(ks=[FAKE, FAKE, FAKE + 8, FAKE]) == h.ERR_BAD_ALIGN
    assert call(scores=None) == h.ERR_NULL_ARG
    assert call(ws_bytes=need1) == h.ERR_WORKSPACE_TOO_SMALL
    assert lib.hippo_score_tokens_layers(1, None, 128, None, 0, C.byref(kv), 16646, C.byref(vid), None, 0, 0, 7, None,
                                         FAKE, None, FAKE, need1, None) == h.ERR_NULL_ARG
