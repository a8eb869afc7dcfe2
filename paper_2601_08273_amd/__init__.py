"""Python binding of the HIPPO hot-path library for MI355X (``libhippo.so``, C ABI in include/hippo.h).

Argument marshalling only: every step runs in the HIP kernels.  torch supplies device memory and
the current stream; nothing here computes.  The calls on tensors are marshalled in C++ (csrc/binding.cpp), the host-side
ones and the C ABI itself through ctypes.  If either shared library is missing the calls raise -- there is no fallback
path.
"""
from __future__ import annotations

import ctypes as C
import os
from typing import Optional, Tuple

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libhippo.so")

DTYPE_F32, DTYPE_BF16, DTYPE_FP8_E4M3 = 0, 1, 2
CALL_SCORE_TOKENS, CALL_SELECT_GATHER_KV, CALL_DRAFT_ATTENTION, CALL_VERIFY_ATTENTION = 0, 1, 2, 3
SCORE_ATTN, SCORE_TEMP, SCORE_SPA, SCORE_ALL, SCORE_ACCUMULATE_ONLY = 1, 2, 4, 7, 8
(OK, ERR_NULL_ARG, ERR_BAD_SHAPE, ERR_BAD_DTYPE, ERR_BAD_ALIGN, ERR_WORKSPACE_TOO_SMALL, ERR_HIP,
 ERR_STATIC_SCRATCH_LIMIT) = range(8)

EXPORTS = ("hippo_status_string", "hippo_workspace_bytes", "hippo_score_tokens",
           "hippo_score_layers_workspace_bytes", "hippo_score_tokens_layers",
           "hippo_select_gather_kv", "hippo_verify_attention", "hippo_draft_attention",
           "hippo_static_scratch_bytes", "hippo_static_scratch_init", "hippo_verify_attention_static",
           "hippo_verify_attention_append", "hippo_draft_attention_append",
           "hippo_verify_attention_paged", "hippo_draft_attention_paged",
           "hippo_verify_attention_fp8kv", "hippo_draft_attention_fp8kv",
           "hippo_quantize_kv_workspace_bytes", "hippo_quantize_kv_e4m3",
           "hippo_spec_verify_workspace_bytes", "hippo_spec_verify", "hippo_vpsd_prefill_buffer",
           "hippo_vpsd_init", "hippo_vpsd_plan", "hippo_vpsd_commit", "hippo_vpsd_simulate")
VPSD_CONSERVATIVE, VPSD_OPTIMISTIC = 0, 1
POLICY_AUTOREGRESSIVE, POLICY_SERIAL_SD, POLICY_VPSD = 0, 1, 2


class VpsdState(C.Structure):
    _fields_ = [("gamma", C.c_int32), ("mode", C.c_int32), ("n_pending", C.c_int32), ("reserved", C.c_int32),
                ("n_emitted", C.c_int64), ("n_rounds", C.c_int64), ("n_target_calls", C.c_int64),
                ("n_draft_tokens", C.c_int64), ("n_draft_wasted", C.c_int64), ("n_mode_switches", C.c_int64)]


class VpsdRound(C.Structure):
    _fields_ = [("mode", C.c_int32), ("draft_serial", C.c_int32), ("verify_len", C.c_int32),
                ("draft_parallel", C.c_int32)]


class VpsdResult(C.Structure):
    _fields_ = [("time", C.c_double), ("speedup", C.c_double), ("n_emitted", C.c_int64), ("n_rounds", C.c_int64),
                ("n_target_calls", C.c_int64), ("n_draft_tokens", C.c_int64), ("n_draft_wasted", C.c_int64),
                ("n_mode_switches", C.c_int64), ("n_flags_used", C.c_int64)]


class PagedKvDesc(C.Structure):
    _fields_ = [("batch", C.c_int32), ("n_q_heads", C.c_int32), ("n_kv_heads", C.c_int32),
                ("head_dim", C.c_int32), ("dtype", C.c_int32), ("page_size", C.c_int32),
                ("max_pages", C.c_int32), ("n_pool_pages", C.c_int32),
                ("stride_page", C.c_int64), ("stride_n", C.c_int64), ("stride_h", C.c_int64)]


class KvDesc(C.Structure):
    _fields_ = [("batch", C.c_int32), ("n_q_heads", C.c_int32), ("n_kv_heads", C.c_int32),
                ("head_dim", C.c_int32), ("dtype", C.c_int32),
                ("stride_b", C.c_int64), ("stride_h", C.c_int64), ("stride_n", C.c_int64)]


class VideoDesc(C.Structure):
    _fields_ = [("n_frames", C.c_int32), ("grid_h", C.c_int32), ("grid_w", C.c_int32),
                ("vis_offset", C.c_int32), ("crop_h", C.c_int32), ("crop_w", C.c_int32)]


class HippoError(RuntimeError):
    def __init__(self, status: int, what: str):
        super().__init__("%s failed: status %d (%s)" % (what, status, status_string(status)))
        self.status = status


_lib = None
_native = None          # csrc/binding.cpp, bound to the library: see _bound


def load():
    """dlopen libhippo.so and declare the signatures.  Raises if the library has not been built."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError("libhippo.so is not built: run `python -m paper_2601_08273_amd.build` "
                           "(there is no fallback implementation)")
    lib = C.CDLL(LIB_PATH)
    vp, i32, i64, u32, f32, sz = C.c_void_p, C.c_int32, C.c_int64, C.c_uint32, C.c_float, C.c_size_t
    kvp, vdp = C.POINTER(KvDesc), C.POINTER(VideoDesc)
    lib.hippo_status_string.argtypes = [C.c_int]
    lib.hippo_status_string.restype = C.c_char_p
    lib.hippo_workspace_bytes.argtypes = [i32, kvp, vdp, i32, i32, i32, i32]
    lib.hippo_workspace_bytes.restype = sz
    lib.hippo_score_tokens.argtypes = [vp, i32, vp, kvp, i32, vdp, vp, i32, i64, u32, vp, vp, vp, vp, sz, vp]
    lib.hippo_score_tokens.restype = C.c_int
    lib.hippo_score_layers_workspace_bytes.argtypes = [kvp, vdp, i32, i32]
    lib.hippo_score_layers_workspace_bytes.restype = C.c_size_t
    lib.hippo_score_tokens_layers.argtypes = [i32, vp, i32, vp, i32, kvp, i32, vdp, vp, i32, i64, u32, vp, vp, vp, vp,
                                              sz, vp]
    lib.hippo_score_tokens_layers.restype = C.c_int
    lib.hippo_select_gather_kv.argtypes = [vp, i32, vp, vp, kvp, i32, vdp, vp, vp, kvp, vp, vp, sz, vp]
    lib.hippo_select_gather_kv.restype = C.c_int
    for fn in (lib.hippo_verify_attention, lib.hippo_draft_attention):
        fn.argtypes = [vp, i32, vp, vp, kvp, i32, f32, i32, vp, vp, vp, sz, vp]
        fn.restype = C.c_int
    lib.hippo_static_scratch_bytes.argtypes = []
    lib.hippo_static_scratch_bytes.restype = sz
    lib.hippo_static_scratch_init.argtypes = []
    lib.hippo_static_scratch_init.restype = C.c_int
    lib.hippo_verify_attention_static.argtypes = [vp, i32, vp, vp, kvp, i32, f32, i32, vp, vp, vp]
    lib.hippo_verify_attention_static.restype = C.c_int
    for fn in (lib.hippo_verify_attention_paged, lib.hippo_draft_attention_paged):
        fn.argtypes = [vp, i32, vp, vp, vp, C.POINTER(PagedKvDesc), i32, f32, i32, vp, vp, vp, sz, vp]
        fn.restype = C.c_int
    for fn in (lib.hippo_verify_attention_append, lib.hippo_draft_attention_append,
               lib.hippo_verify_attention_fp8kv, lib.hippo_draft_attention_fp8kv):
        fn.argtypes = [vp, i32, vp, vp, vp, vp, kvp, i32, f32, i32, vp, vp, vp, sz, vp]
        fn.restype = C.c_int
    lib.hippo_quantize_kv_workspace_bytes.argtypes = [kvp, i32]
    lib.hippo_quantize_kv_workspace_bytes.restype = C.c_size_t
    lib.hippo_quantize_kv_e4m3.argtypes = [vp, vp, kvp, i32, vp, vp, kvp, vp, vp, vp, sz, vp]
    lib.hippo_quantize_kv_e4m3.restype = C.c_int
    f64 = C.c_double
    lib.hippo_vpsd_prefill_buffer.argtypes = [f64, f64, f64]
    lib.hippo_vpsd_prefill_buffer.restype = C.c_int32
    lib.hippo_vpsd_init.argtypes = [C.POINTER(VpsdState), i32, i32]
    lib.hippo_vpsd_plan.argtypes = [C.POINTER(VpsdState), C.POINTER(VpsdRound)]
    lib.hippo_vpsd_commit.argtypes = [C.POINTER(VpsdState), C.POINTER(VpsdRound), i32, i32]
    lib.hippo_vpsd_simulate.argtypes = [i32, i32, f64, f64, i32, vp, i64, i64, C.POINTER(VpsdResult)]
    for fn in (lib.hippo_vpsd_init, lib.hippo_vpsd_plan, lib.hippo_vpsd_commit, lib.hippo_vpsd_simulate):
        fn.restype = C.c_int
    lib.hippo_spec_verify_workspace_bytes.argtypes = [i32, i32, i32, i32]
    lib.hippo_spec_verify_workspace_bytes.restype = C.c_size_t
    lib.hippo_spec_verify.argtypes = [vp, vp, i32, i64, i64, vp, vp, vp, i32, i32, i32, f32, vp, vp, vp, vp, sz, vp]
    lib.hippo_spec_verify.restype = C.c_int
    _lib = lib
    return lib


def _bound():
    """The native marshalling of the calls on tensors, bound to the loaded library."""
    global _native
    load()
    if _native is None:
        _torch()
        try:
            from . import _binding as native
        except ImportError as e:
            raise RuntimeError("_binding.so cannot be imported (%s): it is built for one torch and one Python by `python -m "
                               "paper_2601_08273_amd.build` (there is no fallback implementation)" % e) from e
        native.bind(LIB_PATH, VideoDesc, HippoError)
        _native = native
    return _native


def status_string(status: int) -> str:
    return load().hippo_status_string(int(status)).decode()


# ---------------------------------------------------------------------------------------------
# torch plumbing (device memory + streams)
# ---------------------------------------------------------------------------------------------

def _torch():
    import torch
    return torch


_dtype_codes = {}


def _dtype_code(t) -> int:
    code = _dtype_codes.get(t.dtype)
    if code is None:
        torch = _torch()
        _dtype_codes.update({torch.float32: DTYPE_F32, torch.bfloat16: DTYPE_BF16,
                             torch.uint8: DTYPE_FP8_E4M3, torch.float8_e4m3fn: DTYPE_FP8_E4M3})   # E4M3 cache codes
        code = _dtype_codes.get(t.dtype)
        if code is None:
            raise TypeError("unsupported dtype %s (fp32, bf16, or uint8 / float8_e4m3fn cache codes)" % t.dtype)
    return code


def _ptr(t) -> Optional[int]:
    return None if t is None else t.data_ptr()


def _stream(stream) -> Optional[int]:
    if stream is not None:
        return stream.cuda_stream or None
    torch = _torch()
    if not torch.cuda.is_initialized():
        return torch.cuda.current_stream().cuda_stream or None
    # the current stream's handle without a Stream object around it (0.3 against 2.8 us)
    return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice()) or None


def kv_desc(cache, n_q_heads: int) -> KvDesc:
    """Descriptor of a [B, H_kv, N, d] cache tensor (any strides with unit stride on d)."""
    strides = cache.stride()
    assert len(strides) == 4 and strides[3] == 1
    shape = cache.shape
    return KvDesc(shape[0], n_q_heads, shape[1], shape[3], _dtype_code(cache), *strides[:3])


def video_desc(n_frames, grid_h, grid_w, vis_offset, crop_h=5, crop_w=5) -> VideoDesc:
    return VideoDesc(n_frames, grid_h, grid_w, vis_offset, crop_h, crop_w)


def workspace_bytes(call: int, kv: KvDesc, vid: Optional[VideoDesc], n_rows: int, seq_len: int,
                    k: int = 0, num_splits: int = 0) -> int:
    return int(load().hippo_workspace_bytes(call, C.byref(kv), C.byref(vid) if vid is not None else None,
                                            n_rows, seq_len, k, num_splits))


def _on(stream):
    """Context in which the wrapper allocates what the caller did not pass (workspace, outputs): the
    stream the kernels are enqueued on.  torch's caching allocator ties a block to the stream that was
    current when it was allocated and may hand it out again, on that stream, as soon as the tensor is
    dropped; allocated under another stream than the kernels', a workspace could be recycled while they
    still use it."""
    return _torch().cuda.stream(stream)


def _call(stream, entry, *args):
    """entry(*args) on `stream` (None: the current one), where it also allocates (see _on)."""
    if stream is None:
        return entry(*args)
    with _on(stream):
        return entry(*args)


def _check(status: int, what: str):
    if status != OK:
        raise HippoError(status, what)


# ---------------------------------------------------------------------------------------------
# the four entry points
# ---------------------------------------------------------------------------------------------

def hippo_score_tokens(q_txt, k_cache, vid: VideoDesc, emb=None, flags: int = SCORE_ALL,
                       attn_mass_inout=None, want_components: bool = False, scores_out=None, workspace=None,
                       stream=None):
    """q_txt [B,L,H,d], k_cache [B,Hkv,N,d] -> scores [B,N_v] fp32 (and components [3,B,N_v])."""
    return _call(stream, (_native or _bound()).score_tokens, q_txt, k_cache, vid, emb, flags, attn_mass_inout,
                 want_components, scores_out, workspace)


def hippo_score_tokens_layers(q_txt_layers, k_cache_layers, vid: VideoDesc, emb_layer: int = 0, emb=None,
                              flags: int = SCORE_ALL, attn_mass_inout=None, want_components: bool = False,
                              scores_out=None, workspace=None, stream=None):
    """Eq. 2 with its sum over layers inside one call: lists of per-layer q_txt [B,L,H,d] and
    k_cache [B,Hkv,N,d] (same shapes and strides) -> scores [B,N_v] fp32 (and components)."""
    return _call(stream, (_native or _bound()).score_tokens_layers, q_txt_layers, k_cache_layers, vid, emb_layer, emb,
                 flags, attn_mass_inout, want_components, scores_out, workspace)


def hippo_select_gather_kv(scores, k: int, k_src, v_src, vid: VideoDesc, n_q_heads: Optional[int] = None,
                           gather: bool = True, idx_out=None, k_dst=None, v_dst=None, workspace=None, stream=None):
    """scores [B,N_v] fp32 -> (idx [B,k] int32, k_dst, v_dst [B,Hkv,N-N_v+k,d]).
    idx_out / k_dst / v_dst: optional preallocated outputs (k_dst, v_dst may be strided views)."""
    return _call(stream, (_native or _bound()).select_gather, scores, k, k_src, v_src, vid, n_q_heads, gather, idx_out,
                 k_dst, v_dst, workspace)


def hippo_verify_attention(q, k_cache, v_cache, ctx_len: int, softmax_scale: float = 0.0, num_splits: int = 0,
                           want_lse: bool = False, out=None, workspace=None, stream=None, k_new=None, v_new=None):
    """q [B,q_len,H,d]; caches hold ctx_len+q_len rows; row i attends to [0, ctx_len+i].
    With k_new / v_new [B,q_len,Hkv,d] the new rows are taken from there and appended to the caches
    by the same launch (hippo_verify_attention_append)."""
    return _call(stream, (_native or _bound()).attention, False, q, k_cache, v_cache, ctx_len, softmax_scale,
                 num_splits, want_lse, out, workspace, k_new, v_new)


def hippo_draft_attention(q, k_cache, v_cache, ctx_len: int, softmax_scale: float = 0.0, num_splits: int = 0,
                          want_lse: bool = False, out=None, workspace=None, stream=None, k_new=None, v_new=None):
    return _call(stream, (_native or _bound()).attention, True, q, k_cache, v_cache, ctx_len, softmax_scale, num_splits,
                 want_lse, out, workspace, k_new, v_new)


def hippo_verify_attention_static(q, k_cache, v_cache, ctx_len: int, softmax_scale: float = 0.0, num_splits: int = 0,
                                  lse_out=None, out=None, stream=None):
    """hippo_verify_attention without a workspace: the split partials live in the library's own static
    device array (calls on one GPU must not overlap).  Pass `out` (and `lse_out`) to keep the whole call
    free of allocations."""
    torch = _torch()
    lib = load()
    if stream is not None:
        with _on(stream):
            return hippo_verify_attention_static(q, k_cache, v_cache, ctx_len, softmax_scale, num_splits, lse_out, out)
    assert q.is_contiguous() and q.dim() == 4
    B, q_len, H, d = q.shape
    kv = kv_desc(k_cache, H)
    assert v_cache.stride() == k_cache.stride() and v_cache.shape == k_cache.shape
    if out is None:
        out = torch.empty_like(q)
    st = lib.hippo_verify_attention_static(_ptr(q), q_len, _ptr(k_cache), _ptr(v_cache), C.byref(kv), ctx_len,
                                           float(softmax_scale or 0.0), num_splits, _ptr(out), _ptr(lse_out),
                                           _stream(None))
    _check(st, "hippo_verify_attention_static")
    return out


def hippo_verify_attention_fp8kv(q, k_codes, v_codes, k_scale, v_scale, ctx_len: int, softmax_scale: float = 0.0,
                                 num_splits: int = 0, want_lse: bool = False, out=None, workspace=None,
                                 stream=None):
    """q [B,q_len,H,d] bf16; k_codes / v_codes [B,Hkv,N,d] E4M3 bytes; k_scale / v_scale [B,Hkv] fp32."""
    return _call(stream, (_native or _bound()).attention_fp8kv, False, q, k_codes, v_codes, k_scale, v_scale, ctx_len,
                 softmax_scale, num_splits, want_lse, out, workspace)


def hippo_draft_attention_fp8kv(q, k_codes, v_codes, k_scale, v_scale, ctx_len: int, softmax_scale: float = 0.0,
                                num_splits: int = 0, want_lse: bool = False, out=None, workspace=None,
                                stream=None):
    return _call(stream, (_native or _bound()).attention_fp8kv, True, q, k_codes, v_codes, k_scale, v_scale, ctx_len,
                 softmax_scale, num_splits, want_lse, out, workspace)


def hippo_quantize_kv_e4m3(k_src, v_src, n_rows: Optional[int] = None, k_codes=None, v_codes=None, workspace=None,
                           stream=None):
    """k_src / v_src [B,Hkv,N,d] bf16 or fp32 -> (k_codes, v_codes uint8 [B,Hkv,n_rows,d], k_scale, v_scale
    fp32 [B,Hkv]): the cache format of the *_fp8kv attention calls."""
    return _call(stream, (_native or _bound()).quantize, k_src, v_src, n_rows, k_codes, v_codes, workspace)


def hippo_verify_attention_paged(q, k_pool, v_pool, block_table, ctx_len: int, softmax_scale: float = 0.0,
                                 num_splits: int = 0, want_lse: bool = False, out=None, workspace=None, stream=None):
    """Pools [n_pages, page_size, Hkv, d]; block_table [B, max_pages] int32 on the device."""
    return _call(stream, (_native or _bound()).attention_paged, False, q, k_pool, v_pool, block_table, ctx_len,
                 softmax_scale, num_splits, want_lse, out, workspace)


def hippo_draft_attention_paged(q, k_pool, v_pool, block_table, ctx_len: int, softmax_scale: float = 0.0,
                                num_splits: int = 0, want_lse: bool = False, out=None, workspace=None, stream=None):
    return _call(stream, (_native or _bound()).attention_paged, True, q, k_pool, v_pool, block_table, ctx_len,
                 softmax_scale, num_splits, want_lse, out, workspace)


def hippo_spec_verify(p_logits, q_logits, draft_tokens, u_accept, u_sample, temperature: float,
                      want_alpha: bool = False, n_accept_out=None, next_token_out=None, workspace=None,
                      stream=None):
    """p_logits [B,gamma+1,V] (rows may be padded: stride(1) >= V), q_logits [B,gamma,V] or None
    (greedy), draft_tokens [B,gamma] int32, u_accept [B,gamma] fp32, u_sample [B] fp32 ->
    (n_accept [B] int32, next_token [B] int32[, alpha [B,gamma] fp32])."""
    return _call(stream, (_native or _bound()).spec_verify, p_logits, q_logits, draft_tokens, u_accept, u_sample,
                 temperature, want_alpha, n_accept_out, next_token_out, workspace)


# ---------------------------------------------------------------------------------------------
# host-side control of video parallel speculative decoding (no GPU involved)
# ---------------------------------------------------------------------------------------------

def vpsd_prefill_buffer(t_prefill_target: float, t_prefill_draft: float, t_draft_token: float) -> int:
    return int(load().hippo_vpsd_prefill_buffer(t_prefill_target, t_prefill_draft, t_draft_token))


def vpsd_init(gamma: int, n_prefill_buffer: int = 0) -> VpsdState:
    s = VpsdState()
    _check(load().hippo_vpsd_init(C.byref(s), gamma, n_prefill_buffer), "hippo_vpsd_init")
    return s


def vpsd_plan(state: VpsdState) -> VpsdRound:
    r = VpsdRound()
    _check(load().hippo_vpsd_plan(C.byref(state), C.byref(r)), "hippo_vpsd_plan")
    return r


def vpsd_commit(state: VpsdState, rnd: VpsdRound, n_accept: int, n_drafted_parallel: Optional[int] = None) -> None:
    n = rnd.draft_parallel if n_drafted_parallel is None else n_drafted_parallel
    _check(load().hippo_vpsd_commit(C.byref(state), C.byref(rnd), n_accept, n), "hippo_vpsd_commit")


def vpsd_simulate(policy: int, gamma: int, t_draft: float, t_target: float, accept, n_tokens: int,
                  n_prefill_buffer: int = 0) -> VpsdResult:
    flags = bytes(bytearray(1 if a else 0 for a in accept))
    res = VpsdResult()
    buf = C.create_string_buffer(flags, len(flags)) if flags else None
    _check(load().hippo_vpsd_simulate(policy, gamma, t_draft, t_target, n_prefill_buffer,
                                      C.cast(buf, C.c_void_p) if buf is not None else None, len(flags), n_tokens,
                                      C.byref(res)), "hippo_vpsd_simulate")
    return res
