"""fp32 scoring in one sweep, whose blocks wait for each other's row sums: no result depends on a wait.

The library's bound on a wave's looks at the sums is taken down from the host, so that blocks stop waiting wherever they would
have to, and two calls share the GPU; every result is compared bit for bit with that of the call by itself."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from parity_util import assert_close, dev, host

pytestmark = pytest.mark.gpu


def score(hippo, q, k, vid, polls, flags=7):
    """hippo_score_tokens_layers with its waits bounded by `polls` looks -> scores and components"""
    lib, n_layers = hippo.load(), len(q)
    fn = lib.hippo_score_tokens_layers_polls
    fn.argtypes, fn.restype = lib.hippo_score_tokens_layers.argtypes + [C.c_int32], C.c_int
    B, L, H, _ = q[0].shape
    kv, n_vis = hippo.kv_desc(k[0], H), vid.n_frames * vid.grid_h * vid.grid_w
    ws = torch.empty(lib.hippo_score_layers_workspace_bytes(C.byref(kv), C.byref(vid), L, n_layers), dtype=torch.uint8,
                     device="cuda")
    out = torch.zeros((4, B, n_vis), device="cuda")
    qs, ks = ((C.c_void_p * n_layers)(*[t.data_ptr() for t in x]) for x in (q, k))
    hippo._check(fn(n_layers, qs, L, ks, 0, C.byref(kv), k[0].shape[2], C.byref(vid), None, 0, 0, flags, None,
                    out[0].data_ptr(), out[1].data_ptr(), ws.data_ptr(), ws.numel(), hippo._stream(None), polls),
                 "hippo_score_tokens_layers_polls")
    return out


def inputs(seed, layers, B, L, H, Hkv, d, n, rows_out=None, shift=0.0):
    """logits of a few units; text rows `rows_out` (a slice) are shifted by `shift` nats"""
    r = np.random.default_rng(seed)
    q = [(0.7 * r.standard_normal((B, L, H, d))).astype(np.float32) for _ in range(layers)]
    k = [r.standard_normal((B, Hkv, n, d)).astype(np.float32) for _ in range(layers)]
    for x, y in zip(q, k):
        x[..., 0] = 0.0
        if rows_out is not None:
            x[:, rows_out, :, 0] = np.sqrt(d)
            y[..., 0] = shift
    return q, k


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows_out, shift", [
    # in the words; in the bins; beyond the range of both, one row or all, upwards or downwards
    (None, 0.0), (slice(9, 10), 40.0), (slice(0, None), -40.0), (slice(20, 21), 110.0), (slice(3, 4), -110.0),
    (slice(0, None), 110.0), (slice(0, None), -110.0),
])
def test_no_result_depends_on_a_wait(hippo, rows_out, shift, d):
    layers, B, L, F, gh, gw = 2, 2, 23, 12, 15, 17
    q, k = inputs(d, layers, B, L, 14, 2, d, F * gh * gw + 3, rows_out, shift)
    vid = hippo.video_desc(F, gh, gw, 2)
    qd, kd = [dev(x, "fp32") for x in q], [dev(x, "fp32") for x in k]
    ref = score(hippo, qd, kd, vid, -1)
    for polls in (0, 1, 5):
        got = score(hippo, qd, kd, vid, polls)
        assert torch.equal(got, ref), "%d looks" % polls
    mass = sum(oracle.s_attn(x, y, 2, F * gh * gw) for x, y in zip(q, k))
    # of a logit of `shift`: each of d additions and two products round by up to 2^-24 of it
    bound = (1e-5 + abs(shift) * (d + 2) * 2.0 ** -24) * np.maximum(np.abs(mass), np.sqrt((mass ** 2).mean()))
    assert (np.abs(host(ref)[1] - mass) <= bound).all(), np.abs((host(ref)[1] - mass) / bound).max()


@pytest.mark.parametrize("F, L, H, Hkv, d", [(16, 32, 14, 2, 64), (160, 40, 4, 1, 64), (144, 20, 28, 4, 128)])
def test_two_calls_share_the_gpu(hippo, F, L, H, Hkv, d):
    # 28, 280 and 252 tiles a run: both calls' blocks fit on the chip, one run of theirs or the other's, or two
    vid, n = hippo.video_desc(F, 14, 16, 1), F * 14 * 16
    data = [inputs(s, 1, 1, L, H, Hkv, d, n + 1) for s in (1, 2)]
    data = [(dev(q[0], "fp32"), dev(k[0], "fp32")) for q, k in data]
    alone = [hippo.hippo_score_tokens(q, k, vid, want_components=True) for q, k in data]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in data]
    together = [[], []]
    for _ in range(4):
        for at, (s, (q, k)) in enumerate(zip(streams, data)):
            together[at].append(hippo.hippo_score_tokens(q, k, vid, want_components=True, stream=s))
    torch.cuda.synchronize()
    for ref, got in zip(alone, together):
        for x in got:
            assert torch.equal(x[0], ref[0]) and torch.equal(x[1], ref[1])
    assert_close(host(alone[0][1])[0], oracle.s_attn(host(data[0][0]), host(data[0][1]), 1, n), "fp32", "s_attn")
