"""The binding's own checks, which need no GPU: they come before anything is allocated or enqueued."""
import sys

import numpy as np
import pytest
import torch

import paper_2601_08273_amd as h


def cache(B=1, Hkv=2, N=40, d=64, dtype=torch.bfloat16):
    return torch.zeros((B, Hkv, N, d), dtype=dtype)


def queries(B=1, q_len=2, H=4, d=64, dtype=torch.bfloat16):
    return torch.zeros((B, q_len, H, d), dtype=dtype)


VID = h.video_desc(2, 4, 4, 2)


@pytest.mark.parametrize("call, error", [
    (lambda: h.hippo_verify_attention(queries().transpose(1, 2), cache(), cache(), 38), AssertionError),
    (lambda: h.hippo_verify_attention(queries()[0], cache(), cache(), 38), AssertionError),
    (lambda: h.hippo_verify_attention(queries(), cache(), cache(N=41), 38), AssertionError),
    (lambda: h.hippo_verify_attention(queries(), cache().transpose(2, 3), cache().transpose(2, 3), 38), AssertionError),
    (lambda: h.hippo_verify_attention(queries(), cache(dtype=torch.float16), cache(dtype=torch.float16), 38), TypeError),
    (lambda: h.hippo_verify_attention(queries(), None, cache(), 38), TypeError),
    (lambda: h.hippo_verify_attention(queries(), cache(), cache(), 38.0), TypeError),
    (lambda: h.hippo_draft_attention(queries(), cache(), cache(), 38, out=queries(), workspace=queries(),
                                     k_new=queries(H=2)[0], v_new=queries(H=2)), AssertionError),
    (lambda: h.hippo_verify_attention_fp8kv(queries(dtype=torch.float32), cache(dtype=torch.uint8), cache(dtype=torch.uint8),
                                            torch.ones(1, 2), torch.ones(1, 2), 38), AssertionError),
    (lambda: h.hippo_verify_attention_fp8kv(queries(), cache(dtype=torch.uint8), cache(dtype=torch.uint8),
                                            torch.ones(1, 3), torch.ones(1, 3), 38), AssertionError),
    (lambda: h.hippo_verify_attention_paged(queries(), cache(), cache(), torch.zeros((1, 3)), 38), AssertionError),
    (lambda: h.hippo_verify_attention_paged(queries(), cache(), cache(), torch.zeros((1, 3, 2), dtype=torch.int32), 38), AssertionError),
    (lambda: h.hippo_score_tokens(queries(), cache(), (2, 4, 4, 2, 5, 5)), TypeError),
    (lambda: h.hippo_score_tokens(queries(), cache()[0], VID), AssertionError),
    (lambda: h.hippo_score_tokens(queries(), cache(), VID, scores_out=queries(), workspace=queries(),
                                  emb=torch.zeros((1, 32, 64))[..., ::2]), AssertionError),
    (lambda: h.hippo_score_tokens_layers([queries()], [], VID), AssertionError),
    (lambda: h.hippo_score_tokens_layers([queries(), queries(q_len=3)], [cache(), cache()], VID), AssertionError),
    (lambda: h.hippo_score_tokens_layers(iter([queries()]), iter([cache()]), VID), TypeError),
    (lambda: h.hippo_select_gather_kv(torch.zeros((1, 32), dtype=torch.float64), 4, cache(), cache(), VID), AssertionError),
    (lambda: h.hippo_select_gather_kv(torch.zeros((1, 32)), 4, cache(), cache(), VID, k_dst=cache(N=13), v_dst=cache(N=13)),
     AssertionError),
    (lambda: h.hippo_select_gather_kv(torch.zeros((1, 32)), 4, cache(), cache(), VID, k_dst=cache(N=12)), AssertionError),
    (lambda: h.hippo_quantize_kv_e4m3(cache(), cache(), n_rows=41), AssertionError),
    (lambda: h.hippo_quantize_kv_e4m3(cache(), cache(), k_codes=cache(N=39, dtype=torch.uint8),
                                      v_codes=cache(N=39, dtype=torch.uint8)), AssertionError),
    (lambda: h.hippo_spec_verify(torch.zeros((2, 4, 8)), torch.zeros((2, 3, 9)), None, None, None, 1.0), AssertionError),
    (lambda: h.hippo_spec_verify(torch.zeros((2, 4, 8)), None, torch.zeros((2, 3)), None, None, 0.0), AssertionError),
    (lambda: h.hippo_spec_verify(torch.zeros((4, 8)), None, None, None, None, 0.0), AssertionError),
])
def test_what_is_refused_before_the_library(call, error):
    with pytest.raises(error):
        call()


def test_statuses_of_the_library_come_back_as_errors():
    # 16 tokens of visual keys are missing: refused by the library, before a launch
    with pytest.raises((h.HippoError, RuntimeError)) as e:
        h.hippo_score_tokens(queries(), cache(N=20), VID, scores_out=torch.zeros((1, 32)),
                             workspace=torch.zeros(1 << 16, dtype=torch.uint8))
    if isinstance(e.value, h.HippoError):            # (without a GPU there is no current stream to ask for)
        assert e.value.status == h.ERR_BAD_SHAPE and "hippo_score_tokens failed" in str(e.value)


def test_whole_numbers_of_any_kind_are_taken():
    for n in (np.int64(38), np.int32(38), torch.tensor(38)):
        with pytest.raises(AssertionError):          # the length is read, then the caches' shapes are compared
            h.hippo_verify_attention(queries(), cache(), cache(N=41), n)


def test_layers_take_embeddings_that_are_cut_from_a_longer_sequence():
    # one batch element, whose stride nobody reads: not refused by the binding (without a GPU, by the stream it asks for)
    emb = torch.zeros((1, 40, 64), dtype=torch.bfloat16)[:, 3:35]
    with pytest.raises((h.HippoError, RuntimeError)):
        h.hippo_score_tokens_layers([queries()], [cache(N=20)], VID, emb=emb, scores_out=torch.zeros((1, 32)),
                                    workspace=torch.zeros(1 << 16, dtype=torch.uint8))


def embeddings(B=1, n=32, ch=64, dtype=torch.bfloat16):
    return torch.zeros((B, n, ch), dtype=dtype)


@pytest.mark.parametrize("B, emb", [
    (1, embeddings(ch=128)[..., ::2]),                               # channels that are not side by side
    (2, embeddings(B=2, n=40)[:, 3:35]), (2, embeddings(B=2, n=40)),  # batch elements that are not N_v tokens apart
    (1, embeddings(n=31)), (2, embeddings(B=1)),                     # too few tokens, too few batch elements
    (1, embeddings(dtype=torch.float32)),                            # another type than the cache's
    (1, embeddings()[None]),
])
def test_embeddings_that_the_kernels_would_misread(B, emb):
    q, k = queries(B=B), cache(B=B)
    given = dict(emb=emb, scores_out=torch.zeros((B, 32)), workspace=torch.zeros(1 << 16, dtype=torch.uint8))
    with pytest.raises(AssertionError):
        h.hippo_score_tokens(q, k, VID, **given)
    with pytest.raises(AssertionError):
        h.hippo_score_tokens_layers([q, q], [k, k], VID, **given)


@pytest.mark.parametrize("B, emb", [(1, embeddings(B=2)), (2, embeddings(B=3)), (1, embeddings(B=2, n=40))])
def test_more_embeddings_than_the_caches_have_elements(B, emb):
    given = dict(emb=emb, scores_out=torch.zeros((B, 32)), workspace=torch.zeros(1 << 16, dtype=torch.uint8))
    q, k = queries(B=B), cache(B=B, N=20)
    with pytest.raises((h.HippoError, RuntimeError)):       # (without a GPU, refused by the stream it asks for)
        h.hippo_score_tokens(q, k, VID, **given)
    with pytest.raises((h.HippoError, RuntimeError)):
        h.hippo_score_tokens_layers([q, q], [k, k], VID, **given)


def test_embeddings_that_no_term_reads_are_not_looked_at():
    with pytest.raises((h.HippoError, RuntimeError)):       # (without a GPU, refused by the stream it asks for)
        h.hippo_score_tokens_layers([queries()], [cache(N=20)], VID, emb=embeddings(n=31, dtype=torch.float32),
                                    flags=h.SCORE_ATTN, scores_out=torch.zeros((1, 32)),
                                    workspace=torch.zeros(1 << 16, dtype=torch.uint8))


@pytest.mark.parametrize("as_layers", [list, tuple, torch.stack, lambda t: torch.nn.ParameterList([x for x in t])])
def test_layers_come_in_anything_with_a_length_and_an_index(as_layers):
    given = dict(scores_out=torch.zeros((1, 32)), workspace=torch.zeros(1 << 16, dtype=torch.uint8))
    layers = lambda t: as_layers([t] * 3)
    with pytest.raises((h.HippoError, RuntimeError)):       # (without a GPU, refused by the stream it asks for)
        h.hippo_score_tokens_layers(layers(queries(dtype=torch.float32)), layers(cache(N=20, dtype=torch.float32)), VID, **given)
    with pytest.raises(AssertionError):                     # one layer's queries more than its keys
        h.hippo_score_tokens_layers(layers(queries(dtype=torch.float32)), [cache(dtype=torch.float32)] * 2, VID, **given)
    for no_layers in (torch.tensor(1.0), {queries()}, iter([queries()]), None):
        with pytest.raises(TypeError):
            h.hippo_score_tokens_layers(no_layers, [cache()], VID, **given)


def test_page_tables_with_a_dimension_of_one_behind():
    pool = cache(N=2)
    with pytest.raises((h.HippoError, RuntimeError)):       # (without a GPU, refused by the stream it asks for)
        h.hippo_verify_attention_paged(queries(), pool, pool, torch.zeros((1, 3, 1), dtype=torch.int32), 38,
                                       workspace=torch.zeros(1 << 16, dtype=torch.uint8))


def test_why_the_binding_cannot_be_imported_is_said(monkeypatch):
    class Refuse:                                           # as a module built for another Python or torch is refused
        @staticmethod
        def find_spec(name, path=None, target=None):
            if name == h.__name__ + "._binding":
                raise ImportError("undefined symbol: of another torch")

    monkeypatch.setattr(h, "_native", None)
    monkeypatch.delattr(h, "_binding", raising=False)
    monkeypatch.delitem(sys.modules, h.__name__ + "._binding", raising=False)
    monkeypatch.setattr(sys, "meta_path", [Refuse] + sys.meta_path)
    with pytest.raises(RuntimeError, match="undefined symbol: of another torch.*no fallback"):
        h.hippo_verify_attention(queries(), cache(), cache(), 38)
