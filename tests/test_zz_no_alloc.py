"""ee_verify_static (the entry point for callers that cannot allocate GPU memory) against
ee_verify, through the C ABI: same kernels, scratch in the library's static device array
instead of the session's buffers.  Results must be bit-identical."""
import numpy as np
import pytest

import eegen
import paper_2505_21594_amd as ee

pytestmark = pytest.mark.gpu

MID = eegen.ModelConfig(n_layers=3, d_model=1280, n_heads=10, head_dim=128, d_ffn=1072, vocab=3000,
                        exit_layers=(1, 2))


def _same(a, b, what):
    assert a.accept_len == b.accept_len and a.next_token == b.next_token, what
    assert np.array_equal(a.final_tokens, b.final_tokens), what
    assert np.array_equal(a.exit_tokens, b.exit_tokens) and np.array_equal(a.exit_accept_len, b.exit_accept_len), what
    assert np.array_equal(a.final_conf.view(np.uint32), b.final_conf.view(np.uint32)), what
    assert np.array_equal(a.exit_conf.view(np.uint32), b.exit_conf.view(np.uint32)), what


def test_static_scratch_matches_session_scratch(model_dir):
    path = f"{model_dir}/noalloc_mid.bin"
    eegen.write_model(path, MID, 91, gains="uniform", std=0.03)
    g = ee.Model(path)
    exits = [1, 2]
    prompt = eegen.prompt_tokens(92, 150, MID.vocab)
    a = g.session(256, max_gamma=8, flags=ee.KEEP_LOGITS)    # ee_verify, its own scratch
    b = g.session(256, max_gamma=8, flags=ee.KEEP_LOGITS)    # ee_verify_static
    try:
        assert a.ee_prefill(prompt) == b.ee_prefill(prompt)
        # two calls in a row, the second with a smaller input; the array keeps the first call's contents
        for call, gamma in enumerate((8, 3)):
            drafts = eegen.prompt_tokens(93 + call, gamma, MID.vocab)
            if call == 0:
                drafts[0] = a.ee_pending()      # (any ids would do; makes the passes differ in what they accept)
            a.ee_verify(drafts, exits)
            a.ee_wait_final()
            b.ee_verify_static(drafts, exits)
            b.ee_wait_exit(0)
            b.ee_wait_final()
            ra, rb = a.final_result(), b.final_result()
            _same(ra, rb, f"call {call} gamma {gamma}")
            for e in range(len(exits) + 1):
                la, lb = a.ee_debug_logits(e), b.ee_debug_logits(e)
                assert np.array_equal(la.view(np.uint32), lb.view(np.uint32)), f"call {call} head {e}: logits differ"
            assert a.ee_kv_len() == b.ee_kv_len() and a.ee_pending() == b.ee_pending()
        # the ordinary entry point still works on a session that has used the static one, and the other way round
        drafts = eegen.prompt_tokens(97, 5, MID.vocab)
        b.ee_verify(drafts, exits)
        b.ee_wait_final()
        a.ee_verify_static(drafts, exits)
        a.ee_wait_final()
        _same(a.final_result(), b.final_result(), "entry points swapped")
    finally:
        a.free()
        b.free()
        g.free()


@pytest.mark.parametrize("n_adapters,gamma,max_rows", [(0, 4, 48), (2, 4, 48), (0, 1, 48), (0, 15, 48), (2, 1, 6)])
def test_static_scratch_holds_the_rows_of_grouped_exits(model_dir, n_adapters, gamma, max_rows):
    """Three exits whose heads share one launch (OPT_HEAD_BATCH): the LM head's input then holds the
    rows of all three, and layers run between the first deposit and the launch.  (15, 48): the largest group."""
    cfg = eegen.ModelConfig(n_layers=5, d_model=512, n_heads=4, head_dim=128, d_ffn=1072, vocab=1500, exit_layers=(1, 2, 3),
                            n_adapters=n_adapters, adapter_width=64 if n_adapters else 0)
    path = f"{model_dir}/noalloc_groups_{n_adapters}.bin"
    eegen.write_model(path, cfg, 92, gains="uniform", std=0.04)
    g = ee.Model(path, max_rows=max_rows)
    a, b, c = (g.session(256, max_gamma=gamma, flags=ee.KEEP_LOGITS | ee.NO_AUTOCOMMIT) for _ in range(3))
    try:
        prompt = eegen.prompt_tokens(94, 75, cfg.vocab)
        for s in (a, b, c):
            s.ee_prefill(prompt)
        a.ee_session_option(ee.OPT_HEAD_BATCH, 3)
        b.ee_session_option(ee.OPT_HEAD_BATCH, 3)
        exits = [1, 2, 3]
        drafts = eegen.prompt_tokens(95, gamma, cfg.vocab)
        a.ee_verify(drafts, exits)
        b.ee_verify_static(drafts, exits)
        c.ee_verify(drafts, exits)                       # one launch per exit: what grouping may not change
        for s in (a, b, c):
            s.ee_wait_final()
        _same(a.final_result(), b.final_result(), "grouped exits")
        assert np.array_equal(a.final_result().exit_tokens, c.final_result().exit_tokens)
        for e in range(len(exits) + 1):
            la, lb, lc = (s.ee_debug_logits(e).view(np.uint32) for s in (a, b, c))
            assert np.array_equal(la, lb) and np.array_equal(la, lc), f"head {e}: logits differ"
    finally:
        for s in (a, b, c):
            s.free()
        g.free()


def test_static_scratch_takes_what_just_fits(model_dir):
    """16 rows of this width leave 1408 bytes of the 8 MiB: residual stream and queries 2 * 16 * 64 * 4, five
    inputs 4 * 16 * 64 (or 32 for the adapters' units), activations 4 * 16 * 129024, partial sums and candidates
    24 * 256 * 16, counters 2 * 256, one attention item 16 * (64 + 2) * 4.  A second exit's head rows (4 KB) do not
    fit beside them: grouping then has no effect."""
    cfg = eegen.ModelConfig(n_layers=3, d_model=64, n_heads=1, head_dim=64, d_ffn=129024, vocab=512, exit_layers=(1, 2))
    path = f"{model_dir}/noalloc_edge.bin"
    eegen.write_model(path, cfg, 6, gains="uniform", std=0.02)
    g = ee.Model(path, max_rows=16)
    a, b = (g.session(64, max_gamma=15, flags=ee.KEEP_LOGITS | ee.NO_AUTOCOMMIT) for _ in range(2))
    try:
        prompt, drafts = eegen.prompt_tokens(8, 12, cfg.vocab), eegen.prompt_tokens(9, 15, cfg.vocab)
        for s in (a, b):
            s.ee_prefill(prompt)
            s.ee_session_option(ee.OPT_ATT_SPLITS, 1)     # (the session's own scratch has room for more)
        b.ee_session_option(ee.OPT_HEAD_BATCH, 2)
        a.ee_verify(drafts, [1, 2])
        a.ee_wait_final()
        b.ee_verify_static(drafts, [1, 2])
        b.ee_wait_final()
        _same(a.final_result(), b.final_result(), "at the limit")
    finally:
        a.free()
        b.free()
        g.free()


def test_static_scratch_rejects_what_does_not_fit(model_dir):
    """Sizes beyond the array's 8 MiB are refused with EE_ECAPACITY before anything is enqueued:
    a model whose FFN width makes the gate/up output of 16 rows alone larger than the array."""
    wide = eegen.ModelConfig(n_layers=1, d_model=256, n_heads=4, head_dim=64, d_ffn=140000, vocab=1024)
    path = f"{model_dir}/noalloc_wide.bin"
    eegen.write_model(path, wide, 5)
    g = ee.Model(path)
    s = g.session(64, max_gamma=15)
    try:
        s.ee_prefill(eegen.prompt_tokens(6, 9, wide.vocab))
        kv, pend = s.ee_kv_len(), s.ee_pending()
        with pytest.raises(ee.EEError) as e:
            s.ee_verify_static(eegen.prompt_tokens(7, 15, wide.vocab), [])
        assert e.value.code == ee.EE_ECAPACITY and "static scratch" in str(e.value)
        assert s.ee_kv_len() == kv and s.ee_pending() == pend
        r = s.verify_sync(eegen.prompt_tokens(7, 15, wide.vocab), [])       # the session is unharmed
        assert 0 <= r.accept_len <= 15
        # a single row of the same model fits
        s.ee_verify_static(eegen.prompt_tokens(8, 1, wide.vocab), [])
        s.ee_wait_final()
    finally:
        s.free()
        g.free()
