"""Packed weights (12 bits a weight, the rest in lists) against the oracle, which reads the plain ones.

A model as small as the packing rule admits with every kind of matrix above its line, ragged in K (4112 = 128.5 k-tiles) and in
columns (5003), with weights outside the window of exponents planted where a list or a tile can go wrong."""
import ctypes

import numpy as np
import pytest

import eegen
import paper_2505_21594_amd as ee
from oracle import oracle as eo
from tests.parity import check_first_token, check_pass, gpu_logits, oracle_prefill
from tests.test_gpu_parity import TWO_TERMS, check_two_terms

pytestmark = pytest.mark.gpu

CFG = eegen.ModelConfig(n_layers=2, d_model=4096, n_heads=32, head_dim=128, d_ffn=4112, vocab=5003, exit_layers=(1,))


def _bf16(x):
    return int(eegen.f32_to_bf16(np.array([x]))[0])


def _plant(path):
    t = eegen.open_tensors(path, "r+")
    rng = np.random.default_rng(5)
    for name, w in t.items():
        if w.ndim != 2 or name == "emb":
            continue
        N, K = w.shape
        # outliers at the corners of the matrix and of tiles, on both sides of the groups' and K slices' borders, and anywhere
        for n, k in [(0, 0), (N - 1, K - 1), (0, K - 1), (N - 1, 0), (15, 31), (16, 32), (N // 2, K // 4 - 1), (N // 2, K // 4)]:
            w[n, k] = _bf16(-0.75)
        for n, k in zip(rng.integers(0, N, 60), rng.integers(0, K, 60)):
            w[n, k] = _bf16(rng.choice([-1.0, 1.0]) * rng.uniform(0.6, 1.5))
        # one column with more than a batch of eight, neighbours of it with none
        w[37, rng.permutation(K)[:20]] = _bf16(0.5)
        # zeros of both signs, the smallest normal and a denormal number, and the window's smallest value's neighbours below
        w[50, :4] = [0x0000, 0x8000, 0x0080, 0x0003]
        w[rng.integers(0, N, 80), rng.integers(0, K, 80)] = 0
    t["l2.wd"][::5] = 0       # far too many: this matrix stays plain, those beside it do not


@pytest.fixture(scope="module")
def pair(model_dir):
    p = f"{model_dir}/gpu_packed.bin"
    eegen.write_model(p, CFG, 77, gains="uniform")
    _plant(p)
    g, o = ee.Model(p, max_rows=48), eo.Model(p)
    yield g, o
    g.free()


# rows 2, 5, 8, 9, 16 in one session; 18, 25, 40, 48 over several (K split over workgroups; the last part of every kilobyte count)
@pytest.mark.parametrize("B,gamma", [(1, 1), (1, 4), (1, 7), (1, 8), (1, 15), (3, 5), (5, 4), (8, 4), (6, 7)])
def test_packed_pass(pair, B, gamma):
    """Logits of every head within the two-term bound (check_two_terms: 10 units a layer, two layers and the head: 1.0e-5 by its
    count, the bound is for four), tokens and accept lengths as everywhere; the same pass again gives the same bits.  An outlier missed or
    counted twice moves its column by 0.6 to 1.5 of an input, 3e-3 of the logits and more."""
    g, o = pair
    sess, osess = [], []
    try:
        for b in range(B):
            toks = eegen.prompt_tokens(900, 7 + 3 * b, o.vocab, session=b)
            gs = g.session(64, max_gamma=gamma, flags=ee.NO_AUTOCOMMIT | (ee.KEEP_LOGITS if b == 0 else 0))
            os_ = o.session(64)
            fo, margin = oracle_prefill(os_, toks)
            check_first_token(gs, gs.ee_prefill(toks), fo, margin, f"packed B={B} session {b}")
            sess.append(gs)
            osess.append(os_)
        drafts = [eegen.prompt_tokens(901, gamma, o.vocab, session=b) for b in range(B)]
        seen = []
        for again in range(2):
            ee.ee_verify_batch(sess, drafts, [1])
            for s in sess:
                s.ee_wait_final()
            seen.append([s.ee_debug_logits(e).view(np.uint32) for s in sess for e in range(2)])
        assert all(np.array_equal(x, y) for x, y in zip(*seen))
        for b in range(B):
            ro = osess[b].verify(drafts[b], [1], commit=False, want_logits=True)
            z = gpu_logits(sess[b], 1)
            check_pass(ro, sess[b].final_result(), z, drafts[b], f"packed B={B} gamma={gamma} session {b}")
            check_two_terms(ro, z)
    finally:
        for s in sess:
            s.free()


@pytest.mark.parametrize("name", ["l1.wq", "l2.wo", "l1.wu", "l1.wd", "w_lm"])
def test_one_outlier_is_seen(pair, model_dir, name):
    """A mistake planted in the oracle: without one of a matrix's outliers its logits are far outside the bound, so the test
    above sees a single escape that is lost."""
    g, _ = pair
    p = f"{model_dir}/gpu_packed.bin"
    t = eegen.open_tensors(p, "r+")[name]
    n, kept = 0, int(t[0, 0])
    assert abs(float(eegen.bf16_to_f32(t[0, :1])[0])) == 0.75
    toks, drafts = eegen.prompt_tokens(902, 9, CFG.vocab), eegen.prompt_tokens(903, 4, CFG.vocab)
    gs = g.session(64, max_gamma=4, flags=ee.NO_AUTOCOMMIT | ee.KEEP_LOGITS)
    try:
        first = gs.ee_prefill(toks)
        gs.verify_sync(drafts, [1])
        z = np.stack(gpu_logits(gs, 1)).astype(np.float64)
        t[n, 0] = 0
        o = eo.Model(p)
        os_ = o.session(64)
        os_.prefill(toks, flags=eo.HOLD_LAST)
        # the same rows as the GPU's pass: the prompt's last token, then what it took as pending and the drafts
        os_.verify([(first + 1) % CFG.vocab], commit=True)
        os_.set_pending(first)
        ro = os_.verify(drafts, [1], commit=False, want_logits=True)
        assert np.linalg.norm(z - ro.logits) / np.linalg.norm(ro.logits) > 10 * TWO_TERMS
    finally:
        t[n, 0] = kept
        gs.free()


@pytest.mark.parametrize("split,B,gamma,d", [(False, 1, 4, 512), (False, 3, 7, 512), (False, 2, 15, 2048), (True, 1, 4, 512), (True, 3, 5, 512), (True, 8, 5, 512)])
def test_packed_groups_of_tiles(model_dir, split, B, gamma, d):
    """Matrices whose workgroups own more n-tiles than a group has (gate/up 8 and 10, LM head 9 and 10): every group has lists and sums of
    its own; with K split over workgroups for every kind, every slice."""
    cfg = eegen.ModelConfig(n_layers=2, d_model=d, n_heads=d // 64, head_dim=64, d_ffn=17408, vocab=40000, exit_layers=(1,))
    p = f"{model_dir}/gpu_packed_wide.bin"
    eegen.write_model(p, cfg, 78, gains="uniform", std=0.03)
    t = eegen.open_tensors(p, "r+")
    rng = np.random.default_rng(6)
    for name in ("l1.wg", "l1.wu", "l2.wg", "l2.wu", "w_lm"):
        w = t[name]
        for n, k in [(0, 0), (w.shape[0] - 1, w.shape[1] - 1)] + list(zip(rng.integers(0, w.shape[0], 150), rng.integers(0, w.shape[1], 150))):
            w[n, k] = _bf16(rng.choice([-1.0, 1.0]) * rng.uniform(0.8, 1.6))
    if split:
        ee.ee_tune_k_split(127, 2)
    try:
        g = ee.Model(p, max_rows=48)
    finally:
        ee.ee_tune_k_split(0b1010, 2)   # back to the default
    o = eo.Model(p)
    sess, osess = [], []
    try:
        for b in range(B):
            toks = eegen.prompt_tokens(910, 7 + 3 * b, o.vocab, session=b)
            gs = g.session(64, max_gamma=gamma, flags=ee.NO_AUTOCOMMIT | (ee.KEEP_LOGITS if b == 0 else 0))
            os_ = o.session(64)
            fo, margin = oracle_prefill(os_, toks)
            check_first_token(gs, gs.ee_prefill(toks), fo, margin, f"session {b}")
            sess.append(gs)
            osess.append(os_)
        drafts = [eegen.prompt_tokens(911, gamma, o.vocab, session=b) for b in range(B)]
        ee.ee_verify_batch(sess, drafts, [1])
        for s in sess:
            s.ee_wait_final()
        for b in range(B):
            ro = osess[b].verify(drafts[b], [1], commit=False, want_logits=True)
            z = gpu_logits(sess[b], 1)
            check_pass(ro, sess[b].final_result(), z, drafts[b], f"groups B={B} session {b}")
            check_two_terms(ro, z)
    finally:
        for s in sess:
            s.free()
        g.free()


# d_ffn = 16 (mod 32): half of the down projection's last k-tile is padding.  4112: 129 k-tiles, never split; 4080: 128, split for more than 16 rows
@pytest.mark.parametrize("d_ffn,B,gamma", [(4112, 1, 4), (4112, 3, 5), (4080, 1, 4), (4080, 8, 4)])
def test_padded_k_tile_adds_nothing(model_dir, d_ffn, B, gamma):
    """A padding weight of a packed tile is not zero, so its input has to be: whatever rows an earlier pass had (its activations
    lie where the padding columns of another row count are), a pass gives the same bits, and ee_verify_static those of ee_verify."""
    cfg = eegen.ModelConfig(n_layers=2, d_model=4096, n_heads=32, head_dim=128, d_ffn=d_ffn, vocab=1024, exit_layers=(1,))
    p = f"{model_dir}/gpu_packed_padded.bin"
    eegen.write_model(p, cfg, 79, gains="uniform")
    g = ee.Model(p, max_rows=48)
    drafts = [eegen.prompt_tokens(921, gamma, cfg.vocab, session=b) for b in range(B)]

    def sessions():
        out = [g.session(64, max_gamma=15, flags=ee.NO_AUTOCOMMIT | ee.KEEP_LOGITS) for _ in range(B)]
        for b, s in enumerate(out):
            s.ee_prefill(eegen.prompt_tokens(920, 3 + b, cfg.vocab, session=b))
        return out

    def logits(ss, static=False):
        if static:
            ss[0].ee_verify_static(drafts[0], [1])
        else:
            ee.ee_verify_batch(ss, drafts, [1])
        for s in ss:
            s.ee_wait_final()
        return np.stack([s.ee_debug_logits(e) for s in ss for e in range(2)]).view(np.uint32)

    fresh, used = sessions(), sessions()
    try:
        want = logits(fresh)
        for n, other in ((1, 15), (1, 1), (min(B, 3), 15)):
            ee.ee_verify_batch(used[:n], [eegen.prompt_tokens(922, other, cfg.vocab, session=b) for b in range(n)], [1])
            for s in used[:n]:
                s.ee_wait_final()
            assert np.array_equal(logits(used), want), (n, other)
        if B == 1:
            assert np.array_equal(logits(used, static=True), want)
    finally:
        for s in fresh + used:
            s.free()
        g.free()


def test_a_matrix_that_stays_plain_takes_no_more_memory(model_dir):
    """Zeros in a fifth of the rows are far too many weights outside the window: such a matrix has no packed form and holds no memory
    for one.  Layer 1 alone (layer 2's packed form then moves to its place: a pass against the oracle), then the whole model.  (Places no wave's sequence reaches: up to 5 %; the
    runtime hands out pages of 2 MB and keeps some.)"""
    cfg = eegen.ModelConfig(n_layers=2, d_model=4096, n_heads=32, head_dim=128, d_ffn=4096, vocab=5008, exit_layers=(1,))
    p = f"{model_dir}/gpu_packed_memory.bin"
    eegen.write_model(p, cfg, 80, gains="uniform")
    t = eegen.open_tensors(p, "r+")
    lib = ee.load_library()

    def free_bytes():
        free, total = ctypes.c_size_t(), ctypes.c_size_t()
        assert lib.hipMemGetInfo(ctypes.byref(free), ctypes.byref(total)) == 0
        return free.value

    def used(check=False):
        before = free_bytes()
        g = ee.Model(p)
        took = before - free_bytes()
        if check:
            toks, drafts, o = eegen.prompt_tokens(930, 9, cfg.vocab), eegen.prompt_tokens(931, 4, cfg.vocab), eo.Model(p)
            gs, os_ = g.session(64, max_gamma=4, flags=ee.NO_AUTOCOMMIT | ee.KEEP_LOGITS), o.session(64)
            fo, margin = oracle_prefill(os_, toks)
            check_first_token(gs, gs.ee_prefill(toks), fo, margin, "moved")
            gs.verify_sync(drafts, [1])
            check_two_terms(os_.verify(drafts, [1], commit=False, want_logits=True), gpu_logits(gs, 1))
            gs.free()
        g.free()
        return took

    ee.Model(p).free()
    packed = used()
    for name, w in t.items():
        if name.startswith("l1.w"):
            w[::5] = 0
    half = used(check=True)
    for name, w in t.items():
        if name.startswith("l2.w") or name == "w_lm":
            w[::5] = 0
    plain = used()
    d, F, V = cfg.d_model, cfg.d_ffn, cfg.vocab
    layer, head, emb = 2 * (4 * d * d + 3 * F * d), 2 * V * d, 2 * V * d
    for took, want in ((plain, 2 * layer + head + emb), (packed - half, 0.75 * layer), (half - plain, 0.75 * (layer + head))):
        assert 0.97 * want <= took <= 1.08 * want, (took, want)


@pytest.mark.parametrize("B,gamma", [(1, 4), (8, 4)])
def test_the_caller_chooses_the_form(pair, model_dir, B, gamma):
    """EE_FORM_PLAIN holds nothing packed, EE_FORM_PACKED the same as the default on an empty device, bit for bit; plain and packed weights
    give the same results to rounding: each is within the two-term bound of the oracle, so they are within twice that of each other."""
    auto, _ = pair
    p = f"{model_dir}/gpu_packed.bin"
    plain, packed = ee.Model(p, max_rows=48, form=ee.FORM_PLAIN), ee.Model(p, max_rows=48, form=ee.FORM_PACKED)

    def logits(g):
        ss = [g.session(64, max_gamma=gamma, flags=ee.NO_AUTOCOMMIT | ee.KEEP_LOGITS) for _ in range(B)]
        for b, s in enumerate(ss):
            s.ee_prefill(eegen.prompt_tokens(940, 6 + b, CFG.vocab, session=b))
        ee.ee_verify_batch(ss, [eegen.prompt_tokens(941, gamma, CFG.vocab, session=b) for b in range(B)], [1])
        for s in ss:
            s.ee_wait_final()
        z = np.stack([s.ee_debug_logits(e) for s in ss for e in range(2)])
        for s in ss:
            s.free()
        return z

    try:
        assert plain.packed_bytes() == 0 and packed.packed_bytes() == auto.packed_bytes() > 0
        a, b, c = logits(auto), logits(packed), logits(plain)
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
        assert not np.array_equal(a, c) and np.linalg.norm(a.astype(np.float64) - c) / np.linalg.norm(c.astype(np.float64)) < 2 * TWO_TERMS
    finally:
        plain.free()
        packed.free()


# K of 64 a row: 3072 packs QKV and gate/up at 48 rows, 2048 gate/up (all that is large enough to pack) at 32 and not at 33
@pytest.mark.parametrize("d,F,V,B,gamma,packed", [(3072, 3072, 4096, 3, 15, True), (2048, 5632, 4096, 2, 15, True), (2048, 5632, 4096, 3, 10, False)])
def test_short_k_beside_many_rows_is_streamed_plain(model_dir, d, F, V, B, gamma, packed):
    """The dispatch's line: below it a launch is the plain one, bit for bit; on both sides results are within the two-term bound of the oracle."""
    cfg = eegen.ModelConfig(n_layers=2, d_model=d, n_heads=d // 128, head_dim=128, d_ffn=F, vocab=V, exit_layers=(1,))
    p = f"{model_dir}/gpu_packed_line.bin"
    eegen.write_model(p, cfg, 81, gains="uniform")
    o, z = eo.Model(p), []
    toks = [eegen.prompt_tokens(950, 50 + b, V, session=b) for b in range(B)]   # (more than max_rows rows: their cache is the same in both forms)
    drafts = [eegen.prompt_tokens(951, gamma, V, session=b) for b in range(B)]
    for form in (ee.FORM_PACKED, ee.FORM_PLAIN):
        g = ee.Model(p, max_rows=48, form=form)
        ss = [g.session(80, max_gamma=gamma, flags=ee.NO_AUTOCOMMIT | ee.KEEP_LOGITS) for _ in range(B)]
        firsts = [s.ee_prefill(t) for s, t in zip(ss, toks)]
        for s in ss:
            s.ee_set_pending(7)
        ee.ee_verify_batch(ss, drafts, [1])
        for s in ss:
            s.ee_wait_final()
        z.append(np.stack([s.ee_debug_logits(e) for s in ss for e in range(2)]))
        if form == ee.FORM_PACKED:
            for b, s in enumerate(ss):
                os_ = o.session(80)
                fo, margin = oracle_prefill(os_, toks[b])
                check_first_token(s, firsts[b], fo, margin, f"session {b}")
                os_.set_pending(7)
                ro = os_.verify(drafts[b], [1], commit=False, want_logits=True)
                check_two_terms(ro, gpu_logits(s, 1))
        for s in ss:
            s.free()
        g.free()
    assert np.array_equal(z[0].view(np.uint32), z[1].view(np.uint32)) != packed
