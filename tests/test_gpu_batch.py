"""GPU parity of the panel / batched paths (more than 8 vectors, hypotheses of several sentences
side by side; Section 6's "batching"): every product on the int8 matrix cores.

Per-vector quantization makes a panel's result for vector j the result of the single-vector
call, so each case is checked twice: against the oracle (codes and sums bit-exact through the
taps, floats to 1e-5) and against this library's own streaming kernels (bit for bit).
"""
import ctypes
import time

import numpy as np
import pytest
import torch

from parity import assert_close, assert_same, np_, gpu_gru, gpu_mat
from workloads import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import paper_1804_05038_amd as q
    return q


@pytest.fixture(scope="module")
def ctx(q):
    return q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=160, max_l=256, max_rows=50000, max_ld=2048) + (64 << 20))


def _check_product(oracle, L, x_gpu, tap, j, what):
    xq, xs = oracle.quantize(x_gpu)
    assert_same(tap["xq"][j], xq, what + " xq")
    assert float(tap["xscale"][j]) == float(xs), what + " xscale"
    acc = oracle.accumulate(L.Wq, L.cols, xq)
    assert_same(tap["acc"][j], acc, what + " acc")
    return oracle.dequantize(acc, L.scale, xs, L.bias)


@pytest.mark.parametrize("I,H,n,tiled", [(512, 1024, 9, False), (512, 1024, 70, False), (2048, 1024, 33, False), (36, 20, 12, False),
                                         (620, 1000, 17, False), (256, 256, 130, False), (512, 1024, 70, True), (512, 1024, 145, True),
                                         (2048, 1024, 33, True), (256, 256, 130, True), (1024, 1000, 20, True)])
def test_gru_step_panel(q, ctx, oracle, I, H, n, tiled):
    p = synth.gru_cell(seed=0, I=I, H=H, n_batch=n)
    p["x"] = p["x"] * np.random.default_rng(n).uniform(0.1, 10, (n, 1)).astype(np.float32)
    g = oracle.QGru(p["Wx"], p["Wh"], p["bx"], p["bh"])
    G = q.GruWeights(gpu_mat(q, ctx, p["Wx"], tiled), gpu_mat(q, ctx, p["Wh"], tiled), ctx.f32(p["bx"]), ctx.f32(p["bh"]))
    x, h0 = ctx.f32(p["x"]), ctx.f32(p["h_prev"])
    h, taps = q.gru_step_q8(ctx, G, x, h0, taps=True)
    for j in range(0, n, max(1, n // 7)):
        gx = _check_product(oracle, g.Wx, p["x"][j], taps[0], j, "Wx")
        gh = _check_product(oracle, g.Wh, p["h_prev"][j], taps[1], j, "Wh")
        assert_close(h[j], oracle.gru_gates(gx, gh, p["h_prev"][j]), "h' (teacher-forced)")
        assert_close(h[j], g.step(p["x"][j], p["h_prev"][j]), "h' (free-running)")
    assert_same(q.gru_step_q8(ctx, G, x, h0), np_(h), "no taps")
    # the streaming kernel on groups of at most 8 vectors gives the same bits
    for j0 in (0, n - 5):
        assert_same(q.gru_step_q8(ctx, G, x[j0:j0 + 5].contiguous(), h0[j0:j0 + 5].contiguous()), np_(h)[j0:j0 + 5],
                    "panel vs streaming kernel")


@pytest.mark.parametrize("V,R,n,k", [(50000, 512, 20, 12), (300, 64, 9, 12), (1000, 512, 130, 5), (33658, 640, 11, 12),
                                     (129, 48, 40, 16)])
def test_output_layer_panel_given_t(q, ctx, oracle, V, R, n, k):
    p = synth.output_layer(seed=2, V=V, R=R, n_beam=n)
    L = oracle.QLinear(p["out.W"], p["out.b"])
    W = gpu_mat(q, ctx, p["out.W"])
    t = ctx.f32(p["t"])
    r = q.output_logits_q8(ctx, None, W, ctx.f32(p["out.b"]), t_in=t, k=k, taps=True)
    tap = r["taps"][3]
    for j in range(0, n, max(1, n // 6)):
        logits_ref = _check_product(oracle, L, p["t"][j], tap, j, "W_out")
        assert_same(r["logits"][j], logits_ref, "logits")
        lse, lp, idx = oracle.logsoftmax_topk(logits_ref, k)
        assert_close(r["lse"][j:j + 1], np.array([lse]), "lse")
        assert_same(r["topk_idx"][j], idx, "top-k indices")
        assert_close(r["topk_logp"][j], lp, "top-k logp")
    r2 = q.output_logits_q8(ctx, None, W, ctx.f32(p["out.b"]), t_in=t, k=k, want_logits=False)
    assert_same(r2["topk_idx"], np_(r["topk_idx"]), "logits in the workspace: same top-k")
    r8 = q.output_logits_q8(ctx, None, W, ctx.f32(p["out.b"]), t_in=t[:8].contiguous(), k=k)
    assert_same(r8["logits"], np_(r["logits"])[:8], "panel vs streaming kernel: logits")
    assert_same(r8["topk_idx"], np_(r["topk_idx"])[:8], "panel vs streaming kernel: top-k")
    assert_same(r8["topk_logp"], np_(r["topk_logp"])[:8])


def test_output_layer_panel_with_readout(q, ctx, oracle):
    n = 23
    p = synth.full_model(seed=4, V=3000, E=512, H=1024, A=64, R=512)
    m = oracle.OracleModel(p)
    rng = np.random.default_rng(n)
    s, y, c = (rng.standard_normal((n, d)).astype(np.float32) for d in (1024, 512, 2048))
    ro = q.ReadoutWeights(gpu_mat(q, ctx, p["ro.Ws"]), gpu_mat(q, ctx, p["ro.Wy"]), gpu_mat(q, ctx, p["ro.Wc"]),
                          ctx.f32(p["ro.b"]))
    W = gpu_mat(q, ctx, p["out.W"])
    r = q.output_logits_q8(ctx, ro, W, ctx.f32(p["out.b"]), s=ctx.f32(s), y_emb=ctx.f32(y), ctx_vec=ctx.f32(c),
                           k=12, taps=True)
    T = r["taps"]
    Ls = oracle.QLinear(p["ro.Ws"])
    for j in range(0, n, 4):
        u1 = _check_product(oracle, Ls, s[j], T[0], j, "W_s")
        u2 = _check_product(oracle, m.ro_y, y[j], T[1], j, "W_y")
        u3 = _check_product(oracle, m.ro_c, c[j], T[2], j, "W_c")
        pre = ((u1 + u2) + u3) + p["ro.b"]
        t_gpu = np_(r["t"])[j]
        assert_close(t_gpu, np.tanh(pre.astype(np.float64)).astype(np.float32), "t (teacher-forced)")
        assert_close(t_gpu, m.readout(s[j], y[j], c[j]), "t (free-running)")
        logits = _check_product(oracle, m.out, t_gpu, T[3], j, "W_out")
        lse, lp, idx = oracle.logsoftmax_topk(logits, 12)
        assert_same(r["topk_idx"][j], idx); assert_close(r["topk_logp"][j], lp)
    r5 = q.output_logits_q8(ctx, ro, W, ctx.f32(p["out.b"]), s=ctx.f32(s[:5]), y_emb=ctx.f32(y[:5]), ctx_vec=ctx.f32(c[:5]), k=12)
    assert_same(r5["t"], np_(r["t"])[:5], "panel vs streaming kernels: t")
    assert_same(r5["topk_idx"], np_(r["topk_idx"])[:5]); assert_same(r5["topk_logp"], np_(r["topk_logp"])[:5])


@pytest.mark.parametrize("E,H,A,lens,beam,tiled", [(512, 1024, 1024, (30, 11, 50), 5, False), (36, 40, 28, (7, 1, 3, 12), 3, False),
                                                   (64, 64, 64, (5, 300), 2, True), (512, 1024, 1024, (9,) * 26, 5, False),
                                                   (512, 1024, 1024, (9,) * 26, 5, True), (512, 1024, 1024, (30, 11, 50), 5, True),
                                                   (512, 1024, 1024, (4,) * 67, 3, True), (512, 1024, 1024, (3, 5, 2) * 20, 5, True),
                                                   (64, 64, 64, (2, 7, 1) * 30, 3, False), (64, 64, 64, (3,) * 130, 7, False)])
def test_cgru_decoder_step_batch(q, ctx, oracle, E, H, A, lens, beam, tiled):
    """tiled: the weights also carry their tile-packed copies, which the panel's matrix-core kernels read;
    the single-sentence calls it is compared with read the rows."""
    S, L, n = len(lens), sum(lens), len(lens) * beam
    p = synth.cgru_step(seed=1, E=E, H=H, A=A, l=L, n_beam=n)
    m = oracle.OracleModel(p)
    w = q.CgruWeights(gpu_gru(q, ctx, p, "dec_r", tiled), gpu_mat(q, ctx, p["att.U"], tiled), ctx.f32(p["att.v"]),
                      gpu_gru(q, ctx, p, "dec_q", tiled))
    enc_h = ctx.f32(p["enc_h"])
    P = q.q8_gemm_narrow(ctx, gpu_mat(q, ctx, p["att.W"]), enc_h, ctx.f32(p["att.b"]))
    P_ref = m.attention_precompute(p["enc_h"])
    assert_same(P, P_ref, "P")
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    y, s0 = ctx.f32(p["y_emb"]), ctx.f32(p["s_prev"])
    r = q.cgru_decoder_step_batch_q8(ctx, w, P, enc_h, torch.tensor(off, device=ctx.device), beam, max(lens), y, s0)
    for si in range(S):
        lo, hi, sl = off[si], off[si + 1], slice(si * beam, (si + 1) * beam)
        # the single-sentence entry point on this sentence's slots: the same bits
        r1 = q.cgru_decoder_step_q8(ctx, w, P[lo:hi].contiguous(), enc_h[lo:hi].contiguous(), y[sl].contiguous(), s0[sl].contiguous())
        for key in ("s_mid", "ctx", "s"):
            assert_same(r[key][sl], np_(r1[key]), "sentence %d %s vs single-sentence call" % (si, key))
        assert_same(r["alpha"][sl, :hi - lo], np_(r1["alpha"]), "alpha")
        # and the oracle, free-running, on the sentence's first and last slot
        for j in (si * beam, (si + 1) * beam - 1):
            sm_o, al_o, cx_o, s_o = m.cgru_step(P_ref[lo:hi], p["enc_h"][lo:hi], p["y_emb"][j], p["s_prev"][j])
            assert_close(r["s_mid"][j], sm_o, "s'"); assert_close(r["alpha"][j, :hi - lo], al_o, "alpha")
            assert_close(r["ctx"][j], cx_o, "H_t"); assert_close(r["s"][j], s_o, "s")
    r2 = q.cgru_decoder_step_batch_q8(ctx, w, P, enc_h, torch.tensor(off, device=ctx.device), beam, max(lens), y, s0)
    assert_same(r2["s"], np_(r["s"]), "second call: arrival counters back at zero")


def _translate_all(q, ctx, m_gpu, m_ref, sents, beam, k, max_steps):
    got = q.q8_translate_batch(ctx, m_gpu, sents, beam=beam, k=k, max_steps=max_steps)
    finished = 0
    for src, (toks, score, steps) in zip(sents, got):
        r_toks, r_score, r_steps = m_ref.translate(src, beam=beam, topk=k, max_steps=max_steps)
        assert toks.tolist() == r_toks.tolist(), (src.tolist(), toks.tolist(), r_toks.tolist())
        assert abs(float(score) - float(r_score)) <= 1e-5 * max(1.0, abs(float(r_score)))
        assert steps == r_steps               # a finished sentence stops counting while the batch runs on
        t1, s1, st1 = q.q8_translate(ctx, m_gpu, src, beam=beam, k=k, max_steps=max_steps)
        assert t1.tolist() == toks.tolist() and np.float32(s1) == np.float32(score)
        finished += len(toks) < max_steps
    return finished


@pytest.mark.parametrize("H,A,lens,beam,tiled", [(1024, 1024, (9,), 1, True), (1024, 1024, (5, 3), 4, True), (1024, 1024, (5, 3), 3, False),
                                                 (768, 640, (4, 7, 2), 2, True), (768, 640, (4, 7), 4, False), (1000, 1000, (6, 2), 2, False)])
def test_batched_step_of_up_to_eight_slots(q, H, A, lens, beam, tiled):
    """Its products of rows of 513-1024 bytes run in the panel kernels: the states and contexts that cgru_decoder_step_q8 gives for
    each sentence, bit for bit."""
    E, rng = 512, np.random.default_rng(H + beam)
    p = synth.cgru_step(seed=beam, E=E, H=H, A=A, l=1, n_beam=1)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=16, max_rows=3 * H, max_ld=2048))
    gru = lambda pre: q.GruWeights(gpu_mat(q, ctx, p[pre + ".Wx"], tiled), gpu_mat(q, ctx, p[pre + ".Wh"], tiled), ctx.f32(p[pre + ".bx"]), ctx.f32(p[pre + ".bh"]))
    w = q.CgruWeights(gru("dec_r"), gpu_mat(q, ctx, p["att.U"], tiled), ctx.f32(p["att.v"]), gru("dec_q"))
    off, n = np.concatenate([[0], np.cumsum(lens)]), len(lens) * beam
    f = lambda *s: ctx.f32(rng.standard_normal(s).astype(np.float32))
    P, enc, y, s = f(int(off[-1]), A), f(int(off[-1]), 2 * H), f(n, E), torch.tanh(f(n, H))
    r = q.cgru_decoder_step_batch_q8(ctx, w, P, enc, torch.as_tensor(off.astype(np.int32)).cuda(), beam, max(lens), y, s)
    for i in range(len(lens)):
        rows, sl = slice(int(off[i]), int(off[i + 1])), slice(i * beam, (i + 1) * beam)
        one = q.cgru_decoder_step_q8(ctx, w, P[rows].contiguous(), enc[rows].contiguous(), y[sl].contiguous(), s[sl].contiguous())
        assert_same(r["s"][sl], np_(one["s"]), "s of sentence %d" % i)
        assert_same(r["ctx"][sl], np_(one["ctx"]), "context of sentence %d" % i)


@pytest.mark.parametrize("V,E,H,A,R,beam,k,S", [(13, 16, 24, 20, 12, 5, 6, 4), (50, 32, 48, 40, 24, 3, 5, 7),
                                                (200, 64, 64, 32, 48, 5, 12, 3), (40, 36, 40, 28, 20, 8, 12, 2),
                                                (13, 16, 24, 20, 12, 1, 4, 11)])
def test_translate_batch_small_models(q, ctx, oracle, V, E, H, A, R, beam, k, S):
    p = synth.full_model(seed=V + beam, V=V, E=E, H=H, A=A, R=R, w_std=0.3, b_std=0.1)
    p["out.b"][0] += 1.5                 # make the end token frequent enough to finish hypotheses
    m_ref, m_gpu = oracle.OracleModel(p), q.Model.from_params(ctx, p)
    rng = np.random.default_rng(V + S)
    sents = [rng.integers(1, V, size=int(rng.integers(1, 12))).astype(np.int32) for _ in range(S)]
    finished = _translate_all(q, ctx, m_gpu, m_ref, sents, beam, k, max_steps=15)
    assert finished > 0 or V > 100       # some searches ended early while others went on


def test_translate_batch_full_size_model(q, ctx, oracle):
    p = synth.full_model(seed=4)
    m_ref, m_gpu = oracle.OracleModel(p), q.Model.from_params(ctx, p)
    sents = synth.sentences(seed=4, n=4, V=50000, min_len=5, max_len=14)
    _translate_all(q, ctx, m_gpu, m_ref, sents, beam=5, k=12, max_steps=4)


@pytest.mark.parametrize("E,H,lens", [(512, 1024, (12, 1, 30, 7)), (36, 40, (5, 5, 9, 2, 1, 17)), (100, 60, (3,) * 12 + (40,)),
                                      (512, 1024, (20,))])
def test_encoder_batch(q, ctx, oracle, E, H, lens):
    L = sum(lens)
    p = synth.encoder(seed=3, l=L, E=E, H=H)
    fwd, bwd = gpu_gru(q, ctx, p, "enc_fwd"), gpu_gru(q, ctx, p, "enc_bwd")
    X = ctx.f32(p["X"])
    enc = q.q8_encode_batch(ctx, fwd, bwd, X, list(lens))
    gf = oracle.QGru(p["enc_fwd.Wx"], p["enc_fwd.Wh"], p["enc_fwd.bx"], p["enc_fwd.bh"])
    gb = oracle.QGru(p["enc_bwd.Wx"], p["enc_bwd.Wh"], p["enc_bwd.bx"], p["enc_bwd.bh"])
    o = 0
    for l in lens:
        one = q.q8_encode(ctx, fwd, bwd, X[o:o + l].contiguous())
        assert_same(enc[o:o + l], np_(one), "sentence at row %d vs q8_encode" % o)
        # the oracle's recurrences, free-running, on this sentence
        hf, hb = np.zeros(H, np.float32), np.zeros(H, np.float32)
        ref = np.zeros((l, 2 * H), np.float32)
        for i in range(l):
            hf = gf.step(p["X"][o + i], hf); ref[i, H:] = hf
        for i in range(l - 1, -1, -1):
            hb = gb.step(p["X"][o + i], hb); ref[i, :H] = hb
        assert_close(enc[o:o + l], ref, "sentence at row %d vs oracle" % o)
        o += l


def test_output_layer_panel_ties(q, ctx, oracle):
    """Heavily tied logits overflow the survivor list and take the exact fallback, with the logits
    in the caller's row-major buffer or tile by tile in the workspace.  Equals: lowest index first."""
    V, R, n = 2500, 32, 9
    W = np.zeros((V, R), np.float32); W[:, 0] = 1.0
    b = np.zeros(V, np.float32)
    b[[5, 130, 131, 400, 2499]] = 2.0
    t = np.zeros((n, R), np.float32); t[:, 0] = 0.5
    Wm = gpu_mat(q, ctx, W)
    L = oracle.QLinear(W, b)
    for want in (False, True):
        r = q.output_logits_q8(ctx, None, Wm, ctx.f32(b), t_in=ctx.f32(t), k=12, want_logits=want)
        for j in range(n):
            lse, lp, idx = oracle.logsoftmax_topk(L.gemv(t[j]), 12)
            assert idx[:5].tolist() == [5, 130, 131, 400, 2499] and idx[5:].tolist() == list(range(0, 5)) + [6, 7]
            assert_same(r["topk_idx"][j], idx); assert_close(r["topk_logp"][j], lp)


@pytest.mark.parametrize("V,R,n,k", [(50000, 512, 20, 12), (3001, 512, 300, 12), (2000, 620, 250, 5), (777, 512, 9, 16),
                                     (5000, 640, 1000, 12), (100, 512, 12, 12), (3001, 512, 40, 1), (16, 512, 9, 16),
                                     (4097, 640, 161, 7)])
def test_output_layer_panel_persistent_kernel(q, ctx, oracle, V, R, n, k):
    """Tile-packed vocabulary matrix and no logits requested: the panel kernel that keeps the slots'
    codes in LDS and streams weight tiles (rows of 512 or 640 bytes)."""
    p = synth.output_layer(seed=2, V=V, R=R, n_beam=n)
    L = oracle.QLinear(p["out.W"], p["out.b"])
    W = q.q8_pack_tiles(ctx, q.q8_quantize_matrix(ctx, p["out.W"], ld_out=(R + 63) // 64 * 64))
    t = ctx.f32(p["t"])
    r = q.output_logits_q8(ctx, None, W, ctx.f32(p["out.b"]), t_in=t, k=k, want_logits=False)
    full = q.output_logits_q8(ctx, None, W, ctx.f32(p["out.b"]), t_in=t, k=k)          # stored logits: block kernel
    assert_same(r["topk_idx"], np_(full["topk_idx"]), "panel kernel vs block kernel: top-k")
    assert_same(r["topk_logp"], np_(full["topk_logp"])); assert_same(r["lse"], np_(full["lse"]))
    for j in sorted(set([0, n // 3, n - 1])):
        lse, lp, idx = oracle.logsoftmax_topk(L.gemv(p["t"][j]), k)
        assert_same(r["topk_idx"][j], idx, "top-k indices"); assert_close(r["topk_logp"][j], lp, "top-k logp")
        assert_close(r["lse"][j:j + 1], np.array([lse]), "lse")


def test_output_layer_panel_persistent_kernel_ties(q, ctx, oracle):
    """The panel path keeps no logits and computes those of the qualifying tiles a second time.  With
    nearly all logits equal every tile qualifies and the survivors overflow their list: the exact
    fallback (k rounds over all tiles) has to give the raised entries first, then the lowest indices."""
    V, R, n = 4100, 512, 11
    W = np.zeros((V, R), np.float32); W[:, 0] = 1.0
    b = np.zeros(V, np.float32)
    raised = [7, 130, 131, 2047, 4099]
    b[raised] = 2.0
    t = np.zeros((n, R), np.float32); t[:, 0] = 0.5
    Wm = q.q8_pack_tiles(ctx, q.q8_quantize_matrix(ctx, W, ld_out=512))
    L = oracle.QLinear(W, b)
    r = q.output_logits_q8(ctx, None, Wm, ctx.f32(b), t_in=ctx.f32(t), k=12, want_logits=False)
    for j in range(n):
        lse, lp, idx = oracle.logsoftmax_topk(L.gemv(t[j]), 12)
        assert idx.tolist() == raised + [0, 1, 2, 3, 4, 5, 6]
        assert_same(r["topk_idx"][j], idx); assert_close(r["topk_logp"][j], lp)
        assert_close(r["lse"][j:j + 1], np.array([lse]), "lse")


@pytest.mark.parametrize("dims,S,beam,l", [(dict(), 4, 5, 7), (dict(), 30, 5, 30), (dict(), 3, 3, 5),
                                           (dict(V=33658, E=620, H=1000, A=1000, R=620), 4, 5, 9),
                                           (dict(V=50, E=32, H=48, A=40, R=24, w_std=0.3), 6, 2, 5)])
def test_codes_travel_from_the_batched_step_to_the_output_layer(q, ctx, oracle, dims, S, beam, l):
    """cgru_decoder_step_batch_codes_q8 + output_logits_codes_q8 against the plain calls (identical bits);
    the three sets of codes against the oracle's quantization of the fp32 vectors they belong to."""
    p = synth.full_model(seed=12, **dims)
    m = q.Model.from_params(ctx, p)
    E, H = m.E_tgt.shape[1], m.dec.r.H
    n = S * beam
    rng = np.random.default_rng(S + l)
    enc_h = ctx.f32(rng.standard_normal((S * l, 2 * H)).astype(np.float32))
    P = q.q8_gemm_narrow(ctx, m.att_W, enc_h, m.att_b)
    off = torch.arange(0, (S + 1) * l, l, dtype=torch.int32, device=ctx.device)
    y = ctx.f32(rng.standard_normal((n, E)).astype(np.float32))
    s = ctx.f32(rng.standard_normal((n, H)).astype(np.float32))
    res = []
    for use in (False, True):
        codes = (q.Codes(ctx, n, m.dec.r.Wx.ld), q.Codes(ctx, n, m.dec.q.Wx.ld), q.Codes(ctx, n, m.ro.W_s.ld)) if use else None
        r1 = q.cgru_decoder_step_batch_q8(ctx, m.dec, P, enc_h, off, beam, l, y, s, codes=codes)
        if use:
            assert all(c.valid for c in codes)
            for c, X in ((codes[0], y), (codes[1], r1["ctx"]), (codes[2], r1["s"])):
                for j in (0, n // 2, n - 1):
                    xq, xs = oracle.quantize(np_(X)[j])
                    K = X.shape[1]
                    assert_same(c.q[j, :K], xq, "codes of slot %d" % j)
                    assert not np_(c.q[j, K:]).any() and float(c.scale[j]) == float(xs)
        r2 = q.output_logits_q8(ctx, m.ro, m.W_out, m.b_out, s=r1["s"], y_emb=y, ctx_vec=r1["ctx"], k=12, codes=codes)
        res.append((r1["s"], r1["ctx"], r2["t"], r2["logits"], r2["lse"], r2["topk_logp"], r2["topk_idx"]))
    for a, b, what in zip(res[0], res[1], ("s", "ctx", "t", "logits", "lse", "topk_logp", "topk_idx")):
        assert_same(b, np_(a), what + ": with codes against without")


@pytest.mark.parametrize("dims,S,beam,l", [(dict(), 6, 5, 9), (dict(V=500, E=64, H=128, A=64, R=64, w_std=0.2, b_std=0.1), 20, 3, 5),
                                           (dict(V=700, E=620, H=1000, A=1000, R=620, w_std=0.2, b_std=0.1), 3, 5, 6)])
def test_codes_handed_from_the_batched_search_step_to_the_next_step(q, ctx, oracle, dims, S, beam, l):
    """A batched decoding loop in which q8_beam_update_batch_loop gathers the codes of the rows it gathers and
    cgru_decoder_step_batch_loop_q8 takes them in place of its quantization launch, against the loop that
    quantizes again: every state, context vector, top-k table and gathered row bit for bit at every step; the
    handed codes against the oracle's quantization of the rows.  At 620 / 1000 the gather has no room for them."""
    T = 6
    p = synth.full_model(seed=41, **dims)
    m = q.Model.from_params(ctx, p)
    E, H = m.E_tgt.shape[1], m.dec.r.H
    n = S * beam
    rng = np.random.default_rng(S + l)
    enc_h = ctx.f32(rng.standard_normal((S * l, 2 * H)).astype(np.float32))
    P = q.q8_gemm_narrow(ctx, m.att_W, enc_h, m.att_b)
    off = torch.arange(0, (S + 1) * l, l, dtype=torch.int32, device=ctx.device)

    def loop(hand_on):
        states = torch.zeros(q.q8_beam_state_bytes(T) * S, dtype=torch.uint8, device=ctx.device)
        y, s = ctx.empty(n, E), ctx.empty(n, H)
        done = torch.zeros(S, dtype=torch.int32, device=ctx.device)
        q.q8_beam_init_batch(ctx, states, S, beam, T, enc_h, off, m.E_tgt, y, s, done)
        codes = [q.Codes(ctx, n, m.dec.r.Wx.ld), q.Codes(ctx, n, m.dec.q.Wx.ld), q.Codes(ctx, n, m.ro.W_s.ld)]
        if hand_on:
            codes.append(q.Codes(ctx, n, m.dec.r.Wh.ld))
        trace, used = [], 0
        for _ in range(T):
            given = hand_on and codes[0].c.valid == 2 and codes[3].c.valid == 2
            used += bool(given)
            if given:
                trace += [np_(codes[0].q), np_(codes[0].scale), np_(codes[3].q), np_(codes[3].scale)]
            r = q.cgru_decoder_step_batch_q8(ctx, m.dec, P, enc_h, off, beam, l, y, s, codes=codes)
            o = q.output_logits_q8(ctx, m.ro, m.W_out, m.b_out, s=r["s"], y_emb=y, ctx_vec=r["ctx"], k=8, want_logits=False,
                                   codes=codes[:3])
            q.q8_beam_update_batch(ctx, states, S, beam, T, o["topk_logp"], o["topk_idx"], r["s"], m.E_tgt, y, s, done,
                                   codes=(codes[2], codes[0], codes[3]) if hand_on else None,
                                   E_codes=m.E_tgt_codes if hand_on else None)
            trace += [np_(r["s"]), np_(r["ctx"]), np_(o["topk_logp"]), np_(o["topk_idx"]), np_(y), np_(s)]
        return trace, used, q.q8_beam_result_batch(ctx, states, S, T)

    ref, _, ref_res = loop(False)
    got, used, got_res = loop(True)
    fits = E // 4 + m.dec.r.Wx.ld // 16 + m.ro.W_s.ld // 16 <= 256
    assert used == (T - 1 if fits else 0)
    gi = iter(got)
    for step in range(T):
        if fits and step > 0:
            yq, ys, sq, ss = next(gi), next(gi), next(gi), next(gi)
            y_rows, s_rows = ref[6 * (step - 1) + 4], ref[6 * (step - 1) + 5]
            for j in (0, n // 2, n - 1):
                cq, cs = oracle.quantize(y_rows[j])
                assert_same(yq[j, :E], cq, "codes of y"); assert_same(ys[j:j + 1], np.array([cs], np.float32), "scale of y")
                cq, cs = oracle.quantize(s_rows[j])
                assert_same(sq[j, :H], cq, "codes of s"); assert_same(ss[j:j + 1], np.array([cs], np.float32), "scale of s")
                assert not yq[j, E:].any() and not sq[j, H:].any()
        for i in range(6):
            assert_same(next(gi), ref[6 * step + i], "step %d, output %d" % (step, i))
    for a, b in zip(got_res, ref_res):
        assert a[0].tolist() == b[0].tolist() and a[1:] == b[1:]


def _batched_step_with_codes(q, ctx, m, P, enc_h, off, beam, l, y, s):
    n = y.shape[0]
    codes = (q.Codes(ctx, n, m.dec.r.Wx.ld), q.Codes(ctx, n, m.dec.q.Wx.ld), q.Codes(ctx, n, m.ro.W_s.ld))
    r = q.cgru_decoder_step_batch_q8(ctx, m.dec, P, enc_h, off, beam, l, y, s, codes=codes)
    return {"s_mid": np_(r["s_mid"]), "s": np_(r["s"]), "ctx": np_(r["ctx"]), "alpha": np_(r["alpha"]),
            "sq": np_(codes[2].q), "ss": np_(codes[2].scale), "cq": np_(codes[1].q), "cs": np_(codes[1].scale)}


def _panel_case(q, ctx, S, beam, l, seed=31):
    p = synth.full_model(seed=seed)
    m = q.Model.from_params(ctx, p)
    E, H = m.E_tgt.shape[1], m.dec.r.H
    n = S * beam
    rng = np.random.default_rng(S + l)
    enc_h = ctx.f32(rng.standard_normal((S * l, 2 * H)).astype(np.float32))
    P = q.q8_gemm_narrow(ctx, m.att_W, enc_h, m.att_b)
    off = torch.arange(0, (S + 1) * l, l, dtype=torch.int32, device=ctx.device)
    y = ctx.f32(rng.standard_normal((n, E)).astype(np.float32))
    s = ctx.f32((rng.standard_normal((n, H)) * rng.uniform(0.05, 3.0, (n, 1))).astype(np.float32))
    return m, P, enc_h, off, y, s


@pytest.mark.parametrize("S,beam,l", [(2, 5, 6), (64, 5, 12), (67, 5, 4), (12, 8, 9), (70, 5, 3)])
def test_panel_gru_in_one_launch_equals_products_and_gates_apart(q, ctx, oracle, S, beam, l):
    """The transitions of a batched step as one kernel each, whose blocks exchange their partial maxima for the
    codes of the new states (the default where the grid fits the device: up to 336 slots), against the same
    step with that form switched off (matrix-core products, then a gates kernel): the same bits, states and
    codes.  From 340000 states on (67 and 70 sentences x 5 slots) the second form is the launch in tiles, past the limit either way."""
    m, P, enc_h, off, y, s = _panel_case(q, ctx, S, beam, l)
    one = _batched_step_with_codes(q, ctx, m, P, enc_h, off, beam, l, y, s)
    again = _batched_step_with_codes(q, ctx, m, P, enc_h, off, beam, l, y, s)
    try:
        q.q8_attention_options(ctx, exchange=False)
        apart = _batched_step_with_codes(q, ctx, m, P, enc_h, off, beam, l, y, s)
    finally:
        q.q8_attention_options(ctx, exchange=True)
    q.q8_encode_check(ctx)
    for key in one:
        assert_same(one[key], apart[key], key + ": one launch against products and gates apart")
        assert_same(again[key], one[key], key + ": second call (exchange words cleared by the launch between)")
    j = one["s"].shape[0] - 1
    sq, ss = oracle.quantize(one["s"][j])
    assert_same(one["sq"][j, :sq.shape[0]], sq, "codes of the last slot's new state")
    assert float(one["ss"][j]) == float(ss)


def test_panel_gru_wait_that_gives_up_is_reported_and_the_next_step_is_good(q, ctx, oracle):
    """With a bound of one poll a block of the one-launch panel GRU gives up at once: the kernel still ends,
    q8_encode_check reports it once and clears the exchange words, and the next step with the default bound
    gives the first one's bits again."""
    m, P, enc_h, off, y, s = _panel_case(q, ctx, 40, 5, 5)
    good = _batched_step_with_codes(q, ctx, m, P, enc_h, off, 5, 5, y, s)
    q.q8_encode_check(ctx)
    try:
        q.q8_attention_options(ctx, exchange=True, spin_limit=1)
        _batched_step_with_codes(q, ctx, m, P, enc_h, off, 5, 5, y, s)
        with pytest.raises(q.Q8Error):
            q.q8_encode_check(ctx)
    finally:
        q.q8_attention_options(ctx, exchange=True, spin_limit=0)
    q.q8_encode_check(ctx)
    again = _batched_step_with_codes(q, ctx, m, P, enc_h, off, 5, 5, y, s)
    q.q8_encode_check(ctx)
    for key in good:
        assert_same(again[key], good[key], key + " after the abandoned run")


def _batched_search(q, ctx, m, P, enc_h, off, S, beam, l, T, fused, hand_on, k=8):
    """T steps of a batched search from its start; fused: output_logits_beam_batch_q8, else the output layer and
    q8_beam_update_batch apart.  Returns every step's states, contexts, top-k tables and gathered rows, and the result."""
    E, H = m.E_tgt.shape[1], m.dec.r.H
    n = S * beam
    states = torch.zeros(q.q8_beam_state_bytes(T) * S, dtype=torch.uint8, device=ctx.device)
    y, s = ctx.empty(n, E), ctx.empty(n, H)
    done = torch.zeros(S, dtype=torch.int32, device=ctx.device)
    q.q8_beam_init_batch(ctx, states, S, beam, T, enc_h, off, m.E_tgt, y, s, done)
    codes = [q.Codes(ctx, n, m.dec.r.Wx.ld), q.Codes(ctx, n, m.dec.q.Wx.ld), q.Codes(ctx, n, m.ro.W_s.ld)]
    if hand_on:
        codes.append(q.Codes(ctx, n, m.dec.r.Wh.ld))
    trace, used = [], 0
    for _ in range(T):
        used += bool(hand_on and codes[0].c.valid == 2 and codes[3].c.valid == 2)
        r = q.cgru_decoder_step_batch_q8(ctx, m.dec, P, enc_h, off, beam, l, y, s, codes=codes)
        if fused:
            o = q.output_logits_beam_batch_q8(ctx, m.ro, m.W_out, m.b_out, r["s"], y, r["ctx"], states, S, beam, T, m.E_tgt, s,
                                              done, k=k, codes=(codes[2], codes[0], codes[1]),
                                              s_next_codes=codes[3] if hand_on else None,
                                              E_codes=m.E_tgt_codes if hand_on else None)
        else:
            o = q.output_logits_q8(ctx, m.ro, m.W_out, m.b_out, s=r["s"], y_emb=y, ctx_vec=r["ctx"], k=k, want_logits=False,
                                   codes=codes[:3])
            q.q8_beam_update_batch(ctx, states, S, beam, T, o["topk_logp"], o["topk_idx"], r["s"], m.E_tgt, y, s, done,
                                   codes=(codes[2], codes[0], codes[3]) if hand_on else None,
                                   E_codes=m.E_tgt_codes if hand_on else None)
        trace += [np_(r["s"]), np_(r["ctx"]), np_(o["topk_logp"]), np_(o["topk_idx"]), np_(y), np_(s), np_(done)]
    return trace, used, q.q8_beam_result_batch(ctx, states, S, T)


@pytest.mark.parametrize("dims,S,beam,l,k,hand_on", [
    (dict(), 6, 5, 9, 12, True), (dict(), 64, 5, 7, 12, True), (dict(), 200, 5, 3, 12, True), (dict(), 2, 8, 5, 16, False),
    (dict(), 40, 1, 4, 3, True), (dict(V=700, E=620, H=1000, A=1000, R=620, w_std=0.2, b_std=0.1), 3, 5, 6, 8, True),
    (dict(V=500, E=64, H=128, A=64, R=64, w_std=0.2, b_std=0.1), 20, 3, 5, 8, True), (dict(), 1, 5, 6, 12, False)])
def test_search_steps_inside_the_panel_selection(q, ctx, oracle, dims, S, beam, l, k, hand_on):
    """output_logits_beam_batch_q8 (the sentences' search steps run in the selection kernel's launch where the
    vocabulary matrix is tile-packed with rows of 512 or 640 bytes and there are more than 8 slots; the other
    shapes here take its two-call path) against output layer and q8_beam_update_batch apart: every state,
    context vector, top-k table, gathered row and done flag bit for bit at every step, the same results, and
    as many steps that took their codes from the search step."""
    T = 5
    p = synth.full_model(seed=43, **dims)
    m = q.Model.from_params(ctx, p)
    H = m.dec.r.H
    rng = np.random.default_rng(S + l)
    enc_h = ctx.f32(rng.standard_normal((S * l, 2 * H)).astype(np.float32))
    P = torch.cat([q.q8_gemm_narrow(ctx, m.att_W, enc_h[o:o + 1000].contiguous(), m.att_b) for o in range(0, S * l, 1000)])
    off = torch.arange(0, (S + 1) * l, l, dtype=torch.int32, device=ctx.device)
    ref, ref_used, ref_res = _batched_search(q, ctx, m, P, enc_h, off, S, beam, l, T, False, hand_on, k)
    for rep in range(2):                              # (the second run finds the exchange words as the first left them)
        got, used, got_res = _batched_search(q, ctx, m, P, enc_h, off, S, beam, l, T, True, hand_on, k)
        q.q8_encode_check(ctx)
        assert used == ref_used
        for i, (a, b) in enumerate(zip(got, ref)):
            assert_same(a, b, "run %d, step %d, output %d" % (rep, i // 7, i % 7))
        for a, b in zip(got_res, ref_res):
            assert a[0].tolist() == b[0].tolist() and a[1:] == b[1:]


def test_panel_search_wait_that_gives_up_is_reported_and_the_next_search_is_good(q, ctx, oracle):
    """With a bound of one poll the block that runs a sentence's search step inside the panel selection may stop
    waiting for the sentence's other slots: the kernel still ends normally, q8_encode_check reports it once and
    clears the exchange words, and the same search run again gives the first result."""
    S, beam, l, T = 12, 5, 4, 4
    m = q.Model.from_params(ctx, synth.full_model(seed=43))
    rng = np.random.default_rng(5)
    enc_h = ctx.f32(rng.standard_normal((S * l, 2 * m.dec.r.H)).astype(np.float32))
    P = q.q8_gemm_narrow(ctx, m.att_W, enc_h, m.att_b)
    off = torch.arange(0, (S + 1) * l, l, dtype=torch.int32, device=ctx.device)
    good = _batched_search(q, ctx, m, P, enc_h, off, S, beam, l, T, True, True)
    q.q8_encode_check(ctx)
    gave_up = False
    try:
        q.q8_attention_options(ctx, exchange=True, spin_limit=1)
        for _ in range(5):                            # (a single poll can succeed when the other blocks are quick)
            _batched_search(q, ctx, m, P, enc_h, off, S, beam, l, T, True, True)
            try:
                q.q8_encode_check(ctx)
            except q.Q8Error:
                gave_up = True
                break
    finally:
        q.q8_attention_options(ctx, exchange=True, spin_limit=0)
    assert gave_up
    q.q8_encode_check(ctx)
    again = _batched_search(q, ctx, m, P, enc_h, off, S, beam, l, T, True, True)
    q.q8_encode_check(ctx)
    for a, b in zip(again[0], good[0]):
        assert_same(a, b, "after the abandoned run")
    for a, b in zip(again[2], good[2]):
        assert a[0].tolist() == b[0].tolist() and a[1:] == b[1:]


@pytest.mark.parametrize("beam,A,lens", [
    (2, 4, [1, 7, 3, 2, 9]), (3, 28, [5, 40, 1, 1, 2]), (8, 64, [18, 33, 4]), (5, 256, [70] * 50),                # 32 lanes per position
    (3, 768, [9, 8, 33]), (1, 512, [33] * 12),                                                                   # the same: few positions, beam 1
    (1, 1000, [1, 60, 7] * 9), (1, 1028, [1] * 40), (1, 772, [3, 1, 90] * 4),                                    # a wave per position
    (2, 260, [64] * 50), (5, 512, [60, 66, 64, 3] * 16), (8, 516, [130, 1, 128] * 12),                           # two and four waves
    (4, 1000, [33, 17, 16]), (5, 1028, [1] * 40), (5, 1024, [60, 3, 31, 17]), (6, 2052, [9, 8]), (7, 1024, [130, 2])])
def test_energies_of_a_batch(q, ctx, beam, A, lens):
    """The batched energies by each of their kernels against the definition in 64 bits and against the step of one
    sentence: small arguments, ones that cancel, and entries of P and a beyond the range of the form whose tanh is put
    together from e^{2P} and e^{2a} (there a wave takes one tanh per entry).  An energy is a sum in double rounded once:
    an attention weight is off by twice half a last place of the largest energy and half of its own.  The other kernel
    adds the same floats but for one in some millions in another order, in double: its weights are the same bits but
    where a sum lies that close to a tie, so in all but a few of them (leaving out what the sum P + a lost in rounding,
    or taking an energy's sum in float, changes a third)."""
    E = H = 36
    p = synth.cgru_step(seed=beam, E=E, H=H, A=A, l=1, n_beam=len(lens) * beam)
    rng = np.random.default_rng(A + beam)
    L, n = sum(lens), len(lens) * beam
    P = rng.standard_normal((L, A)).astype(np.float32)
    P[::3] *= 1e-4
    P[1::7, : max(1, A // 5)] *= 60.0                         # some beyond 44
    P[L // 2, 0], P[L - 1, A - 1] = 3e4, -2e30
    big = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=max(lens), max_rows=max(A, 3 * H), max_ld=128))
    enc = big.f32(rng.standard_normal((L, 2 * H)).astype(np.float32))
    p["att.v"] = (rng.standard_normal(A) * 2.0 / np.sqrt(A)).astype(np.float32)
    off = np.array([0] + list(np.cumsum(lens)))
    total = differ = 0
    for gain in (0.05, 400.0):                                # u's weights: small and large a
        U = gpu_mat(q, big, p["att.U"] * np.float32(gain), False)
        gru = lambda pre: gpu_gru(q, big, p, pre)
        w = q.CgruWeights(gru("dec_r"), U, big.f32(p["att.v"]), gru("dec_q"))
        Pd, y, s_prev = big.f32(P), big.f32(p["y_emb"]), big.f32(p["s_prev"])
        r = q.cgru_decoder_step_batch_q8(big, w, Pd, enc, torch.as_tensor(off.astype(np.int32)).to(big.device), beam, max(lens), y, s_prev)
        a = np.concatenate([np_(q.q8_gemm_narrow(big, U, r["s_mid"][j:j + 512].contiguous())) for j in range(0, n, 512)])
        if gain > 1:
            assert np.abs(a).max() > 44
        v = p["att.v"].astype(np.float64)
        for s in sorted({0, 1, 2, len(lens) // 2, len(lens) - 2, len(lens) - 1} & set(range(len(lens)))):
            rows, sl, l = slice(int(off[s]), int(off[s + 1])), slice(s * beam, (s + 1) * beam), lens[s]
            one = np_(q.cgru_decoder_step_q8(big, w, Pd[rows].contiguous(), enc[rows].contiguous(), y[sl].contiguous(), s_prev[sl].contiguous())["alpha"])
            got = np_(r["alpha"][sl, :l])
            total, differ = total + got.size, differ + int((got != one).sum())
            for b in range(beam):
                x = (P[rows] + a[s * beam + b]).astype(np.float32).astype(np.float64)
                e = np.tanh(x) @ v
                al = np.exp(e - e.max()) / np.exp(e - e.max()).sum()
                tol = 2.0 ** -23 * np.abs(e).max() + 2.0 ** -24 + 1e-9
                assert (np.abs(got[b] - al) <= tol * al + 2e-45).all(), "alpha of slot %d" % (s * beam + b)
    assert differ <= 0.02 * total, (differ, total)


@pytest.mark.parametrize("E,H,lens,tiled", [(36, 4, [3, 1], False), (64, 64, [2] * 9 + [5], True), (620, 1000, [4, 9, 1], False), (64, 256, [1, 2, 3] * 6, True),
                                            (48, 96, [3, 1, 4] * 22, False), (48, 100, [2, 1] * 65, False),
                                            # 32 and 64 slots per block, two rounds of blocks, three launches per position instead
                                            (16, 100, [1, 2, 2] * 190, False), (32, 1000, [2, 1, 3] * 33, False), (32, 1024, [1, 3] * 97, True),
                                            (64, 512, [2, 1] * 200, True), (32, 1024, [2, 1] * 200, True), (32, 1024, [1, 3] * 130, True)])
def test_encoder_step_in_one_launch(q, oracle, E, H, lens, tiled):
    """The batched encoder's launches per position (one_launch = 0) at the edges of their blocks (32 units, 16 / 32 / 64 slots,
    one slot group and more), sentences that end at different steps: the states of q8_encode, which runs another kernel per
    position, and of the batch in one launch, bit for bit; with the workspace that q8_encode_batch_bytes asks for, and no
    more than it."""
    rng = np.random.default_rng(H + len(lens))
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=len(lens) + (k == "b"), I=E, H=H).items()}
    big = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=64, max_rows=3 * H, max_ld=1024))
    G = [q.GruWeights(gpu_mat(q, big, p[k + "Wx"], False), gpu_mat(q, big, p[k + "Wh"], tiled), big.f32(p[k + "bx"]), big.f32(p[k + "bh"]))
         for k in ("f", "b")]
    L = sum(lens)
    X = big.f32(rng.standard_normal((L, E)).astype(np.float32))
    from paper_1804_05038_amd import binding
    header = 256 * 1024
    ctx = q.Context(workspace_bytes=header + binding.q8_encode_batch_bytes(G[0], L, len(lens)))
    q.q8_encoder_options(ctx, False)
    for _ in range(2):
        enc = q.q8_encode_batch(ctx, G[0], G[1], X, list(lens))
    q.q8_encoder_options(ctx, True)
    assert_same(q.q8_encode_batch(ctx, G[0], G[1], X, list(lens)), np_(enc), "in one launch")
    q.q8_encoder_options(big, False)
    off = [0] + list(np.cumsum(lens))
    for i in sorted({*range(min(12, len(lens))), *range(max(0, len(lens) - 3), len(lens))}):
        rows = slice(int(off[i]), int(off[i + 1]))
        assert_same(enc[rows], np_(q.q8_encode(big, G[0], G[1], X[rows].contiguous())), "sentence %d" % i)


@pytest.mark.parametrize("H,lens,launches", [(64, [3, 5, 2], 1), (64, [2, 1], 2), (64, [1] * 20, 1), (512, [6] * 385, 6), (512, [7] * 385, 1),
                                             (1024, [3] * 512, 1), (1024, [3] * 513, 3)])
def test_encoder_options_choose_the_launches_of_a_batch(q, H, lens, launches):
    """One launch where it pays, else one of this kind per position; one_launch = 0 takes the kernel whose blocks wait for each
    other out of q8_encode_batch as out of q8_encode.  The same states."""
    E, x = 16, np.random.default_rng(0)
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=k == "b", I=E, H=H).items()}
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=64, max_rows=3 * H, max_ld=1024))
    G = [q.GruWeights(gpu_mat(q, ctx, p[k + "Wx"]), gpu_mat(q, ctx, p[k + "Wh"]), ctx.f32(p[k + "bx"]), ctx.f32(p[k + "bh"])) for k in ("f", "b")]
    ctx = q.Context(workspace_bytes=256 * 1024 + q.q8_encode_batch_bytes(G[0], sum(lens), len(lens)))
    X = ctx.f32(x.standard_normal((sum(lens), E)).astype(np.float32))
    enc = []
    for one_launch in (True, False):
        q.q8_encoder_options(ctx, one_launch)
        q.q8_profile_begin(ctx, "gru", 16)
        enc.append(np_(q.q8_encode_batch(ctx, G[0], G[1], X, lens)))
        assert q.q8_profile_end(ctx)[1] == (launches if one_launch else max(lens))
    assert_same(enc[0], enc[1], "one_launch = 0")


@pytest.mark.parametrize("E,H,ld,lens", [(16, 1028, None, [3, 1, 5, 2, 4, 1, 2]), (16, 1028, None, [2, 1, 3, 1, 2, 1, 4, 2]), (16, 1028, None, [1, 4, 2] * 3),
                                         (16, 1056, None, [2, 3] * 35), (20, 64, 1040, [2, 1, 3]), (20, 64, 1040, [1, 2, 3] * 6)])
def test_encoder_of_a_batch_in_three_launches_per_position(q, E, H, ld, lens):
    """What neither launch takes (more than 1024 hidden units, rows of W_h of more than 1024 bytes): codes, products and gates
    per position, at 7, 8, 9 and more sentences (products of up to 8 vectors are other kernels'), against q8_encode bit for
    bit."""
    rng = np.random.default_rng(H + len(lens))
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=len(lens) + (k == "b"), I=E, H=H).items()}
    big = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=64, max_rows=3 * H, max_ld=1088))
    G = [q.GruWeights(gpu_mat(q, big, p[k + "Wx"]), q.q8_quantize_matrix(big, p[k + "Wh"], ld), big.f32(p[k + "bx"]), big.f32(p[k + "bh"]))
         for k in ("f", "b")]
    off = np.concatenate([[0], np.cumsum(lens)])
    X = big.f32(rng.standard_normal((int(off[-1]), E)).astype(np.float32))
    ctx = q.Context(workspace_bytes=256 * 1024 + q.q8_encode_batch_bytes(G[0], int(off[-1]), len(lens)))
    for one_launch in (True, False):
        q.q8_encoder_options(ctx, one_launch)
        enc = q.q8_encode_batch(ctx, G[0], G[1], X, list(lens))
        for i in range(len(lens)):
            rows = slice(int(off[i]), int(off[i + 1]))
            assert_same(enc[rows], np_(q.q8_encode(big, G[0], G[1], X[rows].contiguous())), "sentence %d" % i)


@pytest.mark.parametrize("E,H,lens,tiled", [(16, 36, [5, 1, 9], False), (16, 4, [3] * 129, False), (32, 1024, [4] * 64 + [7], True),
                                            (32, 1000, [1, 6, 2] * 23, False), (16, 100, [3, 2] * 70, False), (16, 256, [2, 7, 3] * 340, True)])
def test_encoder_of_a_batch_whatever_its_blocks_wait_for(q, oracle, E, H, lens, tiled):
    """The recurrences in one launch at the edges of their sets and groups (one sentence per set, 16 and 17 of them, several
    groups, units and rows past H), with room for their words only: q8_encode's states, bit for bit; and the same with a
    bound of one poll, where members leave and the last of each set works it off by itself.  Neither reports a wait."""
    rng = np.random.default_rng(H + len(lens))
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=len(lens) + (k == "b"), I=E, H=H).items()}
    big = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=64, max_rows=3 * H, max_ld=1024))
    G = [q.GruWeights(gpu_mat(q, big, p[k + "Wx"], False), gpu_mat(q, big, p[k + "Wh"], tiled), big.f32(p[k + "bx"]), big.f32(p[k + "bh"]))
         for k in ("f", "b")]
    L = sum(lens)
    X = big.f32(rng.standard_normal((L, E)).astype(np.float32))
    ctx = q.Context(workspace_bytes=256 * 1024 + q.q8_encode_batch_bytes(G[0], L, len(lens)))
    enc = np_(q.q8_encode_batch(ctx, G[0], G[1], X, list(lens)))
    off = [0] + list(np.cumsum(lens))
    for i in sorted({*range(min(20, len(lens))), *range(max(0, len(lens) - 5), len(lens))}):
        rows = slice(int(off[i]), int(off[i + 1]))
        assert_same(enc[rows], np_(q.q8_encode(big, G[0], G[1], X[rows].contiguous())), "sentence %d" % i)
    q.q8_encoder_options(ctx, True, 1)
    assert_same(q.q8_encode_batch(ctx, G[0], G[1], X, list(lens)), enc, "a bound of one poll")
    q.q8_encode_check(ctx)


@pytest.mark.parametrize("E,H,lens,tiled", [(512, 1024, [1, 9, 4] * 21 + [3], True), (516, 1000, [7, 2, 3], False), (620, 1000, [3] * 17, False),
                                            (640, 1024, [5, 4] * 30, True), (640, 36, [4] * 40, False), (644, 1024, [2, 6, 3] * 20, False),
                                            (1000, 100, [3, 4, 8], False), (4, 4, [3], False)])
def test_encoder_of_a_batch_multiplies_its_rows(q, E, H, lens, tiled):
    """Rows of X of all widths up to the 640 bytes that the recurrences' launch multiplies itself, and past them: q8_encode's states,
    bit for bit, with a bound of one poll as well, and with an infinity in a row of X (whose states are numbers all the same)."""
    rng = np.random.default_rng(E + H)
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=E + (k == "b"), I=E, H=H).items()}
    big = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=64, max_rows=3 * H, max_ld=1024))
    G = [q.GruWeights(gpu_mat(q, big, p[k + "Wx"], tiled and E % 64 == 0), gpu_mat(q, big, p[k + "Wh"], tiled), big.f32(p[k + "bx"]),
                      big.f32(p[k + "bh"]) if k == "f" else None) for k in ("f", "b")]
    L, off = sum(lens), [0] + list(np.cumsum(lens))
    X = rng.standard_normal((L, E)).astype(np.float32)
    ctx = q.Context(workspace_bytes=256 * 1024 + q.q8_encode_batch_bytes(G[0], L, len(lens)))
    for bad in (None, np.inf):
        if bad is not None:
            X[off[1] - 1, E // 2] = bad
        Xd = big.f32(X)
        enc = np_(q.q8_encode_batch(ctx, G[0], G[1], Xd, list(lens)))
        for i in sorted({0, 1 % len(lens), len(lens) // 2, len(lens) - 1}):
            rows = slice(int(off[i]), int(off[i + 1]))
            np.testing.assert_array_equal(enc[rows], np_(q.q8_encode(big, G[0], G[1], Xd[rows].contiguous())), "sentence %d" % i)
    assert np.abs(enc).max() <= 1
    q.q8_encoder_options(ctx, True, 1)
    np.testing.assert_array_equal(np_(q.q8_encode_batch(ctx, G[0], G[1], Xd, list(lens))), enc, "a bound of one poll")
    q.q8_encode_check(ctx)


# inputs, units, vectors, tile-packed, tiles of 32 vectors per block of gru_tile_kernel (checked against the library's rule on the host; 0: the
# kernel whose rows are 512 + 1024 bytes has this one where no codes are wanted)
TILE_GRUS = [(64, 64, 9, True, 1), (16, 36, 33, False, 1), (100, 4, 700, False, 1), (620, 1000, 129, False, 1), (2000, 1000, 353, False, 2),
             (512, 1024, 1000, True, 0), (2048, 1024, 513, True, 3), (1024, 48, 300, False, 1), (512, 2048, 300, True, 3), (256, 512, 1024, True, 2),
             (516, 1000, 801, False, 4), (640, 1024, 1024, True, 4)]


@pytest.mark.parametrize("I,H,n,tiled,columns", TILE_GRUS)
def test_panel_gru_in_tiles_equals_the_streaming_kernel(q, I, H, n, tiled, columns):
    """Products and gates in one launch, at the edges of its blocks (32 units, 32 to 128 vectors, parts of the k range of either
    product, rows that end inside a step): the states of the narrow kernel on the same vectors, bit for bit."""
    p = synth.gru_cell(seed=n, I=I, H=H)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=8, max_rows=3 * H, max_ld=2048))
    G = q.GruWeights(gpu_mat(q, ctx, p["Wx"], tiled), gpu_mat(q, ctx, p["Wh"], tiled), ctx.f32(p["bx"]), ctx.f32(p["bh"]) if H != 48 else None)
    rng = np.random.default_rng(n)
    x, h = ctx.f32(rng.standard_normal((n, I)).astype(np.float32)), ctx.f32(np.tanh(rng.standard_normal((n, H))).astype(np.float32))
    got = np_(q.gru_step_q8(ctx, G, x, h))
    for i in sorted({0, 8, n // 2, n - 8} & set(range(n - 7))):
        assert_same(got[i:i + 8], np_(q.gru_step_q8(ctx, G, x[i:i + 8].contiguous(), h[i:i + 8].contiguous())), "vectors from %d" % i)


# E, H, A, sentences, beam, tile-packed, tiles of 32 vectors per block: batched steps both of whose GRUs run in gru_tile_kernel and leave their
# states' codes (checked against the library's rule on the host)
TILE_STEPS = [(512, 1024, 1024, 72, 5, True, 2), (512, 1024, 64, 337, 1, True, 2), (620, 1000, 64, 68, 5, False, 2), (620, 1000, 1000, 80, 5, False, 2), (512, 1024, 64, 129, 7, True, 4), (16, 1024, 64, 358, 1, False, 2),
              (64, 2048, 64, 44, 4, True, 2)]


@pytest.mark.parametrize("E,H,A,S,beam,tiled,columns", TILE_STEPS)
def test_batched_step_whose_grus_run_in_tiles(q, oracle, E, H, A, S, beam, tiled, columns):
    """Both transitions in one launch each, and the codes of the new states in another: the states of single sentences' steps, bit for
    bit (those of GRU r's states enter through u(s') and GRU q), and the codes that the oracle makes of them.  One product launch is left, u(s')."""
    rng = np.random.default_rng(H + S)
    p, n, l = synth.cgru_step(seed=2, E=E, H=H, A=A, l=1, n_beam=1), S * beam, 3
    lens = [1 + i % l for i in range(S)]
    L, off = sum(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=8, max_rows=3 * H, max_ld=2 * H))
    w = q.CgruWeights(gpu_gru(q, ctx, p, "dec_r", tiled), gpu_mat(q, ctx, p["att.U"], tiled), ctx.f32(p["att.v"]), gpu_gru(q, ctx, p, "dec_q", tiled))
    enc_h, P = ctx.f32(np.tanh(rng.standard_normal((L, 2 * H))).astype(np.float32)), ctx.f32(rng.standard_normal((L, A)).astype(np.float32))
    y, s0 = ctx.f32(rng.standard_normal((n, E)).astype(np.float32)), ctx.f32((rng.standard_normal((n, H)) * rng.uniform(0.05, 3.0, (n, 1))).astype(np.float32))
    codes = q.Codes(ctx, n, w.r.Wx.ld), q.Codes(ctx, n, w.q.Wx.ld), q.Codes(ctx, n, w.r.Wh.ld)
    offd = torch.tensor(off, device=ctx.device)
    for call in range(2):
        q.q8_profile_begin(ctx, "mfma", 16)
        r = q.cgru_decoder_step_batch_q8(ctx, w, P, enc_h, offd, beam, l, y, s0, codes=codes)
        assert q.q8_profile_end(ctx)[1] == 1
    for si in sorted({0, 1, S // 3, S // 2, S - 2, S - 1}):
        lo, hi, sl = off[si], off[si + 1], slice(si * beam, (si + 1) * beam)
        r1 = q.cgru_decoder_step_q8(ctx, w, P[lo:hi].contiguous(), enc_h[lo:hi].contiguous(), y[sl].contiguous(), s0[sl].contiguous())
        for key in ("s_mid", "ctx", "s"):
            assert_same(r[key][sl], np_(r1[key]), "sentence %d %s vs single-sentence call" % (si, key))
    for j in sorted({0, 31, 32, n // 2, n - 1}):
        for key, c in (("s", codes[2]), ("ctx", codes[1])):
            want, scale = oracle.quantize(np_(r[key])[j])
            assert_same(c.q[j, :want.shape[0]], want, "codes of %s, slot %d" % (key, j))
            assert float(c.scale[j]) == float(scale)


@pytest.mark.parametrize("I,H,n", [(64, 64, 9), (620, 1000, 130), (36, 4, 64)])
def test_panel_gru_of_results_between_vectors_of_four(q, I, H, n):
    """Results need the alignment of a float and no more: where they don't begin at 16 bytes, products and gates run apart (the launch of both
    stores four states at a time).  The same bits, and nothing around them touched."""
    p = synth.gru_cell(seed=n, I=I, H=H)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=8, max_rows=3 * H, max_ld=1024))
    G = q.GruWeights(gpu_mat(q, ctx, p["Wx"]), gpu_mat(q, ctx, p["Wh"]), ctx.f32(p["bx"]), ctx.f32(p["bh"]))
    rng = np.random.default_rng(n)
    x, h = ctx.f32(rng.standard_normal((n, I)).astype(np.float32)), ctx.f32(np.tanh(rng.standard_normal((n, H))).astype(np.float32))
    out = []
    for at in (0, 1, 2, 3, 4):
        buf = ctx.empty(n * H + 8)
        assert buf.data_ptr() % 16 == 0
        buf.fill_(7.0)
        q.q8_profile_begin(ctx, "mfma", 16)
        q.gru_step_q8(ctx, G, x, h, h_out=buf[at:at + n * H].view(n, H))
        assert q.q8_profile_end(ctx)[1] == (1 if at % 4 else 0)
        assert (np_(buf)[:at] == 7.0).all() and (np_(buf)[at + n * H:] == 7.0).all()
        out.append(np_(buf)[at:at + n * H])
    for at in (1, 2, 3, 4):
        assert_same(out[at], out[0], "results %d floats further on" % at)


@pytest.mark.parametrize("E,H,l,tiled", [(512, 1024, 97, True), (512, 1024, 1, False), (516, 132, 77, False), (640, 36, 2, False), (620, 1000, 30, False),
                                         (644, 64, 49, False), (1000, 1000, 9, False), (1024, 256, 48, True), (4, 4, 5, False), (1028, 64, 3, False)])
def test_encoder_of_one_sentence_in_one_launch(q, E, H, l, tiled):
    """All widths of X that the launch multiplies itself, sentences that fill its rows in LDS and go past them, one width more: the
    states of a launch per position, bit for bit, from several streams at once as well."""
    rng = np.random.default_rng(E + l)
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=E + (k == "b"), I=E, H=H).items()}
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=128, max_rows=3 * H, max_ld=1040))
    G = [q.GruWeights(gpu_mat(q, ctx, p[k + "Wx"], tiled), gpu_mat(q, ctx, p[k + "Wh"], tiled), ctx.f32(p[k + "bx"]) if k == "b" else None,
                      ctx.f32(p[k + "bh"])) for k in ("f", "b")]
    X = ctx.f32(rng.standard_normal((l, E)).astype(np.float32))
    q.q8_encoder_options(ctx, False)
    want = np_(q.q8_encode(ctx, G[0], G[1], X))
    q.q8_encoder_options(ctx, True)
    for _ in range(3):
        assert_same(q.q8_encode(ctx, G[0], G[1], X), want, "one launch")
    q.q8_encode_check(ctx)
    torch.cuda.synchronize()
    lanes = []
    for _ in range(4):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            own = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=128, max_rows=3 * H, max_ld=1040), stream=st)
            lanes.append((st, own, own.empty(l, 2 * H)))
    for _ in range(5):
        for st, own, out in lanes:
            with torch.cuda.stream(st):
                q.q8_encode(own, G[0], G[1], X, enc_h=out)
    torch.cuda.synchronize()
    for _, own, out in lanes:
        q.q8_encode_check(own)
        assert_same(out, want, "a stream of its own")


@pytest.mark.parametrize("E,H,l,tiled", [(512, 1024, 30, True), (620, 1000, 9, False), (516, 36, 150, False), (1024, 256, 60, True), (4, 4, 5, False)])
def test_encoder_whose_waits_give_up_gives_the_same_states(q, E, H, l, tiled):
    """Bounds of a few polls end some wait at the first position or further on, in one direction or both: a block works the
    direction off, and enc_h is what a launch per position gives, bit for bit.  What the caller's bound ended is reported."""
    rng = np.random.default_rng(E + l)
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=E + (k == "b"), I=E, H=H).items()}
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=160, max_rows=3 * H, max_ld=1040))
    G = [q.GruWeights(gpu_mat(q, ctx, p[k + "Wx"], tiled), gpu_mat(q, ctx, p[k + "Wh"], tiled), ctx.f32(p[k + "bx"]) if k == "b" else None,
                      ctx.f32(p[k + "bh"])) for k in ("f", "b")]
    X = ctx.f32(rng.standard_normal((l, E)).astype(np.float32))
    q.q8_encoder_options(ctx, False)
    want = np_(q.q8_encode(ctx, G[0], G[1], X))
    out, reported = ctx.empty(l, 2 * H), []
    for bound in (1, 2, 3, 4, 6, 8, 0):
        out.fill_(7.0)
        q.q8_encoder_options(ctx, True, bound)
        assert_same(q.q8_encode(ctx, G[0], G[1], X, enc_h=out), want, "a bound of %d polls" % bound)
        try:
            q.q8_encode_check(ctx)
        except q.Q8Error:
            reported.append(bound)
    assert 0 not in reported and (H <= 32 or 1 in reported)


@pytest.mark.parametrize("E,H,lens,tiled", [(512, 1024, [30], True), (620, 1000, [9], False), (516, 36, [150], False), (640, 256, [60], True), (4, 4, [5], False),
                                            (512, 1024, [1, 9, 4] * 21 + [3], True), (516, 1000, [7, 2, 30], False), (644, 1024, [2, 6, 3] * 20, False),
                                            (640, 36, [4, 17] * 20, False)])
def test_encoders_whose_blocks_don_t_share_an_xcd(q, E, H, lens, tiled):
    """States handed over device-coherently, as where a direction's or a set's blocks run on several XCDs: one sentence, and sentences of one group
    per set with the products of X inside and apart.  What a launch per position gives, bit for bit, again and again, and under a bound of a few polls."""
    rng = np.random.default_rng(E + len(lens))
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=E + (k == "b"), I=E, H=H).items()}
    L, one = sum(lens), len(lens) == 1
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=160, max_rows=3 * H, max_ld=1040) + 24 * L * H + (8 << 20))
    G = [q.GruWeights(gpu_mat(q, ctx, p[k + "Wx"], tiled), gpu_mat(q, ctx, p[k + "Wh"], tiled), ctx.f32(p[k + "bx"]), ctx.f32(p[k + "bh"])) for k in ("f", "b")]
    X, out = ctx.f32(rng.standard_normal((L, E)).astype(np.float32)), ctx.empty(L, 2 * H)
    encode = lambda: np_(q.q8_encode(ctx, G[0], G[1], X, enc_h=out) if one else q.q8_encode_batch(ctx, G[0], G[1], X, lens, enc_h=out))
    q.q8_encoder_options(ctx, False)
    want = encode()
    for bound in (0, 0, 0, 1, 3, 0):
        out.fill_(7.0)
        q.q8_encoder_options(ctx, 2, bound)
        q.q8_profile_begin(ctx, "gru", 16)
        assert_same(encode(), want, "a bound of %d polls" % bound)
        assert q.q8_profile_end(ctx)[1] == 1
        if bound == 0:
            q.q8_encode_check(ctx)
        elif one:
            try:
                q.q8_encode_check(ctx)
            except q.Q8Error:
                pass


def test_encoders_beside_a_batched_decoder(q):
    """One sentence's encoder, a batch's and a batched decoder step whose GRUs fill the device, each on a stream of its own and each of
    blocks that wait for each other: whoever gets the compute units first, all results are what they are alone."""
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=320, max_l=64, max_rows=50000, max_ld=2048) + (64 << 20))
    m, P, enc_h, off, y, s = _panel_case(q, ctx, 64, 5, 12)
    p = {k + n: v for k in ("f", "b") for n, v in synth.gru_cell(seed=5 + (k == "b"), I=512, H=1024).items()}
    G = [q.GruWeights(gpu_mat(q, ctx, p[k + "Wx"], True), gpu_mat(q, ctx, p[k + "Wh"], True), ctx.f32(p[k + "bx"]), ctx.f32(p[k + "bh"])) for k in ("f", "b")]
    X, lens = ctx.f32(np.random.default_rng(3).standard_normal((260, 512)).astype(np.float32)), [3, 20, 9, 33] * 4
    step = q.cgru_decoder_step_batch_q8(ctx, m.dec, P, enc_h, off, 5, 12, y, s)
    one, batch = np_(q.q8_encode(ctx, G[0], G[1], X[:40].contiguous())), np_(q.q8_encode_batch(ctx, G[0], G[1], X, lens))
    step = {k: np_(v) for k, v in step.items()}
    torch.cuda.synchronize()
    lanes = []
    for _ in range(3):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            lanes.append((st, q.Context(workspace_bytes=ctx.workspace.numel(), stream=st)))
    X40, got = X[:40].contiguous(), []
    torch.cuda.synchronize()
    for _ in range(12):
        with torch.cuda.stream(lanes[0][0]):
            got.append((q.q8_encode(lanes[0][1], G[0], G[1], X40), one))
        with torch.cuda.stream(lanes[1][0]):
            r = q.cgru_decoder_step_batch_q8(lanes[1][1], m.dec, P, enc_h, off, 5, 12, y, s)
            got += [(r[k], step[k]) for k in ("s", "ctx")]
        with torch.cuda.stream(lanes[2][0]):
            got.append((q.q8_encode_batch(lanes[2][1], G[0], G[1], X, lens), batch))
    torch.cuda.synchronize()
    for _, own in lanes:
        q.q8_encode_check(own)
    for have, want in got:
        assert_same(have, want, "a stream of its own")


@pytest.mark.parametrize("H,S,group", [(1024, 200, 64), (1000, 90, 60), (516, 512, 64)])
def test_encoder_groups_of_a_set_keep_their_scales_apart(q, H, S, group):
    """Sets of several groups, whose states lie orders of magnitude apart (so that another sentence's scale would show): every
    sentence's states are those of batches small enough for one group per set, every time."""
    rng = np.random.default_rng(H)
    E, lens = 16, [int(v) for v in rng.integers(3, 9, size=S)]
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=S + (k == "b"), I=E, H=H).items()}
    off = np.concatenate([[0], np.cumsum(lens)])
    big = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=64, max_rows=3 * H, max_ld=1024))
    G = [q.GruWeights(gpu_mat(q, big, p[k + "Wx"], False), gpu_mat(q, big, p[k + "Wh"], H % 64 == 0), big.f32(p[k + "bx"] * 0), big.f32(p[k + "bh"] * 0))
         for k in ("f", "b")]
    ctx = q.Context(workspace_bytes=256 * 1024 + q.q8_encode_batch_bytes(G[0], int(off[-1]), S))
    X = rng.standard_normal((int(off[-1]), E)) * np.repeat(10.0 ** -rng.integers(0, 4, size=S), lens)[:, None]
    X = big.f32(X.astype(np.float32))
    want = np.concatenate([np_(q.q8_encode_batch(ctx, G[0], G[1], X[int(off[s]):int(off[min(s + group, S)])].contiguous(), lens[s:s + group]))
                           for s in range(0, S, group)])
    for _ in range(5):
        assert_same(q.q8_encode_batch(ctx, G[0], G[1], X, lens), want, "states")


def test_encoders_on_several_streams_take_turns(q):
    """Four streams with a batch each, whose blocks all wait for each other: the states of one stream alone, and no batch takes
    as long as the blocks that give up on each other would (5 ms and more; half a millisecond is ordinary)."""
    E, H, S = 64, 1024, 64
    rng = np.random.default_rng(7)
    lens = [int(v) for v in rng.integers(10, 61, size=S)]
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=k == "b", I=E, H=H).items()}
    big = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=64, max_rows=3 * H, max_ld=1024))
    G = [q.GruWeights(gpu_mat(q, big, p[k + "Wx"], True), gpu_mat(q, big, p[k + "Wh"], True), big.f32(p[k + "bx"]), big.f32(p[k + "bh"]))
         for k in ("f", "b")]
    X = big.f32(rng.standard_normal((sum(lens), E)).astype(np.float32))
    torch.cuda.synchronize()
    lanes = []
    for _ in range(4):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            ctx = q.Context(workspace_bytes=256 * 1024 + q.q8_encode_batch_bytes(G[0], sum(lens), S), stream=st)
            lanes.append((st, ctx, ctx.empty(sum(lens), 2 * H)))

    def run(n, times):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(times):
            for st, ctx, out in lanes[:n]:
                with torch.cuda.stream(st):
                    q.q8_encode_batch(ctx, G[0], G[1], X, lens, enc_h=out)
        torch.cuda.synchronize()
        return (time.perf_counter() - t) / times / n

    run(4, 2)
    want = np_(lanes[0][2])
    for _, _, out in lanes:
        out.fill_(7.0)
    together = min(run(4, 10) for _ in range(3))
    for st, ctx, out in lanes:
        assert_same(out, want, "states")
        q.q8_encode_check(ctx)
    assert together < 1e-3, together


@pytest.mark.parametrize("one_launch", [True, False])
def test_encoder_of_a_batch_replayed_from_a_graph(q, one_launch):
    """Captured with its clearing launch, which waits for a turn on the device: every replay, with eager batches and new inputs
    between them, gives the eager states."""
    from paper_1804_05038_amd import binding
    E, H, lens = 16, 256, [5, 9, 1, 7] * 40
    rng, L, S = np.random.default_rng(3), sum(lens), len(lens)
    p = {k + s: v for k in ("f", "b") for s, v in synth.gru_cell(seed=k == "b", I=E, H=H).items()}
    big = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=8, max_l=64, max_rows=3 * H, max_ld=1024))
    G = [q.GruWeights(gpu_mat(q, big, p[k + "Wx"], False), gpu_mat(q, big, p[k + "Wh"], True), big.f32(p[k + "bx"]), big.f32(p[k + "bh"]))
         for k in ("f", "b")]
    eager = q.Context(workspace_bytes=256 * 1024 + q.q8_encode_batch_bytes(G[0], L, S))
    xs = [eager.f32(rng.standard_normal((L, E)).astype(np.float32)) for _ in range(3)]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    off_dev, X = torch.as_tensor(off).cuda(), xs[0].clone()
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ctx = q.Context(workspace_bytes=256 * 1024 + q.q8_encode_batch_bytes(G[0], L, S), stream=st)
        q.q8_encoder_options(ctx, one_launch)
        out = ctx.empty(L, 2 * H)
        run = lambda: ctx.check(ctx.lib.q8_encode_batch(ctx.handle, ctypes.byref(G[0].c), ctypes.byref(G[1].c), binding._ptr(X), binding._ptr(off_dev),
                                                        off.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), S, binding._ptr(out)))
        run()
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            run()
    torch.cuda.synchronize()
    for i in range(6):
        X.copy_(xs[i % 3])
        out.fill_(7.0)
        want = np_(q.q8_encode_batch(eager, G[0], G[1], xs[i % 3], lens))
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            graph.replay()
        torch.cuda.synchronize()
        assert_same(out, want, "replay %d" % i)


@pytest.mark.parametrize("V,R,n", [(17, 512, 9), (31, 512, 33), (33, 640, 224), (65, 512, 225), (1000, 512, 257), (1009, 640, 289),
                                   (4097, 512, 511), (2051, 640, 1024)])
def test_vocabulary_panel_edges(q, oracle, V, R, n):
    """The panel kernel's units (64 rows x 32 slots) at their remainders, rows past the last packed tile, column groups of
    every size, an odd bias address: the selection on its statistics against the one on stored logits.  The sums behind
    the log-sum-exp differ in order (double, rounded to float once): a last place of lse."""
    rng = np.random.default_rng(V + n)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=8, max_rows=max(V, 4096), max_ld=640))
    W = gpu_mat(q, ctx, (rng.standard_normal((V, R)) * 0.05).astype(np.float32), True)
    b = ctx.f32(np.concatenate([[0], rng.standard_normal(V)]).astype(np.float32))[1:]
    t = ctx.f32(np.tanh(rng.standard_normal((n, R))).astype(np.float32))
    for bias in (b, None):
        kept = q.output_logits_q8(ctx, None, W, bias, t_in=t, k=12, want_logits=True)
        r = q.output_logits_q8(ctx, None, W, bias, t_in=t, k=12, want_logits=False)
        assert_same(r["topk_idx"], np_(kept["topk_idx"]), "indices")
        assert_close(r["lse"], np_(kept["lse"]).astype(np.float64), "lse", rel=2.0 ** -22)
        assert_close(r["topk_logp"], np_(kept["topk_logp"]).astype(np.float64), "logp", rel=2.0 ** -22)


@pytest.mark.parametrize("beam,H,lens", [(1, 36, [3] * 9), (2, 36, [8, 9, 16, 17, 1, 5]), (3, 1000, [7] * 3 + [33]), (5, 1024, [1, 2, 3, 60, 8] * 14),
                                         (5, 20, [4, 11] * 100), (7, 64, [5] * 40), (8, 36, [9, 2] * 64), (4, 36, [900, 3, 30]), (2, 1028, [6] * 5)])
def test_context_of_several_hypotheses_per_block(q, beam, H, lens):
    """The context kernel at every number of hypotheses per block, passes that end past the beam, positions at the edges
    of a round of loads, widths it leaves to the other kernel (C = 2 H > 2048): the single-sentence step, bit for bit."""
    E = A = 36
    p = synth.cgru_step(seed=beam, E=E, H=H, A=A, l=1, n_beam=len(lens) * beam)
    L, n = sum(lens), len(lens) * beam
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=max(lens), max_rows=3 * H, max_ld=2 * H + 64))
    rng = np.random.default_rng(H)
    P, enc = ctx.f32(rng.standard_normal((L, A)).astype(np.float32)), ctx.f32(rng.standard_normal((L, 2 * H)).astype(np.float32))
    gru = lambda pre: gpu_gru(q, ctx, p, pre)
    w = q.CgruWeights(gru("dec_r"), gpu_mat(q, ctx, p["att.U"], False), ctx.f32(p["att.v"]), gru("dec_q"))
    off = np.array([0] + list(np.cumsum(lens)), dtype=np.int32)
    y, s = ctx.f32(p["y_emb"]), ctx.f32(p["s_prev"])
    r = q.cgru_decoder_step_batch_q8(ctx, w, P, enc, torch.as_tensor(off).to(ctx.device), beam, max(lens), y, s)
    for i in sorted({0, 1, 3, len(lens) // 2, len(lens) - 1} & set(range(len(lens)))):
        rows, sl = slice(int(off[i]), int(off[i + 1])), slice(i * beam, (i + 1) * beam)
        one = q.cgru_decoder_step_q8(ctx, w, P[rows].contiguous(), enc[rows].contiguous(), y[sl].contiguous(), s[sl].contiguous())
        assert_same(r["alpha"][sl, :lens[i]], np_(one["alpha"]), "alpha, sentence %d" % i)
        assert_same(r["ctx"][sl], np_(one["ctx"]), "context, sentence %d" % i)
        assert_same(r["s"][sl], np_(one["s"]), "state, sentence %d" % i)


@pytest.mark.parametrize("beam,A,H,lens,s0", [(5, 64, 64, [30, 30, 30, 30, 30, 30], 3), (1, 36, 36, [4] * 30, 20), (8, 1028, 36, [9, 60, 2, 33, 1], 2)])
def test_a_group_of_a_packed_batch_is_stepped_by_its_offsets(q, ctx, beam, A, H, lens, s0):
    """A group of sentences out of a larger packed batch, stepped with the offsets from its first sentence on and the
    batch's own P and encoder states (the first offset is not 0): bit for bit what the same group gives packed alone."""
    E = 36
    S = len(lens) - s0
    p = synth.cgru_step(seed=7, E=E, H=H, A=A, l=1, n_beam=S * beam)
    rng = np.random.default_rng(beam)
    L = sum(lens)
    P, enc = ctx.f32(rng.standard_normal((L, A)).astype(np.float32)), ctx.f32(rng.standard_normal((L, 2 * H)).astype(np.float32))
    gru = lambda pre: gpu_gru(q, ctx, p, pre)
    w = q.CgruWeights(gru("dec_r"), gpu_mat(q, ctx, p["att.U"], False), ctx.f32(p["att.v"]), gru("dec_q"))
    off = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device=ctx.device)
    y, s = ctx.f32(p["y_emb"]), ctx.f32(p["s_prev"])
    first, max_l = int(off[s0]), max(lens[s0:])
    r = q.cgru_decoder_step_batch_q8(ctx, w, P, enc, off[s0:], beam, max_l, y, s)
    alone = q.cgru_decoder_step_batch_q8(ctx, w, P[first:].contiguous(), enc[first:].contiguous(), (off[s0:] - first).contiguous(), beam, max_l, y, s)
    for k in ("alpha", "ctx", "s"):
        assert_same(r[k], np_(alone[k]), k)
