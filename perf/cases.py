"""What decoding with this library consists of, as cases that can be timed and checked one by one.

Each case is one public entry point, or the loop of them that a translation runs, at the sizes this
repository works at: the synthetic model of `workloads/synth.py` (embedding 512, hidden 1024, attention
1024, readout 512, 50000 words), the dimensions of the paper's own systems (620 / 1000 / 1000 / 620, its
vocabularies of 33658 to 63644 words) and a small GRU cell (256).  Sentences are 10 to 60 words, the beam
is 5 (at most 8), 12 continuations are kept per hypothesis.

`exact` is the definition in 64 bits: int8 codes as Section 3's scheme defines them (max-abs in fp32,
round half to even), everything between two quantizations in double.  A vector that is quantized is first
rounded to fp32, as it is one in the library.
"""
import math

import numpy as np
import torch

import paper_1804_05038_amd as q

DEV = "cuda:0"
TOPK = 12
MAX_STEPS = 100
DIMS = {  # E, H, A, R
    "synth": (512, 1024, 1024, 512),
    "paper": (620, 1000, 1000, 620),
}


def listed():
    return [
        # one cell of the smallest configuration: a call whose time is latency
        {"name": "gru_cell_256", "kind": "gru", "I": 256, "H": 256, "n": 1},
        # the matrix x vector product on the largest matrix of the model, the headline product
        {"name": "gemv_50000x512", "kind": "product", "rows": 50000, "cols": 512, "n": 1},
        # w(h_i) of the attention for all source positions of a batch of sentences (a full panel)
        {"name": "panel_1024x2048_n1024", "kind": "product", "rows": 1024, "cols": 2048, "n": 1024},
        # one conditional-GRU step, greedy decoding
        {"name": "cgru_step_greedy", "kind": "cgru", "dims": "synth", "beam": 1, "l": 30},
        # vocabulary layer with the logits kept (rescoring, n-best), beam 5
        {"name": "output_logits_beam5", "kind": "output", "V": 50000, "R": 512, "n": 5},
        # encoder of one sentence
        {"name": "encode_l50", "kind": "encode", "dims": "synth", "l": 50},
        # encoder of a batch of sentences of 10 to 60 words
        {"name": "encode_batch_64", "kind": "encode_batch", "dims": "synth", "sents": 64},
        # the decoding loop of one sentence as q8_translate runs it
        {"name": "decode_beam5", "kind": "decode", "dims": "synth", "V": 50000, "beam": 5, "l": 30, "steps": 8},
        # the same at the dimensions of the paper's systems, its largest vocabulary
        {"name": "decode_paper_beam5", "kind": "decode", "dims": "paper", "V": 63644, "beam": 5, "l": 30, "steps": 8},
        # the batched decoding loop as q8_translate_batch runs it: a serving batch, and a whole test set
        {"name": "decode_batch_64", "kind": "decode_batch", "dims": "synth", "V": 50000, "beam": 5, "sents": 64, "steps": 4},
        {"name": "decode_batch_200", "kind": "decode_batch", "dims": "synth", "V": 50000, "beam": 5, "sents": 200, "steps": 4},
        # a decoder step and output layer of the 32-bit engine
        {"name": "step_f32_beam5", "kind": "step_f32", "dims": "synth", "V": 50000, "beam": 5, "l": 30},
    ]


def _between(rng, lo, hi, step=1):
    """A multiple of step in [lo, hi], even over the logarithm where the range is wide."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1))) if hi > 10 * lo else rng.uniform(lo, hi + 1)
    return max(lo, min(hi, int(v) // step * step))


def draw(rng):
    kind = rng.choice(["gru", "product", "panel", "cgru", "output", "encode", "encode_batch", "decode", "decode_batch",
                       "decode_batch", "step_f32"])
    dims = rng.choice(["synth", "paper"])
    V = rng.randint(33658, 63644)
    if kind == "gru":
        return {"kind": kind, "I": _between(rng, 64, 1024, 4), "H": _between(rng, 64, 1024, 4), "n": rng.randint(1, 8)}
    if kind == "product":
        return {"kind": kind, "rows": _between(rng, 256, 63644), "cols": _between(rng, 256, 2048, 4), "n": rng.randint(1, 8)}
    if kind == "panel":
        return {"kind": "product", "rows": _between(rng, 512, 3072), "cols": _between(rng, 256, 2048, 4), "n": _between(rng, 9, 1024)}
    if kind == "cgru":
        return {"kind": kind, "dims": dims, "beam": rng.randint(1, 8), "l": _between(rng, 1, 300)}
    if kind == "output":
        return {"kind": kind, "V": V, "R": DIMS[dims][3], "n": rng.randint(1, 8)}
    if kind == "encode":
        return {"kind": kind, "dims": dims, "l": _between(rng, 1, 100)}
    if kind == "encode_batch":
        return {"kind": kind, "dims": dims, "sents": _between(rng, 2, 200)}
    if kind == "decode":
        return {"kind": kind, "dims": dims, "V": V, "beam": rng.randint(1, 8), "l": rng.randint(10, 60), "steps": rng.randint(4, 8)}
    if kind == "decode_batch":
        beam = rng.randint(1, 8)
        return {"kind": kind, "dims": dims, "V": V, "beam": beam, "sents": _between(rng, 2, 700 // beam), "steps": rng.randint(2, 4)}
    return {"kind": kind, "dims": dims, "V": V, "beam": rng.randint(1, 8), "l": rng.randint(10, 60)}


# ---- inputs ---------------------------------------------------------------------------------------

def _lengths(sents):
    """Sentence lengths of a batch: part of the case, the same for every seed."""
    return [int(v) for v in np.random.default_rng(1000 + sents).integers(10, 61, size=sents)]


class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def n(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device=DEV, dtype=torch.float32) * std

    def states(self, *shape):
        """Like the states of a GRU: inside (-1, 1)."""
        return torch.tanh(self.n(*shape, std=0.6))


def _gru_params(d, p, name, I, H, std=0.05):
    p[name + ".Wx"], p[name + ".Wh"] = d.n(3 * H, I, std=std), d.n(3 * H, H, std=std)
    p[name + ".bx"], p[name + ".bh"] = d.n(3 * H, std=0.01), d.n(3 * H, std=0.01)


def _decoder_params(d, E, H, A):
    p = {}
    _gru_params(d, p, "dec_r", E, H)
    p["att.U"], p["att.v"] = d.n(A, H, std=0.05), d.n(A, std=0.05)
    _gru_params(d, p, "dec_q", 2 * H, H)
    return p


def _output_params(d, p, E, H, R, V):
    p["ro.Ws"], p["ro.Wy"], p["ro.Wc"], p["ro.b"] = d.n(R, H, std=0.05), d.n(R, E, std=0.05), d.n(R, 2 * H, std=0.05), d.n(R, std=0.01)
    p["out.W"], p["out.b"] = d.n(V, R, std=0.05), d.n(V, std=0.01)


def _raw(case, seed):
    """Every fp32 tensor of a case, from its seed."""
    d, kind = _Draws(seed), case["kind"]
    if kind == "gru":
        p = {}
        _gru_params(d, p, "g", case["I"], case["H"], std=0.1)
        p["x"], p["h"] = d.n(case["n"], case["I"]), d.n(case["n"], case["H"])
        return p
    if kind == "product":
        return {"W": d.n(case["rows"], case["cols"], std=0.05), "b": d.n(case["rows"], std=0.01), "x": d.n(case["n"], case["cols"])}
    if kind == "output":
        p = {"out.W": d.n(case["V"], case["R"], std=0.05), "out.b": d.n(case["V"], std=0.01)}
        p["t"] = torch.tanh(d.n(case["n"], case["R"]))
        return p
    E, H, A, R = DIMS[case["dims"]]
    if kind in ("encode", "encode_batch"):
        p = {}
        _gru_params(d, p, "fwd", E, H)
        _gru_params(d, p, "bwd", E, H)
        p["X"] = d.n(case["l"] if kind == "encode" else sum(_lengths(case["sents"])), E)
        return p
    p = _decoder_params(d, E, H, A)
    L = sum(_lengths(case["sents"])) if kind == "decode_batch" else case["l"]
    # the encoder's states and w(h_i) + b of them, spread as the products of such states are
    p["enc_h"], p["P"] = d.states(L, 2 * H), d.n(L, A, std=0.9)
    if kind in ("cgru", "step_f32"):
        p["y"], p["s"] = d.n(case["beam"], E), d.states(case["beam"], H)
    if kind != "cgru":
        _output_params(d, p, E, H, R, case["V"])
    if kind in ("decode", "decode_batch"):
        p["E_tgt"] = d.n(case["V"], E)
        p["s0"] = d.states(H)
    return p


# ---- states ---------------------------------------------------------------------------------------

def _mat(ctx, W, ld=None):
    """A quantized matrix, with the copy that the matrix cores stream where its rows allow one."""
    m = q.q8_quantize_matrix(ctx, W, ld_out=ld)
    return q.q8_pack_tiles(ctx, m) if m.ld % 64 == 0 else m


def _gru(ctx, p, name):
    return q.GruWeights(_mat(ctx, p[name + ".Wx"]), _mat(ctx, p[name + ".Wh"]), p[name + ".bx"], p[name + ".bh"])


def _cgru(ctx, p):
    return q.CgruWeights(_gru(ctx, p, "dec_r"), _mat(ctx, p["att.U"]), p["att.v"], _gru(ctx, p, "dec_q"))


def _W_out(ctx, W):
    return _mat(ctx, W, (W.shape[1] + 63) // 64 * 64)


def _offsets(lens):
    return torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device=DEV)


class _State:
    pass


def prepare(case, seed):
    p, st, kind = _raw(case, seed), _State(), case["kind"]
    st.kind, st.p = kind, p
    if kind in ("encode_batch", "decode_batch"):
        n = case["sents"] * case.get("beam", 1)
        ws = q.q8_workspace_bytes(max_n=max(n, 8), max_l=60, max_rows=case.get("V", 4096), max_ld=2048)
        st.ctx = ctx = q.Context(DEV, workspace_bytes=ws)
    else:
        n = case.get("n", case.get("beam", 1))
        st.ctx = ctx = q.Context(DEV, workspace_bytes=q.q8_workspace_bytes(max_n=max(n, 8), max_l=max(64, case.get("l", 1)),
                                                                           max_rows=max(65536, case.get("rows", 0))))
    if kind == "gru":
        st.g = _gru(ctx, p, "g")
        st.call = q.gru_step_q8(ctx, st.g, p["x"], p["h"], bind=True)
    elif kind == "product":
        st.W = _mat(ctx, p["W"]) if case["n"] > 8 else q.q8_quantize_matrix(ctx, p["W"])
        st.Y = ctx.empty(case["n"], (case["rows"] + 3) // 4 * 4)[:, :case["rows"]]
        st.x1 = p["x"][0] if case["n"] == 1 else None
    elif kind == "cgru":
        st.call = q.cgru_decoder_step_q8(ctx, _cgru(ctx, p), p["P"], p["enc_h"], p["y"], p["s"], bind=True)
    elif kind == "output":
        st.call = q.output_logits_q8(ctx, None, _W_out(ctx, p["out.W"]), p["out.b"], t_in=p["t"], k=TOPK, bind=True)
    elif kind == "encode":
        st.fwd, st.bwd = _gru(ctx, p, "fwd"), _gru(ctx, p, "bwd")
        st.enc_h = ctx.empty(case["l"], 2 * st.fwd.H)
    elif kind == "encode_batch":
        st.fwd, st.bwd, st.lens = _gru(ctx, p, "fwd"), _gru(ctx, p, "bwd"), _lengths(case["sents"])
        st.enc_h = ctx.empty(sum(st.lens), 2 * st.fwd.H)
        st.ctx = q.Context(DEV, workspace_bytes=ws + q.q8_encode_batch_bytes(st.fwd, sum(st.lens), len(st.lens)))
    elif kind == "decode":
        _prepare_decode(st, ctx, case, p)
    elif kind == "decode_batch":
        _prepare_decode_batch(st, ctx, case, p)
    elif kind == "step_f32":
        mf = lambda k: q.MatF(ctx, p[k].cpu().numpy())
        gru = lambda n: q.GruWeightsF32(mf(n + ".Wx"), mf(n + ".Wh"), p[n + ".bx"], p[n + ".bh"])
        w = q.CgruWeightsF32(gru("dec_r"), mf("att.U"), p["att.v"], gru("dec_q"))
        ro = q.ReadoutWeightsF32(mf("ro.Ws"), mf("ro.Wy"), mf("ro.Wc"), p["ro.b"])
        st.c1 = q.cgru_decoder_step_f32(ctx, w, p["P"], p["enc_h"], p["y"], p["s"], bind=True)
        st.c2 = q.output_logits_f32(ctx, ro, mf("out.W"), p["out.b"], st.c1.out["s"], p["y"], st.c1.out["ctx"], k=TOPK,
                                    want_logits=False, bind=True)
    return st


def _readout(ctx, p):
    return q.ReadoutWeights(_mat(ctx, p["ro.Ws"]), _mat(ctx, p["ro.Wy"]), _mat(ctx, p["ro.Wc"]), p["ro.b"])


def _prepare_decode(st, ctx, case, p):
    n, dec, ro, W_out = case["beam"], _cgru(ctx, p), _readout(ctx, p), _W_out(ctx, p["out.W"])
    gx, E_codes = q.gru_input_table(ctx, dec.r, p["E_tgt"]), q.RowCodes(ctx, p["E_tgt"], dec.r.Wx.ld)
    H, E = dec.r.H, p["E_tgt"].shape[1]
    state = torch.zeros(q.q8_beam_state_bytes(MAX_STEPS), dtype=torch.uint8, device=DEV)
    st.y, s = ctx.empty(n, E), ctx.empty(n, H)
    st.s_mid = [ctx.empty(n, H), ctx.empty(n, H)]
    st.init = q.q8_beam_init(ctx, state, n, MAX_STEPS, p["s0"], p["E_tgt"], st.y, s, bind=True)
    st.first = q.gru_step_q8(ctx, dec.r, st.y, s, h_out=st.s_mid[0], bind=True)
    st.yc, cc, out = q.Codes(ctx, n, dec.r.Wx.ld), q.Codes(ctx, n, dec.q.Wx.ld), None
    st.c1, st.c2, st.steps = [], [], case["steps"]
    for i in (0, 1):
        c1 = q.cgru_decoder_step_ahead_q8(ctx, dec, p["P"], p["enc_h"], st.s_mid[i], out=out, bind=True, ctx_codes=cc)
        out = c1.out
        st.c1.append(c1)
        st.c2.append(q.output_logits_beam_ahead_q8(ctx, ro, W_out, p["out.b"], out["s"], st.y, out["ctx"], state, p["E_tgt"], dec.r,
                                                   gx, st.s_mid[1 - i], k=TOPK, bind=True, y_codes=st.yc, ctx_codes=cc,
                                                   E_codes=E_codes))


def _prepare_decode_batch(st, ctx, case, p):
    S, beam, dec, ro, W_out = case["sents"], case["beam"], _cgru(ctx, p), _readout(ctx, p), _W_out(ctx, p["out.W"])
    lens = _lengths(S)
    n, off, E_codes = S * beam, _offsets(lens), q.RowCodes(ctx, p["E_tgt"], dec.r.Wx.ld)
    H, E = dec.r.H, p["E_tgt"].shape[1]
    states = torch.zeros(q.q8_beam_state_bytes(MAX_STEPS) * S, dtype=torch.uint8, device=DEV)
    st.y, st.s, done = ctx.empty(n, E), ctx.empty(n, H), torch.zeros(S, dtype=torch.int32, device=DEV)
    st.init = q.q8_beam_init_batch(ctx, states, S, beam, MAX_STEPS, p["enc_h"], off, p["E_tgt"], st.y, st.s, done, bind=True)
    codes, st.sp = (q.Codes(ctx, n, dec.r.Wx.ld), q.Codes(ctx, n, dec.q.Wx.ld), q.Codes(ctx, n, ro.W_s.ld)), q.Codes(ctx, n, dec.r.Wh.ld)
    st.yc = codes[0]
    st.c1 = q.cgru_decoder_step_batch_q8(ctx, dec, p["P"], p["enc_h"], off, beam, max(lens), st.y, st.s, bind=True, codes=codes + (st.sp,))
    st.c2 = q.output_logits_beam_batch_q8(ctx, ro, W_out, p["out.b"], st.c1.out["s"], st.y, st.c1.out["ctx"], states, S, beam,
                                          MAX_STEPS, p["E_tgt"], st.s, done, k=TOPK, bind=True, codes=(codes[2], codes[0], codes[1]),
                                          s_next_codes=st.sp, E_codes=E_codes)
    st.steps = case["steps"]


def run(st):
    kind, ctx = st.kind, st.ctx
    if kind == "gru":
        st.call.launch()
        return st.call.out["h"]
    if kind == "product":
        if st.x1 is not None:
            return q.q8_gemv(ctx, st.W, st.x1, st.p["b"], y=st.Y[0])
        return q.q8_gemm_narrow(ctx, st.W, st.p["x"], st.p["b"], Y=st.Y)
    if kind == "cgru":
        st.call.launch()
        return {k: st.call.out[k] for k in ("s", "ctx", "alpha", "s_mid")}
    if kind == "output":
        st.call.launch()
        return {k: st.call.out[k] for k in ("logits", "lse", "topk_logp", "topk_idx")}
    if kind == "encode":
        return q.q8_encode(ctx, st.fwd, st.bwd, st.p["X"], enc_h=st.enc_h)
    if kind == "encode_batch":
        return q.q8_encode_batch(ctx, st.fwd, st.bwd, st.p["X"], st.lens, enc_h=st.enc_h)
    if kind == "decode":
        st.init.launch()
        st.yc.invalidate()                  # y is not what the codes were made of
        st.first.launch()
        for t in range(st.steps):
            st.c1[t & 1].launch()
            st.c2[t & 1].launch()
        i = (st.steps - 1) & 1
        o = st.c2[i].out
        return {"topk_logp": o["topk_logp"], "topk_idx": o["topk_idx"], "s": st.c1[i].out["s"], "ctx": st.c1[i].out["ctx"],
                "alpha": st.c1[i].out["alpha"], "y": st.y, "s_mid": st.s_mid[1 - i]}
    if kind == "decode_batch":
        st.init.launch()
        st.yc.invalidate()
        st.sp.invalidate()
        for t in range(st.steps):
            st.c1.launch()
            st.c2.launch()
        return {"topk_logp": st.c2.out["topk_logp"], "topk_idx": st.c2.out["topk_idx"], "s": st.c1.out["s"], "ctx": st.c1.out["ctx"],
                "alpha": st.c1.out["alpha"], "y": st.y, "s_next": st.s}
    st.c1.launch()
    st.c2.launch()
    return {k: v for c in (st.c1, st.c2) for k, v in c.out.items() if isinstance(v, torch.Tensor)}


# ---- what a pass cannot do without ------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "gru":
        I, H, n = case["I"], case["H"], case["n"]
        return {"bytes": 3 * H * (I + H) + 24 * H + 4 * n * (I + 2 * H), "flops": 2 * n * 3 * H * (I + H)}
    if kind == "product":
        r, c, n = case["rows"], case["cols"], case["n"]
        return {"bytes": r * c + 4 * r + 4 * n * (c + r), "flops": 2 * n * r * c}
    if kind == "output":
        V, R, n = case["V"], case["R"], case["n"]
        return {"bytes": V * R + 4 * V + 4 * n * (R + V), "flops": 2 * n * V * R}
    E, H, A, R = DIMS[case["dims"]]
    if kind in ("encode", "encode_batch"):
        lens = [case["l"]] if kind == "encode" else _lengths(case["sents"])
        L, w = sum(lens), 2 * 3 * H * (E + H)
        # the recurrence multiplies the recurrent matrix at every position of the longest sentence: they are
        # read once here, as they can be kept on the chip
        return {"bytes": w + 4 * L * (E + 2 * H), "flops": 2 * L * w}
    f32 = kind == "step_f32"
    size = 4 if f32 else 1
    n, steps = case["beam"] * case.get("sents", 1), case.get("steps", 1)
    L = sum(_lengths(case["sents"])) if kind == "decode_batch" else case["l"]
    w = 3 * H * (E + H) + A * H + 3 * H * (2 * H + H)
    slot_l = L * case["beam"]                                  # (hypothesis, position) pairs
    flops = 2 * n * w + slot_l * (8 * A + 4 * H)
    # per step: the matrices, P and the encoder's states, the step's inputs and results
    nbytes = size * w + 4 * L * (A + 2 * H) + 4 * n * (E + 5 * H)
    if kind != "cgru":
        w_out = R * (E + 3 * H) + case["V"] * R
        flops += 2 * n * w_out
        nbytes += size * w_out + 4 * case["V"] + 4 * n * (2 * E + H)
    return {"bytes": steps * nbytes, "flops": steps * flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "product":
        return {"rel": 1e-6, "max": 1e-5}          # exact integer sums, two roundings
    if kind == "gru":
        return {"rel": 2e-6, "max": 2e-5}
    if kind == "output":
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.001}
    if kind == "step_f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.001}
    # Chains in which a vector is rounded to fp32 and quantized again: a last-place difference that moves one
    # code of it by one is 1/127 of that entry, and travels through all that follows.
    return {"rel": 5e-3, "max": 0.2, "differ": 0.01}


# ---- the definition in 64 bits ----------------------------------------------------------------------

def _codes(v):
    """fp32 [..., K] -> (codes, scale) per vector, in double."""
    m = v.abs().amax(-1, keepdim=True).cpu().numpy()
    tiny = m < np.float32(2.0 ** -100)
    safe = np.where(tiny, np.float32(1), m)
    inv, scale = np.float32(127) / safe, np.where(tiny, np.float32(1), safe / np.float32(127))
    inv, scale = torch.from_numpy(np.where(tiny, np.float32(0), inv)).to(DEV), torch.from_numpy(scale).to(DEV)
    return torch.clamp(torch.round(v * inv), -127, 127).double(), scale.double()


def _whole(W):
    """A matrix's codes and its one scale."""
    c, s = _codes(W.reshape(1, -1))
    return c.reshape(W.shape), s.reshape(())


def _rows_by_rows(a, b):
    """a @ b.T in double; the second operand is laid out for it first."""
    return torch.mm(a, b.t().contiguous())


def _mul(Wc, x, b=None):
    """One product: x is rounded to fp32 and quantized, vector by vector."""
    c, s = _codes(x.float())
    y = _rows_by_rows(c, Wc[0]) * (Wc[1] * s)
    return y if b is None else y + b.double()


def _cell(gx, gh, h):
    H = h.shape[-1]
    r, z = torch.sigmoid(gx[:, :H] + gh[:, :H]), torch.sigmoid(gx[:, H:2 * H] + gh[:, H:2 * H])
    c = torch.tanh(gx[:, 2 * H:] + r * gh[:, 2 * H:])
    return (1 - z) * c + z * h.float().double()


def _matrices(p, quantized=True):
    return {k: _whole(v) if quantized else v.double() for k, v in p.items()
            if k.endswith((".Wx", ".Wh")) or k in ("att.U", "ro.Ws", "ro.Wy", "ro.Wc", "out.W")}


def _gru_exact(M, p, name, x, h, mul):
    return _cell(mul(M[name + ".Wx"], x, p[name + ".bx"]), mul(M[name + ".Wh"], h, p[name + ".bh"]), h)


def _cgru_exact(M, p, lens, beam, y, s, mul, s_mid=None):
    """One decoder step of len(lens) beams; alpha is padded to the longest sentence."""
    if s_mid is None:
        s_mid = _gru_exact(M, p, "dec_r", y, s, mul)
    a = mul(M["att.U"], s_mid).float().double()
    alpha = torch.zeros(len(lens) * beam, max(lens), dtype=torch.float64, device=DEV)
    ctx, o = [], 0
    v = p["att.v"].double()
    for i, l in enumerate(lens):
        P, h = p["P"][o:o + l].double(), p["enc_h"][o:o + l].double()
        o += l
        sl = slice(i * beam, (i + 1) * beam)
        e = (torch.tanh(P[None] + a[sl][:, None]) * v).sum(-1)
        al = torch.softmax(e, -1)
        alpha[sl, :l] = al
        ctx.append(torch.mm(al, h))
    ctx = torch.cat(ctx)
    return {"s": _gru_exact(M, p, "dec_q", ctx, s_mid, mul), "ctx": ctx, "alpha": alpha, "s_mid": s_mid}


def _top(M, t, b, mul):
    logits = mul(M["out.W"], t, b)
    lse = torch.logsumexp(logits, -1)
    val, idx = torch.topk(logits, TOPK, dim=-1)
    return {"logits": logits, "lse": lse, "topk_logp": val - lse[:, None], "topk_idx": idx.to(torch.int32)}


def _hidden(M, p, s, y, ctx, mul):
    return torch.tanh(mul(M["ro.Ws"], s) + mul(M["ro.Wy"], y) + mul(M["ro.Wc"], ctx) + p["ro.b"].double())


def _search(top, live, beam):
    """One search step of every beam: (parent, token) of each slot of the panel, and the new live hypotheses."""
    lp, ix = top["topk_logp"].cpu().numpy(), top["topk_idx"].cpu().numpy()
    parents, tokens, after = [], [], []
    for i, (width, scores) in enumerate(live):
        if width == 0 or not scores:                     # over: the slots keep what they hold
            return None
        cand = sorted((-(sc + lp[i * beam + j, r]), j, int(ix[i * beam + j, r])) for j, sc in enumerate(scores) for r in range(TOPK))
        kept = cand[:width]
        alive = [c for c in kept if c[2] != 0]
        slots = [(j, t) for _, j, t in alive] + [(alive[0][1], alive[0][2]) if alive else (0, 0)] * (beam - len(alive))
        parents += [i * beam + j for j, _ in slots]
        tokens += [t for _, t in slots]
        after.append((width - (len(kept) - len(alive)), [-c[0] for c in alive]))
    return torch.tensor(parents, device=DEV), torch.tensor(tokens, device=DEV), after


def exact(case, seed):
    p, kind, mul = _raw(case, seed), case["kind"], _mul
    if kind == "product":
        y = _mul(_whole(p["W"]), p["x"], p["b"])
        return y[0] if case["n"] == 1 else y
    M = _matrices(p, kind != "step_f32")
    if kind == "gru":
        return _gru_exact(M, p, "g", p["x"], p["h"], mul)
    if kind == "output":
        return _top(M, p["t"], p["out.b"], mul)
    if kind in ("encode", "encode_batch"):
        lens = [case["l"]] if kind == "encode" else _lengths(case["sents"])
        return _encode_exact(M, p, lens)
    if kind == "cgru":
        return _cgru_exact(M, p, [case["l"]], case["beam"], p["y"], p["s"], mul)
    if kind == "step_f32":
        mul = lambda W, x, b=None: _rows_by_rows(x.float().double(), W) + (0 if b is None else b.double())
        r = _cgru_exact(M, p, [case["l"]], case["beam"], p["y"], p["s"], mul)
        t = _hidden(M, p, r["s"], p["y"], r["ctx"], mul)
        top = _top(M, t, p["out.b"], mul)
        top.pop("logits")
        return {**r, **top, "t": t}
    # the decoding loops
    beam, lens = case["beam"], _lengths(case["sents"]) if kind == "decode_batch" else [case["l"]]
    H = p["s0"].shape[0]
    if kind == "decode_batch":
        first = torch.tensor([0] + list(np.cumsum(lens))[:-1], device=DEV)
        s = p["enc_h"][first, :H].repeat_interleave(beam, 0)
    else:
        s = p["s0"].expand(beam, H).contiguous()
    y, live = p["E_tgt"][:1].expand(len(lens) * beam, -1).contiguous(), [(beam, [0.0])] * len(lens)
    for _ in range(case["steps"]):
        r = _cgru_exact(M, p, lens, beam, y, s, mul)
        top = _top(M, _hidden(M, p, r["s"], y, r["ctx"], mul), p["out.b"], mul)
        found = _search(top, live, beam)
        if found is None:
            return None
        parents, tokens, live = found
        s, y = r["s"][parents], p["E_tgt"][tokens]
    out = {"topk_logp": top["topk_logp"], "topk_idx": top["topk_idx"], "s": r["s"], "ctx": r["ctx"], "alpha": r["alpha"], "y": y}
    if kind == "decode":
        return {**out, "s_mid": _gru_exact(M, p, "dec_r", y, s, mul)}
    return {**out, "s_next": s}


def _encode_exact(M, p, lens):
    """All sentences side by side, both directions; sentences that are over drop out."""
    off = np.concatenate([[0], np.cumsum(lens)])
    H = p["fwd.Wh"].shape[1]
    enc = torch.zeros(int(off[-1]), 2 * H, dtype=torch.float64, device=DEV)
    order = np.argsort(-np.asarray(lens), kind="stable")
    for name, col, back in (("bwd", 0, True), ("fwd", H, False)):
        gx = _mul(M[name + ".Wx"], p["X"], p[name + ".bx"])
        h = torch.zeros(len(lens), H, dtype=torch.float64, device=DEV)
        for t in range(max(lens)):
            on = [i for i in order if lens[i] > t]
            at = torch.tensor([int(off[i + 1]) - 1 - t if back else int(off[i]) + t for i in on], device=DEV)
            gh = _mul(M[name + ".Wh"], h[:len(on)], p[name + ".bh"])
            h = _cell(gx[at], gh, h[:len(on)])
            enc[at, col:col + H] = h
    return enc
