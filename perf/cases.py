"""Performance cases of the DPara drafter path on one MI355X.

Each case is one call, or one natural group of calls, of the public Python entry points
(``paper_2609_27396_amd.dpara``) on device-resident tensors, as a serving loop issues them:

  round       append -> backbone -> verify -> select + head of the small float32 drafter
  update      feature fusion + context append (after a round: gamma + 1 rows; or a prompt)
  precompute  append + all-boundary backbone, every layer (the drafter's stream)
  layer       all-boundary backbone of one drafter layer
  target      the verifying target over the gamma + 1 block rows, with the hidden states the
              drafter fuses
  serial      greedy verify + select + head (the serial step of a round)
  sampled     speculative-sampling verify + sampled head with its draft scores
  candidates  every branch's head candidates + greedy verify + the candidates head

Shapes are the Qwen3-8B, Qwen3-14B and small float32 shapes of ``synth``; weights, context
caches and inputs are drawn on the GPU from the seed.
"""
from __future__ import annotations

import ctypes
import math
from dataclasses import replace

import torch

from paper_2609_27396_amd import dpara as D
from paper_2609_27396_amd import synth

MODELS = {"tiny": synth.TINY, "8b": synth.QWEN3_8B, "14b": synth.QWEN3_14B}
N_FEAT = 3  # target layers whose hidden states are fused
HEAD_KINDS = ("round", "serial", "sampled", "candidates")


def listed():
    return [
        # one whole greedy round of the small float32 drafter: launches and latency
        dict(name="round_tiny_f32", kind="round", model="tiny", batch=1, gamma=4, layers=1, ctx_min=128, ctx_max=128),
        # cache update after a round: the block rows' target features fused and appended
        dict(name="update_8b_b1", kind="update", model="8b", batch=1, gamma=16, layers=5, ctx_min=2048, ctx_max=2048,
             rows=17),
        # prompts of mixed length entering the cache
        dict(name="prefill_8b_b3", kind="update", model="8b", batch=3, gamma=16, layers=5, ctx_min=0, ctx_max=0,
             rows=1250),
        # the drafter's whole work of a round at batch 1 (append + five layers over 289 rows)
        dict(name="precompute_8b_b1", kind="precompute", model="8b", batch=1, gamma=16, layers=5, ctx_min=2048,
             ctx_max=2048, rows=17),
        # one drafter layer, a few requests
        dict(name="layer_8b_b3", kind="layer", model="8b", batch=3, gamma=16, layers=1, ctx_min=700, ctx_max=3000),
        # one drafter layer, full batch with mixed context lengths
        dict(name="layer_8b_b16", kind="layer", model="8b", batch=16, gamma=16, layers=1, ctx_min=512, ctx_max=4096),
        # one layer of the larger drafter over long contexts
        dict(name="layer_14b_b8", kind="layer", model="14b", batch=8, gamma=16, layers=1, ctx_min=8192, ctx_max=8192),
        # target verification of one request's block (four layers and the LM head)
        dict(name="target_8b_b1", kind="target", model="8b", batch=1, gamma=16, layers=4, ctx_min=2048, ctx_max=2048),
        # target verification of a few requests
        dict(name="target_8b_b6", kind="target", model="8b", batch=6, gamma=16, layers=4, ctx_min=600, ctx_max=3500),
        # the serial step of a round at batch 1
        dict(name="serial_8b_b1", kind="serial", model="8b", batch=1, gamma=16),
        # the serial step with sampling at temperature 1
        dict(name="sampled_8b_b8", kind="sampled", model="8b", batch=8, gamma=16),
        # head candidates of every branch off the serial path, then the short serial step
        dict(name="candidates_8b_b4", kind="candidates", model="8b", batch=4, gamma=16),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("round", "update", "update", "precompute", "layer", "layer", "layer", "target", "target",
                       "serial", "sampled", "candidates"))
    if kind == "round":
        n = _log_int(rng, 16, 512)
        return dict(kind=kind, model="tiny", batch=_log_int(rng, 1, 4), gamma=rng.randint(2, 8), layers=1,
                    ctx_min=n, ctx_max=n + rng.randint(0, 64))
    model = rng.choice(("8b", "8b", "14b"))
    gamma = rng.randint(3, 16)
    rows = (gamma + 1) ** 2
    # work that grows with rows or with the batch stays below the largest listed case
    top = {"layer": 2400, "precompute": 420, "candidates": 900}.get(kind)
    most = 16 if top is None else max(1, min(16, top // rows))
    batch = _log_int(rng, 1, most)
    case = dict(kind=kind, model=model, batch=batch, gamma=gamma)
    if kind in ("serial", "sampled", "candidates"):
        return case
    hi = _log_int(rng, 128, min(8192, 65536 // batch))
    lo = hi if rng.random() < 0.5 else max(64, int(hi * rng.uniform(0.15, 0.9)))
    case.update(layers={"layer": 1, "target": rng.randint(1, 4)}.get(kind, 5), ctx_min=lo, ctx_max=hi)
    if kind == "precompute":
        case["rows"] = gamma + 1
    if kind == "update":
        if rng.random() < 0.5:
            case["rows"] = gamma + 1
        else:
            case.update(rows=_log_int(rng, 40, 4000 // batch), ctx_min=0, ctx_max=0)
    return case


# ---------------------------------------------------------------- sizes
def _shape(case):
    return replace(MODELS[case["model"]], gamma=case["gamma"], n_layers=case.get("layers", 1))


def _spread(lo, hi, n):
    """n lengths over [lo, hi], the largest first."""
    return [hi - int((hi - lo) * ((b * 0.6180339887) % 1.0)) for b in range(n)]


def _lens(case):
    return _spread(case["ctx_min"], case["ctx_max"], case["batch"])


def _counts(case):
    """Rows appended per request."""
    return _spread(1, case["rows"], case["batch"])


def _layer_elems(s):
    return s.hidden * s.head_dim * (2 * s.n_q_heads + 2 * s.n_kv_heads) + 3 * s.hidden * s.ffn


def work(case):
    s, B, kind = _shape(case), case["batch"], case["kind"]
    g, H, V, L = s.gamma, s.hidden, s.vocab, s.n_layers
    esz = 4 if s.dtype == "f32" else 2
    kv = 2 * s.n_kv_heads * s.head_dim  # K and V entries of one position
    by = fl = 0.0

    def backbone(rows_per, pairs_in):
        M, ctx = B * rows_per, sum(_lens(case))
        b = L * (_layer_elems(s) + ctx * kv) * esz + M * H * esz
        f = L * (2.0 * M * _layer_elems(s) + 4.0 * s.n_q_heads * s.head_dim * (rows_per * ctx + B * pairs_in))
        return b, f

    def verify():
        return B * (g + 1) * V * (4 if s.dtype == "f32" else 2)

    tree = sum(j + 1 for j in range(g + 1)) + sum(g * (r + 1 + g) for r in range(g + 1))
    if kind in ("round", "precompute", "layer"):
        b, f = backbone((g + 1) ** 2, tree)
        by, fl = by + b + B * (g + 1) * g * H * 4, fl + f
    if kind == "target":
        b, f = backbone(g + 1, sum(j + 1 for j in range(g + 1)))
        M = B * (g + 1)
        by, fl = by + b + V * H * 2 + M * V * 2 + M * N_FEAT * H * 2, fl + f + 2.0 * M * V * H
    if kind in ("update", "precompute", "round"):
        n = sum(_counts(case)) if kind != "round" else B * (g + 1)
        by += n * H * esz + L * kv * (H + n) * esz
        fl += 2.0 * n * H * L * kv
    if kind == "update":
        n = B * case["rows"]
        by += (H * N_FEAT * H + n * N_FEAT * H + n * H) * esz
        fl += 2.0 * n * H * N_FEAT * H
    if kind in HEAD_KINDS:
        rows = B * g * (g + 1 if kind == "candidates" else 1)
        by += verify() + V * H * esz + rows * H * 4 + B * g * H * 4
        fl += 2.0 * rows * V * H
    if kind == "sampled":
        by += 2 * B * g * V * 4 + V * s.ar_rank * 2
        fl += 2.0 * B * g * V * s.ar_rank
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # About four times the error against 64 bits that the path shows.  Tokens and verdicts are
    # whole numbers from float32 logits: the same up to float32 ties.
    if case["kind"] == "round":  # float32 throughout: 2.7e-5 (margins)
        return {"rel": 1e-4, "max": 5e-3}
    if case["kind"] in HEAD_KINDS:  # float32 margins and scores over the vocabulary: 1.9e-5
        return {"rel": 8e-5, "max": 5e-3}
    # bf16: one projection 2.4e-3, a layer 5.1e-3, four or five layers 9e-3 to 1e-2
    return {"update": {"rel": 0.01, "max": 0.1}, "layer": {"rel": 0.02, "max": 0.2}}.get(
        case["kind"], {"rel": 0.03, "max": 0.3})


# ---------------------------------------------------------------- inputs
def _inputs(case, seed):
    """Plain device tensors of one case, from the seed alone."""
    s, B, kind = _shape(case), case["batch"], case["kind"]
    g, H, V, hd, F = s.gamma, s.hidden, s.vocab, s.head_dim, s.ffn
    nq, nkv, L = s.n_q_heads, s.n_kv_heads, s.n_layers
    dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape, std=1.0, mean=0.0, dtype=dt):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=gen)

    def gain(n):
        return normal(n, std=0.1, mean=1.0, dtype=torch.float32)

    w = {"embed": normal(V, H, std=0.02), "mask_emb": normal(H, std=0.02), "final_norm": gain(H),
         "ar_E": normal(V, s.ar_rank, std=0.02), "ar_W": normal(V, s.ar_rank, std=0.02)}
    x = {"w": w}
    if kind in ("round", "precompute", "layer", "update", "target"):
        for l in range(L):
            p = f"L{l}."
            w[p + "attn_norm"], w[p + "mlp_norm"], w[p + "q_norm"], w[p + "k_norm"] = gain(H), gain(H), gain(hd), gain(hd)
            for n, shp in (("wq", (nq * hd, H)), ("wk", (nkv * hd, H)), ("wv", (nkv * hd, H)), ("wo", (H, nq * hd)),
                           ("w_gate", (F, H)), ("w_up", (F, H)), ("w_down", (H, F))):
                w[p + n] = normal(*shp, std=0.02)
        lens = _lens(case)
        x["ctx_len"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
        cap = (max(lens) + case.get("rows", g + 1) + 63) // 64 * 64
        kv = (L, B, nkv)
        if kind == "update":  # a pass reads no earlier position
            x["k"] = torch.zeros(*kv, cap, hd, dtype=dt, device="cuda")
            x["v"] = torch.zeros(*kv, hd, cap, dtype=dt, device="cuda")
        else:  # keys of unit mean square after the k-norm, values of W_v f
            x["k"] = normal(*kv, cap, hd)
            x["v"] = normal(*kv, hd, cap, std=0.02 * math.sqrt(H))
    if kind == "target":
        w["lm_head"] = normal(V, H, std=0.02)
    if kind == "update":
        w["fc"], w["fc_norm"] = normal(H, N_FEAT * H, std=0.02), gain(H)
        x["hidden"] = normal(B * case["rows"], N_FEAT * H)
    if kind in ("update", "precompute"):
        x["n_new"] = torch.tensor(_counts(case), dtype=torch.int32, device="cuda")
    if kind == "precompute":
        x["feats"] = normal(B, case["rows"], H)
    if kind == "round":
        x["feats"] = normal(B, g + 1, H)
        x["n_new"] = torch.randint(1, g + 2, (B,), dtype=torch.int32, device="cuda", generator=gen)
    x["spine"] = torch.randint(0, V, (B, g + 1), dtype=torch.int32, device="cuda", generator=gen)
    if kind in ("serial", "sampled", "candidates"):
        x["reps"] = normal(B, g + 1, g, H, dtype=torch.float32)
    if kind in ("round", "serial", "candidates"):
        # greedy verdicts: accepted lengths ~ min(Geometric(0.2) - 1, gamma); the drafts up to the
        # first rejection are the rows' maxima, the rejecting row's maximum is the bonus
        lg = normal(B, g + 1, V)
        u = torch.rand(B, generator=gen, device="cuda").clamp(1e-6, 1 - 1e-6)
        acc = torch.clamp((torch.log(u) / math.log(0.8)).floor(), 0, g).long()
        alt = torch.randint(0, V, (B, g + 1), device="cuda", generator=gen)
        nxt = torch.cat([x["spine"][:, 1:].long(), alt[:, :1]], 1)
        alt = torch.where(alt == nxt, (alt + 1) % V, alt)
        tok = torch.where(torch.arange(g + 1, device="cuda")[None] < acc[:, None], nxt, alt)
        lg.scatter_(2, tok[..., None], lg.amax(2, keepdim=True) + 1)
        x["logits"] = lg
    if kind == "sampled":
        # drafts drawn from their scores; a target that agrees with them for the most part
        sc = normal(B, g, V, std=1.3, dtype=torch.float32)
        x["spine"][:, 1:] = torch.multinomial(torch.softmax(sc.view(B * g, V), -1), 1,
                                              generator=gen).view(B, g).int()
        x["scores"] = sc
        x["logits"] = (torch.cat([sc, normal(B, 1, V, dtype=torch.float32)], 1)
                       + normal(B, g + 1, V, std=0.5, dtype=torch.float32)).to(dt)
        x["seed"] = seed * 2654435761 % (1 << 62) + 1
    return x


class _Drafter(D.DeviceDrafter):
    """Drafter weights that are on the device already."""

    def __init__(self, shape, w):
        self.shape, self.cfg, self.device, self.t = shape, D.make_config(shape), "cuda", w
        self._layers = (D.DparaLayerWeights * shape.n_layers)()
        for l in range(shape.n_layers):
            for f, _ in D.DparaLayerWeights._fields_:
                setattr(self._layers[l], f, D._ptr(w.get(f"L{l}.{f}")))
        layers = ctypes.cast(self._layers, ctypes.POINTER(D.DparaLayerWeights))
        if "lm_head" in w:  # the target
            self.cfg.ar_rank = 64
            self.w = D.DparaTargetWeights(embed=D._ptr(w["embed"]), lm_head=D._ptr(w["lm_head"]),
                                          final_norm=D._ptr(w["final_norm"]), layers=layers)
        else:
            self.w = D.DparaWeights(embed=D._ptr(w["embed"]), mask_emb=D._ptr(w["mask_emb"]),
                                    final_norm=D._ptr(w["final_norm"]), ar_E=D._ptr(w["ar_E"]),
                                    ar_W=D._ptr(w["ar_W"]), layers=layers)


class _Fusion:
    def __init__(self, shape, w):
        self.cfg, self.fc, self.norm = D.make_config(shape), w["fc"], w["fc_norm"]
        self.w = D.DparaFusionWeights(fc=D._ptr(self.fc), norm=D._ptr(self.norm), n_feat=N_FEAT)


class _State:
    pass


def prepare(case, seed):
    s, B, kind = _shape(case), case["batch"], case["kind"]
    g, H, V = s.gamma, s.hidden, s.vocab
    x = _inputs(case, seed)
    st = _State()
    st.kind, st.x = kind, x
    st.d = _Drafter(s, x["w"])
    cap = 64
    if "k" in x:
        cap = int(x["k"].shape[3])
        st.ctx = D.DeviceContext(s, B, cap)
        st.ctx.k.copy_(x["k"])
        st.ctx.v.copy_(x["v"])
        st.ctx.ctx_len.copy_(x["ctx_len"])
        del x["k"], x["v"]
    st.ws = D.Workspace(st.d.cfg, B, cap, target=kind == "target")
    i32 = dict(dtype=torch.int32, device="cuda")
    f32 = dict(dtype=torch.float32, device="cuda")
    if kind in ("round", "precompute", "layer"):
        st.reps = torch.empty((B, g + 1, g, H), **f32)
    if kind in ("serial", "sampled", "candidates"):
        st.reps = x["reps"]
    if kind in HEAD_KINDS:
        st.accept, st.bonus = torch.empty(B, **i32), torch.empty(B, **i32)
        st.argmax = torch.empty((B, g + 1), **i32)
        st.gathered = torch.empty((B, g, H), **f32)
        st.drafts, st.next_spine = torch.empty((B, g), **i32), torch.empty((B, g + 1), **i32)
        st.margins = torch.empty((B, g), **f32)
        st.d.prepare_head(st.ws)  # weight constants, once per drafter
        if s.dtype == "bf16":
            st.d.prepare_candidates(st.ws)
    if kind == "sampled":
        st.new_scores = torch.empty((B, g, V), **f32)
    if kind == "candidates":
        st.cand = D.branch_candidates_buffer(st.d, B)
    if kind == "target":
        st.logits = torch.empty((B, g + 1, V), dtype=torch.bfloat16, device="cuda")
        st.hidden = torch.empty((B, g + 1, N_FEAT, H), dtype=torch.bfloat16, device="cuda")
        st.feat_layers = [0, (s.n_layers - 1) // 2, s.n_layers - 1]
    if kind == "update":
        st.f = _Fusion(s, x["w"])
        n = B * case["rows"]
        st.fws = torch.empty(D.dpara_fuse_workspace_bytes(st.f.cfg, n, N_FEAT), dtype=torch.uint8, device="cuda")
        st.feats = torch.empty((B, case["rows"], H), dtype=st.d.mat_dtype, device="cuda")
    return st


def run(st):
    x, d, ws, kind = st.x, st.d, st.ws, st.kind
    if kind == "update":
        st.ctx.ctx_len.copy_(x["ctx_len"])
        D.fuse_features(st.f, x["hidden"], st.feats, st.fws)
        D.ctx_append(d, st.ctx, st.feats, x["n_new"], ws)
        return {"feats": st.feats, "k": st.ctx.k, "v": st.ctx.v, "ctx_len": st.ctx.ctx_len}
    if kind == "target":
        D.target_forward_hidden(d, st.ctx, x["spine"], st.logits, st.feat_layers, st.hidden, ws)
        return {"logits": st.logits, "hidden": st.hidden}
    out = {}
    if kind in ("round", "precompute"):
        st.ctx.ctx_len.copy_(x["ctx_len"])
        D.ctx_append(d, st.ctx, x["feats"], x["n_new"], ws)
        out.update(k=st.ctx.k, v=st.ctx.v, ctx_len=st.ctx.ctx_len)
    if kind in ("round", "precompute", "layer"):
        D.backbone_all_boundaries(d, st.ctx, x["spine"], st.reps, ws)
        out["reps"] = st.reps
    if kind in ("precompute", "layer"):
        return out
    if kind == "candidates":
        D.branch_candidates(d, st.reps, st.cand, ws)
    out.update(accept=st.accept, bonus=st.bonus, gathered=st.gathered, drafts=st.drafts, next_spine=st.next_spine,
               margins=st.margins)
    if kind == "sampled":
        D.verify_sampled(d, x["logits"], x["scores"], x["spine"], 1.0, x["seed"], st.accept, st.bonus, ws)
        D.select_and_head_sampled(d, st.reps, st.accept, st.bonus, st.gathered, st.drafts, st.next_spine, st.margins,
                                  1.0, x["seed"] + 1, st.new_scores, ws)
        out["scores"] = st.new_scores
        return out
    D.verify_greedy(d, x["logits"], x["spine"], st.accept, st.bonus, st.argmax, ws)
    out["argmax"] = st.argmax
    if kind == "candidates":
        D.select_and_head_cand(d, st.reps, st.cand, st.accept, st.bonus, st.gathered, st.drafts, st.next_spine,
                               st.margins, ws)
    else:
        D.select_and_head(d, st.reps, st.accept, st.bonus, st.gathered, st.drafts, st.next_spine, st.margins, ws)
    return out


# ---------------------------------------------------------------- the same in 64 bits
def _norm(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _mm(x, w):
    """x w^T in 64 bits, the weight converted a few rows at a time."""
    n = max(1, (1 << 28) // w.shape[1])
    return torch.cat([x @ c.double().T for c in w.split(n)], -1)


def _rope(x, pos, base):
    """x [n, heads, hd] at positions pos [n]."""
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * base ** (-torch.arange(half, device=x.device).double() / half)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _append64(s, x, feats):
    """The caches after the append of feats [B, n, H], in 64 bits."""
    w, hd, nkv = x["w"], s.head_dim, s.n_kv_heads
    K, Vc = x["k"].double(), x["v"].double()
    lens, cnt = x["ctx_len"].tolist(), x["n_new"].tolist()
    for b, (n0, n) in enumerate(zip(lens, cnt)):
        f = feats[b, :n].double()
        pos = torch.arange(n0, n0 + n, device=f.device)
        for l in range(s.n_layers):
            k = _mm(f, w[f"L{l}.wk"]).view(n, nkv, hd)
            if s.qk_norm:
                k = _norm(k, w[f"L{l}.k_norm"], s.rms_eps)
            K[l, b, :, n0:n0 + n] = _rope(k, pos, s.rope_base).permute(1, 0, 2)
            Vc[l, b, :, :, n0:n0 + n] = _mm(f, w[f"L{l}.wv"]).view(n, nkv, hd).permute(1, 2, 0)
    return K, Vc, x["ctx_len"] + x["n_new"]


def _block_layout(g, causal):
    """Position offsets [R] and in-block visibility [R, R] of a request's block rows."""
    if causal:
        return torch.arange(g + 1), torch.ones(g + 1, g + 1).tril().bool()
    R = (g + 1) ** 2
    off, vis = torch.zeros(R, dtype=torch.long), torch.zeros(R, R, dtype=torch.bool)
    for j in range(g + 1):
        off[j] = j
        vis[j, :j + 1] = True
    for r in range(g + 1):
        m = g + 1 + r * g
        off[m:m + g] = r + 1 + torch.arange(g)
        vis[m:m + g, :r + 1] = True
        vis[m:m + g, m:m + g] = True
    return off, vis


def _decoder64(s, x, K, Vc, lens, causal, emit=()):
    """Residual stream [B, R, H] after every layer's pass over the block rows, and the
    residuals after the layers in `emit`."""
    w, hd, nq, nkv, B = x["w"], s.head_dim, s.n_q_heads, s.n_kv_heads, len(lens)
    off, vis = _block_layout(s.gamma, causal)
    R, dev = len(off), K.device
    vis = vis.to(dev)
    X = w["mask_emb"].double().expand(B, R, s.hidden).clone()
    X[:, :s.gamma + 1] = w["embed"][x["spine"].long()].double()
    pos = torch.tensor(lens, device=dev)[:, None] + off.to(dev)[None]
    seen = {}
    for l in range(s.n_layers):
        p = f"L{l}."
        a = _norm(X, w[p + "attn_norm"], s.rms_eps).view(B * R, -1)
        q = _mm(a, w[p + "wq"]).view(B * R, nq, hd)
        k = _mm(a, w[p + "wk"]).view(B * R, nkv, hd)
        v = _mm(a, w[p + "wv"]).view(B, R, nkv, hd)
        if s.qk_norm:
            q, k = _norm(q, w[p + "q_norm"], s.rms_eps), _norm(k, w[p + "k_norm"], s.rms_eps)
        q = _rope(q, pos.reshape(-1), s.rope_base).view(B, R, nq, hd)
        k = _rope(k, pos.reshape(-1), s.rope_base).view(B, R, nkv, hd)
        o = torch.empty(B, R, nq, hd, dtype=torch.float64, device=dev)
        grp = nq // nkv
        for b in range(B):
            ok = torch.cat([torch.ones(R, lens[b], dtype=torch.bool, device=dev), vis], 1)
            for h in range(nkv):
                keys = torch.cat([K[l, b, h, :lens[b]].double(), k[b, :, h]])
                vals = torch.cat([Vc[l, b, h, :, :lens[b]].double().T, v[b, :, h]])
                for j in range(h * grp, (h + 1) * grp):
                    sc = (q[b, :, j] @ keys.T / math.sqrt(hd)).masked_fill(~ok, -math.inf)
                    o[b, :, j] = torch.softmax(sc, -1) @ vals
        X = X + _mm(o.view(B * R, nq * hd), w[p + "wo"]).view(B, R, -1)
        m = _norm(X, w[p + "mlp_norm"], s.rms_eps).view(B * R, -1)
        hid = torch.nn.functional.silu(_mm(m, w[p + "w_gate"])) * _mm(m, w[p + "w_up"])
        X = X + _mm(hid, w[p + "w_down"]).view(B, R, -1)
        if l in emit:
            seen[l] = X
    return X, seen


def _uniform(seed, tag, b, i, v):
    """U of the library's documented generator: Philox4x32-10 (Salmon et al., SC 2011), counter
    (v, i, b, tag), the top 23 bits of word 0; v an int64 tensor."""
    M = 0xFFFFFFFF
    k0, k1 = seed & M, seed >> 32

    def mul(c, x):  # high and low words of the 32 x 32-bit product
        lo, hi = c * (x & 0xFFFF), c * (x >> 16)
        t = lo + ((hi & 0xFFFF) << 16)
        return (hi >> 16) + (t >> 32), t & M

    c = [v, torch.full_like(v, i), torch.full_like(v, b), torch.full_like(v, tag)]
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return (2 * (c[0] >> 9) + 1).double() / (1 << 24)


def _gumbel(seed, tag, b, i, v):
    return -torch.log(-torch.log(_uniform(seed, tag, b, i, v)))


def _head64(s, w, gathered, bonus, seed=None):
    """Drafts, next block, margins and scores of the AR head over gathered [B, g, H]."""
    B, g = gathered.shape[:2]
    drafts = torch.empty(B, g, dtype=torch.int32, device="cuda")
    margins = torch.empty(B, g, dtype=torch.float64, device="cuda")
    scores = torch.empty(B, g, s.vocab, dtype=torch.float64, device="cuda")
    ids = torch.arange(s.vocab, device="cuda")
    W = w["ar_W"].double()
    for b in range(B):
        base = _mm(gathered[b].double(), w["embed"])
        y = int(bonus[b])
        for i in range(g):
            z = base[i] + W @ w["ar_E"][y].double()
            scores[b, i] = z
            if seed is not None:
                z = z + _gumbel(seed, 1, b, i + 1, ids)
            top = torch.topk(z, 2)
            y = int(top.indices[0])
            drafts[b, i], margins[b, i] = y, top.values[0] - top.values[1]
    nxt = torch.cat([torch.as_tensor(bonus, dtype=torch.int32, device="cuda").view(B, 1), drafts], 1)
    return drafts, nxt, margins, scores


def exact(case, seed):
    s, B, kind = _shape(case), case["batch"], case["kind"]
    g = s.gamma
    x = _inputs(case, seed)
    w = x["w"]
    if kind == "update":
        f = _norm(_mm(x["hidden"].double(), w["fc"]), w["fc_norm"], s.rms_eps).view(B, case["rows"], -1)
        K, Vc, n = _append64(s, x, f)
        return {"feats": f, "k": K, "v": Vc, "ctx_len": n}
    if kind == "target":
        emit = [0, (s.n_layers - 1) // 2, s.n_layers - 1]
        X, seen = _decoder64(s, x, x["k"], x["v"], _lens(case), True, emit)
        y = _norm(X, w["final_norm"], s.rms_eps).view(B * (g + 1), -1)
        return {"logits": _mm(y, w["lm_head"]).view(B, g + 1, -1), "hidden": torch.stack([seen[l] for l in emit], 2)}
    out = {}
    if kind in ("round", "precompute"):
        x["k"], x["v"], x["ctx_len"] = _append64(s, x, x["feats"])
        out.update(k=x["k"], v=x["v"], ctx_len=x["ctx_len"])
    if kind in ("round", "precompute", "layer"):
        X, _ = _decoder64(s, x, x["k"], x["v"], x["ctx_len"].tolist(), False)
        reps = _norm(X[:, g + 1:], w["final_norm"], s.rms_eps).view(B, g + 1, g, -1)
        out["reps"] = reps
    if kind in ("precompute", "layer"):
        return out
    reps = reps if kind == "round" else x["reps"]
    spine = x["spine"]
    if kind == "sampled":
        lp, lq = (torch.log_softmax(x[n].double(), -1) for n in ("logits", "scores"))
        accept = torch.zeros(B, dtype=torch.int32, device="cuda")
        bonus = torch.zeros(B, dtype=torch.int32, device="cuda")
        ids, zero = torch.arange(s.vocab, device="cuda"), torch.zeros(1, dtype=torch.long, device="cuda")
        for b in range(B):
            r = 0
            while r < g:
                t = int(spine[b, r + 1])
                if float(torch.log(_uniform(x["seed"], 2, b, r + 1, zero))) >= float(lp[b, r, t] - lq[b, r, t]):
                    break
                r += 1
            p = lp[b, r] if r == g else torch.log(torch.clamp(lp[b, r].exp() - lq[b, r].exp(), min=0))
            accept[b], bonus[b] = r, int(torch.argmax(p + _gumbel(x["seed"], 3, b, 0, ids)))
    else:
        top = torch.argmax(x["logits"].double(), -1).int()
        accept = (top[:, :-1] == spine[:, 1:]).int().cumprod(1).sum(1).int()
        bonus = top.gather(1, accept.long()[:, None])[:, 0]
        out["argmax"] = top
    gathered = reps[torch.arange(B, device="cuda"), accept.long()]
    drafts, nxt, margins, scores = _head64(s, w, gathered, bonus, x["seed"] + 1 if kind == "sampled" else None)
    out.update(accept=accept, bonus=bonus, gathered=gathered.double(), drafts=drafts, next_spine=nxt, margins=margins)
    if kind == "sampled":
        out["scores"] = scores
    return out
