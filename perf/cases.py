"""The calls that users of this library make most, as a fixed set of measured cases.

listed() names them, draw() gives more of the same ranges, prepare() makes what a program
holds before the call (weights, handle, caches, inputs, all from the seed), run() is one
call, exact() is what it computes, in plain float64 torch.

Models are the shapes of paper_2606_09514_amd.synth with fewer blocks (one case has all 32):
a block's work does not depend on how many there are, and small models fit the card several
times.  Cached rows are N(0, 1); a routable block's row is zero where the earlier token
skipped the block, with the share of skipped rows that the budgets give.
"""
import math

import torch

from paper_2606_09514_amd import lib as blib
from paper_2606_09514_amd import synth

# budgets of a mixed batch as shares of the routable blocks (12, 18, 24, 30 of 30)
MIXED = (0.4, 0.6, 0.8, 1.0)
PREDICTOR_HIDDEN = 256


def _case(name, call, shape, layers, batch, ctx, **kw):
    c = dict(name=name, call=call, shape=shape, layers=layers, dtype="bf16", batch=batch, ctx=ctx,
             ragged=False, share=0.5, mixed=False, masked=False, running=False, router_ctx="kv", start=1)
    c.update(kw)
    if not name:
        del c["name"]
    return c


def listed():
    return [
        # whole-model decode of one conversation, the benchmark's headline workload (k = 15 of 30)
        _case("decode_8b_one", "decode", "llama3_8b", 32, 1, 2048),
        # one conversation with a long history (a document in the context)
        _case("decode_8b_long", "decode", "llama3_8b", 8, 1, 30011),
        # a few conversations at different lengths, budgets from the Budget Predictor
        _case("decode_7b_few", "auto", "qwen2_7b", 8, 3, 1500, ragged=True),
        # a small serving batch, mixed budgets, skipped rows masked out of the attention
        _case("decode_8b_small_batch", "decode", "llama3_8b", 8, 11, 1700, ragged=True, mixed=True, masked=True),
        # the batched serving workloads: mixed budgets at equal lengths, GQA and MHA
        _case("decode_8b_batch", "decode", "llama3_8b", 8, 32, 4096, mixed=True),
        _case("decode_13b_batch", "decode", "mha_13b", 4, 96, 2048, mixed=True),
        # a chat-sized prompt
        _case("prefill_8b_short", "prefill", "llama3_8b", 8, 1, 197),
        # the benchmark's prompt
        _case("prefill_8b_2048", "prefill", "llama3_8b", 8, 1, 2048),
        # prompts of different lengths and budgets admitted together
        _case("prefill_7b_ragged", "prefill", "qwen2_7b", 6, 5, 900, ragged=True, mixed=True),
        # planner scores of a batch without a handle (a scheduler that routes ahead)
        _case("planner_8b_batch", "planner", "llama3_8b", 32, 24, 3000, ragged=True),
        # the parity-sized fp32 decoder: latency of a step of tiny kernels
        _case("decode_tiny_f32", "decode", "tiny", 8, 4, 64, dtype="f32"),
        # scheduler calls on a batch's scores: top-k routes, then groups of equal routes
        _case("route_groups", "group", "llama3_8b", 32, 200, 0, mixed=True),
    ]


def draw(rng):
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    call = rng.choice(["decode"] * 4 + ["auto"] + ["prefill"] * 3 + ["planner", "group"])
    shape = rng.choice(["llama3_8b", "llama3_8b", "qwen2_7b", "mha_13b", "tiny"])
    s = synth.SHAPES[shape]
    kw = dict(ragged=rng.random() < 0.6, mixed=rng.random() < 0.5, share=rng.choice([0.3, 0.5, 0.75, 1.0]),
              router_ctx=rng.choice(["kv", "kv", "v"]))
    if shape == "tiny" and rng.random() < 0.5:
        kw["dtype"] = "f32"
    if call == "group":
        return _case("", call, "llama3_8b", rng.randint(12, 80), log_int(8, 1000), 0, mixed=kw["mixed"], share=kw["share"])
    layers = s["n_layers"] if shape == "tiny" or call == "planner" else rng.randint(4, 8)
    if call == "prefill":
        batch = log_int(1, 8)
        ctx = log_int(24, 2048)
        if shape == "mha_13b":
            layers = 4
        ctx = min(ctx, 2048 // batch) if shape != "tiny" else min(ctx, 512 // batch)
        kw["masked"] = rng.random() < 0.3
        return _case("", call, shape, layers, batch, ctx, **kw)
    batch = 1 if rng.random() < 0.25 else log_int(2, 96)
    # cached rows of the whole batch, limited to those of the largest listed case
    row = layers * s["n_kv_heads"] * s["head_dim"]
    most = 4 * 40 * 128 * 96 * 2048 // (row * batch)
    ctx = log_int(16, max(17, min(32000, most)))
    if call == "planner":
        ctx = min(ctx, 4000)
    else:
        kw["masked"] = rng.random() < 0.25
        kw["running"] = not kw["masked"] and rng.random() < 0.15
        kw["start"] = 2 if rng.random() < 0.15 else 1
    return _case("", call, shape, layers, batch, ctx, **kw)


# ------------------------------------------------------------------ inputs


def _cfg(case):
    shape = dict(synth.SHAPES[case["shape"]], n_layers=case["layers"])
    # a cache of whole 64-row pages with room for the answer
    c = synth.model_config(shape, case["dtype"], (case["ctx"] + 64) // 64 * 64 + 64)
    c["router_ctx"] = case["router_ctx"]
    c["start_layer"] = case["start"]
    return c


def _lengths(case, gen):
    """Cached rows (decode) or prompt lengths: all ctx, or from a quarter of it up to it."""
    B, ctx = case["batch"], case["ctx"]
    if not case["ragged"]:
        return [ctx] * B
    lens = [max(1, int(ctx * (0.25 + 0.75 * (b + 1) / B))) for b in range(B)]
    return [lens[i] for i in torch.randperm(B, generator=gen).tolist()]


def _budgets(case, Lm, gen):
    B = case["batch"]
    if not case["mixed"]:
        return [round(case["share"] * Lm)] * B
    ks = [round(MIXED[b % len(MIXED)] * Lm) for b in range(B)]
    return [ks[i] for i in torch.randperm(B, generator=gen).tolist()]


def _mean_share(case):
    return sum(MIXED) / len(MIXED) if case["mixed"] else case["share"]


def _inputs(case, seed):
    """The tensors and host lists of a case, from the seed alone."""
    cfg = _cfg(case)
    L, B, Lm, S = cfg["n_layers"], case["batch"], synth.n_mid(cfg), case["start"]
    gen = torch.Generator().manual_seed(seed)
    dev = torch.Generator(device="cuda").manual_seed(seed + 1)
    s = dict(cfg=cfg, lens=_lengths(case, gen) if case["ctx"] else None, ks=_budgets(case, Lm, gen))
    if case["call"] == "group":
        # scores of the same few prompts' families: equal routes occur
        base = torch.randn((max(1, B // 4), Lm), generator=dev, device="cuda")
        s["scores"] = base[torch.randint(0, base.shape[0], (B,), generator=dev, device="cuda")].contiguous()
        return s
    planner = case["call"] == "planner"
    if not planner:
        W = synth.model_weights(cfg, seed, "cuda")
    else:   # the planner reads no block weights
        H, din = cfg["dm_hidden"], synth.context_dim(cfg)
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        w1, b1, w2, b2 = ((torch.randn(n, generator=dev, device="cuda") * 0.02).to(dt)
                          for n in ((H, din), (H,), (Lm, H), (Lm,)))
        W = dict(layers=[], dm=dict(w1=w1, b1=b1, w2=w2, b2=b2, omega=0.1,
                                    prior=torch.randn(Lm, generator=dev, device="cuda")))
    s["W"] = W
    if case["call"] == "prefill":
        s["k"], s["v"] = synth.kv_cache(cfg, B, 0, seed + 2, "cuda")
        s["x"] = torch.randn((B, max(s["lens"]), cfg["d_model"]), generator=dev, device="cuda")
    else:
        s["k"], s["v"] = synth.kv_cache(cfg, B, max(s["lens"]), seed + 2, "cuda")
        s["x"] = torch.randn((B, cfg["d_model"]), generator=dev, device="cuda")
    T = cfg["max_ctx"]
    if case["call"] != "prefill":
        # which blocks earlier tokens ran: all of them in the always-run blocks
        ran = torch.rand((L, B, T), generator=dev, device="cuda") < _mean_share(case)
        ran[:S] = True
        ran[L - 1] = True
        for l in range(S, L - 1):
            keep = ran[l].view(B, 1, T, 1)
            s["k"][l].mul_(keep)
            s["v"][l].mul_(keep)
        if case["masked"]:
            s["exec"] = ran.to(torch.uint8)
    elif case["masked"]:
        s["exec"] = torch.zeros((L, B, T), dtype=torch.uint8, device="cuda")
    if case["call"] == "auto":
        s["pred"] = synth.predictor_weights(cfg, PREDICTOR_HIDDEN, seed + 3, "cuda")
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    B, Lm = case["batch"], synth.n_mid(s["cfg"])
    u8 = dict(dtype=torch.uint8, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    s["mask"] = torch.zeros((B, Lm), **u8)
    s["out_scores"] = torch.zeros((B, Lm), device="cuda")
    if case["call"] == "group":
        s["perm"], s["starts"], s["n"] = torch.zeros(B, **i32), torch.zeros(B + 1, **i32), torch.zeros(1, **i32)
        return s
    if case["call"] == "planner":
        return s
    s["model"] = blib.Model(s["cfg"], s["W"], max_batch=B)
    s["hidden"] = torch.empty_like(s["x"])
    if case["running"]:
        s["pool"] = s["model"].pool_state()
    if case["call"] == "auto":
        s["model"].set_budget_predictor(s["pred"])
        s["k_out"] = torch.zeros(B, **i32)
    return s


# --------------------------------------------------------------------- run


def run(s):
    case = s["case"]
    call = case["call"]
    if call == "group":
        blib.select_topk(s["scores"], s["ks"], s["mask"])
        blib.group_by_route(s["mask"], s["perm"], s["starts"], s["n"])
        return {"mask": s["mask"], "perm": s["perm"], "starts": s["starts"], "n": s["n"]}
    if call == "planner":
        blib.pool_route_noalloc(s["cfg"], s["W"]["dm"], case["batch"], s["k"], s["v"], s["lens"], s["x"], s["out_scores"])
        return {"scores": s["out_scores"]}
    # the call overwrites its input rows (the new tokens' embeddings) with its output
    s["hidden"].copy_(s["x"])
    out = {"hidden": s["hidden"], "mask": s["mask"], "scores": s["out_scores"], "k": s["k"], "v": s["v"]}
    opt = dict(mask_out=s["mask"], scores_out=s["out_scores"], exec_map=s.get("exec"),
               skip_kv=blib.SKIP_KV_MASK if case["masked"] else blib.SKIP_KV_ZERO, pool=s.get("pool"))
    if call == "prefill":
        s["model"].prefill(s["k"], s["v"], s["hidden"], s["lens"], s["ks"], **opt)
    elif call == "auto":
        s["model"].decode_step_auto(s["k"], s["v"], s["hidden"], s["lens"], k_out=s["k_out"], **opt)
        out["budget"] = s["k_out"]
    else:
        s["model"].decode_step(s["k"], s["v"], s["hidden"], s["lens"], s["ks"], **opt)
    if case["masked"]:
        out["exec"] = s["exec"]
    if case["running"]:
        out["pool_sum"], out["pool_rows"] = s["pool"]
    return out


# -------------------------------------------------------------------- work


def work(case):
    """Bytes: weights of the blocks some sequence runs, cached rows attended, rows written,
    inputs and outputs, once each.  Operations: the projections and both attention products."""
    cfg = _cfg(case)
    B, Lm, S = case["batch"], synth.n_mid(cfg), case["start"]
    if case["call"] == "group":
        return {"bytes": B * Lm * 5 + 4 * (2 * B + 2), "flops": B * Lm * Lm}
    es = 2 if case["dtype"] == "bf16" else 4
    d, hd, nq, nkv, f = cfg["d_model"], cfg["head_dim"], cfg["n_heads"], cfg["n_kv_heads"], cfg["d_ffn"]
    lens = _lengths(case, torch.Generator().manual_seed(0))
    rows = B if case["call"] != "prefill" else sum(lens)
    row = nkv * hd * es
    dm = cfg["dm_hidden"] * (synth.context_dim(cfg) + Lm)
    by = dm * es + rows * d * 8
    fl = 2 * B * dm
    attended = sum(n + 1 for n in lens)
    if case["call"] == "planner":
        return {"bytes": by - rows * d * 4 + 2 * attended * row, "flops": fl + 2 * attended * nkv * hd}
    weights = d * (nq + 2 * nkv) * hd + d * nq * hd + 3 * d * f
    share = round(_mean_share(case) * Lm) / max(Lm, 1)
    run_blocks = S + 1 + share * Lm
    blocks = S + 1 + Lm * (1 - (1 - share) ** B)
    by += blocks * weights * es + 2 * cfg["n_layers"] * rows * row
    fl += 2 * run_blocks * rows * weights
    if case["call"] == "prefill":
        return {"bytes": by, "flops": fl + 4 * run_blocks * sum(n * (n + 1) // 2 for n in lens) * nq * hd}
    return {"bytes": by + 2 * run_blocks * attended * row, "flops": fl + 4 * run_blocks * attended * nq * hd}


def tolerance(case):
    if case["call"] == "group":
        return "exact"
    if case["dtype"] == "f32" or case["call"] == "planner":
        return {"rel": 1e-5, "max": 1e-3}
    # bf16 activations: up to 9e-3 from float64 over 5 blocks
    if case["call"] == "prefill":
        return {"rel": 2e-2, "max": 0.5}
    # 1e-6 (fp32 activations) to 4e-5 (16-bit parts) from float64; a new K/V value next to a
    # rounding boundary moves by one bf16 step, which "max" allows
    return {"rel": 2e-4, "max": 0.05}


# ------------------------------------------------------------------- exact


def _rms(h, gain, eps):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, pos, theta):
    """x [n][heads][hd], pos [n]: rotate-half pairs at angle pos theta^(-2i/hd)."""
    half = x.shape[-1] // 2
    inv = theta ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / x.shape[-1])
    a = pos.double()[:, None, None] * inv
    c, s = a.cos(), a.sin()
    x0, x1 = x[..., :half], x[..., half:]
    return torch.cat([x0 * c - x1 * s, x1 * c + x0 * s], -1)


def _block(s, l, h, b, pos, exec_l):
    """Block l over rows h of sequence b at positions pos (consecutive); writes the cache."""
    cfg, lw = s["cfg"], s["W"]["layers"][l]
    d, hd, nq, nkv = cfg["d_model"], cfg["head_dim"], cfg["n_heads"], cfg["n_kv_heads"]
    n, p0 = h.shape[0], int(pos[0])
    kc, vc = s["k"][l, b], s["v"][l, b]
    y = _rms(h, lw["attn_norm"], cfg["rms_eps"]) @ s["wd"]["wqkv"].T
    q, k, v = y.split([nq * hd, nkv * hd, nkv * hd], -1)
    q = _rope(q.view(n, nq, hd), pos, cfg["rope_theta"])
    kc[:, p0:p0 + n] = _rope(k.view(n, nkv, hd), pos, cfg["rope_theta"]).transpose(0, 1).to(kc.dtype)
    vc[:, p0:p0 + n] = v.view(n, nkv, hd).transpose(0, 1).to(vc.dtype)
    end = p0 + n
    dead = torch.arange(end, device=h.device)[None, :] > pos[:, None]
    if exec_l is not None:
        dead = dead | ((exec_l[b, :end] == 0)[None, :] & (torch.arange(end, device=h.device)[None, :] != pos[:, None]))
    o = torch.empty((n, nq, hd), dtype=torch.float64, device=h.device)
    G = nq // nkv
    for g in range(nkv):
        K, V = kc[g, :end].double(), vc[g, :end].double()
        sc = q[:, g * G:(g + 1) * G].reshape(n * G, hd) @ K.T.contiguous() / math.sqrt(hd)
        sc = sc.view(n, G, end).masked_fill(dead[:, None, :], -math.inf)
        o[:, g * G:(g + 1) * G] = (torch.softmax(sc, -1).view(n * G, end) @ V).view(n, G, hd)
    h = h + o.view(n, nq * hd) @ s["wd"]["wo"].T
    gu = _rms(h, lw["mlp_norm"], cfg["rms_eps"]) @ s["wd"]["wgate_up"].T
    gate, up = gu.chunk(2, -1)
    return h + (torch.nn.functional.silu(gate) * up) @ s["wd"]["wdown"].T


def _mlp(z, w, act):
    y = z @ w["w1"].double().T + w["b1"].double()
    y = torch.nn.functional.gelu(y) if act == "gelu" else torch.nn.functional.silu(y)
    return y @ w["w2"].double().T + w["b2"].double()


def _scores(s, h_last, ends):
    """Router context and fused scores: means of block S-1's rows 0..end, then the hidden row."""
    cfg, dm = s["cfg"], s["W"]["dm"]
    l = cfg["start_layer"] - 1
    z = []
    for b, e in enumerate(ends):
        mk = s["k"][l, b, :, :e + 1].double().mean(1).reshape(-1)
        mv = s["v"][l, b, :, :e + 1].double().mean(1).reshape(-1)
        z.append(torch.cat(([mk, mv] if cfg["router_ctx"] == "kv" else [mv]) + [h_last[b]]))
    z = torch.stack(z)
    sc = _mlp(z, dm, cfg["dm_act"])
    if dm.get("prior") is not None:
        sc = sc + dm["omega"] * dm["prior"].double()
    return z, sc


def exact(case, seed):
    if case["call"] == "group":
        return None
    s = _inputs(case, seed)
    cfg, B, S, L = s["cfg"], case["batch"], case["start"], case["layers"]
    Lm = synth.n_mid(cfg)
    lens = s["lens"]
    if case["call"] == "planner":
        return {"scores": _scores(s, s["x"].double(), lens)[1]}
    prefill = case["call"] == "prefill"
    if prefill:
        pos = [torch.arange(n, device="cuda") for n in lens]
        hs = [s["x"][b, :lens[b]].double() for b in range(B)]
    else:
        pos = [torch.tensor([n], device="cuda") for n in lens]
        hs = [s["x"][b:b + 1].double() for b in range(B)]
    ex = s.get("exec") if not prefill else None
    mask = torch.zeros((B, Lm), dtype=torch.uint8, device="cuda")
    scores, ks = None, s["ks"]
    for l in range(L):
        if l == S:
            z, scores = _scores(s, torch.stack([h[-1] for h in hs]), [n - 1 for n in lens] if prefill else lens)
            if case["call"] == "auto":
                ks = (_mlp(z, s["pred"], cfg["dm_act"]).argmax(-1) + 1).tolist()
            order = torch.sort(scores, dim=-1, descending=True, stable=True).indices
            for b in range(B):
                mask[b, order[b, :ks[b]]] = 1
            chosen = mask.cpu()
        s["wd"] = {n: s["W"]["layers"][l][n].double() for n in ("wqkv", "wo", "wgate_up", "wdown")}
        for b in range(B):
            if S <= l < L - 1 and not chosen[b, l - S]:
                p0 = int(pos[b][0])
                s["k"][l, b, :, p0:p0 + len(pos[b])] = 0
                s["v"][l, b, :, p0:p0 + len(pos[b])] = 0
                continue
            hs[b] = _block(s, l, hs[b], b, pos[b], ex[l] if ex is not None else None)
    # the caches hold values rounded to storage: they have no 64-bit value
    if prefill:
        hidden = s["x"].double()
        for b in range(B):
            hidden[b, :lens[b]] = hs[b]
    else:
        hidden = torch.cat(hs)
    out = {"hidden": hidden, "mask": mask, "scores": scores, "k": None, "v": None}
    if case["call"] == "auto":
        out["budget"] = torch.tensor(ks, dtype=torch.int32, device="cuda")
    if case["masked"]:
        out["exec"] = None
    if case["running"]:
        out["pool_sum"] = out["pool_rows"] = None
    return out
