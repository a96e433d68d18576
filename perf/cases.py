"""The work whose speed is measured: calls that a user of this library makes.

The library decodes with a draft / target pair behind one context: a prompt
forward, then lookahead steps (rollout by the draft, verification by the
target, reward, selection, commit), Alg. 1's step from the prefix, and single
kernels behind their own entry points (a projection, the LM head with its row
statistics, the rows of speculative sampling).  Kinds of case:

  request     what a caller that serves one request does: prefill, whole
              lookahead steps with their commits, and the handle given back
  step        one lookahead step over a batch, up to the selection (the
              rollout, the verification, the linear reward, the argmax)
  rollout     the draft rollout that keeps its logits (speculative sampling)
  alg1        Alg. 1's draft and verification from the prefix: one sequence
              per prompt, so few rows per pass
  prefill     the prompt forward of both models, then the verification of a
              given continuation on the new prefix
  gemm        one projection (weights bf16 or fp32, activations fp32)
  head        the LM head reduced to argmax, top-k and log-probs
  logit_rows  the same reduction on logits that are in memory
  soft_rows   speculative sampling's row kernel

Weights are random, scaled as a freshly initialised residual network (the
residual branches by 1 / sqrt(2 layers)), with a successor for every token
written into the LM head: next-token distributions are then peaked as a
trained model's are, draft and target agree on most tokens, and no greedy
choice hangs on the last bits of a sum.
"""
import math

import numpy as np
import torch

import cdsl_inputs as ci
from paper_2412_10418_amd import binding
from paper_2412_10418_amd.engine import Engine

DEV = "cuda"

# (layers, d_model, heads, kv heads, ffn, vocab) of draft and target, weight type
_1B, _7B = (16, 2048, 32, 8, 8192), (32, 4096, 32, 32, 11008)
PAIRS = {
    "tiny": ((2, 128, 4, 4, 512, 1024), (4, 256, 8, 8, 1024, 1024), "f32"),
    "small": ((12, 1024, 16, 16, 4096, 32000), (24, 2048, 16, 16, 5632, 32000), "bf16"),
    "7b1b": (_1B + (32000,), _7B + (32000,), "bf16"),
    "long": (_1B + (128256,), (32, 4096, 32, 8, 11008, 128256), "bf16"),
}
# how strongly the LM head holds a token's successor: the logit that it adds
# is this times the share of the embedding in the final hidden state
LINK = {"tiny": 8.5, "small": 13.0, "7b1b": 22.0, "long": 22.0}
# (N, K) of the projections of those models: q/k/v, o, gate/up, down
PROJECTIONS = [(3072, 1024), (1024, 1024), (1024, 4096), (6144, 2048), (2048, 2048), (11264, 2048), (2048, 5632),
               (3072, 2048), (16384, 2048), (2048, 8192), (12288, 4096), (6144, 4096), (4096, 4096), (22016, 4096),
               (4096, 11008)]
EPS, THETA, STEPS = 1e-5, 10000.0, 2


def listed():
    return [
        # one prompt on the fp32 plumbing pair: nothing but latency and launches
        {"name": "tiny_request", "kind": "request", "pair": "tiny", "B": 1, "L": 32, "k": 4, "d": 4},
        # a served batch on the small bf16 pair, commits included
        {"name": "small_request", "kind": "request", "pair": "small", "B": 8, "L": 128, "k": 5, "d": 5},
        # the library's main workload: 16 prompts, five beams of ten tokens
        {"name": "step_7b1b", "kind": "step", "pair": "7b1b", "B": 16, "L": 256, "k": 5, "d": 10},
        # long prompts, grouped-query target, large vocabulary
        {"name": "step_long", "kind": "step", "pair": "long", "B": 16, "L": 2048, "k": 8, "d": 4},
        # more draft rows than the decode projections take (k = 10 of the sweep)
        {"name": "rollout_wide", "kind": "rollout", "pair": "7b1b", "B": 16, "L": 512, "k": 10, "d": 5},
        # Alg. 1: one drafted sequence per prompt, ragged prompt length
        {"name": "alg1_7b1b", "kind": "alg1", "pair": "7b1b", "B": 16, "L": 301, "k": 5, "d": 5},
        # prompt forward of the main workload
        {"name": "prefill_7b1b", "kind": "prefill", "pair": "7b1b", "B": 16, "L": 256, "k": 2, "d": 3},
        # one draft projection at the rollout's rows
        {"name": "gemm_decode", "kind": "gemm", "M": 80, "N": 2048, "K": 8192, "dtype": "bf16"},
        # the target's q/k/v projection at the verification's rows
        {"name": "gemm_verify", "kind": "gemm", "M": 800, "N": 12288, "K": 4096, "dtype": "bf16"},
        # the verification's LM head
        {"name": "head_verify", "kind": "head", "M": 800, "V": 32000, "K": 4096, "kk": 5},
        # logits kept in memory (speculative sampling's heads), ragged vocabulary
        {"name": "logit_rows", "kind": "logit_rows", "M": 512, "V": 50257, "kk": 5},
        # speculative sampling over the verified rows
        {"name": "soft_rows", "kind": "soft_rows", "G": 80, "d": 10, "V": 32000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["request", "request", "step", "step", "rollout", "alg1", "prefill", "gemm", "gemm", "gemm",
                       "head", "logit_rows", "soft_rows"])
    if kind == "gemm":
        if rng.random() < 0.2:   # fp32 weights: the plumbing pair's range
            return {"kind": kind, "M": _log_int(rng, 1, 512), "N": rng.randint(33, 2048),
                    "K": 16 * rng.randint(8, 64), "dtype": "f32"}
        N, K = rng.choice(PROJECTIONS)
        if rng.random() < 0.4:   # sizes that no tile divides
            N, K = _log_int(rng, 200, 20000), 32 * rng.randint(20, 350)
        return {"kind": kind, "M": _log_int(rng, 1, 2048), "N": N, "K": K, "dtype": "bf16"}
    if kind == "head":
        V = rng.choice([32000, 50257, 128256])
        return {"kind": kind, "M": _log_int(rng, 1, 1000), "V": V, "K": rng.choice([1024, 2048, 4096]),
                "kk": rng.randint(0, 8)}
    if kind == "logit_rows":
        return {"kind": kind, "M": _log_int(rng, 1, 1000), "V": _log_int(rng, 1000, 128256), "kk": rng.randint(0, 10)}
    if kind == "soft_rows":
        d = rng.randint(1, 12)
        return {"kind": kind, "G": _log_int(rng, 1, max(2, 900 // d)), "d": d, "V": _log_int(rng, 1000, 128256)}
    if kind == "request":
        if rng.random() < 0.4:
            return {"kind": kind, "pair": "tiny", "B": rng.randint(1, 4), "L": rng.randint(5, 64),
                    "k": rng.randint(1, 6), "d": rng.randint(1, 8)}
        return {"kind": kind, "pair": "small", "B": rng.randint(1, 12), "L": _log_int(rng, 16, 256),
                "k": rng.randint(2, 6), "d": rng.randint(2, 8)}
    pair = rng.choice(["small", "7b1b", "7b1b"] + (["long"] if kind == "step" else []))
    B, L = _log_int(rng, 1, 24), _log_int(rng, 24, 640)
    if pair == "long":
        B, L = rng.randint(2, 12), _log_int(rng, 500, 2048)
    if kind == "prefill":
        return {"kind": kind, "pair": pair, "B": min(B, max(1, 4000 // L)), "L": L, "k": rng.randint(1, 4),
                "d": rng.randint(1, 4)}
    if kind == "alg1":
        return {"kind": kind, "pair": pair, "B": B, "L": L, "k": rng.randint(1, 8), "d": rng.randint(2, 10)}
    k, d = rng.randint(1, 10), rng.randint(1, 12)
    if kind == "rollout":
        return {"kind": kind, "pair": pair, "B": B, "L": L, "k": k, "d": min(d, 6)}
    while B * k * d > 800:
        B, d = max(1, B - 1), max(1, d - 1)
    return {"kind": kind, "pair": pair, "B": B, "L": L, "k": k, "d": d}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, *what):
    x = (int(seed) & 0xFFFFFFFF) * 1000003
    for w in what:
        x = (x * 69069 + w + 1) % (1 << 62)
    return torch.Generator(device=DEV).manual_seed(x)


def _weights(pair, which, seed):
    """One model's weights as the binding takes them (which: 0 draft, 1 target).  Token t's successor is
    _successors(...)[t], the same for both models."""
    shape, dtype = PAIRS[pair][which], PAIRS[pair][2]
    n, D, H, Hkv, F, V = shape
    hd = D // H
    g = _gen(seed, 1, which)
    wt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def mat(r, c, std):
        return torch.empty((r, c), dtype=wt, device=DEV).normal_(0.0, std, generator=g)

    def gain():
        return 1.0 + 0.1 * torch.randn(D, generator=g, device=DEV)

    res = 0.02 / math.sqrt(2.0 * n)
    layers = [{"attn_norm": gain(), "wq": mat(H * hd, D, 0.02), "wk": mat(Hkv * hd, D, 0.02),
               "wv": mat(Hkv * hd, D, 0.02), "wo": mat(D, H * hd, res), "mlp_norm": gain(),
               "w_gate": mat(F, D, 0.02), "w_up": mat(F, D, 0.02), "w_down": mat(D, F, res)} for _ in range(n)]
    emb = mat(V, D, 1.0)
    lm = mat(V, D, 0.02)
    lm[_successors(V, seed)] += (emb.float() * (LINK[pair] / D)).to(wt)
    return {"tok_emb": emb, "layers": layers, "final_norm": gain(), "lm_head": lm}


def _successors(V, seed):
    return torch.randperm(V, generator=_gen(seed, 2), device=DEV)


def _prompts(case, seed):
    V = PAIRS[case["pair"]][0][5]
    return torch.randint(0, V, (case["B"], case["L"]), generator=_gen(seed, 3), device=DEV, dtype=torch.int32)


def _lookaheads(case, seed, stray=0.1):
    """[B, k, d + 1]: a token and its chain of successors, with a stray token now and then."""
    B, k, d, V = case["B"], case["k"], case["d"], PAIRS[case["pair"]][0][5]
    succ, g = _successors(V, seed), _gen(seed, 4)
    out = [torch.randint(0, V, (B, k), generator=g, device=DEV)]
    for _ in range(d):
        nxt = succ[out[-1]]
        odd = torch.rand(nxt.shape, generator=g, device=DEV) < stray
        out.append(torch.where(odd, torch.randint(0, V, nxt.shape, generator=g, device=DEV), nxt))
    return torch.stack(out, -1).int().contiguous()


def _beams(case, seed):
    """k different beam heads per prompt, the prompt's successor among them, and their log-probs."""
    B, k, V = case["B"], case["k"], PAIRS[case["pair"]][0][5]
    g = _gen(seed, 6)
    beams = torch.rand((B, V), generator=g, device=DEV).topk(k, -1).indices
    beams[:, 0] = _successors(V, seed)[_prompts(case, seed)[:, -1].long()]
    head_lp = -8.0 * torch.rand((B, k), generator=g, device=DEV)
    return beams.int().contiguous(), head_lp


def _keywords(case, seed):
    """Four distinct words per prompt: two that its greedy continuation has, two that it has not."""
    V = PAIRS[case["pair"]][0][5]
    succ = _successors(V, seed)
    t = _prompts(case, seed)[:, -1].long()
    out = []
    for _ in range(2):
        t = succ[t]
        out.append(t)
    r = torch.randint(0, V - 4, (t.shape[0],), generator=_gen(seed, 7), device=DEV)
    for i in range(2):
        r = r + 1
        for _ in range(2):
            r = torch.where((r == out[0]) | (r == out[1]), r + 1, r)
        out.append(r)
    return torch.stack(out, -1).int().contiguous()


def _workload(case):
    ds, ts, dtype = PAIRS[case["pair"]]
    shape = lambda s: ci.ModelShape(*s, rope_theta=THETA, rms_eps=EPS)  # noqa: E731
    kind = "keyword_count" if case["pair"] == "tiny" else "keyword_coverage"
    return ci.Workload(case["pair"], shape(ds), shape(ts), dtype, batch=case["B"], prompt_len=case["L"], k=case["k"],
                       d=case["d"], steps=STEPS, reward="linear" if case["kind"] in ("step", "prefill") else kind)


def _logits(rows, V, seed, what):
    """Peaked logits: normal, standard deviation 3, one of each row's tokens raised."""
    g = _gen(seed, 8, what)
    z = torch.randn((rows, V), generator=g, device=DEV) * 3.0
    z[torch.arange(rows, device=DEV), torch.randint(0, V, (rows,), generator=g, device=DEV)] += 12.0
    return z


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "gemm":
        g = _gen(seed, 9)
        s["A"] = torch.randn((case["M"], case["K"]), generator=g, device=DEV)
        s["W"] = torch.empty((case["N"], case["K"]), device=DEV,
                             dtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32)
        s["W"].normal_(0.0, 0.02, generator=g)
        s["C"] = torch.zeros((case["M"], case["N"]), device=DEV)
        return s
    if kind == "head":
        g = _gen(seed, 10)
        s["A"] = torch.randn((case["M"], case["K"]), generator=g, device=DEV)
        s["W"] = torch.empty((case["V"], case["K"]), dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
        s["gather"] = torch.randint(0, case["V"], (case["M"],), generator=g, device=DEV, dtype=torch.int32)
        return s
    if kind == "logit_rows":
        s["logits"] = _logits(case["M"], case["V"], seed, 0)
        s["gather"] = torch.randint(0, case["V"], (case["M"],), generator=_gen(seed, 11), device=DEV,
                                    dtype=torch.int32)
        return s
    if kind == "soft_rows":
        G, d, V = case["G"], case["d"], case["V"]
        s["p"] = _logits(G * d, V, seed, 1)
        s["q"] = 0.9 * s["p"] + 0.4 * _logits(G * d, V, seed, 2)
        look = torch.zeros((G, d + 1), dtype=torch.int32, device=DEV)
        look[:, 1:] = s["q"].argmax(-1).view(G, d).int()
        s["look"] = look
        # each uniform is moved to the middle of the interval that it falls in (of one that is not narrower than
        # 1e-5), so that no draw is decided by the last bits of a cumulative sum
        w = (s["p"].double().softmax(-1) - s["q"].double().softmax(-1)).clamp_min(0.0)
        cum = w.cumsum(-1)
        wide = torch.where(w >= 1e-5 * cum[:, -1:], w, torch.zeros_like(w)).cumsum(-1)
        u = torch.rand((G * d, 1), generator=_gen(seed, 12), device=DEV, dtype=torch.float64) * wide[:, -1:]
        at = torch.searchsorted(wide, u, right=True).clamp_max(V - 1)
        mid = cum.gather(-1, at) - 0.5 * w.gather(-1, at)
        s["v"] = (mid / cum[:, -1:]).clamp(0.0, 0.9999999).float().view(-1).contiguous()
        return s
    wl = _workload(case)
    B, L, k, d = case["B"], case["L"], case["k"], case["d"]
    s["eng"] = eng = Engine(wl, _weights(case["pair"], 0, seed), _weights(case["pair"], 1, seed), max_steps=STEPS + 1, device=DEV)
    s["prompts"] = _prompts(case, seed)
    if kind == "request":
        s["keywords"] = _keywords(case, seed)
        return s
    if kind == "prefill":
        s["look"] = _lookaheads(case, seed)
        s["head_lp"] = _beams(case, seed)[1]
        s["out"] = eng.buffers(B, k, d)
        return s
    s["prefix"] = eng.start(s["prompts"]).prefix
    if kind == "alg1":
        s["buf"] = eng._controller_buffers(B, k, d)
        s["keywords"] = _keywords(case, seed)
        return s
    s["beams"], s["head_lp"] = _beams(case, seed)
    if kind == "rollout":
        V = wl.draft.vocab
        s["look"] = torch.zeros((B, k, d + 1), dtype=torch.int32, device=DEV)
        s["logits"] = torch.zeros((B, k, d, V), device=DEV)
        return s
    s["buf"] = eng.buffers(B, k, d)
    s["reward_w"] = 0.02 * torch.randn(wl.target.d_model, generator=_gen(seed, 13), device=DEV)
    return s


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "gemm":
        return binding.cdsl_op_gemm(s["A"], s["W"], s["C"])
    if kind == "head":
        lp, amax, ids, tlp = binding.cdsl_op_lm_head_rows(s["A"], s["W"], s["gather"], case["kk"])
        return {"lp": lp, "amax": amax, "ids": ids, "topk_lp": tlp}
    if kind == "logit_rows":
        lp, amax, ids, tlp = binding.cdsl_op_logit_rows(s["logits"], s["gather"], case["kk"])
        return {"lp": lp, "amax": amax, "ids": ids, "topk_lp": tlp}
    if kind == "soft_rows":
        dlp, rid, rlp = binding.cdsl_op_soft_rows(s["p"], s["q"], case["d"], s["look"], s["v"])
        return {"draft_lp": dlp, "res_ids": rid, "res_lp": rlp}
    eng, k, d = s["eng"], case["k"], case["d"]
    c = eng.ctx
    if kind == "request":
        st = eng.start(s["prompts"])
        heads = st.head_lp.clone()
        for _ in range(STEPS):
            bf = eng.step(st, keywords=s["keywords"])
        st.prefix.free()
        emitted = np.full((case["B"], STEPS * (d + 1)), -1, np.int64)
        for b, e in enumerate(st.emitted):
            emitted[b, :len(e)] = e
        return {"first_heads": heads, "lookaheads": bf.lookaheads, "verify": bf.verify, "reward": bf.reward,
                "beam": bf.beam, "beams": st.beams, "head_lp": st.head_lp, "emitted": emitted}
    if kind == "prefill":
        prefix, beams, head_lp = c.cdsl_prefill(s["prompts"], k)
        v = c.cdsl_verify(prefix, s["look"], k, d, s["head_lp"], out=s["out"].verify)
        prefix.free()
        return {"beams": beams, "head_lp": head_lp, "verify": v}
    if kind == "alg1":
        bf = s["buf"]
        c.cdsl_draft_prefix(s["prefix"], d, bf["look"])
        c.cdsl_verify_prefix(s["prefix"], bf["look"], d, k, bf["verify"])
        c.cdsl_reward_keywords_prefix(s["prefix"], bf["look"], d, bf["verify"]["n_accept"], s["keywords"], True,
                                      bf["reward"])
        return {"lookaheads": bf["look"], "verify": bf["verify"], "reward": bf["reward"]}
    if kind == "rollout":
        c.cdsl_rollout_keep(s["prefix"], s["beams"], k, d, s["look"], s["logits"])
        return {"lookaheads": s["look"], "logits": s["logits"]}
    bf = s["buf"]
    c.cdsl_rollout(s["prefix"], s["beams"], k, d, bf.lookaheads)
    c.cdsl_verify(s["prefix"], bf.lookaheads, k, d, s["head_lp"], out=bf.verify)
    c.cdsl_reward_linear(bf.verify["hidden"], s["reward_w"], bf.reward)
    c.cdsl_select(bf.verify["scores"], bf.reward, 1.0, bf.beam)
    return {"lookaheads": bf.lookaheads, "verify": bf.verify, "reward": bf.reward, "beam": bf.beam}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _params(shape):
    n, D, H, Hkv, F, V = shape
    hd = D // H
    return n * (2 * D * H * hd + 2 * D * Hkv * hd + 3 * D * F), V * D   # layers, head


def _pass_work(shape, wbytes, rows, head_rows, prefix_tokens, suffix_tokens, pairs):
    """One forward pass: weights once, the KV that its rows see once (fp32), the new KV written once."""
    n, D, H, Hkv, F, V = shape
    hd = D // H
    body, head = _params(shape)
    kv = n * 2 * Hkv * hd * 4
    return {"bytes": (body + (head if head_rows else 0)) * wbytes + (prefix_tokens + suffix_tokens + rows) * kv
            + rows * D * wbytes,
            "flops": 2.0 * rows * body + 2.0 * head_rows * head + 4.0 * n * H * hd * pairs}


def _add(*ws):
    return {"bytes": float(sum(w["bytes"] for w in ws)), "flops": float(sum(w["flops"] for w in ws))}


def _rollout_work(shape, wb, B, L, k, d):
    return _add(*[_pass_work(shape, wb, B * k, B * k, B * L, B * k * j, B * k * (L + j + 1)) for j in range(d)])


def _verify_work(shape, wb, B, L, k, d):
    return _pass_work(shape, wb, B * k * d, B * k * d, B * L, 0, B * k * (d * L + d * (d + 1) // 2))


def _prefill_work(ds, ts, wb, B, L):
    pairs = B * (L * (L + 1) // 2)
    return _add(_pass_work(ds, wb, B * L, 0, 0, 0, pairs), _pass_work(ts, wb, B * L, B, 0, 0, pairs))


def work(case):
    kind = case["kind"]
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": M * K * 4.0 + N * K * (2.0 if case["dtype"] == "bf16" else 4.0) + M * N * 4.0,
                "flops": 2.0 * M * N * K}
    if kind == "head":
        M, V, K = case["M"], case["V"], case["K"]
        return {"bytes": M * K * 4.0 + V * K * 2.0 + M * (3 + 2 * case["kk"]) * 4.0, "flops": 2.0 * M * V * K}
    if kind == "logit_rows":
        return {"bytes": case["M"] * (case["V"] + 3 + 2 * case["kk"]) * 4.0, "flops": 0.0}
    if kind == "soft_rows":
        return {"bytes": case["G"] * case["d"] * (2 * case["V"] + 5) * 4.0, "flops": 0.0}
    ds, ts, dtype = PAIRS[case["pair"]]
    wb = 2 if dtype == "bf16" else 4
    B, L, k, d = case["B"], case["L"], case["k"], case["d"]
    if kind == "request":
        steps = [_add(_rollout_work(ds, wb, B, L, k, d), _verify_work(ts, wb, B, L, k, d))] * STEPS
        return _add(_prefill_work(ds, ts, wb, B, L), *steps)
    if kind == "prefill":
        return _add(_prefill_work(ds, ts, wb, B, L), _verify_work(ts, wb, B, L, k, d))
    if kind == "alg1":
        return _add(_rollout_work(ds, wb, B, L, 1, d), _verify_work(ts, wb, B, L, 1, d))
    if kind == "rollout":
        w = _rollout_work(ds, wb, B, L, k, d)
        return _add(w, {"bytes": B * k * d * ds[5] * 4.0, "flops": 0.0})
    return _add(_rollout_work(ds, wb, B, L, k, d), _verify_work(ts, wb, B, L, k, d))


def tolerance(case):
    """About four times the error that was seen against float64, or with the sums in another order."""
    kind = case["kind"]
    if kind == "gemm":
        return {"rel": 1e-5}
    if kind == "head":   # near ties among a row's top tokens
        return {"rel": 3e-6, "differ": 0.003}
    if kind in ("logit_rows", "soft_rows"):
        return {"rel": 1e-6, "differ": 0.0}
    if case["pair"] == "tiny":
        return {"rel": 1e-5, "differ": 0.01}
    return {"rel": 5e-5, "differ": 0.01}


# ---------------------------------------------------------------------------
# the same in 64 bits, with plain torch
# ---------------------------------------------------------------------------
class _Model:
    """A Llama-style decoder in float64, over [B, k, T] tokens that extend a prefix cache shared by the k beams."""

    def __init__(self, shape, w):
        self.n, self.D, self.H, self.Hkv, self.F, self.V = shape
        self.hd, self.w = self.D // self.H, w

    @staticmethod
    def norm(x, g):
        return x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * g.double()

    def rope(self, x, pos):
        half = self.hd // 2
        inv = THETA ** (-(torch.arange(half, device=DEV, dtype=torch.float64) * 2.0) / self.hd)
        a = pos.double()[:, None] * inv
        c, s = a.cos()[:, None, :], a.sin()[:, None, :]
        x1, x2 = x[..., :half], x[..., half:]
        return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)

    def attend(self, q, pre, own, T):
        """q [k, T, H, hd] of one prompt; pre: K, V [L, Hkv, hd]; own: K, V [k, S, Hkv, hd], the last T slots q's own."""
        k, G, S = q.shape[0], self.H // self.Hkv, own[0].shape[1]
        qh = q.reshape(k, T, self.Hkv, G, self.hd).permute(0, 2, 3, 1, 4) / math.sqrt(self.hd)   # k, Hkv, G, T, hd
        qh = qh.reshape(k, self.Hkv, G * T, self.hd)
        ko, vo = (x.permute(0, 2, 1, 3).contiguous() for x in own)                               # k, Hkv, S, hd
        so = torch.matmul(qh, ko.transpose(-1, -2).contiguous())
        row = torch.arange(T, device=DEV).repeat(G) + (S - T)
        so = so.masked_fill(torch.arange(S, device=DEV)[None, :] > row[:, None], -math.inf)
        kp, vp = (x.permute(1, 0, 2).contiguous() for x in pre)                                  # Hkv, L, hd
        sp = torch.matmul(qh, kp.transpose(-1, -2).contiguous())
        a = torch.cat([sp, so], -1).softmax(-1)
        L = kp.shape[1]
        o = torch.matmul(a[..., :L].contiguous(), vp) + torch.matmul(a[..., L:].contiguous(), vo)
        return o.reshape(k, self.Hkv, G, T, self.hd).permute(0, 3, 1, 2, 4).reshape(k, T, self.H * self.hd)

    def extend(self, tok, L, pre, own=None):
        """Normed hidden states [B, k, T, D] of tok [B, k, T] and the layers' caches with these tokens added."""
        B, k, T = tok.shape
        j0 = 0 if own is None else own[0][0].shape[2]
        pos = L + j0 + torch.arange(T, device=DEV)
        x = self.w["tok_emb"][tok.long()].double()
        new = []
        for l in range(self.n):
            w = self.w["layers"][l]
            m = lambda u, name: torch.matmul(u, w[name].double().t())  # noqa: E731
            u = self.norm(x, w["attn_norm"])
            q = self.rope(m(u, "wq").reshape(B * k, T, self.H, self.hd), pos).reshape(B, k, T, self.H, self.hd)
            kk = self.rope(m(u, "wk").reshape(B * k, T, self.Hkv, self.hd), pos).reshape(B, k, T, self.Hkv, self.hd)
            vv = m(u, "wv").reshape(B, k, T, self.Hkv, self.hd)
            if own is not None:
                kk, vv = torch.cat([own[l][0], kk], 2), torch.cat([own[l][1], vv], 2)
            new.append((kk, vv))
            o = torch.stack([self.attend(q[b], (pre[l][0][b], pre[l][1][b]), (kk[b], vv[b]), T) for b in range(B)])
            x = x + m(o, "wo")
            u = self.norm(x, w["mlp_norm"])
            x = x + m(torch.nn.functional.silu(m(u, "w_gate")) * m(u, "w_up"), "w_down")
        return self.norm(x, self.w["final_norm"]), new

    def prefix(self, tokens):
        """The cache over tokens [B, L], and the last position's hidden state [B, D]."""
        B = tokens.shape[0]
        none = torch.zeros((B, 0, self.Hkv, self.hd), dtype=torch.float64, device=DEV)
        h, new = self.extend(tokens[:, None], 0, [(none, none)] * self.n)
        return [(a[:, 0], b[:, 0]) for a, b in new], h[:, 0, -1]

    def logits(self, h):
        return torch.matmul(h, self.w["lm_head"].double().t())


def _cut(cache, n):
    return [(a[:, :n], b[:, :n]) for a, b in cache]


def _exact_rollout(model, cache, L, first, d):
    toks, zs, own = [first.long()], [], None
    for _ in range(d):
        h, own = model.extend(toks[-1][..., None], L, cache, own)
        zs.append(model.logits(h[:, :, 0]))
        toks.append(zs[-1].argmax(-1))
    return torch.stack(toks, -1), torch.stack(zs, 2)


def _exact_verify(model, cache, L, look, kk, head_lp):
    h, _ = model.extend(look[..., :-1], L, cache)
    lsm = model.logits(h).log_softmax(-1)
    lp = lsm.gather(-1, look[..., 1:, None].long())[..., 0]
    top = lsm.topk(kk, -1)
    keep = (lsm.argmax(-1) == look[..., 1:]).int().cumprod(-1).sum(-1)
    return {"logprobs": lp, "target_argmax": None, "n_accept": None, "scores": lp.sum(-1) + head_lp,
            "row_topk_ids": None, "row_topk_lp": top.values, "hidden": h[:, :, -1]}, keep, top


def _floats(v):
    return {a: b for a, b in v.items() if a != "hidden"}


def _exact_request(case, seed, draft, target):
    k, d = case["k"], case["d"]
    prompts, kws = _prompts(case, seed), _keywords(case, seed)
    got = []
    for b in range(case["B"]):
        seq, gen, first = prompts[b:b + 1].long(), [], None
        heads = None
        for _ in range(STEPS):
            L = seq.shape[1]
            dc, _ = draft.prefix(seq)
            tc, h = target.prefix(seq)
            if heads is None:
                heads = first = tuple(target.logits(h).log_softmax(-1).topk(k, -1))
            look, _ = _exact_rollout(draft, dc, L, heads[1], d)
            ver, keep, top = _exact_verify(target, tc, L, look, k, heads[0])
            reward = torch.zeros((1, k), dtype=torch.float64, device=DEV)
            for i in range(k):
                seen = set(gen) | set(look[0, i].tolist())
                reward[0, i] = sum(w in seen for w in kws[b].tolist())
            if case["pair"] != "tiny":
                reward /= 4
            beam = int((ver["scores"] + reward)[0].argmax())
            n = int(keep[0, beam])
            gen += look[0, beam, :n + 1].tolist()
            seq = torch.cat([seq, look[:, beam, :n + 1]], 1)
            if n < d:
                heads = top.values[:, beam, n], top.indices[:, beam, n]
            else:
                heads = tuple(target.logits(target.prefix(seq)[1]).log_softmax(-1).topk(k, -1))
        got.append({"first_heads": first[0], "verify": ver, "reward": reward, "head_lp": heads[0]})
    cat = lambda name: torch.cat([g[name] for g in got])  # noqa: E731
    return {"first_heads": cat("first_heads"), "lookaheads": None, "reward": cat("reward"), "head_lp": cat("head_lp"),
            "verify": {a: None if got[0]["verify"][a] is None else torch.cat([g["verify"][a] for g in got])
                       for a in _floats(got[0]["verify"])}, "beam": None, "beams": None, "emitted": None}


@torch.no_grad()
def exact(case, seed):
    kind = case["kind"]
    if kind in ("gemm", "head", "logit_rows", "soft_rows"):
        s = prepare(case, seed)
        if kind == "gemm":
            return torch.matmul(s["A"].double(), s["W"].double().t())
        if kind == "soft_rows":
            G, d, V = case["G"], case["d"], case["V"]
            p, q = s["p"].double().log_softmax(-1), s["q"].double().log_softmax(-1)
            w = (p.exp() - q.exp()).clamp_min(0.0)
            cum = w.cumsum(-1)
            t = torch.searchsorted(cum, s["v"].double()[:, None] * cum[:, -1:], right=True).clamp_max(V - 1)
            return {"draft_lp": q.gather(-1, s["look"][:, 1:].reshape(-1, 1).long())[:, 0], "res_ids": None,
                    "res_lp": p.gather(-1, t)[:, 0]}
        z = s["logits"].double() if kind == "logit_rows" else torch.matmul(s["A"].double(), s["W"].double().t())
        lsm = z.log_softmax(-1)
        return {"lp": lsm.gather(-1, s["gather"].long()[:, None])[:, 0], "amax": None, "ids": None,
                "topk_lp": lsm.topk(case["kk"], -1).values if case["kk"] else None}
    ds, ts, dtype = PAIRS[case["pair"]]
    B, L, k, d = case["B"], case["L"], case["k"], case["d"]
    if _prefill_work(ds, ts, 2, B, L)["flops"] + work(case)["flops"] > 6e14:
        return None   # too long in 64 bits
    draft, target = (_Model(PAIRS[case["pair"]][i], _weights(case["pair"], i, seed)) for i in (0, 1))
    if kind == "request":
        return _exact_request(case, seed, draft, target)
    prompts = _prompts(case, seed)
    if kind == "prefill":
        tc, h = target.prefix(prompts)
        ver, _, _ = _exact_verify(target, tc, L, _lookaheads(case, seed), k, _beams(case, seed)[1])
        return {"beams": None, "head_lp": target.logits(h).log_softmax(-1).topk(k, -1).values, "verify": ver}
    dc, _ = draft.prefix(prompts)
    if kind == "alg1":
        look, _ = _exact_rollout(draft, _cut(dc, L - 1), L - 1, prompts[:, -1:], d)
        tc, _ = target.prefix(prompts)
        ver, keep, _ = _exact_verify(target, _cut(tc, L - 1), L - 1, look, k, 0.0)
        kws = _keywords(case, seed)
        hit = [[any(w == t for t in look[b, 0, 1:1 + int(keep[b, 0])].tolist()) for w in kws[b].tolist()]
               for b in range(B)]
        ver = {a: None if v is None else v[:, 0] for a, v in _floats(ver).items()}
        return {"lookaheads": None, "verify": ver, "reward": torch.tensor(hit, device=DEV).double().mean(-1)}
    beams, head_lp = _beams(case, seed)
    look, z = _exact_rollout(draft, dc, L, beams, d)
    if kind == "rollout":
        return {"lookaheads": None, "logits": z}
    del dc
    tc, _ = target.prefix(prompts)
    ver, _, _ = _exact_verify(target, tc, L, look, k, head_lp)
    w = 0.02 * torch.randn(ts[1], generator=_gen(seed, 13), device=DEV)
    return {"lookaheads": None, "verify": ver, "reward": torch.matmul(ver["hidden"], w.double()), "beam": None}
