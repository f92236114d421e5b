"""Performance cases of the rollout engine: what a user of the C ABI's Python binding has it do.

Every case goes through `Engine` (rl_decode.py): generation steps, prefill + generation, scoring and
sampling.  The model widths are those of the package's workloads.  Most cases run a few layers of such a
model behind a small vocabulary, so that the layers themselves are what is measured; two run the whole
vocabulary, one of them over the whole model.  Sequence lengths come from the case alone; weights, K/V,
logits and token ids come from the seed.
"""
import math
import random
from dataclasses import replace

import numpy as np
import torch

from paper_2509_15965_amd import configs
from paper_2509_15965_amd.inputs import make_weights
from paper_2509_15965_amd.rl_decode import Engine

MODELS = {"tiny": configs.TINY, "1.5b": configs.QWEN_1_5B, "llama7b": configs.LLAMA2_7B, "7b": configs.QWEN_7B,
          "32b": configs.QWEN_32B, "moe": configs.QWEN3_MOE}
DEV = "cuda"


def listed():
    return [
        # the reference decoder in fp32, start to end: two prompts of 32 tokens with four samples each
        dict(name="tiny_fp32_rollout", kind="rollout", model="tiny", layers=2, vocab=4096, prompts=2, group=4,
             plen_lo=32, plen_hi=32, patches=0, steps=4, page=0, temp=1.0),
        # sampling from logits a caller holds (a serving loop with its own head), 64 rows
        dict(name="sample_64", kind="sample", rows=64, vocab=151936, temp=0.6),
        # the last response of a batch: one row through a whole 1.5B model, head and sampler included
        dict(name="decode_1.5b_last_row", kind="decode", model="1.5b", layers=28, vocab=151936, rows=1, ctx_lo=900,
             ctx_hi=900, page=0, temp=1.0),
        # the long tail of a 7B rollout: a few long responses left
        dict(name="decode_7b_tail", kind="decode", model="7b", layers=4, vocab=4096, rows=11, ctx_lo=1500,
             ctx_hi=4500, page=0, temp=1.0),
        # the middle of a 7B rollout
        dict(name="decode_7b_mid", kind="decode", model="7b", layers=4, vocab=4096, rows=101, ctx_lo=600,
             ctx_hi=3400, page=0, temp=0.6),
        # the full 7B batch
        dict(name="decode_7b_batch", kind="decode", model="7b", layers=4, vocab=4096, rows=512, ctx_lo=400,
             ctx_hi=1600, page=0, temp=1.0),
        # a 32B rollout's batch at half its length
        dict(name="decode_32b", kind="decode", model="32b", layers=2, vocab=4096, rows=48, ctx_lo=1000,
             ctx_hi=6000, page=0, temp=1.0),
        # a mixture of experts in the middle of its rollout, on a paged pool
        dict(name="decode_moe_mid", kind="decode", model="moe", layers=2, vocab=4096, rows=131, ctx_lo=300,
             ctx_hi=1300, page=256, temp=1.0),
        # the start of a GRPO rollout: ragged prompts, 16 samples each, first steps over the shared prompts
        dict(name="grpo_start_7b", kind="rollout", model="7b", layers=2, vocab=4096, prompts=8, group=16, plen_lo=256,
             plen_hi=1024, patches=0, steps=4, page=256, temp=1.0),
        # an embodied policy's environment step: image patches + instruction, then action tokens
        dict(name="embodied_env_step", kind="rollout", model="llama7b", layers=2, vocab=32000, prompts=32, group=1,
             plen_lo=288, plen_hi=288, patches=256, steps=3, page=0, temp=1.0),
        # the inference stage over one GRPO group, whole vocabulary
        dict(name="score_7b_group", kind="score", model="7b", layers=2, vocab=152064, prompts=1, group=16,
             plen_lo=640, plen_hi=640, rlen=1100, temp=1.0),
        # the inference stage of a mixture of experts
        dict(name="score_moe_group", kind="score", model="moe", layers=2, vocab=32000, prompts=2, group=8,
             plen_lo=300, plen_hi=900, rlen=700, temp=0.6),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["decode", "decode", "decode", "decode_moe", "rollout", "rollout", "score", "score_moe", "sample"])
    temp = rng.choice([1.0, 1.0, 0.6])
    if kind == "sample":
        return dict(kind="sample", rows=log_int(1, 512), vocab=rng.choice([32000, 151936, 152064]),
                    temp=rng.choice([1.0, 0.6, 0.0]))
    if kind in ("decode", "decode_moe"):
        model = "moe" if kind == "decode_moe" else rng.choice(["1.5b", "7b", "7b", "32b", "llama7b"])
        lo = log_int(64, 2000)
        hi = int(lo * rng.uniform(1.0, 4.0))
        rows = max(1, min(log_int(1, 512), 600000 // hi))
        page = rng.choice([64, 256]) if model == "moe" else 0
        if page:   # the K/V is made on the host: a bounded amount
            rows = max(1, min(rows, 160000 // hi))
        return dict(kind="decode", model=model, layers=2, vocab=4096, rows=rows, ctx_lo=lo, ctx_hi=hi, page=page,
                    temp=temp)
    if kind == "rollout":
        model = rng.choice(["tiny", "1.5b", "7b", "llama7b", "moe"])
        lo = log_int(16, 500)
        hi = int(lo * rng.uniform(1.0, 3.0))
        prompts = max(1, min(log_int(1, 32), 12000 // hi))
        if model == "tiny":
            prompts, lo, hi = min(prompts, 4), min(lo, 64), min(hi, 128)
        return dict(kind="rollout", model=model, layers=2, vocab=4096, prompts=prompts,
                    group=rng.choice([1, 3, 4, 8, 16]) if model != "tiny" else 4, plen_lo=lo, plen_hi=hi,
                    patches=rng.choice([0, lo // 2]) if model == "llama7b" else 0, steps=rng.randint(1, 6),
                    page=rng.choice([0, 64, 256]), temp=temp)
    model = "moe" if kind == "score_moe" else rng.choice(["1.5b", "7b", "llama7b"])
    group = rng.choice([2, 4, 8, 16])
    prompts = rng.randint(1, 3)
    rlen = max(16, min(log_int(50, 1500), 12000 // (prompts * group)))
    lo = log_int(32, 800)
    return dict(kind="score", model=model, layers=2, vocab=rng.choice([4096, 32000]), prompts=prompts, group=group,
                plen_lo=lo, plen_hi=int(lo * rng.uniform(1.0, 1.5)), rlen=rlen, temp=temp)


# ---- sizes of a case ---------------------------------------------------------------------------------------
def shape_of(case):
    return replace(MODELS[case["model"]], n_layers=case["layers"], vocab=case["vocab"])


def _ints(case, what, n, lo, hi):
    r = random.Random("%s %s %d %d %d" % (what, case.get("model"), n, lo, hi))
    return [r.randint(lo, hi) for _ in range(n)]


def contexts(case):
    return _ints(case, "ctx", case["rows"], case["ctx_lo"], case["ctx_hi"])


def prompt_lens(case):
    return _ints(case, "prompt", case["prompts"], case["plen_lo"], case["plen_hi"])


def resp_lens(case):
    n = case["prompts"] * case["group"]
    if case["kind"] == "rollout":
        return [case["steps"]] * n
    r = random.Random("resp %d %d" % (n, case["rlen"]))
    return [max(2, min(2 * case["rlen"], int(r.lognormvariate(math.log(case["rlen"]), 0.5)))) for _ in range(n)]


def offsets(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


# ---- inputs ------------------------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def weights(case, seed):
    s = shape_of(case)
    w = make_weights(s, int(seed), device=DEV, init="normal" if case["model"] == "tiny" else "fanin")
    if s.moe:
        w["w_router"] *= 4   # a trained router is peaked: the last expert chosen weighs a few percent
    return w


def tokens(seed, salt, n, vocab):
    return torch.randint(0, vocab, (n,), generator=_gen(seed, salt), device=DEV, dtype=torch.int32)


def kv_pool(seed, nbytes):
    """A contiguous pool of N(0, 1) keys and values (what projections of normalised rows look like)."""
    return torch.empty(nbytes // 2, dtype=torch.bfloat16, device=DEV).normal_(generator=_gen(seed, 11))


def packed_kv(case, seed):
    """Host K/V of every slot in the layout rl_kv_onload documents."""
    s = shape_of(case)
    per = [s.n_layers * s.n_kv_heads * (n + (n + 7) // 8 * 8) * s.head_dim for n in contexts(case)]
    t = torch.empty(sum(per), dtype=torch.bfloat16, device=DEV).normal_(generator=_gen(seed, 12))
    return t, per


def packed_prompts(case, seed):
    """Prompt ids (negative: caller rows), the caller rows, and response ids."""
    s = shape_of(case)
    plens = prompt_lens(case)
    tok = tokens(seed, 21, sum(plens), s.vocab)
    embeds = None
    if case.get("patches"):
        p, off = case["patches"], offsets(plens)
        embeds = torch.empty((len(plens) * p, s.hidden), dtype=torch.bfloat16, device=DEV).normal_(
            generator=_gen(seed, 22))
        for i in range(len(plens)):
            tok[off[i]:off[i] + p] = -1 - torch.arange(i * p, (i + 1) * p, dtype=torch.int32, device=DEV)
    resp = tokens(seed, 23, sum(resp_lens(case)), s.vocab)
    return tok, embeds, resp


def sample_inputs(case, seed):
    r = np.random.RandomState(int(seed) % (1 << 31))
    uids = r.randint(0, 1 << 30, case["rows"]).astype(np.uint64)
    pos = r.randint(1, 5000, case["rows"]).astype(np.int32)
    z = torch.empty((case["rows"], case["vocab"]), dtype=torch.float32, device=DEV).normal_(
        0.0, 2.0, generator=_gen(seed, 31))
    return z, uids, pos


def prepare(case, seed):
    st = {"case": case, "kind": case["kind"], "T": case["temp"], "seed": int(seed)}
    i32 = dict(dtype=torch.int32, device=DEV)
    f32 = dict(dtype=torch.float32, device=DEV)
    if case["kind"] == "sample":
        n = case["rows"]
        s = replace(configs.TINY, vocab=case["vocab"])   # the engine whose workspace the call uses
        st["eng"] = Engine(s, make_weights(s, 1, device=DEV), max_seqs=n, max_ctx=32, max_prefill_tokens=32, device=DEV)
        st["z"], st["uids"], st["pos"] = sample_inputs(case, seed)
        st["tok"], st["logp"] = torch.empty(n, **i32), torch.empty(n, **f32)
        return st
    s = shape_of(case)
    w = weights(case, seed)
    if case["kind"] == "decode":
        n, ctx = case["rows"], contexts(case)
        eng = Engine(s, w, max_seqs=n, max_ctx=max(ctx) + 8, max_prefill_tokens=1024, device=DEV,
                     kv_page_size=case["page"])
        slots = np.arange(n, dtype=np.int32)
        if case["page"]:
            host, _ = packed_kv(case, seed)
            eng.kv_onload(slots, ctx, host.view(torch.uint8).cpu())
            torch.cuda.synchronize()
        else:
            eng.kv.view(torch.bfloat16).copy_(kv_pool(seed, eng.kv_nbytes))
        st.update(eng=eng, slots=slots, ctx=np.asarray(ctx, dtype=np.int32), uids=np.arange(n, dtype=np.uint64),
                  in_tok=tokens(seed, 1, n, s.vocab), forced=tokens(seed, 2, n, s.vocab), tok=torch.empty(n, **i32),
                  logp=torch.empty(n, **f32), logits=torch.empty((n, s.vocab), **f32))
        return st
    plens, rlens, g = prompt_lens(case), resp_lens(case), case["group"]
    n = len(rlens)
    tok, embeds, resp = packed_prompts(case, seed)
    total = sum(plens) + (sum(rlens) if case["kind"] == "score" else 0)
    st["eng"] = Engine(s, w, max_seqs=n, max_ctx=max(p + max(rlens[i * g:(i + 1) * g]) for i, p in enumerate(plens)) + 8,
                       max_prefill_tokens=total, device=DEV, kv_page_size=case.get("page", 0))
    st.update(slots=np.arange(n, dtype=np.int32), uids=np.arange(n, dtype=np.uint64), poff=offsets(plens), group=g,
              ptok=tok, embeds=embeds)
    if case["kind"] == "score":
        st.update(roff=offsets(rlens), rtok=resp, logp=torch.empty(sum(rlens), **f32))
        return st
    k = case["steps"]
    st["in_tok"] = [resp.view(n, k)[:, j].contiguous() for j in range(k)]
    st["forced"] = tokens(seed, 24, n, s.vocab)
    st["tok"] = torch.empty(n, **i32)
    st["logp"] = [torch.empty(n, **f32) for _ in range(k + 1)]
    st["logits"] = [torch.empty((len(plens), s.vocab), **f32)] + [torch.empty((n, s.vocab), **f32) for _ in range(k)]
    return st


def run(st):
    e = st["eng"]
    if st["kind"] == "sample":
        e.sample_logits(st["z"], st["uids"], st["pos"], st["tok"], st["logp"], seed=st["seed"], temperature=st["T"])
        return st["tok"], st["logp"]
    if st["kind"] == "decode":
        e.set_lengths(st["slots"], st["ctx"])
        e.step(st["slots"], st["uids"], st["in_tok"], st["tok"], st["logp"], forced=st["forced"], seed=3,
               temperature=st["T"], out_logits=st["logits"])
        return st["logits"], st["logp"]
    if st["kind"] == "score":
        e.score(st["slots"], st["poff"], st["ptok"], st["roff"], st["rtok"], st["logp"], group=st["group"],
                temperature=st["T"])
        return st["logp"]
    # teacher-forced: the tokens fed back are given, so that every step's logits can be compared
    e.prefill(st["slots"], st["uids"], st["poff"], st["ptok"], st["tok"], st["logp"][0], group=st["group"],
              embeds=st["embeds"], forced=st["in_tok"][0], seed=3, temperature=st["T"], out_logits=st["logits"][0])
    k = len(st["in_tok"])
    for j in range(k):
        e.step(st["slots"], st["uids"], st["in_tok"][j], st["tok"], st["logp"][j + 1],
               forced=st["in_tok"][j + 1] if j + 1 < k else st["forced"], seed=3, temperature=st["T"],
               out_logits=st["logits"][j + 1])
    return {"logits": st["logits"], "logp": st["logp"]}


# ---- what a pass cannot do without -------------------------------------------------------------------------
def _pass_work(s, rows, head_rows, kv_read, kv_write, scored):
    """One forward over `rows` tokens: weights once, K/V positions read and written once, logits once."""
    reach = s.n_experts * (1.0 - (1.0 - s.top_k / s.n_experts) ** rows) if s.moe else None
    kvb = s.kv_bytes_per_token()
    out = 4.0 * rows if scored else 4.0 * head_rows * s.vocab
    nbytes = s.decode_params(reach) * s.elem_bytes + rows * s.hidden * s.elem_bytes + (kv_read + kv_write) * kvb + out
    per_row = s.decode_params(s.top_k if s.moe else None) - s.hidden * s.vocab
    return nbytes, 2.0 * rows * per_row + 2.0 * head_rows * s.hidden * s.vocab


def work(case):
    if case["kind"] == "sample":
        n, v = case["rows"], case["vocab"]
        return {"bytes": 4.0 * n * v + 20.0 * n, "flops": 4.0 * n * v}
    s = shape_of(case)
    att = 4.0 * s.n_q_heads * s.head_dim * s.n_layers   # FLOPs per (token, key)
    if case["kind"] == "decode":
        ctx = contexts(case)
        b, f = _pass_work(s, len(ctx), len(ctx), sum(ctx), len(ctx), False)
        return {"bytes": b, "flops": f + att * (sum(ctx) + len(ctx))}
    plens, rlens, g = prompt_lens(case), resp_lens(case), case["group"]
    if case["kind"] == "score":
        rows = sum(plens) + sum(rlens)
        b, f = _pass_work(s, rows, len(plens) + sum(rlens) - len(rlens), 0, 0, True)
        keys = sum(p * (p + 1) / 2 for p in plens) + sum(m * (plens[i // g] + (m + 1) / 2) for i, m in enumerate(rlens))
        return {"bytes": b, "flops": f + att * keys}
    n = len(rlens)
    # a paged pool holds a prompt's full pages once per group; a contiguous one needs them in every slot
    page = case["page"]
    copies = sum((p // page * page + g * (p % page)) if page else g * p for p in plens)
    b, f = _pass_work(s, sum(plens), len(plens), 0, copies, False)
    f += att * sum(p * (p + 1) / 2 for p in plens)
    for j in range(case["steps"]):
        own = n * j
        bb, ff = _pass_work(s, n, n, sum(plens) + own, n, False)
        b, f = b + bb, f + ff + att * (g * sum(plens) + own + n)
    return {"bytes": b, "flops": f}


def tolerance(case):
    # about four times what the path differs from 64 bits by (two correct versions differ by about as much)
    if case["kind"] == "sample":
        return {"rel": 5e-7, "max": 5e-6, "differ": 0.0}
    if case["model"] == "tiny":
        return {"rel": 4e-6, "max": 4e-5}
    if case["model"] == "moe":
        # a row whose routing decision is a near tie may take another last expert
        return {"rel": 0.01, "max": 0.3}
    return {"rel": 0.01, "max": 0.06}


# ---- the same in 64 bits -----------------------------------------------------------------------------------
def _rms(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, theta):
    """x [rows][heads][d] rotated by the angle of each row's position (halves paired)."""
    d = x.shape[-1]
    w = theta ** (-2.0 * torch.arange(d // 2, device=DEV, dtype=torch.float64) / d)
    a = pos.double()[:, None] * w[None, :]
    c, s = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
    u, v = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([u * c - v * s, v * c + u * s], -1)


def _mlp(s, w, l, h):
    if not s.moe:
        gu = h @ w["w_gate_up"][l].double().t()
        a, b = gu[:, :s.ffn], gu[:, s.ffn:]
        return (torch.nn.functional.silu(a) * b) @ w["w_down"][l].double().t()
    top, idx = (h @ w["w_router"][l].double().t()).topk(s.top_k, dim=-1)
    p = torch.softmax(top, -1)
    out = torch.zeros_like(h)
    for e in range(s.n_experts):
        r, j = (idx == e).nonzero(as_tuple=True)
        if not len(r):
            continue
        gu = h[r] @ w["w_exp_gate_up"][l, e].double().t()
        a, b = gu[:, :s.expert_ffn], gu[:, s.expert_ffn:]
        y = (torch.nn.functional.silu(a) * b) @ w["w_exp_down"][l, e].double().t()
        out.index_add_(0, r, p[r, j][:, None] * y)
    return out


def _attend(q, k, v, first):
    """q [m][Hq][d] at positions first.. over k, v [t][Hkv][d] (query i sees keys 0 .. first + i)."""
    m, hq, d = q.shape
    t, hkv, _ = k.shape
    qh = q.view(m, hkv, hq // hkv, d).permute(1, 2, 0, 3).reshape(hkv, -1, d)
    s = torch.matmul(qh, k.permute(1, 2, 0).contiguous()).view(hkv, hq // hkv, m, t) / math.sqrt(d)
    if m > 1 or first + 1 < t:
        s = s.masked_fill(torch.arange(t, device=DEV)[None, :] > first + torch.arange(m, device=DEV)[:, None], -math.inf)
    o = torch.matmul(torch.softmax(s, -1).view(hkv, -1, t), v.permute(1, 0, 2).contiguous())
    return o.view(hkv, hq // hkv, m, d).permute(2, 0, 1, 3).reshape(m, hq * d)


def _forward(s, w, x, pos, attend):
    """Final normed rows of a forward pass; attend(l, q, k, v) returns the attention of every row."""
    hq, hkv, d = s.n_q_heads, s.n_kv_heads, s.head_dim
    for l in range(s.n_layers):
        qkv = (_rms(x, w["attn_norm"][l], s.rms_eps) @ w["w_qkv"][l].double().t()).view(len(x), hq + 2 * hkv, d)
        q, k = _rope(qkv[:, :hq], pos, s.rope_theta), _rope(qkv[:, hq:hq + hkv], pos, s.rope_theta)
        x = x + attend(l, q, k, qkv[:, hq + hkv:]) @ w["w_o"][l].double().t()
        x = x + _mlp(s, w, l, _rms(x, w["mlp_norm"][l], s.rms_eps))
    return _rms(x, w["final_norm"], s.rms_eps)


def _logp(z, tok, temp):
    z = z / (temp if temp > 0 else 1.0)
    return z.gather(-1, tok.long()[:, None])[:, 0] - torch.logsumexp(z, -1)


def _slot_kv(case, seed, s):
    """(l, i) -> keys and values [len][Hkv][d] of the decode cases' slots."""
    ctx = contexts(case)
    hkv, d = s.n_kv_heads, s.head_dim
    if not case["page"]:
        cap, n = (max(ctx) + 8 + 31) // 32 * 32, len(ctx)
        pool = kv_pool(seed, 2 * s.n_layers * n * hkv * cap * d * 2)
        kk = pool[:pool.numel() // 2].view(s.n_layers, n, hkv, cap, d)
        vv = pool[pool.numel() // 2:].view(s.n_layers, n, hkv, cap // 8, d, 8)

        def get(l, i):
            m = ctx[i]
            v = vv[l, i].permute(1, 3, 0, 2).reshape(cap, hkv, d)
            return kk[l, i, :, :m].permute(1, 0, 2).double(), v[:m].double()
        return get
    flat, per = packed_kv(case, seed)
    base = offsets(per).astype(np.int64) if sum(per) < (1 << 31) else np.concatenate([[0], np.cumsum(per)])

    def get(l, i):
        m = ctx[i]
        m8 = (m + 7) // 8 * 8
        t = flat[int(base[i]):int(base[i + 1])].view(s.n_layers, hkv, (m + m8) * d)[l]
        k = t[:, :m * d].view(hkv, m, d).permute(1, 0, 2)
        v = t[:, m * d:].reshape(hkv, m8 // 8, d, 8).permute(1, 3, 0, 2).reshape(m8, hkv, d)[:m]
        return k.double(), v.double()
    return get


def _philox(case, seed):
    """Noise words [rows][vocab] of the sampler's counter-based generator (Philox4x32-10)."""
    _, uids, pos = sample_inputs(case, seed)
    lo, u32 = np.uint64(0xFFFFFFFF), np.uint64(32)
    out = np.empty((case["rows"], case["vocab"]), dtype=np.uint32)
    for i in range(case["rows"]):
        c = [np.arange(case["vocab"] // 4, dtype=np.uint64)] + [
            np.full(case["vocab"] // 4, x, dtype=np.uint64) for x in (pos[i], uids[i] & lo, uids[i] >> u32)]
        k0, k1 = int(seed) & 0xFFFFFFFF, int(seed) >> 32
        for r in range(10):
            p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
            c = [(p1 >> u32) ^ c[1] ^ np.uint64(k0), p1 & lo, (p0 >> u32) ^ c[3] ^ np.uint64(k1), p0 & lo]
            k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
        out[i] = np.stack(c, -1).reshape(-1).astype(np.uint32)
    return out


def exact(case, seed):
    if case["kind"] == "sample":
        z, _, _ = sample_inputs(case, seed)
        score = z if case["temp"] == 0 else z / case["temp"]
        if case["temp"] > 0:
            u = (_philox(case, seed).astype(np.float64) + 0.5) * 2.0 ** -32
            score = score + torch.from_numpy((-np.log(-np.log(u))).astype(np.float32)).to(DEV)
        return None, _logp(z.double(), score.argmax(-1), case["temp"])
    s, w = shape_of(case), weights(case, seed)
    head = w["lm_head"].double().t()
    if case["kind"] == "decode":
        ctx, n = contexts(case), case["rows"]
        get = _slot_kv(case, seed, s)

        def attend(l, q, k, v):
            rows = []
            for i in range(n):
                kc, vc = get(l, i)
                rows.append(_attend(q[i:i + 1], torch.cat([kc, k[i:i + 1]]), torch.cat([vc, v[i:i + 1]]), ctx[i]))
            return torch.cat(rows)
        x = w["embed"][tokens(seed, 1, n, s.vocab).long()].double()
        z = _forward(s, w, x, torch.tensor(ctx, device=DEV), attend) @ head
        return z, _logp(z, tokens(seed, 2, n, s.vocab), case["temp"])
    plens, rlens, g = prompt_lens(case), resp_lens(case), case["group"]
    tok, embeds, resp = packed_prompts(case, seed)
    po, ro, np_rows = offsets(plens), offsets(rlens), sum(plens)
    x = w["embed"][torch.cat([tok.clamp(min=0), resp]).long()].double()
    if embeds is not None:
        own = (tok < 0).nonzero()[:, 0]
        x[own] = embeds[(-tok[own] - 1).long()].double()
    pos = torch.cat([torch.arange(p, device=DEV) for p in plens] +
                    [torch.arange(plens[i // g], plens[i // g] + m, device=DEV) for i, m in enumerate(rlens)])

    def attend(l, q, k, v):
        rows = [_attend(q[po[p]:po[p + 1]], k[po[p]:po[p + 1]], v[po[p]:po[p + 1]], 0) for p in range(len(plens))]
        for i in range(len(rlens)):
            a, b, p = np_rows + ro[i], np_rows + ro[i + 1], i // g
            rows.append(_attend(q[a:b], torch.cat([k[po[p]:po[p + 1]], k[a:b]]), torch.cat([v[po[p]:po[p + 1]], v[a:b]]),
                                plens[p]))
        return torch.cat(rows)
    h = _forward(s, w, x, pos, attend)
    last = torch.tensor([po[p + 1] - 1 for p in range(len(plens))], device=DEV)
    if case["kind"] == "rollout":
        k = case["steps"]
        rows = h[np_rows:].view(len(rlens), k, -1)
        z = [h[last] @ head] + [rows[:, j] @ head for j in range(k)]
        targets = [resp.view(len(rlens), k)[:, j] for j in range(k)] + [tokens(seed, 24, len(rlens), s.vocab)]
        logp = [_logp(z[0].repeat_interleave(g, 0), targets[0], case["temp"])]
        return {"logits": z, "logp": logp + [_logp(z[j], targets[j], case["temp"]) for j in range(1, k + 1)]}
    src = torch.cat([torch.cat([last[i // g:i // g + 1], torch.arange(np_rows + ro[i], np_rows + ro[i + 1] - 1, device=DEV)])
                     for i in range(len(rlens))])
    return torch.cat([_logp(h[src[a:a + 2048]] @ head, resp[a:a + 2048], case["temp"]) for a in range(0, len(src), 2048)])
