"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case is one call of an online-DPO step's generation side: completions drawn from the policy (`generate`), the
teacher-forced log-probs of finished sequences (`score`), the next-token logits of prompts (`logits`), the sampling stage
alone (`sample`), and the learner's terms from the log-probs (`terms`).  Models are the widths the paper trains
(Pythia 410M / 1B / 2.8B, Llama-3.1 8B) with as many blocks as keep a case short: every kernel of a block runs once per
block, so two or four blocks are the same work per block as all of them.  Weights and inputs are random draws of the
distributions of the synthetic workloads: N(0, 0.02) matrices, gains 1 + N(0, 0.02), uniform token ids.

Where a call draws tokens that feed the next step, the tokens are given (`forced`): a draw that falls on the other side of
a bucket of width 2e-5 would send two correct implementations down different sequences.  The sampler still does all of its
work for every one of them.  The draw itself is in the `sample` cases.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

NEOX, LLAMA = 0, 1

# name: (arch, all blocks, d_model, query heads, kv heads, head dim, FFN width, vocabulary, rotary dims, theta)
MODELS = {
    "tiny": (NEOX, 2, 128, 4, 4, 32, 512, 1024, 8, 1e4),
    "410m": (NEOX, 24, 1024, 16, 16, 64, 4096, 50304, 16, 1e4),
    "1b": (NEOX, 16, 2048, 8, 8, 256, 8192, 50304, 64, 1e4),
    "2.8b": (NEOX, 32, 2560, 32, 32, 80, 10240, 50304, 20, 1e4),
    "8b": (LLAMA, 32, 4096, 32, 8, 128, 14336, 128256, 128, 5e5),
}


def _case(name, op, model, layers, B, lo, hi, k=1, new=0, temperature=0.7, share=False, eos=False, precise=False, f32=False):
    return {"name": name, "op": op, "model": model, "layers": layers, "B": B, "lo": lo, "hi": hi, "k": k, "new": new,
            "temperature": temperature, "share": share, "eos": eos, "precise": precise, "f32": f32}


def listed():
    return [
        # the learner's side of one step: pair selection, DPO loss and the Proximal RLOO objective of 512 scored pairs
        _case("terms-512x2", "terms", "2.8b", 1, 512, 256, 512, k=2, new=64),
        # the sampling stage on its own in a serving loop: final norm, LM head and draw for 64 rows
        _case("sample-64", "sample", "2.8b", 1, 64, 1, 1),
        # the smallest model there is, fp32 weights: launches and latency
        _case("generate-tiny", "generate", "tiny", 2, 4, 32, 32, k=2, new=16, f32=True),
        # next-token logits of three prompts with the whole 1B-shaped model: a prompt pass that cannot fill the chip
        _case("logits-1b-3", "logits", "1b", 16, 3, 64, 400),
        # evaluation: greedy completions of 16 prompts that end at an EOS token, whole 1B-shaped model: weight-bound decode
        _case("greedy-eos-1b-16", "generate", "1b", 16, 16, 128, 512, new=64, temperature=0.0, eos=True),
        # the TL;DR workload at 410M: the whole model, 128 sequences
        _case("generate-410m-64x2", "generate", "410m", 24, 64, 128, 512, k=2, new=64),
        # the TL;DR workload at 1B: 512 sequences, head size 256
        _case("generate-1b-256x2", "generate", "1b", 4, 256, 128, 512, k=2, new=64),
        # the TL;DR workload at 2.8B (the headline): 1024 sequences, a cache that outweighs the weights
        _case("generate-2.8b-512x2", "generate", "2.8b", 4, 512, 256, 512, k=2, new=64),
        # the training-bound setting: four samples of a prompt read one copy of its cache
        _case("generate-2.8b-96x4-shared", "generate", "2.8b", 4, 96, 100, 512, k=4, new=64, share=True),
        # the chatbot workload at 8B: grouped-query attention, SwiGLU, long contexts
        _case("generate-8b-128x2", "generate", "8b", 2, 128, 256, 1024, k=2, new=96),
        # log-probs of 512 prompts with their two completions, each prompt once
        _case("score-2.8b-512x2", "score", "2.8b", 4, 512, 256, 512, k=2, new=64),
        # sequences of all lengths, each on its own, in the mode that keeps pairs of 16-bit numbers
        _case("score-8b-24-precise", "score", "8b", 2, 24, 5, 1024, precise=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# seconds a pass would take at 5 TB/s and 0.7 PFLOP/s and with 50 us for each block and step, and the bytes of a context
def _seconds(case):
    w = work(case)
    steps = case["new"] if case["op"] == "generate" else 1
    return w["bytes"] / 5e12 + w["flops"] / (0.35e15 if case["precise"] else 0.7e15) + steps * case["layers"] * 50e-6


def draw(rng):
    most = max(_seconds(c) for c in listed())
    while True:
        op = rng.choice(["generate"] * 5 + ["score"] * 2 + ["logits", "sample", "terms"])
        model = rng.choice(["410m", "1b", "2.8b", "8b"])
        arch, _, d, hq, hkv, h, F, V, r, theta = MODELS[model]
        pairs = h <= 128          # the mode that keeps pairs of 16-bit numbers has no larger heads
        if op == "terms":
            c = _case("", op, model, 1, _log_int(rng, 16, 2000), 64, rng.randint(100, 600), k=rng.choice([2, 2, 3, 4]), new=_log_int(rng, 16, 512))
        elif op == "sample":
            c = _case("", op, model, 1, rng.randint(1, 64), 1, 1, temperature=rng.choice([0.7, 1.0]))
        elif op == "logits":
            c = _case("", op, model, rng.randint(1, 4), _log_int(rng, 1, 64), rng.randint(1, 64), rng.randint(65, 1024))
        elif op == "score":
            k = rng.choice([1, 2, 2, 4])     # more than one: a prompt and its completions
            c = _case("", op, model, rng.randint(1, 2), _log_int(rng, 2, 384), rng.randint(1, 128), rng.randint(129, 768), k=k,
                      new=_log_int(rng, 8, 128) if k > 1 else 0, precise=pairs and rng.random() < 0.2)
        else:
            share = rng.random() < 0.25
            k = rng.choice([1, 2, 2, 2, 3, 4])
            if share:
                k = min(k, 16 * hkv // hq)
            c = _case("", op, model, rng.randint(1, 3), _log_int(rng, 1, 400), rng.randint(1, 256), rng.randint(257, 1024), k=k,
                      new=_log_int(rng, 4, 128), temperature=rng.choice([0.7, 0.7, 1.0, 0.0]), share=share,
                      eos=rng.random() < 0.25, precise=pairs and rng.random() < 0.1)
        del c["name"]
        cache = 4.0 * c["layers"] * hkv * h * c["B"] * c["k"] * (c["hi"] + c["new"] + 32) * (2 if c["precise"] else 1)
        if _seconds(c) <= 0.9 * most and cache < 24e9:
            return c


def _shape(case):
    arch, _, d, hq, hkv, h, F, V, r, theta = MODELS[case["model"]]
    return SimpleNamespace(arch=arch, n_layers=case["layers"], d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=h, d_ffn=F,
                           vocab=V, rotary_dim=r, rope_theta=theta, norm_eps=1e-5)


# ------------------------------------------------------------------------------------------------ inputs


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _weights(case, seed):
    """Canonical tensors of the model, drawn on the device: bf16, or fp32 where the caller keeps them so."""
    m = _shape(case)
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(int(seed) * 1000003 + 17)
    dt = torch.float32 if case["f32"] else torch.bfloat16
    d, F, V, qd, kvd = m.d_model, m.d_ffn, m.vocab, m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    neox = m.arch == NEOX

    def mat(*shape, scale=1.0):
        t = torch.empty(*shape, dtype=torch.float32, device=dev).normal_(0.0, 0.02 * scale, generator=g)
        return t.to(dt)

    def gain():
        return (1.0 + torch.empty(d, dtype=torch.float32, device=dev).normal_(0.0, 0.02, generator=g)).to(dt)

    # the sampling stage meets a peaked distribution, as a trained model's: a few tokens hold most of the mass
    w = {"embed_in": mat(V, d), "final_norm_g": gain(), "lm_head": mat(V, d, scale=5.0 if case["op"] == "sample" else 1.0)}
    if neox:
        w["final_norm_b"] = mat(d)
    for l in range(m.n_layers):
        t = {"norm1_g": gain(), "norm2_g": gain(), "wq": mat(qd, d), "wk": mat(kvd, d), "wv": mat(kvd, d), "wo": mat(d, qd),
             "w_up": mat(F, d), "w_down": mat(d, F)}
        if neox:
            t.update(norm1_b=mat(d), norm2_b=mat(d), bq=mat(qd), bk=mat(kvd), bv=mat(kvd), bo=mat(d), b_up=mat(F), b_down=mat(d))
        else:
            t["w_gate"] = mat(F, d)
        for name, x in t.items():
            w["layers.%d.%s" % (l, name)] = x
    return w


def _lens(case, seed):
    """Prompt (or sequence) lengths, uniform in the stated range, the shortest and the longest among them."""
    n = np.random.default_rng([int(seed), 1]).integers(case["lo"], case["hi"], size=case["B"], endpoint=True).astype(np.int32)
    n[0] = case["hi"]
    if case["B"] > 1:
        n[-1] = case["lo"]
    return n


def _tokens(case, seed, lens, k, new):
    """Prompts [B, hi] padded with an id that nothing may read, and completions [B, k, new]."""
    rng = np.random.default_rng([int(seed), 2])
    V = MODELS[case["model"]][7]
    prompts = rng.integers(1, V, size=(case["B"], case["hi"])).astype(np.int32)
    prompts[np.arange(case["hi"])[None, :] >= lens[:, None]] = -1
    forced = rng.integers(1, V, size=(case["B"], k, max(new, 1))).astype(np.int32)
    if case["eos"]:       # token 0 ends a completion, at a step drawn uniformly
        ends = rng.integers(1, new + 1, size=(case["B"], k))
        np.put_along_axis(forced, (ends - 1)[..., None], 0, axis=2)
    return prompts, forced


def _full(case, seed):
    """The sequences a learner scores: every prompt with each of its k completions, [B k, hi + new], their lengths and
    the length of the prompt part (1 where the sequences are on their own: all of it is scored)."""
    k, new, lens = case["k"], case["new"], _lens(case, seed)
    prompts, comp = _tokens(case, seed, lens, k, new)
    seqs = np.full((case["B"] * k, case["hi"] + new), -1, np.int32)
    for b in range(case["B"]):
        n = int(lens[b])
        seqs[b * k:(b + 1) * k, :n] = prompts[b, :n]
        if new:
            seqs[b * k:(b + 1) * k, n:n + new] = comp[b, :, :new]
    total = np.repeat(lens, k).astype(np.int32) + new
    start = np.repeat(lens, k).astype(np.int32) if k > 1 else np.ones(case["B"], np.int32)
    return seqs, total, start


def _hidden(case, seed, weights):
    """Residual rows and one uniform per row for the sampling stage.  The uniform lies in the middle of the bucket of a
    token of probability above 2 % (or of the most probable one), so that the draw does not hang on rounding."""
    m = _shape(case)
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 5)
    hidden = torch.empty(case["B"], m.d_model, dtype=torch.float32, device=dev).normal_(0.0, 1.5, generator=g)
    z = _logits64(m, weights, hidden.double()) / _t32(case)
    p = torch.softmax(z, dim=-1)
    cum = p.cumsum(-1)
    pick = torch.multinomial((p * (p > 0.02) + 1e-12 * (p == p.max(-1, keepdim=True).values)).float(), 1, generator=g)
    u = (cum.gather(1, pick) - 0.5 * p.gather(1, pick)).squeeze(1).clamp(0.0, 1.0 - 1e-6).float()
    return hidden, u.contiguous()


def _t32(case):
    return float(np.float32(case["temperature"]))     # the entry points take the temperature as a 32-bit number


def _terms(case, seed):
    dev = _device()
    B, k, stride = case["B"], case["k"], case["hi"] + case["new"]
    g = torch.Generator(device=dev).manual_seed(int(seed) * 104729 + 3)
    n = torch.from_numpy(np.repeat(_lens(case, seed), k)).to(dev)
    pol = -torch.rand(B * k, stride, device=dev, generator=g) * 6.0
    # the reference and the generating policy are close to the policy
    ref = pol + 0.05 * torch.randn(B * k, stride, device=dev, generator=g)
    old = pol + 0.002 * torch.randn(B * k, stride, device=dev, generator=g)
    rewards = torch.randn(B, k, device=dev, generator=g)
    return {"pol": pol, "ref": ref, "old": old, "start": n, "lens": n + case["new"], "rewards": rewards}


# ------------------------------------------------------------------------------------------------ the calls


def prepare(case, seed):
    import paper_2410_18252_amd.rlgen as R

    op, k, new = case["op"], case["k"], case["new"]
    if op == "terms":
        return {"op": op, "R": R, "k": k, **_terms(case, seed)}
    w = _weights(case, seed)
    cap = case["hi"] + new if op != "sample" else 32
    S = case["B"] * k
    r32 = lambda n: (n + 31) // 32 * 32  # noqa: E731
    kv = case["B"] * (r32(case["hi"]) + k * r32(new)) if case["share"] else S * r32(cap)
    if op == "sample":
        kv = 64 * 32
    cfg = R.make_cfg(_shape(case), weight_dtype=R.DTYPE_F32 if case["f32"] else R.DTYPE_BF16, max_seqs=max(S, 2), max_seq_len=max(cap, 2),
                     max_kv_tokens=max(kv, r32(cap)), share_prompt_kv=int(case["share"]), precise=int(case["precise"]))
    st = {"op": op, "R": R, "k": k, "new": new, "temperature": case["temperature"], "policy": R.Policy(cfg, w)}
    if op == "sample":
        st["hidden"], st["u"] = _hidden(case, seed, w)
        st["out"] = (torch.empty(case["B"], dtype=torch.int32, device="cuda"), torch.empty(case["B"], dtype=torch.float32, device="cuda"))
    elif op == "generate":
        st["lens"] = _lens(case, seed)
        prompts, forced = _tokens(case, seed, st["lens"], k, new)
        st["prompts"], st["forced"] = torch.from_numpy(prompts).cuda(), torch.from_numpy(forced).cuda()
        st["u"] = torch.from_numpy(np.random.default_rng([int(seed), 3]).random((case["B"], k, new), dtype=np.float32)).cuda()
        if case["eos"]:
            R.rlgen_set_eos(st["policy"], 0)
    elif op == "score":
        seqs, st["lens"], st["start"] = _full(case, seed)
        st["seqs"] = torch.from_numpy(seqs).cuda()
        if k > 1:
            R.rlgen_set_score_groups(st["policy"], k)
    else:
        st["lens"] = _lens(case, seed)
        st["seqs"] = torch.from_numpy(_tokens(case, seed, st["lens"], 1, 0)[0]).cuda()
    return st


def run(st):
    R, op = st["R"], st["op"]
    if op == "generate":
        tokens, logprobs = R.rlgen_generate(st["policy"], st["prompts"], st["lens"], st["k"], st["new"], st["temperature"], st["u"], st["forced"])
        return {"tokens": tokens, "logprobs": logprobs}
    if op == "score":
        return {"logprobs": R.rlgen_score(st["policy"], st["seqs"], st["lens"], st["temperature"], st["start"])}
    if op == "logits":
        return {"logits": R.rlgen_debug_logits(st["policy"], st["seqs"], st["lens"])}
    if op == "sample":
        tokens, logprobs = R.rlgen_sample_static(st["policy"], st["hidden"], st["temperature"], st["u"], out=st["out"])
        return {"tokens": tokens, "logprobs": logprobs}
    B, k = st["rewards"].shape
    pol, ref, old = (R.rlgen_sequence_logprob(st[n], st["start"], st["lens"]).view(B, k) for n in ("pol", "ref", "old"))
    best, worst = R.rlgen_select_pairs(st["rewards"])
    p, n = best.long()[:, None], worst.long()[:, None]
    loss = R.rlgen_dpo_loss(pol.gather(1, p), ref.gather(1, p), pol.gather(1, n), ref.gather(1, n), 0.1)
    return {"pol": pol, "ref": ref, "old": old, "best": best, "worst": worst, "loss": loss,
            "rloo": R.rlgen_proximal_rloo(pol, old, st["rewards"], 0.2)}


# ------------------------------------------------------------------------------------------------ what a pass needs


def work(case):
    """Weights once per pass over the blocks (once per decode step), cached keys and values once per decode step, inputs
    and outputs once; the products' flops with attention over the visible keys only."""
    arch, _, d, hq, hkv, h, F, V, r, theta = MODELS[case["model"]]
    op, B, k, new, L = case["op"], case["B"], case["k"], case["new"], case["layers"]
    if op == "terms":
        return {"bytes": 4.0 * B * k * (3 * new + 12), "flops": 4.0 * B * k * new}
    body = L * ((hq + 2 * hkv) * h * d + hq * h * d + (3 if arch == LLAMA else 2) * d * F)
    head = V * d
    pair = 2.0 if case["precise"] else 1.0          # 16-bit values per element, products per weight
    if op == "sample":
        return {"bytes": 2.0 * head + 4.0 * B * d, "flops": 2.0 * B * head}
    mean = 0.5 * (case["lo"] + case["hi"])
    rows = B * mean
    tri = B * 0.5 * mean * mean
    att = 4.0 * h * hq * L
    if op == "logits":
        return {"bytes": 2.0 * (body + head) + 4.0 * B * V, "flops": 2.0 * rows * body + 2.0 * B * head + att * tri}
    if op == "score":
        tail = B * k * new
        scored = tail if k > 1 else rows
        flops = 2.0 * (rows + tail) * body + 2.0 * scored * head + att * (tri + B * k * (new * mean + 0.5 * new * new))
        return {"bytes": 2.0 * (body + head) + 8.0 * B * k * (mean + new), "flops": pair * flops}
    share = B if case["share"] else B * k
    live = 0.5 if case["eos"] else 1.0
    steps = (new - 1) * live
    kv = 4.0 * L * hkv * h * pair
    keys = (share * mean * (new - 1) + B * k * 0.5 * new * (new - 1)) * live
    flops = 2.0 * (rows + B * k * steps) * body + 2.0 * B * k * (1 + steps) * head + att * (tri + B * k * steps * (mean + 0.5 * new))
    return {"bytes": 2.0 * (body + head) * new + kv * (keys + rows + B * k * steps) + 12.0 * B * k * new, "flops": pair * flops}


def tolerance(case):
    """About four times the distance measured between what the entry points return and the 64-bit values.  Log-probs of
    nearly uniform distributions are about -11, so their relative errors are a tenth of the logits'."""
    llama = MODELS[case["model"]][0] == LLAMA
    if case["op"] == "terms":
        return {"rel": 4e-5}       # exp of a difference of two sums of 64 terms (measured 1e-5)
    if case["precise"]:
        return {"rel": 1e-5}       # measured 2.5e-6
    if case["op"] == "sample":
        return {"rel": 2e-3}       # measured 4.6e-4: log-probs of likely tokens are small
    if case["op"] == "logits":
        return {"rel": 2.8e-2 if llama else 3.2e-3}       # measured 8e-4 on NeoX shapes
    return {"rel": 3e-3 if llama else 2.6e-4}             # measured 7.6e-4 and 6.5e-5


# ------------------------------------------------------------------------------------------------ the same in 64 bits


def _norm64(x, g, b, eps):
    if b is not None:
        x = x - x.mean(-1, keepdim=True)
    y = x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()
    return y if b is None else y + b.double()


def _logits64(m, w, x):
    y = _norm64(x, w["final_norm_g"], w.get("final_norm_b"), m.norm_eps)
    return torch.cat([y @ t.double().t() for t in w["lm_head"].split(16384)], dim=-1)


def _rope64(x, pos, r, theta):
    half = r // 2
    ang = pos.double()[:, None] * (theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / r))[None, :]
    c, s = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :half], x[..., half:r]
    return torch.cat([a * c - b * s, b * c + a * s, x[..., r:]], dim=-1)


def _attend64(q, k, v, first):
    """Causal attention of one sequence's rows from position `first` on; q [n, Hq, h], k, v [first + n, Hkv, h]."""
    n, hq, h = q.shape
    rep = hq // k.shape[1]
    kk = k.permute(1, 2, 0).repeat_interleave(rep, 0).contiguous()
    vv = v.permute(1, 0, 2).repeat_interleave(rep, 0).contiguous()
    s = torch.matmul(q.permute(1, 0, 2).contiguous(), kk) / math.sqrt(h)
    at = torch.arange(n, device=q.device) + first
    s.masked_fill_(torch.arange(k.shape[0], device=q.device)[None, :] > at[:, None], -math.inf)
    return torch.matmul(torch.softmax(s, -1), vv).permute(1, 0, 2).reshape(n, hq * h)


def _hidden64(case, w, groups, last=None):
    """Residual rows after all blocks of groups of sequences: a group is (prompt ids, [tails ids]); a prompt runs once.
    Returns for each group (prompt rows, [tail rows])."""
    m = _shape(case)
    dev = _device()
    out = []
    at = 0
    while at < len(groups):
        part, rows = [], 0
        while at < len(groups) and (not part or rows < 12000):
            part.append(groups[at])
            rows += len(groups[at][0]) + sum(len(t) for t in groups[at][1])
            at += 1
        segs, ids, pos = [], [], []
        for prompt, tails in part:
            mine = []
            for ext, first in [(prompt, 0)] + [(t, len(prompt)) for t in tails]:
                mine.append((len(ids), len(ids) + len(ext), first))
                ids += [int(i) for i in ext]
                pos += range(first, first + len(ext))
            segs.append(mine)
        pos = torch.tensor(pos, device=dev)
        x = w["embed_in"][torch.tensor(ids, device=dev)].double()
        for l in range(m.n_layers):
            t = {n[len("layers.%d." % l):]: v for n, v in w.items() if n.startswith("layers.%d." % l)}
            t = {n: v.double() for n, v in t.items()}
            lin = lambda y, a, b: y @ t[a].t() + (t[b] if b in t else 0.0)  # noqa: E731
            n1 = _norm64(x, t["norm1_g"], t.get("norm1_b"), m.norm_eps)
            q = _rope64(lin(n1, "wq", "bq").view(-1, m.n_q_heads, m.head_dim), pos, m.rotary_dim, m.rope_theta)
            kk = _rope64(lin(n1, "wk", "bk").view(-1, m.n_kv_heads, m.head_dim), pos, m.rotary_dim, m.rope_theta)
            vv = lin(n1, "wv", "bv").view(-1, m.n_kv_heads, m.head_dim)
            o = torch.empty(x.shape[0], m.n_q_heads * m.head_dim, dtype=torch.float64, device=dev)
            for mine in segs:
                p0, p1, _ = mine[0]
                for a, b, first in mine:
                    keys = (kk[a:b], vv[a:b]) if first == 0 else (torch.cat([kk[p0:p1], kk[a:b]]), torch.cat([vv[p0:p1], vv[a:b]]))
                    if b > a:
                        o[a:b] = _attend64(q[a:b], keys[0], keys[1], first)
            if m.arch == NEOX:
                n2 = _norm64(x, t["norm2_g"], t["norm2_b"], m.norm_eps)
                y = lin(n2, "w_up", "b_up")
                x = x + lin(o, "wo", "bo") + lin(0.5 * y * (1.0 + torch.erf(y / math.sqrt(2.0))), "w_down", "b_down")
            else:
                x = x + lin(o, "wo", "bo")
                n2 = _norm64(x, t["norm2_g"], None, m.norm_eps)
                y = lin(n2, "w_gate", "")
                x = x + lin(y * torch.sigmoid(y) * lin(n2, "w_up", ""), "w_down", "b_down")
        for mine in segs:
            out.append((x[mine[0][0]:mine[0][1]], [x[a:b] for a, b, _ in mine[1:]]))
    return out


def _logprob64(case, w, rows, targets):
    temperature = _t32(case) if case["temperature"] > 0 else 1.0
    got = []
    for x, t in zip(rows.split(2048), targets.split(2048)):
        z = _logits64(_shape(case), w, x) / temperature
        got.append(z.gather(1, t[:, None]).squeeze(1) - torch.logsumexp(z, -1))
    return torch.cat(got)


def exact(case, seed):
    op, B, k, new = case["op"], case["B"], case["k"], case["new"]
    dev = _device()
    if op == "terms":
        s = _terms(case, seed)
        at = torch.arange(case["hi"] + new, device=dev)[None, :]
        inside = (at >= s["start"][:, None]) & (at < s["lens"][:, None])
        pol, ref, old = ((s[n].double() * inside).sum(1).view(B, k) for n in ("pol", "ref", "old"))
        best, worst = s["rewards"].argmax(1), s["rewards"].argmin(1)
        pick = lambda x, i: x.gather(1, i[:, None]).squeeze(1)  # noqa: E731
        margin = (pick(pol, best) - pick(ref, best)) - (pick(pol, worst) - pick(ref, worst))
        r = s["rewards"].double()
        adv = r - (r.sum(1, keepdim=True) - r) / (k - 1)
        ratio = torch.exp(pol - old)
        return {"pol": pol, "ref": ref, "old": old, "best": best.int(), "worst": worst.int(),
                "loss": torch.nn.functional.softplus(-float(np.float32(0.1)) * margin),
                "rloo": torch.minimum(ratio * adv, ratio.clamp(1 - float(np.float32(0.2)), 1 + float(np.float32(0.2))) * adv)}
    need = work(dict(case, precise=False))["flops"]
    if need > 6e14:
        return None
    # a context keeps its matrices in bf16 whatever type they are given in, and vectors as they are
    w = {n: v.to(torch.bfloat16) if v.dim() == 2 else v for n, v in _weights(case, seed).items()}
    m = _shape(case)
    if op == "sample":
        hidden, u = _hidden(case, seed, w)
        p = torch.log_softmax(_logits64(m, w, hidden.double()) / _t32(case), -1)
        tok = (p.exp().cumsum(-1) <= u.double()[:, None]).sum(-1).clamp(max=m.vocab - 1)
        return {"tokens": tok.int(), "logprobs": p.gather(1, tok[:, None]).squeeze(1)}
    if op == "logits":
        lens = _lens(case, seed)
        seqs = _tokens(case, seed, lens, 1, 0)[0]
        rows = _hidden64(case, w, [(seqs[b, :lens[b]], []) for b in range(B)])
        return {"logits": _logits64(m, w, torch.stack([r[0][-1] for r in rows]))}
    lens = _lens(case, seed)
    prompts, comp = _tokens(case, seed, lens, k, new)
    if op == "score":
        out = torch.zeros(B * k, case["hi"] + new, dtype=torch.float64, device=dev)
        if k == 1 and new == 0:
            rows = _hidden64(case, w, [(prompts[b, :lens[b]], []) for b in range(B)])
            for b in range(B):
                if lens[b] > 1:
                    out[b, 1:lens[b]] = _logprob64(case, w, rows[b][0][:-1], torch.from_numpy(prompts[b, 1:lens[b]]).long().to(dev))
            return {"logprobs": out}
    rows = _hidden64(case, w, [(prompts[b, :lens[b]], [comp[b, j, :new - 1] for j in range(k)]) for b in range(B)])
    x = torch.cat([torch.cat([r[0][-1:], t]) for r in rows for t in r[1]])
    targets = torch.from_numpy(comp[:, :, :new].reshape(-1).astype(np.int64)).to(dev)
    lp = _logprob64(case, w, x, targets).view(B, k, new)
    if op == "score":
        for b in range(B):
            out[b * k:(b + 1) * k, lens[b]:lens[b] + new] = lp[b]
        return {"logprobs": out}
    tok = torch.from_numpy(comp[:, :, :new]).to(dev)
    if case["eos"]:
        ended = (tok == 0).long().cumsum(-1) - (tok == 0).long() > 0
        tok, lp = tok.masked_fill(ended, 0), lp.masked_fill(ended, 0.0)
    return {"tokens": tok, "logprobs": lp}
