"""Performance cases: the work a program asks of this library, through its public calls.

Three families, with the sizes of the repository's own model shapes and training benchmark:

* draft calls -- the draft step at batch 1 (truncate, append the accepted rows, draft a
  block), the ingestion of a prompt followed by its first block, and the batched step of
  several sequences with contexts of their own, greedy and sampled;
* anchor attention of one draft layer in training, forward, backward and both;
* the position-weighted cross-entropy with its gradient.

A draft call is read through its logits as well as its tokens: the program keeps a pinned
host buffer and takes the logits there (the only way the library gives them out).  For
batched calls with many rows the vocabulary is cut to 4,096, so that the pass is the draft
layers and not a copy of hundreds of megabytes to the host; the full LM head at batch is
covered by the sampled case of four sequences.

Weights, target rows and ids are synthetic, drawn on the GPU from the seed alone with the
distributions of paper_2606_02091_amd/synth.py.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2606_02091_amd import dflare as dfl
from paper_2606_02091_amd import synth

SMALL_VOCAB = 4096
PREFILL_CHUNK = 512   # rows of one append while a prompt is read in


def listed():
    return [
        # the smallest call: launches, barriers and host path of a step that moves a few MB
        dict(name="step_tiny", kind="step", model="tiny", vocab=1024, block=8, context=64, n_new=5),
        # the headline step: batch 1, a 4,096-row context, the mean number of accepted rows
        dict(name="step_qwen3_8b", kind="step", model="qwen3_8b", vocab=151936, block=16, context=4096, n_new=8),
        # 64-wide heads, the long context and the largest vocabulary, one drafted block mostly rejected
        dict(name="step_gpt_oss_20b", kind="step", model="gpt_oss_20b", vocab=201088, block=16, context=8192,
             n_new=3),
        # a prompt is read in by 512-row appends, then the first block: time to the first draft
        dict(name="prefill_qwen3_4b", kind="prefill", model="qwen3_4b", vocab=151936, block=16, context=2048),
        # a lightly loaded server: four sequences, sampled at temperature 1, full LM head
        dict(name="batched_4_sampled", kind="batched", model="qwen3_8b", vocab=151936, block=16, n_seq=4,
             lo=301, hi=3000, temperature=1.0),
        # the serving benchmark's 32 ragged sequences through the draft layers
        dict(name="batched_32", kind="batched", model="qwen3_8b", vocab=SMALL_VOCAB, block=16, n_seq=32,
             lo=512, hi=4096, temperature=0.0),
        # training, one draft layer at the benchmark's sequence length and number of anchors
        dict(name="attn_fwd", kind="attn_fwd", n_blocks=512, block=16, T=3072, n_q=32, n_kv=8, hd=128),
        dict(name="attn_bwd", kind="attn_bwd", n_blocks=512, block=16, T=3072, n_q=32, n_kv=8, hd=128),
        # a short sequence with few anchors: 64-wide heads, blocks of 11, ragged everywhere
        dict(name="attn_train_short", kind="attn_train", n_blocks=45, block=11, T=777, n_q=64, n_kv=8, hd=64),
        # the loss over the 151,936-word vocabulary, 256 blocks
        dict(name="ce_151936", kind="ce", n_blocks=256, block=16, vocab=151936),
        # the largest vocabulary, fewer blocks
        dict(name="ce_201088", kind="ce", n_blocks=65, block=16, vocab=201088),
        # a small odd vocabulary: rows that start on no 16-byte boundary
        dict(name="ce_odd", kind="ce", n_blocks=23, block=9, vocab=32003),
    ]


def _log_int(rng, lo, hi):
    """Uniform over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "prefill", "batched", "batched", "attn_fwd", "attn_bwd", "attn_train", "ce", "ce"])
    if kind in ("step", "prefill", "batched"):
        model = rng.choice(["qwen3_4b", "qwen3_8b", "gpt_oss_20b"])
        c = dict(kind=kind, model=model, vocab=SMALL_VOCAB, block=rng.choice([16, 16, rng.randint(4, 15)]))
        if kind == "step":
            c["vocab"] = rng.choice([SMALL_VOCAB, synth.CONFIGS[model].vocab])
            c.update(context=_log_int(rng, 16, synth.CONFIGS[model].context), n_new=rng.randint(1, 16))
        elif kind == "prefill":
            c.update(context=_log_int(rng, 17, 2048))
        else:
            lo = _log_int(rng, 16, 1024)
            c.update(n_seq=_log_int(rng, 2, 32), lo=lo, hi=_log_int(rng, lo + 1, 4096),
                     temperature=rng.choice([0.0, 0.0, 0.7]))
        return c
    if kind == "ce":
        vocab = rng.choice([151936, 201088, _log_int(rng, 1000, 200000), 4 * _log_int(rng, 500, 50000)])
        blocks = max(1, _log_int(rng, 4, max(5, int(256 * 151936 / max(vocab, 40000)))))
        return dict(kind=kind, n_blocks=blocks, block=rng.choice([16, rng.randint(2, 16)]), vocab=vocab)
    n_q, n_kv, hd = rng.choice([(32, 8, 128), (64, 8, 64), (16, 8, 128), (12, 4, 64)])
    return dict(kind=kind, n_blocks=_log_int(rng, 4, 512), block=rng.choice([16, rng.randint(3, 15)]),
                T=_log_int(rng, 50, 3072), n_q=n_q, n_kv=n_kv, hd=hd)


# ---- inputs ---------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _config(case):
    return synth.CONFIGS[case["model"]].replace(vocab=case["vocab"], block_size=case["block"])


def _weights(cfg, seed):
    """Weights (bf16, N(0, 0.02), gains 1 + N(0, 0.02)) and fusion logits N(0, 1)."""
    g = _gen(1000 * seed + 1)
    H, F, V, D, q, kv = cfg.hidden, cfg.ffn, cfg.vocab, cfg.n_draft_layers, cfg.q_dim, cfg.kv_dim
    shapes = {"embed": (V, H), "lm_head": (V, H), "final_norm": (H,), "fuse_norm": (D, H), "attn_norm": (D, H),
              "mlp_norm": (D, H), "wq": (D, q, H), "wk_d": (D, kv, H), "wv_d": (D, kv, H), "wk_t": (D, kv, H),
              "wv_t": (D, kv, H), "wo": (D, H, q), "w_gate": (D, F, H), "w_up": (D, F, H), "w_down": (D, H, F)}
    w = {}
    for name, shape in shapes.items():
        t = torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
        w[name] = t.add_(1.0) if name.endswith("norm") else t
    logits = np.random.default_rng(1000 * seed + 2).standard_normal((D, cfg.n_target_layers)).astype(np.float32)
    return w, logits


def _hidden(cfg, n, seed):
    """n target rows [S, n, H]: N(0, 1), layer s scaled by 1 + 0.2 s."""
    S = cfg.n_target_layers
    h = torch.empty((S, n, cfg.hidden), dtype=torch.bfloat16, device="cuda").normal_(generator=_gen(1000 * seed + 3))
    return h.mul_((1.0 + 0.2 * torch.arange(S, device="cuda")).to(torch.bfloat16)[:, None, None])


def _ids(cfg, n_seq, seed):
    """[x_t, mask, mask, ...] of every sequence."""
    ids = np.full((n_seq, cfg.block_size), cfg.vocab - 1, np.int32)
    ids[:, 0] = np.random.default_rng(1000 * seed + 4).integers(0, cfg.vocab - 1, size=n_seq)
    return ids


def _layout(case, seed):
    """(contexts, rows appended in the pass, first row in the shared stream) per sequence."""
    if case["kind"] == "batched":
        rng = np.random.default_rng(1000 * seed + 5)
        L = rng.integers(case["lo"], case["hi"] + 1, size=case["n_seq"])
        n = np.minimum(rng.integers(1, 17, size=case["n_seq"]), L)
        return [int(x) for x in L], [int(x) for x in n], [16 * i for i in range(case["n_seq"])]
    n = case["context"] if case["kind"] == "prefill" else min(case["n_new"], case["context"])
    return [case["context"]], [n], [0]


class _Draft:
    """A draft model in use: the handle, the inputs of a pass and the buffers it fills."""

    def __init__(self, case, seed):
        cfg = self.cfg = _config(case)
        self.case = case
        self.L, self.n, base = _layout(case, seed)
        n_seq = len(self.L)
        w, logits = _weights(cfg, seed)
        batched = case["kind"] == "batched"
        max_new = max(PREFILL_CHUNK, 16 * n_seq) if batched or case["kind"] == "prefill" else 16
        conf = dfl.make_config(cfg, max(self.L) + 16, max_new, max_batch=n_seq)
        self.h = dfl.dflare_init(conf, w, logits)
        del w
        stream = _hidden(cfg, max(b + l for b, l in zip(base, self.L)), seed)
        for i in range(n_seq):  # the context before the pass
            for s in range(0, self.L[i] - self.n[i], max_new):
                k = min(max_new, self.L[i] - self.n[i] - s)
                rows = stream[:, base[i] + s:base[i] + s + k].contiguous()
                if batched:
                    dfl.dflare_fuse_append_batched(self.h, [i], [k], rows)
                else:
                    dfl.dflare_fuse_append(self.h, rows)
        self.seqs = np.arange(n_seq, dtype=np.int32)
        new = torch.cat([stream[:, b + l - n:b + l] for b, l, n in zip(base, self.L, self.n)], dim=1)
        if case["kind"] == "prefill":
            self.new = [new[:, s:s + PREFILL_CHUNK].contiguous() for s in range(0, new.shape[1], PREFILL_CHUNK)]
        else:
            self.new = [new.contiguous()]
        ids = torch.from_numpy(_ids(cfg, n_seq, seed)).cuda()
        self.ids = ids if batched else ids[0].contiguous()
        self.tokens = torch.empty_like(self.ids)
        self.logits = torch.empty((*self.ids.shape, cfg.vocab), dtype=torch.float32, pin_memory=True)
        self.logits_ptr = ctypes.cast(self.logits.data_ptr(), ctypes.POINTER(ctypes.c_float))
        # logits are kept by the launch that is used without them, too
        dfl.dflare_set_option(self.h, dfl.OPT_CAPTURE_PERSISTENT, 1)
        dfl.dflare_debug_capture(self.h, True)
        dfl.dflare_debug_capture(self.h, False)
        torch.cuda.synchronize()

    def __del__(self):
        if getattr(self, "h", None):
            dfl.dflare_destroy(self.h)
            self.h = None

    def step(self):
        h, case = self.h, self.case
        if case["kind"] == "batched":
            dfl.dflare_set_sampling(h, case["temperature"], 1)
            for i, (L, n) in enumerate(zip(self.L, self.n)):
                if dfl.dflare_context_len_seq(h, i) != L - n:
                    dfl.dflare_truncate_seq(h, i, L - n)
            dfl.dflare_fuse_append_batched(h, self.seqs, self.n, self.new[0])
        else:
            dfl.dflare_truncate(h, min(self.L[0] - self.n[0], dfl.dflare_context_len(h)))
            for rows in self.new:
                dfl.dflare_fuse_append(h, rows)
        dfl.dflare_debug_capture(h, True)  # keep the logits of the drafted block (not the fused rows above)
        if case["kind"] == "batched":
            dfl.dflare_draft_block_batched(h, self.seqs, self.ids, self.tokens)
            what = dfl.DBG_BLOGITS
        else:
            dfl.dflare_draft_block(h, self.ids, self.tokens)
            what = dfl.DBG_LOGITS
        dfl.dflare_debug_capture(h, False)
        rc = dfl.lib().dflare_debug_read(h, what, 0, self.logits_ptr, self.logits.numel())
        if rc != dfl.OK:
            raise dfl.DFlareError(rc, "reading the logits")
        return [self.tokens, self.logits]


def _attn_inputs(case, seed):
    g = _gen(1000 * seed + 6)
    n, B, T, hd = case["n_blocks"], case["block"], case["T"], case["hd"]

    def bf(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g)

    q, kc, vc = bf(n * B, case["n_q"], hd), bf(T, case["n_kv"], hd), bf(T, case["n_kv"], hd)
    kb, vb = bf(n * B, case["n_kv"], hd), bf(n * B, case["n_kv"], hd)
    # anchors lie anywhere in the sequence that leaves room for the block
    anchors = torch.randint(0, max(T - B, 0) + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
    dout = torch.empty((n * B, case["n_q"], hd), dtype=torch.float32, device="cuda").normal_(generator=g)
    return q, kc, vc, kb, vb, anchors, dout


def _ce_inputs(case, seed):
    g = _gen(1000 * seed + 7)
    rows, V = case["n_blocks"] * case["block"], case["vocab"]
    z = torch.empty((rows, V), dtype=torch.float32, device="cuda").normal_(0.0, 3.0, generator=g)
    y = torch.randint(0, V, (rows,), generator=g, device="cuda", dtype=torch.int32)
    y[torch.rand(rows, generator=g, device="cuda") < 0.05] = -1  # positions without a target
    return z, y


GAMMA = 4.5


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "prefill", "batched"):
        return _Draft(case, seed)
    if kind == "ce":
        return kind, case, _ce_inputs(case, seed)
    x = _attn_inputs(case, seed)
    saved = dfl.anchor_attention_fwd(*x[:6], case["block"]) if kind == "attn_bwd" else None
    return kind, case, x, saved


def run(state):
    if isinstance(state, _Draft):
        return state.step()
    kind, case = state[0], state[1]
    B = case["block"]
    if kind == "ce":
        z, y = state[2]
        return list(dfl.weighted_ce(z, y, B, GAMMA))
    *inp, dout = state[2]
    if kind == "attn_bwd":
        return list(dfl.anchor_attention_bwd(*inp, B, *state[3], dout))
    out, lse = dfl.anchor_attention_fwd(*inp, B)
    if kind == "attn_fwd":
        return [out, lse]
    return [out, lse, *dfl.anchor_attention_bwd(*inp, B, out, lse, dout)]


# ---- work -----------------------------------------------------------------------------------

def work(case):
    if case["kind"] == "ce":
        rows, V = case["n_blocks"] * case["block"], case["vocab"]
        return {"bytes": 8 * rows * V + 8 * rows, "flops": 6 * rows * V}
    if case["kind"].startswith("attn"):
        n, B, T, hd, n_q, n_kv = (case[k] for k in ("n_blocks", "block", "T", "hd", "n_q", "n_kv"))
        fwd = 4.0 * n * B * n_q * hd * (max(T - B, 0) / 2 + B)   # anchors are uniform
        inputs = 2 * (n * B * n_q * hd + 2 * (T + n * B) * n_kv * hd)
        rows4 = 4 * n * B * n_q * hd
        grads = rows4 + 8 * (T + n * B) * n_kv * hd
        stats = 4 * n * B * n_q
        passes = {"attn_fwd": (inputs + rows4 + stats, fwd),
                  "attn_bwd": (inputs + 2 * rows4 + stats + grads, 2.5 * fwd),
                  "attn_train": (inputs + 2 * rows4 + stats + grads, 3.5 * fwd)}
        b, f = passes[case["kind"]]
        return {"bytes": int(b), "flops": int(f)}
    cfg = _config(case)
    L, n, _ = _layout(case, 0)
    H, F, V, D, S, B = cfg.hidden, cfg.ffn, cfg.vocab, cfg.n_draft_layers, cfg.n_target_layers, cfg.block_size
    q, kv = cfg.q_dim, cfg.kv_dim
    layer = H * q + 2 * H * kv + q * H + 3 * H * F
    rows, new, ctx = len(L) * B, sum(n), sum(L)
    weights = 2 * (D * (layer + 2 * H * kv) + V * H)
    cache = 2 * D * 2 * kv * ctx                      # context keys and values, read once (16 bits)
    moved = 2 * S * new * H + 2 * D * 2 * kv * new + 2 * rows * H + 4 * rows * V
    flops = 2 * rows * (D * layer + V * H) + 2 * new * D * (2 * H * kv + S * H) \
        + 4 * D * q * B * sum(l + B for l in L)
    return {"bytes": weights + cache + moved, "flops": flops}


def tolerance(case):
    """About four times the largest relative error against 64 bits over the declared ranges."""
    kind = case["kind"]
    if kind == "ce":
        return {"rel": 1e-6, "max": 1e-5}
    if kind.startswith("attn"):
        return {"rel": 1e-2, "max": 0.1}
    # random weights leave near ties between the best logits; one row of a batch-1 block may flip
    return {"rel": 1e-2, "max": 0.06, "differ": 0.13}


# ---- 64-bit results ---------------------------------------------------------------------------

def _rms(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, pos, base):
    """x [n, heads, hd] at positions pos [n], rotate-half convention."""
    half = x.shape[-1] // 2
    freq = base ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / x.shape[-1])
    th = pos.double()[:, None] * freq
    c, s = torch.cos(th)[:, None], torch.sin(th)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _exact_draft(case, seed):
    cfg = _config(case)
    L, _, base = _layout(case, seed)
    w, fusion = _weights(cfg, seed)
    R = max(b + l for b, l in zip(base, L))
    stream = _hidden(cfg, R, seed)
    ids = torch.from_numpy(_ids(cfg, len(L), seed)).cuda().long()
    alpha = torch.softmax(torch.from_numpy(fusion).double().cuda(), dim=-1)
    B, nq, nkv, hd, eps, rb = cfg.block_size, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.rms_eps, cfg.rope_base
    G = nq // nkv
    X = w["embed"][ids.reshape(-1)].double()
    blk = [torch.arange(l, l + B, device="cuda") for l in L]
    for i in range(cfg.n_draft_layers):
        wk, wv = w["wk_t"][i].double().t().contiguous(), w["wv_t"][i].double().t().contiguous()
        ck, cv = [], []
        for s in range(0, R, 512):
            u = torch.zeros((min(512, R - s), cfg.hidden), dtype=torch.float64, device="cuda")
            for j in range(cfg.n_target_layers):
                u.add_(stream[j, s:s + 512].double(), alpha=float(alpha[i, j]))
            f = _rms(u, w["fuse_norm"][i], eps)
            ck.append(f @ wk)
            cv.append(f @ wv)
        ck, cv = torch.cat(ck).view(R, nkv, hd), torch.cat(cv).view(R, nkv, hd)
        a = _rms(X, w["attn_norm"][i], eps)
        pos = torch.cat(blk)
        q = _rope((a @ w["wq"][i].double().t()).view(-1, nq, hd), pos, rb)
        kb = _rope((a @ w["wk_d"][i].double().t()).view(-1, nkv, hd), pos, rb)
        vb = (a @ w["wv_d"][i].double().t()).view(-1, nkv, hd)
        o = torch.empty_like(q)
        for m, (l, b0) in enumerate(zip(L, base)):
            r = slice(m * B, (m + 1) * B)
            k = torch.cat([_rope(ck[b0:b0 + l], torch.arange(l, device="cuda"), rb), kb[r]])
            v = torch.cat([cv[b0:b0 + l], vb[r]])
            for g in range(nkv):
                qq = q[r, g * G:(g + 1) * G].reshape(B * G, hd)
                p = torch.softmax(qq @ k[:, g].t().contiguous() / math.sqrt(hd), dim=-1)
                o[r, g * G:(g + 1) * G] = (p @ v[:, g].contiguous()).view(B, G, hd)
        X = X + o.reshape(-1, nq * hd) @ w["wo"][i].double().t()
        a = _rms(X, w["mlp_norm"][i], eps)
        gate = a @ w["w_gate"][i].double().t()
        X = X + (gate * torch.sigmoid(gate) * (a @ w["w_up"][i].double().t())) @ w["w_down"][i].double().t()
    a = _rms(X, w["final_norm"], eps)
    z = torch.cat([a @ w["lm_head"][s:s + 16384].double().t() for s in range(0, cfg.vocab, 16384)], dim=-1)
    tokens = None if case.get("temperature", 0.0) > 0 else z.argmax(-1).int()  # the draws have no 64-bit form here
    shape = tuple(ids.shape) if case["kind"] == "batched" else (B,)
    return [None if tokens is None else tokens.view(shape), z.view(*shape, cfg.vocab)]


def _exact_attn(case, seed):
    n, B, T, nq, nkv, hd = (case[k] for k in ("n_blocks", "block", "T", "n_q", "n_kv", "hd"))
    q, kc, vc, kb, vb, anchors, dout = (t.double() if t.is_floating_point() else t for t in _attn_inputs(case, seed))
    G, scale = nq // nkv, 1.0 / math.sqrt(hd)
    hidden_keys = torch.arange(T, device="cuda")[None, :] >= anchors.repeat_interleave(G * B)[:, None]  # [n G B, T]
    out, lse, dq = torch.empty_like(q), torch.empty((n * B, nq), dtype=torch.float64, device="cuda"), torch.empty_like(q)
    dkc, dvc, dkb, dvb = (torch.empty_like(t) for t in (kc, vc, kb, vb))

    def rows(x, g):  # [n B, n_q, hd] -> the rows of KV head g, block by block: [n G B, hd]
        return x.view(n, B, nq, -1)[:, :, g * G:(g + 1) * G].permute(0, 2, 1, 3).reshape(n * G * B, -1)

    def unrows(x):
        return x.view(n, G, B, -1).permute(0, 2, 1, 3).reshape(n * B, G, -1)

    for g in range(nkv):
        k, v = kc[:, g].contiguous(), vc[:, g].contiguous()
        k1, v1 = kb[:, g].reshape(n, B, hd), vb[:, g].reshape(n, B, hd)
        k1t, v1t = k1.transpose(1, 2).contiguous(), v1.transpose(1, 2).contiguous()
        qq, do = rows(q, g), rows(dout, g)
        blocks = lambda x: x.view(n, G * B, -1)
        s = torch.cat([(qq @ k.t()).masked_fill(hidden_keys, -math.inf),
                       torch.bmm(blocks(qq), k1t).view(n * G * B, B)], dim=1) * scale
        ls = torch.logsumexp(s, dim=1, keepdim=True)
        p = torch.exp(s - ls)
        pc, pb = p[:, :T].contiguous(), blocks(p[:, T:].contiguous())
        o = pc @ v + torch.bmm(pb, v1).view(n * G * B, hd)
        out[:, g * G:(g + 1) * G], lse[:, g * G:(g + 1) * G] = unrows(o), unrows(ls)[..., 0]
        d = (do * o).sum(1, keepdim=True)
        dsc = pc * (do @ v.t() - d) * scale
        dsb = pb * (torch.bmm(blocks(do), v1t) - blocks(d)) * scale
        dq[:, g * G:(g + 1) * G] = unrows(dsc @ k + torch.bmm(dsb, k1).view(n * G * B, hd))
        dkc[:, g], dvc[:, g] = dsc.t() @ qq, pc.t() @ do
        dkb[:, g] = torch.bmm(dsb.transpose(1, 2).contiguous(), blocks(qq)).reshape(n * B, hd)
        dvb[:, g] = torch.bmm(pb.transpose(1, 2).contiguous(), blocks(do)).reshape(n * B, hd)
    grads = [dq, dkc, dvc, dkb, dvb]
    return {"attn_fwd": [out, lse], "attn_bwd": grads, "attn_train": [out, lse, *grads]}[case["kind"]]


def _exact_ce(case, seed):
    z, y = _ce_inputs(case, seed)
    rows, B = z.shape[0], case["block"]
    b = torch.arange(rows, device="cuda") % B
    on = (b > 0) & (y >= 0)
    w = torch.exp(-(b - 1).double() / GAMMA) * on
    total = w.sum().clamp_min(1e-300)
    ce = torch.zeros(rows, dtype=torch.float64, device="cuda")
    dz = torch.empty(z.shape, dtype=torch.float64, device="cuda")
    for s in range(0, rows, 512):
        x = z[s:s + 512].double()
        r = torch.arange(x.shape[0], device="cuda")
        label = y[s:s + 512].clamp_min(0).long()
        lse = torch.logsumexp(x, dim=1)
        ce[s:s + 512] = torch.where(on[s:s + 512], lse - x[r, label], 0.0)
        p = torch.exp(x - lse[:, None])
        p[r, label] -= 1.0
        dz[s:s + 512] = p * (w[s:s + 512] / total)[:, None]
    return [((w * ce).sum() / total).view(1), ce, dz]


def exact(case, seed):
    with torch.no_grad():
        if case["kind"] == "ce":
            return _exact_ce(case, seed)
        if case["kind"].startswith("attn"):
            return _exact_attn(case, seed)
        return _exact_draft(case, seed)
