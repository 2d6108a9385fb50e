"""GPU parity of the batched draft step: several sequences, each with its own context
cache and length, appended to and drafted together through the batched C-ABI calls,
against one fp64 oracle per sequence on the same seeded inputs (the bar of
tests/parity.py).

Sizes finish in seconds on the oracle yet span several 128-row GEMM groups, ragged
row counts (B = 5 gives sequences that straddle 16-row tiles), empty and one-row
contexts, contexts on and off the 64-key block and 512-key range grids of the
attention, 64 and 128 query rows per KV head, vocabularies that are not a multiple of
16, slots listed out of order and calls on subsets of the slots.

Besides the oracle bar, two batched results are compared directly: the same sequence
drafted by batched calls of other shapes (other rows, other K splits), and by the
batch-1 path.  The batched GEMMs take fp16 operands, rounded to 2^-11 relative; which
way each rounding falls depends on the order of the fp32 sums before it (the K split),
and the draft layers carry such differences forward, so a batched result sits about
2.5e-3 of the logit range from the exact one at full size (1e-3 on the small cases
here) and any two of them, or one and the batch-1 path's, agree within AGREE_TOL =
5e-3, a quarter of the oracle bar.
"""
import numpy as np
import pytest
import torch

from oracle import dflare_oracle as orc
from paper_2606_02091_amd import dflare as dfl
from paper_2606_02091_amd import synth
import parity as P

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

AGREE_TOL = 5e-3

CASES = {
    # name: (config, context length per listed slot, slots, max_batch)
    "hd128_b16": (synth.ModelConfig("bhd128", hidden=256, n_q_heads=4, n_kv_heads=1, head_dim=128, ffn=512,
                                    vocab=4001, n_draft_layers=2, n_target_layers=8, block_size=16, context=300),
                  [0, 1, 40, 128, 129, 200, 300, 77, 255], [3, 0, 7, 1, 9, 4, 11, 2, 5], 12),
    "hd64_gqa_b5": (synth.ModelConfig("bhd64", hidden=96, n_q_heads=6, n_kv_heads=2, head_dim=64, ffn=160,
                                      vocab=1000, n_draft_layers=3, n_target_layers=5, block_size=5, context=130,
                                      random_block=True),
                    [33, 0, 130, 7, 64], [1, 4, 0, 2, 3], 5),
    # 8 query heads per KV head (128 query rows per work item) and contexts spanning
    # several 512-key attention ranges, one of them ending a single key into a range
    "hd128_gqa8_long": (synth.ModelConfig("bgqa8", hidden=128, n_q_heads=8, n_kv_heads=1, head_dim=128,
                                          ffn=256, vocab=700, n_draft_layers=2, n_target_layers=3,
                                          block_size=16, context=1030),
                        [497, 1030, 0, 700, 511], [2, 0, 4, 1, 3], 5),
    "hd64_gqa8_long": (synth.ModelConfig("bgqa8h64", hidden=128, n_q_heads=16, n_kv_heads=2, head_dim=64,
                                         ffn=256, vocab=900, n_draft_layers=2, n_target_layers=3,
                                         block_size=16, context=1100),
                       [1100, 496, 40], [1, 0, 2], 3),
}


def dev(bits):
    return dfl.bf16_tensor(bits)


def ids_tensor(ids):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(ids, np.int32))).cuda()


def slot_rows(cfg, slot, start, n):
    return synth.hidden_rows(cfg, start, n, seed=100 + slot)


def slot_ids(cfg, slot, step=0):
    return synth.block_ids(cfg, step=step, seed=200 + slot)


def build_batched(cfg, lengths, slots, max_batch, seed=5):
    """Fill every slot's context with batched appends of 1..16 rows per listed sequence,
    in rounds where the order of the sequences changes and some sequences sit out."""
    w, lg = P.weights_for(cfg)
    maxc = max(lengths) + 64
    model = dfl.DraftModel(cfg, w, lg, max_context=maxc, max_new=16 * max_batch, max_batch=max_batch)
    dfl.dflare_debug_capture(model.h, True)
    orcs = {s: P.oracle_for(cfg, w, lg, maxc) for s in slots}
    target = dict(zip(slots, lengths))
    filled = {s: 0 for s in slots}
    rng = np.random.default_rng(seed)
    last = None
    while any(filled[s] < target[s] for s in slots):
        seq, nn, parts, fused = [], [], [], []
        for s in rng.permutation(slots):
            s = int(s)
            left = target[s] - filled[s]
            if left <= 0 or rng.random() < 0.3:
                continue
            n = int(min(left, rng.integers(1, 17)))
            rows = slot_rows(cfg, s, filled[s], n)
            seq.append(s)
            nn.append(n)
            parts.append(rows)
            fused.append(orcs[s].append(rows))
            filled[s] += n
        if seq:
            model.fuse_append_batched(seq, nn, dev(np.concatenate(parts, axis=1)))
            last = np.concatenate(fused, axis=1)
    torch.cuda.synchronize()
    return model, orcs, last


def compare_draft(model, orcs, cfg, seq, step=0):
    B, V = cfg.block_size, cfg.vocab
    ids = np.stack([slot_ids(cfg, s, step) for s in seq])
    out = model.draft_block_batched(seq, ids_tensor(ids))
    torch.cuda.synchronize()
    tokens = out.cpu().numpy()
    logits = dfl.dflare_debug_read(model.h, dfl.DBG_BLOGITS, 0, (len(seq), B, V))
    worst = 0.0
    for i, s in enumerate(seq):
        ref = orcs[s].draft_block(ids[i])
        e = P.relinf(logits[i], ref["logits"])
        assert e <= P.REL_TOL, (s, e)
        P.check_tokens(tokens[i], ref["logits"])
        worst = max(worst, e)
    return tokens, logits, worst


@pytest.mark.parametrize("name", list(CASES))
def test_batched_matches_oracles(name):
    cfg, lengths, slots, max_batch = CASES[name]
    print(f"[batched] {name}: slots {slots} lengths {lengths}", flush=True)
    model, orcs, last_fused = build_batched(cfg, lengths, slots, max_batch)
    for s, L in zip(slots, lengths):
        assert dfl.dflare_context_len_seq(model.h, s) == L
    # fused rows of the last batched append (all of its rows, in call order)
    for i in range(cfg.n_draft_layers):
        got = dfl.dflare_debug_read(model.h, dfl.DBG_FUSED, i, (last_fused.shape[1], cfg.hidden))
        assert P.relinf(got, last_fused[i]) <= P.REL_TOL
    # every slot's cache
    for s, L in zip(slots, lengths):
        for i in range(cfg.n_draft_layers):
            for what, ref in ((dfl.DBG_KCACHE, orcs[s].k_cache[i]), (dfl.DBG_VCACHE, orcs[s].v_cache[i])):
                got = dfl.dflare_debug_read_seq(model.h, what, s, i, (L, cfg.n_kv_heads, cfg.head_dim))
                assert P.relinf(got, ref) <= P.REL_TOL, (s, i, what)
    # all slots, in the listed order
    tokens, logits, worst = compare_draft(model, orcs, cfg, slots)
    print(f"[batched] {name}: {len(slots)} sequences, logits rel err {worst:.2e}", flush=True)
    # a subset in another order gives the same rows
    sub = slots[::-2]
    t2, l2, _ = compare_draft(model, orcs, cfg, sub)
    for j, s in enumerate(sub):
        i = slots.index(s)
        assert P.relinf(l2[j], logits[i]) <= AGREE_TOL
    model.close()


# calls of one to eight row tiles (the weight-streaming GEMM picks its shape by them), ragged rows
# (B = 13); k-tiles per wave from none (H = 96: three k-tiles for four waves) to several, residual
# projections with and without a K split (q = 1,024, F = 2,080), four output tiles per work-group for
# three and four row tiles (Q/K/V, gate/up and LM head of more than 1,020 output tiles; 1,027 in the LM
# head, so that its last work-group has three), greedy and sampled
@pytest.mark.parametrize("hidden,n_q,n_kv,hd,ffn,vocab", [(96, 4, 2, 64, 160, 1001), (1056, 8, 2, 128, 2080, 1001),
                                                          (160, 64, 32, 128, 8224, 16421)])
def test_batched_few_rows(hidden, n_q, n_kv, hd, ffn, vocab):
    cfg = synth.ModelConfig("few", hidden=hidden, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=hd, ffn=ffn, vocab=vocab,
                            n_draft_layers=2, n_target_layers=3, block_size=13, context=40, random_block=True)
    slots = [5, 0, 3, 9, 1, 7, 2, 8, 4]
    print(f"[batched] few rows H={hidden}", flush=True)
    model, orcs, _ = build_batched(cfg, [40, 7, 0, 16, 33, 1, 12, 25, 18], slots, 10)
    for n in (1, 2, 3, 4, 5, 6, 9):
        tokens, logits, worst = compare_draft(model, orcs, cfg, slots[:n])
        print(f"[batched] few rows H={hidden}: {n} sequences, logits rel err {worst:.2e}", flush=True)
        dfl.dflare_set_sampling(model.h, 0.8, 11)
        ids = np.stack([slot_ids(cfg, s) for s in slots[:n]])
        drawn = model.draft_block_batched(slots[:n], ids_tensor(ids)).cpu().numpy()
        for i, s in enumerate(slots[:n]):
            want, scores = orc.sample_tokens(logits[i].astype(np.float64), 0.8, 11, 0, slot=s)
            # the scores of the kernel's own logits, in fp32: the noise's logarithms err by 1e-5 at most
            for b in range(cfg.block_size):
                assert scores[b][drawn[i][b]] >= scores[b][want[b]] - 1e-4, (n, s, b)
        dfl.dflare_set_sampling(model.h, 0.0, 0)
    model.close()


# calls of nine and ten row tiles on the tiled GEMM, whose residual projections leave their K parts to
# the norm: a second group of row tiles that is not full, a last column group that is not (66
# output tiles), parts of unequal length (33 and 65 k-tiles), ragged rows (B = 13); and projections too
# short for a split (8 and 5 k-tiles), which add to the residual stream themselves
@pytest.mark.parametrize("hidden,n_q,hd,ffn", [(1056, 8, 128, 2080), (96, 4, 64, 160)])
def test_batched_residual_parts(hidden, n_q, hd, ffn):
    cfg = synth.ModelConfig("parts", hidden=hidden, n_q_heads=n_q, n_kv_heads=2, head_dim=hd, ffn=ffn, vocab=501,
                            n_draft_layers=2, n_target_layers=3, block_size=13, context=40, random_block=True)
    slots = [5, 0, 3, 9, 1, 7, 2, 8, 4, 11, 6, 10]
    print("[batched] residual parts", flush=True)
    model, orcs, _ = build_batched(cfg, [40, 7, 0, 16, 33, 1, 12, 25, 18, 3, 39, 22], slots, 12)
    for n in (11, 12):
        _, _, worst = compare_draft(model, orcs, cfg, slots[:n])
        print(f"[batched] residual parts: {n} sequences, logits rel err {worst:.2e}", flush=True)
    model.close()


# attention items of 512, 256 and 128 keys (264 items of 512 with twelve sequences; eight and three
# sequences have fewer than there are CUs), keys ending at a range, one past it and inside
def test_batched_attention_ranges():
    cfg = synth.ModelConfig("ranges", hidden=128, n_q_heads=8, n_kv_heads=8, head_dim=64, ffn=160, vocab=501,
                            n_draft_layers=1, n_target_layers=2, block_size=16, context=1100)
    slots = list(range(12))
    print("[batched] attention ranges", flush=True)
    lengths = [1100, 496, 1009, 1008, 1030, 1024, 1070, 1100, 1010, 1050, 1090, 1023]
    model, orcs, _ = build_batched(cfg, lengths, slots, 12)
    for n in (12, 8, 3):
        _, _, worst = compare_draft(model, orcs, cfg, slots[:n])
        print(f"[batched] attention ranges: {n} sequences, logits rel err {worst:.2e}", flush=True)
    model.close()


# an LM-head row of NaN: its id loses to every finite score, in calls of few rows (the weight-streaming GEMM)
# and of more (n = 11), greedy and sampled.  The row is the first of 16 output columns, in the tile and the group of
# tiles of the token that the first block row gets without it
def test_batched_nan_logit_loses():
    cfg = synth.ModelConfig("nan", hidden=96, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=160, vocab=1001,
                            n_draft_layers=1, n_target_layers=3, block_size=13, context=40, random_block=True)
    w, lg = P.weights_for(cfg)
    slots = list(range(11))
    orcs = {s: P.oracle_for(cfg, w, lg, 64) for s in slots}
    for s in slots:
        orcs[s].append(slot_rows(cfg, s, 0, 5))
    ids = np.stack([slot_ids(cfg, s) for s in slots])
    clean = np.stack([np.array(orcs[s].draft_block(ids[i])["logits"]) for i, s in enumerate(slots)])
    bad = sorted({int(t) // 64 * 64 for t in clean[0].argmax(-1)} | {int(t) // 16 * 16 for t in clean[0].argmax(-1)})
    w["lm_head"] = w["lm_head"].copy()
    w["lm_head"][bad] = 0x7FC0
    clean[:, :, bad] = -np.inf
    model = dfl.DraftModel(cfg, w, lg, max_context=64, max_new=16 * len(slots), max_batch=len(slots))
    model.fuse_append_batched(slots, [5] * len(slots), dev(np.concatenate([slot_rows(cfg, s, 0, 5) for s in slots], axis=1)))
    for n in (1, 2, 4, 5, 9, 11):
        print(f"[batched] NaN logit: {n} sequences", flush=True)
        tokens = model.draft_block_batched(slots[:n], ids_tensor(ids[:n])).cpu().numpy()
        for i in range(n):
            P.check_tokens(tokens[i], clean[i])
        dfl.dflare_set_sampling(model.h, 0.8, 11)
        drawn = model.draft_block_batched(slots[:n], ids_tensor(ids[:n])).cpu().numpy()
        dfl.dflare_set_sampling(model.h, 0.0, 0)
        for i, s in enumerate(slots[:n]):
            _, scores = orc.sample_tokens(clean[i], 0.8, 11, 0, slot=s)
            for b in range(cfg.block_size):
                assert scores[b][drawn[i][b]] >= scores[b].max() - P.MARGIN, (n, s, b)
    model.close()


# the tuning overrides of the K split and the tile width act in calls of few rows too: another split adds in
# another order, so the bits differ, and the result stays at the oracle
def test_batched_overrides_act_in_small_calls(monkeypatch):
    cfg = synth.ModelConfig("over", hidden=1056, n_q_heads=8, n_kv_heads=2, head_dim=128, ffn=2080, vocab=501,
                            n_draft_layers=2, n_target_layers=3, block_size=13, context=40, random_block=True)
    slots = [1, 0, 2]
    got = {}
    for name in ("", "QKV", "O", "DOWN"):
        for kg in (1, 3) if name else (0,):
            for k in ("QKV", "O", "DOWN"):  # the others without a split
                monkeypatch.setenv(f"DFLARE_BSPLIT_{k}", str(kg) if k == name else "1")
            if not name:
                for k in ("QKV", "O", "DOWN"):
                    monkeypatch.delenv(f"DFLARE_BSPLIT_{k}")
            model, orcs, _ = build_batched(cfg, [40, 7, 16], slots, 3)
            _, got[name, kg], worst = compare_draft(model, orcs, cfg, slots)
            print(f"[batched] DFLARE_BSPLIT_{name}={kg}: logits rel err {worst:.2e}", flush=True)
            model.close()
    for name in ("QKV", "O", "DOWN"):
        assert not np.array_equal(got[name, 1], got[name, 3]), name
    assert np.array_equal(got["QKV", 1], got["O", 1]) and np.array_equal(got["QKV", 1], got["DOWN", 1])


# an override set after the handle was made cannot ask for more than its partial area holds
def test_batched_override_after_init_stays_in_bounds(monkeypatch):
    cfg = synth.ModelConfig("late", hidden=1056, n_q_heads=8, n_kv_heads=2, head_dim=128, ffn=2080, vocab=501,
                            n_draft_layers=2, n_target_layers=3, block_size=13, context=40, random_block=True)
    slots = [1, 0, 2]
    print("[batched] late override", flush=True)
    model, orcs, _ = build_batched(cfg, [40, 7, 16], slots, 3)
    for name in ("QKV", "O", "GU", "DOWN"):
        monkeypatch.setenv(f"DFLARE_BSPLIT_{name}", "8")
    compare_draft(model, orcs, cfg, slots)
    model.close()


def test_batched_single_equals_batch1():
    """Slot 0 through the batch-1 calls, slot 1 through the batched calls, same rows."""
    cfg = CASES["hd128_b16"][0]
    w, lg = P.weights_for(cfg)
    L = 190
    model = dfl.DraftModel(cfg, w, lg, max_context=L + 64, max_new=16, max_batch=2)
    dfl.dflare_debug_capture(model.h, True)
    orc = P.oracle_for(cfg, w, lg, L + 64)
    s = 0
    for n in synth.append_sizes(40, seed=6):
        n = int(min(n, L - s))
        if n <= 0:
            break
        rows = slot_rows(cfg, 0, s, n)
        model.fuse_append(dev(rows))
        model.fuse_append_batched([1], [n], dev(rows))
        orc.append(rows)
        s += n
    torch.cuda.synchronize()
    assert model.context_len == L and dfl.dflare_context_len_seq(model.h, 1) == L
    for i in range(cfg.n_draft_layers):
        for what in (dfl.DBG_KCACHE, dfl.DBG_VCACHE):
            a = dfl.dflare_debug_read_seq(model.h, what, 0, i, (L, cfg.n_kv_heads, cfg.head_dim))
            b = dfl.dflare_debug_read_seq(model.h, what, 1, i, (L, cfg.n_kv_heads, cfg.head_dim))
            assert P.relinf(b, a) <= AGREE_TOL, (i, what)
    for step in range(2):
        ids = slot_ids(cfg, 0, step)
        t1 = model.draft_block(ids_tensor(ids)).cpu().numpy()
        z1 = dfl.dflare_debug_read(model.h, dfl.DBG_LOGITS, 0, (cfg.block_size, cfg.vocab))
        tb = model.draft_block_batched([1], ids_tensor(ids[None])).cpu().numpy()[0]
        zb = dfl.dflare_debug_read(model.h, dfl.DBG_BLOGITS, 0, (1, cfg.block_size, cfg.vocab))[0]
        ref = orc.draft_block(ids)
        assert P.relinf(zb, ref["logits"]) <= P.REL_TOL
        assert P.relinf(zb, z1) <= AGREE_TOL
        P.check_tokens(t1, ref["logits"])
        P.check_tokens(tb, ref["logits"])
        # the batched call on slot 0 reads the batch-1 context
        t0 = model.draft_block_batched([0], ids_tensor(ids[None])).cpu().numpy()[0]
        z0 = dfl.dflare_debug_read(model.h, dfl.DBG_BLOGITS, 0, (1, cfg.block_size, cfg.vocab))[0]
        assert P.relinf(z0, z1) <= AGREE_TOL
        assert P.relinf(z0, zb) <= AGREE_TOL
        P.check_tokens(t0, ref["logits"])
    model.close()


def test_batched_truncate_and_validation():
    cfg = CASES["hd64_gqa_b5"][0]
    w, lg = P.weights_for(cfg)
    model = dfl.DraftModel(cfg, w, lg, max_context=24, max_new=20, max_batch=3)
    dfl.dflare_debug_capture(model.h, True)
    orcs = {s: P.oracle_for(cfg, w, lg, 24) for s in range(3)}
    rows = {s: slot_rows(cfg, s, 0, 30) for s in range(3)}
    model.fuse_append_batched([2, 0], [10, 6], dev(np.concatenate([rows[2][:, :10], rows[0][:, :6]], axis=1)))
    orcs[2].append(rows[2][:, :10])
    orcs[0].append(rows[0][:, :6])
    h = model.h

    def err(fn, *a):
        with pytest.raises(dfl.DFlareError) as e:
            fn(*a)
        return e.value.status

    x = dev(rows[1][:, :4])
    assert err(dfl.dflare_fuse_append_batched, h, [1, 1], [2, 2], x) == dfl.ERR_INVALID_ARG   # repeated slot
    assert err(dfl.dflare_fuse_append_batched, h, [3], [4], x) == dfl.ERR_INVALID_ARG         # slot out of range
    assert err(dfl.dflare_fuse_append_batched, h, [1], [0], x) == dfl.ERR_INVALID_ARG         # empty append
    big = dev(np.concatenate([rows[1][:, :15], rows[0][:, :6]], axis=1))
    assert err(dfl.dflare_fuse_append_batched, h, [1, 0], [15, 6], big) == dfl.ERR_INVALID_ARG  # sum > max_new
    full = dev(np.concatenate([rows[1][:, :4], rows[2][:, :16]], axis=1))
    assert err(dfl.dflare_fuse_append_batched, h, [1, 2], [4, 16], full) == dfl.ERR_CONTEXT_FULL
    ids = ids_tensor(np.zeros((2, cfg.block_size)))
    assert err(dfl.dflare_draft_block_batched, h, [0, 0], ids, ids) == dfl.ERR_INVALID_ARG
    assert err(dfl.dflare_truncate_seq, h, 2, 11) == dfl.ERR_INVALID_ARG
    # failed calls changed nothing
    assert [dfl.dflare_context_len_seq(h, s) for s in range(3)] == [6, 0, 10]
    # truncate one slot, append to it again, draft all three (slot 1 empty)
    dfl.dflare_truncate_seq(h, 2, 7)
    orcs[2].truncate(7)
    model.fuse_append_batched([2], [3], dev(rows[1][:, 20:23]))
    orcs[2].append(rows[1][:, 20:23])
    assert [dfl.dflare_context_len_seq(h, s) for s in range(3)] == [6, 0, 10]
    assert model.context_len == 6
    compare_draft(model, orcs, cfg, [1, 2, 0])
    model.close()
