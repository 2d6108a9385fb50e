"""GPU parity of the training-side kernels against the fp64 oracle (oracle/training_oracle.py)
on the same seeded bf16 inputs: anchor attention (Sec. 3.3) forward and backward, and the
progressive position-weighted cross-entropy (Eq. 5).

Shapes span several 32-key tiles with ragged tails, block sizes 16 and 5, GQA groups of 4 and
3, more blocks than one 64-block gradient chunk, anchors 0 (no context) and T (all of it), and
T = 0.  The attention's products run on bf16 matrix cores with probabilities and gradients
rounded to bf16 as operands; the bar is the per-tensor relative error of tests/parity.py
(2e-2 of the tensor's largest magnitude).  Gradients must repeat bit for bit.
"""
import numpy as np
import pytest
import torch

from oracle import training_oracle as tr
from paper_2606_02091_amd import dflare as dfl
from paper_2606_02091_amd import synth
import parity as P

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

CASES = {
    # name: (n_blocks, B, T, n_q, n_kv, hd)
    "b16_hd128": (5, 16, 200, 8, 2, 128),
    "b5_hd64_gqa3": (7, 5, 77, 6, 2, 64),
    "chunks_hd64": (150, 4, 300, 4, 1, 64),
    "no_context": (3, 8, 0, 4, 2, 128),
}


def inputs(n, B, T, nq, nkv, hd, seed=0):
    rng = np.random.default_rng(seed)

    def bf(shape):
        return synth.round_bf16(rng.standard_normal(shape).astype(np.float32))

    x = dict(q=bf((n * B, nq, hd)), k_ctx=bf((T, nkv, hd)), v_ctx=bf((T, nkv, hd)),
             k_blk=bf((n * B, nkv, hd)), v_blk=bf((n * B, nkv, hd)))
    anchors = rng.integers(0, T + 1, size=n).astype(np.int32)
    if n >= 2:
        anchors[0], anchors[1] = 0, T
    dout = rng.standard_normal((n * B, nq, hd))
    return x, anchors, dout


def dev(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda()


@pytest.mark.parametrize("name", list(CASES))
def test_anchor_attention_matches_oracle(name):
    n, B, T, nq, nkv, hd = CASES[name]
    print(f"[training] attention {name}", flush=True)
    x, anchors, dout = inputs(n, B, T, nq, nkv, hd)
    f64 = {k: synth.bf16_to_f32(v).astype(np.float64) for k, v in x.items()}
    d = {k: dev(v) for k, v in x.items()}
    a = torch.from_numpy(anchors).cuda()
    out, lse = dfl.anchor_attention_fwd(d["q"], d["k_ctx"], d["v_ctx"], d["k_blk"], d["v_blk"], a, B)
    ro, rl = tr.anchor_attention_fwd(**f64, anchors=list(anchors), B=B)
    e_out, e_lse = P.relinf(out.cpu().numpy(), ro), P.relinf(lse.cpu().numpy(), rl)
    assert e_out <= P.REL_TOL and e_lse <= P.REL_TOL, (e_out, e_lse)
    do = torch.from_numpy(dout.astype(np.float32)).cuda()
    g = dfl.anchor_attention_bwd(d["q"], d["k_ctx"], d["v_ctx"], d["k_blk"], d["v_blk"], a, B, out, lse, do)
    ref = tr.anchor_attention_bwd(**f64, anchors=list(anchors), B=B, dout=dout)
    errs = {}
    for nm, got, want in zip(("dq", "dk_ctx", "dv_ctx", "dk_blk", "dv_blk"), g, ref):
        if want.size == 0:
            continue
        errs[nm] = P.relinf(got.cpu().numpy(), want)
        assert errs[nm] <= P.REL_TOL, (nm, errs[nm])
    g2 = dfl.anchor_attention_bwd(d["q"], d["k_ctx"], d["v_ctx"], d["k_blk"], d["v_blk"], a, B, out, lse, do)
    for u, v in zip(g, g2):
        assert torch.equal(u, v)
    print(f"[training] {name}: out {e_out:.2e} lse {e_lse:.2e} "
          + " ".join(f"{k} {v:.2e}" for k, v in errs.items()), flush=True)


# Edges of the attention kernels' forms: rows per (block, KV head) of one to four 32-row waves, with
# and without padding; blocks few enough for split key tiles and more (257 blocks x 1 head: a last
# work-group that is not full); contexts at the edges of the 32-key and 128-key tiles; anchors
# at tile edges.  The bar is that of the cases above.
@pytest.mark.parametrize("n,B,T,nq,nkv,hd", [
    (3, 16, 1, 2, 1, 128), (257, 16, 33, 2, 1, 64), (258, 3, 31, 3, 1, 128),      # one wave per block
    (5, 16, 129, 4, 1, 64), (261, 11, 65, 4, 1, 128), (129, 16, 127, 8, 2, 64),   # two
    (9, 11, 128, 8, 1, 64), (33, 16, 160, 6, 1, 128),                             # three
    (7, 16, 257, 8, 1, 128), (70, 13, 96, 16, 2, 64),                             # four
    (130, 1, 4096, 16, 16, 64), (128, 1, 4096, 16, 16, 64),  # context gradients in chunks of 44 and of 64 blocks
])
def test_anchor_attention_kernel_forms(n, B, T, nq, nkv, hd):
    print(f"[training] attention form {(n, B, T, nq, nkv, hd)}", flush=True)
    x, anchors, dout = inputs(n, B, T, nq, nkv, hd, seed=5)
    edges = [a for a in (0, 1, 31, 32, 33, 127, 128, 129, T - 1, T) if 0 <= a <= T][:n]
    anchors[:len(edges)] = edges
    f64 = {k: synth.bf16_to_f32(v).astype(np.float64) for k, v in x.items()}
    d = {k: dev(v) for k, v in x.items()}
    a = torch.from_numpy(anchors).cuda()
    inp = (d["q"], d["k_ctx"], d["v_ctx"], d["k_blk"], d["v_blk"], a, B)
    out, lse = dfl.anchor_attention_fwd(*inp)
    got = (out, lse, *dfl.anchor_attention_bwd(*inp, out, lse, torch.from_numpy(dout.astype(np.float32)).cuda()))
    want = (*tr.anchor_attention_fwd(**f64, anchors=list(anchors), B=B),
            *tr.anchor_attention_bwd(**f64, anchors=list(anchors), B=B, dout=dout))
    for nm, u, v in zip(("out", "lse", "dq", "dk_ctx", "dv_ctx", "dk_blk", "dv_blk"), got, want):
        assert P.relinf(u.cpu().numpy(), v) <= P.REL_TOL, (nm, P.relinf(u.cpu().numpy(), v))


# context rows past the last anchor (a buffer's unused end) may hold anything: no block reads them, their
# gradients are zero, and the others are not touched.  Anchors at multiples of 64, the last inside a 128-key tile
@pytest.mark.parametrize("hd", [64, 128])
def test_anchor_attention_unused_context_rows(hd):
    n, B, T, nq, nkv, top = 40, 16, 1152, 8, 2, 1088
    print(f"[training] unused context rows hd={hd}", flush=True)
    x, _, dout = inputs(n, B, T, nq, nkv, hd, seed=9)
    anchors = (64 * np.random.default_rng(9).integers(0, top // 64 + 1, size=n)).astype(np.int32)
    anchors[3] = top
    x["k_ctx"][top:] = x["v_ctx"][top:] = 0  # as the oracle sees them
    f64 = {k: synth.bf16_to_f32(v).astype(np.float64) for k, v in x.items()}
    x["k_ctx"][top:] = x["v_ctx"][top:] = 0x7FC0  # NaN
    d = {k: dev(v) for k, v in x.items()}
    a = torch.from_numpy(anchors).cuda()
    inp = (d["q"], d["k_ctx"], d["v_ctx"], d["k_blk"], d["v_blk"], a, B)
    out, lse = dfl.anchor_attention_fwd(*inp)
    got = (out, lse, *dfl.anchor_attention_bwd(*inp, out, lse, torch.from_numpy(dout.astype(np.float32)).cuda()))
    want = (*tr.anchor_attention_fwd(**f64, anchors=list(anchors), B=B),
            *tr.anchor_attention_bwd(**f64, anchors=list(anchors), B=B, dout=dout))
    for nm, u, v in zip(("out", "lse", "dq", "dk_ctx", "dv_ctx", "dk_blk", "dv_blk"), got, want):
        assert P.relinf(u.cpu().numpy(), v) <= P.REL_TOL, nm
    assert not got[3][top:].any() and not got[4][top:].any()


# (V, blocks): rows held in registers (up to 98,307 values: odd row starts, the last value of each
# size), rows with a part past the registers (98,309; 152,516 and 201,088), and rows held on chip (V a
# multiple of 4 in 111,616 .. 152,512): none in LDS, the Qwen3 vocabulary, LDS full; 17 blocks = 272
# rows: a last turn of 16 rows cut into pieces, 23 = 368: one of 112 rows that is not
@pytest.mark.parametrize("V,n", [(3, 2), (1000, 6), (1003, 6), (1000, 70), (2051, 3), (8195, 3), (16387, 3), (32003, 9),
                                 (49155, 2), (65539, 2), (65543, 2), (81923, 2), (81927, 2), (98307, 2), (98309, 2),
                                 (111616, 17), (111616, 23), (151936, 2), (152512, 2), (152516, 17), (201088, 2)])
def test_weighted_ce_matches_oracle(V, n):
    B = 16
    rng = np.random.default_rng(3)
    z = (3.0 * rng.standard_normal((n * B, V))).astype(np.float32)
    y = rng.integers(0, V, size=n * B).astype(np.int32)
    y[rng.random(n * B) < 0.1] = -1
    y[1], y[2], y[3] = V - 1, 0, min(V - 1, 111616)  # last value, first value, first value past the registers
    gamma = 4.5
    loss, ce, dz = dfl.weighted_ce(torch.from_numpy(z).cuda(), torch.from_numpy(y).cuda(), B, gamma)
    rloss, rce, rdz = tr.weighted_ce(z.astype(np.float64), y, B, gamma)
    assert abs(float(loss.cpu()[0]) - rloss) <= 1e-5 * max(1.0, abs(rloss))
    assert P.relinf(ce.cpu().numpy(), rce) <= 1e-5
    assert P.relinf(dz.cpu().numpy(), rdz) <= 1e-5
    with pytest.raises(dfl.DFlareError):
        dfl.weighted_ce(torch.from_numpy(z[:17]).cuda(), torch.from_numpy(y[:17]).cuda(), B, gamma)


# a masked run of logits (-inf, or the lowest float) at the head, in the middle, at the tail, all but the last
# five and all but the first value: longer than a piece, and than all a thread holds in registers; and a row
# without a loss that is masked as a whole: exact zeros
MASKS = ((0.0, 0.6), (0.3, 0.7), (0.55, 1.0), (0.0, -5), (1, 1.0))


def masked_ce_case(V, n, low, B=16):
    rng = np.random.default_rng(8)
    z = (3.0 * rng.standard_normal((n * B, V))).astype(np.float32)
    y = np.empty(n * B, np.int32)
    for r in range(n * B):
        lo, hi = MASKS[r % len(MASKS)]
        lo = lo if isinstance(lo, int) else int(lo * V)
        hi = V + hi if isinstance(hi, int) else int(hi * V)
        z[r, lo:hi] = low
        free = np.r_[0:lo, hi:V]
        y[r] = free[rng.integers(0, free.size)]
    z[0] = low
    return z, y


# rows held in registers, their form with a rest (odd V, and V a multiple of 4), a last turn in pieces (an
# on-chip vocabulary and a longer one), and rows held on chip (none in LDS, and the Qwen3 vocabulary)
@pytest.mark.parametrize("low", [-np.inf, float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("V,n", [(1003, 3), (32003, 3), (98307, 1), (98309, 5), (201088, 5), (151936, 1),
                                 (201088, 1), (111616, 5), (151936, 5)])
def test_weighted_ce_masked_logits(V, n, low):
    print(f"[training] masked CE V={V} n={n} low={low}", flush=True)
    z, y = masked_ce_case(V, n, low)
    loss, ce, dz = (t.cpu().numpy() for t in dfl.weighted_ce(torch.from_numpy(z).cuda(), torch.from_numpy(y).cuda(),
                                                             16, 4.5))
    assert not dz[0].any() and ce[0] == 0.0
    z[0] = 0.0  # (the oracle would form 0 x NaN)
    rloss, rce, rdz = tr.weighted_ce(z.astype(np.float64), y, 16, 4.5)
    assert abs(float(loss[0]) - rloss) <= 1e-5 * max(1.0, abs(rloss))
    assert P.relinf(ce, rce) <= 1e-5
    assert P.relinf(dz, rdz) <= 1e-5


# gradients aligned otherwise than the logits: rows held in registers and their form with a rest
@pytest.mark.parametrize("V", [1003, 32004, 98309, 201088])
def test_weighted_ce_gradient_alignment(V):
    B, rows = 16, 80
    print(f"[training] CE gradient alignment V={V}", flush=True)
    g = torch.Generator("cuda").manual_seed(4)
    z = torch.randn(rows, V, device="cuda", generator=g)
    y = torch.randint(0, V, (rows,), device="cuda", dtype=torch.int32, generator=g)
    want = dfl.weighted_ce(z, y, B, 4.5)
    for shift in (1, 2, 3):
        buf = torch.full((rows * V + 8,), 7.0, device="cuda")
        loss, ce = torch.empty(1, device="cuda"), torch.empty(rows, device="cuda")
        dz = buf[shift:shift + rows * V]
        dfl.weighted_ce_noalloc(z, y, B, 4.5, loss, ce, dz)
        torch.cuda.synchronize()
        assert torch.equal(loss, want[0]) and torch.equal(ce, want[1]) and torch.equal(dz.view(rows, V), want[2])
        assert (buf[:shift] == 7.0).all() and (buf[shift + rows * V:] == 7.0).all()


# more rows than one launch has work-groups for (2^32 threads)
def test_weighted_ce_many_rows():
    B, V, gamma = 16, 2, 4.5
    rows = (1 << 24) + B
    print(f"[training] CE of {rows} rows", flush=True)
    z = torch.randn(rows, V, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    y = torch.arange(rows, device="cuda", dtype=torch.int32) % 3 - 1
    loss, ce, dz = dfl.weighted_ce(z, y, B, gamma)
    b = torch.arange(rows, device="cuda") % B
    w = torch.exp(-(b - 1).double() / gamma) * ((b > 0) & (y >= 0))
    lse = torch.logsumexp(z.double(), dim=1)
    want = torch.where(w > 0, lse - z.double().gather(1, y.clamp_min(0).long()[:, None])[:, 0], 0.0)
    total = w.sum()
    p = torch.exp(z.double() - lse[:, None])
    p.scatter_add_(1, y.clamp_min(0).long()[:, None], -torch.ones_like(p[:, :1]))
    p *= (w / total)[:, None]
    rloss = (w * want).sum() / total
    assert abs(float(loss) - float(rloss)) <= 1e-5 * max(1.0, abs(float(rloss)))
    assert float((ce - want).abs().max()) <= 1e-5 * float(want.abs().max())
    assert float((dz - p).abs().max()) <= 1e-5 * float(p.abs().max())


def test_anchor_attention_full_training_shape_sampled():
    """The training shape the benchmark times (T = 3,072, 512 blocks of B = 16, 32 query / 8 KV
    heads x 128): every kernel runs on the whole problem in its benchmark launch configuration
    (8 gradient chunks, XCD-grouped work order), and sampled blocks are checked against the
    oracle run on that block alone — its outputs, lse, dQ and block-key gradients depend on
    nothing else.  Anchors lie in 0 .. 2,900 except one block's, T - B: the context keys from
    2,901 up to it are seen by that block only, so their gradients are that block's too, and
    keys at or past T - B are seen by no block (zero gradients)."""
    n, B, T, nq, nkv, hd = 512, 16, 3072, 32, 8, 128
    print("[training] full shape sampled", flush=True)
    rng = np.random.default_rng(11)

    def bf(shape):
        return synth.round_bf16(rng.standard_normal(shape).astype(np.float32))

    x = dict(q=bf((n * B, nq, hd)), k_ctx=bf((T, nkv, hd)), v_ctx=bf((T, nkv, hd)),
             k_blk=bf((n * B, nkv, hd)), v_blk=bf((n * B, nkv, hd)))
    anchors = rng.integers(0, 2901, size=n).astype(np.int32)
    top = 7
    anchors[0], anchors[top] = 0, T - B
    dout = rng.standard_normal((n * B, nq, hd)).astype(np.float32)
    d = {k: dev(v) for k, v in x.items()}
    a = torch.from_numpy(anchors).cuda()
    out, lse = dfl.anchor_attention_fwd(d["q"], d["k_ctx"], d["v_ctx"], d["k_blk"], d["v_blk"], a, B)
    g = dfl.anchor_attention_bwd(d["q"], d["k_ctx"], d["v_ctx"], d["k_blk"], d["v_blk"], a, B, out, lse,
                                 torch.from_numpy(dout).cuda())
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    dq, dkc, dvc, dkb, dvb = (t.cpu().numpy() for t in g)
    assert not dkc[T - B:].any() and not dvc[T - B:].any()
    kc64 = synth.bf16_to_f32(x["k_ctx"]).astype(np.float64)
    vc64 = synth.bf16_to_f32(x["v_ctx"]).astype(np.float64)
    for i in (0, top, 200, n - 1):
        rows = slice(i * B, (i + 1) * B)
        blk = {k: synth.bf16_to_f32(x[k][rows]).astype(np.float64) for k in ("q", "k_blk", "v_blk")}
        ro, rl = tr.anchor_attention_fwd(blk["q"], kc64, vc64, blk["k_blk"], blk["v_blk"], [int(anchors[i])], B)
        rdq, rdkc, rdvc, rdkb, rdvb = tr.anchor_attention_bwd(blk["q"], kc64, vc64, blk["k_blk"], blk["v_blk"],
                                                               [int(anchors[i])], B, dout[rows].astype(np.float64))
        errs = {"out": P.relinf(out[rows], ro), "lse": P.relinf(lse[rows], rl), "dq": P.relinf(dq[rows], rdq),
                "dk_blk": P.relinf(dkb[rows], rdkb), "dv_blk": P.relinf(dvb[rows], rdvb)}
        if i == top:
            only = slice(2901, T - B)
            errs["dk_ctx_own"] = P.relinf(dkc[only], rdkc[only])
            errs["dv_ctx_own"] = P.relinf(dvc[only], rdvc[only])
        print(f"[training] full shape block {i} (anchor {anchors[i]}): "
              + " ".join(f"{k} {v:.2e}" for k, v in errs.items()), flush=True)
        for k, v in errs.items():
            assert v <= P.REL_TOL, (i, k, v)
