"""GPU parity of the backward pass (fine-tuning, Sec. 4.5) against the gradient oracle (fp64 autograd
of the forward definitions, pinned by finite differences): the forward's log-sum-exp, and the
gradients of the block-sparse attention for fixed block lists."""

import math

import numpy as np
import pytest
import torch

import oracle as O
from oracle import rola_grad as G
from paper_2609_06712_amd import synth

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts too; every test here is skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2609_06712_amd import rola as R  # noqa: E402
from tests import _parity as T  # noqa: E402


def _f64(t):
    return t.detach().to("cpu", torch.float64).numpy()


def _rel(got, want):
    return float(np.linalg.norm(got - want) / max(np.linalg.norm(want), 1e-300))


@pytest.mark.parametrize("grid,block,s,B", [((3, 10, 13), 64, 0.5, 1), ((3, 10, 13), 128, 0.5, 1),
                                            ((2, 9, 20), 64, 0.7, 2), ((4, 8, 16), 64, 0.0, 1)],
                         ids=["ragged-b64", "ragged-b128", "batch2", "keep-all"])
def test_sparse_backward(grid, block, s, B):
    w = synth.WAN_1_3B_480P.replace(grid=grid, H=2, B=B, block=block, sparsity=s)
    inp = synth.make_inputs(w, 7)
    d = {k: v.cuda() for k, v in inp.items()}
    g = w.grid
    prob = R.problem(w.B, w.H, w.N, w.d_h, g, w.dtype)
    cos, sin = R.rola_rope_tables(prob, w.split)
    qr = R.rola_rope_apply(d["Qn"], cos, sin, g)
    kr = R.rola_rope_apply(d["Kn"], cos, sin, g)
    idx = R.rola_block_select(qr, kr, g, block, s)
    os_, lse = R.rola_sparse_attn_lse(qr, kr, d["V"], g, block, s, idx)
    ref_os = R.rola_sparse_attn(qr, kr, d["V"], g, block, s, idx)
    gen = torch.Generator().manual_seed(3)
    dos = torch.randn(qr.shape, generator=gen).to(torch.bfloat16).cuda()
    dq, dk, dv = R.rola_sparse_attn_backward(qr, kr, d["V"], g, block, s, idx, os_, lse, dos)
    torch.cuda.synchronize()
    assert torch.equal(os_, ref_os)  # the lse variant computes the same O^s
    scale = 1.0 / math.sqrt(w.d_h)
    for b in range(w.B):
        for h in range(w.H):
            q, k, v = _f64(qr[b, h]), _f64(kr[b, h]), _f64(d["V"][b, h])
            ix = idx[b, h].cpu().numpy()
            # lse (log2 units) from its definition over the selected keys
            mask = np.zeros((w.N, w.N), bool)
            blk = np.arange(w.N) // block
            sel = np.zeros((ix.shape[0], ix.shape[0]), bool)
            sel[np.arange(ix.shape[0])[:, None], ix] = True
            mask = sel[blk[:, None], blk[None, :]]
            sc = np.where(mask, q @ k.T * scale, -np.inf)
            mx = sc.max(1, keepdims=True)
            lse_ref = (mx[:, 0] + np.log(np.exp(sc - mx).sum(1))) / math.log(2)
            # the forward's denominator sums the bf16-rounded probabilities that enter P V (relative
            # error <= 2^-9), so its log2 is within 2^-9 / ln 2 = 2.8e-3 of the exact one
            np.testing.assert_allclose(_f64(lse[b, h]), lse_ref, rtol=0, atol=2.9e-3)
            want = G.sparse_attention_grads(q, k, v, ix, block, scale, _f64(dos[b, h]))
            errs = {n: _rel(_f64(t[b, h]), want[n]) for n, t in (("dqr", dq), ("dkr", dk), ("dv", dv))}
            print(f"[parity] sparse backward grid {grid} block {block} s {s} b{b} h{h}: " +
                  ", ".join(f"{n} rel {e:.2e}" for n, e in errs.items()), flush=True)
            for n, e in errs.items():
                assert e <= 1e-2, (n, e)
            # shifting all keys leaves O^s unchanged: the key gradients sum to zero
            colsum = np.abs(_f64(dk[b, h]).sum(0)).max()
            assert colsum <= 1e-2 * np.abs(_f64(dk[b, h])).sum(0).max() + 1e-6


@pytest.mark.parametrize("block", [64, 128])
def test_sparse_backward_uneven_transposed_lists(block):
    """4096 tokens at 90 % sparsity: the transposed lists (query blocks per key block) differ in
    length, some key blocks are selected by no query block, and the dK/dV workgroups take the key
    blocks longest list first while walking each list in its bit-reversed order. Every head
    against the gradient oracle; unselected key blocks must get exactly zero gradients."""
    w = synth.WAN_1_3B_480P.replace(grid=(8, 16, 32), H=2, B=1, block=block, sparsity=0.9)
    inp = synth.make_inputs(w, 21)
    d = {k: v.cuda() for k, v in inp.items()}
    g = w.grid
    prob = R.problem(w.B, w.H, w.N, w.d_h, g, w.dtype)
    cos, sin = R.rola_rope_tables(prob, w.split)
    qr = R.rola_rope_apply(d["Qn"], cos, sin, g)
    kr = R.rola_rope_apply(d["Kn"], cos, sin, g)
    idx = R.rola_block_select(qr, kr, g, block, w.sparsity)
    os_, lse = R.rola_sparse_attn_lse(qr, kr, d["V"], g, block, w.sparsity, idx)
    gen = torch.Generator().manual_seed(5)
    dos = torch.randn(qr.shape, generator=gen).to(torch.bfloat16).cuda()
    dq, dk, dv = R.rola_sparse_attn_backward(qr, kr, d["V"], g, block, w.sparsity, idx, os_, lse, dos)
    torch.cuda.synchronize()
    scale = 1.0 / math.sqrt(w.d_h)
    nb = -(-w.N // block)
    for h in range(w.H):
        ix = idx[0, h].cpu().numpy()
        counts = np.bincount(ix.ravel(), minlength=nb)
        print(f"[parity] transposed list lengths block {block} h{h}: min {counts.min()} max "
              f"{counts.max()} unselected {int((counts == 0).sum())} of {nb}", flush=True)
        assert counts.max() > counts.min()  # uneven lists, as the case intends
        want = G.sparse_attention_grads(_f64(qr[0, h]), _f64(kr[0, h]), _f64(d["V"][0, h]), ix, block,
                                        scale, _f64(dos[0, h]))
        errs = {n: _rel(_f64(t[0, h]), want[n]) for n, t in (("dqr", dq), ("dkr", dk), ("dv", dv))}
        print(f"[parity] sparse backward uneven lists block {block} h{h}: " +
              ", ".join(f"{n} rel {e:.2e}" for n, e in errs.items()), flush=True)
        for n, e in errs.items():
            assert e <= 1e-2, (n, e)
        for J in np.flatnonzero(counts == 0):  # no query selected these keys
            rows = slice(J * block, min(w.N, (J + 1) * block))
            assert torch.count_nonzero(dk[0, h, rows]) == 0 and torch.count_nonzero(dv[0, h, rows]) == 0


@pytest.mark.parametrize("grid,block,H,B", [((3, 20, 33), 64, 3, 3), ((5, 17, 31), 128, 10, 1),
                                            ((1, 9, 7), 64, 1, 1)])
def test_sparse_backward_heads_over_xcds(grid, block, H, B):
    """Key blocks dealt over the XCDs (whole heads plus a remainder: 9 and 10 heads; 1 head), and
    transposed lists of block counts off the powers of two and the 64-position steps, against the
    gradient oracle."""
    w = synth.WAN_1_3B_480P.replace(grid=grid, H=H, B=B, block=block, sparsity=0.8)
    d = {k: v.cuda() for k, v in synth.make_inputs(w, 21).items()}
    g = w.grid
    prob = R.problem(w.B, w.H, w.N, w.d_h, g, w.dtype)
    cos, sin = R.rola_rope_tables(prob, w.split)
    qr = R.rola_rope_apply(d["Qn"], cos, sin, g)
    kr = R.rola_rope_apply(d["Kn"], cos, sin, g)
    idx = R.rola_block_select(qr, kr, g, block, w.sparsity)
    os_, lse = R.rola_sparse_attn_lse(qr, kr, d["V"], g, block, w.sparsity, idx)
    dos = torch.randn(qr.shape, generator=torch.Generator().manual_seed(4)).to(torch.bfloat16).cuda()
    dq, dk, dv = R.rola_sparse_attn_backward(qr, kr, d["V"], g, block, w.sparsity, idx, os_, lse, dos)
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(H):
            want = G.sparse_attention_grads(_f64(qr[b, h]), _f64(kr[b, h]), _f64(d["V"][b, h]),
                                            idx[b, h].cpu().numpy(), block, w.d_h ** -0.5, _f64(dos[b, h]))
            for n, t in (("dqr", dq), ("dkr", dk), ("dv", dv)):
                assert _rel(_f64(t[b, h]), want[n]) <= 1e-2, (b, h, n)


@pytest.mark.parametrize("block,ragged", [(64, 0), (64, 37), (128, 0), (128, 101)])
def test_sparse_backward_short_transposed_lists(block, ragged):
    """Eleven key blocks selected by 0, 1, .., 10 query blocks: dK/dV walks of no step, of fewer steps
    than LDS stages and of every remainder of a turn, with a whole and a ragged last query block.
    Tolerance as the other backward tests (bf16 operands, relative error of a tensor); blocks that no
    query selects get exactly zero."""
    nb, keep = 11, 5
    w = synth.WAN_1_3B_480P.replace(grid=(1, 1, nb * block - ragged), H=1, B=1, block=block, sparsity=0.55)
    assert R.keep_blocks(nb, w.sparsity) == keep
    left = np.full(nb, keep)
    rows = [[] for _ in range(nb)]
    for J in range(nb - 1, -1, -1):  # key block J goes to the J query blocks with the most room left
        for I in np.argsort(-left, kind="stable")[:J]:
            rows[I].append(J)
            left[I] -= 1
    assert not left.any()
    idx = torch.tensor([sorted(r) for r in rows], dtype=torch.int32)[None, None].cuda()
    d = {k: v.cuda() for k, v in synth.make_inputs(w, 8).items()}
    q, k, v = d["Qn"], d["Kn"], d["V"]
    os_, lse = R.rola_sparse_attn_lse(q, k, v, w.grid, block, w.sparsity, idx)
    dos = torch.randn(q.shape, generator=torch.Generator().manual_seed(6)).to(torch.bfloat16).cuda()
    grads = R.rola_sparse_attn_backward(q, k, v, w.grid, block, w.sparsity, idx, os_, lse, dos)
    torch.cuda.synchronize()
    want = G.sparse_attention_grads(_f64(q[0, 0]), _f64(k[0, 0]), _f64(v[0, 0]), idx[0, 0].cpu().numpy(),
                                    block, w.d_h ** -0.5, _f64(dos[0, 0]))
    for n, t in zip(("dqr", "dkr", "dv"), grads):
        assert _rel(_f64(t[0, 0]), want[n]) <= 1e-2, n
        for J in range(nb):  # every block by itself: a step lost in a short list shows
            r = slice(J * block, (J + 1) * block)
            err = np.abs(_f64(t[0, 0])[r] - want[n][r]).max()
            assert err <= 2e-2 * np.abs(want[n]).max(), (n, J, err)
    assert torch.count_nonzero(grads[1][0, 0, :block]) == 0 and torch.count_nonzero(grads[2][0, 0, :block]) == 0


def test_sparse_backward_many_groups():
    """200 heads of 390 tokens: 800 (head, pair) groups, more than the chip holds at once, so the dQ
    pass's resident workgroups each take several groups from the work queues. Sampled heads against
    the gradient oracle."""
    w = synth.WAN_1_3B_480P.replace(grid=(3, 10, 13), H=200, B=1, sparsity=0.5)
    inp = synth.make_inputs(w, 13)
    d = {k: v.cuda() for k, v in inp.items()}
    g = w.grid
    prob = R.problem(w.B, w.H, w.N, w.d_h, g, w.dtype)
    cos, sin = R.rola_rope_tables(prob, w.split)
    qr = R.rola_rope_apply(d["Qn"], cos, sin, g)
    kr = R.rola_rope_apply(d["Kn"], cos, sin, g)
    idx = R.rola_block_select(qr, kr, g, 64, w.sparsity)
    os_, lse = R.rola_sparse_attn_lse(qr, kr, d["V"], g, 64, w.sparsity, idx)
    gen = torch.Generator().manual_seed(4)
    dos = torch.randn(qr.shape, generator=gen).to(torch.bfloat16).cuda()
    dq, dk, dv = R.rola_sparse_attn_backward(qr, kr, d["V"], g, 64, w.sparsity, idx, os_, lse, dos)
    torch.cuda.synchronize()
    scale = 1.0 / math.sqrt(w.d_h)
    for h in (0, 77, 199):
        want = G.sparse_attention_grads(_f64(qr[0, h]), _f64(kr[0, h]), _f64(d["V"][0, h]),
                                        idx[0, h].cpu().numpy(), 64, scale, _f64(dos[0, h]))
        errs = {n: _rel(_f64(t[0, h]), want[n]) for n, t in (("dqr", dq), ("dkr", dk), ("dv", dv))}
        print(f"[parity] sparse backward 800 groups h{h}: " +
              ", ".join(f"{n} rel {e:.2e}" for n, e in errs.items()), flush=True)
        for n, e in errs.items():
            assert e <= 1e-2, (n, e)


@pytest.mark.parametrize("r,B,eps_lr", [(32, 1, 1e-6), (16, 2, 1e-6), (64, 1, 1e-6), (64, 2, 0.0),
                                         (32, 1, 0.0)])
def test_lowrank_backward(r, B, eps_lr):
    """The low-rank branch + fusion backward against the oracle, per head, from the GPU's own O^s.
    390 tokens: the last 64-token chunk holds 6, so padding tokens run through every step; with
    eps_lr = 0 they must still contribute nothing (their RMSNorm denominator is 0)."""
    w = synth.WAN_1_3B_480P.replace(grid=(3, 10, 13), H=2, B=B, r=r)
    inp = synth.make_inputs(w, 8)
    d = {k: v.cuda() for k, v in inp.items()}
    g = w.grid
    prob = R.problem(w.B, w.H, w.N, w.d_h, g, w.dtype)
    cos, sin = R.rola_rope_tables(prob, w.split)
    C, _ = R.rola_lowrank_summary(d["Kn"], d["V"], d["Pk"], r, cos, sin, g)
    gen = torch.Generator().manual_seed(5)
    os_ = torch.randn(d["Qn"].shape, generator=gen).to(torch.bfloat16).cuda()
    dO = torch.randn(d["Qn"].shape, generator=gen).to(torch.bfloat16).cuda()
    dOs, dQn, dKn, dV, dPq, dPk, dlog = R.rola_lowrank_backward(
        d["Qn"], d["Kn"], d["V"], d["Pq"], d["Pk"], r, cos, sin, C, os_, d["logits"], dO, g,
        eps_lr=eps_lr)
    torch.cuda.synchronize()
    ocos, osin = O.rope_tables(*g, w.split)
    f = synth.to_f64(inp)
    want = {(b, h): G.lowrank_combine_grads(f["Qn"][b, h], f["Kn"][b, h], f["V"][b, h], f["Pq"][h],
                                            f["Pk"][h], _f64(os_[b, h]), f["logits"][b], ocos, osin,
                                            _f64(dO[b, h]), eps_lr=eps_lr)
            for b in range(w.B) for h in range(w.H)}
    for name, t in (("dPq", dPq), ("dPk", dPk), ("dlogits", dlog)):
        assert torch.isfinite(t).all(), name
    for (b, h), wt in want.items():
        errs = {n: _rel(_f64(t[b, h]), wt[k]) for n, t, k in
                (("dOs", dOs, "dos"), ("dQn", dQn, "dqn"), ("dKn", dKn, "dkn"), ("dV", dV, "dv"))}
        print(f"[parity] lowrank backward r{r} eps_lr {eps_lr:g} b{b} h{h}: " +
              ", ".join(f"{n} rel {e:.2e}" for n, e in errs.items()), flush=True)
        for n, e in errs.items():
            assert e <= 1e-2, (n, e)
    # parameter gradients summed over the batch, gate-logit gradients over the heads
    for name, k in (("dPq", dPq), ("dPk", dPk)):
        ref = np.stack([sum(want[(b, h)][name] for b in range(w.B)) for h in range(w.H)])
        assert _rel(_f64(k), ref) <= 1e-2, name
    ref = np.stack([sum(want[(b, h)]["dlogits"] for h in range(w.H)) for b in range(w.B)])
    assert _rel(_f64(dlog), ref) <= 1e-2


@pytest.mark.parametrize("r", [32, 64])
def test_lowrank_backward_multistep(r):
    """40 heads of 7800 tokens: every chunk of the low-rank backward then spans two 64-token steps
    (the last one ragged), so the outer products accumulate across steps. Sampled heads against
    the oracle; dP summed over the batch (B = 1: the head's own)."""
    w = synth.WAN_1_3B_480P.replace(grid=(5, 30, 52), H=40, B=1, r=r)
    inp = synth.make_inputs(w, 11)
    d = {k: v.cuda() for k, v in inp.items()}
    g = w.grid
    prob = R.problem(w.B, w.H, w.N, w.d_h, g, w.dtype)
    cos, sin = R.rola_rope_tables(prob, w.split)
    C, _ = R.rola_lowrank_summary(d["Kn"], d["V"], d["Pk"], w.r, cos, sin, g)
    gen = torch.Generator().manual_seed(6)
    os_ = torch.randn(d["Qn"].shape, generator=gen).to(torch.bfloat16).cuda()
    dO = torch.randn(d["Qn"].shape, generator=gen).to(torch.bfloat16).cuda()
    dOs, dQn, dKn, dV, dPq, dPk, _ = R.rola_lowrank_backward(
        d["Qn"], d["Kn"], d["V"], d["Pq"], d["Pk"], w.r, cos, sin, C, os_, d["logits"], dO, g)
    torch.cuda.synchronize()
    ocos, osin = O.rope_tables(*g, w.split)
    f = synth.to_f64(inp)
    for h in (0, 21, 39):
        wt = G.lowrank_combine_grads(f["Qn"][0, h], f["Kn"][0, h], f["V"][0, h], f["Pq"][h],
                                     f["Pk"][h], _f64(os_[0, h]), f["logits"][0], ocos, osin,
                                     _f64(dO[0, h]))
        errs = {n: _rel(_f64(t), wt[k]) for n, t, k in
                (("dOs", dOs[0, h], "dos"), ("dQn", dQn[0, h], "dqn"), ("dKn", dKn[0, h], "dkn"),
                 ("dV", dV[0, h], "dv"), ("dPq", dPq[h], "dPq"), ("dPk", dPk[h], "dPk"))}
        print(f"[parity] lowrank backward r{r} 40 heads x 7800 tokens h{h}: " +
              ", ".join(f"{n} rel {e:.2e}" for n, e in errs.items()), flush=True)
        for n, e in errs.items():
            assert e <= 1e-2, (n, e)


def test_gate_backward():
    gen = torch.Generator().manual_seed(6)
    X = torch.randn((2, 300, 1536), generator=gen).to(torch.bfloat16)
    Wg = (torch.randn((1536,), generator=gen) / 40).to(torch.bfloat16)
    dl = torch.randn((2, 300), generator=gen)
    dX, dWg, dbg = R.rola_gate_logits_backward(X.cuda(), Wg.cuda(), dl.cuda(), (300, 1, 1))
    torch.cuda.synchronize()
    want = G.gate_grads(X.double().numpy().reshape(-1, 1536), Wg.double().numpy(), dl.double().numpy().ravel())
    assert _rel(_f64(dX).reshape(-1, 1536), want["dX"]) <= 1e-6
    assert _rel(_f64(dWg), want["dWg"]) <= 1e-5
    assert float(dbg.cpu()) == pytest.approx(want["dbg"], rel=1e-5)


@pytest.mark.parametrize("dtype,B,N,dm", [("bf16", 1, 1, 8), ("bf16", 1, 513, 136), ("f32", 2, 700, 2056),
                                          ("bf16", 1, 5003, 640), ("bf16", 1, 131, 5120)])
def test_gate_backward_edges(dtype, B, N, dm):
    """One row, ragged row chunks, every column tile width (16 to 256 columns of eight channels) and
    few / many chunk partials. Every sum is fp32 over B N terms, in whatever order: its error is at
    most B N 2^-24 sum |term|."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(N + dm)
    X = torch.randn((B, N, dm), generator=gen).to(tdt)
    Wg = (torch.randn((dm,), generator=gen) / dm ** 0.5).to(tdt)
    dl = torch.randn((B, N), generator=gen)
    dX, dWg, dbg = R.rola_gate_logits_backward(X.cuda(), Wg.cuda(), dl.cuda(), (N, 1, 1))
    none, dWg2, _ = R.rola_gate_logits_backward(X.cuda(), Wg.cuda(), dl.cuda(), (N, 1, 1), want_dX=False)
    torch.cuda.synchronize()
    Xf, df = X.double().numpy().reshape(-1, dm), dl.double().numpy().ravel()
    want = G.gate_grads(Xf, Wg.double().numpy(), df)
    assert none is None and torch.equal(dWg, dWg2)
    np.testing.assert_allclose(_f64(dX).reshape(-1, dm), want["dX"], rtol=2.0 ** -23)
    u = B * N * 2.0 ** -24
    assert np.all(np.abs(_f64(dWg) - want["dWg"]) <= u * (np.abs(df) @ np.abs(Xf)) + 1e-30)
    assert abs(float(dbg.cpu()) - want["dbg"]) <= u * np.abs(df).sum()


@pytest.mark.parametrize("grid,s", [((3, 10, 13), 0.5), ((4, 8, 16), 0.75)])
def test_module_backward(grid, s):
    """The composed backward (paper_2609_06712_amd.train) against fp64 autograd of the whole module,
    per head, with the GPU's block lists."""
    from paper_2609_06712_amd import train
    w = synth.WAN_1_3B_480P.replace(grid=grid, H=2, sparsity=s)
    inp = synth.make_inputs(w, 9)
    d = {k: v.cuda() for k, v in inp.items()}
    out, saved = train.forward(d["Qn"], d["Kn"], d["V"], d["Pq"], d["Pk"], d["logits"], w.grid,
                               w.split, 64, s, w.r)
    gen = torch.Generator().manual_seed(7)
    dO = torch.randn(out.shape, generator=gen).to(torch.bfloat16).cuda()
    gr = train.backward(d["Qn"], d["Kn"], d["V"], d["Pq"], d["Pk"], d["logits"], saved, dO)
    torch.cuda.synchronize()
    f = synth.to_f64(inp)
    ocos, osin = O.rope_tables(*w.grid, w.split)
    tot = {"dPq": 0, "dPk": 0, "dlogits": 0}
    for h in range(w.H):
        want = G.module_grads(f["Qn"][0, h], f["Kn"][0, h], f["V"][0, h], f["Pq"][h], f["Pk"][h],
                              f["logits"][0], ocos, osin, saved["idx"][0, h].cpu().numpy(), 64,
                              _f64(dO[0, h]))
        errs = {n: _rel(_f64(gr[n][0, h]), want[k]) for n, k in
                (("dQn", "dqn"), ("dKn", "dkn"), ("dV", "dv"))}
        errs["dPq"] = _rel(_f64(gr["dPq"][h]), want["dPq"])
        errs["dPk"] = _rel(_f64(gr["dPk"][h]), want["dPk"])
        tot["dlogits"] = tot["dlogits"] + want["dlogits"]
        print(f"[parity] module backward {grid} s{s} h{h}: " +
              ", ".join(f"{n} rel {e:.2e}" for n, e in errs.items()), flush=True)
        for n, e in errs.items():
            assert e <= 2e-2, (n, e)
    assert _rel(_f64(gr["dlogits"][0]), tot["dlogits"]) <= 2e-2


@pytest.mark.parametrize("grid,block", [((3, 10, 13), 64), ((3, 10, 13), 128), ((4, 8, 16), 64)])
def test_sparse_backward_accumulate(grid, block):
    """The accumulating sparse backward against the plain one followed by the rotation's backward: the
    same products added to the same values, up to the fusing of three multiply-adds per element."""
    w = synth.WAN_1_3B_480P.replace(grid=grid, H=3, B=2, block=block, sparsity=0.5)
    d = {k: v.cuda() for k, v in synth.make_inputs(w, 22).items()}
    g = w.grid
    prob = R.problem(w.B, w.H, w.N, w.d_h, g, w.dtype)
    cos, sin = R.rola_rope_tables(prob, w.split)
    qr = R.rola_rope_apply(d["Qn"], cos, sin, g)
    kr = R.rola_rope_apply(d["Kn"], cos, sin, g)
    idx = R.rola_block_select(qr, kr, g, block, w.sparsity)
    os_, lse = R.rola_sparse_attn_lse(qr, kr, d["V"], g, block, w.sparsity, idx)
    gen = torch.Generator().manual_seed(5)
    dos = torch.randn(qr.shape, generator=gen).to(torch.bfloat16).cuda()
    base = [torch.randn(qr.shape, generator=gen).cuda() for _ in range(3)]
    args = (qr, kr, d["V"], g, block, w.sparsity, idx, os_, lse, dos)
    grads = R.rola_sparse_attn_backward(*args)
    want = [t.clone() for t in base]
    for i, (dy, dx) in enumerate(zip(grads, want)):
        R.rola_rope_backward_accumulate(dy, cos, sin, g, dx, rotate=i < 2)
    got = R.rola_sparse_attn_backward_accumulate(*args, cos, sin, *base)
    torch.cuda.synchronize()
    for i, (x, y, dy, b) in enumerate(zip(got, want, grads, base)):
        assert x is b
        # each term is rounded at most twice more in one form than in the other
        bound = 2.0 ** -22 * (y.abs() + dy.abs().unflatten(-1, (-1, 2)).sum(-1).repeat_interleave(2, -1))
        assert bool(((x - y).abs() <= bound).all()), i


def test_rope_backward_accumulate():
    """dX += R(p)^T dY (the gradient through the main-path rotation) and dX += dY, against the
    oracle's rotation by the negated angle (R(p)^T = R(-p)) in fp64, on a ragged 3x10x13 grid."""
    w = synth.WAN_1_3B_480P.replace(grid=(3, 10, 13), H=2, B=2)
    g = w.grid
    gen = torch.Generator().manual_seed(11)
    dY = torch.randn((w.B, w.H, w.N, 128), generator=gen)
    dX0 = torch.randn((w.B, w.H, w.N, 128), generator=gen)
    prob = R.problem(w.B, w.H, w.N, 128, g, "f32")
    cos, sin = R.rola_rope_tables(prob, w.split)
    rot = R.rola_rope_backward_accumulate(dY.cuda(), cos, sin, g, dX0.clone().cuda())
    add = R.rola_rope_backward_accumulate(dY.cuda(), cos, sin, g, dX0.clone().cuda(), rotate=False)
    torch.cuda.synchronize()
    ocos, osin = O.rope_tables(*g, w.split)
    want = dX0.double().numpy() + O.rotate(dY.double().numpy(), ocos, -osin)
    np.testing.assert_allclose(_f64(rot), want, rtol=0, atol=2e-5)
    np.testing.assert_allclose(_f64(add), (dX0.double() + dY.double()).numpy(), rtol=0, atol=1e-6)
