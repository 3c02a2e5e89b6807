"""Products of few rows (the ring kernel): every tile it is built in, at the edges of the tiles and of the rule that picks
them - 64- to 384-row and 64- to 160-column tiles, row tails and a last tile column cut short, K shares of unequal length,
the sizes just beyond - and, through a prefill of large enough products, the epilogues that only a prefill uses: rotation,
outputs per segment, the row list, partial tiles left to the RMSNorm.

A bf16 result is off by half a unit in the last place (2^-9 of the value, a quarter of that in the 2-norm: 1.7e-3, bound
2.5e-3); fp32 sums of K products of bf16 values stay within sqrt(K) 2^-24 < 1e-5 of theirs."""
import numpy as np
import pytest
import torch

import fastav_inputs as fi
import paper_2601_13143_amd as fa
from gpu_util import assert_close, dev, host, make_decoder, prune_tuples, rel_l2
from oracle import fastav_oracle as orc

TILES = None      # the large-tile kernel
CASES = [         # epilogue, rows, columns, K, (tile rows, tile columns, K shares)
    (fa.EPI_STORE, 17, 4096, 1024, (64, 64, 1)), (fa.EPI_STORE, 64, 4608, 1024, (64, 64, 1)), (fa.EPI_STORE, 65, 4096, 1088, (64, 64, 1)),
    (fa.EPI_STORE, 193, 8192, 512, (128, 64, 1)), (fa.EPI_STORE, 129, 16384, 256, (192, 64, 1)), (fa.EPI_STORE, 144, 15360, 320, (192, 64, 1)),
    (fa.EPI_STORE, 145, 15360, 320, TILES), (fa.EPI_STORE, 257, 8192, 2048, (192, 64, 1)), (fa.EPI_STORE, 385, 4224, 2112, (192, 64, 1)),
    (fa.EPI_STORE, 576, 4608, 2048, (192, 64, 1)), (fa.EPI_STORE, 577, 4608, 2048, TILES), (fa.EPI_STORE, 64, 4096, 960, TILES),
    (fa.EPI_RESADD, 17, 4096, 1024, (64, 64, 2)), (fa.EPI_RESADD, 64, 1024, 4160, (64, 64, 8)), (fa.EPI_RESADD, 65, 1024, 4096, (128, 64, 8)),
    (fa.EPI_RESADD, 128, 2048, 2112, (128, 64, 4)), (fa.EPI_RESADD, 193, 4096, 4096, (128, 64, 2)), (fa.EPI_RESADD, 130, 3584, 4096, (192, 64, 4)),
    (fa.EPI_RESADD, 257, 2048, 2112, (192, 64, 4)), (fa.EPI_RESADD, 300, 3584, 3584, (192, 64, 2)), (fa.EPI_RESADD, 576, 2048, 2048, (192, 64, 2)),
    (fa.EPI_RESADD, 65, 4096, 8192, (128, 128, 8)), (fa.EPI_RESADD, 129, 4096, 8256, (192, 128, 8)), (fa.EPI_RESADD, 250, 4096, 8192, (256, 128, 8)),
    (fa.EPI_RESADD, 257, 4096, 8192, TILES), (fa.EPI_RESADD, 17, 4096, 960, TILES),
    (fa.EPI_SWIGLU, 17, 4096, 1024, (64, 64, 1)), (fa.EPI_SWIGLU, 65, 4160, 1088, (128, 64, 1)), (fa.EPI_SWIGLU, 129, 8192, 512, (192, 64, 1)),
    (fa.EPI_SWIGLU, 257, 4096, 2048, (192, 64, 1)), (fa.EPI_SWIGLU, 64, 14336, 320, (64, 128, 1)), (fa.EPI_SWIGLU, 65, 14336, 320, (128, 128, 1)),
    (fa.EPI_SWIGLU, 129, 14336, 384, (192, 128, 1)), (fa.EPI_SWIGLU, 256, 14336, 320, (256, 128, 1)), (fa.EPI_SWIGLU, 64, 18944, 256, (64, 160, 1)),
    (fa.EPI_SWIGLU, 128, 18944, 320, (128, 160, 1)), (fa.EPI_SWIGLU, 191, 18944, 256, (192, 160, 1)), (fa.EPI_SWIGLU, 193, 18880, 256, (256, 160, 1)),
    (fa.EPI_SWIGLU, 257, 18944, 256, (384, 160, 1)), (fa.EPI_SWIGLU, 331, 18944, 320, (384, 160, 1)), (fa.EPI_SWIGLU, 384, 16448, 256, (384, 160, 1)),
    (fa.EPI_SWIGLU, 300, 18944, 448, (384, 160, 1)),
    (fa.EPI_STORE, 100, 4096, 1152, (64, 64, 1)), (fa.EPI_STORE, 200, 8192, 576, (128, 64, 1)),       # odd numbers of stages
    (fa.EPI_SWIGLU, 100, 14336, 2048, (128, 128, 1)), (fa.EPI_SWIGLU, 250, 14336, 4096, (256, 128, 1)),   # K walked from another place
    (fa.EPI_RESADD, 257, 4096, 4096, (128, 128, 2)), (fa.EPI_RESADD, 512, 2048, 8256, (128, 128, 4)), (fa.EPI_RESADD, 331, 2560, 6912, (128, 128, 4)),
    (fa.EPI_RESADD, 576, 3584, 3648, (192, 128, 3)), (fa.EPI_RESADD, 513, 2560, 6912, (192, 128, 4)),   # several tile rows of 128 columns
    (fa.EPI_SWIGLU, 48, 8192, 2048, (64, 64, 1)), (fa.EPI_SWIGLU, 100, 8192, 2048, (128, 64, 1)), (fa.EPI_SWIGLU, 129, 8192, 2048, (192, 64, 1)),
    (fa.EPI_SWIGLU, 60, 14336, 2048, (64, 128, 1)), (fa.EPI_SWIGLU, 60, 18944, 2048, (64, 160, 1)), (fa.EPI_SWIGLU, 300, 18944, 2048, (384, 160, 1)),
    (fa.EPI_SWIGLU, 450, 2048, 2048, (128, 64, 1)),                            # several tile rows: all from the first stage
    (fa.EPI_SWIGLU, 385, 18944, 256, TILES), (fa.EPI_SWIGLU, 145, 8192, 512, TILES),
]


def _plan(epi, m, n, k, room=None):
    p = fa.fastav_linear_plan(m, n, k, epi, fa.BF16, room)
    assert p.kernel in (fa.LINEAR_RING, fa.LINEAR_TILES)
    return (p.tile_rows, p.tile_cols, p.splits) if p.kernel == fa.LINEAR_RING else TILES


def test_cases_reach_every_tile():
    """Host-side: the sizes take the tiles they are here for, and all tiles the kernel is built in are among them."""
    for epi, m, n, k, plan in CASES:
        assert _plan(epi, m, n, k) == plan, (epi, m, n, k)
    few = {(64, 64), (128, 64), (192, 64)}
    wide = {(128, 128), (192, 128), (256, 128)}
    want = {fa.EPI_STORE: few, fa.EPI_RESADD: few | wide, fa.EPI_SWIGLU: few | wide | {(64, 128)} | {(r, 160) for r in (64, 128, 192, 256, 384)}}
    for epi, tiles in want.items():
        assert {c[4][:2] for c in CASES if c[0] == epi and c[4]} == tiles, epi


@pytest.mark.gpu
@pytest.mark.parametrize("epi,m,n,k,plan", CASES)
def test_linear(epi, m, n, k, plan):
    gen = torch.Generator(device="cuda").manual_seed(m * 7 + n)
    a, w, w2, c = (torch.randn(s, device="cuda", generator=gen) for s in ((m, k), (n, k), (n, k), (m, n)))
    a, w, w2 = a.bfloat16(), (w / k ** 0.5).bfloat16(), (w2 / k ** 0.5).bfloat16()
    want = a.double() @ w.double().T
    if epi == fa.EPI_SWIGLU:
        want = want / (1 + torch.exp(-want)) * (a.double() @ w2.double().T)
    if epi != fa.EPI_RESADD:
        got = fa.fastav_linear(a, w, epi, w2 if epi == fa.EPI_SWIGLU else None)
        assert ((got.double() - want).norm() / want.norm()).item() < 2.5e-3
        return
    want += c
    for workspace in (True, False):
        got = fa.fastav_linear(a, w, epi, c=c.clone(), use_workspace=workspace)
        assert ((got.double() - want).norm() / want.norm()).item() < 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k,shares", [(64, 1024, 4160, 5), (250, 4096, 8192, 4), (250, 4096, 8192, 3), (100, 2048, 2112, 3)])
def test_linear_with_room_for_some_of_the_partial_tiles(m, n, k, shares):
    """A workspace for fewer partial tiles than planned: nothing is written behind it, the sum is the same to rounding."""
    room = shares * m * n * 4 + 128
    plan = _plan(fa.EPI_RESADD, m, n, k, room)
    assert plan is TILES or plan[2] == shares
    gen = torch.Generator(device="cuda").manual_seed(m + n)
    a, w, c = (torch.randn(s, device="cuda", generator=gen) for s in ((m, k), (n, k), (m, n)))
    a, w = a.bfloat16(), (w / k ** 0.5).bfloat16()
    want = a.double() @ w.double().T + c
    ws = torch.full((room + 4096,), 171, dtype=torch.uint8, device="cuda")
    fa.binding._check(fa.lib().fastav_linear(a.data_ptr(), w.data_ptr(), None, c.data_ptr(), m, n, k, fa.EPI_RESADD, fa.BF16, ws.data_ptr(), room,
                                             torch.cuda.current_stream().cuda_stream))
    assert ((c.double() - want).norm() / want.norm()).item() < 1e-5
    assert bool((ws[room:] == 171).all())


def _model(dh, samples, prunes):
    m = fi.Model(3, 2048, 2048 // dh, 512 // dh, dh, 2560, 1.0e4, 1e-6, "bf16")
    w = fi.Workload("ring", m, samples, prunes, seed=97)
    weights = [fi.layer_weights(m, l, 31) for l in range(m.n_layers)]
    for rows in (sum(w.seqlens), 17):
        for epi, n, k in ((fa.EPI_STORE, 3072, 2048), (fa.EPI_RESADD, 2048, 2048), (fa.EPI_SWIGLU, 2560, 2048), (fa.EPI_RESADD, 2048, 2560)):
            assert _plan(epi, rows, n, k) is not TILES, (rows, epi, n, k)
    return w, weights, fi.embeddings(w), make_decoder(m, weights)


RAGGED = [[(fi.VIDEO, 200), (fi.AUDIO, 110), (fi.TEXT, 21)], [(fi.VIDEO, 97), (fi.AUDIO, 60), (fi.TEXT, 9)]]


@pytest.mark.gpu
@pytest.mark.parametrize("dh", [128, 64])
def test_prefill_against_the_oracle_and_the_separate_launches(dh):
    """497 rows, then about 350 and 280 behind two FINE prunes: every product of the layers runs in the ring kernel.  Rotation in
    the projection's epilogue against the separate kernel (bf16 rounding), with K and V in the caller's caches (an output per
    segment) or in the workspace (the same bits); the row list of the O projection and the partial tiles left to the RMSNorm
    against their separate launches (the same bits); all of it against the oracle."""
    w, weights, x, d = _model(dh, RAGGED, [fi.Prune(1, fi.FINE, 0.7), fi.Prune(2, fi.FINE, 0.8)])
    spans, offs = fi.span_table(w)
    xd = dev(x, "bf16")
    res = {}
    for name, option, value, kv in (("all", None, 1, True), ("workspace", None, 1, False), ("rope", fa.OPT_FUSED_ROPE, 0, True),
                                    ("rows", fa.OPT_FUSED_GATHER_OPROJ, 0, True), ("sums", fa.OPT_FUSED_SPLITK_NORM, 0, True)):
        try:
            if option is not None:
                fa.fastav_set_option(option, value)
            o = d.fastav_prefill(xd, fi.cu_seqlens(w), spans, offs, prune_tuples(w), 1, want_kv=kv)
            torch.cuda.synchronize()
        finally:
            if option is not None:
                fa.fastav_set_option(option, 1)
        res[name] = [o["x_out"].clone(), o["kept_pos"].clone()] + ([t.clone() for p in o["kv"] for t in p] if kv else [])
    for name in ("rows", "sums", "workspace"):
        assert all(torch.equal(a, b) for a, b in zip(res["all"], res[name])), name
    assert torch.equal(res["all"][3], res["rope"][3])                          # V of layer 0: not rotated
    k_f, k_u = host(res["all"][2]), host(res["rope"][2])
    assert np.max(np.abs(k_f - k_u)) <= 2e-2 * max(1.0, np.abs(k_u).max())
    ref = orc.prefill(w, weights, x)
    for t, what in ((2, "K"), (3, "V")):
        want = np.concatenate([r["kv"][0][t - 2] for r in ref])
        assert_close(host(res["all"][t]).reshape(want.shape), want, "bf16", what=f"{what} layer 0")
    pos, cu = res["all"][1].cpu().numpy(), np.concatenate([[0], np.cumsum([len(r["kept_pos"]) for r in ref])])
    for b, r in enumerate(ref):
        mine = pos[cu[b]:cu[b + 1]]
        common, gi, ri = np.intersect1d(mine, r["kept_pos"], return_indices=True)
        assert len(common) >= 0.97 * len(mine)                                 # scores around 1 / n: bf16 exchanges near-ties
        assert rel_l2(host(res["all"][0])[cu[b]:cu[b + 1]][gi], r["x_out"][ri]) <= 1e-2


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,mlp,rows,shares", [(1024, 8192, 60, 16), (2048, 8192, 100, 8), (1536, 5120, 60, 10), (4224, 2048, 100, 3), (5120, 2048, 120, 3), (8192, 1024, 60, 2)])
def test_prefill_partial_tiles_left_to_the_rmsnorm(hidden, mlp, rows, shares):
    """Up to 16 partial tiles per residual row, rows of one to eight registers per thread in the RMSNorm that adds them (it reads two
    or four partial rows at a time): the bits of the separate reduction."""
    assert _plan(fa.EPI_RESADD, rows, hidden, mlp)[2] == shares
    m = fi.Model(3, hidden, 8, 2, 128, mlp, 1.0e4, 1e-6, "bf16")
    w = fi.Workload("partial", m, [[(fi.VIDEO, rows - 20), (fi.TEXT, 20)]], [], seed=5)
    d = make_decoder(m, [fi.layer_weights(m, l, 37) for l in range(m.n_layers)])
    spans, offs = fi.span_table(w)
    xd = dev(fi.embeddings(w), "bf16")
    res = []
    try:
        for fused in (1, 0):
            fa.fastav_set_option(fa.OPT_FUSED_SPLITK_NORM, fused)
            o = d.fastav_prefill(xd, fi.cu_seqlens(w), spans, offs, [], 1, want_kv=True)
            torch.cuda.synchronize()
            res.append([o["x_out"].clone()] + [t.clone() for p in o["kv"] for t in p])
    finally:
        fa.fastav_set_option(fa.OPT_FUSED_SPLITK_NORM, 1)
    assert all(torch.isfinite(t.float()).all() for t in res[0])
    assert all(torch.equal(a, b) for a, b in zip(*res))


@pytest.mark.gpu
def test_prefill_of_a_batch_agrees_with_its_samples_to_rounding():
    """Tiles and K shares follow the number of rows, and with them the order of the fp32 sums: a batch and its samples alone
    agree to bf16 rounding (every layer's rounding of the hidden state differs in the last place here and there)."""
    w, _, x, d = _model(128, RAGGED, [fi.Prune(1, fi.GLOBAL, 0.6)])
    spans, offs = fi.span_table(w)
    cu = fi.cu_seqlens(w)
    both = d.fastav_prefill(dev(x, "bf16"), cu, spans, offs, prune_tuples(w), 1)
    torch.cuda.synchronize()
    xb, pb, cb = host(both["x_out"]), both["kept_pos"].cpu().numpy(), both["cu_seqlens_out"].cpu().numpy()
    for b, s in enumerate(w.samples):
        one = fi.Workload("one", w.model, [s], w.prunes, seed=w.seed)
        sp, of = fi.span_table(one)
        o = d.fastav_prefill(dev(x[cu[b]:cu[b + 1]], "bf16"), fi.cu_seqlens(one), sp, of, prune_tuples(one), 1)
        torch.cuda.synchronize()
        assert np.array_equal(o["kept_pos"].cpu().numpy(), pb[cb[b]:cb[b + 1]])
        assert rel_l2(host(o["x_out"]), xb[cb[b]:cb[b + 1]]) <= 1e-2
