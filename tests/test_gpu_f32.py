"""The fp32 matrix-core kernels at the edges of their tiles: 32 x 32 tiles, 16-wide k chunks, the three workgroup
forms of the products (8 and 4 waves on a tile, waves of 64 x 64 from 2048 tiles on), 16-row / 16-key attention tiles;
and a prefill whose sizes are multiples of none of them.  Tolerances: gpu_util's fp32 ones."""
import numpy as np
import pytest
import torch

import fastav_inputs as fi
import paper_2601_13143_amd as fa
from gpu_util import assert_close, dev, host, make_decoder, model_struct, prune_tuples
from oracle import fastav_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(1, 16, 4), (33, 48, 20), (31, 33, 64), (128, 256, 688), (520, 1040, 36), (2050, 1060, 132),
                                   (2017, 1041, 16), (4000, 530, 12), (1100, 2000, 48), (65, 32800, 64)])
@pytest.mark.parametrize("epi", [fa.EPI_STORE, fa.EPI_RESADD, fa.EPI_SWIGLU])
def test_linear(m, n, k, epi):
    rng = np.random.default_rng(m * 7 + n)
    a, w, w2, c = (rng.standard_normal(s).astype(np.float32) for s in ((m, k), (n, k), (n, k), (m, n)))
    w /= np.sqrt(k)
    got = fa.fastav_linear(dev(a, "f32"), dev(w, "f32"), epi, dev(w2, "f32") if epi == fa.EPI_SWIGLU else None,
                           dev(c, "f32") if epi == fa.EPI_RESADD else None)
    want = a.astype(np.float64) @ w.astype(np.float64).T
    if epi == fa.EPI_RESADD:
        want += c
    elif epi == fa.EPI_SWIGLU:
        want = orc.silu(want) * (a.astype(np.float64) @ w2.astype(np.float64).T)
    assert_close(host(got), want, "f32", scale=max(1.0, np.abs(want).std()), what=f"linear {m}x{n}x{k} epi {epi}")


@pytest.mark.parametrize("dh,hq,hkv", [(64, 4, 2), (128, 6, 2), (64, 3, 3)])
@pytest.mark.parametrize("lens", [[1], [15, 16, 17], [127, 300], [513]])
def test_attention(dh, hq, hkv, lens):
    rng = np.random.default_rng(sum(lens) + dh)
    T = sum(lens)
    q, k, v = (rng.standard_normal((T, h, dh)).astype(np.float32) for h in (hq, hkv, hkv))
    model = fa.make_model(1, 64, hq, hkv, dh, 64, dtype=fa.F32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    o, ll, ml = fa.fastav_attention(model, dev(q, "f32"), dev(k, "f32"), dev(v, "f32"), torch.from_numpy(cu).cuda(), max(lens), want_last=True)
    o, ll, ml = host(o), host(ll), host(ml)
    for b in range(len(lens)):
        lo, hi = cu[b], cu[b + 1]
        qs, ks, vs = (t[lo:hi].astype(np.float64) for t in (q, k, v))
        assert_close(o[lo:hi], orc.causal_gqa_attention(qs, ks, vs), "f32", what=f"attention {lens} sample {b}")
        for h in range(hq):
            z = ks[:, h // (hq // hkv)] @ qs[-1, h] / np.sqrt(dh)
            np.testing.assert_allclose(ll[h, lo:hi], z, atol=2e-5 * max(1.0, np.abs(z).max()))
            np.testing.assert_allclose(ml[b, h], [z.max(), np.exp(z - z.max()).sum()], rtol=2e-5, atol=2e-5)


def _masked_attention(dh, n, masked):
    """One fp32 sample whose keys of the ranges `masked` have the logit -inf for every query: q . k overflows to -inf there
    (the first dimension is 3e38 on those keys against -4 on every query) and is ordinary elsewhere."""
    rng = np.random.default_rng(dh + n)
    q, k, v = (rng.standard_normal((n, h, dh)).astype(np.float32) for h in (4, 2, 2))
    q[:, :, 0], k[:, :, 0] = -4.0, 0.0
    off = np.zeros(n, dtype=bool)
    for lo, hi in masked:
        off[lo:hi] = True
        k[lo:hi, :, 0] = 3.0e38
    model = fa.make_model(1, 64, 4, 2, dh, 64, dtype=fa.F32)
    got = fa.fastav_attention(model, dev(q, "f32"), dev(k, "f32"), dev(v, "f32"), torch.tensor([0, n], dtype=torch.int32, device="cuda"), n, want_last=True)
    z = np.einsum("ihd,jhd->hij", q[:, :, 1:].astype(np.float64), k.repeat(2, axis=1)[:, :, 1:].astype(np.float64)) / np.sqrt(dh)
    z[:, np.triu(np.ones((n, n), dtype=bool), 1)] = -np.inf
    z[:, :, off] = -np.inf
    return [host(t) for t in got], z, v.repeat(2, axis=1).astype(np.float64)


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("n,masked", [(512, [(32, 48)]), (300, [(16, 200)]), (130, [(64, 80), (112, 128)]), (40, [(0, 16)])])
def test_attention_with_logits_of_minus_infinity(dh, n, masked):
    """Whole 16-key tiles at -inf, among them the first ones a wave takes and the first of the sample: rows that see a finite
    logit are what the softmax over their finite logits gives; rows that see none are 0 / 0."""
    (o, ll, ml), z, v = _masked_attention(dh, n, masked)
    m = z.max(axis=2)
    live = m[0] > -np.inf
    p = np.exp(z[:, live] - m[:, live, None])
    want = np.einsum("hij,jhd->ihd", p / p.sum(axis=2, keepdims=True), v)
    assert_close(o[live], want, "f32", what=f"attention {n}, -inf at {masked}")
    assert np.isnan(o[~live]).all()
    assert np.array_equal(np.isneginf(ll), np.isneginf(z[:, -1]))
    np.testing.assert_allclose(ml[0, :, 0], m[:, -1], rtol=2e-5, atol=2e-5)
    np.testing.assert_allclose(ml[0, :, 1], p[:, -1].sum(axis=1), rtol=2e-5)


def test_attention_whose_last_row_sees_no_finite_logit():
    """(max, sum) of such a row are (-inf, 0)."""
    (o, _, ml), _, _ = _masked_attention(64, 70, [(0, 70)])
    assert np.isnan(o).all() and np.isneginf(ml[0, :, 0]).all() and (ml[0, :, 1] == 0).all()


@pytest.mark.parametrize("hidden,hq,hkv,dh,mlp,samples", [
    (100, 3, 1, 64, 76, [[(fi.VIDEO, 40), (fi.AUDIO, 29), (fi.TEXT, 6)]]),
    (132, 2, 2, 128, 90, [[(fi.VIDEO, 33), (fi.TEXT, 1)], [(fi.AUDIO, 150), (fi.TEXT, 20)]]),
    (128, 16, 2, 64, 530, [[(fi.VIDEO, 700), (fi.AUDIO, 390), (fi.TEXT, 21)], [(fi.AUDIO, 1080), (fi.TEXT, 20)]]),   # 64 x 64 per wave
    (66, 2, 1, 64, 70, [[(fi.VIDEO, 50), (fi.TEXT, 5)]]),          # hidden no multiple of 4: the separate launches
])
def test_prefill(hidden, hq, hkv, dh, mlp, samples):
    m = fi.Model(3, hidden, hq, hkv, dh, mlp, 1.0e4, 1e-6, "f32")
    w = fi.Workload("odd", m, samples, [fi.Prune(1, fi.GLOBAL, 0.8), fi.Prune(2, fi.FINE, 0.7)], seed=5)
    weights = [fi.layer_weights(m, l, 3) for l in range(m.n_layers)]
    x = fi.embeddings(w)
    dec = make_decoder(m, weights)
    spans, offs = fi.span_table(w)
    out = dec.fastav_prefill(dev(x, "f32"), fi.cu_seqlens(w), spans, offs, prune_tuples(w), 1, want_kv=True)
    ref = orc.prefill(w, weights, x, keep_kv=True)
    cu = out["cu_seqlens_out"].cpu().numpy()
    for b, r in enumerate(ref):
        assert np.array_equal(out["kept_pos"].cpu().numpy()[cu[b]:cu[b + 1]], r["kept_pos"])
        assert_close(host(out["x_out"])[cu[b]:cu[b + 1]], r["x_out"], "f32", what=f"x_out {b}")
    for l in range(m.n_layers):
        for t in range(2):
            got = host(out["kv"][l][t])
            want = np.concatenate([r["kv"][l][t] for r in ref])
            assert_close(got, want.reshape(got.shape), "f32", what=f"kv {l} {t}")
