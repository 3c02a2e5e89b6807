"""GPU parity of the attention-rollout analysis (Eq. 2-3) against the CPU oracle, through the C ABI."""
import ctypes as C

import numpy as np
import pytest
import torch

import fastav_inputs as fi
from oracle import fastav_oracle as orc
import paper_2601_13143_amd as fa
from gpu_util import dev, host, make_decoder, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,dh,n", [(8, 2, 128, 300), (4, 4, 64, 132), (28, 4, 128, 260), (32, 8, 128, 1028), (4, 2, 128, 4)])
def test_attention_map_matches_oracle(Hq, Hkv, dh, n):
    """Head-mean causal attention map of one layer on identical bf16 inputs: entries are probabilities (<= 1),
    written as bf16, so they are compared relative to the row's own scale."""
    rng = np.random.default_rng(Hq + n)
    q = fi.round_bf16((rng.standard_normal((n, Hq, dh)) * 1.3).astype(np.float32))
    k = fi.round_bf16((rng.standard_normal((n, Hkv, dh)) * 1.3).astype(np.float32))
    m = fa.make_model(1, 64, Hq, Hkv, dh, 64)
    got = host(fa.fastav_attention_map(m, dev(q, "bf16"), dev(k, "bf16")))
    want = orc.head_mean_attention_map(q.astype(np.float64), k.astype(np.float64))
    assert np.all(np.triu(got, 1) == 0.0)
    assert np.max(np.abs(got.sum(axis=1) - 1.0)) <= 5e-3               # bf16 entries: each within 2^-9 of itself
    assert rel_l2(got, want) <= 5e-3, rel_l2(got, want)
    assert np.max(np.abs(got - want) / np.maximum(want, 1.0 / n)) <= 2e-2


def _small(n_layers=3):
    m = fi.Model(n_layers, 512, 8, 2, 128, 1024, 1.0e4, 1e-6, "bf16")
    w = fi.Workload("roll", m, [[(fi.TEXT, 8), (fi.VIDEO, 144), (fi.AUDIO, 92), (fi.TEXT, 12)]], [], seed=51)
    weights = [fi.layer_weights(m, l, 13) for l in range(m.n_layers)]
    for W in weights:                                # sharper attention than N(0, 0.02) weights give
        W["wq"] = fi.round_bf16((W["wq"] * 6.0).astype(np.float32))
        W["wk"] = fi.round_bf16((W["wk"] * 6.0).astype(np.float32))
    return m, w, weights, fi.embeddings(w)


@pytest.mark.parametrize("alpha", [0.5, 1.0, 0.0])
def test_rollout_matches_oracle(alpha):
    m, w, weights, x = _small()
    dec = make_decoder(m, weights)
    n = x.shape[0]
    want = orc.attention_rollout(m, weights, x, alpha)
    for upto in (1, 2, 3):
        got = host(dec.fastav_rollout(dev(x, "bf16"), alpha, upto))
        torch.cuda.synchronize()
        assert np.max(np.abs(got.sum(axis=1) - 1.0)) <= 1e-2            # rows of a rollout sum to 1
        assert np.all(np.abs(np.triu(got, 1)) <= 1e-6)
        assert rel_l2(got, want[upto - 1]) <= 1e-2, (alpha, upto, rel_l2(got, want[upto - 1]))
    if alpha == 0.0:
        assert np.array_equal(got, np.eye(n))


def test_rollout_is_deterministic_and_rejects_bad_arguments():
    m, w, weights, x = _small(2)
    dec = make_decoder(m, weights)
    a = dec.fastav_rollout(dev(x, "bf16"), 0.7).clone()
    b = dec.fastav_rollout(dev(x, "bf16"), 0.7)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    with pytest.raises(fa.FastavError):
        dec.fastav_rollout(dev(x, "bf16"), 1.5)
    with pytest.raises(fa.FastavError):
        dec.fastav_rollout(dev(x, "bf16"), 0.5, 3)             # more layers than the model has
    with pytest.raises(fa.FastavError):
        dec.fastav_rollout(dev(x[:254], "bf16"), 0.5)          # n not a multiple of 4


def _cutoff_from(infl32: np.ndarray, prot: np.ndarray, thr: float) -> int:
    """The integer decision on given fp32 influences, in the precision the library compares in."""
    hit = np.nonzero((~prot) & (infl32.astype(np.float32) * np.float32(len(infl32)) >= np.float32(thr)))[0]
    return int(hit[-1]) + 1 if hit.size else 0


@pytest.mark.parametrize("n", [4, 132, 1028, 4100])
def test_rollout_influence_and_cutoff_on_given_matrices(n):
    """Column means and the threshold -> cut-off position on identical fp32 rollout matrices (a lower-triangular
    row-stochastic matrix with early columns favoured and a few late outliers)."""
    rng = np.random.default_rng(n)
    R = np.tril(rng.random((n, n)) * np.exp(-np.arange(n) / (0.3 * n))[None, :] + 1e-4)
    for j in rng.integers(n // 2, n, 3):
        R[:, j] *= 6.0
    R = (R / R.sum(axis=1, keepdims=True)).astype(np.float32)
    prot = np.zeros(n, dtype=bool)
    prot[: max(1, n // 50)] = True; prot[-max(1, n // 40):] = True
    r_dev = torch.from_numpy(np.ascontiguousarray(R.T)).cuda().t()       # the layout fastav_rollout returns
    p_dev = torch.from_numpy(prot.astype(np.uint8)).cuda()
    want = orc.rollout_influence(R)
    for thr in (0.0, 0.5, 1.0, 2.0, 5.0, 1e9):
        infl, cut = fa.fastav_rollout_cutoff(r_dev, p_dev, thr)
        g = infl.cpu().numpy()
        np.testing.assert_allclose(g, want, rtol=2e-5, atol=1e-9)
        assert abs(g.sum() - 1.0) < 1e-4
        c = int(cut.cpu()[0])
        assert c == _cutoff_from(g, prot, thr)                            # integer work on the same values: exact
        margin = np.min(np.abs(want[~prot] * n - thr)) if (~prot).any() else 1.0
        if margin > 1e-4 * max(1.0, thr):                                 # no influence sits on the threshold
            assert c == orc.rollout_cutoff(R, prot, thr), (thr, c)
    assert int(fa.fastav_rollout_cutoff(r_dev, torch.ones_like(p_dev), 0.0)[1].cpu()[0]) == 0   # no candidates


def test_rollout_cutoff_after_a_rollout_and_bad_arguments():
    m, w, weights, x = _small()
    dec = make_decoder(m, weights)
    r = dec.fastav_rollout(dev(x, "bf16"), 0.5, 3)
    prot = orc.protected_mask(w.samples[0], 1)
    infl, cut = fa.fastav_rollout_cutoff(r, torch.from_numpy(prot.astype(np.uint8)).cuda(), 1.0)
    got_r = host(r)
    np.testing.assert_allclose(infl.cpu().numpy(), orc.rollout_influence(got_r), rtol=2e-5, atol=1e-9)
    assert int(cut.cpu()[0]) == _cutoff_from(infl.cpu().numpy(), prot, 1.0)
    want = orc.attention_rollout(m, weights, x, 0.5)[2]
    assert rel_l2(infl.cpu().numpy(), orc.rollout_influence(want)) <= 1e-2
    lib = fa.lib()
    ok = (r.t().data_ptr(), 256, torch.zeros(256, dtype=torch.uint8, device="cuda").data_ptr())
    assert lib.fastav_rollout_cutoff(None, 256, ok[2], 1.0, infl.data_ptr(), cut.data_ptr(), None) == 1
    assert lib.fastav_rollout_cutoff(ok[0], 255, ok[2], 1.0, infl.data_ptr(), cut.data_ptr(), None) == 1
    assert lib.fastav_rollout_cutoff(ok[0], 0, ok[2], 1.0, infl.data_ptr(), cut.data_ptr(), None) == 1
    assert lib.fastav_rollout_cutoff(ok[0], 256, ok[2], -1.0, infl.data_ptr(), cut.data_ptr(), None) == 1
    assert lib.fastav_rollout_cutoff(ok[0], 256, ok[2], float("nan"), infl.data_ptr(), cut.data_ptr(), None) == 1


@pytest.mark.parametrize("Hq,Hkv,dh,n", [(3, 3, 64, 36), (9, 3, 128, 64), (12, 4, 128, 516), (16, 1, 64, 68)])
def test_attention_map_heads_and_keys_dealt_over_waves(Hq, Hkv, dh, n):
    """Head counts that are no multiple of a workgroup's eight waves (or fewer), and key counts below, at and just beyond
    the blocks that the waves take in turn."""
    test_attention_map_matches_oracle(Hq, Hkv, dh, n)


@pytest.mark.parametrize("n", [8, 64, 68, 128, 196, 388])
def test_rollout_at_the_edges_of_its_tiles(n):
    """One to seven 64 x 64 tiles a side, whole and ragged, and more K slices than a workgroup has waves."""
    m = fi.Model(3, 512, 8, 2, 128, 1024, 1.0e4, 1e-6, "bf16")
    w = fi.Workload("roll", m, [[(fi.TEXT, 4), (fi.VIDEO, n - 4)]], [], seed=n)
    weights = [fi.layer_weights(m, l, 17) for l in range(m.n_layers)]
    for W in weights:
        W["wq"] = fi.round_bf16((W["wq"] * 6.0).astype(np.float32))
        W["wk"] = fi.round_bf16((W["wk"] * 6.0).astype(np.float32))
    x = fi.embeddings(w)
    dec = make_decoder(m, weights)
    want = orc.attention_rollout(m, weights, x, 0.6)
    for upto in (1, 3):                                # the statistics of the map's own pass, and those of the attention
        got = host(dec.fastav_rollout(dev(x, "bf16"), 0.6, upto))
        assert rel_l2(got, want[upto - 1]) <= 1e-2, (n, upto, rel_l2(got, want[upto - 1]))   # the bound of the rollout above
        assert np.all(np.triu(got, 1) == 0.0)


@pytest.mark.parametrize("Hq,Hkv,dh,n", [(4, 2, 128, 1476), (8, 4, 64, 1476), (4, 4, 64, 900), (20, 4, 128, 396), (2, 1, 64, 2052), (60, 12, 128, 1300), (64, 8, 64, 1412)])
def test_rollout_with_the_statistics_of_every_attention_form(Hq, Hkv, dh, n):
    """Ragged prompts whose map takes the 64 x 64 tiles of two waves' shares (beyond 256 tiles) or of four, and the short form; row
    statistics from attention with split keys and with a tile per workgroup of many key tiles; the step's sums over up to nine slices
    a wave; heads of 64 and of 128."""
    m = fi.Model(2, 256, Hq, Hkv, dh, 256, 1.0e4, 1e-6, "bf16")
    w = fi.Workload("roll", m, [[(fi.TEXT, 4), (fi.VIDEO, n - 4)]], [], seed=n)
    weights = [fi.layer_weights(m, l, 19) for l in range(m.n_layers)]
    for W in weights:
        W["wq"] = fi.round_bf16((W["wq"] * 6.0).astype(np.float32))
        W["wk"] = fi.round_bf16((W["wk"] * 6.0).astype(np.float32))
    x = fi.embeddings(w)
    want = orc.attention_rollout(m, weights, x, 0.6)
    got = host(make_decoder(m, weights).fastav_rollout(dev(x, "bf16"), 0.6, 2))
    assert rel_l2(got, want[1]) <= 1e-2, rel_l2(got, want[1])          # the bound of the rollout above
    assert np.max(np.abs(got.sum(axis=1) - 1.0)) <= 1e-2
    assert np.all(np.triu(got, 1) == 0.0)


@pytest.mark.parametrize("Hq,Hkv,dh,n", [(3, 1, 128, 1412), (5, 5, 64, 1476), (1, 1, 64, 68)])
def test_attention_map_with_more_tiles_than_cus(Hq, Hkv, dh, n):
    """Beyond 256 tiles the heads are dealt over two waves a block instead of four; head counts that no share divides."""
    test_attention_map_matches_oracle(Hq, Hkv, dh, n)


@pytest.mark.parametrize("n", [64, 200, 1480, 1476])
def test_attention_map_into_memory_off_a_16_byte_boundary(n):
    """The map's rows may lie at 8-byte addresses: the base 8 bytes past a 16-byte boundary, or a pitch that is no multiple of 16 bytes."""
    m = fa.make_model(1, 64, 4, 2, 64, 64)
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, k = (torch.randn((n, h, 64), device="cuda", generator=gen).bfloat16() for h in (4, 2))
    want = fa.fastav_attention_map(m, q, k)
    buf = torch.full((n * n + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(fa.lib().fastav_attention_map_workspace_bytes(n, 4), dtype=torch.uint8, device="cuda")
    fa.binding._check(fa.lib().fastav_attention_map(C.byref(m), q.data_ptr(), q.stride(0), k.data_ptr(), k.stride(0), n, buf.data_ptr() + 8, ws.data_ptr(),
                                                    ws.numel(), torch.cuda.current_stream().cuda_stream))
    assert torch.equal(buf[4:-4].view(n, n), want)
    assert bool((buf[:4] == 7.0).all()) and bool((buf[-4:] == 7.0).all())


@pytest.mark.parametrize("Hq,Hkv,dh,n", [(6, 3, 64, 896), (6, 3, 64, 900), (4, 2, 128, 832), (4, 2, 128, 836), (24, 6, 128, 200), (24, 8, 128, 200), (8, 2, 128, 68)])
def test_attention_map_on_both_sides_of_the_short_form(Hq, Hkv, dh, n):
    """Short prompts take 32 x 64 tiles read straight from memory, up to 896 tokens (heads of 64) or 832 (few heads of 128, or many
    to a key head)."""
    test_attention_map_matches_oracle(Hq, Hkv, dh, n)


def test_attention_map_of_rows_far_apart():
    """Keys 68 MB apart: the rows of one tile lie further from each other than a 32-bit byte offset reaches."""
    n, pitch = 840, 34_100_000
    m = fa.make_model(1, 64, 8, 2, 128, 64)
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k = (torch.randn((n, h, 128), device="cuda", generator=gen).bfloat16() for h in (8, 2))
    apart = torch.empty((n - 1) * pitch + 256, dtype=torch.bfloat16, device="cuda").as_strided((n, 2, 128), (pitch, 128, 1))
    apart.copy_(k)
    got, want = host(fa.fastav_attention_map(m, q, apart)), host(fa.fastav_attention_map(m, q, k))
    assert rel_l2(got, want) <= 1e-3                       # the heads' sums in another order, entries rounded to bf16
    assert np.all(np.triu(got, 1) == 0.0)
