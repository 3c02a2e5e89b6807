"""The bf16 attention kernel in each of the forms its launcher cuts a launch into, at the edges of the rule."""
import numpy as np
import pytest
import torch

import fastav_inputs as fi
import paper_2601_13143_amd as fa
from gpu_util import assert_close, dev, host

pytestmark = pytest.mark.gpu


def _reference(q, k, v, lens):
    """Causal GQA attention in 64 bits on the CPU, and the last row's logits with their (max, sum)."""
    T, Hq, dh = q.shape
    G = Hq // k.shape[1]
    out, at, last, ml = np.empty((T, Hq, dh)), 0, np.empty((Hq, T)), np.empty((len(lens), Hq, 2))
    for b, n in enumerate(lens):
        sl = slice(at, at + n)
        for h in range(Hq):
            z = q[sl, h] @ k[sl, h // G].T / np.sqrt(dh)
            z[np.triu_indices(n, 1)] = -np.inf
            m = z.max(axis=1, keepdims=True)
            p = np.exp(z - m)
            out[sl, h] = p @ v[sl, h // G] / p.sum(axis=1, keepdims=True)
            last[h, sl], ml[b, h] = z[-1], (m[-1, 0], p[-1].sum())
        at += n
    return out, last, ml


# tiles: fewer than three query tiles, or more items than CUs; split: up to 256 items, ten tiles and up to 512 items
# (heads of 64: 576 from five tiles on, 672 from ten, 1024 from sixteen); pairs: 480 to 512 pairs of even samples
@pytest.mark.parametrize("Hq,Hkv,dh,lens", [
    (8, 2, 128, [256]), (8, 2, 128, [257]), (8, 2, 128, [384]), (8, 2, 128, [385, 1, 130]), (8, 8, 64, [319]), (28, 4, 128, [331]),
    (32, 8, 128, [1024]), (32, 8, 128, [1025]), (32, 8, 128, [1153]), (16, 4, 64, [1300]), (32, 8, 128, [331, 300, 290]),
    (64, 8, 64, [250] * 8), (60, 6, 128, [129] * 8), (64, 8, 64, [250] * 7 + [100]),
    (64, 8, 64, [600, 590]), (64, 8, 64, [512, 500]), (48, 8, 64, [1300]), (64, 8, 64, [1409]), (16, 4, 64, [1930, 1700, 1600])])
def test_forms_against_float64(Hq, Hkv, dh, lens):
    rng = np.random.default_rng(Hq + dh + sum(lens))
    T = sum(lens)
    q, k, v = (fi.round_bf16(rng.standard_normal((T, h, dh)).astype(np.float32)) for h in (Hq, Hkv, Hkv))
    m = fa.make_model(1, 64, Hq, Hkv, dh, 64)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    args = (m, dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), cu, max(lens))
    o, ll, ml = fa.fastav_attention(*args, want_last=True)
    # two builds of one form, and pairs against tiles, add the same key tiles in the same order
    assert torch.equal(o, fa.fastav_attention(*args))
    want, last, wml = _reference(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), lens)
    assert_close(host(o), want, "bf16", what=f"attention {lens}")
    assert np.max(np.abs(host(ll) - last)) <= 1e-3 * max(1.0, np.abs(last).max())
    assert np.max(np.abs(host(ml)[..., 0] - wml[..., 0])) <= 1e-3 * max(1.0, np.abs(wml[..., 0]).max())
    assert np.max(np.abs(host(ml)[..., 1] / wml[..., 1] - 1.0)) <= 4e-3          # the kernel sums probabilities rounded to bf16


def test_short_sample_gives_the_same_bits_beside_a_long_one():
    """One or two query tiles run on one key group also where the batch's longest sample splits its keys over two."""
    rng = np.random.default_rng(3)
    lens = [250, 700, 90]
    T, m = sum(lens), fa.make_model(1, 64, 8, 2, 128, 64)
    q, k, v = (dev(fi.round_bf16(rng.standard_normal((T, h, 128)).astype(np.float32)), "bf16") for h in (8, 2, 2))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    both = fa.fastav_attention(m, q, k, v, torch.from_numpy(cu).cuda(), max(lens))
    for b, n in enumerate(lens):
        sl = slice(cu[b], cu[b + 1])
        one = fa.fastav_attention(m, q[sl], k[sl], v[sl], torch.tensor([0, n], dtype=torch.int32, device="cuda"), n)
        assert torch.equal(one, both[sl])


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("group", [1, 2])
def test_split_keys_with_one_group_at_minus_infinity(dh, group):
    """A row whose keys in one group's tiles all have the logit -inf is what the softmax over the other group's keys gives.
    group 1: key tiles 1, 3, ..; group 2: key tile 1 only, so that group 1 starts on -inf and meets finite keys later."""
    n, Hq, Hkv = 400, 4, 2
    rng = np.random.default_rng(dh)
    q, k, v = (fi.round_bf16(rng.standard_normal((n, h, dh)).astype(np.float32)) for h in (Hq, Hkv, Hkv))
    q[:, :, 0], k[:, :, 0] = -4.0, 0.0
    tile = np.arange(n) // 64
    off = tile % 2 == 1 if group == 1 else tile == 1
    k[off, :, 0] = 3.0e38                                                        # q . k overflows to -inf
    k = fi.round_bf16(k)
    cu = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    o = host(fa.fastav_attention(fa.make_model(1, 64, Hq, Hkv, dh, 64), dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), cu, n))
    kk = k.astype(np.float64).copy()
    kk[:, :, 0] = 0.0
    want = np.empty((n, Hq, dh))
    for h in range(Hq):
        z = q[:, h].astype(np.float64) @ kk[:, h // 2].T / np.sqrt(dh)
        z[np.triu_indices(n, 1)] = -np.inf
        z[:, off] = -np.inf
        p = np.exp(z - z.max(axis=1, keepdims=True))
        want[:, h] = p @ v[:, h // 2].astype(np.float64) / p.sum(axis=1, keepdims=True)
    assert_close(o, want, "bf16", what=f"attention, group {group} at -inf")
