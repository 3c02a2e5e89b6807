"""Eq. 4 scores of a batch large enough for the wide launch forms (eight KV heads per workgroup, four positions per thread)
against its samples one by one, which take the narrow ones: the sums are the same, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2601_13143_amd as fa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,dh,extra", [(32, 8, 128, 0), (28, 4, 128, 0), (12, 3, 64, 0), (8, 2, 128, 1)])
def test_batch_equals_samples(hq, hkv, dh, extra):
    rng = np.random.default_rng(hq + extra)
    lens = rng.integers(1, 300, 170)
    lens[-1] += -int(lens.sum()) % 4 + extra          # planes 16-byte aligned, or not (extra)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randn((int(cu[-1]), hq, dh), device="cuda", generator=gen).bfloat16()
    k = torch.randn((int(cu[-1]), hkv, dh), device="cuda", generator=gen).bfloat16()
    model = fa.make_model(1, 64, hq, hkv, dh, 64)
    got = fa.fastav_score(model, q, k, torch.from_numpy(cu).cuda(), int(lens.max()))
    for b in (0, 1, 2, 3, 63, 128, 168, 169):
        rows = slice(int(cu[b]), int(cu[b + 1]))
        n = int(lens[b])
        one = fa.fastav_score(model, q[rows], k[rows], torch.tensor([0, n], dtype=torch.int32, device="cuda"), n)
        assert torch.equal(got[rows], one), (b, n)
        kk = k[rows].double().repeat_interleave(hq // hkv, dim=1)
        p = torch.softmax((q[rows][-1].double()[None] * kk).sum(-1) / dh ** 0.5, dim=0).mean(1)
        assert ((one.double() - p).norm() / p.norm()).item() < 2e-6
