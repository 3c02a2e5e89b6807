"""The prefill's first launch (schedule, positions, protected rows, fp32 embeddings, rotary table) and outputs that are written in place."""
import numpy as np
import pytest
import torch

import fastav_inputs as fi
import paper_2601_13143_amd as fa
from gpu_util import dev, host, make_decoder, prune_tuples
from oracle import fastav_oracle as orc

pytestmark = pytest.mark.gpu


def _case(samples, prunes, dtype, hidden=192, seed=5):
    m = fi.Model(2, hidden, 4, 2, 64, 256, 1.0e4, 1e-6, dtype)
    w = fi.Workload("setup", m, samples, prunes, seed=seed)
    weights = [fi.layer_weights(m, l, 3) for l in range(m.n_layers)]
    return w, weights, fi.embeddings(w)


def _run(dec, w, x, **kw):
    spans, offs = fi.span_table(w)
    o = dec.fastav_prefill(x, fi.cu_seqlens(w), spans, offs, prune_tuples(w), 1, **kw)
    torch.cuda.synchronize()
    return o


def _check(w, weights, x, o, tol):
    ref = orc.prefill(w, weights, x, keep_kv=False)
    cu = o["cu_seqlens_out"].cpu().numpy()
    assert cu.tolist() == np.concatenate([[0], np.cumsum([len(r["kept_pos"]) for r in ref])]).tolist()
    for b, r in enumerate(ref):
        assert np.array_equal(o["kept_pos"].cpu().numpy()[cu[b]:cu[b + 1]], r["kept_pos"])
        g = host(o["x_out"])[cu[b]:cu[b + 1]]
        assert np.linalg.norm(g - r["x_out"]) <= tol * np.linalg.norm(r["x_out"]), b


@pytest.mark.parametrize("dtype,tol", [("f32", 2e-5), ("bf16", 1e-2)])
@pytest.mark.parametrize("prunes", [[], [fi.Prune(1, fi.GLOBAL, 0.5)]])
@pytest.mark.parametrize("batch", [1, 3, 200])
def test_setup_and_outputs(batch, prunes, dtype, tol):
    """One sample to 200 (whose schedule and spans do not fit the kernel arguments: separate launches), with the last stage's
    rows written to the outputs by the set-up (no prune) or by the last compaction; spans that start mid-sample, rows that
    end inside a workgroup."""
    samples = [[(fi.TEXT, 1 + b % 3), (fi.VIDEO, 4 + b % 5), (fi.AUDIO, 3), (fi.TEXT, 2)] for b in range(batch)]
    if batch == 3:
        samples[1] = [(fi.VIDEO, 300), (fi.TEXT, 7), (fi.AUDIO, 211)]
    w, weights, x = _case(samples, prunes, dtype, hidden=200 if dtype == "f32" else 192)
    _check(w, weights, x, _run(make_decoder(w.model, weights), w, dev(x, dtype)), tol)


@pytest.mark.parametrize("hidden", [64, 1028, 4096, 4100, 8192, 8196])
@pytest.mark.parametrize("prune", [[], [fi.Prune(0, fi.GLOBAL, 0.5)]])
def test_first_normalisation_in_the_setup(hidden, prune):
    """The first layer's RMSNorm is made by the set-up for rows of up to 4096 and up to 8192 elements, by its own launch beyond and
    where a prune comes before it; rows that end inside a workgroup's last round of loads."""
    w, weights, x = _case([[(fi.VIDEO, 30), (fi.TEXT, 3)], [(fi.AUDIO, 7), (fi.TEXT, 2)]], prune, "bf16", hidden=hidden)
    _check(w, weights, x, _run(make_decoder(w.model, weights), w, dev(x, "bf16")), 1e-2)


def test_output_over_the_input():
    """x_out in the memory of x (an fp32 model without a prune): the residual stream then stays in the workspace."""
    w, weights, x = _case([[(fi.VIDEO, 40), (fi.TEXT, 9)]], [], "f32")
    dec, xd = make_decoder(w.model, weights), dev(x, "f32")
    want = _run(dec, w, xd.clone())
    outputs = {k: torch.empty_like(want[k]) for k in ("cu_seqlens_out", "kept_pos")}
    got = _run(dec, w, xd, outputs={"x_out": xd, **outputs})
    assert got["x_out"].data_ptr() == xd.data_ptr()
    assert torch.equal(got["x_out"], want["x_out"]) and torch.equal(got["kept_pos"], want["kept_pos"]) and torch.equal(got["cu_seqlens_out"], want["cu_seqlens_out"])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("prunes", [[], [fi.Prune(0, fi.FINE, 0.5)], [fi.Prune(0, fi.GLOBAL, 0.7), fi.Prune(1, fi.FINE, 0.6)]])
@pytest.mark.parametrize("shared", ["kept_pos in x", "cu in x", "kept_pos over the last kept rows", "x_out over a cache", "kept_pos in a layer's output"])
def test_outputs_that_share_memory_with_another_buffer(shared, prunes, dtype):
    """The hidden states, positions and prefix sums are the call's last writes, whatever buffer of the call their memory was before."""
    w, weights, x = _case([[(fi.VIDEO, 300), (fi.TEXT, 9)], [(fi.AUDIO, 55), (fi.TEXT, 3)]], prunes, dtype, hidden=64)
    dec = make_decoder(w.model, weights)
    xd = dev(x, dtype)
    want = _run(dec, w, xd.clone(), want_kv=True, want_trace=True, want_layers=True)
    o = {k: v if not torch.is_tensor(v) else torch.empty_like(v) for k, v in want.items()}
    o["kv"] = [tuple(torch.empty_like(t) for t in kv) for kv in want["kv"]]
    o["prune_keep_idx"] = [torch.empty_like(t) for t in want["prune_keep_idx"]]
    o["layer_x"] = [torch.empty_like(t) for t in want["layer_x"]]
    words = lambda t, n: t.view(-1).view(torch.int32)[-n:]
    if shared == "kept_pos in x":
        o["kept_pos"] = words(xd, o["kept_pos"].numel())
    elif shared == "cu in x":
        o["cu_seqlens_out"] = words(xd, o["cu_seqlens_out"].numel())
    elif shared == "kept_pos over the last kept rows":
        o["kept_pos"] = (o["prune_keep_idx"] or [o["kept_pos"]])[-1]
    elif shared == "x_out over a cache":
        k = torch.empty(max(want["kv"][0][0].numel() * want["kv"][0][0].element_size(), o["x_out"].numel() * 4) // 4, dtype=torch.float32, device="cuda")
        o["x_out"] = k[:o["x_out"].numel()].view(o["x_out"].shape)
        o["kv"][0] = (k.view(want["kv"][0][0].dtype)[:want["kv"][0][0].numel()].view(want["kv"][0][0].shape), o["kv"][0][1])
    else:
        o["kept_pos"] = words(o["layer_x"][0], o["kept_pos"].numel())
    got = _run(dec, w, xd, outputs=o)
    for k in ("x_out", "kept_pos", "cu_seqlens_out"):
        assert torch.equal(got[k], want[k]), k


@pytest.mark.parametrize("batch", [1, 32, 33])
@pytest.mark.parametrize("scored", [True, False])
def test_select_with_prefix_sums_in_the_arguments(batch, scored):
    """Up to 32 samples the prefix sums travel with the launch, beyond they are uploaded; empty samples, samples that keep nothing
    and all of their rows; the caller's prefix sums of the kept rows come out either way."""
    rng = np.random.default_rng(batch)
    n = rng.integers(1, 400, batch)
    n[batch // 2] = 0 if batch > 1 else n[0]
    cu = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    keep = np.array([0 if b % 5 == 3 else m if b % 5 == 4 else (m + 1) // 2 for b, m in enumerate(n)], dtype=np.int32)
    T = int(cu[-1])
    scores = rng.permutation(T).astype(np.float32)
    rows = rng.standard_normal((T, 3)).astype(np.float32)
    prot = torch.zeros(T, dtype=torch.uint8, device="cuda")
    idx, cu_out, (got,) = fa.fastav_select_gather(torch.from_numpy(scores).cuda() if scored else None, prot, cu, keep, [torch.from_numpy(rows).cuda()])
    want = []
    for b in range(batch):
        order = np.argsort(-scores[cu[b]:cu[b + 1]], kind="stable") if scored else np.arange(n[b])
        want.append(cu[b] + np.sort(order[:keep[b]]))
    want = np.concatenate(want)
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(cu_out.cpu().numpy(), np.concatenate([[0], np.cumsum(keep)]))
    assert np.array_equal(got.cpu().numpy(), rows[want])


@pytest.mark.parametrize("n", [4097, 8193, 16385, 28673, 30000, 32768, 32769])
@pytest.mark.parametrize("scored", [True, False])
def test_selection_of_long_samples(n, scored):
    """Rows dealt to the threads in odd numbers of 16-byte pieces (4 to 36 rows a thread), up to the last sample whose keys fit LDS
    and one beyond; equal scores across the cut."""
    rng = np.random.default_rng(n)
    cu, keep = np.array([0, n, n + 700], dtype=np.int32), np.array([n * 2 // 3, 333], dtype=np.int32)
    scores = np.floor(rng.random(n + 700) * 50).astype(np.float32)
    prot = rng.random(n + 700) < 0.02
    idx, _, _ = fa.fastav_select_gather(torch.from_numpy(scores).cuda() if scored else None, torch.from_numpy(prot.astype(np.uint8)).cuda(), cu, keep)
    want = []
    for b in range(2):
        s = np.where(prot[cu[b]:cu[b + 1]], np.inf, scores[cu[b]:cu[b + 1]] if scored else 0.0)
        want.append(cu[b] + np.sort(np.argsort(-s, kind="stable")[:keep[b]]))
    assert np.array_equal(idx.cpu().numpy(), np.concatenate(want))


def test_calls_go_to_the_current_stream():
    """The stream handed to the library is torch's current one: default, side streams, nested, and back."""
    public = lambda: torch.cuda.current_stream().cuda_stream
    assert fa.binding._stream() == public()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        assert fa.binding._stream() == public() == a.cuda_stream
        with torch.cuda.stream(b):
            assert fa.binding._stream() == public() == b.cuda_stream != a.cuda_stream
        assert fa.binding._stream() == a.cuda_stream
    assert fa.binding._stream() == public()
