"""MoE routing: the chosen experts, weights, offsets and pair order, exactly, at
the edges of its paths (one thread or eight lanes per token; one work-group up
to 512 tokens, chunks of 64 beyond, more chunks than groups that add them up,
and so many that they are scanned), with ties, infinities, NaN and skewed loads."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_01891_amd import aflex, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("E,k", [(8, 2), (16, 8), (17, 1), (33, 8), (63, 4), (64, 8)])
@pytest.mark.parametrize("T", [1, 33, 64, 65, 512, 513, 640, 1025, 2177])
def test_routing_exact(gpu_lib, T, E, k):
    rng = np.random.default_rng([T, E, k])
    logits = np.round(rng.standard_normal((T, E)).astype(np.float32) * 2) / 2  # many ties
    logits[rng.random((T, E)) < 0.05] = -np.inf
    logits[:, E - 1] += (np.arange(T) % 3 == 0) * np.float32(9)  # a crowded last expert
    logits[T // 2] = 0.0  # a token without any order
    logits[T // 3, :] = -1e30
    logits = torch.from_numpy(logits)
    x, w, _ = synth.custom_ffn(41, T, 64, 64, E=E)
    _, r = aflex.moe_ffn(x.to(DEV), w.to(DEV), logits.to(DEV), k, routing=True)
    ids, wts = oracle.route_topk(logits, k)
    assert torch.equal(r["topk_ids"].cpu().long(), ids)
    # expf and one division in fp32: a few units in the last place
    assert torch.allclose(r["topk_w"].cpu().double(), wts.double(), rtol=1e-5, atol=1e-7)
    flat = ids.reshape(-1).numpy()
    order = np.lexsort((np.arange(flat.size), flat))  # by expert, then token and slot
    assert np.array_equal(r["sorted_pairs"].cpu().numpy(), order)
    counts = np.bincount(flat, minlength=E)
    assert np.array_equal(r["expert_offsets"].cpu().numpy(), np.concatenate([[0], np.cumsum(counts)]))


# the last count of chunks that every work-group adds up, the first that is scanned,
# and more chunks than the scan takes at a time
@pytest.mark.parametrize("T,E,k", [(32768, 8, 2), (32769, 8, 2), (32769, 64, 8), (65601, 9, 1), (65601, 17, 3)])
def test_routing_exact_many_chunks(gpu_lib, T, E, k):
    test_routing_exact(gpu_lib, T, E, k)


def _topk_serial(row, k):
    """The largest untaken logit k times, ties to the lower id, as one pass over the
    untaken logits finds it: a NaN is kept when it is the first of them and never
    replaces another."""
    taken, out = set(), []
    for _ in range(k):
        best = None
        for e in range(len(row)):
            if e not in taken and (best is None or row[e] > row[best]):
                best = e
        taken.add(best)
        out.append(best)
    return out


@pytest.mark.parametrize("E,k", [(8, 2), (16, 8), (17, 3), (33, 8), (64, 8)])
@pytest.mark.parametrize("T", [70, 640])
def test_nan_and_infinite_logits(gpu_lib, T, E, k):
    """NaN at every place, +inf and -inf beside each other: the experts that the
    serial rule chooses, by one thread per token and by eight lanes."""
    rng = np.random.default_rng([T, E, k, 1])
    logits = np.round(rng.standard_normal((T, E)).astype(np.float32) * 2) / 2
    for v in (np.nan, np.inf, -np.inf):
        logits[rng.random((T, E)) < 0.15] = v
    for t in range(min(T, E)):  # one NaN alone, at each place
        logits[t] = np.where(np.isnan(logits[t]), 0.25, logits[t])
        logits[t, t] = np.nan
    logits[E:E + 3] = np.float32([[np.nan], [np.inf], [-np.inf]])
    x, w, _ = synth.custom_ffn(42, T, 64, 64, E=E)
    _, r = aflex.moe_ffn(x.to(DEV), w.to(DEV), torch.from_numpy(logits).to(DEV), k, routing=True)
    ids = np.array([_topk_serial(row, k) for row in logits])
    assert np.array_equal(r["topk_ids"].cpu().numpy(), ids)
    with np.errstate(invalid="ignore"):
        sel = np.take_along_axis(logits.astype(np.float64), ids, 1)
        ex = np.exp(sel - sel[:, :1])  # (the softmax is taken from the first choice)
        ref = ex / ex.sum(1, keepdims=True)
    assert np.allclose(r["topk_w"].cpu().numpy(), ref, rtol=1e-5, atol=1e-7, equal_nan=True)
    flat = ids.reshape(-1)
    assert np.array_equal(r["sorted_pairs"].cpu().numpy(), np.lexsort((np.arange(flat.size), flat)))
    counts = np.bincount(flat, minlength=E)
    assert np.array_equal(r["expert_offsets"].cpu().numpy(), np.concatenate([[0], np.cumsum(counts)]))
