"""Sampled one-workgroup rows with no small kept set and no top-k (the distance histogram, the staged
crossing bucket and the grouped draw), and candidate lists past 128 entries (the digit selections),
against the oracle: lengths at the edges of a slot group (4 slots of 512 threads), of the instantiated
sizes and with a ragged tail, misaligned rows, penalties, top-n, rows of one value (the crossing bucket
overflows its staging), masked rows, the ends of the uniforms and of top-p.  Logprobs within the parity tests' 1e-5.  Rows that
keep most of a vocabulary have values of 1e-5 of the mass and less, which the parity tests' band of 1e-5
would leave out: here ids are compared outside a band of 2e-6.  A weight 2^a with |a| <= 24 carries a
relative error of at most 24 * 2^-24 ln 2 + 2^-22 = 1.2e-6 (the argument's rounding, the exponential's), and so
does any sum of weights; the fixed-point and double sums add less than 1e-8."""
from __future__ import annotations

import numpy as np
import pytest

import workloads
from tests.parity import compare_sample, np_

pytestmark = pytest.mark.gpu

GROUP = 4 * 512  # slots
TIGHT = 2e-6


def _check(ref, out, n_top):
    """The parity comparison, then the ids again outside the tight band; the number of rows in that."""
    compare_sample(ref, out, n_top=n_top)
    sure = (ref["cdf_margin"] >= TIGHT) & (ref["topp_margin"] >= TIGHT) & ((ref["flags"] & 6) == 0)
    assert np.array_equal(np_(out[0])[sure], ref["ids"][sure])
    return int(sure.sum())


def _run(w, offset=0, n_top=0):
    import torch

    import paper_2606_01927_amd as alb
    from workloads.device import to_device

    logits, u, p = to_device(w, row_offset_bytes=offset)
    assert alb.sample_route(w.B, w.V, logits.dtype, p) == alb.ROUTE_ONE_WORKGROUP
    out = alb.sample(logits, u, p, n_top=n_top, V=w.V)
    torch.cuda.synchronize()
    return out


def _rows(dtype, V, B, kind, seed, hist):
    """A workload of V logits: flat rows (thousands kept), every filter combination without top-k."""
    w = workloads.generate(5 if dtype == "bf16" else 4, B=B, V=V, H=hist or None, variant=seed)
    rng = np.random.default_rng(seed)
    w.temperature = rng.uniform(0.8, 2.0, B).astype(np.float32)
    w.top_k = w.min_p = w.top_p = None
    if dtype == "f32":  # the generator's heavy tails would put fp32 logprobs past the tolerance by rounding alone
        w.logits = rng.normal(0, 2, (B, w.ld)).astype(np.float32)
    if kind == "nucleus":
        w.top_p = rng.choice([0.3, 0.9, 0.99, 0.99995, 0.0, 1.0], B).astype(np.float32)
    elif kind == "minp":
        w.min_p = rng.choice([1e-3, 1e-2, 0.05], B).astype(np.float32)
        w.top_p = rng.choice([1.0, 0.95], B).astype(np.float32)
    elif kind == "topk":  # lists of more than 128 entries
        w.top_k = rng.choice([130, 200, 500], B).astype(np.int32)
        w.top_p = rng.choice([0.5, 0.9, 1.0], B).astype(np.float32)
    if not hist:
        w.hist_offsets = w.hist_ids = w.repetition_penalty = w.frequency_penalty = w.presence_penalty = None
    u = rng.integers(0, 1 << 24, B)
    u[:2] = 0, (1 << 24) - 1
    w.uniforms = (u * 2.0 ** -24).astype(np.float32)
    w.n_top = 0
    return w


@pytest.mark.parametrize("kind", ["plain", "nucleus", "minp", "topk"])
@pytest.mark.parametrize("dtype,slots,extra", [
    ("bf16", 300, 5), ("f32", GROUP - 1, 0), ("f32", GROUP, 1), ("bf16", GROUP + 1, 7), ("f32", 3 * GROUP, 3),
    ("bf16", 8 * 512, 0), ("f32", 16 * 512 + 1, 2), ("bf16", 32 * 512 + 3, 1), ("f32", 38 * 512, 1)])
def test_open_and_mid_rows(dtype, slots, extra, kind, oracle_mod):
    vec, es = (8, 2) if dtype == "bf16" else (4, 4)
    V = slots * vec + extra
    big = V > 60000
    compared = 0
    for offset, hist, n_top in ((0, 0, 0), (es, 0, 5), (0, 700, 20)):
        w = _rows(dtype, V, 10 if big else 12, kind, slots % 97 + offset, hist)
        print(dtype, V, kind, "offset", offset, "hist", hist, "n_top", n_top, flush=True)
        out = _run(w, offset, n_top)
        w.n_top = n_top
        compared += _check(oracle_mod.sample(w), out, n_top)
    assert compared >= 3


@pytest.mark.parametrize("kind", ["plain", "nucleus", "minp"])
def test_ties_and_masks(kind, oracle_mod):
    V, B = 20011, 8
    w = _rows("f32", V, B, kind, 3, 0)
    x = np.array(w.logits[:, :V], copy=True)
    x[0] = 1.5                                      # one value: its bucket does not fit the staging
    x[1, :] = -np.inf
    x[1, 17] = 2.0                                  # a single finite value
    x[2, ::2] = -np.inf
    x[3] = np.float32(0.25) * np.round(x[3] * 4)    # heavy ties
    x[4, :100] = 200.0                              # distances past the last bucket
    x[5] = -0.0
    x[5, 5000:] = 0.0
    x[6] = -np.inf                                  # empty
    x[7] += 3e5                                     # a maximum past the path's range: the re-reading path
    w.logits, w.ld, w.temperature = x, V, np.ones(B, np.float32)
    for n_top in (0, 5):
        out = _run(w, 0, n_top)
        w.n_top = n_top
        _check(oracle_mod.sample(w), out, n_top)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["list", "head", "penalised"])
def test_uniform_zero_draws_the_smallest_weight(where, dtype):
    """At u = 0 the draw is the first token of positive probability, whatever its weight (2^-40 to 2^-52 of the
    largest here: the oracle's margins would leave such a row out): the first entry of a candidate list, of the
    unaligned head, and a penalised one."""
    import torch

    import paper_2606_01927_amd as alb

    V, es = 20011, 2 if dtype == "bf16" else 4
    drops = (28.5, 32.0, 36.0)
    B = len(drops)
    rng = np.random.default_rng(4)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.from_numpy(rng.normal(0, 0.5, (B, V)).astype(np.float32)).to(dt)
    first = 0 if where != "penalised" else 7  # 7: past the head
    x[:, :first] = -float("inf")
    if where == "list":  # 300 finite values, one to a thread, all of them kept by top-k
        keep = torch.arange(300) * (16 // es)
        x[:, ~torch.isin(torch.arange(V), keep)] = -float("inf")
    if where == "head":  # nothing else in the head
        x[:, 1:16] = -float("inf")
    x[:, 400] = 8.0
    x[:, first] = torch.tensor([8.0 - d for d in drops]).to(dt)
    ld = V + (16 // es - V % (16 // es))
    buf = torch.zeros(B * ld + 16, dtype=dt, device="cuda")
    off = 1 if where == "head" else 0
    rows = buf[off:off + B * ld].view(B, ld)
    rows[:, :V] = x.cuda()
    p = alb.SamplingParams(temperature=torch.ones(B, device="cuda"))
    if where == "list":
        p.top_k = torch.full((B,), 300, dtype=torch.int32, device="cuda")
    if where == "penalised":  # a penalty of 0: the token takes the path of the penalised ones
        p.hist_offsets = torch.arange(B + 1, dtype=torch.int64, device="cuda")
        p.hist_ids = torch.full((B,), first, dtype=torch.int32, device="cuda")
        p.presence_penalty = torch.zeros(B, device="cuda")
    u = torch.zeros(B, device="cuda")
    assert alb.sample_route(B, V, dt, p) == alb.ROUTE_ONE_WORKGROUP
    ids = alb.sample(rows[:, :V], u, p, V=V)[0].cpu().numpy()
    assert (ids == first).all(), ids


@pytest.mark.parametrize("dtype,V", [("f32", 20011), ("bf16", 128256)])
@pytest.mark.parametrize("allowed", [1, 3, 64, 128, 129, 511, 2000, 2500])
def test_masked_rows(allowed, dtype, V, oracle_mod):
    """Rows of a few finite values, from one to past the candidate list: threads and waves without any, more
    top-n slots than values, and the normaliser evaluated before or beside the counting (with and without
    top-p alone)."""
    B = 4
    for kind in ("plain", "nucleus", "minp", "topk", "greedy"):
        w = _rows(dtype, V, B, "plain" if kind == "greedy" else kind, allowed, 0)
        rng = np.random.default_rng(allowed)
        neg = np.float32(-np.inf) if dtype == "f32" else np.uint16(0xff80)
        x = np.array(w.logits[:, :V], copy=True)
        for i in range(B):
            at = rng.permutation(V)[:allowed] if i else np.arange(allowed)  # row 0: all in the first threads
            row = np.full(V, neg)
            row[at] = x[i, at]
            x[i] = row
        w.logits, w.ld = x, V
        if kind == "greedy":
            w.temperature = np.zeros(B, np.float32)
        for n_top in (0, 5, 32):
            out = _run(w, 0, n_top)
            w.n_top = n_top
            _check(oracle_mod.sample(w), out, n_top)
