"""albireo_topk_topp through the chunk-parallel kernels: row lengths at the edges of a chunk (19456 values),
of a 16-byte slot and of one register chunk, strided rows at any 4-byte boundary, every combination of the
filters, and the rows that leave the histogram's cut to a selection over memory (one value many times, kept
sets past the staging), and maxima of any magnitude.  Against plain torch in 64 bits on the fp32 processed logits:
threshold, kept count and flags exactly (top-p is moved to the middle of the interval its group falls into),
probabilities and log-normaliser within 1e-5: a weight 2^a, |a| <= 24, carries a relative error of at most
24 * 2^-24 ln 2 + 2^-22 = 1.2e-6, and so does a sum of them.  Where a group's interval is narrower than that error
(half of it below 2e-6) rounding may decide the group: the cut then has to be one that some top-p within
2e-6 of the row's gives."""
from __future__ import annotations

import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CHUNK = 4864 * 4
TIGHT = 2e-6
ONE_WG = 38 * 512 * 4 + 3  # the longest row of one register chunk


def _reference(x, T, k, p, mp):
    """(kept mask, processed logits, p moved inside its interval) of one row."""
    V = x.size
    r = np.float32(1.0 / np.float64(T)) if T >= 1e-5 else np.float32(1)
    z = (x * r).astype(np.float32)
    m = z.max()
    if T < 1e-5:
        keep = np.zeros(V, bool)
        keep[int(np.argmax(z))] = True
        return keep, z, p
    zs = np.sort(z)[::-1]
    fin = zs[zs > -np.inf]
    tau = -np.inf
    if 0 < k < V and k <= fin.size:
        tau = zs[k - 1]
    if mp > 0:
        tau = max(tau, np.float32(m + np.float32(math.log(min(np.float64(np.float32(mp)), 1.0)))))
    if p < 1:
        if p <= 0:
            tau = m
        else:
            s2 = fin[fin >= tau].astype(np.float64)
            vals, cnt = np.unique(s2, return_counts=True)
            vals, cnt = vals[::-1], cnt[::-1]
            cum = np.cumsum(cnt * np.exp(vals - np.float64(m)))
            g = min(int(np.searchsorted(cum, p * cum[-1])), vals.size - 1)
            mid = np.float32(((cum[g - 1] if g else 0.0) + cum[g]) / 2 / cum[-1])
            p = min(mid, np.float32(1 - 2.0 ** -24)) if vals.size > 1 else p
            tau = max(tau, np.float32(vals[g]))
    return (z >= tau) & (z > -np.inf), z, p


def _floor(x, T, k, mp):
    """The cut of top-k and min-p alone."""
    keep, z, _ = _reference(x, T, k, 1.0, mp)
    return z[keep].min()


def _run(x, T, k, p, mp, ld=None, offset=0):
    import torch

    import paper_2606_01927_amd as alb

    B, V = x.shape
    ld = ld or V
    buf = torch.full((B * ld + 8,), float("nan"), device="cuda")
    rows = buf[offset:offset + B * ld].view(B, ld)
    rows[:, :V] = torch.from_numpy(x).cuda()
    ref = []
    p = p.copy()
    for i in range(B):
        row = x[i]
        if np.isnan(row).any() or (row == np.inf).any() or not (row > -np.inf).any():
            ref.append(None)
            continue
        keep, z, p[i] = _reference(row, T[i], int(k[i]), p[i], mp[i])
        ref.append((keep, z))
    prm = alb.SamplingParams(temperature=torch.from_numpy(T).cuda(), top_p=torch.from_numpy(p).cuda())
    if (k > 0).any():
        prm.top_k = torch.from_numpy(k).cuda()
    if (mp > 0).any():
        prm.min_p = torch.from_numpy(mp).cuda()
    ws = alb.Workspace(buf.device)
    for _ in range(2):  # the second call finds the workspace as the first left it
        pr, thr, kept, ln, fl = alb.topk_topp(rows[:, :V], prm, V=V, workspace=ws)
        torch.cuda.synchronize()
        assert int(ws.buf.count_nonzero()) == 0
        pr_, thr, kept, ln, fl = (t.cpu().numpy() for t in (pr, thr, kept, ln, fl))
        for i in range(B):
            if ref[i] is None:
                assert thr[i] == -np.inf and kept[i] == 0 and not pr_[i].any(), i
                continue
            keep, z = ref[i]
            if 0 < p[i] < 1 and T[i] >= 1e-5 and kept[i] != keep.sum():
                w = np.where((z > -np.inf) & (z >= _floor(x[i], T[i], int(k[i]), mp[i])), np.exp(z.astype(np.float64) - z.max()), 0.0)
                at, above = w[z >= thr[i]].sum() / w.sum(), w[z > thr[i]].sum() / w.sum()
                assert at - above < 2 * TIGHT and above - TIGHT <= p[i] <= at + TIGHT, (i, V, above, p[i], at)
                keep = (w > 0) & (z >= thr[i])
            case = (i, V, float(T[i]), int(k[i]), float(p[i]), float(mp[i]))
            assert kept[i] == keep.sum(), (case, kept[i], keep.sum())
            assert thr[i] == z[keep].min(), case
            assert not pr_[i][~keep].any(), case
            m = np.float64(z.max())
            w = np.where(keep, np.exp(z.astype(np.float64) - m), 0.0)
            if T[i] < 1e-5:
                w = keep.astype(np.float64)
            assert abs(ln[i] - (m + math.log(w.sum()))) <= 1e-5 * max(1.0, abs(m)), case
            assert np.abs(pr_[i] - w / w.sum()).max() <= 1e-5, case
    return fl


COMBOS = [  # temperature, k, p, min-p
    (1.0, 40, 1.0, 0.0), (0.7, 0, 0.9, 0.0), (0.8, 50, 0.8, 0.0), (1.0, 0, 1.0, 0.02), (1.0, 0, 0.95, 0.05),
    (1.3, 0, 1.0, 0.0), (0.0, 5, 0.5, 0.1), (1.0, 30, 0.0, 0.0), (0.9, 700, 0.9, 0.0), (1.0, 20, 0.9, 0.1),
    (0.5, 0, 0.999, 0.0), (1.0, 9000, 0.99, 0.0), (1.0, 15000, 1.0, 0.0), (2.0, 0, 0.99, 0.001),
    (1.0, 2 ** 30, 0.5, 0.0)]


def _params(combos):
    T, k, p, mp = zip(*combos)
    return (np.array(T, np.float32), np.array(k, np.int32), np.array(p, np.float32), np.array(mp, np.float32))


@pytest.mark.parametrize("V,ld,offset", [
    (ONE_WG + 1, None, 0), (4 * CHUNK, None, 0), (4 * CHUNK + 1, None, 1), (5 * CHUNK - 1, 5 * CHUNK + 3, 2),
    (128256, None, 0), (100003, 100007, 3), (200000, None, 0)])
def test_filter_combinations(V, ld, offset):
    rng = np.random.default_rng(V)
    B = len(COMBOS)
    x = (rng.normal(0, 2.5, (B, V)) - 1.1 * np.log(rng.permutation(V) + 1)).astype(np.float32)
    x[::3] = rng.normal(0, 2, x[::3].shape)
    x[1, rng.random(V) < 0.3] = -np.inf
    _run(x, *_params(COMBOS), ld=ld, offset=offset)


@pytest.mark.parametrize("V", [4, 5, 7, 2047, CHUNK - 1, CHUNK, CHUNK + 1, 3 * CHUNK + 2, ONE_WG])
def test_top_p_alone_short_rows(V):
    rng = np.random.default_rng(V)
    combos = [(t, 0, p, 0.0) for t in (0.0, 0.6, 1.0) for p in (0.0, 0.3, 0.9, 0.999, 1.0)]
    x = rng.normal(0, 2, (len(combos), V)).astype(np.float32)
    _run(x, *_params(combos))


def test_rows_selected_over_memory():
    """Kept sets and buckets past the staging, one value throughout, large maxima, far-away chunks."""
    V = 90000
    rng = np.random.default_rng(5)
    rows, combos = [], []
    for combo in [(1.0, 0, 0.9, 0.0), (1.0, 100, 0.9, 0.0), (1.0, 5000, 0.7, 0.0), (1.0, 0, 0.8, 0.01), (1.0, 7, 1.0, 0.0)]:
        ties = np.round(rng.normal(0, 1, V) * 4) / 4
        rows += [np.full(V, 1.5), ties, rng.normal(0, 0.3, V), rng.normal(0, 1, V) * 3e5,
                 np.concatenate([rng.normal(0, 2, V // 2), rng.normal(-500, 2, V - V // 2)]),
                 np.concatenate([np.full(V // 2, -np.inf), rng.normal(0, 2, V - V // 2)]),
                 np.where(np.arange(V) < 50, rng.normal(0, 1, V), -np.inf)]
        combos += [combo] * 7
    _run(np.stack(rows).astype(np.float32), *_params(combos))


def test_empty_and_bad_rows():
    import paper_2606_01927_amd as alb

    V = 80001
    rng = np.random.default_rng(6)
    x = rng.normal(0, 2, (6, V)).astype(np.float32)
    x[0] = -np.inf
    x[1, 70000] = np.nan
    x[2, 3] = np.inf
    x[3, 1:] = -np.inf
    x[4, :-1] = -np.inf
    combos = [(1.0, 10, 0.9, 0.0)] * 6
    fl = _run(x, *_params(combos))
    empty, bad = alb.FLAG_EMPTY, alb.FLAG_BAD_INPUT
    assert fl[0] & empty and fl[1] & bad and fl[2] & bad and not (fl[3:] & (empty | bad)).any()


@pytest.mark.parametrize("V", [20003, 90000])
def test_maxima_of_any_magnitude(V):
    """Maxima from 2^18 to 1e30 in both signs, the values below them spaced by the type's own steps: weights and
    bucket edges hold at any magnitude.  V on both sides of one register chunk (top-p alone in the first)."""
    rng = np.random.default_rng(11)
    rows, combos = [], []
    for combo in [(1.0, 0, 0.5, 0.0), (1.0, 0, 0.9, 0.0), (1.0, 100, 0.8, 0.0), (1.0, 30, 1.0, 0.0), (1.0, 0, 0.7, 1e-4)]:
        if V < ONE_WG and (combo[1] or combo[3]):
            continue
        for m in (2.6e5, 3e5, 6e5, 1.1e6, 1e7, -1e7, 2.5e7, 4e7, 1e8, -1e8, 1e30, -1e30):
            x = (m - abs(m) * rng.uniform(0.01, 1, V)).astype(np.float32)
            at, top = rng.permutation(V), np.float32(m)
            x[at[0]] = top
            step, used = float(top) - float(np.nextafter(top, np.float32(-np.inf))), 1
            for k in range(1, 200):  # k steps below the maximum: the more values, the less each weighs
                n = int(min(math.ceil(math.exp(min(k * step, 50.0)) / 2), 1500))
                if used + n > 6000 or n == 1500:
                    break
                x[at[used:used + n]] = np.float32(float(top) - k * step)
                used += n
            rows.append(x)
            combos.append(combo)
    for scale in (100.0, 400.0):  # ordinary logits at a temperature next to greedy
        rows.append(rng.normal(0, scale, V).astype(np.float32))
        combos.append((2e-5, 0, 0.9, 0.0))
    _run(np.stack(rows).astype(np.float32), *_params(combos))


def test_cuts_in_the_last_bucket():
    """Two filters whose count or min-p cut lies 32 and more below the maximum, or is never reached: fewer finite
    values than k, steep rows, tiny min-p.  The staged list then ends above the last bucket, and holds at most
    4096 values or leaves the row to the selection over memory."""
    rng = np.random.default_rng(12)
    rows, combos = [], []
    for V_fin in (1, 20, 39, 1000, 4096, 4097, 20000):
        x = np.full(90000, -np.inf)
        x[rng.permutation(90000)[:V_fin]] = rng.normal(0, 2, V_fin)
        for k, p in ((40, 0.9), (V_fin + 1, 0.999), (30000, 1 - 2.0 ** -24)):
            rows.append(x)
            combos.append((1.0, k, p, 0.0))
    for spread in (31.9, 33.0, 200.0, 3e5):
        for combo in ((1.0, 40, 0.9, 0.0), (1.0, 9000, 0.99, 0.0), (1.0, 0, 0.9, 1e-20), (1.0, 80000, 0.5, 1e-30)):
            rows.append(-rng.random(90000) ** 0.5 * spread)
            combos.append(combo)
    _run(np.stack(rows).astype(np.float32), *_params(combos))


@pytest.mark.parametrize("V", [2048, 2049])
def test_top_p_alone_at_the_candidate_list(V):
    """The longest row that the one-workgroup kernel keeps (its list holds 2048), and the next."""
    rng = np.random.default_rng(V)
    combos = [(t, 0, p, 0.0) for t in (0.0, 0.6, 1.0) for p in (0.0, 0.3, 0.9, 0.999, 1.0)]
    x = rng.normal(0, 2, (len(combos), V)).astype(np.float32)
    x[::2, 7] += 12.0
    _run(x, *_params(combos))


@pytest.mark.parametrize("V", [30000, 90000])
def test_smaller_workspace(V):
    """A workspace below the chunk-parallel kernels' need but enough for the register-resident ones (none at all
    where a row takes one workgroup): the same distribution from those."""
    import ctypes

    import torch

    import paper_2606_01927_amd as alb

    B = 6
    rng = np.random.default_rng(V)
    x = torch.from_numpy(rng.normal(0, 2.5, (B, V)).astype(np.float32)).cuda()
    T, _, p, _ = _params([(t, 0, p, 0.0) for t, p in ((1.0, 0.9), (0.7, 0.5), (0.5, 0.99), (1.0, 1.0), (0.0, 0.5), (2.0, 0.3))])
    # top-p in the middle of the interval its group falls into
    p = np.array([_reference(x[i].cpu().numpy(), T[i], 0, p[i], 0.0)[2] for i in range(B)], np.float32)
    rows = alb.SamplingParams(temperature=torch.from_numpy(T).cuda(), top_p=torch.from_numpy(p).cuda())
    prm = alb._params(rows, x.device)
    full = int(alb._lib.albireo_workspace_size(B, V, alb.F32, 0))
    buf = torch.zeros(full + 256, dtype=torch.uint8, device="cuda")
    base = buf.data_ptr() + (-buf.data_ptr()) % 256
    got = []
    for ws, n in ((base, full), (base, full * 3 // 4) if V > ONE_WG else (None, 0)):
        o = [torch.empty((B, V), device="cuda")] + [torch.empty(B, dtype=d, device="cuda") for d in
                                                    (torch.float32, torch.int32, torch.float32, torch.int32)]
        rc = alb._lib.albireo_topk_topp(x.data_ptr(), B, V, V, ctypes.byref(prm), *[t.data_ptr() for t in o], ws, n, None)
        assert rc == 0
        torch.cuda.synchronize()
        assert int(buf.count_nonzero()) == 0
        got.append([t.cpu().numpy() for t in o])
    (pr, thr, kept, ln, fl), (pr2, thr2, kept2, ln2, fl2) = got
    assert np.array_equal(thr, thr2) and np.array_equal(kept, kept2) and np.array_equal(fl, fl2)
    assert np.abs(pr - pr2).max() <= 1e-5 and np.abs(ln - ln2).max() <= 1e-5
