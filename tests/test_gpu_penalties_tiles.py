"""albireo_apply_penalties at the edges of its tiles (8192 elements from the output's first 16-byte
boundary) and of its 16-byte groups: short rows, rows of every length modulo four, strided and misaligned
inputs, an fp32 input in place.  The penalties are defined fp32 operation by operation, so the results are
compared bit for bit with the same operations in numpy fp32."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TILE = 8192


def _reference(x, rep, freq, pres, out_counts, in_prompt):
    """fp32 penalties of one row: repetition over output and prompt ids, frequency and presence over
    the output counts."""
    x = x.astype(np.float32).copy()
    c = out_counts.astype(np.float32)
    seen = (out_counts > 0) | in_prompt
    with np.errstate(invalid="ignore"):
        x = np.where(seen, np.where(x > 0, x / rep, x * rep), x)
        return np.where(out_counts > 0, (x - freq * c) - pres, x).astype(np.float32)


@pytest.mark.parametrize("dtype", ["bf16", "f32", "f32_in_place"])
@pytest.mark.parametrize("V", [1, 3, 4, 7, TILE - 1, TILE, TILE + 1, TILE + 3, 3 * TILE + 2])
def test_tile_edges_bit_exact(V, dtype):
    import torch

    import paper_2606_01927_amd as alb

    B, pad, skip = 5, 3, 1  # rows of stride V + pad from an address one element past 16 bytes
    rng = np.random.default_rng(V)
    x = rng.normal(0, 3, size=(B, V)).astype(np.float32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    if dtype == "f32_in_place":
        pad = skip = 0
    buf = torch.zeros(skip + B * (V + pad), dtype=dt, device="cuda")
    logits = buf[skip:].view(B, V + pad)[:, :V] if pad == 0 else buf[skip:].as_strided((B, V), (V + pad, 1))
    logits.copy_(torch.from_numpy(x))
    xs = logits.float().cpu().numpy()
    # histories that name the row's ends, the tiles' ends, repeats and ids outside the vocabulary
    edges = [i for i in (0, 1, 2, V - 2, V - 1, TILE - 1, TILE, TILE + 1, 2 * TILE, 2 * TILE + 3) if 0 <= i < V]
    hist = [np.concatenate([edges, rng.integers(0, V, 300), [V, -1, 2**31 - 1], edges]) if b else [] for b in range(B)]
    prompt = [rng.integers(0, V, 40 * b) for b in range(B)]
    out_counts = np.stack([np.bincount([i for i in h if 0 <= i < V], minlength=V) for h in hist])
    in_prompt = np.stack([np.bincount(q.astype(np.int64), minlength=V) > 0 for q in prompt])

    def csr(rows):
        offs = np.cumsum([0] + [len(r) for r in rows]).astype(np.int64)
        ids = np.concatenate([np.asarray(r, np.int32) for r in rows]).astype(np.int32)
        return torch.from_numpy(offs).cuda(), torch.from_numpy(ids).cuda()

    pen = [rng.uniform(lo, hi, size=B).astype(np.float32) for lo, hi in ((1.05, 1.5), (0.0, 0.5), (-0.2, 0.4))]
    p = alb.SamplingParams()
    p.repetition_penalty, p.frequency_penalty, p.presence_penalty = [torch.from_numpy(a).cuda() for a in pen]
    p.hist_offsets, p.hist_ids = csr(hist)
    p.prompt_offsets, p.prompt_ids = csr(prompt)
    out = logits if dtype == "f32_in_place" else torch.full((B, V), 7.0, device="cuda")
    got = alb.apply_penalties(logits, p, V=V, out=out).cpu().numpy()
    for b in range(B):
        ref = _reference(xs[b], pen[0][b], pen[1][b], pen[2][b], out_counts[b], in_prompt[b])
        assert np.array_equal(got[b].view(np.uint32), ref.view(np.uint32)), (V, dtype, b)
    # without penalties the rows are copied
    plain = alb.apply_penalties(logits if dtype != "f32_in_place" else got_copy(got), alb.SamplingParams(), V=V)
    want = xs if dtype != "f32_in_place" else got
    assert np.array_equal(plain.cpu().numpy().view(np.uint32), want.view(np.uint32))


def got_copy(a):
    import torch

    return torch.from_numpy(a.copy()).cuda()
