"""The build of the penalty state on both sides of its vocabulary limit (393216 ids: the LDS bitmap up to
it, the sort past it), at rows of no id, of one, of the most a build takes and of more, and where the ids
fill whole bitmap words.  Counts and marks are whole numbers: compared exactly with a Python dictionary."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LIMIT = 393216
MAXS = 8192


def _rows(V, rng):
    """(prompt, output) ids of each row."""
    ends = np.array([0, V - 1, 31, 32, 33, 63, 64, V - 2], np.int64)
    ends = ends[(ends >= 0) & (ends < V)]
    run = np.arange(min(V, 500))  # whole bitmap words
    z = (rng.zipf(1.3, 5000) - 1) % V
    return [
        (np.zeros(0), np.zeros(0)),
        (np.array([V - 1]), np.zeros(0)),
        (np.zeros(0), np.array([0, 0, 0])),
        (ends, np.concatenate([ends, ends])),
        (run, run[::2]),
        (z[:3000], z[2000:]),
        (np.array([V, -1, 5 % V, 2**31 - 1]), np.array([-7, V + 3, 5 % V])),      # ids outside the vocabulary
        (rng.integers(0, V, MAXS - 100), rng.integers(0, V, 100)),                 # exactly the most
        (rng.integers(0, V, MAXS - 100), rng.integers(0, V, 300)),                 # 200 left out
    ]


@pytest.mark.parametrize("V", [1, 31, 33, 128256, LIMIT - 1, LIMIT, LIMIT + 1, 600000])
@pytest.mark.parametrize("cap", [8192, 900])
def test_state_init_matches_the_definition(V, cap):
    import torch

    import paper_2606_01927_amd as alb

    rng = np.random.default_rng(V + cap)
    rows = _rows(V, rng)

    def csr(which):
        offs = np.cumsum([0] + [len(r[which]) for r in rows]).astype(np.int64)
        ids = np.concatenate([np.asarray(r[which], np.int32) for r in rows]).astype(np.int32)
        return torch.from_numpy(offs).cuda(), torch.from_numpy(ids).cuda()

    st = alb.PenaltyState(len(rows), cap)
    st.init(V, *csr(0), *csr(1))
    ids, counts = st.ids.cpu().numpy(), st.counts.cpu().numpy().view(np.uint32)
    lens, flags = st.len.cpu().numpy(), st.flags.cpu().numpy()
    for b, (prompt, output) in enumerate(rows):
        occ = [(int(i), True) for i in prompt] + [(int(i), False) for i in output]
        want_flags = alb.FLAG_LIMIT if len(occ) > MAXS else 0
        want = {}
        for i, from_prompt in occ[:MAXS]:
            if not 0 <= i < V:
                want_flags |= alb.FLAG_BAD_INPUT
                continue
            c = want.get(i, 0)
            want[i] = c | 0x80000000 if from_prompt else c + 1
        entries = sorted(want.items())
        if len(entries) > cap:
            want_flags |= alb.FLAG_LIMIT
            entries = entries[:cap]
        assert lens[b] == len(entries), (V, cap, b)
        assert flags[b] == want_flags, (V, cap, b)
        assert [int(v) for v in ids[b, :lens[b]]] == [i for i, _ in entries], (V, cap, b)
        assert [int(v) for v in counts[b, :lens[b]]] == [c for _, c in entries], (V, cap, b)
