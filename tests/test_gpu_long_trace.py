"""GPU scoring of the longest trace that the calls accept (top-1, 2^32 - 1 tokens): token positions reach the end of 32 bits in
every trace pass.  The ids repeat with a short period, so the exact costs and loads follow from the number of tokens of every
residue."""
import numpy as np
import pytest
import torch

import paper_2606_01007_amd as tacg
from paper_2606_01007_amd import synth

pytestmark = pytest.mark.gpu

N, PERIOD, SPLIT = (1 << 32) - 1, 1013, 1001  # two families: a short one, and the rest


@pytest.fixture(scope="module")
def trace():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return {}


def _trace(cache, E):
    """int16 [1][N][1] and one period of its ids (one trace, of 8.6 GB, is held at a time)."""
    if E not in cache:
        cache.clear()
        ids = np.random.default_rng(E).integers(0, E, PERIOD).astype(np.int16)
        cache[E] = torch.as_tensor(ids).cuda().repeat(N // PERIOD + 1)[:N].view(1, N, 1), ids
    return cache[E]


def _counts(ids, E, lo, hi, hz):
    """[hz][E]: tokens of [lo, hi) by anchor position (t - lo) mod hz and id."""
    r = np.arange(PERIOD * hz, dtype=np.int64)  # t - lo = r + j PERIOD hz
    n = np.maximum(0, (hi - lo - r + PERIOD * hz - 1) // (PERIOD * hz))
    out = np.zeros((hz, E), dtype=np.int64)
    np.add.at(out, (r % hz, ids[(lo + r) % PERIOD].astype(np.int64)), n)
    return out


# lane = token; bit planes with bands of one and of three GPUs; lane = placement with four and two placements per lane, the
# last with a band wider than the packed fallbacks
@pytest.mark.parametrize("E,G,P,sizes", [(16, 9, 1, (1, 3)), (16, 8, 7, (2, 1)), (16, 8, 7, (1, 3)), (16, 9, 41, (2, 3)),
                                         (70, 9, 41, (3, 6))])
def test_longest_trace(trace, E, G, P, sizes):
    print(f"longest trace E={E} G={G} P={P} bands {sizes}", flush=True)
    tr, ids = _trace(trace, E)
    off, start = [0, SPLIT, N], [0, sizes[0]]
    rng = np.random.default_rng(P + E)
    prim = rng.integers(0, G, (P, 1, E)).astype(np.uint8)
    sec = np.full((P, 1, E, 1), synth.NONE, dtype=np.uint8)
    sec[:, 0, 3, 0] = (prim[:, 0, 3] + 1 + rng.integers(0, G - 1, P)) % G  # one replicated expert
    ref = rng.integers(0, 1000, (P, 1, G))
    out = tacg.eval_placements(tr, off, E, start, sizes, G, torch.as_tensor(prim).cuda(), torch.as_tensor(sec).cuda(),
                               torch.as_tensor(ref).cuda(), theta=None)
    torch.cuda.synchronize()
    assert int(out["err"].item()) == 0
    load = np.zeros((P, 1, G), dtype=np.int64)
    fam = np.zeros((P, 2), dtype=np.int64)
    for f in range(2):
        n = _counts(ids, E, off[f], off[f + 1], sizes[f])
        assert n.sum() == off[f + 1] - off[f]
        for p in range(P):
            for pos in range(sizes[f]):
                h = start[f] + pos
                for e in range(E):
                    cand = sorted({int(prim[p, 0, e])} | {int(g) for g in sec[p, 0, e] if g != synth.NONE})
                    g = cand[0] if len(cand) == 1 else h if h in cand else min(cand, key=lambda m: (ref[p, 0, m], m))
                    load[p, 0, g] += n[pos, e]
                    fam[p, f] += n[pos, e] if g != h else 0
    np.testing.assert_array_equal(out["cost_span"].cpu().numpy(), np.zeros(P, dtype=np.int64))
    np.testing.assert_array_equal(out["cost_home_fam"].cpu().numpy(), fam)
    np.testing.assert_array_equal(out["cost_home"].cpu().numpy(), fam.sum(1))
    np.testing.assert_array_equal(tacg.as_u32(out["load"]).cpu().numpy(), load)
