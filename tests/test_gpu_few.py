"""GPU parity of the scoring of few placements (lane = token), of the dispatch counts taken with the id validation and of the
candidate sets, at their edges: one to four placements of a workgroup, the most placements the pass takes and one
more, chunks of a family that end inside a tile, families without tokens, tokens with every slot replicated, ids out of
range and repeated at layer and family boundaries, and loads beyond 32 bits in the guard.  All values are whole: they must equal
the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_01007_amd as tacg
from paper_2606_01007_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build()


@pytest.mark.parametrize("E,k,counts,G,P,R,n_rep,bad,big", [
    (16, 2, [1, 0, 63], 9, 1, 0, 0, 0, 0),
    (33, 5, [4097, 64, 65], 12, 2, 2, 5, 3, 0),
    (64, 16, [300, 301], 32, 3, 4, 16, 2, 0),
    (20, 16, [500], 17, 4, 4, 16, 0, 1),
    (256, 8, [9000, 8191, 1], 32, 5, 3, 16, 4, 1),
    (100, 7, [777] * 6, 31, 40, 3, 16, 0, 0),
    (100, 7, [777] * 6, 31, 41, 3, 16, 0, 0),
    (70, 6, [500, 3], 12, 64, 0, 0, 1, 0),
    (70, 6, [500, 3], 12, 65, 0, 0, 1, 0),
    (70, 6, [500, 3], 8, 6, 2, 8, 1, 0),                     # at most 8 GPUs: few placements, then bit planes
    (70, 6, [500, 3], 8, 7, 2, 8, 1, 0),
    (40, 1, [300, 0, 0, 300], 10, 7, 1, 3, 2, 0),
])
def test_few_placements(E, k, counts, G, P, R, n_rep, bad, big):
    print(f"few E={E} k={k} counts={counts} G={G} P={P} R={R}x{n_rep} bad={bad}", flush=True)
    seed, L, F = 17 * E + P, 3, len(counts)
    off = synth.fam_offsets(counts)
    N = int(off[-1])
    gen = torch.Generator().manual_seed(seed)
    tr = torch.topk(torch.rand((L, N, E), generator=gen), k, dim=2).indices.to(torch.int16)
    rng = np.random.default_rng(seed)
    edges = [(l, t) for l in range(L) for t in (0, N - 1, int(off[1]) - 1)]
    for i in range(bad):
        l, t = edges[int(rng.integers(len(edges)))]
        tr[l, t, int(rng.integers(k))] = -1 if i % 2 else (int(tr[l, t, 0]) if k > 1 else E)
    prim = synth.random_placements(P, L, E, G, -(-E // G), seed)
    sec = None
    if R:
        rep = np.stack([np.sort(rng.choice(E, n_rep, replace=False)) for _ in range(L)])
        sec = synth.random_secondaries(prim, G, rep, R, seed)
        sec[rng.random(sec.shape[:3]) < 0.2] = synth.NONE
    hs, hz = synth.home_bands(F, G)
    Do, _, _ = oracle.coact(tr, off, E)
    ref = oracle.placement_load(Do, prim, G) if R else None
    if R and big:  # loads beyond 32 bits, some equal
        ref = (ref.astype(np.int64) // 7 + 1) * (1 << 38)
    want = oracle.score(tr, off, E, hs, hz, G, prim, sec, ref, (3, 20), stats=True)
    args = (tr.cuda(), off, E, hs, hz, G, torch.as_tensor(prim).cuda(), torch.as_tensor(sec).cuda() if R else None,
            torch.as_tensor(ref).cuda() if R else None)
    for name, call in (("stats", tacg.eval_trace_stats), ("plain", tacg.eval_placements)):
        out = call(*args, theta=(3, 20))
        torch.cuda.synchronize()
        assert int(out["err"].item()) == want["err"], name
        keys = ("span_fam", "cross_fam", "home_mass_fam") if name == "stats" else ("cost_home_fam",)
        for key in ("cost_home", "cost_span") + keys:
            np.testing.assert_array_equal(out[key].cpu().numpy(), want[key], err_msg=f"{name} {key}")
        np.testing.assert_array_equal(tacg.as_u32(out["load"]).cpu().numpy(), want["load"])
