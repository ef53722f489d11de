"""GPU parity of the bit-plane scoring pass (at most 8 GPUs) at the sizes where it can go wrong: group and
block edges of the placements (32 per group, 512 per workgroup, padded and split remainders), the plane counts
(G up to 4 and up to 8), the narrowest and widest token descriptors, the largest table that fits the LDS and
the first that does not, classes shorter than a tile or empty, and tokens with every slot replicated.
Costs and loads are whole numbers: they must equal the oracle's."""
import sys

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


@pytest.mark.parametrize("E,k,counts,G,P,R,n_rep,bad", [
    (8, 2, [640, 1, 0, 65], 4, 7, 0, 0, 0),        # the fewest placements of this pass
    (9, 1, [130], 1, 31, 0, 0, 0),
    (16, 8, [63, 200], 4, 32, 3, 16, 0),
    (24, 5, [1, 2, 3, 700], 8, 33, 4, 16, 3),
    (33, 7, [500] * 9, 5, 97, 2, 6, 0),          # more families than GPUs
    (64, 6, [900, 17], 7, 352, 2, 16, 5),        # 11 groups: blocks of 8, 2 and 1
    (60, 4, [3000, 2999], 6, 416, 2, 4, 0),      # 13 groups: one padded block
    (100, 9, [700, 800], 8, 512, 3, 12, 2),      # two words of replica rows
    (128, 8, [1500, 10, 1490], 8, 545, 2, 8, 0),  # a full block, then one group and one placement
    (40, 16, [257, 300], 8, 64, 4, 16, 0),
    (256, 8, [600, 600], 8, 40, 2, 16, 1),       # the largest table
    (256, 16, [300, 200], 3, 40, 2, 16, 1),
    (248, 8, [300, 200], 8, 40, 2, 16, 0),       # 768 threads and, with one expert more, 512
    (249, 8, [300, 200], 8, 40, 2, 16, 1),
    (252, 10, [300, 200], 8, 40, 2, 16, 0),      # the largest tables above top-8 ...
    (244, 11, [300, 200], 5, 40, 2, 16, 0),
    (236, 16, [300, 200], 8, 40, 2, 16, 1),
    (253, 9, [300, 200], 8, 40, 2, 16, 0),       # ... and the first too large for the LDS: the general pass
    (245, 12, [300, 200], 5, 40, 2, 16, 1),
    (237, 13, [300, 200], 8, 40, 2, 16, 0),
    (256, 12, [300, 200], 8, 40, 2, 16, 0),
    (12, 3, [40000, 30000], 2, 700, 1, 3, 0),    # long runs
])
def test_planes_parity(E, k, counts, G, P, R, n_rep, bad):
    print(f"planes E={E} k={k} counts={counts} G={G} P={P} R={R}x{n_rep}", flush=True)
    sys.stdout.flush()
    seed, L, F = 31 * E + k, 2, len(counts)
    off = synth.fam_offsets(counts)
    N = int(off[-1])
    gen = torch.Generator().manual_seed(seed)
    tr = torch.topk(torch.rand((L, N, E), generator=gen), k, dim=2).indices.to(torch.int16)
    rng = np.random.default_rng(seed)
    for i in range(bad):  # invalid token-layers: an id out of range or a repeated one
        l, t = int(rng.integers(L)), int(rng.integers(N))
        tr[l, t, int(rng.integers(k))] = E if i % 2 else int(tr[l, t, 0])
    prim = synth.random_placements(P, L, E, G, -(-E // G), seed)
    sec = None
    if R:
        rep = np.stack([np.sort(rng.choice(E, n_rep, replace=False)) for _ in range(L)])
        sec = synth.random_secondaries(prim, G, rep, min(R, G - 1), seed)
        sec[rng.random(sec.shape[:3]) < 0.3] = synth.NONE  # some placements keep a single candidate
    hs, hz = synth.home_bands(F, G)
    Do, _, err = oracle.coact(tr, off, E)
    ref = oracle.placement_load(Do, prim, G) if R else None
    want = oracle.score(tr, off, E, hs, hz, G, prim, sec, ref, (3, 20))
    out = tacg.eval_placements(tr.cuda(), off, E, hs, hz, G, torch.as_tensor(prim).cuda(),
                               torch.as_tensor(sec).cuda() if R else None,
                               torch.as_tensor(ref).cuda() if R else None, theta=(3, 20))
    torch.cuda.synchronize()
    assert int(out["err"].item()) == want["err"]
    np.testing.assert_array_equal(out["cost_home"].cpu().numpy(), want["cost_home"])
    np.testing.assert_array_equal(out["cost_span"].cpu().numpy(), want["cost_span"])
    np.testing.assert_array_equal(tacg.as_u32(out["load"]).cpu().numpy(), want["load"])
    np.testing.assert_array_equal(out["cost_home_fam"].cpu().numpy(), want["cost_home_fam"])
