"""GPU parity of scoring and statistics of short traces, where the work split and the choice of the passes change: many short,
empty or one-token families, fewer token-layers than a wave, and the sizes on both sides of the rules (named at the rows).
All values are whole: they must equal the oracle's."""
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


@pytest.mark.parametrize("E,k,L,counts,G,P,R,n_rep", [
    # validation and dispatch counts: several families per workgroup, workgroups that end inside one, a single token
    (128, 16, 1, [30] * 64, 9, 65, 0, 0),
    (60, 2, 4, [9] * 63 + [0], 16, 64, 3, 5),
    (8, 2, 4, [0, 1] * 32, 8, 100, 0, 0),
    (256, 1, 3, [700, 0, 1, 2000], 8, 10, 2, 4),
    (16, 6, 2, [0, 1, 0], 6, 3, 0, 0),
    (40, 3, 58, [5, 70], 9, 5, 1, 3),
    # one preparation launch up to 4096 table entries a layer, with secondaries up to 64 placements
    (64, 4, 2, [200], 9, 64, 2, 6),
    (64, 4, 2, [200], 9, 65, 2, 6),
    (32, 3, 2, [100, 50], 12, 65, 1, 4),
    (32, 3, 3, [100, 50], 12, 128, 0, 0),
    (32, 3, 3, [100, 50], 12, 129, 0, 0),
    # lane = token from 25 placements on: token-layers enough, or few workgroups (2048; 4096 with secondaries)
    (48, 2, 4, [40] * 64, 10, 24, 0, 0),
    (48, 2, 4, [40] * 64, 10, 32, 0, 0),
    (48, 2, 5, [40] * 64, 10, 28, 0, 0),
    (20, 3, 6, [30] * 64, 12, 40, 2, 4),
    (20, 3, 7, [30] * 64, 12, 40, 2, 4),
    (33, 16, 9, [256] * 8, 11, 64, 0, 0),
    (33, 16, 9, [255] * 16, 11, 64, 0, 0),
    # bit planes or not: few experts, a short choice, no replicas, 128 tokens a family
    (16, 2, 2, [128] * 4, 6, 520, 0, 0),
    (16, 2, 2, [129, 128, 128], 6, 520, 0, 0),
    (32, 1, 2, [1] * 64, 8, 97, 0, 0),
    (33, 1, 2, [1] * 64, 8, 97, 0, 0),
    (16, 2, 2, [100] * 4, 6, 70, 1, 2),
    # the last block of placements in one piece, padded: 16 layers and 768 tiles of work; split below that
    (40, 5, 16, [9] * 48, 8, 65, 2, 5),
    (40, 5, 15, [9] * 48, 8, 65, 2, 5),
    (40, 5, 16, [9] * 47, 8, 160, 2, 5),
    (20, 3, 20, [70] * 40, 3, 340, 1, 4),
    (24, 4, 16, [40] * 50, 5, 577, 0, 0),
    (24, 4, 16, [500] * 3, 5, 300, 3, 6),
])
def test_short(E, k, L, counts, G, P, R, n_rep):
    print(f"short E={E} k={k} L={L} F={len(counts)} N={sum(counts)} G={G} P={P} R={R}x{n_rep}", flush=True)
    seed, F = 13 * E + P, len(counts)
    off = synth.fam_offsets(counts)
    gen = torch.Generator().manual_seed(seed)
    tr = torch.topk(torch.rand((L, int(off[-1]), E), generator=gen), k, dim=2).indices.to(torch.int16)
    rng = np.random.default_rng(seed)
    prim = synth.random_placements(P, L, E, G, -(-E // G), seed)
    sec = ref = None
    if R:
        rep = np.stack([np.sort(rng.choice(E, n_rep, replace=False)) for _ in range(L)])
        sec = synth.random_secondaries(prim, G, rep, R, seed)
        sec[rng.random(sec.shape[:3]) < 0.2] = synth.NONE
        Do, _, _ = oracle.coact(tr, off, E)
        ref = oracle.placement_load(Do, prim, G)
    hs, hz = synth.home_bands(F, G)
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
