"""GPU parity of the lane = placement scoring pass on traces with invalid token-layers: four placements per lane (at most 64
experts) and two, at most and more than eight ids a token, bands of up to four GPUs and wider ones, with and without
secondaries; single invalid token-layers, and a layer, a family and a long run of them.  All sizes are above the numbers of
placements and GPUs of the other two passes.  All values are whole: they must equal the oracle's."""
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


@pytest.mark.parametrize("E,k,counts,G,P,R,n_rep", [
    (16, 2, [500, 3], 9, 130, 0, 0), (64, 6, [700, 900, 65], 12, 257, 2, 8), (33, 16, [300, 301], 32, 130, 3, 16),
    (40, 9, [333], 10, 257, 0, 0), (60, 4, [130] * 16, 9, 259, 1, 5), (256, 10, [300, 200], 16, 130, 2, 8),
    (100, 16, [250, 0, 260], 9, 70, 4, 16), (65, 8, [1000], 17, 66, 0, 0),
])
@pytest.mark.parametrize("dense", [False, True])
def test_invalid_token_layers(E, k, counts, G, P, R, n_rep, dense):
    print(f"lanes E={E} k={k} counts={counts[:4]} G={G} P={P} R={R}x{n_rep} dense={dense}", flush=True)
    seed, L, F = 7 * E + P, 4, len(counts)
    off = synth.fam_offsets(counts)
    N = int(off[-1])
    gen = torch.Generator().manual_seed(seed)
    tr = torch.topk(torch.rand((L, N, E), generator=gen), k, dim=2).indices.to(torch.int16)
    rng = np.random.default_rng(seed)
    if dense:
        tr[1, :, k - 1] = tr[1, :, 0]                          # a whole layer: repeated ids
        tr[2, int(off[F - 1]):, 0] = E                         # the last family: an id out of range
        tr[3, N // 4:N // 4 + min(150, N // 2), k // 2] = -1   # a run across tiles
    for l, t in ((0, 0), (0, N - 1), (3, N // 2), (0, int(rng.integers(N)))):
        tr[l, t, int(rng.integers(k))] = E + 3
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
