"""GPU parity of the decayed-load scoring at the GPU counts where the number of loads held per lane changes (8, 16, 24, 32) and at
expert counts around the eight whose tables are read together.  Costs, loads and the final float64 loads (one
rounding a step in trace order) must equal the oracle's."""
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


@pytest.mark.parametrize("E,k,G,R,P", [(8, 2, 8, 2, 3), (9, 3, 9, 0, 65), (33, 9, 16, 3, 2), (40, 8, 17, 4, 5), (63, 5, 24, 1, 7),
                                       (65, 12, 25, 3, 64), (255, 8, 32, 4, 2), (256, 4, 11, 2, 66)])
def test_online_gpu_counts(E, k, G, R, P):
    print(f"online E={E} k={k} G={G} R={R} P={P}", flush=True)
    counts, L = [150, 0, 211], 2
    off = synth.fam_offsets(counts)
    gen = torch.Generator().manual_seed(E + G)
    tr = torch.topk(torch.rand((L, int(off[-1]), E), generator=gen), k, dim=2).indices.to(torch.int16)
    prim = synth.random_placements(P, L, E, G, -(-E // G), E)
    rng = np.random.default_rng(E)
    sec = None
    if R:
        rep = np.stack([np.sort(rng.choice(E, min(16, E // 2), replace=False)) for _ in range(L)])
        sec = synth.random_secondaries(prim, G, rep, R, E)
        sec[rng.random(sec.shape[:3]) < 0.2] = synth.NONE
    hs, hz = synth.home_bands(len(counts), G)
    want = oracle.score_online(tr, off, E, hs, hz, G, prim, sec, 0.995, (3, 20))
    out = tacg.eval_online(tr.cuda(), off, E, hs, hz, G, torch.as_tensor(prim).cuda(),
                           torch.as_tensor(sec).cuda() if R else None, rho=0.995, theta=(3, 20))
    torch.cuda.synchronize()
    assert int(out["err"].item()) == want["err"] == 0
    for key in ("cost_home", "cost_span", "cost_home_fam", "state"):
        np.testing.assert_array_equal(out[key].cpu().numpy(), want[key], err_msg=key)
    np.testing.assert_array_equal(tacg.as_u32(out["load"]).cpu().numpy(), want["load"])
