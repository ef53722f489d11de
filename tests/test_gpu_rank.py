"""GPU parity of the grouping objective and the snapshot loads at the edges of their work split: one, two and four
sets of 64 placements per workgroup, partial sets, dword-aligned and unaligned placement rows, one GPU holding
every expert and GPUs holding one, more placements than a workgroup's run, and the numbers of placements and layers on
both sides of the change between the objective's two kernels (1152 to 3456 by the experts per GPU), and of the runs of placements
that the loads take (1 up to 1152 in all, then 4, 8 and up to 64 a workgroup).
Loads are whole numbers.  The objective is a float64 sum of n = E^2 non-negative terms at most: two orders of it
differ by at most 2 n 2^-53 relative."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_01007_amd as tacg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build()


@pytest.mark.parametrize("E,G,P,L,shift", [
    (1, 1, 1, 1, 0), (3, 2, 63, 2, 0), (4, 4, 64, 3, 0), (16, 1, 65, 2, 0), (16, 16, 130, 3, 1), (20, 3, 257, 100, 0),
    (6, 5, 257, 100, 0), (64, 8, 200, 96, 0), (60, 7, 129, 2, 3), (255, 32, 70, 2, 0), (256, 32, 300, 3, 0), (256, 1, 5, 1, 2),
    (256, 32, 1536, 2, 0), (256, 32, 1537, 2, 0), (252, 8, 2048, 1, 0), (252, 8, 2049, 1, 1), (255, 2, 768, 2, 0),
    (256, 2, 769, 2, 0), (4, 4, 1025, 2, 0),
    (3, 1, 2050, 1, 0), (33, 32, 500, 60, 0), (72, 9, 500, 60, 3), (40, 8, 300, 17, 0), (252, 4, 70, 12, 0), (16, 4, 1024, 40, 0),
    (255, 2, 576, 2, 0), (255, 2, 577, 2, 0), (80, 2, 704, 2, 0), (80, 2, 705, 2, 0), (252, 8, 1857, 1, 1), (100, 9, 2561, 1, 0),
    (256, 32, 1728, 2, 0), (256, 32, 1729, 2, 0), (33, 16, 2433, 1, 0), (36, 4, 2241, 1, 0),
])
def test_objective_and_loads(E, G, P, L, shift):
    print(f"rank E={E} G={G} P={P} L={L} shift={shift}", flush=True)
    rng = np.random.default_rng(E * 1000 + P)
    a = rng.random((L, E, E)).astype(np.float32)
    prim = rng.integers(0, G, (P, L, E)).astype(np.uint8)      # uneven groups, some empty
    D = rng.integers(0, 1 << 31, (5, L, E)).astype(np.int32)
    buf = torch.zeros(P * L * E + shift, dtype=torch.uint8, device="cuda")
    prim_t = buf[shift:].view(P, L, E)
    prim_t.copy_(torch.as_tensor(prim))
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    obj = tacg.group_objective(torch.as_tensor(a).cuda(), prim_t, G, err=err).cpu().numpy()
    load = tacg.placement_load(torch.as_tensor(D).cuda(), prim_t, G, err=err).cpu().numpy()
    assert int(err.item()) == 0
    np.testing.assert_array_equal(load, oracle.placement_load(D.view(np.uint32), prim, G))
    np.testing.assert_allclose(obj, oracle.grouping_objective(a, prim, G), rtol=2 * E * E * 2.0 ** -53, atol=0)
