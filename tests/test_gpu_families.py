"""GPU parity of the passes over the family counts (reweighting, GESR scores, distances, top pairs) where their
work split changes: one wave per eight families (1 to 64 families; up to 2 and 4 apart), 1 to 16 rows per workgroup, 64 columns per lane step,
rows paired from both ends of the triangle (odd and even E), and families without tokens.
float64 results: sums of at most E F terms in another order, 2 E F 2^-53 relative to the sum of magnitudes, and a square
root; float32 results: one rounding (2^-24) of values whose z-scores lose at most about 1e4 x 2^-53."""
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


def _counts(F, L, E, k, seed, empty):
    """Dispatch and co-activation counts of random token-layers."""
    rng = np.random.default_rng(seed)
    n = 200
    off = np.concatenate([[0], np.cumsum([0 if f in empty else n + f for f in range(F)])]).astype(np.int64)
    pop = rng.random((L, 1, E)) * 2
    tr = np.argsort(-(pop + rng.random((L, int(off[-1]), E))), axis=2)[..., :k].astype(np.int16)
    D, C, err = oracle.coact(torch.as_tensor(np.ascontiguousarray(tr)), off, E)
    assert err == 0
    return D, C


@pytest.mark.parametrize("F,L,E,k,empty", [
    (2, 2, 3, 2, ()), (8, 1, 16, 4, ()), (9, 2, 17, 3, (8,)), (16, 2, 64, 6, (0, 9)), (17, 1, 65, 8, ()),
    (24, 2, 128, 8, ()), (33, 1, 130, 5, (32,)), (64, 1, 40, 4, ()), (3, 2, 255, 8, ()), (16, 1, 256, 8, ()),
    (1, 2, 70, 4, ()), (2, 1, 256, 8, ()), (2, 13, 255, 4, ()), (3, 40, 64, 4, (1,)), (4, 1, 129, 6, ()), (5, 12, 129, 6, (0,)),
    (9, 30, 8, 2, ()), (24, 1, 256, 8, ()),  # the last: 64 KB of dynamic LDS and some static
])
def test_family_passes(F, L, E, k, empty):
    print(f"families F={F} L={L} E={E} k={k} empty={empty}", flush=True)
    D, C = _counts(F, L, E, k, 100 * F + E, empty)
    D_t, C_t = torch.as_tensor(D.astype(np.int32)).cuda(), torch.as_tensor(C.astype(np.int32)).cuda()
    tol = 2 * E * F * 2.0 ** -53
    for got, want in zip(tacg.gesr_scores(D_t, C_t, k), oracle.gesr_scores(D, C, k)):
        np.testing.assert_allclose(got.cpu().numpy(), want, rtol=4 * tol, atol=tol)
    np.testing.assert_allclose(tacg.activation_distance(D_t, k).cpu().numpy(), oracle.activation_distance(D, k),
                               rtol=4 * tol * L, atol=tol * L)
    for n in (1, 40, 500):
        pairs, jac = tacg.pair_jaccard(C_t, n)
        np.testing.assert_array_equal(pairs.cpu().numpy(), oracle.top_pairs(C, n))
        np.testing.assert_array_equal(jac.cpu().numpy(), oracle.pair_jaccard(C, n))
    if F >= 2:
        for got, want in zip(tacg.reweight(D_t, C_t, k, want_hat=True), oracle.reweight(D, C, k)):
            np.testing.assert_allclose(got.cpu().double().numpy(), want, rtol=2e-7, atol=1e-30)
