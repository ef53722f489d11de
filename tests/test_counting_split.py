"""The split of a counting call: how many workgroups count (from the workspace size, which holds a slot of pair counts for each
and one for every segment), and GPU parity where the number changes: one segment, one long family among empty ones, many
short ones, each class of expert count and both counting paths.  Counts are whole numbers: they must equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_01007_amd as tacg
from paper_2606_01007_amd import synth


def _workgroups(E, k, L, F, N):
    bins = E if k == 1 else E * (E - 1) // 2
    return int(tacg.lib().tacg_coact_workspace_bytes(N, L, k, E, F)) // (4 * bins) - L * F


# the reduction of a segment reads the slots of its workgroups one after the other: few segments, few workgroups
@pytest.mark.parametrize("E,k,L,F,N,lo,hi", [
    (256, 2, 1, 1, 374006, 8, 16), (160, 6, 1, 1, 200000, 7, 32), (128, 2, 4, 4, 306464, 38, 256), (100, 2, 24, 16, 437668, 321, 800), (128, 8, 1, 1, 200000, 25, 128), (60, 1, 12, 64, 124060, 400, 750),
    (64, 8, 2, 1, 500000, 64, 256), (256, 8, 58, 16, 4096, 230, 240), (128, 8, 48, 16, 16384, 700, 800), (256, 8, 58, 16, 1 << 21, 256, 256),
    (8, 2, 1, 1, 0, 1, 1),
])
def test_workgroups(E, k, L, F, N, lo, hi):
    assert lo <= _workgroups(E, k, L, F, N) <= hi


@pytest.mark.parametrize("E,k", [(256, 2), (160, 6), (128, 2), (100, 1), (128, 8), (60, 4)])
def test_workgroups_grow_with_the_size(E, k):
    """A workspace for longer traces, more layers or more families also holds a smaller call."""
    for L, F in ((1, 1), (3, 2), (12, 8), (48, 64)):
        w = [_workgroups(E, k, L, F, n) for n in (*range(0, 60000, 97), 300000, 1 << 21, 1 << 24)]
        assert w == sorted(w)
        assert _workgroups(E, k, L, F, 40000) <= _workgroups(E, k, L, F + 1, 40000)


def test_sizes_beyond_the_limits_have_a_workspace_size_too():
    assert _workgroups(100000, 2, 1, 1, 1 << 20) >= 1 and _workgroups(300, 40, 3, 100, 1000) >= 1


@pytest.mark.gpu
@pytest.mark.parametrize("E,k,L,counts", [
    (256, 2, 1, [60001]), (160, 6, 1, [40000]), (129, 3, 2, [0, 30000, 0, 7]), (128, 2, 3, [25000, 1]), (100, 1, 1, [50000]),
    (256, 1, 2, [20000, 30]), (128, 8, 1, [40000]), (128, 12, 2, [9000, 0, 1]), (60, 4, 1, [50001]), (64, 8, 2, [30, 30000]),
    (40, 2, 4, [17] * 64), (24, 5, 3, [0] * 63 + [5000]),
])
def test_counts(E, k, L, counts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build()
    print(f"counting split E={E} k={k} L={L} counts={counts[:4]}", flush=True)
    off = synth.fam_offsets(counts)
    gen = torch.Generator().manual_seed(E + k)
    tr = torch.topk(torch.rand((L, int(off[-1]), E), generator=gen), k, dim=2).indices.to(torch.int16)
    D, C, err = tacg.coact_build(tr.cuda(), off, E)
    Do, Co, _ = oracle.coact(tr, off, E)
    assert int(err.item()) == 0
    np.testing.assert_array_equal(tacg.as_u32(D).cpu().numpy(), Do)
    np.testing.assert_array_equal(tacg.as_u32(C).cpu().numpy(), Co)
