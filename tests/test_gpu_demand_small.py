"""The one-launch demand against the oracle, element by element, at the edges
of its range (rows of up to 4,096 ids, up to 1,024 experts) and just past
them, where the two passes take over."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vp():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2609_34340_amd as vp
    vp.lib()
    return vp


@pytest.mark.parametrize("T,k,E,N,R,sort_row", [
    (1, 1, 8, 8, 1, 0), (1, 1, 1, 1, 1, 0), (63, 1, 16, 8, 2, 1), (64, 1, 16, 8, 2, -1), (65, 1, 24, 8, 3, 0),
    (341, 3, 48, 16, 2, 1), (1024, 1, 256, 64, 2, 0), (1025, 1, 256, 64, 2, 1), (256, 8, 256, 256, 4, 3),
    (683, 3, 1024, 64, 2, 0), (512, 4, 1024, 1024, 2, 1), (293, 7, 512, 8, 3, 2), (1024, 4, 512, 32, 2, 0),
    (585, 7, 1016, 8, 2, 1), (4096, 1, 8, 8, 2, 0), (4097, 1, 8, 8, 2, 0), (1025, 4, 256, 32, 2, 1),
    (1024, 4, 1032, 8, 2, 1), (16, 255, 256, 8, 2, 0)])
def test_edges(vp, T, k, E, N, R, sort_row):
    rng = np.random.default_rng(T * k + E)
    # skewed experts, repeats among a token's slots included
    ids = np.minimum((rng.random((R, T, k)) ** 2 * E).astype(np.int32), E - 1)
    first = N - R if N >= R else 0
    rows = torch.from_numpy(ids).cuda()
    out = vp.demand(rows, N, E, 4096, first_rank=first, sort_row=sort_row)
    torch.cuda.synchronize()
    assert vp.read_status(out["status"]) == 0
    for r in range(R):
        ref = oracle.demand(ids[r], N, E, first + r, 4096)
        assert np.array_equal(out["demand"][r].cpu().numpy(), ref["row"]), r
        assert np.array_equal(out["counts"][r].cpu().numpy(), ref["counts"]), r
    if sort_row >= 0:
        ref = oracle.demand(ids[sort_row], N, E, first + sort_row, 4096)
        for key in ("sorted_tok", "sorted_slot"):
            assert np.array_equal(out[key].cpu().numpy()[:T * k], ref[key]), key
        assert np.array_equal(out["dest_off"].cpu().numpy(), ref["dest_off"])


@pytest.mark.parametrize("T,k,E", [(5, 2, 16), (4096, 1, 1024)])
@pytest.mark.parametrize("bad", [-1, 1 << 30])
def test_bad_id_is_reported(vp, T, k, E, bad):
    ids = torch.zeros((2, T, k), dtype=torch.int32, device="cuda")
    ids[1, T - 1, k - 1] = bad
    for sort_row in (-1, 0, 1):
        out = vp.demand(ids, 8, E, 4096, sort_row=sort_row)
        torch.cuda.synchronize()
        assert vp.read_status(out["status"]) == vp.INVALID_ARGUMENT
        assert int(out["counts"].sum()) == 2 * T * k - 1


# a row's demand from its experts' sums or from their offsets: destinations of one expert to all of them
@pytest.mark.parametrize("E,N", [(1, 1), (1024, 1), (1024, 8), (136, 8), (128, 8), (120, 8), (1020, 60), (1024, 64),
                                 (1024, 1024)])
@pytest.mark.parametrize("T,k", [(1, 1), (77, 8), (4096, 1)])
def test_demand_row_of_many_experts(vp, E, N, T, k):
    rng = np.random.default_rng(E + N + T)
    R = min(N, 3)
    ids = rng.integers(0, E, (R, T, k)).astype(np.int32)
    for sort_row in (-1, R - 1):
        out = vp.demand(torch.from_numpy(ids).cuda(), N, E, 4112, first_rank=N - R, sort_row=sort_row)
        torch.cuda.synchronize()
        assert vp.read_status(out["status"]) == 0
        for r in range(R):
            ref = oracle.demand(ids[r], N, E, N - R + r, 4112)
            assert np.array_equal(out["demand"][r].cpu().numpy(), ref["row"]), r
            assert np.array_equal(out["counts"][r].cpu().numpy(), ref["counts"]), r
        if sort_row >= 0:
            assert np.array_equal(out["sorted_tok"].cpu().numpy()[:T * k], ref["sorted_tok"])
            assert np.array_equal(out["dest_off"].cpu().numpy(), ref["dest_off"])
