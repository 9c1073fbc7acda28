"""mps_workspace_size holds the room that the direct eigensolver of the splits
uses behind the plan, for every operation that splits (host only)."""
import pytest

from paper_1703_00387_amd import _lib, api


def _slot(m, n):
    """Lower bound of one matrix's scratch: the Gram, the reflectors and the exchange of the tridiagonalisation."""
    return 16 * (m * m + m * m + max(2 * m * m, m * n))


@pytest.mark.parametrize("chi,d", [(256, 2), (512, 2), (512, 5), (40, 2)])
def test_tdvp_size_holds_the_splits_room(chi, d):
    """The Lanczos vectors, theta, environments and MPO products of mps_tdvp2_step, counted here from its
    arguments, plus one slot: the size may not be smaller."""
    L, w, nk, e = 8, 4, 20, 16
    N, X = chi * d * d * chi, chi * w * d * d * chi
    plan = e * (2 * (L + 1) * chi * w * chi + 3 * X + (nk + 1) * N + 3 * N + 3 * N)
    size = api.workspace_size(_lib.MPS_OP_TDVP, "c128", 1, L, d, chi, w, nk)
    assert size >= plan + _slot(d * chi, d * chi)


@pytest.mark.parametrize("chi,d", [(256, 2), (512, 5)])
def test_truncate_size_holds_the_room(chi, d):
    m = d * chi
    assert api.workspace_size(_lib.MPS_OP_TRUNCATE, "c128", 1, 2, d, chi) >= 16 * m * m + _slot(m, m)
