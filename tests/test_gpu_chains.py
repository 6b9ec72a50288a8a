"""How many products the library adds up one after the other: the rounding error of K and of the
adjoint grows with the length of such a chain.

The first product of a sum is 2^56, all others are 1.  A partial sum that holds the first one loses
every 1 added to it (they are under half of its last place, four of them together still are), the
other partial sums are whole numbers and exact, so the sum falls short by the length of the first
chain.  Adding the partial sums up rounds each to a multiple of 16, at most 8 off per addition."""
import pytest

torch = pytest.importorskip("torch")

from paper_2505_03755_amd import dfmi

pytestmark = pytest.mark.gpu
BIG = 2.0 ** 28   # its square is the first product


def ones_with_big_column(naux, nao):
    """Packed b^P_ij = 1, but 2^28 where P = 0 and i or j is 0."""
    B = torch.ones((naux, nao * (nao + 1) // 2), dtype=torch.float64, device="cuda")
    i = torch.arange(nao, device="cuda")
    B[0, i * (i + 1) // 2] = BIG
    return B


def unit_columns(nao, n):
    return torch.eye(nao, dtype=torch.float64, device="cuda")[:, :n].contiguous()


# 640 slabs of 16 products a chain; 12000 products where 40 chains are more than that needs.  The contraction is in whole
# slabs, runs on across the auxiliary rows, or is weighted.
@pytest.mark.parametrize("nao,naux,nocc,weighted,limit", [
    (800, 800, 800, False, 10240), (800, 801, 799, False, 10240), (800, 800, 800, True, 10240),
    (1200, 400, 1200, False, 12000)])
def test_k_chains(nao, naux, nocc, weighted, limit):
    B = ones_with_big_column(naux, nao)
    w = torch.ones((1, nocc), dtype=torch.float64, device="cuda") if weighted else None
    _, K, _ = dfmi.jk(B, nao, unit_columns(nao, nocc)[None].contiguous(), w=w, want_j=False, want_v=False)
    # K_ij = sum_{P, c} b^P_ic b^P_jc for i, j >= 1
    lost = (BIG * BIG - K[0, 1:, 1:]) + float(naux * nocc - 1)
    assert lost.min().item() >= -8 * 128
    worst = lost.max().item()
    assert worst <= limit + 8 * 128, worst


# 2048 slabs a chain of the 128-wide tiles, counted over slabs of 16 of each row of b^P, and none longer in the columns
# and rows past them
@pytest.mark.parametrize("nao,naux,nocc", [(600, 600, 150), (1200, 2400, 300), (450, 900, 300)])
def test_adjoint_chains(nao, naux, nocc):
    B = ones_with_big_column(naux, nao)
    C = unit_columns(nao, nocc)
    # S = gK + gK^T = 1, so dCocc_mc = sum_P b^P Y_P with Y_P = b^P C
    gK = 0.5 * torch.eye(nao, dtype=torch.float64, device="cuda")
    dC = dfmi.step_backward(B, nao, C, unit_columns(nao, 0), None, gK, None)[0]
    scale = round(dC[1, 1].item() / (BIG * BIG))   # a whole factor of the cotangent
    lost = BIG * BIG * scale - dC[1:, 1:] + scale * float(naux * nao - 1)
    assert lost.min().item() >= -8 * 512 * scale
    wide = lost[:nao // 128 * 128 - 1, :nocc // 128 * 128 - 1].max().item()
    assert wide <= scale * (2048 * 16 + 8 * 512), wide
    assert lost.max().item() <= wide + 16 * 512 * scale, (lost.max().item(), wide)


def test_v_chain():
    """v_0 = sum_m b_mm with 2^56 in the first row and 7 in one row of every other 64-row band: added to 2^56 one at a
    time a 7 is lost.  With 128-row bands seven were; the partial sums that are kept round by 8 each."""
    nao = 1024
    B = torch.zeros((1, nao * (nao + 1) // 2), dtype=torch.float64, device="cuda")
    m = torch.arange(0, nao, 64, device="cuda")
    B[0, m * (m + 3) // 2] = 7.0
    B[0, 0] = BIG * BIG
    ones = torch.ones((nao, 1), dtype=torch.float64, device="cuda")
    v = dfmi.step(B, nao, ones, unit_columns(nao, 0), unit_columns(nao, 1))["v"]
    lost = BIG * BIG - v.item() + 7.0 * (len(m) - 1)
    assert abs(lost) <= 7 * 7 + 8 * 3, lost
