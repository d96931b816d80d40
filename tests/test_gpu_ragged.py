"""GPU parity on lattices smaller than, or not a multiple of, the 64-site pieces
that the import, clover and hop kernels work in: extents of 2 (both neighbours
of a site in a direction are the same site), V = 32, 48, 240 and 720.  The last
two have time slices of 38.5 and 137.3 pieces, which the clover kernel's tile
order cuts into 8 and 16 column groups of unequal width (two waves a piece).

FP64 operators against the oracle, relative 2-norm <= 1e-12: a few hundred
roundings of 2^-53 per component, the bound of the other operator tests.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2503_16994_amd import inputs, lqcd

pytestmark = pytest.mark.gpu

P, SF, OPEN = 0, 1, 2
CASES = [((2, 2, 2, 4), P), ((2, 2, 2, 6), OPEN), ((6, 2, 2, 10), SF), ((10, 6, 2, 6), P),
         ((22, 14, 16, 8), P), ((26, 26, 26, 4), OPEN)]


@pytest.mark.parametrize("mu", [0.0, 0.07], ids=["mu0", "mu"])
@pytest.mark.parametrize("two_row", [False, True], ids=["full", "two_row"])
@pytest.mark.parametrize("L,bc", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "PSO"[v])
def test_operators_on_ragged_lattices(L, bc, two_row, mu):
    print(f"\n[gpu case] ragged {L} bc {bc} two_row {two_row} mu {mu}", flush=True)
    theta = (1, 1, 1, -1) if bc == P else tuple(np.exp(1j * np.array([0.3, -1.2, 2.2, 0.0])))
    kappa, csw, cF = 0.125, 1.7, 1.2
    U = inputs.gauge_field(L, 0.25, seed=sum(L), bc=bc)
    A = orc.clover_matrix(L, bc, U, orc.m0_from_kappa(kappa), csw, cF, mu)
    lat = lqcd.Lattice(L, bc, theta)
    g = lqcd.GaugeField(lat, torch.from_numpy(U), lqcd.PM_F64 | (lqcd.PM_TWO_ROW if two_row else 0))
    ws = lqcd.Workspace(lat, lqcd.PM_F64, 2)
    d = lqcd.dirac(kappa, csw, cF, mu)
    psi = np.stack([inputs.gaussian_spinor(L, 5 + k, bc) for k in range(2)])
    x = torch.from_numpy(psi).cuda()
    got = lqcd.dw_apply(g, d, x, op=lqcd.OP_DW, ws=ws).cpu().numpy()
    back = lqcd.dw_apply(g, d, x, op=lqcd.OP_DW_DAG, ws=ws).cpu().numpy()
    schur = lqcd.dw_apply(g, d, x, op=lqcd.OP_SCHUR, ws=ws).cpu().numpy()
    Ainv = orc.inverse_blocks(A)
    odd = orc.parity_mask(L)
    for j in range(2):
        for have, want in ((got[j], orc.dw(L, bc, theta, U, A, psi[j])), (back[j], orc.dw_dag(L, bc, theta, U, A, psi[j]))):
            assert np.linalg.norm(have - want) <= 1e-12 * np.linalg.norm(want), j
        pe = psi[j].copy()
        pe[odd] = 0
        want = orc.schur_dhat(L, bc, theta, U, A, Ainv, pe)
        want[odd] = 0
        assert np.linalg.norm(schur[j] - want) <= 1e-12 * np.linalg.norm(want), j
