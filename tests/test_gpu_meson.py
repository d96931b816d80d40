"""GPU parity of the meson contraction (lqcd_meson) against the oracle's
meson_G / meson_correlator, on the same seeded 12-column fields.

Tolerance: relative 1e-12 (max-norm over the tensor, resp. over each
correlator): both sides sum the same FP64 products, in different orders,
over at most a few thousand sites per slice.
"""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2503_16994_amd import inputs, lqcd

pytestmark = pytest.mark.gpu

# every diagonal pair and a few mixed ones (g5 with g_t, 1 with g5, g_x with g_y)
PAIRS = [(m, m) for m in range(16)] + [(15, 8), (0, 15), (1, 2)]


def rel_max(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def random_columns(L, seed):
    rng = np.random.default_rng(seed)
    shape = (12, L[3], L[2], L[1], L[0], 4, 3)
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


# 6x4x4x6: V3 = 96 (one partial chunk); 12x10x8x6: V3 = 960 = 3 x 256 + 192
# (ragged last chunk); 16x16x8x4: V3 = 2048 (eight full chunks)
@pytest.mark.parametrize("L", [(6, 4, 4, 6), (12, 10, 8, 6), (16, 16, 8, 4)], ids=lambda L: "x".join(map(str, L)))
def test_meson_matches_oracle_on_random_columns(L):
    print(f"\n[gpu case] meson {L}", flush=True)
    psi = random_columns(L, seed=sum(L))
    lat = lqcd.Lattice(L, lqcd.BC_PERIODIC, (1, 1, 1, -1))
    ws = lqcd.Workspace(lat, lqcd.PM_F64, 1)
    C, G = lqcd.meson(lat, torch.from_numpy(psi).cuda(), PAIRS, ws)
    torch.cuda.synchronize()
    G_ref = orc.meson_G(L, psi)
    assert rel_max(G.cpu().numpy(), G_ref) < 1e-12
    Cg = C.cpu().numpy()
    for p, (m1, m2) in enumerate(PAIRS):
        ref = orc.meson_correlator(G_ref, m1, m2)
        assert rel_max(Cg[p], ref) < 1e-12, (m1, m2)
    # only C, then only G: the same numbers
    C2, none = lqcd.meson(lat, torch.from_numpy(psi).cuda(), PAIRS[:3], ws, want_G=False)
    assert none is None and np.array_equal(C2.cpu().numpy(), Cg[:3])
    none, G2 = lqcd.meson(lat, torch.from_numpy(psi).cuda(), [], ws)
    assert none is None and np.array_equal(G2.cpu().numpy(), G.cpu().numpy())


# 2x2x2x4: half of one 16-site step of a workgroup; 6x2x2x4: V3 = 24, a ragged
# second step; 10x6x2x4: V3 = 120, a ragged second 64-site chunk; 2x2x2x2046
# and 2x2x2x2048: both sides of the line where the chunk grows to 1024 sites.
# Sums of at most 9 V3 products of O(1) numbers: 1e-12 as above.
@pytest.mark.parametrize("L", [(2, 2, 2, 4), (6, 2, 2, 4), (10, 6, 2, 4), (2, 2, 2, 2046), (2, 2, 2, 2048)],
                         ids=lambda L: "x".join(map(str, L)))
def test_meson_chunk_edges(L):
    print(f"\n[gpu case] meson {L}", flush=True)
    psi = random_columns(L, seed=sum(L))
    lat = lqcd.Lattice(L, lqcd.BC_PERIODIC, (1, 1, 1, -1))
    ws = lqcd.Workspace(lat, lqcd.PM_F64, 1)
    C, G = lqcd.meson(lat, torch.from_numpy(psi).cuda(), PAIRS, ws)
    G_ref = orc.meson_G(L, psi)
    assert rel_max(G.cpu().numpy(), G_ref) < 1e-12
    for p, (m1, m2) in enumerate(PAIRS):
        assert rel_max(C[p].cpu().numpy(), orc.meson_correlator(G_ref, m1, m2)) < 1e-12, (m1, m2)


def test_meson_of_a_solved_propagator():
    """12 point sources solved by lqcd_solve (8^3x16, FP64 eo-CG, two-row
    links), contracted on the GPU: equal to the oracle's contraction of the
    same solution; the pion correlator is positive."""
    L = (8, 8, 8, 16)
    U = inputs.gauge_field(L, 0.2, seed=7)
    lat = lqcd.Lattice(L, lqcd.BC_PERIODIC, (1, 1, 1, -1))
    g = lqcd.GaugeField(lat, torch.from_numpy(U), lqcd.PM_F64 | lqcd.PM_TWO_ROW)
    eta = torch.from_numpy(inputs.point_sources_12(L, (0, 0, 0, 0))).cuda()
    ws = lqcd.Workspace(lat, lqcd.PM_F64, 12)
    r = lqcd.solve(g, eta, 0.1345, 1.9, tol=1e-10, ws=ws)
    assert r.status == lqcd.OK
    C, G = lqcd.meson(lat, r.psi, PAIRS, ws)
    torch.cuda.synchronize()
    psi = r.psi.cpu().numpy()
    G_ref = orc.meson_G(L, psi)
    assert rel_max(G.cpu().numpy(), G_ref) < 1e-12
    pion = C.cpu().numpy()[15]
    assert rel_max(pion, orc.meson_correlator(G_ref, 15, 15)) < 1e-12
    assert np.all(pion.real > 0) and np.max(np.abs(pion.imag)) < 1e-10 * np.max(pion.real)
    print("pion correlator:", np.array2string(pion.real, precision=4))


def test_meson_full_size_sampled_slices():
    """32^3x64 (the C3 lattice), random columns: the GPU contraction over the
    whole lattice, checked on four time slices against the oracle on those
    slices alone."""
    L = (32, 32, 32, 64)
    rng = np.random.default_rng(5)
    shape = (12, 64, 32, 32, 32, 4, 3)
    psi = torch.complex(torch.randn(shape, dtype=torch.float64, device="cuda"),
                        torch.randn(shape, dtype=torch.float64, device="cuda"))
    lat = lqcd.Lattice(L, lqcd.BC_PERIODIC, (1, 1, 1, -1))
    ws = lqcd.Workspace(lat, lqcd.PM_F64, 1)
    C, G = lqcd.meson(lat, psi, [(15, 15), (8, 8)], ws)
    torch.cuda.synchronize()
    Gg, Cg = G.cpu().numpy(), C.cpu().numpy()
    for t in sorted(rng.choice(64, 4, replace=False)):
        sl = psi[:, t:t + 1].cpu().numpy()
        G_ref = orc.meson_G((32, 32, 32, 1), sl)[0]
        assert rel_max(Gg[t], G_ref) < 1e-12, t
        assert abs(Cg[0, t] - orc.meson_correlator(G_ref[None], 15, 15)[0]) < 1e-12 * abs(Cg[0, t])
    del psi
    torch.cuda.empty_cache()


# Columns that differ by a phase that barely varies, or by that and a factor i
# (spins tied by a gamma matrix): every entry of G has one large part and one
# that all but cancels.  That part is held to the rounding of its own terms:
# 9 V3 pairs of products |z_i z_j| ~ 1, a rounding of u = 2^-53 of each pair's
# size, adding up like a random walk, times 8.  (A sum of one product over the
# slice, subtracted from its transpose afterwards, is off by the rounding of that
# sum, which is as large as the other part.)  16^3: 64-site chunks, summed by the
# second kernel; 8^3: one chunk a slice, summed in the first.
@pytest.mark.parametrize("L", [(16, 16, 16, 4), (8, 8, 8, 2048)], ids=lambda L: "x".join(map(str, L)))
def test_meson_parts_that_cancel(L):
    print(f"\n[gpu case] meson cancelling parts {L}", flush=True)
    T, V3 = L[3], L[0] * L[1] * L[2]
    gen = torch.Generator(device="cuda").manual_seed(3)
    ph = torch.randn((12, T, V3, 4, 3), generator=gen, dtype=torch.float64, device="cuda").mul_(0.05).add_(0.7)
    spin = torch.arange(4, device="cuda")
    col = torch.arange(12, device="cuda") // 3
    ph += (math.pi / 2) * ((col[:, None] + spin[None, :]) % 2)[:, None, None, :, None]
    psi = torch.polar(1 + 0.3 * torch.rand(ph.shape, generator=gen, dtype=torch.float64, device="cuda"), ph)
    del ph
    lat = lqcd.Lattice(L, lqcd.BC_PERIODIC, (1, 1, 1, -1))
    _, G = lqcd.meson(lat, psi.reshape(12, T, L[2], L[1], L[0], 4, 3), [], lqcd.Workspace(lat, lqcd.PM_F64, 1))
    G = G.cpu().numpy()
    par = (np.arange(4)[:, None] + np.arange(4)[None, :]) % 2  # [al][be]
    for t in {0, T // 2, T - 1}:
        z = psi[:, t].cpu().numpy().reshape(4, 3, V3, 4, 3).transpose(3, 0, 2, 4, 1).reshape(16, -1)  # [(al, be)][x, a, c]
        zr, zi = z.real.astype(np.longdouble), z.imag.astype(np.longdouble)
        # term by term, in 64-bit mantissas (products summed one by one would cancel here too)
        re = np.stack([(zr[i] * zr + zi[i] * zi).sum(axis=1) for i in range(16)])
        im = np.stack([(zi[i] * zr - zr[i] * zi).sum(axis=1) for i in range(16)])
        small = (par.reshape(-1)[:, None] != par.reshape(-1)[None, :])  # Re is the small part
        g = G[t].reshape(16, 16)
        err = np.where(small, np.abs(g.real - re), np.abs(g.imag - im)).astype(np.float64)
        tol = 8 * 2.0 ** -53 * math.sqrt(9 * V3) * 1.3 ** 2
        assert err.max() <= tol, (t, err.max(), tol)
        assert rel_max(g, (re + 1j * im).astype(np.complex128)) < 1e-12


# Chunks of 128 (6^3x1024), 256 (10^3x512), 512 (14x14x10x512) and 1024 sites
# (14^3x768), each with a ragged last one (88, 232, 424 and 696 sites, which half
# fill their last step of 16): sampled slices against the oracle on those slices
# alone, relative 1e-12 as above; a correlator has 16 terms of G.
@pytest.mark.parametrize("L", [(6, 6, 6, 1024), (10, 10, 10, 512), (14, 14, 10, 512), (14, 14, 14, 768)],
                         ids=lambda L: "x".join(map(str, L)))
def test_meson_ragged_chunks(L):
    print(f"\n[gpu case] meson ragged chunk {L}", flush=True)
    T = L[3]
    gen = torch.Generator(device="cuda").manual_seed(T)
    psi = torch.randn((12, T, L[2], L[1], L[0], 4, 3), generator=gen, dtype=torch.complex128, device="cuda")
    lat = lqcd.Lattice(L, lqcd.BC_PERIODIC, (1, 1, 1, -1))
    C, G = lqcd.meson(lat, psi, PAIRS, lqcd.Workspace(lat, lqcd.PM_F64, 1))
    G, C = G.cpu().numpy(), C.cpu().numpy()
    for t in (0, 1, T // 2 + 1, T - 1):
        G_ref = orc.meson_G((*L[:3], 1), psi[:, t:t + 1].cpu().numpy())
        assert rel_max(G[t], G_ref[0]) < 1e-12, t
        for p, (m1, m2) in enumerate(PAIRS):
            ref = orc.meson_correlator(G_ref, m1, m2)[0]
            assert abs(C[p, t] - ref) < 16e-12 * np.max(np.abs(G_ref)), (t, m1, m2)
    del psi
    torch.cuda.empty_cache()
