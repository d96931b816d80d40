// Clover term (the Csw! step of paper Sec. 3.3), computed in FP64.
//
// Per site: the clover-leaf field strength of the six planes, made
// anti-Hermitian and traceless; then, in the chiral basis, the diagonal term
// splits into two Hermitian 6x6 blocks (row index 3*spin + colour within a
// chirality):
//   A_+- = (4 + m0 + d_bnd (cF-1)) 1 + (csw/2) [[ i E3, i E1 + E2 ],
//                                              [ i E1 - E2, -i E3 ]],
//   E_k = +-F_{t k} - B_k,  B_1 = F_{yz}, B_2 = F_{zx}, B_3 = F_{xy}.
// This is the sigma_{mu nu} (x) F_{mu nu} sum written out for the chiral
// basis (sigma_{kl} = -eps_{klm} diag(s_m, s_m), sigma_{tk} = diag(s_k, -s_k)).
// The inverse of each block on the odd sites is formed by an unpivoted
// LDL^H factorisation, with Gauss-Jordan elimination under partial pivoting
// as the fallback for an indefinite block with a tiny LDL^H pivot
// (clover_inv.h); a block that is singular to working precision is reported
// as a numerical error.
//
// Work decomposition: a workgroup of W waves owns the 64 sites of one layout
// tile.  Each wave computes the field strength of 6/W planes, one after the
// other (a lane per site), and leaves the nine independent reals of each in LDS;
// then wave b < 2 assembles, stores and inverts the blocks of chirality b.  One
// thread per site doing all of it keeps six 3x3 matrices, four leaves and two
// 6x6 blocks alive: that needed 9 KB of scratch per lane and took 3.26 ms at
// 24^3x48 with three precisions stored.
// Bound: the links through L2 (twelve per plane and site), and their latency:
// with W = 6 four of six waves end at the barrier while the last two hold the
// workgroup's place, and only 1.5 waves per SIMD are resident on average.  W = 2
// keeps every wave to the end: 24^3x48 (two rows, three precisions stored) 664 ->
// 538 us, and with the tile order below and stores past L2 433 to 455 (FP64 alone
// 349).  W = 6 is the shorter chain while the chip is not full: a changed operator
// and its Dw at 12x10x8x14 (210 workgroups) 53 us with W = 6, 58 with 2; 12^3x24
// (648) 93 and 86; 32^3x64 2707 and 2172.  Two waves per SIMD: at three, 25 to 36 registers spill (W = 2: 598
// against 495 us).
#include "clover_inv.h"
#include "lqcd_kernels.h"

namespace lqcd {

using cd = cpx<double>;

constexpr int kCloverPlanes = 6;  // xy, xz, xt, yz, yt, zt
constexpr int kCloverWide = 512;  // from this many workgroups on, two waves each

// Tile order.  In site order every XCD walks whole time slices, and from some
// 10^4 sites a slice its t neighbours have left its L2 when it returns to them.
// Here a time slice is a row of tiles (about: tiles may straddle slices, which
// only costs locality), cut into column groups of at most kGroupTiles tiles, a
// multiple of eight groups; an XCD walks one group through all rows, then the
// next.  24^3x48 538 -> 495 us; a changed operator and its Dw at 32^3x64 2314 ->
// 2172 us, 16^3x32 166 both; groups of 8, 16 and 32 tiles 503, 471 and 476 us.
constexpr int kRowTiles = 32;  // tiles per slice from which the order is used
constexpr int kGroupTiles = 16;

struct M3 {
  cd m[9];
};

__device__ inline M3 m3_mul(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cd v = cmul(a.m[3 * i], b.m[j]);
      v = cmac(v, a.m[3 * i + 1], b.m[3 + j]);
      r.m[3 * i + j] = cmac(v, a.m[3 * i + 2], b.m[6 + j]);
    }
  return r;
}

// a * b^+
__device__ inline M3 m3_mul_nd(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cd v = cmulc(b.m[3 * j], a.m[3 * i]);
      v = cmacc(v, b.m[3 * j + 1], a.m[3 * i + 1]);
      r.m[3 * i + j] = cmacc(v, b.m[3 * j + 2], a.m[3 * i + 2]);
    }
  return r;
}

// a^+ * b
__device__ inline M3 m3_mul_dn(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cd v = cmulc(a.m[i], b.m[j]);
      v = cmacc(v, a.m[3 + i], b.m[3 + j]);
      r.m[3 * i + j] = cmacc(v, a.m[6 + i], b.m[6 + j]);
    }
  return r;
}

// a - b^+
__device__ inline M3 m3_sub_dag(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      r.m[3 * i + j] = {a.m[3 * i + j].re - b.m[3 * j + i].re, a.m[3 * i + j].im + b.m[3 * j + i].im};
  return r;
}

// link U_mu of the site with lexical index lex and parity p
template <bool TWO_ROW>
__device__ inline M3 load_link(const KGeom& g, const double2* U, int lex, int p, int mu) {
  constexpr int ne = TWO_ROW ? 6 : 9;  // stored complex per link
  const double2* u = U + (size_t)p * 4 * ne * g.V2p + tix((size_t)(lex >> 1), 4 * ne) + mu * ne * kTile;
  M3 r;
#pragma unroll
  for (int e = 0; e < ne; ++e) {
    double2 v = u[e * kTile];
    r.m[e] = {v.x, v.y};
  }
  if constexpr (TWO_ROW) su3_third_row(r.m);
  return r;
}

// Traceless anti-Hermitian part of (Q - Q^+)/8 for the (mu, nu) plane at a
// site, Q the sum of the four counter-clockwise leaves.  Leaves 1 and 4 start
// and end with U_mu(x), leaves 2 and 3 with U_mu(x - mu), and only Q - Q^+
// counts, so
//   l1 - l4^+ = U_mu(x) (A - B^+),  l2 - l3^+ = (C - D) U_mu(x - mu)
// take ten products instead of twelve.
template <bool TWO_ROW>
__device__ inline M3 field_strength(const KGeom& g, const double2* U, const Coord& c, int lex, int p, int mu, int nu) {
  // steps of the lexical index to the neighbours, wrapped
  auto step = [&](int d, int dir) {
    int stride = 1;
    for (int k = 0; k < d; ++k) stride *= g.L[k];
    const int x = coord_of(c, d), last = g.L[d] - 1;
    if (dir > 0) return x == last ? -last * stride : stride;
    return x == 0 ? last * stride : -stride;
  };
  const int fm = step(mu, 1), bm = step(mu, -1), fn = step(nu, 1), bn = step(nu, -1);
#define LNK(off, par, d) load_link<TWO_ROW>(g, U, lex + (off), (par), (d))
  const M3 Un_x = LNK(0, p, nu);
  M3 A = m3_mul_nd(LNK(fm, 1 - p, nu), LNK(fn, 1 - p, mu));
  A = m3_mul_nd(A, Un_x);
  M3 B = m3_mul_dn(LNK(bn, 1 - p, nu), LNK(bn, 1 - p, mu));
  B = m3_mul(B, LNK(fm + bn, p, nu));
  A = m3_mul(LNK(0, p, mu), m3_sub_dag(A, B));
  B = m3_mul_nd(Un_x, LNK(bm + fn, p, mu));
  M3 C = m3_mul_nd(B, LNK(bm, 1 - p, nu));
  B = m3_mul(LNK(bm + bn, p, mu), LNK(bn, 1 - p, nu));
  B = m3_mul_dn(B, LNK(bm + bn, p, nu));
#pragma unroll
  for (int e = 0; e < 9; ++e) C.m[e] = csub(C.m[e], B.m[e]);
  C = m3_mul(C, LNK(bm, 1 - p, mu));
#undef LNK
  M3 F;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const cd q = cadd(A.m[3 * i + j], C.m[3 * i + j]), qt = cadd(A.m[3 * j + i], C.m[3 * j + i]);
      F.m[3 * i + j] = {(q.re - qt.re) * 0.125, (q.im + qt.im) * 0.125};
    }
  const double tr_im = (F.m[0].im + F.m[4].im + F.m[8].im) / 3.0;
  F.m[0].im -= tr_im;
  F.m[4].im -= tr_im;
  F.m[8].im -= tr_im;
  return F;
}

// The nine independent reals of an anti-Hermitian 3x3 matrix: the imaginary
// diagonal, then the entries (1,0), (2,0), (2,1).
struct AH3 {
  double d[3];
  cd o[3];
};
// a * X + b * Y
__device__ inline AH3 ah3_comb(double a, const AH3& x, double b, const AH3& y) {
  AH3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    r.d[i] = a * x.d[i] + b * y.d[i];
    r.o[i] = {a * x.o[i].re + b * y.o[i].re, a * x.o[i].im + b * y.o[i].im};
  }
  return r;
}
__device__ inline cd ah3_at(const AH3& x, int i, int j) {
  if (i == j) return {0.0, x.d[i]};
  if (i > j) return x.o[i + j - 1];
  const cd v = x.o[i + j - 1];
  return {-v.re, v.im};  // -conj
}

__device__ inline cd times_i(cd a) { return {-a.im, a.re}; }

// Hermitian 6x6 block from E1, E2, E3 (anti-Hermitian 3x3): the lower
// triangle is computed, the upper one is its adjoint
__device__ inline void make_block(const AH3& E1, const AH3& E2, const AH3& E3, double c, double d, cd (&B)[6][6]) {
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (a >= b) {
        const cd v = cscale(c, times_i(ah3_at(E3, a, b)));
        B[a][b] = v;
        B[3 + a][3 + b] = {-v.re, -v.im};
      }
      B[3 + a][b] = cscale(c, csub(times_i(ah3_at(E1, a, b)), ah3_at(E2, a, b)));
    }
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    B[i][i] = {B[i][i].re + d, 0.0};
#pragma unroll
    for (int j = i + 1; j < 6; ++j) B[i][j] = {B[j][i].re, -B[j][i].im};
  }
}

// block B into components c0 .. c0+17 of site s of a tiled 36-component field
template <typename S>
__device__ inline void store_packed(S* field, size_t s, int c0, const cd (&B)[6][6]) {
  S* base = field + tix(s, 36) + c0 * kTile;
  st_nt(base + 0 * kTile, cd{B[0][0].re, B[1][1].re});
  st_nt(base + 1 * kTile, cd{B[2][2].re, B[3][3].re});
  st_nt(base + 2 * kTile, cd{B[4][4].re, B[5][5].re});
#pragma unroll
  for (int i = 1; i < 6; ++i)
#pragma unroll
    for (int j = 0; j < i; ++j) st_nt(base + tri_index(i, j) * kTile, B[i][j]);
}

template <bool TWO_ROW, int W>
__global__ __launch_bounds__(64 * W, 2) void k_clover(const CloverLaunch c) {
  __shared__ double sh[kCloverPlanes][9][kTile];
  const KGeom& g = c.g;
  // the two parities of a tile side by side
  int tile, p;
  if (c.groups > 0) {
    const int j = (int)(blockIdx.x >> 3), per = 2 * c.rows * c.cols;  // workgroups of a group
    const int grp = (int)(blockIdx.x & 7) + 8 * (j / per), i = (j % per) >> 1;
    const int col = (int)((long)grp * c.row_tiles / c.groups) + i % c.cols;
    if (col >= (int)((long)(grp + 1) * c.row_tiles / c.groups)) return;
    tile = i / c.cols * c.row_tiles + col;
    p = j & 1;
  } else {
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    tile = blk >> 1;
    p = blk & 1;
  }
  const int l = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int s = tile * kTile + l;
  const Coord co = site_coord(g, s < g.V2 ? s : 0, p);
  if (s < g.V2) {
#pragma unroll 1
    for (int q = w * (kCloverPlanes / W); q < (w + 1) * (kCloverPlanes / W); ++q) {
      const int mu = q < 3 ? 0 : (q < 5 ? 1 : 2);
      const int nu = q < 3 ? q + 1 : (q < 5 ? q - 1 : 3);
      const M3 F = field_strength<TWO_ROW>(g, c.U64, co, 2 * s + (co.x & 1), p, mu, nu);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        sh[q][i][l] = F.m[4 * i].im;
        const cd v = F.m[i == 0 ? 3 : 5 + i];  // (1,0), (2,0), (2,1)
        sh[q][3 + 2 * i][l] = v.re;
        sh[q][4 + 2 * i][l] = v.im;
      }
    }
  }
  __syncthreads();
  if (w >= 2 || s >= g.V2) return;
  const int b = w;  // chirality
  auto plane = [&](int q) {
    AH3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      r.d[i] = sh[q][i][l];
      r.o[i] = {sh[q][3 + 2 * i][l], sh[q][4 + 2 * i][l]};
    }
    return r;
  };
  const int T = g.L[3];
  bool bnd = false;
  if (g.bc == BC_SF) bnd = (co.t == 1) || (co.t == T - 1);
  if (g.bc == BC_OPEN) bnd = (co.t == 0) || (co.t == T - 1);
  const double d = 4.0 + c.m0 + (bnd ? (c.cF - 1.0) : 0.0);
  const double cc = 0.5 * c.csw;
  const size_t par = (size_t)p * 36 * g.V2p;  // parity p of the clover field

  // E_k = sg F_{tk} - B_k with F_{tk} = -F_{kt}; planes 0 xy, 1 xz, 2 xt, 3 yz, 4 yt, 5 zt
  const double sg = (b == 0) ? 1.0 : -1.0;
  auto block = [&](cd(&B)[6][6]) {
    make_block(ah3_comb(-sg, plane(2), -1.0, plane(3)), ah3_comb(-sg, plane(4), 1.0, plane(1)),
               ah3_comb(-sg, plane(5), -1.0, plane(0)), cc, d, B);
  };
  // the matrix to invert: the block, or with a twisted mass (the block of
  // chirality b is B + i sg mu) Q = B^2 + mu^2: B is Hermitian, so
  // (B + i m)^{-1} = Q^{-1} (B - i m) for m = +-mu (and the adjoint is the same
  // with -m); the odd sites store the Hermitian positive definite Q^{-1}, the
  // hop kernels apply B and the i m term themselves
  auto to_invert = [&](cd(&B)[6][6]) {
    if (c.mu == 0.0) return;
    cd Q[6][6];
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) {
        cd v = {i == j ? c.mu * c.mu : 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 6; ++k) v = cmac(v, B[i][k], B[k][j]);
        Q[i][j] = v;
      }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      B[i][i] = {Q[i][i].re, 0.0};
#pragma unroll
      for (int j = 0; j < i; ++j) {
        B[i][j] = Q[i][j];
        B[j][i] = {Q[i][j].re, -Q[i][j].im};
      }
    }
  };
  cd B[6][6];
  block(B);
  store_packed(c.C64 + par, s, 18 * b, B);
  if (c.C32) store_packed(c.C32 + par, s, 18 * b, B);
  if (c.C16) store_packed(c.C16 + par, s, 18 * b, B);
  if (p == 0) return;
  to_invert(B);
  const double bound = blk6::norm_inf_bound(B);
  blk6::NormBound rb;
  const size_t base = tix((size_t)s, 36) + 18 * b * kTile;
  auto put = [&](int e, cd v) {
    st_nt(c.Ci64 + base + e * kTile, v);
    if (c.Ci32) st_nt(c.Ci32 + base + e * kTile, v);
    if (c.Ci16) st_nt(c.Ci16 + base + e * kTile, v);
  };
  double diag[6];
  const bool ldl = blk6::inverse_ldl_each(B, [&](int i, int j, cd v) {
    rb.add(i, j, v);
    if (i != j) return put(tri_index(i, j), v);
    diag[i] = v.re;
    if (i & 1) put(i >> 1, cd{diag[i - 1], diag[i]});
  });
  if (!(ldl && blk6::accepted(bound, rb.max()))) {  // rare: the norms decide, or the pivoted route
    cd A[6][6], R[6][6];
    block(A);
    to_invert(A);
    blk6::inverse_ldl(A, R);
    if (blk6::herm_inverse_careful(A, R, ldl) == blk6::INV_SINGULAR) atomicOr(c.err_flag, 1);
    store_packed(c.Ci64, s, 18 * b, R);
    if (c.Ci32) store_packed(c.Ci32, s, 18 * b, R);
    if (c.Ci16) store_packed(c.Ci16, s, 18 * b, R);
  }
}

template <int W>
static void launch_clover_w(const CloverLaunch& c, unsigned grid, hipStream_t st) {
  if (c.two_row)
    k_clover<true, W><<<grid, 64 * W, 0, st>>>(c);
  else
    k_clover<false, W><<<grid, 64 * W, 0, st>>>(c);
}

hipError_t launch_clover(const CloverLaunch& c0, hipStream_t st) {
  CloverLaunch c = c0;
  const int tiles = (int)((c.g.V2 + kTile - 1) / kTile);
  unsigned grid = 2u * (unsigned)tiles;
  c.row_tiles = (int)((c.g.V2 / c.g.L[3] + kTile - 1) / kTile);
  c.groups = 0;
  if (c.row_tiles >= kRowTiles) {
    c.groups = 8 * ((c.row_tiles + 8 * kGroupTiles - 1) / (8 * kGroupTiles));
    c.rows = (tiles + c.row_tiles - 1) / c.row_tiles;
    c.cols = (c.row_tiles + c.groups - 1) / c.groups;
    grid = (unsigned)c.groups * 2u * (unsigned)c.rows * (unsigned)c.cols;
  }
  if (2 * tiles < kCloverWide)
    launch_clover_w<6>(c, grid, st);
  else
    launch_clover_w<2>(c, grid, st);
  return hipGetLastError();
}

}  // namespace lqcd
