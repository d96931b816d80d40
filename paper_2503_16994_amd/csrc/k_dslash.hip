// Hopping-term (Wilson "Dslash") kernels with the clover block fused in.
//
// Work decomposition.  A thread owns one output site of parity p_out and NR
// right-hand sides; RL consecutive lanes share one site and own RL different
// rhs groups (so a 128-thread workgroup covers 128/RL sites and RL*NR rhs;
// 128 rather than 256 threads gives the one-rhs launches on a 16^3x32 lattice
// two workgroups per CU instead of one).  Per
// hop a thread loads the link (9 site-coalesced complex loads, or 6 when the
// field keeps two rows per link and the third is rebuilt in registers; the RL
// lanes of a site issue identical addresses, which the memory pipeline serves once)
// and, for each of its NR rhs, the neighbour spinor (12 loads), spin-projects
// it to a half spinor, multiplies by U or U^+ and accumulates.  The clover
// blocks (two Hermitian 6x6 blocks) are loaded one chirality at a time and
// applied to all NR rhs.  Links and clover blocks are read once per launch, so
// they are loaded non-temporally, leaving L2 to the spinors that neighbouring
// sites re-read.  The only cross-lane work is the optional per-rhs |out|^2
// block reduction (wave64 butterfly over the lanes of one rhs, then LDS
// across the block's waves), which is deterministic.
//
// This is a 3x3 complex mat-vec stencil: there is no dense contraction to
// give to the matrix cores; the kernel is bound by HBM bandwidth and is
// written for coalescing (unit-stride SoA loads over sites), L2 reuse (the
// block orders below) and occupancy (RL instead of NR keeps registers low).
#include <type_traits>

#include "cg_dev.h"

namespace lqcd {

constexpr int kHopBlock = 128;  // threads per workgroup

// Raw operands of one hop (the link and the NR neighbour spinors, in their
// storage types), so that a hop's loads can be issued before the arithmetic
// of the hop before it.
template <int NR, typename SG, typename SI>
struct HopOperands {
  SG u[9];
  SI y[NR][12];
};

template <typename S>
__device__ inline S raw_ld(const S* p) {
  return *p;
}
__device__ inline double2 raw_ld_nt(const double2* p) {
  nt_d2 v = __builtin_nontemporal_load(reinterpret_cast<const nt_d2*>(p));
  return make_double2(v.x, v.y);
}
__device__ inline float2 raw_ld_nt(const float2* p) {
  nt_f2 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f2*>(p));
  return make_float2(v.x, v.y);
}
__device__ inline bf16x2 raw_ld_nt(const bf16x2* p) {
  return bf16x2{__builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p))};
}
template <typename A, typename S>
__device__ inline cpx<A> widen(const S& v) {
  const auto c = StoreTraits<S>::load(&v);
  return {(A)c.re, (A)c.im};
}

// Phase of the hop x -> x + DIR mu at a site: the boundary phase on the edge,
// zero where the hop is cut (the Schroedinger-functional backward hop from
// t = 1 lands on the Dirichlet slice t = 0, whose field is ignored).
template <int MU, int DIR, typename A>
__device__ inline bool hop_phase(const KGeom& g, const Coord& c, bool& edge, A& pr, A& pi) {
  const int coord = coord_of(c, MU);
  edge = (DIR > 0) ? (coord == g.L[MU] - 1) : (coord == 0);
  pr = 1;
  pi = 0;
  if (edge) {
    pr = (A)(DIR > 0 ? g.fwd_re[MU] : g.bwd_re[MU]);
    pi = (A)(DIR > 0 ? g.fwd_im[MU] : g.bwd_im[MU]);
  }
  if (MU == 3 && DIR < 0 && g.bc == BC_SF && c.t == 1) {
    pr = 0;
    pi = 0;
  }
  return !(pr == (A)0 && pi == (A)0);
}

// the link of a hop (neighbour index sn)
template <int MU, int DIR, int NR, typename SG, typename SI>
__device__ inline void link_fetch(HopOperands<NR, SG, SI>& f, const HopLaunch& a, int p, int s, int sn) {
  const KGeom& g = a.g;
  const int ne = a.two_row ? 6 : 9;                // stored complex per link
  const size_t par = (size_t)4 * ne * g.V2p;      // one parity of the link field
  const SG* Ub = static_cast<const SG*>(a.U);
  const SG* up = (DIR > 0) ? Ub + p * par + tix(s, 4 * ne) + MU * ne * kTile
                           : Ub + (1 - p) * par + tix(sn, 4 * ne) + MU * ne * kTile;
#pragma unroll
  for (int e = 0; e < 6; ++e) f.u[e] = a.cached_gauge ? raw_ld(up + e * kTile) : raw_ld_nt(up + e * kTile);
  if (!a.two_row) {
#pragma unroll
    for (int e = 6; e < 9; ++e) f.u[e] = a.cached_gauge ? raw_ld(up + e * kTile) : raw_ld_nt(up + e * kTile);
  }
}

template <int MU, int DIR, int NR, typename SG, typename SI>
__device__ inline void hop_fetch(HopOperands<NR, SG, SI>& f, const HopLaunch& a, const SI* yb, int p, int s,
                                 const Coord& c, int rhs0) {
  const int sn = nb_index(a.g, s, c, MU, DIR);
  link_fetch<MU, DIR>(f, a, p, s, sn);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const SI* yp = yb + (size_t)(rhs0 + r) * a.y_rs + tix(sn, 12);
#pragma unroll
    for (int k = 0; k < 12; ++k) f.y[r][k] = raw_ld(yp + k * kTile);
  }
}

template <int NR, typename A, typename SG, typename SI>
__device__ inline void hop_link(cpx<A> (&U)[9], const HopOperands<NR, SG, SI>& f, const HopLaunch& a) {
#pragma unroll
  for (int e = 0; e < 6; ++e) U[e] = widen<A>(f.u[e]);
  if (a.two_row) {
    su3_third_row(U);
  } else {
#pragma unroll
    for (int e = 6; e < 9; ++e) U[e] = widen<A>(f.u[e]);
  }
}

// w = ph U h (forward) or ph U^+ h (backward), h the projected half spinor of y
template <int MU, int DIR, typename A, typename SI>
__device__ inline void hop_half(const cpx<A> (&U)[9], const SI (&y)[12], bool edge, A pr, A pi, cpx<A> (&w)[2][3]) {
  cpx<A> psi[4][3];
#pragma unroll
  for (int k = 0; k < 12; ++k) psi[k / 3][k % 3] = widen<A>(y[k]);
  cpx<A> h[2][3];
  spin_project<MU, DIR>(psi, h);
  if (DIR > 0) su3_mul(U, h, w);
  else su3_dag_mul(U, h, w);
  if (edge) {
    const cpx<A> ph = {pr, pi};
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int a2 = 0; a2 < 3; ++a2) w[q][a2] = cmul(ph, w[q][a2]);
  }
}

template <int MU, int DIR, int NR, typename A, typename SG, typename SI>
__device__ inline void hop_apply(cpx<A> (&acc)[NR][4][3], const HopOperands<NR, SG, SI>& f, const HopLaunch& a,
                                 const Coord& c) {
  bool edge;
  A pr, pi;
  if (!hop_phase<MU, DIR, A>(a.g, c, edge, pr, pi)) return;
  cpx<A> U[9];
  hop_link(U, f, a);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    cpx<A> w[2][3];
    hop_half<MU, DIR>(U, f.y[r], edge, pr, pi, w);
    spin_accumulate<MU, DIR>(acc[r], w);
  }
}

// Hop k of the eight: direction k / 2, forward for even k.
template <int K, int NR, typename SG, typename SI>
__device__ inline void fetch_k(HopOperands<NR, SG, SI>& f, const HopLaunch& a, const SI* yb, int p, int s,
                               const Coord& c, int rhs0) {
  hop_fetch<K / 2, (K & 1) ? -1 : 1, NR, SG, SI>(f, a, yb, p, s, c, rhs0);
}

// Hops K .. K1-1 in order, one hop ahead: the loads of hop k+1 are issued
// before the arithmetic of hop k (f[k & 1] holds hop k).  The accumulation
// order is that of the plain sequence.
template <int K, int K1, int NR, typename A, typename SG, typename SI>
__device__ inline void hops_ahead(cpx<A> (&acc)[NR][4][3], HopOperands<NR, SG, SI> (&f)[2], const HopLaunch& a,
                                  const SI* yb, int p, int s, const Coord& c, int rhs0) {
  if constexpr (K + 1 < K1) fetch_k<K + 1>(f[(K + 1) & 1], a, yb, p, s, c, rhs0);
  hop_apply<K / 2, (K & 1) ? -1 : 1, NR, A, SG, SI>(acc, f[K & 1], a, c);
  if constexpr (K + 1 < K1) hops_ahead<K + 1, K1>(acc, f, a, yb, p, s, c, rhs0);
}

// Hops K0 .. K1-1 accumulated into acc.  With AHEAD the loads run one hop
// ahead of the arithmetic (two hops' operands live in registers); without,
// each hop loads and computes in turn and a cut hop loads nothing.
template <bool AHEAD, int K0, int K1, int NR, typename A, typename SG, typename SI>
__device__ inline void hop_range(cpx<A> (&acc)[NR][4][3], const HopLaunch& a, const SI* yb, int p, int s,
                                 const Coord& c, int rhs0) {
  if constexpr (AHEAD) {
    HopOperands<NR, SG, SI> f[2];
    fetch_k<K0>(f[K0 & 1], a, yb, p, s, c, rhs0);
    hops_ahead<K0, K1>(acc, f, a, yb, p, s, c, rhs0);
  } else {
    HopOperands<NR, SG, SI> f;
    bool edge;
    A pr, pi;
    if (hop_phase<K0 / 2, (K0 & 1) ? -1 : 1, A>(a.g, c, edge, pr, pi)) {
      fetch_k<K0>(f, a, yb, p, s, c, rhs0);
      hop_apply<K0 / 2, (K0 & 1) ? -1 : 1, NR, A, SG, SI>(acc, f, a, c);
    }
    if constexpr (K0 + 1 < K1) hop_range<false, K0 + 1, K1, NR, A, SG, SI>(acc, a, yb, p, s, c, rhs0);
  }
}

// Loads one hop ahead where one hop's raw operands take at most 48 registers
// per lane (BF16 with up to 3 rhs per thread, FP32 with one): the
// reduced-precision multi-rhs launches are latency-bound, and FP64 would
// give up too much occupancy.
template <int NR, typename SG, typename SI>
constexpr bool kHopAhead = 9 * sizeof(SG) + 12 * NR * sizeof(SI) <= 192;

// out6 += i m in6 (m = +-mu: the twisted-mass term of one chirality block)
template <typename A>
__device__ inline void add_tm(A m, const cpx<A> (&in6)[6], cpx<A> (&o6)[6]) {
#pragma unroll
  for (int i = 0; i < 6; ++i) o6[i] = {o6[i].re - m * in6[i].im, o6[i].im + m * in6[i].re};
}

template <typename A, typename SG>
__device__ inline void load_block(const SG* C, int blk, int s, bool cached, cpx<A> (&m)[18]) {
  const SG* c = C + tix(s, 36) + blk * 18 * kTile;
#pragma unroll
  for (int e = 0; e < 18; ++e) {
    auto v = cached ? ld(c + e * kTile) : ld_nt(c + e * kTile);
    m[e] = {(A)v.re, (A)v.im};
  }
}

// Mapping of the 1-D grid (nbs site blocks x ntiles rhs tiles) to work.
// Workgroup b runs on XCD b mod 8 (round-robin dispatch), each XCD with its
// own L2.
//   order 0: site block b mod nbs, rhs tile b / nbs (plain order);
//   order 1: XCD-contiguous: every XCD walks one contiguous range of
//            (site block, tile) pairs with the tiles of a site block adjacent;
//   order 2: XCD z-slabs: XCD x owns z-planes [x Lz/8, (x+1) Lz/8) for all t;
//            it walks, innermost first, the rhs tiles, the site blocks of a
//            (z, t) plane, the planes of its slab, then t.  The t-neighbours
//            of a site are then a slab plane (a few blocks) away.  Requires
//            Lz % 8 == 0 and a whole number of site blocks per (z, t) plane
//            (else order 1).
//   order 3: as 1, with the rhs tile outermost (the whole lattice per tile);
//   order 4: as 2, with the rhs tile outermost;
//   orders 5, 6: as 2 with slabs of 1 or 2 planes: XCD x sweeps t over the
//            planes z = d (x + 8 k) .. d (x + 8 k) + d - 1 for pass k = 0, 1,
//            ... (d = 1 or 2); a t-step then holds d/(Lz/8) of the data of
//            order 2, so the t-neighbours stay in L2 with many rhs per site,
//            at the price of z-neighbours in another XCD's L2 (6 requires
//            Lz % 16 == 0).
// Tile-inner orders read each link once for all tiles but need a reuse window
// holding all rhs; tile-outer orders read the links once per tile and keep
// the reuse window of a single tile.  A launch over both parities maps each parity like a one-parity launch (nb
// and nbs per parity); the parities alternate every round of eight
// workgroups (see hop_thread).
__device__ inline void block_order(const HopLaunch& a, int b, int nb, int nbs, int ntiles, int& sb, int& tile) {
  if (a.order == 0) {
    sb = b % nbs;
    tile = b / nbs;
    return;
  }
  const int x = b & 7, j = b >> 3;
  if (a.order == 3) {
    const int l = xcd_remap(b, nb);
    tile = l / nbs;
    sb = l % nbs;
    return;
  }
  if (a.order == 2 || a.order >= 4) {
    const int bpp = a.bpp, Lz = a.g.L[2];
    const int depth = (a.order == 5) ? 1 : (a.order == 6 ? 2 : (Lz >> 3));  // planes per slab
    int q;
    if (a.order != 4) {
      tile = j % ntiles;
      q = j / ntiles;
    } else {
      const int per_tile = nbs >> 3;  // site blocks per XCD and tile
      tile = j / per_tile;
      q = j % per_tile;
    }
    const int pb = q % bpp;
    q /= bpp;
    const int zl = q % depth;
    q /= depth;
    const int t = q % a.g.L[3];
    const int pass = q / a.g.L[3];  // 0 unless depth < Lz / 8
    sb = pb + bpp * (depth * (x + 8 * pass) + zl + Lz * t);
    return;
  }
  const int l = xcd_remap(b, nb);
  tile = l % ntiles;
  sb = l / ntiles;
}

// per-rhs block sum: lanes l and l' hold the same rhs iff l = l' mod RL
template <int RL>
__device__ inline double block_sum_rl(double v, double* sh) {
#pragma unroll
  for (int off = 32; off >= RL; off >>= 1) v += __shfl_xor(v, off, 64);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l < RL) sh[w * RL + l] = v;
  __syncthreads();
  double s = 0.0;
  if ((int)threadIdx.x < RL) {
#pragma unroll
    for (int i = 0; i < kHopBlock / 64; ++i) s += sh[i * RL + threadIdx.x];
  }
  return s;
}

// Everything a hop launch computes for one thread before the output stage:
// block decode, the 8 hops, the clover blocks.  Leaves the NR output
// spinors in v (scaled hop sum plus pre(z), then post), and the site, its
// coordinates and the rhs indices in the outputs.
struct ThreadSite {
  int sb, rhs_tile0, rhs0, s, p;
  int c0;  // first output component this thread owns (0, or 6 w when split)
  bool active, masked;
};

// Direction split (SPLIT; one rhs per thread only).  The two waves of a
// workgroup share its 64 sites: wave w computes the hops in directions 2w and
// 2w+1, the waves swap halves of their partial sums through LDS (xch, 2 x 6 x 64
// complex), and wave w then owns the six output components of chirality w
// (spins 2w, 2w+1) and their clover block.  Twice the waves per site at half
// the dependent loads each: for lattices too small to fill the GPU.  The hop
// sum is (x, y terms) + (z, t terms) instead of one chain over the eight, so
// results differ from the unsplit kernel in the last bits.
template <typename SG, typename SI, int PRE, int POST, bool HOP, int NR, int RL, bool SPLIT, bool TM, typename A>
__device__ inline bool hop_thread(const HopLaunch& a, ThreadSite& ts, cpx<A> (&v)[NR][12], cpx<A>* xch) {
  static_assert(!SPLIT || (NR == 1 && RL == 1 && HOP), "direction split: one rhs per thread");
  static_assert(!TM || (NR == 1 && RL == 1), "twisted mass: one rhs per thread");
  constexpr int SPB = SPLIT ? 64 : kHopBlock / RL;  // sites per block
  // wave index (uniform over the wave; only the split uses it)
  const int wv = SPLIT ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
  ts.c0 = 6 * wv;
  const KGeom& g = a.g;
  int tile, p = a.p_out, b = blockIdx.x, nb = gridDim.x, nbs = a.nbs;
  if (a.both) {
    // Both parities: with a whole number of XCD rounds per parity, the
    // parities alternate every XCD round (workgroups 8j .. 8j+7 run parity
    // j mod 2, one per XCD), so that each XCD handles parity-0 and parity-1
    // blocks of the same sites together and the links that a parity-1 site
    // reads backward (stored with its parity-0 neighbour) were just read
    // forward by the parity-0 block, and are L2 hits; otherwise parity 0
    // takes the first half of the grid and parity 1 the second.
    nb >>= 1;
    nbs >>= 1;
    if ((nb & 7) == 0) {
      const int j = b >> 3;
      p = j & 1;
      b = ((j >> 1) << 3) | (b & 7);
    } else {
      p = (b >= nb) ? 1 : 0;
      b -= p * nb;
    }
  }
  int bx;  // site block within the parity
  block_order(a, b, nb, nbs, a.nrhs / (NR * RL), bx, tile);
  ts.sb = p * nbs + bx;  // partial-sum slot
  const int lane_r = (RL > 1) ? (int)(threadIdx.x % RL) : 0;
  ts.rhs_tile0 = tile * NR * RL;
  ts.rhs0 = ts.rhs_tile0 + lane_r * NR;  // this lane's first rhs
  if (a.done) {
    bool all = true;
    for (int r = 0; r < NR * RL; ++r)
      all = all && (a.done[(ts.rhs_tile0 + r) * (int)(sizeof(CGState) / sizeof(int))] != 0);
    if (all) return false;
  }
  ts.p = p;
  const int s = bx * SPB + (SPLIT ? (int)(threadIdx.x & 63) : (int)(threadIdx.x / RL));
  ts.s = s;
  ts.active = s < g.V2;
  const SI* yb = static_cast<const SI*>(a.y);
  const SI* zb = static_cast<const SI*>(a.z);
  const SG* cpre = static_cast<const SG*>(a.Cpre);
  if (a.both) {
    yb += (1 - p) * a.par_stride;
    if (zb) zb += p * a.par_stride;
    if (cpre) cpre += p * a.cpre_par;
  }
  const int rhs0 = ts.rhs0;

  cpx<A> acc[NR][4][3];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int b = 0; b < 3; ++b) acc[r][q][b] = {(A)0, (A)0};

  Coord c;
  c.t = 0;
  if (ts.active) {
    c = site_coord(g, s, p);
    if (HOP) {
      constexpr bool AH = kHopAhead<NR, SG, SI>;
      if (!SPLIT) {
        hop_range<AH, 0, 8, NR, A, SG, SI>(acc, a, yb, p, s, c, rhs0);
      } else if (wv == 0) {
        hop_range<AH, 0, 4, NR, A, SG, SI>(acc, a, yb, p, s, c, rhs0);
      } else {
        hop_range<AH, 4, 8, NR, A, SG, SI>(acc, a, yb, p, s, c, rhs0);
      }
    }
  }
  ts.masked = (g.bc == BC_SF) && (c.t == 0);
  const A scale = (A)a.scale;

  if constexpr (SPLIT) {
    // region 0 of xch receives wave 1's spins 0, 1 (for wave 0), region 1
    // wave 0's spins 2, 3 (for wave 1); every thread of the workgroup gets here
    const int l = threadIdx.x & 63;
    if (wv == 0) {
#pragma unroll
      for (int k = 0; k < 6; ++k) xch[(6 + k) * 64 + l] = acc[0][2 + k / 3][k % 3];
    } else {
#pragma unroll
      for (int k = 0; k < 6; ++k) xch[k * 64 + l] = acc[0][k / 3][k % 3];
    }
    __syncthreads();
    if (wv == 0) {
#pragma unroll
      for (int k = 0; k < 6; ++k) v[0][k] = cscale(scale, cadd(acc[0][k / 3][k % 3], xch[k * 64 + l]));
    } else {
#pragma unroll
      for (int k = 0; k < 6; ++k)
        v[0][k] = cscale(scale, cadd(xch[(6 + k) * 64 + l], acc[0][2 + k / 3][k % 3]));
    }
    if (ts.active && PRE != PRE_NONE) {
      cpx<A> Cm[18];
      if (PRE == PRE_CLOV) load_block(cpre, wv, s, a.cached_gauge != 0, Cm);
      const SI* zp = zb + (size_t)rhs0 * a.z_rs + tix(s, 12) + 6 * wv * kTile;
      cpx<A> in6[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        auto t = ld(zp + i * kTile);
        in6[i] = {(A)t.re, (A)t.im};
      }
      if (PRE == PRE_IDENT) {
#pragma unroll
        for (int i = 0; i < 6; ++i) v[0][i] = cadd(v[0][i], in6[i]);
      } else {
        cpx<A> o6[6];
        herm6_mul(Cm, in6, o6);
        if constexpr (TM) add_tm((A)(wv == 0 ? a.tm_mu : -a.tm_mu), in6, o6);
#pragma unroll
        for (int i = 0; i < 6; ++i) v[0][i] = cadd(v[0][i], o6[i]);
      }
    }
    if (ts.active && POST == POST_CLOV) {
      cpx<A> in6[6], o6[6], Ci[18];
#pragma unroll
      for (int i = 0; i < 6; ++i) in6[i] = v[0][i];
      if constexpr (TM) {  // (A + i m)^{-1} = Q^{-1} (A - i m), m = tm_mu g5
        load_block(static_cast<const SG*>(a.Ctm), wv, s, a.cached_gauge != 0, Ci);
        herm6_mul(Ci, in6, o6);
        add_tm((A)(wv == 0 ? -a.tm_mu : a.tm_mu), in6, o6);
#pragma unroll
        for (int i = 0; i < 6; ++i) in6[i] = o6[i];
      }
      load_block(static_cast<const SG*>(a.Cpost), wv, s, a.cached_gauge != 0, Ci);
      herm6_mul(Ci, in6, o6);
#pragma unroll
      for (int i = 0; i < 6; ++i) v[0][i] = o6[i];
    }
    if (a.g5 && wv == 1) {
#pragma unroll
      for (int k = 0; k < 6; ++k) v[0][k] = {-v[0][k].re, -v[0][k].im};
    }
    if (ts.masked) {
#pragma unroll
      for (int k = 0; k < 6; ++k) v[0][k] = {(A)0, (A)0};
    }
    return true;
  }

#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int k = 0; k < 12; ++k) v[r][k] = cscale(scale, acc[r][k / 3][k % 3]);
  if (ts.active && PRE != PRE_NONE) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      cpx<A> Cm[18];
      if (PRE == PRE_CLOV) load_block(cpre, b, s, a.cached_gauge != 0, Cm);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const SI* zp = zb + (size_t)(rhs0 + r) * a.z_rs + tix(s, 12);
        cpx<A> in6[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          auto t = ld(zp + (6 * b + i) * kTile);
          in6[i] = {(A)t.re, (A)t.im};
        }
        if (PRE == PRE_IDENT) {
#pragma unroll
          for (int i = 0; i < 6; ++i) v[r][6 * b + i] = cadd(v[r][6 * b + i], in6[i]);
        } else {
          cpx<A> o6[6];
          herm6_mul(Cm, in6, o6);
          if constexpr (TM) add_tm((A)(b == 0 ? a.tm_mu : -a.tm_mu), in6, o6);
#pragma unroll
          for (int i = 0; i < 6; ++i) v[r][6 * b + i] = cadd(v[r][6 * b + i], o6[i]);
        }
      }
    }
  }
  if (TM && ts.active && POST == POST_CLOV) {
    // twisted mass: (A + i m)^{-1} = Q^{-1} (A - i m) per chirality
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      {
        cpx<A> Cm[18];
        load_block(static_cast<const SG*>(a.Ctm), b, s, a.cached_gauge != 0, Cm);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          cpx<A> in6[6], o6[6];
#pragma unroll
          for (int i = 0; i < 6; ++i) in6[i] = v[r][6 * b + i];
          herm6_mul(Cm, in6, o6);
          add_tm((A)(b == 0 ? -a.tm_mu : a.tm_mu), in6, o6);
#pragma unroll
          for (int i = 0; i < 6; ++i) v[r][6 * b + i] = o6[i];
        }
      }
      cpx<A> Ci[18];
      load_block(static_cast<const SG*>(a.Cpost), b, s, a.cached_gauge != 0, Ci);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        cpx<A> in6[6], o6[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) in6[i] = v[r][6 * b + i];
        herm6_mul(Ci, in6, o6);
#pragma unroll
        for (int i = 0; i < 6; ++i) v[r][6 * b + i] = o6[i];
      }
    }
  } else if (ts.active && POST == POST_CLOV) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      cpx<A> Ci[18];
      load_block(static_cast<const SG*>(a.Cpost), b, s, a.cached_gauge != 0, Ci);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        cpx<A> in6[6], o6[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) in6[i] = v[r][6 * b + i];
        herm6_mul(Ci, in6, o6);
#pragma unroll
        for (int i = 0; i < 6; ++i) v[r][6 * b + i] = o6[i];
      }
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (a.g5) {
#pragma unroll
      for (int k = 6; k < 12; ++k) v[r][k] = {-v[r][k].re, -v[r][k].im};
    }
    if (ts.masked) {
#pragma unroll
      for (int k = 0; k < 12; ++k) v[r][k] = {(A)0, (A)0};
    }
  }
  return true;
}

// alpha = rr / pAp for the rhs this workgroup owns (see HopLaunch::alpha_cg):
// a fixed-order sum (thread-strided partial sums, wavefront butterfly, the
// waves in order)
__device__ inline void fused_alpha(const HopLaunch& a, double* sh) {
  for (int r = blockIdx.x; r < a.nrhs; r += gridDim.x) {
    CGState& c = a.alpha_cg[r];
    if (c.done) {  // uniform over the workgroup
      if (a.alpha_slot >= 0 && threadIdx.x == 0) c.alpha_w[a.alpha_slot] = 0.0;
      continue;
    }
    const double* p = a.alpha_parts + (size_t)r * parts_stride(a.alpha_nparts);
    double acc = 0.0;
    for (int i = threadIdx.x; i < parts_count(a.alpha_nparts); i += kHopBlock) acc += parts_at(p, a.alpha_nparts, i);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double v = 0.0;
      for (int w = 0; w < kHopBlock / 64; ++w) v += sh[w];  // waves in order
      c.pAp = v;
      c.alpha = (v > 0.0) ? c.rr / v : 0.0;
      c.rr_prev = c.rr;
      if (a.alpha_slot >= 0) c.alpha_w[a.alpha_slot] = c.alpha;
    }
  }
  __syncthreads();
}

// Canonical output of k_hop (FP64): the NC components of each of a wave's 64
// sites pass through LDS (a pitch of NC + 1 complex keeps the 16-byte accesses
// free of bank conflicts) and leave as contiguous runs of NC 16-byte words per
// site, instead of an internal vector that a second pass reads back: Dw at
// 32^3x64 from canonical to canonical 1028 -> 863 us, of 12 fields on 16^3x32 525
// -> 407 us.
template <int NC>
__device__ inline void canon_store(const HopLaunch& a, const cpx<double> (&v)[12], int p, int s, int rhs, int c0,
                                   double2* sh) {
  const KGeom& g = a.g;
  const int l = threadIdx.x & 63;
  double2* w = sh + (threadIdx.x >> 6) * 64 * (NC + 1);
#pragma unroll
  for (int k = 0; k < NC; ++k) w[l * (NC + 1) + k] = make_double2(v[k].re, v[k].im);
  const Coord c = site_coord(g, s < g.V2 ? s : 0, p);
  // this lane's site as an offset into the rhs's field (-1: padding)
  const int own = s < g.V2 ? 2 * s + (c.x & 1) : -1;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  double2* base = a.cout + (size_t)rhs * 24 * g.V2;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int idx = i * 64 + l, site = idx / NC, k = idx % NC;
    const int lex = __shfl(own, site, 64);
    if (lex < 0) continue;
    const double2 t = w[site * (NC + 1) + k];
    const nt_d2 tv = {t.x, t.y}, zero = {0.0, 0.0};
    __builtin_nontemporal_store(tv, reinterpret_cast<nt_d2*>(base + (size_t)lex * 12 + c0 + k));
    if (a.cout_zero)
      __builtin_nontemporal_store(zero, reinterpret_cast<nt_d2*>(base + (size_t)(lex ^ 1) * 12 + c0 + k));
  }
  // the next rhs overwrites the LDS
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
static unsigned canon_lds(bool split) { return (kHopBlock / 64) * 64 * (split ? 7 : 13) * (unsigned)sizeof(double2); }

template <typename SG, typename SI, typename SO, int PRE, int POST, bool HOP, int NR, int RL, bool SPLIT, bool TM,
          bool CANON = false>
__global__ __launch_bounds__(kHopBlock) void k_hop(const HopLaunch a) {
  static_assert(!CANON || (RL == 1 && std::is_same<SO, double2>::value), "canonical output: FP64, one lane per site");
  using A = typename StoreTraits<SG>::acc;
  constexpr int NC = SPLIT ? 6 : 12;  // output components per thread
  __shared__ double red[(kHopBlock / 64) * RL > 4 ? (kHopBlock / 64) * RL : 4];
  __shared__ cpx<A> xch[SPLIT ? 2 * 6 * 64 : 1];
  if (a.alpha_cg) fused_alpha(a, red);
  ThreadSite ts;
  cpx<A> v[NR][12];
  if (!hop_thread<SG, SI, PRE, POST, HOP, NR, RL, SPLIT, TM>(a, ts, v, xch)) return;
  if constexpr (CANON) {
    extern __shared__ double2 canon_sh[];
#pragma unroll
    for (int r = 0; r < NR; ++r) canon_store<NC>(a, v[r], ts.p, ts.s, ts.rhs0 + r, ts.c0, canon_sh);
    return;
  }
  // launches that may form a residual (HopLaunch::res)
  constexpr bool RES = PRE == PRE_CLOV && POST == POST_NONE && std::is_same<SG, double2>::value;
  SO* ob = static_cast<SO*>(a.out);
  if (a.both && ob) ob += ts.p * a.par_stride;
  // padding sites of the last tile (inactive, v = 0) are written too, so
  // every output vector holds zeros there
  const bool store = ts.s < a.g.V2p;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    double nrm = 0.0;
    if (store) {
      const size_t site = tix(ts.s, 12) + ts.c0 * kTile;
      bool put = !a.masked_out || a.done[(ts.rhs0 + r) * (int)(sizeof(CGState) / sizeof(int))] == 0;
      if constexpr (RES) {
        if (a.res) {  // uniform over the launch
          const double2* bp = a.res + (a.both ? ts.p * a.par_stride : 0) + (size_t)(ts.rhs0 + r) * a.res_rs + site;
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            const auto bv = ld(bp + k * kTile);
            v[r][k] = csub(bv, v[r][k]);
            if (a.res_g5 && ts.c0 + k >= 6) v[r][k] = {-v[r][k].re, -v[r][k].im};
          }
          if (a.out32) {
            float2* op = a.out32 + (size_t)(ts.rhs0 + r) * a.out32_rs + site;
#pragma unroll
            for (int k = 0; k < NC; ++k) st(op + k * kTile, v[r][k]);
          }
          put = put && ob != nullptr;
        }
      }
      if (put) {
        SO* op = ob + (size_t)(ts.rhs0 + r) * a.out_rs + site;
        if (a.nt_out) {
#pragma unroll
          for (int k = 0; k < NC; ++k) st_nt(op + k * kTile, v[r][k]);
        } else {
#pragma unroll
          for (int k = 0; k < NC; ++k) st(op + k * kTile, v[r][k]);
        }
      }
      if (a.partials) {
#pragma unroll
        for (int k = 0; k < NC; ++k) nrm += cnorm2(v[r][k]);
      }
    }
    if (a.partials) {
      const double bs = block_sum_rl<RL>(nrm, red);
      if ((int)threadIdx.x < RL)
        a.partials[(size_t)(ts.rhs_tile0 + (int)threadIdx.x * NR + r) * a.nbs + ts.sb] = bs;
    }
  }
}

// The last hop of a CG iteration fused with the vector update: with
// Ap = g5 (A_ee q + 1/2 H t) computed in registers, every rhs that is not done
// gets r -= alpha Ap (r of type SV) and the per-block |r|^2 partial.  Ap is
// never stored; x += alpha p is left to the flush of the deferred updates.
template <typename SG, typename SI, typename SV, int NR, int RL, bool SPLIT, bool TM>
__global__ __launch_bounds__(kHopBlock) void k_hop_xr(const HopLaunch a) {
  using A = typename StoreTraits<SG>::acc;
  using AV = typename StoreTraits<SV>::acc;
  constexpr int NC = SPLIT ? 6 : 12;  // output components per thread
  __shared__ double red[(kHopBlock / 64) * RL];
  __shared__ cpx<A> xch[SPLIT ? 2 * 6 * 64 : 1];
  ThreadSite ts;
  cpx<A> v[NR][12];
  if (!hop_thread<SG, SI, PRE_CLOV, POST_NONE, true, NR, RL, SPLIT, TM>(a, ts, v, xch)) return;
  SV* rb = static_cast<SV*>(a.xr_r);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int q = ts.rhs0 + r;
    const CGState& cs = a.cg[q];
    double nrm = 0.0;
    if (ts.active && !cs.done) {
      const AV alpha = (AV)cs.alpha;
      const size_t o = (size_t)q * a.xr_rs + tix(ts.s, 12) + ts.c0 * kTile;
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        auto rv = ld(rb + o + k * kTile);
        rv.re -= alpha * (AV)v[r][k].re;
        rv.im -= alpha * (AV)v[r][k].im;
        st(rb + o + k * kTile, rv);
        nrm += cnorm2(rv);
      }
    }
    const double bs = block_sum_rl<RL>(nrm, red);
    if ((int)threadIdx.x < RL)
      a.partials[(size_t)(ts.rhs_tile0 + (int)threadIdx.x * NR + r) * a.nbs + ts.sb] = bs;
  }
}

// ---------------------------------------------------------------------------
// Small launches: one site and rhs spread over eight waves.
//
// With too few sites to hide latency, the time of a launch is the length of
// one thread's chain: eight rounds of loads and SU(3) products, then the
// clover blocks.  Here a workgroup of eight waves owns 64 sites and one rhs:
// wave d computes hop d alone (one round of loads) and leaves its two-spin
// result in LDS; then each of six waves owns two output components (colour
// w % 3 of both spins of chirality w / 3), adds the eight hops in the order of
// the one-thread chain and applies its two rows of the clover block, whose
// loads were issued before the hops.  Every sum is formed by the same
// operations in the same order as in k_hop, so results agree bit for bit: a
// launch's size never shows in them (the |out|^2 partials, per 64 sites, are
// paired by their readers, see parts_count).  Modes are run-time uniform: the
// launch is bound by latency, not by issue.  alpha has workgroups of its own.
// 8^4, one rhs: 10.1 -> 5.9 us per FP64 hop, 9.5 -> 5.5 FP32, 7.6 -> 4.7 BF16.
constexpr int kSpreadSites = 64;
constexpr int kSpreadBlock = 512;

// entry q of the reconstructed half spinor: component (chirality B, spin q)
// of the contribution of a hop whose two-spin result is w (one colour each)
template <int MU, int DIR, typename A>
__device__ inline cpx<A> spread_add(cpx<A> acc, int b, int q, const cpx<A>* w, int col, int l) {
  // upper chirality: w_q itself; lower: +-1 or +-i times w_{1-q} (x, y) or w_q (z, t)
  const int sp = (b == 1 && MU < 2) ? 1 - q : q;
  const cpx<A> v = w[(3 * sp + col) * kSpreadSites + l];
  if (b == 0) return cadd(acc, v);
  // sign of the forward hop: x: -i, -i; y: -, +; z: -i, +i; t: +, +
  const bool neg = (DIR > 0) == (MU == 0 || (MU < 3 && q == 0));
  if (MU == 0 || MU == 2) return neg ? csub_i(acc, v) : cadd_i(acc, v);
  return neg ? csub(acc, v) : cadd(acc, v);
}

// component k of a canonical field's site, rounded to the storage type of an
// internal vector (as the layout conversion rounds it)
template <typename SI>
__device__ inline SI canon_ld(const double2* site, int k, bool g5) {
  double2 v = site[k];
  if (g5 && k >= 6) v = make_double2(-v.x, -v.y);
  SI t;
  st(&t, cpx<double>{v.x, v.y});
  return t;
}

// PF: the operand is r + beta y (HopLaunch::pf_r)
template <int K, bool CANON, bool PF, typename A, typename SG, typename SI>
__device__ inline void spread_hop(const HopLaunch& a, const SI* yb, int p, int s, const Coord& c, int rhs, cpx<A>* w,
                                  int l, const double* rr2) {
  constexpr int MU = K / 2, DIR = (K & 1) ? -1 : 1;
  bool edge;
  A pr, pi;
  cpx<A> v[2][3];
  if (hop_phase<MU, DIR, A>(a.g, c, edge, pr, pi)) {
    HopOperands<1, SG, SI> f;
    bool internal = true;
    if constexpr (CANON) {
      if (a.cy) {  // uniform over the launch
        internal = false;
        const int sn = nb_index(a.g, s, c, MU, DIR);
        link_fetch<MU, DIR>(f, a, p, s, sn);
        const double2* yp = a.cy + ((size_t)rhs * 2 * a.g.V2 + 2 * sn + ((c.x + (MU == 0 ? 1 : 0)) & 1)) * 12;
#pragma unroll
        for (int k = 0; k < 12; ++k) f.y[0][k] = canon_ld<SI>(yp, k, a.g5_in);
      }
    }
    if (internal) fetch_k<K>(f, a, yb, p, s, c, rhs);
    if constexpr (PF) {
      using SR = std::conditional_t<std::is_same<SI, double2>::value, double2, float2>;
      const int sn = nb_index(a.g, s, c, MU, DIR);
      const SR* rp = static_cast<const SR*>(a.pf_r) + (size_t)rhs * a.pf_rs + tix(sn, 12);
      cpx<A> r[12];
#pragma unroll
      for (int k = 0; k < 12; ++k) r[k] = ld(rp + k * kTile);
      const A beta = (A)(rr2[1] > 0.0 ? rr2[0] / rr2[1] : 0.0);
#pragma unroll
      for (int k = 0; k < 12; ++k) st(&f.y[0][k], p_next(beta, r[k], widen<A>(f.y[0][k])));
    }
    cpx<A> U[9];
    hop_link(U, f, a);
    hop_half<MU, DIR>(U, f.y[0], edge, pr, pi, v);
  } else {
#pragma unroll
    for (int e = 0; e < 6; ++e) v[e / 3][e % 3] = {(A)0, (A)0};
  }
#pragma unroll
  for (int e = 0; e < 6; ++e) w[(6 * K + e) * kSpreadSites + l] = v[e / 3][e % 3];
}

// row i of a packed Hermitian 6x6 block: the six elements of row i, the
// stored lower-triangle entry for each column and the diagonal pair
template <typename A, typename SG>
__device__ inline void load_row(const SG* C, int blk, int i, int s, cpx<A> (&m)[6]) {
  const SG* c = C + tix(s, 36) + blk * 18 * kTile;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const int e = j == i ? (i >> 1) : (j < i ? 3 + i * (i - 1) / 2 + j : 3 + j * (j - 1) / 2 + i);
    const auto v = ld(c + e * kTile);
    m[j] = {(A)v.re, (A)v.im};
  }
}
// that row times v, in the order of herm6_mul
template <typename A>
__device__ inline cpx<A> row_mul(const cpx<A> (&m)[6], int i, const cpx<A> (&v)[6]) {
  cpx<A> acc = {(A)0, (A)0};
#pragma unroll
  for (int j = 0; j < 6; ++j)
    if (j == i) {
      const A re = m[j].re, im = m[j].im;
      acc = cscale((i & 1) ? im : re, v[j]);
    }
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    if (j < i) acc = cmac(acc, m[j], v[j]);
    if (j > i) acc = cmacc(acc, m[j], v[j]);
  }
  return acc;
}

// CANON: input and output may be canonical fields (HopLaunch::cy, cz, cout),
// which saves a small operator application its two layout conversions.
// PF: applied to the updated search direction (HopLaunch::pf_r), which saves a
// small iteration the launch of the update (4.5 us eager, 1.6 us and its drain
// in a graph) for twelve more loads a lane and a barrier in the third hop:
// solves of 2^9 to 2^14 sites up to 5% (3516 -> 3330, 8714 -> 8580, 10941 ->
// 10600 us), 8^4 FP32 3885 both.
template <typename SG, typename SI, typename SO, bool XR, bool CANON, bool PF = false>
__global__ __launch_bounds__(kSpreadBlock) void k_hop_spread(const HopLaunch a) {
  using A = typename StoreTraits<SG>::acc;
  __shared__ __attribute__((aligned(16))) cpx<A> wls[8 * 6 * kSpreadSites];  // the hops; later the site vectors
  __shared__ double nls[12 * kSpreadSites];  // |component|^2 of the sites
  const KGeom& g = a.g;
  const int l = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nwork = a.nbs * a.nrhs;
  if ((int)blockIdx.x >= nwork) {  // the extra workgroups: alpha of one rhs each (see HopLaunch::alpha_cg)
    const int r = blockIdx.x - nwork;
    CGState& c = a.alpha_cg[r];
    if (c.done) {
      if (a.alpha_slot >= 0 && threadIdx.x == 0) c.alpha_w[a.alpha_slot] = 0.0;
      return;
    }
    if (a.beta_parts) {
      const double rr = wave_psum(a.beta_parts + (size_t)r * parts_stride(a.beta_nparts), a.beta_nparts);
      __syncthreads();  // every wave has read done
      if (threadIdx.x == 0) {
        beta_step(c, rr);
        nls[kHopBlock / 64] = c.done;
      }
      __syncthreads();
      if (nls[kHopBlock / 64] != 0.0) {
        if (a.alpha_slot >= 0 && threadIdx.x == 0) c.alpha_w[a.alpha_slot] = 0.0;
        return;
      }
    }
    const double* pp = a.alpha_parts + (size_t)r * parts_stride(a.alpha_nparts);
    double acc = 0.0;  // as in fused_alpha: the first kHopBlock threads
    if (w < kHopBlock / 64)
      for (int i = threadIdx.x; i < parts_count(a.alpha_nparts); i += kHopBlock) acc += parts_at(pp, a.alpha_nparts, i);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (l == 0 && w < kHopBlock / 64) nls[w] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double v = 0.0;
      for (int k = 0; k < kHopBlock / 64; ++k) v += nls[k];  // waves in order
      c.pAp = v;
      c.alpha = (v > 0.0) ? c.rr / v : 0.0;
      c.rr_prev = c.rr;
      if (a.alpha_slot >= 0) c.alpha_w[a.alpha_slot] = c.alpha;
    }
    return;
  }
  const int lb = xcd_remap(blockIdx.x, nwork);  // the rhs of a site block side by side on one XCD
  const int rhs = lb % a.nrhs, sb = lb / a.nrhs;
  if (a.beta_parts) {
    // this launch's beta step may set the flag: one read decides for the workgroup
    if (threadIdx.x == 0) nls[0] = a.done[rhs * (int)(sizeof(CGState) / sizeof(int))];
    __syncthreads();
    if (nls[0] != 0.0) return;
  } else if (a.done && a.done[rhs * (int)(sizeof(CGState) / sizeof(int))] != 0) {
    return;
  }
  const int p = a.both ? (sb & 1) : a.p_out;
  const int bx = a.both ? sb >> 1 : sb, s = bx * kSpreadSites + l;  // site block of the parity, site
  const bool active = s < g.V2;
  const SI* yb = static_cast<const SI*>(a.y);
  const SI* zb = static_cast<const SI*>(a.z);
  const SG* cpre = static_cast<const SG*>(a.Cpre);
  if (a.both) {
    yb += (1 - p) * a.par_stride;
    if (zb) zb += p * a.par_stride;
    if (cpre) cpre += p * a.cpre_par;
  }
  const Coord c = site_coord(g, active ? s : 0, p);
  // this wave's output components: rows col and 3 + col of chirality b
  const int b = w / 3, col = w % 3;
  const bool owner = w < 6;
  const bool tm = a.tm_post != 0 || a.tm_mu != 0.0;
  // first clover product of the launch: A z before the hops, or the first matrix after them
  const SG* first = a.pre == PRE_CLOV ? cpre
                    : a.post == POST_CLOV ? static_cast<const SG*>(tm ? a.Ctm : a.Cpost) : nullptr;
  cpx<A> m0[6], m1[6], z[6];
  if (owner && active) {
    if (first) {
      load_row(first, b, col, s, m0);
      load_row(first, b, 3 + col, s, m1);
    }
    if (a.pre != PRE_NONE) {
      bool internal = true;
      if constexpr (CANON) {
        if (a.cz) {
          internal = false;
          const double2* zp = a.cz + ((size_t)rhs * 2 * g.V2 + 2 * s + (c.x & 1)) * 12 + 6 * b;
          const bool neg = a.g5_in && b == 1;
#pragma unroll
          for (int i = 0; i < 6; ++i) {
            const SI t = canon_ld<SI>(zp, i, false);
            z[i] = widen<A>(t);
            if (neg) z[i] = {-z[i].re, -z[i].im};
          }
        }
      }
      if (internal) {
        const SI* zp = zb + (size_t)rhs * a.z_rs + tix(s, 12) + 6 * b * kTile;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          const auto t = ld(zp + i * kTile);
          z[i] = {(A)t.re, (A)t.im};
        }
      }
    }
  }
  // |r|^2 and the one before, for beta
  double rr2[2] = {0.0, 0.0};
  if constexpr (PF) {
    using SR = std::conditional_t<std::is_same<SI, double2>::value, double2, float2>;
    rr2[1] = a.pf_cg[rhs].rr_prev;
    // this site's components of the new direction (input parity, same index)
    const size_t o = tix(s, 12) + (6 * b + col) * kTile;
    cpx<A> pv[2], rv[2];
    if (owner && active) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        pv[q] = ld(yb + (size_t)rhs * a.y_rs + o + 3 * q * kTile);
        rv[q] = ld(static_cast<const SR*>(a.pf_r) + (size_t)rhs * a.pf_rs + o + 3 * q * kTile);
      }
    }
    rr2[0] = wave_psum(a.pf_parts + (size_t)rhs * parts_stride(a.pf_nparts), a.pf_nparts);
    if (owner && active) {
      const A beta = (A)(rr2[1] > 0.0 ? rr2[0] / rr2[1] : 0.0);
#pragma unroll
      for (int q = 0; q < 2; ++q)
        st(static_cast<SI*>(a.pf_next) + (size_t)rhs * a.pf_rs + o + 3 * q * kTile, p_next(beta, rv[q], pv[q]));
    }
  }
  if (active) {
    switch (w) {
      case 0: spread_hop<0, CANON, PF, A, SG, SI>(a, yb, p, s, c, rhs, wls, l, rr2); break;
      case 1: spread_hop<1, CANON, PF, A, SG, SI>(a, yb, p, s, c, rhs, wls, l, rr2); break;
      case 2: spread_hop<2, CANON, PF, A, SG, SI>(a, yb, p, s, c, rhs, wls, l, rr2); break;
      case 3: spread_hop<3, CANON, PF, A, SG, SI>(a, yb, p, s, c, rhs, wls, l, rr2); break;
      case 4: spread_hop<4, CANON, PF, A, SG, SI>(a, yb, p, s, c, rhs, wls, l, rr2); break;
      case 5: spread_hop<5, CANON, PF, A, SG, SI>(a, yb, p, s, c, rhs, wls, l, rr2); break;
      case 6: spread_hop<6, CANON, PF, A, SG, SI>(a, yb, p, s, c, rhs, wls, l, rr2); break;
      default: spread_hop<7, CANON, PF, A, SG, SI>(a, yb, p, s, c, rhs, wls, l, rr2); break;
    }
  }
  __syncthreads();
  cpx<A> v[2] = {{(A)0, (A)0}, {(A)0, (A)0}};
  if (owner && active) {
    const A scale = (A)a.scale;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      cpx<A> t = {(A)0, (A)0};
      t = spread_add<0, 1>(t, b, q, wls + 0 * 6 * kSpreadSites, col, l);
      t = spread_add<0, -1>(t, b, q, wls + 1 * 6 * kSpreadSites, col, l);
      t = spread_add<1, 1>(t, b, q, wls + 2 * 6 * kSpreadSites, col, l);
      t = spread_add<1, -1>(t, b, q, wls + 3 * 6 * kSpreadSites, col, l);
      t = spread_add<2, 1>(t, b, q, wls + 4 * 6 * kSpreadSites, col, l);
      t = spread_add<2, -1>(t, b, q, wls + 5 * 6 * kSpreadSites, col, l);
      t = spread_add<3, 1>(t, b, q, wls + 6 * 6 * kSpreadSites, col, l);
      t = spread_add<3, -1>(t, b, q, wls + 7 * 6 * kSpreadSites, col, l);
      v[q] = cscale(scale, t);
    }
    if (a.pre != PRE_NONE) {
      const auto pick = [col](A x, A y, A t) { return col == 0 ? x : (col == 1 ? y : t); };
      const cpx<A> z0 = {pick(z[0].re, z[1].re, z[2].re), pick(z[0].im, z[1].im, z[2].im)};
      const cpx<A> z1 = {pick(z[3].re, z[4].re, z[5].re), pick(z[3].im, z[4].im, z[5].im)};
      cpx<A> o0 = z0, o1 = z1;
      if (a.pre == PRE_CLOV) {
        o0 = row_mul(m0, col, z);
        o1 = row_mul(m1, 3 + col, z);
        if (tm) {
          const A m = (A)(b == 0 ? a.tm_mu : -a.tm_mu);
          o0 = {o0.re - m * z0.im, o0.im + m * z0.re};
          o1 = {o1.re - m * z1.im, o1.im + m * z1.re};
        }
      }
      v[0] = cadd(v[0], o0);
      v[1] = cadd(v[1], o1);
    }
  }
  if (a.post == POST_CLOV) {  // uniform over the launch
    // one or (twisted mass) two products; each needs the six components of the
    // chirality, which the other waves hold
    for (int step = tm ? 0 : 1; step < 2; ++step) {
      __syncthreads();  // wls is free
      if (owner) {
#pragma unroll
        for (int q = 0; q < 2; ++q) wls[(6 * b + 3 * q + col) * kSpreadSites + l] = v[q];
      }
      __syncthreads();
      if (owner && active) {
        cpx<A> in6[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) in6[i] = wls[(6 * b + i) * kSpreadSites + l];
        if (a.pre == PRE_CLOV || (tm && step == 1)) {
          const SG* C = static_cast<const SG*>(step == 0 ? a.Ctm : a.Cpost);
          load_row(C, b, col, s, m0);
          load_row(C, b, 3 + col, s, m1);
        }
        const cpx<A> o0 = row_mul(m0, col, in6), o1 = row_mul(m1, 3 + col, in6);
        if (step == 0) {  // (A + i m)^{-1} = Q^{-1} (A - i m), m = tm_mu g5
          const A m = (A)(b == 0 ? -a.tm_mu : a.tm_mu);
          const cpx<A> i0 = v[0], i1 = v[1];
          v[0] = {o0.re - m * i0.im, o0.im + m * i0.re};
          v[1] = {o1.re - m * i1.im, o1.im + m * i1.re};
        } else {
          v[0] = o0;
          v[1] = o1;
        }
      }
    }
  }
  double n2[2] = {0.0, 0.0};
  if (owner) {
    const bool masked = g.bc == BC_SF && c.t == 0;
    if (a.g5 && b == 1) {
#pragma unroll
      for (int q = 0; q < 2; ++q) v[q] = {-v[q].re, -v[q].im};
    }
    if (masked) {
#pragma unroll
      for (int q = 0; q < 2; ++q) v[q] = {(A)0, (A)0};
    }
    const size_t site = tix(s, 12) + (6 * b + col) * kTile;
    if constexpr (XR) {
      using AV = typename StoreTraits<SO>::acc;
      SO* rb = static_cast<SO*>(a.xr_r);
      const CGState& cs = a.cg[rhs];
      if (active && !cs.done) {
        const AV alpha = (AV)cs.alpha;
        const size_t o = (size_t)rhs * a.xr_rs + site;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          auto rv = ld(rb + o + 3 * q * kTile);
          rv.re -= alpha * (AV)v[q].re;
          rv.im -= alpha * (AV)v[q].im;
          st(rb + o + 3 * q * kTile, rv);
          n2[q] = cnorm2(rv);
        }
      }
    } else if (CANON && a.cout) {
      // through LDS below
    } else if (s < g.V2p) {  // padding sites (v = 0) too
      const long po = a.both ? p * a.par_stride : 0;
      if constexpr (std::is_same<SG, double2>::value) {
        if (a.res) {
          const double2* bp = a.res + po + (size_t)rhs * a.res_rs + site;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            v[q] = csub(ld(bp + 3 * q * kTile), v[q]);
            if (a.res_g5 && b == 1) v[q] = {-v[q].re, -v[q].im};
            if (a.out32) st(a.out32 + (size_t)rhs * a.out32_rs + site + 3 * q * kTile, v[q]);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {  // one rhs per workgroup: masked_out is the early exit above
        if (a.out) st(static_cast<SO*>(a.out) + po + (size_t)rhs * a.out_rs + site + 3 * q * kTile, v[q]);
        n2[q] = cnorm2(v[q]);
      }
    }
  }
  if constexpr (CANON) {
    if (a.cout) {
      // lane-per-site components to contiguous runs of 12 words per site; the
      // value is what the output storage type holds
      __syncthreads();
      static_assert(13 * kSpreadSites * sizeof(double2) <= sizeof(wls), "output staging");
      double2* sh = reinterpret_cast<double2*>(wls);
      if (owner) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          SO t;
          st(&t, v[q]);
          const auto r = ld(&t);
          sh[l * 13 + 6 * b + 3 * q + col] = make_double2((double)r.re, (double)r.im);
        }
      }
      __syncthreads();
      double2* base = a.cout + (size_t)rhs * 24 * g.V2;
      for (int idx = threadIdx.x; idx < 12 * kSpreadSites; idx += kSpreadBlock) {
        const int site = idx / 12, k = idx % 12, so = bx * kSpreadSites + site;
        if (so >= g.V2) break;
        const int lex = 2 * so + (site_coord(g, so, p).x & 1);
        base[(size_t)lex * 12 + k] = sh[site * 13 + k];
        if (a.cout_zero) base[(size_t)(lex ^ 1) * 12 + k] = make_double2(0.0, 0.0);
      }
      return;
    }
  }
  if (a.partials) {
    if (owner) {
#pragma unroll
      for (int q = 0; q < 2; ++q) nls[(6 * b + 3 * q + col) * kSpreadSites + l] = n2[q];
    }
    __syncthreads();
    if (w == 0) {  // the sum of one wave of k_hop
      double nrm = 0.0;
#pragma unroll
      for (int k = 0; k < 12; ++k) nrm += nls[k * kSpreadSites + l];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
      if (l == 0) {
        const int per = (a.nbs / (a.both ? 2 : 1) + 1) & ~1;  // slots per parity: whole pairs
        double* pt = a.partials + (size_t)rhs * (a.both ? 2 * per : per) + p * (a.both ? per : 0);
        pt[bx] = nrm;
        if (bx == a.nbs / (a.both ? 2 : 1) - 1 && (bx & 1) == 0) pt[bx + 1] = 0.0;
      }
    }
  }
}

static int sites_per_block(int rl, bool split = false) {
  return split ? 64 : kHopBlock / (rl < 1 ? 1 : rl);
}
// the direction split applies to launches with one rhs per thread only
static bool split_on(const HopLaunch& h) { return h.dir_split && h.nr_tile == 1 && h.rhs_lanes == 1; }
// twisted-mass kernels exist for one rhs per thread (the launch helpers of
// the library set nr_tile = rhs_lanes = 1 whenever mu != 0)
static bool tm_on(const HopLaunch& h) { return h.tm_post != 0 || h.tm_mu != 0.0; }

// Launches of k_hop_spread (a site and rhs is one thread of k_hop): those whose
// workgroups are all resident at once, one per CU in FP64 (183 registers), two in
// FP32 and BF16.  One more starts a second round that few CUs take part in.
// Measured as time of k_hop over time of k_hop_spread, by output sites x rhs:
// even-odd solves, one field / with a twisted mass: FP64 16384 1.32 / 1.34, 18432
// 0.97 / 0.95, 28672 0.93 / 0.92; FP32 32768 1.15 / 1.17, 36864 0.99 / 0.98, 45056
// 0.98 / 0.98; BF16 20480 1.13 / 1.14, 32768 1.13 / 1.14, 36864 0.96 / 0.94, 40960
// 0.95 / 0.91; twelve fields: FP64 30720 0.95, FP32 43008 0.92, BF16 30720 1.14,
// 43008 0.98; full-lattice solves 20480 0.96; Dw 20480 0.93.
// The caller's direction split sums in another order and keeps its own kernel, and
// so does a launch that asks for the general form: a workgroup of eight waves finds
// no place on a GPU that another stream's launches keep full.
constexpr long kCUs = 256;
static int spread_nblocks(const HopLaunch& h) {
  return (h.both ? 2 : 1) * ((h.g.V2 + kSpreadSites - 1) / kSpreadSites);
}
static long spread_workgroups(const HopLaunch& h) { return (long)spread_nblocks(h) * h.nrhs; }
static bool spread_on(const HopLaunch& h) {
  return h.hop && !h.general && !split_on(h) && spread_workgroups(h) <= (h.prec == P_F64 ? 1 : 2) * kCUs;
}

// Unused dynamic LDS that caps the workgroups resident per CU (160 KiB of LDS
// per CU, plus each workgroup's small static reduction array): level 1 -> 4,
// 2 -> 3, 3 -> 2 workgroups.  A smaller live set per XCD keeps more neighbour
// spinors in L2 when every site carries many rhs.
static unsigned lds_cap_bytes(int level) {
  switch (level) {
    case 1: return 39u << 10;
    case 2: return 53u << 10;
    case 3: return 63u << 10;
    default: return 0u;
  }
}

// most partial sums per rhs a launch of k_hop writes on V2 sites per parity: 4 rhs
// lanes (fewest sites per workgroup), or both parities split (a small launch
// writes at most 514: 512 workgroups, whole pairs per parity)
int hop_max_parts(long V2) {
  const long one = (V2 + sites_per_block(4) - 1) / sites_per_block(4);
  const long both = 2 * ((V2 + sites_per_block(1, true) - 1) / sites_per_block(1, true));
  return (int)(one > both ? one : both);
}

int hop_nblocks(const HopLaunch& h) {
  const int spb = sites_per_block(h.rhs_lanes, split_on(h));
  const int nb = (h.g.V2 + spb - 1) / spb;
  return h.both ? 2 * nb : nb;
}

// partial sums per rhs of a small launch, as a count of half sums (see parts_count): whole
// pairs for each parity
static int spread_nparts(const HopLaunch& h) {
  const int per = (h.g.V2 + kSpreadSites - 1) / kSpreadSites;
  return -(h.both ? 2 : 1) * ((per + 1) & ~1);
}

// The direction update is fused where a launch is small (spread_on) and every
// wave can sum the partials itself without a barrier (at most 64, 2^14 sites).
bool hop_fuses_p(const HopLaunch& h0) {
  HopLaunch h = h0;
  if (h.prec == P_F64) h.rhs_lanes = 1;
  return spread_on(h) && parts_count(spread_nparts(h)) <= 64;
}

// Canonical input is read site by site (192 contiguous bytes per lane, no
// coalescing over lanes), which pays while the launch is one round of a
// workgroup per CU (every small FP64 launch): Dw of 8^3x12 (12288 sites and
// fields) 11.7 us with the conversion, 9.8 without; 12^4 (20736) 19.7 and 19.2,
// and D^+ D there 31.5 and 33.2.
bool hop_reads_canonical(const HopLaunch& h0) {
  HopLaunch h = h0;
  if (h.prec == P_F64) h.rhs_lanes = 1;
  return spread_on(h) && spread_workgroups(h) <= kCUs;
}

template <typename SG, typename SI, typename SO, bool XR>
static hipError_t launch_spread(HopLaunch h, hipStream_t st) {
  h.nbs = spread_nblocks(h);
  const unsigned grid = (unsigned)h.nbs * (unsigned)h.nrhs + (h.alpha_cg ? (unsigned)h.nrhs : 0u);
  if constexpr (!XR && std::is_same<SI, SO>::value) {
    if (h.cy || h.cz || h.cout) {
      k_hop_spread<SG, SI, SO, false, true><<<grid, kSpreadBlock, 0, st>>>(h);
      return hipGetLastError();
    }
  }
  if (h.cy || h.cz || h.cout) return hipErrorInvalidValue;
  if (h.beta_parts && (parts_count(h.beta_nparts) > 64 || !h.done || !h.alpha_cg)) return hipErrorInvalidValue;
  if constexpr (!XR && std::is_same<SI, SO>::value) {
    if (h.pf_r) {
      if (parts_count(h.pf_nparts) > 64 || h.both || h.pre != PRE_NONE) return hipErrorInvalidValue;
      k_hop_spread<SG, SI, SO, false, false, true><<<grid, kSpreadBlock, 0, st>>>(h);
      return hipGetLastError();
    }
  }
  if (h.pf_r) return hipErrorInvalidValue;
  k_hop_spread<SG, SI, SO, XR, false><<<grid, kSpreadBlock, 0, st>>>(h);
  return hipGetLastError();
}

// An empty kernel that takes the registers (whole granules of eight) and, by its
// launch, the LDS of k_hop_spread.  Ending k_hop_spread itself early for a launch
// without sites cost every small launch 0.1 to 0.4 us (12x10x8x14, one field:
// 19.85 / 19.97 and 20.27 us, by where the test stood).
template <typename SG>
__global__ __launch_bounds__(kSpreadBlock) void k_hop_place() {
  if constexpr (std::is_same_v<SG, double2>) asm volatile("" ::: "v191");
  else if constexpr (std::is_same_v<SG, float2>) asm volatile("" ::: "v103");
  else asm volatile("" ::: "v95");
}

template <typename SG>
static void place(hipStream_t st) {
  using A = typename StoreTraits<SG>::acc;
  constexpr size_t lds = sizeof(cpx<A>) * 8 * 6 * kSpreadSites + sizeof(double) * 12 * kSpreadSites;
  k_hop_place<SG><<<32, kSpreadBlock, lds, st>>>();
}

hipError_t launch_hop_place(int prec, hipStream_t st) {
  if (prec == P_F64) place<double2>(st);
  else if (prec == P_F32) place<float2>(st);
  else place<bf16x2>(st);
  return hipGetLastError();
}

// per-rhs partial sums a launch of the tiled shapes writes (its site blocks;
// negative: halves of them, see parts_count)
int hop_nparts(const HopLaunch& h0) {
  HopLaunch h = h0;
  if (h.prec == P_F64) h.rhs_lanes = 1;
  if (spread_on(h)) return spread_nparts(h);
  return hop_nblocks(h);
}

// the block order that a launch of this shape runs: the slab orders need whole
// workgroups per (z, t) plane and a whole number of slabs
int hop_order(const HopLaunch& h) {
  const bool slab_ok =
      (h.g.L[2] % 8) == 0 && ((long)h.g.Lxh * h.g.L[1]) % sites_per_block(h.rhs_lanes, split_on(h)) == 0;
  if ((h.order == 2 || h.order == 5) && !slab_ok) return 1;
  if (h.order == 6 && !(slab_ok && (h.g.L[2] % 16) == 0)) return 1;
  if (h.order == 4 && !slab_ok) return 3;
  return h.order < 0 || h.order > 6 ? 1 : h.order;
}

// fill in nbs/bpp and validate the block order for this launch
static bool prepare(HopLaunch& h) {
  if (h.rhs_lanes != 1 && h.rhs_lanes != 2 && h.rhs_lanes != 4) return false;
  if (h.nr_tile < 1 || h.nr_tile > 3) return false;
  if (h.nrhs % (h.nr_tile * h.rhs_lanes) != 0) return false;
  h.nbs = hop_nblocks(h);
  h.lds_cap = lds_cap_bytes(h.occ_cap);
  h.bpp = (int)((long)h.g.Lxh * h.g.L[1] / sites_per_block(h.rhs_lanes, split_on(h)));
  h.order = hop_order(h);
  return true;
}

// canonical output (HopLaunch::cout), FP64
template <bool SPLIT, bool TM, int NR>
static hipError_t launch_canon(const HopLaunch& h, hipStream_t st) {
  const unsigned grid = (unsigned)h.nbs * (unsigned)(h.nrhs / NR), lds = canon_lds(SPLIT);
  k_hop<double2, double2, double2, PRE_CLOV, POST_NONE, true, NR, 1, SPLIT, TM, true>
      <<<grid, kHopBlock, lds > h.lds_cap ? lds : h.lds_cap, st>>>(h);
  return hipGetLastError();
}
static hipError_t launch_canon(const HopLaunch& h, hipStream_t st) {
  if (tm_on(h)) {
    if (h.nr_tile != 1) return hipErrorInvalidValue;
    return split_on(h) ? launch_canon<true, true, 1>(h, st) : launch_canon<false, true, 1>(h, st);
  }
  switch (h.nr_tile) {
    case 1: return split_on(h) ? launch_canon<true, false, 1>(h, st) : launch_canon<false, false, 1>(h, st);
    case 2: return launch_canon<false, false, 2>(h, st);
    case 3: return launch_canon<false, false, 3>(h, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename SG, typename SI, typename SO, int PRE, int POST, bool HOP, int RL>
static hipError_t launch_rl(const HopLaunch& h, hipStream_t st) {
  const unsigned grid = (unsigned)h.nbs * (unsigned)(h.nrhs / (h.nr_tile * RL));
  switch (h.nr_tile) {
    case 1:
      if constexpr (RL == 1) {
        if (tm_on(h)) {
          if (split_on(h))
            k_hop<SG, SI, SO, PRE, POST, HOP, 1, 1, true, true><<<grid, kHopBlock, h.lds_cap, st>>>(h);
          else
            k_hop<SG, SI, SO, PRE, POST, HOP, 1, 1, false, true><<<grid, kHopBlock, h.lds_cap, st>>>(h);
          break;
        }
        if (split_on(h)) {
          k_hop<SG, SI, SO, PRE, POST, HOP, 1, 1, true, false><<<grid, kHopBlock, h.lds_cap, st>>>(h);
          break;
        }
      }
      if (tm_on(h)) return hipErrorInvalidValue;
      k_hop<SG, SI, SO, PRE, POST, HOP, 1, RL, false, false><<<grid, kHopBlock, h.lds_cap, st>>>(h);
      break;
    case 2:
      if (tm_on(h)) return hipErrorInvalidValue;
      k_hop<SG, SI, SO, PRE, POST, HOP, 2, RL, false, false><<<grid, kHopBlock, h.lds_cap, st>>>(h);
      break;
    case 3:
      if (tm_on(h)) return hipErrorInvalidValue;
      k_hop<SG, SI, SO, PRE, POST, HOP, 3, RL, false, false><<<grid, kHopBlock, h.lds_cap, st>>>(h);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// the two hot shapes: every (nr_tile, rhs_lanes); FP64 only with rhs_lanes 1
template <typename SG, typename SI, typename SO, int PRE, int POST, bool HOP>
static hipError_t launch_tiled(const HopLaunch& h0, hipStream_t st) {
  HopLaunch h = h0;
  if (std::is_same<SG, double2>::value) h.rhs_lanes = 1;
  if (spread_on(h)) return launch_spread<SG, SI, SO, false>(h, st);
  if (!prepare(h)) return hipErrorInvalidValue;
  if (h.cy || h.cz || h.pf_r || h.beta_parts) return hipErrorInvalidValue;  // the small form only
  if (h.cout) {
    if constexpr (std::is_same<SG, double2>::value && PRE == PRE_CLOV && POST == POST_NONE)
      return h.partials ? hipErrorInvalidValue : launch_canon(h, st);
    return hipErrorInvalidValue;
  }
  if constexpr (std::is_same<SG, double2>::value) {
    return launch_rl<SG, SI, SO, PRE, POST, HOP, 1>(h, st);
  } else {
    switch (h.rhs_lanes) {
      case 1: return launch_rl<SG, SI, SO, PRE, POST, HOP, 1>(h, st);
      case 2: return launch_rl<SG, SI, SO, PRE, POST, HOP, 2>(h, st);
      case 4: return launch_rl<SG, SI, SO, PRE, POST, HOP, 4>(h, st);
      default: return hipErrorInvalidValue;
    }
  }
}

template <typename SG, typename SI, typename SV, int RL>
static hipError_t launch_xr_rl(const HopLaunch& h, hipStream_t st) {
  const unsigned grid = (unsigned)h.nbs * (unsigned)(h.nrhs / (h.nr_tile * RL));
  switch (h.nr_tile) {
    case 1:
      if constexpr (RL == 1) {
        if (tm_on(h)) {
          if (split_on(h))
            k_hop_xr<SG, SI, SV, 1, 1, true, true><<<grid, kHopBlock, h.lds_cap, st>>>(h);
          else
            k_hop_xr<SG, SI, SV, 1, 1, false, true><<<grid, kHopBlock, h.lds_cap, st>>>(h);
          break;
        }
        if (split_on(h)) {
          k_hop_xr<SG, SI, SV, 1, 1, true, false><<<grid, kHopBlock, h.lds_cap, st>>>(h);
          break;
        }
      }
      if (tm_on(h)) return hipErrorInvalidValue;
      k_hop_xr<SG, SI, SV, 1, RL, false, false><<<grid, kHopBlock, h.lds_cap, st>>>(h);
      break;
    case 2:
      if (tm_on(h)) return hipErrorInvalidValue;
      k_hop_xr<SG, SI, SV, 2, RL, false, false><<<grid, kHopBlock, h.lds_cap, st>>>(h);
      break;
    case 3:
      if (tm_on(h)) return hipErrorInvalidValue;
      k_hop_xr<SG, SI, SV, 3, RL, false, false><<<grid, kHopBlock, h.lds_cap, st>>>(h);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename SG, typename SI, typename SV>
static hipError_t launch_xr(const HopLaunch& h0, hipStream_t st) {
  HopLaunch h = h0;
  if (std::is_same<SG, double2>::value) h.rhs_lanes = 1;
  if (h.both || !h.partials || !h.cg) return hipErrorInvalidValue;
  if (spread_on(h)) return launch_spread<SG, SI, SV, true>(h, st);
  if (!prepare(h)) return hipErrorInvalidValue;
  if constexpr (std::is_same<SG, double2>::value) {
    return launch_xr_rl<SG, SI, SV, 1>(h, st);
  } else {
    switch (h.rhs_lanes) {
      case 1: return launch_xr_rl<SG, SI, SV, 1>(h, st);
      case 2: return launch_xr_rl<SG, SI, SV, 2>(h, st);
      case 4: return launch_xr_rl<SG, SI, SV, 4>(h, st);
      default: return hipErrorInvalidValue;
    }
  }
}

hipError_t launch_hop_xr(const HopLaunch& h, hipStream_t st) {
  if (h.g.V2 <= 0 || h.nrhs <= 0 || !h.hop || h.pre != PRE_CLOV || h.post != POST_NONE)
    return hipErrorInvalidValue;
  if (h.prec == P_F64 && h.in_prec == P_F64 && h.xr_prec == P_F64)
    return launch_xr<double2, double2, double2>(h, st);
  if (h.prec == P_F32 && h.in_prec == P_F32 && h.xr_prec == P_F32)
    return launch_xr<float2, float2, float2>(h, st);
  if (h.prec == P_BF16 && h.in_prec == P_BF16 && h.xr_prec == P_F32)
    return launch_xr<bf16x2, bf16x2, float2>(h, st);
  return hipErrorInvalidValue;
}

// set-up shapes (source preparation, reconstruction, block application):
// one rhs per thread
template <typename SG, typename SI, typename SO, int PRE, int POST, bool HOP>
static hipError_t launch_single(const HopLaunch& h0, hipStream_t st) {
  HopLaunch h = h0;
  h.nr_tile = 1;
  h.rhs_lanes = 1;
  h.dir_split = 0;
  if (spread_on(h)) return launch_spread<SG, SI, SO, false>(h, st);
  if (!prepare(h)) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)h.nbs * (unsigned)h.nrhs;
  if (tm_on(h))
    k_hop<SG, SI, SO, PRE, POST, HOP, 1, 1, false, true><<<grid, kHopBlock, 0, st>>>(h);
  else
    k_hop<SG, SI, SO, PRE, POST, HOP, 1, 1, false, false><<<grid, kHopBlock, 0, st>>>(h);
  return hipGetLastError();
}

template <typename SG, typename SI, typename SO>
static hipError_t dispatch_mode(const HopLaunch& h, hipStream_t st) {
  if (h.hop && h.pre == PRE_NONE && h.post == POST_CLOV)
    return launch_tiled<SG, SI, SO, PRE_NONE, POST_CLOV, true>(h, st);
  if (h.hop && h.pre == PRE_CLOV && h.post == POST_NONE)
    return launch_tiled<SG, SI, SO, PRE_CLOV, POST_NONE, true>(h, st);
  if (h.hop && h.pre == PRE_IDENT && h.post == POST_NONE)
    return launch_single<SG, SI, SO, PRE_IDENT, POST_NONE, true>(h, st);
  if (h.hop && h.pre == PRE_IDENT && h.post == POST_CLOV)
    return launch_single<SG, SI, SO, PRE_IDENT, POST_CLOV, true>(h, st);
  if (!h.hop && h.pre == PRE_IDENT && h.post == POST_CLOV)
    return launch_single<SG, SI, SO, PRE_IDENT, POST_CLOV, false>(h, st);
  if (!h.hop && h.pre == PRE_CLOV && h.post == POST_NONE)
    return launch_single<SG, SI, SO, PRE_CLOV, POST_NONE, false>(h, st);
  if (h.hop && h.pre == PRE_NONE && h.post == POST_NONE)
    return launch_single<SG, SI, SO, PRE_NONE, POST_NONE, true>(h, st);
  return hipErrorInvalidValue;
}

hipError_t launch_hop(const HopLaunch& h, hipStream_t st) {
  if (h.g.V2 <= 0 || h.nrhs <= 0) return hipErrorInvalidValue;
  if (h.prec == P_F64 && h.in_prec == P_F64 && h.out_prec == P_F64)
    return dispatch_mode<double2, double2, double2>(h, st);
  if (h.prec == P_F32 && h.in_prec == P_F32 && h.out_prec == P_F32)
    return dispatch_mode<float2, float2, float2>(h, st);
  if (h.prec == P_BF16 && h.in_prec == P_BF16 && h.out_prec == P_BF16)
    return dispatch_mode<bf16x2, bf16x2, bf16x2>(h, st);
  return hipErrorInvalidValue;
}

}  // namespace lqcd
