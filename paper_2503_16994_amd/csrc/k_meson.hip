// Meson two-point functions from a 12-column point-source propagator.
//
// The paper's propagator functions produce the quark propagator from which
// correlation functions are contracted (Sec. 3.3); this is that contraction.
// With S(x)[al a][be c] = psi_(3 be + c)(x)[al][a] (column j = 3 s + c of the
// propagator: source spin s, colour c), the colour-traced spin tensor per
// time slice
//   G_t[al][be][al'][be'] = sum_{x in slice t} sum_{a, c} S(x)[al a][be c] conj(S(x)[al' a][be' c])
// carries every meson correlator: by g5-hermiticity the backward propagator
// is g5 S^+ g5, so
//   C_t(Gamma, Gamma') = sum_x tr[Gamma S(x) Gamma' g5 S(x)^+ g5]
//                      = sum Gamma[de][al] Gamma'[be][ga] g5[ga] g5[de] G_t[al][be][de][ga].
// Gamma is named by a 4-bit mask m: Gamma_m = g_t^{m3} g_x^{m0} g_y^{m1} g_z^{m2}
// (ordered product, t first, so m = 15 is g5 = g_t g_x g_y g_z).
//
// As a matrix product, G_t = Z Z^H with Z[(al, be)][(x, a, c)] the 16 x 9 V3
// matrix of slice t, so it runs on the FP64 matrix cores: with Z = Zr + i Zi,
//   Re G = Zr Zr^T + Zi Zi^T,   Im G = Zi Zr^T - Zr Zi^T.
// An entry of G may be far smaller than the terms it is summed from (columns that
// differ by nearly a phase: Im, or Re for spins tied by a factor i), so the two
// products of Re and of Im go into one accumulator each, term by term.  (Im G as
// X - X^T of one product is a product less, and the error of such an entry grew a
// thousandfold against sums of its own terms.)
//
// Kernel 1 (k_meson_partial): workgroup (b, t) takes one chunk of slice t,
// each of its four waves every fourth group of four sites.  In
// v_mfma_f64_16x16x4 lane l holds row l % 16 and inner index l / 16 of both
// operands, so the lane that loads component (al, a) of column (be, c) at
// site l / 16 of the group holds one entry of the left and of the right
// operand at once: nine 16-byte loads and 36 matrix instructions per four
// sites, no LDS and no barrier inside the loop, and the next group's loads in
// flight meanwhile.  v_permlane16_swap first puts the two terms of a site next to
// each other along the inner index (re of two sites in one register, im of them
// in the other), so that they meet in the sum before the next site's do.  Every
// four groups (288 terms) the sums are added to a second pair, which keeps the
// chains of a sum as short as its error wants them.  The waves' sums are added
// in wave order.
// Kernel 2 (k_meson_reduce): workgroup t sums the chunk partials of every
// entry in chunk order, forms G (Im antisymmetrised) and contracts with the
// requested Gamma pairs (a fixed-order block sum).  FP64 throughout;
// deterministic, no atomics.
//
// Bound: HBM, 2304 B per site read once.  At 32^3x64 the call takes 885 us
// (5.5 TB/s, against 6.0 TB/s of a plain read-only sum on the same card), with Im G
// from X - X^T 863 (and at four waves per SIMD, 931); staged in LDS 16 sites at a
// time and accumulated with vector FMAs, 168 registers and two barriers per 16
// sites, it took 1578 us.
#include "lqcd_kernels.h"

namespace lqcd {

constexpr int kMesonBlock = 256;
constexpr int kMesonGroup = 4;       // sites of one wave's step (the inner dimension of the matrix instruction)
constexpr int kMesonMaxChunk = 1024; // sites per workgroup, halved until the grid fills the GPU
constexpr int kMesonMinChunk = 64;
constexpr long kMesonGrid = 2048;    // workgroups wanted: eight per CU, two rounds of four

using cd = cpx<double>;
typedef double d4 __attribute__((ext_vector_type(4)));

// exchanges the odd 16-lane rows of a with the even ones of b
__device__ inline void swap_rows(double& a, double& b) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 av = __builtin_bit_cast(u2, a), bv = __builtin_bit_cast(u2, b);
  const auto lo = __builtin_amdgcn_permlane16_swap(av.x, bv.x, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(av.y, bv.y, false, false);
  a = __builtin_bit_cast(double, u2{lo[0], hi[0]});
  b = __builtin_bit_cast(double, u2{lo[1], hi[1]});
}

__global__ __launch_bounds__(kMesonBlock) void k_meson_partial(const double2* __restrict__ psi, long V, long V3,
                                                               int chunk, int nchunk, double2* partials) {
  const int t = blockIdx.y, b = blockIdx.x, tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63, row = l & 15, al = row >> 2, be = row & 3;
  const long s_end = min((long)(t + 1) * V3, (long)t * V3 + (long)(b + 1) * chunk);
  constexpr int kStep = kMesonGroup * (kMesonBlock / 64);
  long x = (long)t * V3 + (long)b * chunk + kMesonGroup * w + (l >> 4);  // this lane's site
  // element (c, a) of this lane's (al, be): column 3 be + c, component 3 al + a
  const double2* p = psi + ((size_t)(3 * be) * V + x) * 12 + 3 * al;
  double2 z[9], zn[9];
  auto load = [&](double2 (&v)[9]) {
    const bool in = x < s_end;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int a = 0; a < 3; ++a) v[3 * c + a] = in ? p[(size_t)c * V * 12 + a] : make_double2(0.0, 0.0);
    x += kStep;
    p += kStep * 12;
  };
  const d4 zero = {0.0, 0.0, 0.0, 0.0};
  d4 re = zero, im = zero, re_sum = zero, im_sum = zero;
  const int steps = (int)((s_end - ((long)t * V3 + (long)b * chunk) + kStep - 1) / kStep);  // uniform
  load(z);
  for (int k = 0; k < steps; ++k) {
    load(zn);  // past the chunk: zeros, nothing read
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      // inner index 0..3: re, im of sites 0 and 2, then of sites 1 and 3
      double p0 = z[e].x, p1 = z[e].y, n0 = z[e].y, n1 = -z[e].x;
      swap_rows(p0, p1);
      swap_rows(n0, n1);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(p0, p0, re, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(p1, p1, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(n0, p0, im, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(n1, p1, im, 0, 0, 0);
    }
    if ((k & 3) == 3) {
      re_sum += re;
      im_sum += im;
      re = im = zero;
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) z[e] = zn[e];
  }
  re_sum += re;
  im_sum += im;
  // result element r of lane l: row l / 16 + 4 r, column l % 16
  __shared__ double2 red[kMesonBlock / 64][256];
#pragma unroll
  for (int r = 0; r < 4; ++r) red[w][((l >> 4) + 4 * r) * 16 + row] = make_double2(re_sum[r], im_sum[r]);
  __syncthreads();
  double2 s = make_double2(0.0, 0.0);
#pragma unroll
  for (int ww = 0; ww < kMesonBlock / 64; ++ww) {
    s.x += red[ww][tid].x;
    s.y += red[ww][tid].y;
  }
  partials[((size_t)t * nchunk + b) * 256 + tid] = s;  // entry (tid / 16, tid % 16)
}

// chiral-basis gamma matrices g_x, g_y, g_z, g_t (mu = 0..3): each has one
// non-zero per row; row r of g_mu holds `val` in column `col`
__device__ inline void gamma_row(int mu, int r, int& col, cd& val) {
  switch (mu) {
    case 0:  // g_x = [[0, -i s1], [i s1, 0]]
      col = 3 - r;
      val = (r < 2) ? cd{0.0, -1.0} : cd{0.0, 1.0};
      break;
    case 1:  // g_y = [[0, -i s2], [i s2, 0]]
      col = 3 - r;
      val = (r == 0 || r == 3) ? cd{-1.0, 0.0} : cd{1.0, 0.0};
      break;
    case 2:  // g_z = [[0, -i s3], [i s3, 0]]
      col = r ^ 2;
      val = (r == 0 || r == 3) ? cd{0.0, -1.0} : cd{0.0, 1.0};
      break;
    default:  // g_t = [[0, -1], [-1, 0]]
      col = r ^ 2;
      val = cd{-1.0, 0.0};
      break;
  }
}

// entry (r, c) of Gamma_m = g_t^{m3} g_x^{m0} g_y^{m1} g_z^{m2}: the single
// non-zero of row r is followed through the ordered product
__device__ inline cd gamma_entry(int m, int r, int c) {
  int k = r;
  cd p = {1.0, 0.0};
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const int mu = (f == 0) ? 3 : f - 1;
    if ((m >> mu) & 1) {
      int col;
      cd v;
      gamma_row(mu, k, col, v);
      p = cmul(p, v);
      k = col;
    }
  }
  return (k == c) ? p : cd{0.0, 0.0};
}

struct MesonPairs {
  int n;
  int m[kMaxMesonPairs][2];
  double scale;                   // applied to every correlator
  double2* out[kMaxMesonPairs];   // correlator of pair p: out[p][t]
};

__global__ __launch_bounds__(256) void k_meson_reduce(const double2* __restrict__ partials, int nchunk, double2* G,
                                                      MesonPairs pairs) {
  __shared__ double red[2][4];
  __shared__ double xs[256];
  const int t = blockIdx.x, i = threadIdx.x;
  double2 g = make_double2(0.0, 0.0);
#pragma unroll 8
  for (int b = 0; b < nchunk; ++b) {
    const double2 v = partials[((size_t)t * nchunk + b) * 256 + i];
    g.x += v.x;
    g.y += v.y;
  }
  xs[i] = g.y;
  __syncthreads();
  g.y = 0.5 * (g.y - xs[(i & 15) * 16 + (i >> 4)]);  // G is Hermitian
  if (G) G[(size_t)t * 256 + i] = g;
  // entry i = G[al][be][de][ga]
  const int al = i >> 6, be = (i >> 4) & 3, de = (i >> 2) & 3, ga = i & 3;
  const double g5ga = ga < 2 ? 1.0 : -1.0, g5de = de < 2 ? 1.0 : -1.0;
  for (int p = 0; p < pairs.n; ++p) {
    const cd coef = cmul(gamma_entry(pairs.m[p][0], de, al), gamma_entry(pairs.m[p][1], be, ga));
    cd term = cmul(coef, cd{g.x, g.y});
    term = {term.re * g5ga * g5de, term.im * g5ga * g5de};
    double re = term.re, im = term.im;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      re += __shfl_xor(re, off, 64);
      im += __shfl_xor(im, off, 64);
    }
    const int w = i >> 6, l = i & 63;
    if (l == 0) {
      red[0][w] = re;
      red[1][w] = im;
    }
    __syncthreads();
    if (i == 0) {
      double sr = 0.0, si = 0.0;
      for (int ww = 0; ww < 4; ++ww) {
        sr += red[0][ww];
        si += red[1][ww];
      }
      pairs.out[p][t] = make_double2(pairs.scale * sr, pairs.scale * si);
    }
    __syncthreads();
  }
}

// Sites per workgroup: as many as leave kMesonGrid workgroups (fewer partials
// to write and sum again), down to one group of 16 sites a wave where the
// lattice is too small to fill the GPU (there the loop's length is the time).
static int meson_chunk(long V3, int T) {
  int c = kMesonMaxChunk;
  while (c > kMesonMinChunk && T * ((V3 + c - 1) / c) < kMesonGrid) c >>= 1;
  return c;
}
// A chunk below 256 sites means that twice its length left fewer than
// kMesonGrid workgroups, so there are never more than
// max(T ceil(V3 / 256), 2 kMesonGrid) partials (4 KiB each, 16 MiB).
int meson_nchunk(long V3, int T) {
  const int c = meson_chunk(V3, T);
  return (int)((V3 + c - 1) / c);
}

hipError_t launch_meson(const KGeom& g, const double2* psi, int npairs, const int* masks, double2* const* outs,
                        double scale, double2* G, double2* scratch, hipStream_t st) {
  if (npairs < 0 || npairs > kMaxMesonPairs) return hipErrorInvalidValue;
  const long V3 = (long)g.L[0] * g.L[1] * g.L[2], V = V3 * g.L[3];
  const int chunk = meson_chunk(V3, g.L[3]), nchunk = meson_nchunk(V3, g.L[3]);
  MesonPairs pairs;
  pairs.n = npairs;
  pairs.scale = scale;
  for (int p = 0; p < kMaxMesonPairs; ++p) {
    pairs.m[p][0] = p < npairs ? masks[2 * p] : 0;
    pairs.m[p][1] = p < npairs ? masks[2 * p + 1] : 0;
    pairs.out[p] = p < npairs ? outs[p] : nullptr;
  }
  k_meson_partial<<<dim3(nchunk, g.L[3]), kMesonBlock, 0, st>>>(psi, V, V3, chunk, nchunk, scratch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_meson_reduce<<<g.L[3], 256, 0, st>>>(scratch, nchunk, G, pairs);
  return hipGetLastError();
}

}  // namespace lqcd
