// Internal host-side state behind the opaque handles of lqcd.h.
#pragma once

#include <stdarg.h>
#include <stdio.h>

#include <string>
#include <vector>

#include "../../include/lqcd.h"
#include "lqcd_kernels.h"

struct lqcd_geom {
  lqcd_geom_desc desc;
  lqcd::KGeom kg;
  int64_t V;
  int V2;
  int V2p;  // V2 rounded up to the 64-site layout tile
};

struct lqcd_gauge {
  const lqcd_geom_t* g;
  int pmask;
  uint64_t uid;  // distinguishes gauge fields for the clover cache
  int two_row;   // links stored as their first two rows
  double2* U64;
  float2* U32;
  lqcd::bf16x2* U16;
};

// Device memory map of a workspace (all pointers into the caller's memory).
struct WsLayout {
  size_t bytes = 0;
  // clover: A on both parities (tiled 36-component fields), inverse on the odd sites
  double2 *C64 = nullptr, *Ci64 = nullptr;
  float2 *C32 = nullptr, *Ci32 = nullptr;
  lqcd::bf16x2 *C16 = nullptr, *Ci16 = nullptr;
  int* err_flag = nullptr;
  // FP64 full-lattice vectors [nrhs][2 parities] of tiled 12-component fields
  double2 *E = nullptr, *X = nullptr, *TMP = nullptr, *R = nullptr, *P = nullptr, *Q = nullptr,
          *AP = nullptr, *EH = nullptr;
  // inner-precision half vectors [nrhs] of tiled 12-component fields (FP32) and BF16 copies
  float2 *xl = nullptr, *rl = nullptr, *pl = nullptr, *ql = nullptr, *apl = nullptr, *tl = nullptr;
  lqcd::bf16x2 *pb = nullptr, *qb = nullptr, *tb = nullptr;
  // reductions
  double* partials = nullptr;  // [nrhs][max_parts]
  double* partials2 = nullptr; // [nrhs][max_parts]
  int max_parts = 0;
  lqcd::CGState* cg = nullptr; // [nrhs]
  double* scal = nullptr;      // [8][nrhs]
};

// A captured chunk of solver iterations, valid for the workspace's lifetime
// (its kernels read and write only the gauge field and workspace memory).
// A captured chunk of CG iterations.  Its launches depend on the gauge
// field, the solver, the precision of the recursion, the rhs count, the chunk
// length and the hop-kernel tunings of that precision and of FP64 (reliable
// updates); the workspace's buffers are fixed for its lifetime.
struct GraphEntry {
  uint64_t gauge_uid;
  int solver, inner_prec, nrhs, chunk;
  double mu;  // twisted mass (a kernel argument of the captured launches)
  bool shared;  // general hop launches only
  lqcd_tuning tune_inner, tune_f64, tune_f32;
  hipGraph_t graph;
  hipGraphExec_t exec;
};

inline bool same_tuning(const lqcd_tuning& a, const lqcd_tuning& b) {
  return a.nr_tile == b.nr_tile && a.block_order == b.block_order && a.rhs_lanes == b.rhs_lanes &&
         a.flags == b.flags;
}

// the configuration of a workspace nobody tuned (nr, order, lanes, flags): it
// stands for own_tuning, and setting it gives the choice back to the launches
constexpr lqcd_tuning kDefaultTuning = {1, 1, 1, 0};

struct lqcd_ws {
  const lqcd_geom_t* g;
  int pmask;
  int nrhs;
  WsLayout m;
  // clover cache key
  bool clover_valid = false;
  uint64_t clover_uid = 0;
  double kappa = 0, csw = 0, cF = 0, mu = 0;
  int clover_pmask = 0;
  std::vector<GraphEntry> graphs;
  hipEvent_t probe[2] = {nullptr, nullptr};  // around the look for a place of a small solve
  lqcd_tuning tune[3] = {kDefaultTuning, kDefaultTuning, kDefaultTuning};
  bool tune_set[3] = {false, false, false};  // not the default (else: own_tuning)
};

namespace lqcd {

void set_error(const char* fmt, ...);
int fail(int status, const char* fmt, ...);
WsLayout plan_ws(const lqcd_geom_t* g, int pmask, int nrhs, char* base);
int ensure_clover(const lqcd_gauge_t* u, const lqcd_dirac* d, lqcd_ws_t* w, hipStream_t st);
int check_dirac(const lqcd_dirac* d);
// argument checks shared by the meson entry points (status, last error set)
int meson_check(const char* who, const lqcd_geom_t* g, const void* psi, int npairs, const int32_t* pairs,
                const void* C, const void* G);
// FP64 complex partials of the meson contraction: T x chunks x 256 entries
size_t meson_scratch_bytes(const lqcd_geom_t* g);
// adds an autotuning result to the process-wide tuning cache (lqcd_tune.hip)
void tune_cache_put(const lqcd_gauge_t* u, int prec, int nrhs, int twisted, const lqcd_tuning& t, double us);

inline int hip_status(hipError_t e, const char* what) {
  if (e == hipSuccess) return LQCD_OK;
  return fail(LQCD_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

#define LQCD_HIP(call)                                        \
  do {                                                        \
    hipError_t _e = (call);                                   \
    if (_e != hipSuccess) return ::lqcd::hip_status(_e, #call); \
  } while (0)

// Description of one hop launch over a full-layout vector: parity p_out of
// `out` from parity 1-p_out of `y` (and p_out of `z`).
struct HopSpec {
  int prec;  // links/clover precision
  int in_prec, out_prec;
  int pre, post;
  bool hop = true;
  bool g5 = false;
  double scale = 0.0;
};

// Launch configuration of a workspace that nobody tuned, by sites V, storage
// precision and rhs count n (no configuration changes a result).
//  * Links and clover blocks in FP64 and FP32: with several rhs per site they are
//    re-read, and up to a few 10^5 sites they stay in the last-level cache from
//    launch to launch, so ordinary loads beat non-temporal ones; one rhs (or two,
//    and in FP32 three) of a larger lattice streams them once and keeps the
//    non-temporal ones.  In BF16 the two are the same to 1%: non-temporal.
//    A launch over both parities (`both`) reads every link twice, so in FP32 it
//    keeps the ordinary loads to 10^6 sites.
//  * rhs per thread: one while the launch needs its threads to hide latency,
//    two (or three for an odd n, in FP32 for any multiple of three) once there
//    are enough.
//  * From 10^6 sites on, z-slabs per XCD; in FP64 with several rhs from 10^6
//    sites times rhs on (plain order where planes do not divide, see hop_order).
// Against non-temporal loads and one rhs per thread everywhere, us per pair of
// hops on fields of zeros: FP64 12^3x24 12 rhs 123 / 89, 16^3x32 1 rhs 47.5 / 43.1,
// 4 rhs 136 / 98, 12 rhs 391 / 295, 24^3x48 12 rhs 2632 / 1701, 32^3x64 1 rhs
// 753 / 645, 12 rhs 7936 / 4379; FP32 16^3x32 12 rhs 216 / 147, 24^3x48 1 rhs 127
// / 113, 32^3x64 12 rhs 4076 / 2395; BF16 32^3x64 12 rhs 1533 / 1188.
// The lines, ms of even-odd solves of 40 iterations from noise sources:
//   cached / non-temporal loads: FP32 1 rhs 524288 sites 10.6 / 11.1, 663552 13.8 /
//   13.8, 786432 16.4 / 15.8, 983040 20.2 / 19.2, 2 rhs (one / two a thread) 262144
//   8.4 / 8.8, 663552 22.2 / 21.1, 3 rhs 262144 11.9 / 11.7, 393216 18.1 / 18.4, 663552
//   31.0 / 29.1; FP64 1 rhs 212992 7.86 / 8.00, 221184 8.34 / 8.50, 245760 8.93 / 8.55,
//   2 rhs 212992 11.95 / 11.99, 245760 13.45 / 13.21, 3 rhs (one / three a thread)
//   245760 18.6 / 19.1, 524288 39.6 / 40.7;
//   the same, us per internal Dw of 1 rhs: FP32 331776 52.2 / 60.6, 663552 108.7 /
//   115.2; FP64 229376 76.8 / 77.4, 331776 120.4 / 116.4;
//   one / two rhs a thread, by sites times rhs: BF16 393216 4.76 / 4.80, 524288 5.29 /
//   5.44, 786432 7.27 / 7.10, 1048576 9.12 / 9.33, 1327104 12.05 / 12.24, 1572864
//   12.92 / 12.76, 2654208 23.2 / 22.3; FP32 327680 5.46 / 5.55, 360448 5.95 / 5.75,
//   497664 7.58 / 7.07; FP64 497664 10.80 / 10.91, 786432 17.7 / 17.3, 1048576 23.1 /
//   23.0, and 22.3 with slabs;
//   plain order / slabs, 1 rhs: FP64 524288 17.4 / 17.7, 983040 32.9 / 31.5, 1048576
//   34.5 / 33.1; FP32 1048576 20.1 / 19.8; BF16 983040 11.3 / 11.0.
// The slabs and tiles of FP64 batches, us per canonical Dw / per four hops of the
// Schur normal operator, plain order against slabs at two rhs per thread:
// 16^3x32 4 rhs 154 / 275 and 150 / 285, 8 rhs 281 / 526 and 273 / 511, 12 rhs
// 410 / 762 and 389 / 732; 32^3x64 12 rhs, slabs at three and two rhs per thread:
// 7194 / 11236 and 6937 / 10882.
inline lqcd_tuning own_tuning(int64_t V, int prec, int n, bool both = false) {
  constexpr int kCached = LQCD_TUNE_NT_STORE | LQCD_TUNE_CACHED_GAUGE, kStream = LQCD_TUNE_NT_STORE;
  const int64_t vn = V * n, large = 1000000;
  lqcd_tuning t = {1, 1, 1, 0};
  if (V >= large) {
    t.block_order = 2;
    const bool three = n % 3 == 0 && (prec == LQCD_F32 || (prec == LQCD_F64 && n % 2 != 0));
    if (n > 1) t.nr_tile = three || n == 3 ? 3 : 2;
  }
  if (prec == LQCD_BF16) {
    if (n >= 4 && vn >= 1400000) t.nr_tile = 2;
  } else if (n < 4) {
    const int64_t line = prec == LQCD_F32 ? (both ? large : 600000) : n == 3 ? large : both ? 250000 : 230000;
    const bool fits = V <= line;
    t.flags = fits ? kCached : kStream;
    if (!fits && n > 1) t.nr_tile = n;
  } else {
    t.flags = kCached;
    if (V < large && vn >= (prec == LQCD_F64 ? large : 360000)) {
      t.nr_tile = 2;
      if (prec == LQCD_F64) t.block_order = 2;
    }
  }
  return t;
}
// the configuration of launches over n rhs in precision prec
inline lqcd_tuning tuning_of(const lqcd_ws* w, int prec, int n, bool both = false) {
  return w->tune_set[prec] ? w->tune[prec] : own_tuning(w->g->V, prec, n, both);
}

// The same for an operator on canonical fields whose result the layout conversion
// reads next (one_hop: a single launch over one parity).
//  * Up to 8 MB of (sites x rhs x element) the conversion finds the result in the
//    last-level cache, so it is stored the ordinary way.
//  * The conversions before and after sweep that cache: links and clover blocks of
//    few rhs stay in it from call to call only if everything the call moves fits
//    its 256 MB.
// us per call of FP32 HOP_EO, stores and loads ordinary / non-temporal stores and
// ordinary loads / this choice: 16^3x32 1 rhs 36.6 / 37.2 / 36.6, 4 rhs 111 / 117 /
// 110; 24^4 1 rhs 88.5 / 90.2 / 84.8, with a twisted mass 101 / 104 / 92, 4 rhs 279 /
// 274 / 274; 24^3x48 1 rhs 168 / 169 / 163.  FP64 16^3x32 49.6 / 50.6 / 49.6, 24^4 136 /
// 139 / 125.  BF16 the same to 1% in every form.
inline lqcd_tuning own_tuning_converted(int64_t V, int prec, int n, bool both, bool one_hop, bool two_row) {
  lqcd_tuning t = own_tuning(V, prec, n, both);
  const int64_t e = (int64_t)elem_bytes(prec);
  if (prec == LQCD_BF16 || V * n * e > 8000000) return t;
  t.flags &= ~LQCD_TUNE_NT_STORE;
  // links of both parities and clover blocks of one; canonical and internal fields
  const int64_t bytes = V * (((two_row ? 24 : 36) + 18) * e + n * 24 * (16 + e));
  if (!both && (n < 4 || one_hop) && bytes > 256000000) t.flags &= ~LQCD_TUNE_CACHED_GAUGE;
  return t;
}

// rhs tiling of a launch over nrhs fields: rhs_lanes lanes per site, each
// with nr_tile rhs; both are reduced until their product divides nrhs
inline void apply_tuning(HopLaunch& h, const lqcd_tuning& t) {
  int rl = (t.rhs_lanes == 2 || t.rhs_lanes == 4) ? t.rhs_lanes : 1;
  int nr = t.nr_tile < 1 ? 1 : (t.nr_tile > 3 ? 3 : t.nr_tile);
  while (h.nrhs % rl) rl >>= 1;
  while (h.nrhs % (nr * rl)) --nr;
  h.nr_tile = nr;
  h.rhs_lanes = rl;
  h.order = t.block_order;
  h.nt_out = (t.flags & LQCD_TUNE_NT_STORE) ? 1 : 0;
  h.cached_gauge = (t.flags & LQCD_TUNE_CACHED_GAUGE) ? 1 : 0;
  h.occ_cap = (t.flags >> LQCD_TUNE_OCC_SHIFT) & 3;
  h.dir_split = (t.flags & LQCD_TUNE_DIR_SPLIT) ? 1 : 0;  // used where nr_tile = rhs_lanes = 1
}
inline void single_tile(HopLaunch& h) {
  h.nr_tile = 1;
  h.rhs_lanes = 1;
}

}  // namespace lqcd
