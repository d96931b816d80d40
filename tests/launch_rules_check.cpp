// Host check of the rules by which the library chooses its launches, linked
// against the built library (no device work).  Each check is named on the
// command line; a failure prints what differs and ends with status 1.
#include <stdio.h>
#include <string.h>

#include "../paper_2503_16994_amd/csrc/lqcd_internal.h"

using namespace lqcd;

static int failures = 0;
#define CHECK(cond, ...)                  \
  do {                                    \
    if (!(cond)) {                        \
      printf("%s: ", #cond);              \
      printf(__VA_ARGS__);                \
      printf("\n");                       \
      ++failures;                         \
    }                                     \
  } while (0)

static HopLaunch hop(int prec, long V2, int nrhs, bool both, double mu) {
  HopLaunch h;
  memset(&h, 0, sizeof(h));
  h.g.V2 = (int)V2;
  h.prec = prec;
  h.nrhs = nrhs;
  h.hop = true;
  h.both = both;
  h.tm_mu = mu;
  h.tm_post = mu != 0.0;
  apply_tuning(h, lqcd_tuning{1, 1, 1, 0});
  return h;
}

// A small launch (negative partial counts) is one whose 64-site workgroups are
// resident together: 256 in FP64, 512 in FP32 and BF16.
static void small_launches() {
  for (int prec = P_F64; prec <= P_BF16; ++prec) {
    const long line = 256 * (prec == P_F64 ? 1 : 2);
    for (int nrhs : {1, 4, 12})
      for (int both = 0; both < 2; ++both)
        for (double mu : {0.0, 0.01})
          for (long V2 = 16; V2 * nrhs < 64 * 2 * line; V2 += 16) {
            const bool small = hop_nparts(hop(prec, V2, nrhs, both != 0, mu)) < 0;
            const long n = (both ? 2 : 1) * ((V2 + 63) / 64) * nrhs;
            HopLaunch g = hop(prec, V2, nrhs, both != 0, mu);
            g.general = true;  // asked for
            CHECK(hop_nparts(g) > 0 && !hop_reads_canonical(g) && !hop_fuses_p(g), "prec %d V2 %ld: general form", prec, V2);
            CHECK(small == (n <= line), "prec %d nrhs %d both %d mu %g workgroups %ld", prec, nrhs, both, mu, n);
            if (failures > 10) return;
          }
  }
}

// The configuration of a workspace nobody tuned, at measured points on both
// sides of its lines (the faster of the two is the one expected).
static void own_configurations() {
  struct {
    int prec;
    int64_t V;
    int n, tile;
    bool cached, both = false;
  } const want[] = {
      {LQCD_F32, 524288, 1, 1, true},  {LQCD_F32, 786432, 1, 1, false}, {LQCD_F32, 983040, 1, 1, false},
      {LQCD_F32, 262144, 2, 1, true},  {LQCD_F32, 663552, 2, 2, false}, {LQCD_F32, 393216, 3, 1, true},
      {LQCD_F32, 663552, 3, 3, false}, {LQCD_F64, 221184, 1, 1, true},  {LQCD_F64, 245760, 1, 1, false},
      {LQCD_F64, 212992, 2, 1, true},  {LQCD_F64, 245760, 2, 2, false}, {LQCD_F64, 245760, 3, 1, true},
      {LQCD_F64, 524288, 3, 1, true},  {LQCD_BF16, 131072, 4, 1, false}, {LQCD_BF16, 131072, 8, 1, false},
      {LQCD_BF16, 331776, 4, 1, false}, {LQCD_BF16, 131072, 12, 2, false}, {LQCD_BF16, 663552, 4, 2, false},
      {LQCD_F32, 81920, 4, 1, true},   {LQCD_F32, 90112, 4, 2, true},   {LQCD_F64, 41472, 12, 1, true},
      {LQCD_F64, 131072, 8, 2, true},
      // launches over both parities
      {LQCD_F32, 663552, 1, 1, true, true}, {LQCD_F64, 229376, 1, 1, true, true}, {LQCD_F64, 331776, 1, 1, false, true},
  };
  for (const auto& w : want) {
    const lqcd_tuning t = own_tuning(w.V, w.prec, w.n, w.both);
    CHECK(t.nr_tile == w.tile, "prec %d V %ld n %d: tile %d", w.prec, (long)w.V, w.n, t.nr_tile);
    CHECK(((t.flags & LQCD_TUNE_CACHED_GAUGE) != 0) == w.cached, "prec %d V %ld n %d: flags %d", w.prec, (long)w.V,
          w.n, t.flags);
  }
}

// The same where a layout conversion reads the result next (canonical FP32
// operators, FP64 HOP_EO).
static void converted_configurations() {
  constexpr int N = LQCD_TUNE_NT_STORE, C = LQCD_TUNE_CACHED_GAUGE;
  struct {
    int prec;
    int64_t V;
    int n;
    bool both, one_hop;
    int flags;
  } const want[] = {
      {LQCD_F32, 131072, 1, false, true, C},  {LQCD_F32, 331776, 1, false, true, 0}, {LQCD_F32, 663552, 1, false, true, 0},
      {LQCD_F32, 331776, 1, false, false, 0}, {LQCD_F32, 331776, 1, true, false, C}, {LQCD_F32, 131072, 4, false, true, 0},
      {LQCD_F32, 131072, 4, false, false, C}, {LQCD_F32, 331776, 4, false, true, N | C},
      {LQCD_F64, 131072, 1, false, true, C},  {LQCD_F64, 331776, 1, false, true, 0}, {LQCD_F64, 663552, 1, false, true, N},
      {LQCD_BF16, 331776, 1, false, true, 0},
  };
  for (const auto& w : want) {
    const int flags = own_tuning_converted(w.V, w.prec, w.n, w.both, w.one_hop, true).flags;
    CHECK(flags == w.flags, "prec %d V %ld n %d both %d one hop %d: flags %d", w.prec, (long)w.V, w.n, w.both, w.one_hop,
          flags);
  }
}

// Setting what lqcd_ws_get_tuning returned for a workspace nobody tuned changes
// nothing: at once, and after another setting it gives the choice back to the
// launches.
static void tuning_round_trip() {
  for (int prec = LQCD_F64; prec <= LQCD_BF16; ++prec)
    for (int nrhs : {1, 3, 4, 12})
      for (int T : {8, 32, 256}) {
        lqcd_geom_desc d;
        memset(&d, 0, sizeof(d));
        for (int mu = 0; mu < 4; ++mu) {
          d.L[mu] = mu == 3 ? T : 16;
          d.theta_re[mu] = 1.0;
        }
        lqcd_geom_t* g = nullptr;
        lqcd_ws_t* w = nullptr;
        CHECK(lqcd_geom(&d, &g) == LQCD_OK, "geometry");
        // only recorded, never dereferenced here
        CHECK(lqcd_ws_create(g, 7, nrhs, (void*)(uintptr_t)(1 << 20), ~size_t(0), &w) == LQCD_OK, "workspace");
        const auto untouched = [&](const char* when) {
          for (int n : {1, nrhs})
            CHECK(same_tuning(tuning_of(w, prec, n), own_tuning(w->g->V, prec, n)), "prec %d nrhs %d T %d n %d: %s", prec,
                  nrhs, T, n, when);
        };
        lqcd_tuning first;
        CHECK(lqcd_ws_get_tuning(w, prec, &first) == LQCD_OK, "get");
        CHECK(same_tuning(first, lqcd_tuning{1, 1, 1, 0}), "prec %d: the documented default", prec);
        CHECK(lqcd_ws_set_tuning(w, prec, &first) == LQCD_OK, "set");
        untouched("set(get())");
        lqcd_tuning other = first;  // one field changed
        other.flags |= LQCD_TUNE_DIR_SPLIT;
        lqcd_tuning back;
        CHECK(lqcd_ws_set_tuning(w, prec, &other) == LQCD_OK && lqcd_ws_get_tuning(w, prec, &back) == LQCD_OK, "set");
        CHECK(same_tuning(back, other) && same_tuning(tuning_of(w, prec, 1), other), "a set configuration is used");
        CHECK(lqcd_ws_set_tuning(w, prec, &first) == LQCD_OK, "set");
        untouched("restored");
        lqcd_ws_free(w);
        lqcd_geom_free(g);
      }
}

// Workspaces keep their size, and hold the partial sums of every launch form.
static void workspace_bytes() {
  const struct {
    int L[4];
    size_t one, twelve;  // FP64 for one rhs; every precision for twelve
  } want[] = {{{16, 16, 16, 32}, 314606336, 3180727808}, {{24, 24, 24, 48}, 1592691456, 16102419968},
              {{32, 32, 32, 64}, 5033689856, 50891591168}, {{26, 26, 26, 30}, 1265796864, 12797448704},
              {{32, 32, 32, 32}, 2516845312, 25445797376}};
  for (const auto& w : want) {
    lqcd_geom_desc d;
    memset(&d, 0, sizeof(d));
    for (int mu = 0; mu < 4; ++mu) {
      d.L[mu] = w.L[mu];
      d.theta_re[mu] = 1.0;
    }
    lqcd_geom_t* g = nullptr;
    CHECK(lqcd_geom(&d, &g) == LQCD_OK, "geometry");
    CHECK(lqcd_ws_bytes(g, LQCD_PM_F64, 1) == w.one, "T %d: %zu", w.L[3], lqcd_ws_bytes(g, LQCD_PM_F64, 1));
    CHECK(lqcd_ws_bytes(g, 7, 12) == w.twelve, "T %d: %zu", w.L[3], lqcd_ws_bytes(g, 7, 12));
    lqcd_geom_free(g);
  }
  for (int prec = P_F64; prec <= P_BF16; ++prec)
    for (int nrhs : {1, 2, 4, 12})
      for (int both = 0; both < 2; ++both)
        for (long V2 = 16; V2 < 40000; V2 += 8) {
          const int n = parts_stride(hop_nparts(hop(prec, V2, nrhs, both != 0, 0.0)));
          const int max = hop_max_parts(V2) > 2048 ? hop_max_parts(V2) : 2048;
          CHECK(n <= max, "prec %d nrhs %d both %d V2 %ld: %d partials", prec, nrhs, both, V2, n);
          if (failures > 10) return;
        }
}

// Partial sums of the meson contraction: within the bound the header gives, hence
// within the fixed array for every lattice that lqcd_meson_noalloc accepts, and
// within the smallest workspace.
static void meson_scratch() {
  constexpr size_t kPartial = 256 * 2 * sizeof(double);
  CHECK(64 * meson_nchunk(32 * 32 * 32, 64) * kPartial == 8u << 20, "32^3x64: %d", meson_nchunk(32 * 32 * 32, 64));
  for (int T = 4; T <= 4096; T += T < 128 ? 2 : 62)
    for (long V3 = 8; V3 <= 262144; V3 += V3 < 4096 ? 8 : V3 / 64 * 4) {
      const size_t limit = (size_t)T * ((V3 + 255) / 256), n = (size_t)T * meson_nchunk(V3, T);
      CHECK(n <= (limit > 4096 ? limit : 4096), "T %d V3 %ld: %zu partials", T, V3, n);
      if (limit * kPartial <= LQCD_NOALLOC_SCRATCH_BYTES)
        CHECK(n * kPartial <= LQCD_NOALLOC_SCRATCH_BYTES, "T %d V3 %ld: %zu partials", T, V3, n);
      const size_t ws = (size_t)8 * 24 * padded_sites(V3 * T / 2) * 16;  // the FP64 vectors of one rhs
      CHECK(n * kPartial <= ws, "T %d V3 %ld: %zu partials, workspace %zu", T, V3, n, ws);
      if (failures > 10) return;
    }
}

int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) {
    if (!strcmp(argv[i], "small_launches")) small_launches();
    else if (!strcmp(argv[i], "own_configurations")) own_configurations();
    else if (!strcmp(argv[i], "workspace_bytes")) workspace_bytes();
    else if (!strcmp(argv[i], "meson_scratch")) meson_scratch();
    else if (!strcmp(argv[i], "tuning_round_trip")) tuning_round_trip();
    else if (!strcmp(argv[i], "converted_configurations")) converted_configurations();
    else {
      printf("unknown check %s\n", argv[i]);
      return 2;
    }
  }
  return failures ? 1 : 0;
}
