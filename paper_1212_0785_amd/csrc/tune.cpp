// Launch-shape and link-form decisions and their persisted tuning table
// (the auto-tuner of Sec. 4, for the choices this library offers): per
// lattice and storage, the Dslash shape (one site per work-item, two
// wavefronts per 64 sites, or one wavefront per hop), its link streaming, site
// order and workgroups per CU, the staple-force shape (one link per work-item,
// plane split, or four directions of 64 sites per block in the tiled walk), and
// the compact link form of the hop and staple kernels (two rows, or row 0 and
// column 2).
//
// Precedence: environment override (HMC_DSLASH_SPLIT, HMC_GFORCE_PLANES,
// HMC_LINK_FORM, HMC_LINK_STREAM, HMC_DSLASH_ORDER, HMC_DSLASH_OCC) > tuned
// entry > built-in rule measured on MI355X.
// HMC_TUNE_DB names a table file loaded on first use; hmc_autotune fills and
// saves entries.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "internal.h"

namespace hmc {

namespace {

using Key = std::tuple<int, int, int, int, int, int>;  // L0..L3, kind, prec

struct Entry {
  int choice;
  double us;
};

struct Table {
  std::mutex mu;
  std::map<Key, Entry> map;
  bool env_loaded = false;
};

// Bumped whenever an entry may have changed (recorded solver launches
// depend on the decisions in force when they were recorded).
std::atomic<uint64_t> g_generation{1};

Table& table() {
  static Table t;
  return t;
}

Key make_key(const int* L, int kind, int prec) { return Key(L[0], L[1], L[2], L[3], kind, prec); }

const char* const kKindNames[] = {"dslash",        "gauge_force",  "dslash_links",    "gauge_force_links",
                                  "dslash_stream", "dslash_order", "dslash_occupancy"};
constexpr int kNumKinds = 7;

const char* kind_name(int kind) { return kKindNames[kind]; }

int kind_of(const char* name) {
  for (int k = 0; k < kNumKinds; ++k)
    if (std::strcmp(name, kKindNames[k]) == 0) return k;
  return -1;
}

bool valid_choice(int kind, int c) {
  switch (kind) {
    case TUNE_DSLASH: return c == 1 || c == 2 || c == 4;
    case TUNE_GFORCE: return c == 0 || c == 1 || c == 2;
    case TUNE_DSLASH_STREAM: return c == 0 || c == 1;
    case TUNE_DSLASH_ORDER: return c >= 0 && c <= kMaxYBlock;
    case TUNE_DSLASH_OCC: return c == 0 || c == 2;
    default: return c == LINK_ROWS2 || c == LINK_ROWCOL;
  }
}

// Parses "kind L0 L1 L2 L3 prec choice us" lines; others are skipped.
int load_locked(Table& t, const char* path) {
  FILE* f = std::fopen(path, "r");
  if (!f) return -1;
  char line[256];
  int n = 0;
  while (std::fgets(line, sizeof line, f)) {
    char kind[32];
    int L[4], prec, choice;
    double us;
    if (std::sscanf(line, "%31s %d %d %d %d %d %d %lf", kind, &L[0], &L[1], &L[2], &L[3], &prec, &choice, &us) != 8)
      continue;
    const int k = kind_of(kind);
    if (k < 0 || !valid_choice(k, choice) || prec < 0 || prec > 3) continue;
    t.map[make_key(L, k, prec)] = Entry{choice, us};
    ++n;
  }
  std::fclose(f);
  return n;
}

void ensure_env_loaded(Table& t) {
  if (t.env_loaded) return;
  t.env_loaded = true;
  if (const char* p = std::getenv("HMC_TUNE_DB")) load_locked(t, p);
}

int env_int(const char* name) {
  const char* e = std::getenv(name);
  return e ? std::atoi(e) : -1;
}

}  // namespace

int tune_lookup(const int* L, int kind, int prec) {
  Table& t = table();
  std::lock_guard<std::mutex> lk(t.mu);
  ensure_env_loaded(t);
  auto it = t.map.find(make_key(L, kind, prec));
  return it == t.map.end() ? -1 : it->second.choice;
}

void tune_store(const int* L, int kind, int prec, int choice, double us) {
  Table& t = table();
  std::lock_guard<std::mutex> lk(t.mu);
  ensure_env_loaded(t);
  t.map[make_key(L, kind, prec)] = Entry{choice, us};
  ++g_generation;
}

int tune_load(const char* path) {
  Table& t = table();
  std::lock_guard<std::mutex> lk(t.mu);
  ensure_env_loaded(t);
  ++g_generation;
  return load_locked(t, path);
}

uint64_t tune_generation() { return g_generation.load(); }

int tune_save(const char* path) {
  Table& t = table();
  std::lock_guard<std::mutex> lk(t.mu);
  // merge: entries already in the file that this process does not hold are kept
  std::map<Key, Entry> merged;
  {
    Table tmp;
    if (load_locked(tmp, path) >= 0) merged = tmp.map;
  }
  for (const auto& kv : t.map) merged[kv.first] = kv.second;
  const std::string tmp_path = std::string(path) + ".tmp";
  FILE* f = std::fopen(tmp_path.c_str(), "w");
  if (!f) return -1;
  std::fprintf(f,
               "# kind L0 L1 L2 L3 prec choice us\n"
               "# dslash: choice 1 = one site per work-item, 2 = two wavefronts per site, 4 = one wavefront per hop; us per "
               "CG iteration in a solve\n"
               "# gauge_force: choice 0 = one link per work-item, 1 = plane split, 2 = four directions of 64 sites per "
               "block; us per launch\n"
               "# dslash_links, gauge_force_links: reals read per SU(3) link, 12 = two rows, 10 = row 0 and column 2\n"
               "# dslash_stream: 1 = non-temporal link loads and output stores\n"
               "# dslash_order: 1 = tiled site order (one site per work-item shape), n >= 2 = tiled in y-blocks of n "
               "64-site chunks\n"
               "# dslash_occupancy: workgroups per CU of the tiled order, 2 = at most two, 0 = as registers allow\n");
  for (const auto& kv : merged) {
    const Key& k = kv.first;
    std::fprintf(f, "%s %d %d %d %d %d %d %.3f\n", kind_name(std::get<4>(k)), std::get<0>(k), std::get<1>(k),
                 std::get<2>(k), std::get<3>(k), std::get<5>(k), kv.second.choice, kv.second.us);
  }
  std::fclose(f);
  return std::rename(tmp_path.c_str(), path) == 0 ? (int)merged.size() : -1;
}

bool tune_env_forced() {
  return env_int("HMC_DSLASH_SPLIT") >= 0 || env_int("HMC_GFORCE_PLANES") >= 0 || env_int("HMC_LINK_FORM") >= 0 ||
         env_int("HMC_LINK_STREAM") >= 0 || env_int("HMC_DSLASH_ORDER") >= 0 || env_int("HMC_DSLASH_OCC") >= 0;
}

namespace {
// HMC_LINK_FORM: 18 = all entries even on SU(3) links, 12, 10; else unset.
int forced_link_form() {
  static const int forced = [] {
    const int v = env_int("HMC_LINK_FORM");
    return (v == LINK_FULL || v == LINK_ROWS2 || v == LINK_ROWCOL) ? v : -1;
  }();
  return forced;
}
}  // namespace

int dslash_link_form(const LatArg& g, hmc_prec prec) {
  if (forced_link_form() > 0) return forced_link_form();
  const int t = tune_lookup(g.L, TUNE_DSLASH_LINKS, prec);
  if (t > 0) return t;
  // Two rows below 2^20 half-lattice sites: they rebuild a reunitarised FP64
  // link bit for bit, row 0 and column 2 do not (error of Mhat at 24^3x44, two
  // rows / row 0 + column 2: FP64 9.34e-17 / 9.92e-17, FP32 4.83e-8 / 4.97e-8,
  // FP16 2.78e-4 / 2.80e-4).  From there a sixth fewer link bytes decide.
  // Measured (Mhat, us, the same order): FP64 20^3x40 70.1 / 64.3, 24^3x44 140 /
  // 128, 28^3x60 298 / 273; FP32 20^3x40 35.6 / 33.4, 28^3x60 171 / 159; FP16
  // 24^3x48 51.8 / 45.9, 32^3x64 155 / 149; BF16 24^3x48 44.7 / 42.6, 32^3x64
  // 149 / 138
  return g.Vh >= 1 << 20 ? LINK_ROWCOL : LINK_ROWS2;
}

namespace {
// Bytes of all links in the ten-real form at storage prec.
double compact_link_bytes(const LatArg& g, hmc_prec prec) {
  return 8.0 * g.Vh * (prec == HMC_F64 ? 80 : prec == HMC_F32 ? 40 : 20);
}
}  // namespace

bool dslash_link_stream(const LatArg& g, hmc_prec prec) {
  static const int forced = env_int("HMC_LINK_STREAM");
  if (forced >= 0) return forced != 0;
  const int t = tune_lookup(g.L, TUNE_DSLASH_STREAM, prec);
  if (t >= 0) return t != 0;
  // Streaming pays once the links a hop reads no longer stay in the 256 MB
  // last-level cache from one hop to the next, beside the vectors; before that
  // the hints only bypass it.  Measured (Mhat, us, plain / streamed, in the link
  // form and shape of the rules, with the ten-real links' MB): FP64 20^3x40 (102
  // MB) 70.1 / 75.6, 20x24x24x44 (162) 114 / 115 and 281 / 280 per iteration of a
  // solve, 24^3x44 (195) 145 / 140, 32^3x64 (671) 565 / 445; FP32 24^3x44 (97) 66.8
  // / 81.4, 24x28x28x52 (157) 123 / 127 and 396 / 394, 28^3x60 (211) 180 / 171,
  // 32^3x64 (336) 298 / 258; BF16 32^3x64 (168) 140 / 141 and 538 / 537, 40^3x80
  // (410) 358 / 325
  return compact_link_bytes(g, prec) >= 150e6;
}

int dslash_tiled_order(const LatArg& g, hmc_prec prec) {
  if (!tiled_order_valid(g)) return 0;
  static const int forced = env_int("HMC_DSLASH_ORDER");
  // an order the lattice does not admit falls back to whole z-planes
  if (forced >= 0) return forced == 0 ? 0 : tiled_order_valid(g, forced) ? forced : 1;
  const int t = tune_lookup(g.L, TUNE_DSLASH_ORDER, prec);
  if (t >= 0) return t == 0 ? 0 : tiled_order_valid(g, t) ? t : 1;
  // Whole z-planes for FP64 where its rule has one site per work-item, once a
  // t-slice outgrows an XCD's L2 (linear / tiled with two blocks per CU, Mhat:
  // 32^3x64 495 / 502 us, 40^3x80 1333 / 1255).  The narrower storages stay
  // linear: the cap costs them (40^3x80, linear / tiled with / without it: FP32
  // 680 / 682 / 666 us, FP16 341 / 434 / 336, BF16 323 / 424 / 320), and what
  // is left without it is nothing at 32^3x64 (258 / 259, 150 / 151, 146 / 142).
  return prec == HMC_F64 && g.Vh >= 3 << 19 && dslash_shape(g, prec) == 1 ? 1 : 0;
}

int dslash_tiled_occupancy(const LatArg& g, hmc_prec prec) {
  static const int forced = env_int("HMC_DSLASH_OCC");
  if (forced >= 0) return forced == 0 ? 0 : 2;
  const int t = tune_lookup(g.L, TUNE_DSLASH_OCC, prec);
  if (t >= 0) return t;
  return 2;
}

int staple_link_form(const LatArg& g) {
  if (forced_link_form() > 0) return forced_link_form();
  const int t = tune_lookup(g.L, TUNE_GFORCE_LINKS, HMC_F64);
  if (t > 0) return t;
  // measured on MI355X, ten reals a link against twelve: 8^4 10.4 and 8.3 us,
  // 18x10x14x26 34.1 and 27.4, 20^3x40 141 and 112, 32^3x64 893 and 782, 48^3x96
  // 4.64 and 3.98 ms (the kernel waits for its arithmetic before its bytes).
  // Below 256 half-lattice sites the launch follows the answer that callers
  // have had from the query there, ten, though twelve are faster (4^3x6 10.2
  // and 8.1 us).
  return g.Vh < kThreads ? LINK_ROWCOL : LINK_ROWS2;
}

int dslash_shape(const LatArg& g, hmc_prec prec) {
  static const int forced = [] {
    const int v = env_int("HMC_DSLASH_SPLIT");
    return v < 0 ? -1 : v == 1 ? 4 : (v == 2 || v == 4) ? v : 1;
  }();
  if (forced > 0) return forced;
  const int t = tune_lookup(g.L, TUNE_DSLASH, prec);
  if (t > 0) return t;
  // One wavefront per hop until the launch fills the chip so many times over
  // that the one-site kernel's smaller traffic wins, for the narrower storages
  // sooner, whose hop is bound by its instructions and whose p-update adds four
  // times the partial sums of the split shapes.  Measured with the link form and
  // streaming of the rules, us, shapes 1 / 2 / 4, Mhat and per iteration of a
  // solve: FP64 20^3x40 95 / 79 / 70, 224 / 195 / 172; 24^3x44 160 / 150 / 140, 382
  // / 367 / 344; 28^3x60 347 / 318 / 298, 846 / 808 / 772; 32^3x64 477 / 472 / 445,
  // 1225 / 1204 / 1156; 40^3x80, where the tiled order keeps neighbours in L2, 1256
  // / 1310 / 1292, 3097 / 3284 / 3244.  (Lattices that do not admit that order go
  // the same way without gaining by it: 36^3x72 872 / 805 / 768, 2094 / 2009 / 1947;
  // 40^3x84 1385 / 1288 / 1238, 3394 / 3319 / 3245.)  FP32 20^3x40 43 / 41 / 36, 133
  // / 134 / 122; 24x28x28x52 139 / 136 / 127, 402 / 416 / 394; 28^3x60 188 / 183 /
  // 171, 546 / 562 / 536; 32^3x64 258 / 261 / 247, 796 / 850 / 825.  FP16 20^3x40 32
  // / 31 / 26, 117 / 121 / 110; 20x24x24x44 38 / 42 / 38, 147 / 163 / 155; 28^3x60
  // 90 / 82 / 86, 365 / 383 / 383.  BF16 20^3x40 28 / 26 / 24, 107 / 109 / 103;
  // 20x24x24x44 34 / 36 / 34, 136 / 147 / 143; 28^3x60 82 / 74 / 75, 342 / 362 / 360.
  // Two wavefronts (2) lead nowhere in a solve; tables and overrides
  // may ask for them.
  // (below one block choice 1 runs as 4: dslash_run_shape)
  if (prec == HMC_F64) return g.Vh < kThreads ? 1 : g.Vh < 3 << 19 ? 4 : 1;
  return g.Vh < (prec == HMC_F32 ? 1 << 19 : 1 << 18) ? 4 : 1;
}

bool exp_update_stream(const LatArg& g) {
  static const int forced = env_int("HMC_EXP_STREAM");
  if (forced >= 0) return forced != 0;
  // measured on MI355X: 16^3x32 27.4 -> 29.8 us (the fields stay in the
  // last-level cache between launches, which the hints bypass); 24^3x48
  // 156 -> 144 us, 32^4 270 -> 250 us; 48^3x96 2.56-2.58 ms either way
  return g.Vh >= (1 << 18);
}

bool fermion_force_stream(const LatArg& g) {
  static const int forced = env_int("HMC_FF_STREAM");
  if (forced >= 0) return forced != 0;
  // measured on MI355X: 24^3x48 174 -> 156 us, 48^3x96 2.99 -> 2.90 ms;
  // 16^3x32 31.6 against 31.7 us
  return g.Vh >= (1 << 18);
}

bool gauge_force_stream(const LatArg& g) {
  static const int forced = env_int("HMC_GF_STREAM");
  if (forced >= 0) return forced != 0;
  // measured on MI355X (site-blocked staple force): 24^3x48 321 -> 295 us,
  // 48^3x96 4.65 -> 4.57 ms
  return g.Vh >= (1 << 18);
}

int plaquette_shape(const LatArg&) {
  static const int forced = env_int("HMC_PLAQ_PAIRS");
  if (forced >= 0) return forced == 0 ? 0 : 1;
  // measured on MI355X: 1.78 -> 1.36 ms at 48^3x96, 26.5 -> 21.3 us at 16^3x32
  return 1;
}

int plaquette_link_form(const LatArg& g) {
  static const int forced = env_int("HMC_PLAQ_FORM");
  if (forced == LINK_ROWS2 || forced == LINK_ROWCOL) return forced;
  // measured on MI355X (plane-paired sum): two rows 1.33 ms against 1.69 ms
  // with row 0 + column 2 at 48^3x96, 21.4 against 29.6 us at 16^3x32 (the
  // reconstruction lengthens the latency-bound chain); the per-site form
  // follows the staple force
  return plaquette_shape(g) == 1 ? (int)LINK_ROWS2 : staple_link_form(g);
}


int gauge_force_shape(const LatArg& g) {
  static const int forced = env_int("HMC_GFORCE_PLANES");
  if (forced >= 0) return forced == 0 ? 0 : forced == 2 ? 2 : 1;
  const int t = tune_lookup(g.L, TUNE_GFORCE, HMC_F64);
  if (t >= 0) return t;
  // measured on MI355X: four directions per block in the tiled walk are
  // 27% faster than one link per work-item at 48^3x96 and 13% faster at
  // 16^3x32 (the plane split: 6% slower and 20% slower)
  return 2;
}

}  // namespace hmc
