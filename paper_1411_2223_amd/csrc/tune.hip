// tune.hip -- autotuner for the Dslash launch (QUDA's automatic choice of
// running parameters is the idea, section "CPS & QUDA"; this one is written
// for gfx950): times each candidate RHS tile (columns per thread) on the
// caller's own buffers and keeps the fastest per (device, lattice, link tier,
// vector tiers, epilogue, columns).  Results live in memory and, when the
// environment variable ASQ_TUNE_CACHE names a file, in that file as one JSON
// object mapping each key to its launch variant code.
// ASQ_TUNE=0 turns timing off and uses the built-in defaults.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "asq_internal.h"

namespace asq {
namespace {

std::mutex g_mu;
std::map<std::string, int> g_cache;
bool g_loaded = false;

// The architecture name of a device, asked for once: the query costs more than the
// rest of a lookup.
std::string arch_of(int device) {
  static std::mutex mu;
  static std::map<int, std::string> names;
  std::lock_guard<std::mutex> lk(mu);
  auto it = names.find(device);
  if (it != names.end()) return it->second;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) return "gfx";
  return names[device] = prop.gcnArchName;
}

// What a configuration's string key is made of.  g_quick maps it to the recorded
// variant, so that a call that was tuned before builds no string (a public operator
// call at 8^4 takes 5.3 us on the GPU; the two string lookups took 1.6 us of its host
// time).  Filled from g_cache and emptied when that changes, under g_mu.
using QuickKey = std::array<int, 10>;
std::map<QuickKey, int> g_quick;

QuickKey quick_key(const asq_gauge* g, int link, int in, int out, int epi, int ncol) {
  return {g->device, g->geom.X, g->geom.Y, g->geom.Z, g->geom.T, link, in, out, epi, ncol};
}

std::string key_of(const asq_gauge* g, int link, int in, int out, int epi, int ncol) {
  char buf[160];
  const std::string name = arch_of(g->device);
  const char* arch = name.c_str();
  snprintf(buf, sizeof(buf), "%s/%dx%dx%dx%d/L%d/I%d/O%d/E%d/N%d", arch, g->geom.X, g->geom.Y, g->geom.Z,
           g->geom.T, link, in, out, epi, ncol);
  for (char* c = buf; *c; ++c)
    if (*c == ' ' || *c == ':') *c = '_';
  return buf;
}

void load_cache_locked() {
  if (g_loaded) return;
  g_loaded = true;
  const char* path = getenv("ASQ_TUNE_CACHE");
  if (!path || !*path) return;
  FILE* f = fopen(path, "r");
  if (!f) return;
  // the file this library writes: one "key": code pair per line
  char line[256], k[200];
  int v;
  while (fgets(line, sizeof(line), f))
    if (sscanf(line, " \"%199[^\"]\" : %d", k, &v) == 2) g_cache[k] = v;
  fclose(f);
}

void save_cache_locked() {
  const char* path = getenv("ASQ_TUNE_CACHE");
  if (!path || !*path) return;
  FILE* f = fopen(path, "w");
  if (!f) return;
  fprintf(f, "{\n");
  size_t n = 0;
  for (auto& kv : g_cache)
    fprintf(f, "  \"%s\": %d%s\n", kv.first.c_str(), kv.second, ++n < g_cache.size() ? "," : "");
  fprintf(f, "}\n");
  fclose(f);
}

// The recorded variant of a configuration, or -1.
int recorded_locked(const asq_gauge* g, int link, int in, int out, int epi, int ncol) {
  load_cache_locked();
  const QuickKey q = quick_key(g, link, in, out, epi, ncol);
  auto f = g_quick.find(q);
  if (f != g_quick.end()) return f->second;
  auto it = g_cache.find(key_of(g, link, in, out, epi, ncol));
  if (it == g_cache.end() || it->second < 0) return -1;
  return g_quick[q] = it->second;
}

int default_rtile(int link, int ncol) {
  if (ncol <= 1) return 1;
  if (link == LINK_F64_R18) return 2;
  return ncol >= 4 ? 4 : 2;
}

// How far from the best a candidate of the tuner may be to be timed further.  The LDS
// form shortens a launch by up to 10 %, and wherever it was the best the same launch
// without it was within 6 % of the best without it (44 configurations, 8^4 to 48^3 x 96,
// 1 to 96 columns); launches repeat to a few percent.  First call of 12 FP64
// columns at 16^3 x 32 with every LDS form, and every candidate timed twice, 220 ms, so
// 109; of 96 FP16 columns at 20^3 x 64 4.6 and 2.2 s.
constexpr float kTuneNear = 1.15f;

bool tuning_on() {
  const char* e = getenv("ASQ_TUNE");
  return !(e && e[0] == '0');
}

}  // namespace

// ASQ_VARIANT=<code> (decimal) replaces the tuned launch variant wherever the
// library builds that variant for the tier (tests use it to run every variant
// through the solver epilogues).
int forced_variant(int link, int in) {
  const char* e = getenv("ASQ_VARIANT");
  if (!e || !*e) return -1;
  const int v = atoi(e);
  return variant_built(link, in, v) ? v : -1;
}

int tuned_rtile(const asq_gauge* g, int link, int in, int out, int epi, int ncol) {
  const int fv = forced_variant(link, in);
  // a forced tile wider than the batch, or whose LDS window does not fit this
  // lattice, is ignored, except the matrix-core form, which masks its idle
  // columns; that form is for many columns and not forced on one or two
  if (fv >= 0 && !(fv & kMfmaBit) && tile_cols(fv) <= (ncol > 1 ? ncol : 1) && variant_fits(g->geom, in, fv)) return fv;
  if (fv >= 0 && (fv & kMfmaBit) && ncol > 2) return fv;
  std::lock_guard<std::mutex> lk(g_mu);
  const int v = recorded_locked(g, link, in, out, epi, ncol);
  // a cache file may come from another build: only variants the tuner itself
  // could have chosen are taken from it
  if (v >= 0 && variant_built(link, in, v) && !(v & kMfmaBit) && tile_cols(v) <= (ncol > 1 ? ncol : 1) &&
      variant_fits(g->geom, in, v))
    return v;
  return default_rtile(link, ncol);
}

// True when tune_dslash would time candidates for this configuration (timing
// on, no recorded winner), so the caller can put trial data in place first.
bool tune_pending(const asq_gauge* g, int link, int in, int ncol, int epi_timed) {
  if (!tuning_on()) return false;
  std::lock_guard<std::mutex> lk(g_mu);
  load_cache_locked();
  return g_cache.count(key_of(g, link, in, in, epi_timed, ncol)) == 0;
}

// Time the PLAIN Dslash (the loop shared by every epilogue) for each tile on
// in_buf -> out_buf and record the winner for every epilogue; with
// epi = EPI_CANON, time and record the public operator on the canonical
// layouts instead.  Buffers are the caller's: in_buf is only read, out_buf is
// scratch.  persist = false keeps the winners out of the ASQ_TUNE_CACHE file
// (timings taken while other work may share the device).
int tune_dslash(const asq_gauge* g, int link, int in, int ncol, const void* in_buf, void* out_buf,
                hipStream_t s, int epi_timed, bool persist) {
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (recorded_locked(g, link, in, in, epi_timed, ncol) >= 0) return ASQ_OK;
    if (g_cache.count(key_of(g, link, in, in, epi_timed, ncol))) return ASQ_OK;
  }
  const std::string kp = key_of(g, link, in, in, epi_timed, ncol);
  int best = default_rtile(link, ncol);
  int best_update = best;  // the UPDATE epilogue's pick: no tile wider than 8 columns
  if (tuning_on()) {
    DslashArgs a;
    memset(&a, 0, sizeof(a));
    a.g = g->geom;
    a.out_parity = 1;
    a.ncol = ncol;
    a.links = g->links[link];
    a.in = in_buf;
    a.out = out_buf;
    a.mask = MASK_ALL;
    a.nblk = g->nblk;
    a.coeff_fat = g->desc.fat_scale;
    a.coeff_long = g->desc.long_scale;
    hipEvent_t e0, e1;
    ASQ_HIP_TRY(hipEventCreate(&e0));
    ASQ_HIP_TRY(hipEventCreate(&e1));
    float best_ms = 1e30f, best_update_ms = 1e30f;
    // columns per thread x hop-loop form x block order (orders differ only when
    // there are several tiles) x XCD slabs or one global sweep (of single blocks
    // or of runs of blocks per XCD)
    std::vector<int> cands;
    for (int gs = 0; gs < 2; ++gs)
      for (int order = 0; order < 4; ++order)
        for (int pipe = 0; pipe < 2; ++pipe)
          for (int cols : {1, 2, kThreeCols, 4, 6, 8, 12})
            if (order == 0 || ncol > tile_cols(cols)) cands.push_back(make_rtile(cols, pipe, order, gs != 0));
    // runs of 16, 64 or 256 blocks per XCD inside the sweep: pipelined loop, the
    // first two block orders
    for (int chunk = 1; chunk <= 3; ++chunk)
      for (int order = 0; order < 2; ++order)
        for (int cols : {1, 2, kThreeCols, 4, 6, 8, 12})
          if (order == 0 || ncol > tile_cols(cols)) cands.push_back(make_rtile(cols, true, order, true, chunk));
    // one-column tiles with streamed links, where the tier has that form
    {
      const size_t n = cands.size();
      for (size_t q = 0; q < n; ++q)
        if ((cands[q] & 0xff) == 1 && variant_built(link, in, cands[q] | kStreamBit)) cands.push_back(cands[q] | kStreamBit);
    }
    // launches of few blocks: the split form
    if ((long)g->nblk * ncol <= kSplitMaxBlocks) cands.push_back(kSplitCode);
    // The solver runs D_oe forwards and D_eo backwards, so each sweep starts on
    // the links and vectors the previous one left in the memory-side cache; the
    // candidates are timed in that pattern (pairs of launches), best of two.
    auto pair = [&](int r) {
      bool ok = true;
      for (int k = 0; k < 2 && ok; ++k) {
        a.out_parity = k ? 0 : 1;
        a.reverse = k;
        ok = launch_dslash(link, in, in, epi_timed, r, a, s) == ASQ_OK;
      }
      return ok;
    };
    // A candidate whose first timing is far from the best is not timed again, and its
    // LDS form is not tried (kTuneNear).
    auto time_one = [&](int r) {
      const int cols = tile_cols(r);
      float ms = 1e30f;
      if (cols > 1 && cols > ncol) return ms;  // a wider tile than the batch only wastes lanes
      if (!pair(r)) return ms;  // warm-up
      // the UPDATE epilogue also keeps r, x and the direction of every column of
      // the tile live: the 12-column tile loses occupancy there that the plain
      // loop timed here does not show
      const bool three_ok = cols != 3 || (long)g->nblk * ((ncol + 2) / 3) >= kThreeUpdateMinBlocks;
      const bool update_ok = cols <= 8 && three_ok;
      for (int rep = 0; rep < 2; ++rep) {
        float t = 0;
        // a candidate whose timing fails is skipped
        if (hipEventRecord(e0, s) != hipSuccess || !pair(r) || !pair(r) || hipEventRecord(e1, s) != hipSuccess ||
            hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&t, e0, e1) != hipSuccess)
          return 1e30f;
        if (t < ms) ms = t;
        if (ms > kTuneNear * best_ms && !(update_ok && ms <= kTuneNear * best_update_ms)) break;
      }
      if (log_enabled()) fprintf(stderr, "[asq] tune %s R=%d %.4f ms\n", kp.c_str(), r, ms / 4);
      if (ms < best_ms) {
        best_ms = ms;
        best = r;
      }
      if (update_ok && ms < best_update_ms) {
        best_update_ms = ms;
        best_update = r;
      }
      return ms;
    };
    std::vector<float> took;
    for (int r : cands) took.push_back(time_one(r));
    // the pipelined candidates near the best with the LDS window (windows too large for
    // LDS are refused; a candidate that fails to launch is skipped)
    const float near_ms = kTuneNear * std::max(best_ms, best_update_ms);
    for (size_t q = 0; q < cands.size(); ++q)
      if (took[q] <= near_ms && variant_built(link, in, cands[q] | kLdsBit)) time_one(cands[q] | kLdsBit);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
  }
  std::lock_guard<std::mutex> lk(g_mu);
  g_quick.clear();
  if (epi_timed == EPI_CANON) {
    g_cache[kp] = best;
  } else {
    for (int epi = EPI_PLAIN; epi <= EPI_RESID; ++epi)
      for (int out = VEC_F64; out <= VEC_F16; ++out)
        g_cache[key_of(g, link, in, out, epi, ncol)] = epi == EPI_UPDATE ? best_update : best;
  }
  if (persist) save_cache_locked();
  return ASQ_OK;
}

}  // namespace asq
