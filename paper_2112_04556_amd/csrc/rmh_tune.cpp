// Stencil launch configuration cache.  Entries are keyed by lattice extents, dtype, the number of
// link fields per launch and the purpose of the launch (rmh_purpose); the autotuner
// (rmh_autotune_laplacian) fills them from timed candidates, rmh_tune_save / rmh_tune_load keep
// them in a JSON file stamped with the device architecture and the HIP runtime version, and
// otherwise the built-in defaults apply.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cstdlib>
#include <initializer_list>
#include <map>
#include <mutex>
#include <string>
#include <tuple>

#include "rmh.h"
#include "rmh_tune.h"

namespace rmh {

namespace {
using Key = std::tuple<int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t>;  // L0..L3, dtype, n, purpose
struct Entry {
  HopConfig cfg;
  double ms;
};
std::mutex g_mu;
std::map<Key, Entry> g_cache;

Key key_of(const Geom& g, int32_t dtype, int32_t n_rhs, int32_t purpose) {
  return Key(g.L0, g.L1, g.L2, g.L3, dtype, n_rhs, purpose);
}

// The first of the given x3 walks that divides L3 (0: none does).
int32_t walk_of(const Geom& g, std::initializer_list<int> ks) {
  for (int k : ks)
    if (g.L3 % k == 0) return k;
  return 0;
}

// The tiled walk's tile and segment length for a launch: the shape with the least estimated time.  A CU
// holds 8 waves in FP64 (16 in FP32) and 160 KB of LDS; its time is the number of blocks it gets, each
// w waves walking K planes after a prologue worth 1.5, lengthened by the halo rows read from memory and
// by having few waves to hide latency with.  Of the up to 40 best shapes timed on each of 17 lattices
// (8x12x16x20 to 32^3x64, odd extents among them) the estimate's pick was the fastest or within 5 %.
bool tile_shape(const Geom& g, int32_t dtype, int32_t n_rhs, HopConfig* out) {
  const int max_waves = dtype == RMH_F64 ? 8 : 16;
  const double lds_column = 2.0 * (dtype == RMH_F64 ? 272 : 144);
  double best = 0.0;
  for (int R2 = 1; R2 <= g.L2 && g.L0 * R2 <= 256; ++R2)
    for (int R1 = 1; R1 <= g.L1 && g.L0 * R1 * R2 <= 256; ++R1) {
      HopConfig c;
      c.form = kFormMatrix;
      c.nv = 2;
      c.order = 1;
      c.xcd_remap = 1;
      c.block = g.L0 * R1 * R2;
      c.tile2 = R2;
      c.walk = g.L3;
      HopTile t;
      if (!hop_tile_of(g, c, &t) || t.R1 != R1 || t.R2 != R2) continue;
      const int w = (c.block + 31) / 32;
      const int fit = std::max(1, std::min(max_waves / w, (int)(160 * 1024 / (lds_column * c.block))));
      const double halo = (R1 < g.L1 ? 0.2 / R1 : 0.0) + (R2 < g.L2 ? 0.2 / R2 : 0.0) + (w < 4 ? 0.08 : 0.0);
      for (int nseg = 1, K; nseg <= g.L3; nseg = (g.L3 - 1) / (K - 1) + 1) {   // each K = ceil(L3 / nseg) once
        K = (g.L3 + nseg - 1) / nseg;
        const int64_t per_cu = ((int64_t)t.n1 * t.n2 * nseg * n_rhs + 255) / 256;
        const double waves = (double)w * std::min<int64_t>(fit, per_cu);
        const double cost = (double)per_cu * w * (K + 1.5) * (1.0 + halo) * (1.0 + 0.5 * max_waves / waves);
        HopConfig ck = c;
        ck.walk = K;
        if ((best == 0.0 || cost < best) && hop_tile_of(g, ck, &t)) {
          best = cost;
          *out = ck;
        }
        if (K == 1) break;
      }
    }
  return best > 0.0;
}

// Microseconds of one FP64 application by a tile (rounds of blocks on a CU, each K planes of the field at 2.9 or,
// with two waves on a SIMD, 3.9 us, more where the lattice's end cuts tiles, and the traffic of a thousand
// site-fields) and by one thread per site with the 3x3 form.  Fitted to 227 launches of 2^16 to 4 M site-fields on
// lattices of any extents; the standard deviations are 6.6 and 5.8 %.
double tile_us(const Geom& g, int32_t n_rhs, const HopConfig& c) {
  HopTile t;
  if (!hop_tile_of(g, c, &t)) return 0.0;
  const int w = (g.L0 * t.R1 * t.R2 + 31) / 32, fit = std::max(1, 8 / w);
  const int64_t blocks = (int64_t)t.n1 * t.n2 * ((g.L3 + t.K - 1) / t.K) * n_rhs, per_cu = (blocks + 255) / 256;
  const int m = w * std::min<int64_t>(fit, per_cu) > 4 ? 2 : 1;   // waves on a SIMD
  const double planes = (double)((per_cu + fit - 1) / fit) * (t.K + 1.5), k = 1e-3 * g.V * n_rhs;
  const int cut = (g.L1 % t.R1 ? 1 : 0) + (g.L2 % t.R2 ? 1 : 0);
  const double halo = (t.R1 < g.L1 ? 1.0 / t.R1 : 0.0) + (t.R2 < g.L2 ? 1.0 / t.R2 : 0.0);
  return planes * ((m == 1 ? 2.9 : 3.9) + 0.3 * m * cut) + k * (0.13 + 0.028 * halo + (g.L0 % 8 ? 0.024 : 0.0)) +
         0.03 * std::max(0.0, k - 700.0);
}
double site_us(const Geom& g, int32_t n_rhs) {
  const double k = 1e-3 * g.V * n_rhs;
  return 3.5 + k * (0.254 + 0.064 / n_rhs) + 0.065 * std::max(0.0, k - 700.0);
}

// Untuned defaults, from sweeps on MI355X.  FP64 and the FP32 launches below 2^20 sites, but for the FP32 moments,
// use the 3x3 form, which needs the fewest operations per hop.
//  - FP64 from 2^16 site-fields on: the tiled walk where its estimate is the lower (36x32x24x28 213 us against 275;
//    16^4 20.0 against 22.5; 24x16x16x24 x 2 68.7 against 82.3), else one thread per site (20^3x16 x 4 146.6 us
//    against 189.1 tiled, 14x13x13x23 x 8 115 against 149), or the hop split below 98304 site-fields where the
//    components' rows begin on whole cache lines (8x12x12x8 x 8 22.4 us against 24.7 by sites, 25.5 tiled;
//    9x11x12x14 x 5, whose rows do not, 36.8 against 27.5).
//  - FP32 from 2^20 sites on: the tiled walk where its waves are full and its runs of sites along x0 and x1 are
//    whole 128-byte lines or 96 sites at least, else the walk with four directions per thread, 4 planes or, from
//    2^21 sites on, 8 (tiled against that walk: 32^3x64 0.260 ms against 0.306; 28x32x48x48 0.288 against 0.308;
//    22x40x44x36 0.343 against 0.232; 40x44x36x28 x 2 0.582 against 0.504).
//  - In smaller FP32 lattices the tile's vector work, the link rebuilt by both lane halves, is the bound: a batch of
//    at least 2^19 site-fields walks with four directions per thread (24^4 x 8 360 us against 372 tiled) where blocks
//    of 64 columns fill the (x0, x1) planes (32x20x24x28 x 3 154 us against 169 by sites), else takes one thread per
//    site in blocks of 256 (20x24x20x32 x 5 199 us against 225 walking, 20x24x24x24 x 2 74.7 against 82.5); smaller
//    launches take one thread per site and direction pair (16^4 x 4 37 us against 43 for the hop split).
//  - smaller launches (FP32: below 2^16 site-fields): four lanes per site, one per direction (hop split),
//    whose four times as many waves hide the latency that one thread per site leaves exposed.  Two
//    directions per lane (FP32 from 24576 site-fields on: four; 16^3x12 9.3 us against 10.4 with two, 8x12x8x8
//    6.8 against 5.2), in blocks of 128 threads where these give the CUs less work than blocks of 256
//    (FP64, 128 against 256: 8^4 5.6 us against 6.3; 8x12x8x8 7.2 against 6.4; 12^4 12.4 against 11.5).
// FP32 Chebyshev moments below 2^20 sites keep the streamed adjoint form.  It is no loss of time (tuned, a batch of 32
// sources at 24^4 takes it too, two fields a thread); another form would move the moments by a few 1e-9, which is
// within their own error (8e-9 at 24^4) and so no gain either.
HopConfig defaults(const Geom& g, int32_t dtype, int32_t n_rhs, int32_t purpose) {
  const bool f64 = dtype == RMH_F64;
  const int64_t work = (int64_t)g.V * n_rhs;
  HopConfig c;
  if (!f64 && purpose == RMH_PURPOSE_MOMENTS && g.V < (1 << 20)) {
    const bool batch = work >= (1 << 19);
    c.form = kFormStream;
    c.nv = 4;
    c.block = batch ? 64 : 256;
    c.xcd_remap = batch ? 1 : 0;
    c.order = batch ? 1 : 2;
    if (batch && !hop_order_ok(g, c)) c.order = 0;
    return c;
  }
  if (!f64 && g.V >= (1 << 20)) {
    HopTile t;
    if (tile_shape(g, dtype, n_rhs, &c) && hop_tile_of(g, c, &t) && c.block % 32 == 0 &&
        ((g.L0 * t.R1) % 32 == 0 || g.L0 * t.R1 >= 96))
      return c;
    c = HopConfig();
    c.form = kFormAdjoint;
    c.block = 256;
    c.xcd_remap = 1;
    c.nv = 4;
    c.order = 0;
    c.walk = g.V < (1 << 21) ? walk_of(g, {4, 8, 16, 2}) : walk_of(g, {8, 4, 16, 2});
    return c;
  }
  c.form = kFormMatrix;
  c.xcd_remap = 1;
  if (f64 && work >= (1 << 16) && tile_shape(g, dtype, n_rhs, &c)) {
    if (tile_us(g, n_rhs, c) <= site_us(g, n_rhs)) return c;
    const bool split = work < 98304 && g.V % 32 == 0;
    c = HopConfig();
    c.form = kFormMatrix;
    c.xcd_remap = split ? 0 : 1;
    c.nv = split ? 2 : 4;
    c.block = split ? 256 : 64;
    c.order = split ? 2 : 0;
  } else if (work >= (1 << 19)) {
    // (also the FP64 lattices too large for the tile: more than 2^24 sites, or rows longer than a block)
    const bool sites = !f64 && (int64_t)g.L0 * g.L1 % 64 != 0;
    c.nv = 4;
    c.block = f64 ? 128 : sites ? 256 : 64;
    c.walk = f64 ? walk_of(g, {8, 4, 2}) : sites ? 0 : walk_of(g, {4, 8, 2});
  } else if (!f64 && work >= (1 << 16)) {
    c.nv = 2;
    c.block = 128;
  } else {
    // a block of 128 threads holds 16 sites' two direction pairs, one of 256 threads 32
    const int64_t small = (work + 16 * 256 - 1) / (16 * 256), large = 2 * ((work + 32 * 256 - 1) / (32 * 256));
    c.nv = f64 || work < 24576 ? 2 : 4;
    c.block = c.nv == 2 && small < large ? 128 : 256;
    c.order = 2;
    c.xcd_remap = 0;
  }
  return c;
}

// The shapes found so far (the search takes microseconds to tens of them, a small launch as much), by
// lattice, dtype, batch and purpose; dropped when it grows past 256 entries.
std::map<Key, HopConfig> g_shapes;
HopConfig defaults_kept(const Geom& g, int32_t dtype, int32_t n_rhs, int32_t purpose) {
  const Key k = key_of(g, dtype, n_rhs, purpose);
  const auto it = g_shapes.find(k);
  if (it != g_shapes.end()) return it->second;
  if (g_shapes.size() >= 256) g_shapes.clear();
  return g_shapes[k] = defaults(g, dtype, n_rhs, purpose);
}

// nearest batch size among the entries of (L, dtype, purpose)
const HopConfig* nearest(const Geom& g, int32_t dtype, int32_t n_rhs, int32_t purpose) {
  const HopConfig* best = nullptr;
  int32_t dist = 0;
  for (auto& kv : g_cache) {
    const Key& k = kv.first;
    if (std::get<0>(k) != g.L0 || std::get<1>(k) != g.L1 || std::get<2>(k) != g.L2 || std::get<3>(k) != g.L3 ||
        std::get<4>(k) != dtype || std::get<6>(k) != purpose)
      continue;
    const int32_t d = std::abs(std::get<5>(k) - n_rhs);
    if (!best || d < dist) {
      best = &kv.second.cfg;
      dist = d;
    }
  }
  return best;
}

// a configuration that was stored for another batch size keeps only what fits this one
HopConfig fit_batch(HopConfig c, int32_t n_rhs) {
  if (c.ns > 1 && n_rhs % c.ns) c.ns = 1;
  return c;
}
}  // namespace

const char* hop_config_error(const Geom& g, const HopConfig& c, int32_t dtype) {
  // The tiled walk's block counts columns and its tile and walk fit any extents, so on a lattice that takes it their
  // whole range is valid (the built-in shapes are among it); anywhere else the launch would be one of the others.
  HopTile t;
  if (c.block >= 1 && c.block <= 256 && c.tile2 >= 1 && hop_tile_of(g, c, &t))
    return c.xcd_remap == 0 || c.xcd_remap == 1 ? nullptr : "xcd_remap must be 0 or 1";
  if (c.form < kFormAdjoint || c.form > kFormStream) return "form must be 0, 1 or 2";
  if (c.block != 64 && c.block != 128 && c.block != 256) return "block must be 64, 128 or 256";
  if (c.nv != 1 && c.nv != 2 && c.nv != 4) return "nv must be 1, 2 or 4";
  if (c.nv == 1 && c.form != kFormMatrix) return "nv = 1 needs form 1 (3x3 products)";
  if ((c.block * c.nv / 4) % 64) return "block * nv / 4 must be a multiple of 64";
  if (c.order < 0 || c.order > 3) return "order must be 0, 1, 2 or 3";
  if (c.walk < 0 || c.walk > 64) return "walk must be in [0, 64]";
  if (c.xcd_remap != 0 && c.xcd_remap != 1) return "xcd_remap must be 0 or 1";
  if (c.ns != 1 && c.ns != 2 && c.ns != 4) return "ns must be 1, 2 or 4";
  if (c.tile2 != 1 && c.tile2 != 2 && c.tile2 != 4) return "tile2 must be 1, 2 or 4";
  if (c.tile2 > 1 && c.walk == 0) return "tile2 > 1 needs a walk";
  if (c.ns > 1) {
    if (c.nv != 4 || c.walk != 0 || c.order > 1 || c.form == kFormMatrix)
      return "ns > 1 needs nv = 4, form 0 or 2, order 0 or 1 and no walk";
    if (c.ns == 4 && dtype == RMH_F64) return "ns = 4 is FP32 only";
  }
  return nullptr;
}

HopConfig tune_hop(const Geom& g, int32_t dtype, int32_t n_rhs, int32_t purpose) {
  std::lock_guard<std::mutex> lk(g_mu);
  auto it = g_cache.find(key_of(g, dtype, n_rhs, purpose));
  if (it != g_cache.end()) return it->second.cfg;
  it = g_cache.find(key_of(g, dtype, n_rhs, RMH_PURPOSE_ANY));
  if (it != g_cache.end()) return it->second.cfg;
  if (const HopConfig* c = nearest(g, dtype, n_rhs, purpose)) return fit_batch(*c, n_rhs);
  if (const HopConfig* c = nearest(g, dtype, n_rhs, RMH_PURPOSE_ANY)) return fit_batch(*c, n_rhs);
  return defaults_kept(g, dtype, n_rhs, purpose);  // under the lock
}

HopConfig tune_default(const Geom& g, int32_t dtype, int32_t n_rhs, int32_t purpose) {
  std::lock_guard<std::mutex> lk(g_mu);
  return defaults_kept(g, dtype, n_rhs, purpose);
}

void tune_clear() {
  std::lock_guard<std::mutex> lk(g_mu);
  g_cache.clear();
}

void tune_store(const Geom& g, int32_t dtype, int32_t n_rhs, int32_t purpose, const HopConfig& cfg, double ms) {
  std::lock_guard<std::mutex> lk(g_mu);
  g_cache[key_of(g, dtype, n_rhs, purpose)] = Entry{cfg, ms};
}

// ------------------------------------------------------------------------------------------
// JSON file: {"format": "rmh-tune-1", "arch": "...", "hip_runtime": N, "entries": [{...}, ...]}

static const char* kFields[] = {"L0", "L1", "L2", "L3", "dtype", "n_rhs", "purpose", "form", "block",
                                "xcd_remap", "nv", "order", "walk", "ns", "tile2"};
constexpr int kNumFields = 15;

int tune_save_file(const char* path, const std::string& arch, int32_t runtime, int32_t* n_saved) {
  std::lock_guard<std::mutex> lk(g_mu);
  FILE* f = fopen(path, "w");
  if (!f) return -1;
  fprintf(f, "{\"format\": \"rmh-tune-1\", \"arch\": \"%s\", \"hip_runtime\": %d, \"entries\": [", arch.c_str(),
          runtime);
  int n = 0;
  for (auto& kv : g_cache) {
    const Key& k = kv.first;
    const HopConfig& c = kv.second.cfg;
    const int32_t v[kNumFields] = {std::get<0>(k), std::get<1>(k), std::get<2>(k), std::get<3>(k), std::get<4>(k),
                                   std::get<5>(k), std::get<6>(k), c.form, c.block, c.xcd_remap, c.nv, c.order,
                                   c.walk, c.ns, c.tile2};
    fprintf(f, "%s\n  {", n ? "," : "");
    for (int i = 0; i < kNumFields; ++i) fprintf(f, "%s\"%s\": %d", i ? ", " : "", kFields[i], v[i]);
    fprintf(f, ", \"ms\": %.6g}", kv.second.ms);
    ++n;
  }
  fprintf(f, "\n]}\n");
  const bool ok = ferror(f) == 0;
  if (fclose(f) != 0 || !ok) return -1;
  if (n_saved) *n_saved = n;
  return 0;
}

// value of "name": <int> inside [b, e); false when absent or not an integer
static bool json_int(const char* b, const char* e, const char* name, long* out) {
  const std::string key = std::string("\"") + name + "\"";
  const char* p = b;
  while (p < e) {
    const char* q = strstr(p, key.c_str());
    if (!q || q >= e) return false;
    q += key.size();
    while (q < e && (*q == ' ' || *q == '\t' || *q == '\n' || *q == '\r')) ++q;
    if (q < e && *q == ':') {
      ++q;
      char* end = nullptr;
      const long v = strtol(q, &end, 10);
      if (end == q || end > e) return false;
      *out = v;
      return true;
    }
    p = q;
  }
  return false;
}

static bool json_str(const char* b, const char* e, const char* name, std::string* out) {
  const std::string key = std::string("\"") + name + "\"";
  const char* q = strstr(b, key.c_str());
  if (!q || q >= e) return false;
  q += key.size();
  while (q < e && *q != '"') {
    if (*q != ' ' && *q != ':' && *q != '\t' && *q != '\n' && *q != '\r') return false;
    ++q;
  }
  if (q >= e) return false;
  const char* s = ++q;
  while (q < e && *q != '"') ++q;
  if (q >= e) return false;
  out->assign(s, q);
  return true;
}

// 0: loaded (or skipped for another device/runtime), -1: unreadable, -2: malformed or invalid
int tune_load_file(const char* path, const std::string& arch, int32_t runtime, int32_t* n_loaded) {
  if (n_loaded) *n_loaded = 0;
  FILE* f = fopen(path, "rb");
  if (!f) return -1;
  std::string text;
  char buf[4096];
  size_t r;
  while ((r = fread(buf, 1, sizeof buf, f)) > 0) text.append(buf, r);
  const bool bad = ferror(f) != 0;
  fclose(f);
  if (bad) return -1;
  const char* b = text.c_str();
  const char* e = b + text.size();
  std::string fmt, farch;
  long frt = 0;
  if (!json_str(b, e, "format", &fmt) || fmt != "rmh-tune-1" || !json_str(b, e, "arch", &farch) ||
      !json_int(b, e, "hip_runtime", &frt))
    return -2;
  if (farch != arch || frt != runtime) return 0;
  const char* ent = strstr(b, "\"entries\"");
  if (!ent) return -2;
  const char* p = strchr(ent, '[');
  if (!p) return -2;
  // parse every entry first, store only if all are valid
  std::map<Key, Entry> add;
  for (;;) {
    const char* ob = strchr(p, '{');
    const char* close = strchr(p, ']');
    if (!ob || (close && close < ob)) break;
    const char* cb = strchr(ob, '}');
    if (!cb) return -2;
    long v[kNumFields];
    for (int i = 0; i < kNumFields; ++i)
      if (!json_int(ob, cb, kFields[i], &v[i])) return -2;
    HopConfig c;
    c.form = (int32_t)v[7];
    c.block = (int32_t)v[8];
    c.xcd_remap = (int32_t)v[9];
    c.nv = (int32_t)v[10];
    c.order = (int32_t)v[11];
    c.walk = (int32_t)v[12];
    c.ns = (int32_t)v[13];
    c.tile2 = (int32_t)v[14];
    const int32_t dtype = (int32_t)v[4];
    if ((dtype != RMH_F64 && dtype != RMH_F32) || v[5] < 1 || v[5] > (1L << 24) || v[6] < RMH_PURPOSE_ANY ||
        v[6] > RMH_PURPOSE_HEATBATH)
      return -2;
    int64_t V = 1;   // (saturated: an entry for more sites than any call takes is kept like the others)
    for (int i = 0; i < 4; ++i) {
      if (v[i] < 2 || v[i] > (1 << 20)) return -2;
      V = std::min<int64_t>(V * v[i], INT32_MAX);
    }
    const Geom g{(int32_t)v[0], (int32_t)v[1], (int32_t)v[2], (int32_t)v[3], (int32_t)V};
    if (hop_config_error(g, c, dtype)) return -2;
    add[Key((int32_t)v[0], (int32_t)v[1], (int32_t)v[2], (int32_t)v[3], dtype, (int32_t)v[5], (int32_t)v[6])] =
        Entry{c, 0.0};
    p = cb + 1;
  }
  std::lock_guard<std::mutex> lk(g_mu);
  for (auto& kv : add) g_cache[kv.first] = kv.second;
  if (n_loaded) *n_loaded = (int32_t)add.size();
  return 0;
}

}  // namespace rmh
