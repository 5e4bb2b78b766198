// Host runtime: tile choice, the tuned-shape cache (optionally persisted as
// JSON), launch geometry, per-device workspaces.
#include "cell_model.hpp"
#include "runtime.hpp"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <unordered_map>

#include "plan.hpp"

namespace dfr {

namespace {

std::mutex g_tune_mutex;
std::map<std::string, int> g_tune;
bool g_tune_loaded = false;
uint64_t g_tune_generation = 0;  // bumped whenever g_tune changes

const char *cache_path() {
  const char *p = std::getenv("DFR_TUNE_CACHE");
  return (p && *p) ? p : nullptr;
}

// The cache file is a flat JSON object {"key": tile, ...}.
void load_cache_locked() {
  if (g_tune_loaded) return;
  g_tune_loaded = true;
  const char *path = cache_path();
  if (!path) return;
  FILE *f = std::fopen(path, "rb");
  if (!f) return;
  std::string text;
  char buf[4096];
  size_t n;
  while ((n = std::fread(buf, 1, sizeof(buf), f)) > 0) text.append(buf, n);
  std::fclose(f);
  size_t i = 0;
  while (true) {
    size_t q0 = text.find('"', i);
    if (q0 == std::string::npos) break;
    size_t q1 = text.find('"', q0 + 1);
    if (q1 == std::string::npos) break;
    size_t colon = text.find(':', q1);
    if (colon == std::string::npos) break;
    int v = std::atoi(text.c_str() + colon + 1);
    if (v >= 1 && v <= kTileCount) g_tune[text.substr(q0 + 1, q1 - q0 - 1)] = v;
    i = colon + 1;
  }
}

void save_cache_locked() {
  const char *path = cache_path();
  if (!path) return;
  std::string tmp = std::string(path) + ".tmp";
  FILE *f = std::fopen(tmp.c_str(), "wb");
  if (!f) return;
  std::fprintf(f, "{");
  bool first = true;
  for (auto &kv : g_tune) {
    std::fprintf(f, "%s\n  \"%s\": %d", first ? "" : ",", kv.first.c_str(), kv.second);
    first = false;
  }
  std::fprintf(f, "\n}\n");
  std::fclose(f);
  std::rename(tmp.c_str(), path);
}

}  // namespace

int lds_need(const FramePlan &P, int32_t out_h, int32_t out_w, int interp, int tile,
             LdsNeeds &known) {
  int &need = known.floats[tile];
  if (need == 0) {
    TileShape s;
    tile_shape(tile, s);
    need = estimate_lds_floats(P, out_h, out_w, s, interp);
  }
  return need;
}

std::string tune_key(const FramePlan &P, int32_t out_h, int32_t out_w, int interp, bool batch) {
  double mag = max_magnification(P, out_h, out_w);
  int mb = mag > 0 ? (int)std::lround(std::log2(mag) * 2.0) : -99;
  // rotation class from the map's Jacobian at the frame centre
  double xs0, ys0, xs1, ys1;
  int rb = 0;
  double cx = 0.5 * (out_w - 1), cy = 0.5 * (out_h - 1);
  if (position_f64(P, cx, cy, xs0, ys0) && position_f64(P, cx + 8.0, cy, xs1, ys1)) {
    double ang = std::atan2(std::fabs(ys1 - ys0), std::fabs(xs1 - xs0)) * 180.0 / M_PI;
    rb = (int)(ang / 10.0);
  }
  int sord = std::min(P.s_order, 6);
  char key[128];
  std::snprintf(key, sizeof(key), "%s:i%d:s%d:t%d:m%d:r%d", batch ? "batch" : "single", interp,
                sord, P.t_order > 0 ? 1 : 0, mb, rb);
  return key;
}

std::mutex &tune_mutex_for_batch() { return g_tune_mutex; }

int tuned_tile(const std::string &key) {
  load_cache_locked();
  auto it = g_tune.find(key);
  return it == g_tune.end() ? 0 : it->second;
}

void tune_store(const std::string &key, int tile) {
  std::lock_guard<std::mutex> lk(g_tune_mutex);
  load_cache_locked();
  g_tune[key] = tile;
  ++g_tune_generation;
  save_cache_locked();
}

int choose_tile(const FramePlan &P, int32_t out_h, int32_t out_w, int interp, int requested,
                bool batch, LdsNeeds &known, int lds_factor, int pref, int64_t images) {
  if (requested >= 1 && requested <= kTileCount) return requested;
  {
    std::lock_guard<std::mutex> lk(g_tune_mutex);
    load_cache_locked();
    if (!g_tune.empty()) {
      auto it = g_tune.find(tune_key(P, out_h, out_w, interp, batch));
      if (it != g_tune.end()) return it->second;
    }
  }
  // heuristic: the measured default for the kernel and interpolation unless
  // the map turns its source box much larger per output pixel than the
  // 64x32 tile's (a rotated map and a flat tile); then 64x32 when its box
  // fits the LDS budget (or the square 64x64 tile when its box is smaller
  // per output pixel still: 218 against 225 us on the 8192^2 frame rotated
  // by 45 degrees), else the largest tile whose box does
  {
    if (pref < 1 || pref > kTileCount) pref = forward_default_tile(interp, images, out_h, out_w);
    TileShape a, b;
    tile_shape(pref, a);
    tile_shape(kDefaultTile, b);
    const double na = lds_need(P, out_h, out_w, interp, pref, known);
    const double nb = lds_need(P, out_h, out_w, interp, kDefaultTile, known);
    // the flat 128x16 tile gives way to 64x64 where that one's box is at most
    // 0.7 of its own per output pixel: a map turned by 3 degrees or more, or by
    // 90, where the flat tile's box is tall and its rows short (6000x4000
    // bilinear, tile kernel, 128x16 and 64x64: 67 and 71 us at 2 degrees, 70 and
    // 69 at 3, 85 and 75 at 10, 64 and 54 at 92)
    if (pref == kFlatTile) {
      TileShape c;
      tile_shape(kSquareTile, c);
      const double nc = lds_need(P, out_h, out_w, interp, kSquareTile, known);
      if (lds_factor * nc <= kLdsMaxFloats &&
          nc / (c.width * c.height) <= 0.7 * na / (a.width * a.height))
        return kSquareTile;
    }
    if (lds_factor * na <= kLdsMaxFloats &&
        na / (a.width * a.height) <= 1.5 * nb / (b.width * b.height))
      return pref;
  }
  const double nb = lds_need(P, out_h, out_w, interp, kDefaultTile, known);
  if (lds_factor * nb <= kLdsMaxFloats) {
    TileShape b, c;
    tile_shape(kDefaultTile, b);
    tile_shape(kSquareTile, c);
    const double nc = lds_need(P, out_h, out_w, interp, kSquareTile, known);
    if (lds_factor * nc <= kLdsMaxFloats &&
        nc / (c.width * c.height) <= 0.95 * nb / (b.width * b.height))
      return kSquareTile;
    return kDefaultTile;
  }
  const int order[] = {4, 8, 1, 7, 10};
  for (int t : order)
    if (lds_factor * lds_need(P, out_h, out_w, interp, t, known) <= kLdsMaxFloats) return t;
  return 7;
}

void make_geom(const FramePlan &P, int32_t out_h, int32_t out_w, int interp, int tile,
               const dfr_options &o, TileGeom &G, TileShape &ts, LdsNeeds &known, int lds_factor) {
  tile_shape(tile, ts);
  std::memset(&G, 0, sizeof(G));
  G.out_h = out_h;
  G.out_w = out_w;
  G.txt_log2 = ts.txt_log2;
  G.tiles_x = (out_w + ts.width - 1) / ts.width;
  int64_t ty = (out_h + ts.height - 1) / ts.height;
  G.n_tiles = (int32_t)(G.tiles_x * ty);
  int64_t need = (int64_t)lds_factor * lds_need(P, out_h, out_w, interp, tile, known);
  G.lds_cap = need <= kLdsMaxFloats ? (int32_t)need : 0;
  G.cubic_a = (float)o.cubic_a;
  G.nan_outside = o.nan_outside ? 1 : 0;
  G.debug = o.debug_positions;
  G.allow_skip = o.debug_positions ? 0 : 1;
}

// ------------------------------------------------ cached single set-up --

namespace {

struct SetupEntry {
  FramePlan P;
  TileGeom G;
  TileShape ts;
};

std::mutex g_setup_mutex;
std::unordered_map<std::string, SetupEntry> g_setup;
constexpr size_t kSetupCacheMax = 256;

void put_bytes(std::string &k, const void *p, size_t n) {
  k.append(static_cast<const char *>(p), n);
}

void put_wcs(std::string &k, const dfr_wcs &w) {
  put_bytes(k, w.crpix, sizeof(w.crpix));
  put_bytes(k, w.crval, sizeof(w.crval));
  put_bytes(k, w.cd, sizeof(w.cd));
  const int32_t orders[4] = {w.a_order, w.b_order, w.ap_order, w.bp_order};
  put_bytes(k, orders, sizeof(orders));
  const double *coef[4] = {w.a, w.b, w.ap, w.bp};
  for (int i = 0; i < 4; ++i)
    if (orders[i] > 0 && coef[i])
      put_bytes(k, coef[i], sizeof(double) * (orders[i] + 1) * (orders[i] + 1));
}

}  // namespace

void single_setup(const float *src, int32_t src_h, int32_t src_w, int64_t src_pitch,
                  const dfr_wcs &sw, const dfr_wcs &tw, int32_t out_h, int32_t out_w,
                  float *out, float *footprint, int interp, const dfr_options &o, FramePlan &P,
                  TileGeom &G, TileShape &ts, int lds_factor, int pref, bool two_rows) {
  std::string key;
  key.reserve(1024);
  uint64_t gen;
  {
    std::lock_guard<std::mutex> lk(g_tune_mutex);
    load_cache_locked();
    gen = g_tune_generation;
  }
  const int64_t ints[9] = {src_h, src_w, out_h, out_w, interp, o.tile, lds_factor, pref,
                           two_rows ? 1 : 0};
  put_bytes(key, ints, sizeof(ints));
  put_bytes(key, &gen, sizeof(gen));
  put_wcs(key, sw);
  put_wcs(key, tw);
  bool hit = false;
  {
    std::lock_guard<std::mutex> lk(g_setup_mutex);
    auto it = g_setup.find(key);
    if (it != g_setup.end()) {
      P = it->second.P;
      G = it->second.G;
      ts = it->second.ts;
      hit = true;
    }
  }
  if (!hit) {
    build_plan(nullptr, src_h, src_w, src_w, sw, tw, out_h, out_w, nullptr, nullptr, P);
    std::memset(&G, 0, sizeof(G));
    std::memset(&ts, 0, sizeof(ts));
    if (out_h > 0 && out_w > 0) {
      LdsNeeds known;
      int tile = choose_tile(P, out_h, out_w, interp, o.tile, false, known, lds_factor, pref);
      TileShape t4;
      if (two_rows && tile_shape(tile, t4) && t4.np == 4) tile -= 1;
      dfr_options base;
      dfr_options_init(&base);
      make_geom(P, out_h, out_w, interp, tile, base, G, ts, known, lds_factor);
    }
    std::lock_guard<std::mutex> lk(g_setup_mutex);
    if (g_setup.size() >= kSetupCacheMax) g_setup.clear();
    g_setup[key] = SetupEntry{P, G, ts};
  }
  // the per-call parts
  P.src = (src_h > 0 && src_w > 0) ? src : nullptr;
  P.pitch = src_pitch;
  P.out = out;
  P.fp = footprint;
  G.cubic_a = (float)o.cubic_a;
  G.nan_outside = o.nan_outside ? 1 : 0;
  G.debug = o.debug_positions;
  G.allow_skip = o.debug_positions ? 0 : 1;
}

// ------------------------------------------------------------ workspaces --

namespace {
std::mutex g_ws_mutex;
std::map<std::pair<int, void *>, Workspace> g_ws;
}  // namespace

std::mutex &workspace_mutex() { return g_ws_mutex; }

bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &status) == hipSuccess)
    return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

Workspace *workspace(hipStream_t stream) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  Workspace &w = g_ws[std::make_pair(dev, reinterpret_cast<void *>(stream))];
  w.device = dev;
  w.stream = stream;
  return &w;
}

dfr_status workspace_buffer(Workspace *w, size_t bytes, void **buf) {
  *buf = nullptr;
  if (!w) return DFR_E_DEVICE;
  if (w->cap >= bytes && w->buf) {
    *buf = w->buf;
    return DFR_OK;
  }
  if (w->buf) {
    // work already queued on this stream may still use the old buffer; a
    // failed wait is a device error (the old buffer is kept)
    if (hipStreamSynchronize(w->stream) != hipSuccess) return DFR_E_DEVICE;
    (void)hipFree(w->buf);
    w->buf = nullptr;
    w->cap = 0;
  }
  size_t cap = std::max<size_t>(bytes + bytes / 4, 1 << 20);
  if (hipMalloc(&w->buf, cap) != hipSuccess) {
    // (taken here: it would stay the thread's last error, and a caller that does
    // without the memory would find it after its next launch)
    (void)hipGetLastError();
    w->buf = nullptr;
    return DFR_E_NOMEM;
  }
  w->cap = cap;
  *buf = w->buf;
  return DFR_OK;
}

dfr_status workspace_control(Workspace *w, int **ctl) {
  *ctl = nullptr;
  if (!w) return DFR_E_DEVICE;
  if (!w->ctl) {
    if (hipMalloc(&w->ctl, 256) != hipSuccess) {
      w->ctl = nullptr;
      return DFR_E_NOMEM;
    }
    w->ctl_dirty = true;
  }
  if (w->ctl_dirty) {
    if (launch_zero_i32(w->ctl, 64, w->stream) != hipSuccess) return DFR_E_DEVICE;
    w->ctl_dirty = false;
  }
  *ctl = w->ctl;
  return DFR_OK;
}

namespace {

void destroy_graphs(Workspace &w) {
  for (auto &g : w.graphs) {
    (void)hipGraphExecDestroy(g.exec);
    (void)hipGraphDestroy(g.graph);
  }
  w.graphs.clear();
}

}  // namespace

namespace {

dfr_status staging_wait(StagingRing &r, int k) {
  if (r.pending[k] && hipEventSynchronize(r.copied[k]) != hipSuccess) return DFR_E_DEVICE;
  r.pending[k] = false;
  return DFR_OK;
}

// The ring's next slot, of at least `bytes` bytes and not read by a copy any more.
dfr_status staging_slot(StagingRing &r, size_t bytes, void **buf, int *slot) {
  for (hipEvent_t &e : r.copied)
    if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
      e = nullptr;
      return DFR_E_DEVICE;
    }
  const int k = r.next;
  dfr_status s = staging_wait(r, k);
  if (s != DFR_OK) return s;
  if (r.slot < bytes) {
    for (int i = 0; i < kStagings; ++i)
      if ((s = staging_wait(r, i)) != DFR_OK) return s;
    if (r.buf) (void)hipHostFree(r.buf);
    r.buf = nullptr;
    r.slot = 0;
    void *mem = nullptr;
    const size_t size = (bytes + 255) & ~(size_t)255;
    if (hipHostMalloc(&mem, kStagings * size, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      return DFR_E_NOMEM;
    }
    r.buf = static_cast<char *>(mem);
    r.slot = size;
  }
  r.next = (k + 1) % kStagings;
  *buf = r.buf + (size_t)k * r.slot;
  *slot = k;
  return DFR_OK;
}

}  // namespace

void release_workspaces() {
  std::lock_guard<std::mutex> lk(g_ws_mutex);
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return;
  for (auto it = g_ws.begin(); it != g_ws.end();) {
    if (it->first.first != dev) {
      ++it;
      continue;
    }
    Workspace &w = it->second;
    (void)hipStreamSynchronize(w.stream);
    destroy_graphs(w);
    if (w.buf) (void)hipFree(w.buf);
    if (w.ctl) (void)hipFree(w.ctl);
    if (w.staging.buf) (void)hipHostFree(w.staging.buf);
    for (hipEvent_t e : w.staging.copied)
      if (e) (void)hipEventDestroy(e);
    it = g_ws.erase(it);
  }
}

// ----------------------------------------------------------------- batch --

dfr_status run_batch(const std::vector<FramePlan> &plans, const TileGeom &G, int interp, int np,
                     int max_sord, bool models, hipStream_t stream, bool graph,
                     const BatchRun &run) {
  const CoaddOut *coadd = run.coadd;
  const int total = (int)plans.size() * G.n_tiles;
  // A stack call cannot be recorded: the copy of its frame table would read, on
  // replay, whatever a later call has put into the staging buffer, and a graph
  // launched into a capturing stream runs at once, on the table of an earlier
  // call.  Refused before anything is queued.
  if (capturing(stream)) return DFR_E_DEVICE;
  if (coadd || run.crop_items >= 0 || run.reach_host || total > kBatchItems) graph = false;
  std::lock_guard<std::mutex> lk(g_ws_mutex);
  Workspace *w = workspace(stream);
  if (!w) return DFR_E_DEVICE;
  const int n = (int)plans.size();
  const size_t table = (size_t)n * sizeof(FramePlan);
  // reach boxes (4 ints per frame) | frame table | reach boxes of the models'
  // blocks | per-frame model tables (when used)
  // a target with SIP has no reach boxes: every tile visits every frame
  const int tord = plans[0].t_order;
  // (nor has a cropped call: its windows are the boxes of an earlier prepass, so
  // its items end early by their cells' marks alone)
  const bool boxes = models && tord == 0 && run.crop_items < 0;
  int msord = 0;  // the models' source order
  for (const FramePlan &P : plans) msord = std::max(msord, P.s_order);
  const int ncx = (G.out_w + kCell - 1) / kCell, ncy = (G.out_h + kCell - 1) / kCell;
  const int64_t ncells = (int64_t)ncx * ncy;
  const size_t tofs = ((size_t)n * 16 + 255) & ~(size_t)255;
  int ncx_i = ncx, ncy_i = ncy, bcols = (ncx + 7) / 8, bpf = bcols * ((ncy + 7) / 8);
  const size_t pofs = (tofs + table + 255) & ~(size_t)255;
  const size_t mofs = (pofs + (boxes ? (size_t)n * bpf * sizeof(int4) : 0) + 255) & ~(size_t)255;
  size_t mbytes = models && !run.reach_host ? (size_t)n * ncells * sizeof(CellModel) : 0;
  void *wsbuf = nullptr;
  dfr_status ws = workspace_buffer(w, mofs + mbytes, &wsbuf);
  if (ws == DFR_E_NOMEM && tord > 0 && mbytes) {
    // a target with SIP does without the tables: the anchored chain
    models = false;
    mbytes = 0;
    ws = workspace_buffer(w, mofs, &wsbuf);
  }
  if (ws != DFR_OK) return ws;
  char *dev = static_cast<char *>(wsbuf);
  int32_t *reach = reinterpret_cast<int32_t *>(dev);
  FramePlan *plans_dev = reinterpret_cast<FramePlan *>(dev + tofs);
  CellModel *models_dev = mbytes ? reinterpret_cast<CellModel *>(dev + mofs) : nullptr;
  // the next staging slot, once its last copy has ended: with one slot a
  // call would wait here for the whole previous batch on the stream (its copy
  // is ordered behind that batch's kernels), so the GPU ran dry between calls
  void *stage = nullptr;
  int slot = 0;
  if ((ws = staging_slot(w->staging, tofs + table, &stage, &slot)) != DFR_OK) return ws;
  std::memset(stage, 0, tofs);
  FramePlan *host_plans = reinterpret_cast<FramePlan *>(static_cast<char *>(stage) + tofs);
  std::memcpy(host_plans, plans.data(), table);
  for (int i = 0; i < n; ++i) {
    host_plans[i].models = mbytes ? models_dev + i * ncells : nullptr;
    host_plans[i].reach = boxes ? reach + 4 * i : nullptr;
  }
  // (the reach boxes' place goes with it, zero; the prepass writes them)
  if (hipMemcpyAsync(dev, stage, tofs + table, hipMemcpyHostToDevice, stream) != hipSuccess)
    return DFR_E_DEVICE;
  if (hipEventRecord(w->staging.copied[slot], stream) != hipSuccess) {
    (void)hipStreamSynchronize(stream);  // the copy may still read the buffer
    return DFR_E_DEVICE;
  }
  w->staging.pending[slot] = true;
  const int lds_bytes = G.lds_cap * (int)sizeof(float);
  int4 *parts = boxes ? reinterpret_cast<int4 *>(dev + pofs) : nullptr;
  const void *mkernel = cell_models_batch_ptr(msord, tord);
  const void *parts_in = parts;
  void *rargs[] = {&plans_dev, &parts_in, &bpf};
  if (!graph) {
    // (a launch has fewer than 2^32 threads: whole frames, as many as that allows)
    const int step = std::max(1, ((1 << 26) - 1) / bpf);
    for (int f = 0; f < n && (run.reach_host ? boxes : models); f += step) {
      const FramePlan *plans_f = plans_dev + f;
      CellModel *models_f = models_dev ? models_dev + f * ncells : nullptr;
      int4 *parts_f = parts ? parts + (int64_t)f * bpf : nullptr;
      void *args[] = {&plans_f, &ncx_i, &ncy_i, &bcols, &bpf, &models_f, &parts_f};
      if (launch_kernel(mkernel, dim3((unsigned)std::min(step, n - f) * (unsigned)bpf), dim3(64),
                        args, 0, stream) != hipSuccess)
        return DFR_E_DEVICE;
    }
    if (boxes &&
        launch_kernel(reach_kernel_ptr(), dim3(n), dim3(256), rargs, 0, stream) != hipSuccess)
      return DFR_E_DEVICE;
    if (run.reach_host) {
      // the reach boxes the prepass recorded, back to the host (none:
      // every frame may reach everywhere, reported as -1)
      if (boxes && hipMemcpyAsync(run.reach_host, reach, (size_t)16 * n, hipMemcpyDeviceToHost,
                                   stream) != hipSuccess)
        return DFR_E_DEVICE;
      if (hipStreamSynchronize(stream) != hipSuccess) return DFR_E_DEVICE;
      if (!boxes)
        for (int i = 0; i < 4 * n; ++i) run.reach_host[i] = -1;
      return DFR_OK;
    }
    const hipError_t e =
        coadd ? launch_coadd_f32(plans_dev, n, max_sord, G, interp, np, *coadd, stream)
        : run.crop_items >= 0
            ? launch_batch_cropped(plans_dev, n, (int)run.crop_items, max_sord, G, interp, np,
                                   stream)
            : launch_batch_f32(plans_dev, n, max_sord, G, interp, np, stream);
    if (e != hipSuccess) return DFR_E_DEVICE;
  } else {
    BatchGraph *found = nullptr;
    for (auto &g : w->graphs)
      if (g.n == n && g.interp == interp && g.np == np && g.sord == max_sord &&
          g.models == (models ? mkernel : nullptr) && g.plans_dev == plans_dev &&
          std::memcmp(&g.geom, &G, sizeof(G)) == 0)
        found = &g;
    if (!found) {
      BatchGraph bg;
      std::memset(&bg, 0, sizeof(bg));
      bg.geom = G;
      bg.n = n;
      bg.interp = interp;
      bg.np = np;
      bg.sord = max_sord;
      bg.models = models ? mkernel : nullptr;
      bg.plans_dev = plans_dev;
      if (hipGraphCreate(&bg.graph, 0) != hipSuccess) return DFR_E_DEVICE;
      hipGraphNode_t mod = nullptr, box = nullptr, kern = nullptr;
      bool ok = true;
      void *margs[] = {&plans_dev, &ncx_i, &ncy_i, &bcols, &bpf, &models_dev, &parts};
      if (models) {
        hipKernelNodeParams mp;
        std::memset(&mp, 0, sizeof(mp));
        mp.func = const_cast<void *>(mkernel);
        // (kBatchItems bounds the cells of a graph's frames far below a launch's limit)
        mp.gridDim = dim3((unsigned)n * (unsigned)bpf);
        mp.blockDim = dim3(64);
        mp.kernelParams = margs;
        ok = hipGraphAddKernelNode(&mod, bg.graph, nullptr, 0, &mp) == hipSuccess;
      }
      if (boxes) {
        hipKernelNodeParams bp;
        std::memset(&bp, 0, sizeof(bp));
        bp.func = const_cast<void *>(reach_kernel_ptr());
        bp.gridDim = dim3(n);
        bp.blockDim = dim3(256);
        bp.kernelParams = rargs;
        ok = ok && hipGraphAddKernelNode(&box, bg.graph, &mod, 1, &bp) == hipSuccess;
        mod = box;
      }
      TileGeom geom = G;
      int first = 0, nitems = total;
      void *kargs[] = {&plans_dev, &first, &nitems, &geom};
      hipKernelNodeParams kp;
      std::memset(&kp, 0, sizeof(kp));
      kp.func = const_cast<void *>(batch_kernel_ptr(interp, np, max_sord));
      kp.gridDim = dim3(total);
      kp.blockDim = dim3(kThreads);
      kp.sharedMemBytes = lds_bytes;
      kp.kernelParams = kargs;
      ok = ok && hipGraphAddKernelNode(&kern, bg.graph, models ? &mod : nullptr, models ? 1 : 0,
                                       &kp) == hipSuccess;
      ok = ok && hipGraphInstantiate(&bg.exec, bg.graph, nullptr, nullptr, 0) == hipSuccess;
      if (!ok) {
        (void)hipGraphDestroy(bg.graph);
        return DFR_E_DEVICE;
      }
      w->graphs.push_back(bg);
      found = &w->graphs.back();
    }
    if (hipGraphLaunch(found->exec, stream) != hipSuccess) return DFR_E_DEVICE;
  }
  return DFR_OK;
}

}  // namespace dfr
