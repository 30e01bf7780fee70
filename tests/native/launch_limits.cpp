// The limits of one launch, checked on the CPU for geometries and list lengths that no test pool could hold.
//
// The real launch code (runtime.hip.inc) is compiled with launches that are recorded instead of queued.  For a sweep of
// geometries it is given lists longer than one launch may carry; every recorded launch must hold what its kernel's
// 32-bit arithmetic assumes: counts that equal their 64-bit value, divisions by multiplication (FastDiv) that
// equal plain division up to the largest number the launch divides, a grid whose thread count fits 32 bits, and the
// launches together exactly the list.  No memory is touched: descriptor pointers are only counted with.
//
// A check of what kv_evict_and_load reports sits beside them, on a handle whose launches are recorded.
//
// usage: launch_limits   (prints "launches ok" and the number of launches looked at)
#include <hip/hip_runtime.h>

#include <algorithm>

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kern, grid, block, lds_bytes, stream, ...) record((grid), (block), __VA_ARGS__)

template <class... Args>
void record(dim3 grid, dim3 block, const Args&... args);

#include "kvswap.hip"

struct Launch {
  uint64_t grid, threads, bytes;
  HbmArgs a;
};
static std::vector<Launch> launches;
template <class Args, class = std::enable_if_t<std::is_base_of_v<HbmArgs, Args>>>
void take(uint64_t grid, uint64_t threads, const Args& a) {
  launches.push_back({grid, threads, sizeof(Args), a});
  // a launch that is not run has finished: the other stream may wait for its number, and its times are asked
  if (a.stamp) a.stamp[0] = 1, a.stamp[1] = 2;
  if (a.done) *a.done = a.done_value;
}
struct MoveLaunch {
  uint64_t grid, threads, bytes;
  MoveArgs a;
};
static std::vector<MoveLaunch> move_launches;
void take(uint64_t grid, uint64_t threads, const MoveArgs& a) { move_launches.push_back({grid, threads, sizeof(a), a}); }
void take(...) {}
template <class... Args>
void record(dim3 grid, dim3 block, const Args&... args) {
  if constexpr (sizeof...(args) == 1) take((uint64_t)grid.x, (uint64_t)block.x, args...);
}

namespace {

long looked_at = 0;

[[noreturn]] void die(const char* what, const kv_pool& p, uint64_t a, uint64_t b) {
  std::printf("FAILED: %s: %llu, expected %llu (L %d H %d D %d B %d chunk %lld S %lld)\n", what, (unsigned long long)a,
              (unsigned long long)b, p.cfg.num_layers, p.cfg.num_kv_heads, p.cfg.head_dim, p.cfg.block_size, (long long)p.chunk,
              (long long)p.S);
  std::exit(1);
}

// f divides as plain division does at the largest numbers up to `top` (where the error of the multiplication is largest: the
// last multiple of d, its neighbour below, and top itself) and at a few others
void divides(const kv_pool& p, const char* what, const FastDiv& f, uint64_t d, uint64_t top) {
  const uint64_t last = top / d * d;
  for (uint64_t n : {top, last, last ? last - 1 : 0, last >= d ? last - d : 0, last > d ? last - d - 1 : 0, top / 2, (uint64_t)0})
    if ((uint64_t)((uint32_t)n / f) != n / d) die(what, p, (uint32_t)n / f, n / d);
}

const Desc* const kBase = (const Desc*)(uintptr_t)4096;

void hbm(kv_pool& p, int mode, uint64_t n, bool pm) {
  launches.clear();
  launch_hbm(&p, mode, kBase, nullptr, (size_t)n, nullptr, pm, nullptr);
  const uint64_t L2 = 2 * (uint64_t)p.cfg.num_layers, vpb = (uint64_t)p.block_bytes / 16;
  uint64_t at = 0;
  for (size_t i = 0; i < launches.size(); i++) {
    const HbmArgs& a = launches[i].a;
    if ((uint64_t)(a.desc - kBase) != at) die("first descriptor of a launch", p, (uint64_t)(a.desc - kBase), at);
    const uint64_t end = i + 1 < launches.size() ? (uint64_t)(launches[i + 1].a.desc - kBase) : n, m = end - at;
    uint64_t data;
    if (pm && mode != 0) {
      data = L2 * a.ppc * m;
      if (a.n_plane != m * a.ppc) die("jobs per plane", p, a.n_plane, m * a.ppc);
      divides(p, "plane of a job", a.per_plane, m * a.ppc, data - 1);
      divides(p, "chunk of a piece", a.by_ppc, a.ppc, m * a.ppc - 1);
    } else if (p.hbm_all) {
      data = (m * vpb + 255) / 256;
      if (a.n_vec != m * vpb) die("vectors of a launch", p, a.n_vec, m * vpb);
      divides(p, "block of a vector", a.by_vpb, vpb, m * vpb - 1);
      divides(p, "chunk of a vector", a.by_vpc, (uint64_t)p.chunk / 16, vpb - 1);
    } else {
      data = m * a.ppb;
      divides(p, "block of a job", a.by_ppb, a.ppb, data - 1);
      if (p.hbm_wave)
        divides(p, "chunk of a piece", a.by_ppc, a.ppc, a.ppb - 1);
      else
        divides(p, "chunk of a vector", a.by_vpc, (uint64_t)p.chunk / 16, vpb - 1);
    }
    if (a.n_data_jobs != data) die("data jobs", p, a.n_data_jobs, data);
    if (a.n_jobs != data + m * a.side_ppb) die("jobs", p, a.n_jobs, data + m * a.side_ppb);
    if (a.side_ppb) {
      divides(p, "block of a side job", a.by_side, a.side_ppb, m * a.side_ppb - 1);
      divides(p, "head of a scale word", a.by_H, a.H, (uint64_t)a.side_ppb * 256 - 1);
    }
    if (launches[i].grid != a.n_jobs && !(pm && mode == 1 && p.max_wgs_device)) die("grid", p, launches[i].grid, a.n_jobs);
    if (launches[i].grid * launches[i].threads >> 32) die("threads of a launch", p, launches[i].grid * launches[i].threads, 0);
    at = end;
    looked_at++;
  }
  if (at != n) die("descriptors launched", p, at, n);
}

void link(kv_pool& p, int mode, uint64_t n, int64_t wgs) {
  launches.clear();
  launch_link(&p, mode, kBase, nullptr, (size_t)n, nullptr, wgs, nullptr);
  const uint64_t vps = (uint64_t)p.S / 16;
  uint64_t at = 0;
  for (size_t i = 0; i < launches.size(); i++) {
    const HbmArgs& a = launches[i].a;
    if ((uint64_t)(a.desc - kBase) != at) die("first descriptor of a link launch", p, (uint64_t)(a.desc - kBase), at);
    const uint64_t end = i + 1 < launches.size() ? (uint64_t)(launches[i + 1].a.desc - kBase) : n, m = end - at;
    uint64_t jobs;
    if (p.link_all) {
      jobs = (m * vps + 255) / 256;
      if (a.n_vec != m * vps) die("vectors of a link launch", p, a.n_vec, m * vps);
      divides(p, "slot of a vector", a.by_vps, vps, m * vps - 1);
    } else {
      jobs = m * ((vps + 255) / 256);
      divides(p, "slot of a link job", a.by_link, a.link_ppb, jobs - 1);
    }
    if (a.n_jobs != jobs) die("link jobs", p, a.n_jobs, jobs);
    if ((a.n_jobs + launches[i].grid) >> 32) die("numbers the counter hands out", p, a.n_jobs + launches[i].grid, 0);
    divides(p, "chunk of a vector", a.by_vpc, (uint64_t)p.chunk / 16, vps - 1);
    if (a.scale_words) divides(p, "head of a scale word", a.by_H, a.H, a.scale_words - 1);
    if (launches[i].grid < 1 || launches[i].grid > a.n_jobs) die("link grid", p, launches[i].grid, a.n_jobs);
    if (launches[i].grid * launches[i].threads >> 32) die("threads of a link launch", p, launches[i].grid * launches[i].threads, 0);
    at = end;
    looked_at++;
  }
  if (at != n) die("descriptors launched on the link", p, at, n);
}

// A handle under a workgroup cap: launches of 256 lanes within the cap, the data jobs (in either order of the scatter) with
// the build that has nothing else in it, the scale jobs behind them.
void capped(kv_pool& p, int64_t cap) {
  p.max_wgs_device = cap;
  p.dev_staging = true;
  if (!p.stream[kEvict]) (void)hipStreamCreateWithFlags(&p.stream[kEvict], hipStreamNonBlocking);
  const Desc list[3] = {{0, 0}, {1, 1}, {2, 2}};
  for (int mode = 0; mode < 3; mode++)
    for (int pm = 0; pm < (mode == 1 && p.chunk >= 4096 ? 2 : 1); pm++) {
      launches.clear();
      move_launches.clear();
      Call c;
      if (enqueue_kernel(&p, c, mode, list, 3, nullptr, 0, /*sole=*/true, pm == 1) != KV_OK) die("capped launch", p, 0, 0);
      if (!launches.empty()) die("launches of one-wavefront workgroups under a cap", p, launches.size(), 0);
      if (move_launches.size() != (p.cfg.scale_dev ? 2u : 1u)) die("launches under a cap", p, move_launches.size(), 1);
      int64_t at = 0;
      for (const MoveLaunch& l : move_launches) {
        if (l.threads != 256 || l.grid > (uint64_t)cap) die("workgroups under a cap", p, l.grid, (uint64_t)cap);
        if (l.a.first_job != at) die("first job of a capped launch", p, (uint64_t)l.a.first_job, (uint64_t)at);
        if (&l == &move_launches[0] && (l.a.scale_words || l.a.n_jobs != l.a.n_data_jobs || (l.a.per_plane > 0) != (pm == 1)))
          die("data jobs of a capped launch", p, (uint64_t)l.a.n_jobs, (uint64_t)l.a.n_data_jobs);
        at = l.a.n_jobs;
        looked_at++;
      }
      if (at != move_launches[0].a.n_data_jobs + (p.cfg.scale_dev ? 3 : 0)) die("jobs under a cap", p, (uint64_t)at, 0);
    }
  p.max_wgs_device = 0;
}

// A list inside the kernel arguments: short ones leave the arguments (with 256 hidden bytes) below 1 KiB, and a list beyond
// what they hold is uploaded (a short move's beyond those 1 KiB), also where a knob selects kv_move_kernel.
void arguments() {
  kv_pool p;
  p.cfg.num_layers = 2;
  p.cfg.num_kv_heads = 1;
  p.cfg.num_blocks = 1000;
  p.chunk = 4096;
  p.cfg.block_stride = 4096;
  p.cfg.kv_stride = p.cfg.layer_stride = INT64_MAX / 4;
  p.S = p.block_bytes = 16384;
  static uint32_t counters[64];
  p.tickets = counters;
  hbm_setup(&p);
  (void)hipStreamCreateWithFlags(&p.stream[kEvict], hipStreamNonBlocking);
  if (grow_ring(&p, 4096) != KV_OK) die("ring", p, 0, 0);
  std::vector<Desc> list(449, Desc{0, 1});
  for (int64_t cap : {0, 4})
    for (int kind = 0; kind < 3; kind++)
      for (int mode = 0; mode < (kind == 0 ? 3 : 2); mode++)
        for (size_t n : {1, 8, 9, 60, 61, 448, 449}) {
          p.max_wgs_device = cap;
          launches.clear();
          move_launches.clear();
          Call c;
          const size_t ring = p.ring_head;
          if (enqueue_kernel(&p, c, mode, list.data(), n, nullptr, kind, /*sole=*/true) != KV_OK) die("launch", p, n, 0);
          const bool uploaded = p.ring_head != ring, knob = cap && kind != 1;
          const uint64_t bytes = knob ? move_launches.at(0).bytes : launches.at(0).bytes;
          const bool inside = knob ? move_launches[0].a.use_inl : bytes > sizeof(HbmArgs);
          if (inside == uploaded || inside != (n <= (knob ? 8u : mode == 2 ? 60u : 448u))) die("a list inside the arguments", p, n, inside);
          if (bytes > (n <= 60 || knob || uploaded ? 1024u - 256u : 4096u)) die("bytes of arguments", p, bytes, n);
          looked_at++;
        }
}

void geometry(int L, int H, int D, int B, int e, bool scales) {
  const int64_t chunk = (int64_t)B * H * D * e;
  if (chunk % 16 || chunk > (1 << 30) || (scales && 2ll * L * H * 4 % 16)) return;  // kv_pool_create refuses these
  kv_pool p;
  p.cfg.num_layers = L;
  p.cfg.num_kv_heads = H;
  p.cfg.head_dim = D;
  p.cfg.block_size = B;
  p.cfg.num_blocks = INT32_MAX;
  p.chunk = chunk;
  p.block_bytes = 2 * (int64_t)L * chunk;
  p.cfg.block_stride = chunk;
  p.cfg.kv_stride = p.cfg.layer_stride = INT64_MAX / 4;
  if (scales) {
    p.cfg.scale_dev = (void*)(uintptr_t)4096;
    p.block_scale_bytes = 2ll * L * H * 4;
  }
  p.S = p.block_bytes + p.block_scale_bytes;
  static uint32_t counters[64];
  p.tickets = counters;
  hbm_setup(&p);
  auto list = [&](size_t most) { return std::min<uint64_t>(INT32_MAX, 2 * (uint64_t)most + 3); };
  if (hbm_kernels(&p))
    for (int mode = 0; mode < 3; mode++) {
      hbm(p, mode, list(p.hbm_most), false);
      hbm(p, mode, 1, false);
      if (mode && p.hbm_wave) hbm(p, mode, list(p.hbm_most), true);
    }
  if ((L == 2 || L == 3) && B <= 16) capped(p, 3);
  if (p.S < ((int64_t)1 << 34))
    for (int mode = 0; mode < 2; mode++)
      for (int64_t wgs : {(int64_t)0, (int64_t)1, (int64_t)1 << 30, INT64_MAX}) {
        link(p, mode, list(p.link_most), wgs);
        link(p, mode, 1, wgs);
      }
}

}  // namespace

// Phases of kv_evict_and_load: small ones are for the host link, where the first and the last run alone.
void phases() {
  kv_pool p;
  const int64_t MiB = 1 << 20;
  for (int64_t larger : {1 * MiB, 32 * MiB, 256 * MiB, 320 * MiB, 4096 * MiB}) {
    p.dev_staging = true;
    if (phase_of(&p, larger) != 256 * MiB) die("phase in HBM", p, (uint64_t)phase_of(&p, larger), (uint64_t)larger);
    p.dev_staging = false;
    const int64_t host = phase_of(&p, larger);
    if (host < 16 * MiB || host > 64 * MiB || (host > 16 * MiB && host > larger / 8)) die("phase over the link", p, (uint64_t)host, (uint64_t)larger);
  }
}

// kv_evict_and_load whose eviction or load moves nothing: the plan and the statistics afterwards are still the load's.
void evict_and_load_with_an_empty_side() {
  kv_pool none;
  void *pool = nullptr, *arena = nullptr;
  kv_pool_config kc{};
  kc.struct_size = sizeof(kc);
  kc.num_layers = 1; kc.num_kv_heads = 1; kc.head_dim = 64; kc.block_size = 8; kc.dtype = KV_F16; kc.num_blocks = 16;
  kc.block_stride = 1024; kc.kv_stride = 16 * 1024; kc.layer_stride = 32 * 1024;
  (void)hipMalloc(&pool, 32 * 1024);
  (void)hipMalloc(&arena, 16 * 2048);
  kc.pool_dev = pool; kc.staging_host = arena; kc.staging_bytes = 16 * 2048; kc.flags = KV_STAGING_DEVICE;
  kv_pool* p = nullptr;
  if (kv_pool_create(&kc, &p) != KV_OK) die("kv_pool_create", none, 0, 0);
  const uint64_t id[4] = {1, 2, 3, 4};
  const int32_t blk[3] = {5, 6, 7}, two[2] = {0, 2}, nothing[2] = {0, 0}, tok[1] = {16}, zero[1] = {0};
  if (kv_swap_out(p, 1, &id[0], two, blk, tok, nullptr) != KV_OK || kv_swap_out(p, 1, &id[1], nothing, blk, zero, nullptr) != KV_OK)
    die("kv_swap_out", none, 0, 0);
  kv_stats st;
  // an eviction of nothing beside a load of two blocks
  if (kv_evict_and_load(p, 1, &id[2], nothing, blk, zero, 1, &id[0], two, blk, 0, nullptr) != KV_OK) die("kv_evict_and_load", none, 0, 0);
  st.struct_size = sizeof(st);
  if (kv_last_plan(p, nullptr, nullptr, 0) != 2) die("plan after an empty eviction", none, (uint64_t)kv_last_plan(p, nullptr, nullptr, 0), 2);
  if (kv_last_stats(p, &st) != KV_OK || st.op != 3 || st.blocks != 2) die("statistics after an empty eviction", none, (uint64_t)st.blocks, 2);
  // an eviction of two blocks beside a load of nothing
  if (kv_evict_and_load(p, 1, &id[3], two, blk, tok, 1, &id[1], nothing, blk, 0, nullptr) != KV_OK) die("kv_evict_and_load", none, 1, 0);
  st.struct_size = sizeof(st);
  if (kv_last_plan(p, nullptr, nullptr, 0) != 0) die("plan after an empty load", none, (uint64_t)kv_last_plan(p, nullptr, nullptr, 0), 0);
  if (kv_last_stats(p, &st) != KV_OK || st.op != 3 || st.blocks != 0) die("statistics after an empty load", none, (uint64_t)st.blocks, 0);
  if (kv_pool_destroy(p) != KV_OK) die("kv_pool_destroy", none, 0, 0);
  (void)hipFree(pool);
  (void)hipFree(arena);
}

int main() {
  arguments();
  evict_and_load_with_an_empty_side();
  phases();
  {  // the division itself, over its whole range
    kv_pool none;
    const uint64_t top = (1ull << 31) - 1;
    for (uint64_t d = 1; d <= 200000; d++) divides(none, "division", fast_div((uint32_t)d), d, top);
    for (uint64_t d = 200000; d < (1ull << 30); d += d / 5000 + 1) divides(none, "division", fast_div((uint32_t)d), d, top);
    for (int b = 1; b <= 30; b++)
      for (uint64_t d : {(1ull << b) - 1, 1ull << b, (1ull << b) + 1}) divides(none, "division", fast_div((uint32_t)d), d, top);
  }
  for (int L : {1, 2, 3, 16, 24, 28, 32, 40, 80, 96})
    for (int H : {1, 2, 3, 4, 5, 8, 9, 10, 32, 128})
      for (int D : {8, 16, 64, 65, 72, 80, 96, 112, 120, 128, 192, 256})
        for (int B : {1, 2, 3, 4, 8, 16, 32, 256})
          for (int e : {1, 2}) {
            geometry(L, H, D, B, e, false);
            if (e == 1) geometry(L, H, D, B, e, true);
          }
  geometry(80, 128, 256, 4096, 1, true);    // blocks of 20 GiB
  geometry(40, 128, 256, 4096, 1, false);   // 10 GiB
  geometry(64, 129, 257, 2048, 1, true);    // 8.1 GiB, ragged
  std::printf("launches ok: %ld\n", looked_at);
  return 0;
}
