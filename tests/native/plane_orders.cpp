// The plane-by-plane order of a launch with both ends in HBM and the block-by-block one against plain loops over the bytes, on the CPU:
// the library's host code and its kernels, on the stand-in HIP runtime, over every way a pool can be laid out that the order accepts (layer-major,
// padded, block-major, planes in descending layers' places), chunks of one KiB to several and ragged ones, with and without scales, lists in any order,
// inside the arguments and uploaded, launches that finish with a number and the clock and launches that do not.  And the rule that
// says which pools' planes collide, at the distances it was measured at.
#include <random>

#include "kvswap.hip"

namespace {

[[noreturn]] void die(const char* what, long a, long b) {
  std::printf("FAILED: %s (%ld, %ld)\n", what, a, b);
  std::exit(1);
}

long compared = 0;

void compare(std::mt19937_64& rng, int L, int H, int D, int B, bool scales, int layout, size_t n) {
  const int64_t chunk = (int64_t)B * H * D, N = 3 * (int64_t)n + 2;  // one byte per element
  kv_pool p;
  p.cfg.num_layers = L;
  p.cfg.num_kv_heads = H;
  p.cfg.num_blocks = N;
  p.chunk = chunk;
  p.block_bytes = 2 * L * chunk;
  if (layout == 0) {  // layer-major
    p.cfg.block_stride = chunk;
    p.cfg.kv_stride = N * chunk;
    p.cfg.layer_stride = 2 * N * chunk;
  } else if (layout == 1) {  // the same, padded
    p.cfg.block_stride = chunk + 48;
    p.cfg.kv_stride = N * p.cfg.block_stride + 160;
    p.cfg.layer_stride = 2 * p.cfg.kv_stride + 16;
  } else if (layout == 2) {  // block-major
    p.cfg.kv_stride = chunk;
    p.cfg.layer_stride = 2 * chunk;
    p.cfg.block_stride = p.block_bytes;
  } else {  // all layers' K, then all layers' V
    p.cfg.block_stride = chunk;
    p.cfg.layer_stride = N * chunk;
    p.cfg.kv_stride = L * N * chunk;
  }
  const int64_t pool_bytes = (L - 1) * p.cfg.layer_stride + p.cfg.kv_stride + (N - 1) * p.cfg.block_stride + chunk;
  std::vector<char> pool((size_t)pool_bytes), scale;
  p.cfg.pool_dev = pool.data();
  int64_t side = 0;
  if (scales) {
    side = 2ll * L * H * 4;
    scale.resize((size_t)(N * side));
    p.cfg.scale_dev = scale.data();
    p.cfg.scale_block_stride = H * 4;
    p.cfg.scale_kv_stride = N * H * 4;
    p.cfg.scale_layer_stride = 2 * N * H * 4;
  }
  p.S = p.block_bytes + side;
  p.dev_staging = true;
  hbm_setup(&p);
  hipStream_t st[2];
  for (int s = 0; s < 2; s++) {
    (void)hipStreamCreateWithFlags(&st[s], hipStreamNonBlocking);
    p.stream[s] = st[s];
  }
  if (grow_ring(&p, 4096) != KV_OK) die("ring", 0, 0);
  static uint32_t words[2][kLeaveWords];
  static uint64_t done[2], stamp[2];

  std::vector<int32_t> perm((size_t)N);
  for (size_t i = 0; i < perm.size(); i++) perm[i] = (int32_t)i;
  std::shuffle(perm.begin(), perm.end(), rng);
  std::vector<Desc> list(n);
  std::vector<int32_t> slot(n);
  for (size_t i = 0; i < n; i++) slot[i] = (int32_t)i;
  std::shuffle(slot.begin(), slot.end(), rng);
  for (int mode = 0; mode < 3; mode++)
    for (int finish = 0; finish < 2; finish++) {
      for (int s = 0; s < 2; s++) {
        p.leave[s] = finish ? words[s] : nullptr;
        p.done_word[s] = finish ? &done[s] : nullptr;
      }
      p.by_number = finish;
      std::vector<char> pool0((size_t)pool_bytes), scale0(scale.size());
      for (char& c : pool0) c = (char)rng();
      for (char& c : scale0) c = (char)rng();
      std::vector<char> slots0((size_t)((int64_t)n * p.S));
      for (size_t i = 0; i < slots0.size(); i++) slots0[i] = (char)(i * 131 >> 3);
      // what the descriptors say, chunk by chunk
      std::vector<char> want_pool = pool0, want_scale = scale0, want_slots = slots0;
      for (size_t i = 0; i < n; i++)
        for (int k = 0; k < 2 * L; k++) {
          const int64_t plane = (k >> 1) * p.cfg.layer_stride + (k & 1) * p.cfg.kv_stride;
          const int64_t splane = (k >> 1) * p.cfg.scale_layer_stride + (k & 1) * p.cfg.scale_kv_stride, words = scales ? H * 4 : 0;
          char* blk = want_pool.data() + plane + perm[i] * p.cfg.block_stride;
          char* blk_scale = want_scale.data() + splane + perm[i] * p.cfg.scale_block_stride;
          char* other = mode == 2 ? want_pool.data() + plane + perm[n + i] * p.cfg.block_stride : want_slots.data() + slot[i] * p.S + k * chunk;
          char* other_scale = mode == 2 ? want_scale.data() + splane + perm[n + i] * p.cfg.scale_block_stride
                                        : want_slots.data() + slot[i] * p.S + p.block_bytes + k * words;
          std::memcpy(mode == 1 ? blk : other, mode == 1 ? other : blk, (size_t)chunk);
          if (words) std::memcpy(mode == 1 ? blk_scale : other_scale, mode == 1 ? other_scale : blk_scale, (size_t)words);
        }
      if ((mode == 0 ? want_slots == slots0 : want_pool == pool0) || (scales && mode && want_scale == scale0)) die("a case that moves nothing", mode, layout);
      for (int pm = 0; pm < 2; pm++) {
        pool = pool0;
        scale = scale0;
        p.cfg.pool_dev = pool.data();
        if (scales) p.cfg.scale_dev = scale.data();
        hbm_setup(&p);
        std::vector<char> slots = slots0;
        for (size_t i = 0; i < n; i++) list[i] = {perm[i], mode == 2 ? perm[n + i] : slot[i]};
        if (pm) {
          std::vector<Desc> tmp;
          sort_desc(&list, &tmp, mode == 2 ? &Desc::b : &Desc::a, N);
        }
        Call c;
        c.stream = mode == 1 ? kLoad : kEvict;
        c.st.op = mode == 0 ? 1 : mode == 1 ? 3 : 4;
        c.seq = ++p.seq;
        stamp[0] = stamp[1] = 0;
        c.stamp = finish ? stamp : nullptr;  // (begun by the launch's first workgroup, or by the upload in front of it)
        if (enqueue_kernel(&p, c, mode, list.data(), n, mode == 2 ? nullptr : slots.data(), 0, /*sole=*/true, pm == 1) != KV_OK) die("launch", n, mode);
        (void)hipStreamSynchronize(st[c.stream]);
        if (finish && mode != 2 && done[c.stream] != p.done_last[c.stream]) die("number of a launch", (long)done[c.stream], (long)p.done_last[c.stream]);
        if (c.stamp && !(stamp[0] && stamp[1] > stamp[0])) die("clock of a launch", (long)stamp[0], (long)stamp[1]);
        for (int s = 0; s < 2; s++)
          for (uint32_t w : words[s])
            if (w) die("a counter that is not zero after its launch", w, s);
        p.ring_inflight.clear();
        if (pool != want_pool || scale != want_scale || slots != want_slots) die("other bytes than the list says: mode, layout", mode, layout * 10 + pm);
        compared++;
      }
    }
  (void)hipHostFree(p.ring_host);
  (void)hipFree(p.ring_dev);
  for (int s = 0; s < 2; s++) (void)hipStreamDestroy(st[s]);
}

// What a handle over such a pool does with its planes.  layout: 0 layer-major, 1 block-major, 2 layer-major with a block's K and V
// side by side.
bool rule(int L, int64_t chunk, int64_t N, int layout = 0, kv_pool* p = nullptr) {
  kv_pool own;
  if (!p) p = &own;
  p->cfg.num_layers = L;
  p->cfg.num_kv_heads = 1;
  p->cfg.num_blocks = N;
  p->chunk = chunk;
  p->S = p->block_bytes = 2 * L * chunk;
  p->cfg.kv_stride = layout ? chunk : N * chunk;
  p->cfg.layer_stride = layout == 1 ? 2 * chunk : 2 * N * chunk;
  p->cfg.block_stride = layout == 0 ? chunk : layout == 1 ? 2 * L * chunk : 2 * chunk;
  p->dev_staging = true;
  hbm_setup(p);
  return p->planes_collide;
}

void rules() {
  for (int64_t N : {508, 516, 1016, 1032, 2032, 2064})
    if (!rule(32, 32768, N) || !rule(80, 32768, N)) die("planes that collide", N, 0);
  for (int64_t N : {448, 500, 504, 507, 509, 512, 524, 576, 960, 1000, 1020, 1024, 1088, 2040, 2048, 4096, 38146, 40000})
    if (rule(32, 32768, N)) die("planes that do not collide", N, 0);
  for (int64_t N : {127, 129, 254, 258, 508, 516})
    if (!rule(32, 131072, N)) die("planes of 128 KiB chunks that collide", N, 0);
  for (int64_t N : {4064, 4128})
    if (!rule(32, 4096, N)) die("planes of 4 KiB chunks that collide", N, 0);
  if (!rule(64, 32768, 127, 2)) die("planes that collide, K and V of a block side by side", 127, 0);
  // block-major: a block is one run, whatever its chunks
  for (int64_t chunk : {1024, 2048, 4096, 32768})
    for (int L : {2, 16, 32, 80})
      for (int64_t N : {508, 700, 1584, 14400})
        if (rule(L, chunk, N, 1)) die("a block-major pool", chunk, L);
  // planes on few channels, but of blocks so small that enough others are in flight beside them
  const int64_t small[][3] = {{4, 1024, 13208}, {16, 1024, 27348}, {2, 4096, 7224}, {16, 3072, 2794}, {64, 3072, 7138}, {8, 65536, 2580}, {24, 32768, 1270}, {80, 8192, 344}};
  for (auto& s : small)
    if (rule((int)s[0], s[1], s[2])) die("small blocks", s[1], s[2]);
  // which transfers of a pool whose planes collide: long ones, and scatters only of long chunks into a quarter of the pool
  const struct {
    int L, layout;
    int64_t chunk, N;
    size_t n;
    bool out, in;
  } sizes[] = {{32, 0, 32768, 508, 29, false, false}, {32, 0, 32768, 508, 30, true, false}, {32, 0, 32768, 508, 126, true, false},
               {32, 0, 32768, 508, 127, true, true}, {32, 0, 32768, 1032, 500, true, true}, {64, 0, 8192, 508, 200, true, false},
               {48, 0, 16384, 127, 60, true, true}, {32, 2, 32768, 1032, 256, true, false}, {32, 2, 32768, 1032, 300, false, false}};
  for (auto& s : sizes) {
    kv_pool p;
    (void)rule(s.L, s.chunk, s.N, s.layout, &p);
    if (plane_by_plane_move(&p, (size_t)s.N / 2) != (s.layout == 0)) die("moves of long chunks", s.chunk, s.N);
    if (collides(&p, true, s.n) != s.out || collides(&p, false, s.n) != s.in) die("which transfers go plane by plane", s.chunk, (long)s.n);
  }
  // moves whose lists are worth ordering
  const struct {
    int L;
    int64_t chunk;
    size_t n;
    bool pm;
  } moves[] = {{1, 144, 27601, false}, {1, 448, 28933, false},  {2, 768, 28606, false},  {24, 64, 38056, false}, {8, 144, 11274, false},  {24, 128, 9819, false},
               {2, 1920, 42627, false}, {16, 384, 996, false},   {4, 1344, 50386, true},  {24, 160, 40116, true}, {48, 80, 4608, true},    {80, 16, 2866, true},
               {32, 256, 5170, true},   {24, 224, 6552, true},   {80, 960, 6983, true},   {8, 2560, 2584, true},  {1, 1024, 300, true},    {32, 32768, 64, true}};
  for (auto& m : moves) {
    kv_pool p;
    (void)rule(m.L, m.chunk, 3 * (int64_t)m.n, 0, &p);
    if (plane_by_plane_move(&p, m.n) != m.pm) die("which moves go plane by plane", m.chunk, m.L);
  }
}

}  // namespace

// Under a profiling tool, which may run one kernel at a time, a handle has no words to wait for numbers in.
void handle_under_a_profiler() {
  void *pool = nullptr, *arena = nullptr;
  (void)hipMalloc(&pool, 32 * 1024);
  (void)hipMalloc(&arena, 16 * 2048);
  kv_pool_config kc{};
  kc.struct_size = sizeof(kc);
  kc.num_layers = 1; kc.num_kv_heads = 1; kc.head_dim = 64; kc.block_size = 8; kc.dtype = KV_F16; kc.num_blocks = 16;
  kc.block_stride = 1024; kc.kv_stride = 16 * 1024; kc.layer_stride = 32 * 1024;
  kc.pool_dev = pool; kc.staging_host = arena; kc.staging_bytes = 16 * 2048; kc.flags = KV_STAGING_DEVICE;
  for (const char* tool : {"", "ROCP_TOOL_LIBRARIES", "HSA_TOOLS_LIB"}) {
    if (*tool) setenv(tool, "tool.so", 1);
    kv_pool* p = nullptr;
    if (kv_pool_create(&kc, &p) != KV_OK) die("kv_pool_create", 0, 0);
    if ((p->done_word[0] || p->done_word[1]) == (*tool != 0)) die("words of a handle under a profiler", *tool, 0);
    const uint64_t id = 1;
    const int32_t off[2] = {0, 2}, blk[2] = {5, 6}, tok = 16;
    if (kv_swap_out(p, 1, &id, off, blk, &tok, nullptr) != KV_OK || kv_swap_in(p, 1, &id, off, blk, 0, nullptr) != KV_OK || kv_sync(p) != KV_OK)
      die("swap of a handle under a profiler", *tool, 0);
    if (kv_pool_destroy(p) != KV_OK) die("kv_pool_destroy", 0, 0);
    if (*tool) unsetenv(tool);
  }
  (void)hipFree(pool);
  (void)hipFree(arena);
}

int main() {
  handle_under_a_profiler();
  rules();
  std::mt19937_64 rng(17);
  for (int layout = 0; layout < 4; layout++)
    for (int scales = 0; scales < 2; scales++)
      for (size_t n : {1, 2, 63, 64, 65, 130, 449}) {
        const int L = n > 200 ? 1 : 1 + (int)(rng() % 3), K = n > 100 ? 1 : 1 + (int)(rng() % 3);
        compare(rng, L, 4, 64, 4 * K, scales, layout, n);
        // 16 to 7200 bytes, no whole KiB: whole lines and ragged ones, below and from 4 KiB on
        const int odd[] = {4, 36, 40, 64, 288, 520, 1152, 1800};
        compare(rng, L + 1, 4, odd[rng() % (n > 100 ? 4 : 8)], 1, scales, layout, n);
      }
  std::printf("orders agree with the lists: %ld\n", compared);
  return 0;
}
