// Paths of the runtime that the serving histories of runtime_on_mock_hip.cpp do not take, on the stand-in HIP runtime, against
// plain loops over the pool's bytes.  One section per run, named by the argument.
#include <random>

#include "kvswap.hip"

namespace {

[[noreturn]] void die(const char* what, long a = 0, long b = 0) {
  std::printf("FAILED: %s (%ld, %ld)\n", what, a, b);
  std::exit(1);
}
#define OK(expr)                                        \
  do {                                                  \
    const int rc_ = (expr);                             \
    if (rc_ != KV_OK) die(#expr, rc_, __LINE__);        \
  } while (0)

// A layer-major pool of N blocks of 2 x 2 chunks, its arena and a handle on streams of its own.
struct Pool {
  static constexpr int64_t planes = 4;
  int64_t N, chunk;
  char *pool = nullptr, *arena = nullptr;
  hipStream_t st[2];
  kv_pool_config kc{};
  kv_pool* h = nullptr;
  explicit Pool(int64_t n, int64_t slots = 16, uint32_t flags = KV_STAGING_DEVICE, int64_t chunk_bytes = 64) : N(n), chunk(chunk_bytes) {
    (void)hipMalloc((void**)&pool, (size_t)(N * planes * chunk));
    if (flags & KV_STAGING_DEVICE)
      (void)hipMalloc((void**)&arena, (size_t)(slots * planes * chunk));
    else
      (void)hipHostMalloc((void**)&arena, (size_t)(slots * planes * chunk), 0);
    for (auto& s : st) (void)hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    kc.struct_size = sizeof(kc);
    kc.num_layers = 2; kc.num_kv_heads = 1; kc.head_dim = (int32_t)(chunk / 2); kc.block_size = 1; kc.dtype = KV_F16; kc.num_blocks = N;
    kc.block_stride = chunk; kc.kv_stride = N * chunk; kc.layer_stride = 2 * N * chunk;
    kc.pool_dev = pool; kc.staging_host = arena; kc.staging_bytes = slots * planes * chunk;
    kc.evict_stream = st[0]; kc.load_stream = st[1]; kc.flags = flags;
    OK(kv_pool_create(&kc, &h));
    std::mt19937_64 rng(7);
    for (int64_t i = 0; i < N * planes * chunk; i++) pool[i] = (char)rng();
  }
  ~Pool() {
    OK(kv_pool_destroy(h));
    for (auto& s : st) (void)hipStreamDestroy(s);
    (void)hipFree(pool);
    (void)hipFree(arena);
  }
  std::vector<char> bytes() const { return std::vector<char>(pool, pool + N * planes * chunk); }
};

struct Moves {
  std::vector<int32_t> src, dst;
  Moves(std::mt19937_64& rng, int64_t N, size_t n) {
    std::vector<int32_t> perm((size_t)N);
    for (size_t i = 0; i < perm.size(); i++) perm[i] = (int32_t)i;
    std::shuffle(perm.begin(), perm.end(), rng);
    src.assign(perm.begin(), perm.begin() + (long)n);
    dst.assign(perm.begin() + (long)n, perm.begin() + 2 * (long)n);
  }
  void apply(const Pool& p, std::vector<char>* to) const {
    for (size_t i = 0; i < src.size(); i++)
      for (int64_t k = 0; k < Pool::planes; k++)
        std::memcpy(to->data() + (k * p.N + dst[i]) * p.chunk, to->data() + (k * p.N + src[i]) * p.chunk, (size_t)p.chunk);
  }
  int run(const Pool& p, hipEvent_t wait = nullptr) const {
    return kv_move_blocks_noalloc(p.h, (int64_t)src.size(), src.data(), dst.data(), wait);
  }
};

// An allocation-free move inside a graph moves the blocks it was captured with, whatever the handle does between the
// capture and a replay.  The evict stream joins the capture through the caller's event, or through the load stream's fence.
void capture() {
  std::mt19937_64 rng(1);
  for (int through = 0; through < 2; through++)
    for (size_t n : {7, 61, 100, 449, 1000}) {
      Pool p(2 * (int64_t)n + 3);
      hipStream_t origin;
      hipEvent_t fork, join;
      (void)hipStreamCreateWithFlags(&origin, hipStreamNonBlocking);
      (void)hipEventCreate(&fork);
      (void)hipEventCreate(&join);
      const Moves first(rng, p.N, n);
      std::vector<char> want = p.bytes();
      mockhip::begin_capture(origin);
      (void)hipEventRecord(fork, origin);
      if (through == 1) (void)hipStreamWaitEvent(p.st[1], fork, 0);
      OK(first.run(p, through == 0 ? fork : nullptr));
      hipStreamCaptureStatus on;
      (void)hipStreamIsCapturing(p.st[0], &on);
      if (on != hipStreamCaptureStatusActive) die("the evict stream is not in the capture", through, (long)n);
      (void)hipEventRecord(join, p.st[0]);
      (void)hipStreamWaitEvent(origin, join, 0);
      const mockhip::Graph g = mockhip::end_capture();
      if (p.bytes() != want) die("a captured move has run", through, (long)n);
      for (int turn = 0; turn < 6; turn++) {  // more calls than the handle has upload buffers
        const Moves other(rng, p.N, n);
        OK(other.run(p));
        other.apply(p, &want);
        OK(kv_sync(p.h));
        if (turn % 2) {
          mockhip::replay(origin, g);
          first.apply(p, &want);
          (void)hipStreamSynchronize(origin);
        }
        if (p.bytes() != want) die("a replay moves other blocks: through, n", through, (long)n);
      }
      if (mockhip::capture_errors()) die("calls that a capture does not allow", mockhip::capture_errors(), (long)n);
      (void)hipStreamDestroy(origin);
      (void)hipEventDestroy(fork);
      (void)hipEventDestroy(join);
    }
}

// A capture that streams of a handle are drawn into through `fork`, in the relaxed mode where asked.
struct Captured {
  hipStream_t origin;
  hipEvent_t fork, join;
  hipStreamCaptureMode mode;
  explicit Captured(bool relaxed) : mode(relaxed ? hipStreamCaptureModeRelaxed : hipStreamCaptureModeGlobal) {
    (void)hipStreamCreateWithFlags(&origin, hipStreamNonBlocking);
    (void)hipEventCreate(&fork);
    (void)hipEventCreate(&join);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    mockhip::begin_capture(origin);
    (void)hipEventRecord(fork, origin);
  }
  mockhip::Graph end(std::initializer_list<hipStream_t> joined) {
    for (hipStream_t s : joined) {
      (void)hipEventRecord(join, s);
      (void)hipStreamWaitEvent(origin, join, 0);
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    return mockhip::end_capture();
  }
  void replay(const mockhip::Graph& g) {
    mockhip::replay(origin, g);
    (void)hipStreamSynchronize(origin);
  }
  ~Captured() {
    (void)hipStreamDestroy(origin);
    (void)hipEventDestroy(fork);
    (void)hipEventDestroy(join);
  }
};

// Calls that keep a record go into a graph as well, and the handle goes on behind them: what is captured runs with each replay and not
// before, and eager calls on both streams, polls, waits and telemetry work as ever.  `front`: in front of it nothing, an allocation-free move
// that stores a number, one with an event, a swap-out; the program itself has waited for that, and the handle has not looked.
// (A swap-in that is captured asks for the swap-out in front of it, which only the relaxed mode allows.)
void captured_calls() {
  const std::vector<int32_t> a{1, 2, 3}, b{4, 5, 6}, c{7, 8, 9}, d{10, 11, 12}, e{13, 14, 15};
  const int32_t off[2] = {0, 3}, tok = 3;
  const uint64_t id1 = 1, id2 = 2, id4 = 4, id7 = 7, id8 = 8;
  const std::vector<int32_t> f{20, 21, 22}, h{23, 24, 25};
  for (uint32_t flags : {(uint32_t)KV_STAGING_DEVICE, (uint32_t)KV_PATH_ZEROCOPY})
    for (int front = 0; front < 4; front++)
      for (int kind = 0; kind < 4; kind++) {  // a move a to d, a swap-out of a, a swap-in to d of what has been swapped out of c, both
        Pool p(40, 16, flags);
        std::mt19937_64 rng(4);
        std::vector<char> want = p.bytes();
        Moves m(rng, p.N, 1);
        auto moved = [&](const std::vector<int32_t>& src, const std::vector<int32_t>& dst) {
          m.src = src, m.dst = dst;
          m.apply(p, &want);
        };
        if (kind >= 2) {
          OK(kv_swap_out(p.h, 1, &id7, off, c.data(), &tok, nullptr));
          OK(kv_swap_out(p.h, 1, &id4, off, b.data(), &tok, nullptr));
          OK(kv_sync(p.h));
        }
        if (front == 3) {
          OK(kv_swap_out(p.h, 1, &id8, off, f.data(), &tok, nullptr));
          (void)hipStreamSynchronize(p.st[0]);
        } else if (front) {
          p.h->by_number = front == 1;
          OK(kv_move_blocks_noalloc(p.h, 3, f.data(), h.data(), nullptr));
          p.h->by_number = true;
          moved(f, h);
          if (!p.h->na_done == (front == 1)) die("number of an allocation-free move", front, kind);
          (void)hipStreamSynchronize(p.st[0]);
        }
        Captured cap(kind >= 2);
        if (front) (void)hipStreamWaitEvent(p.st[0], cap.fork, 0);  // (it is in the capture before the call)
        if (kind == 0)
          OK(kv_move_blocks(p.h, 3, a.data(), d.data(), cap.fork));
        else if (kind == 1)
          OK(kv_swap_out(p.h, 1, &id1, off, a.data(), &tok, cap.fork));
        else if (kind == 2)
          OK(kv_swap_in(p.h, 1, &id7, off, d.data(), KV_KEEP_STAGING, cap.fork));
        else
          OK(kv_evict_and_load(p.h, 1, &id1, off, a.data(), &tok, 1, &id7, off, d.data(), KV_KEEP_STAGING, cap.fork));
        const mockhip::Graph g = kind == 0 || kind == 1 ? cap.end({p.st[0]}) : kind == 2 && !front ? cap.end({p.st[1]}) : cap.end({p.st[0], p.st[1]});
        if (mockhip::capture_errors()) die("calls that a capture does not allow, kind", mockhip::capture_errors(), kind);
        if (p.bytes() != want) die("a captured call has run, kind", kind, flags);
        for (int turn = 0; turn < 3; turn++) {
          for (int32_t blk : a)
            for (int64_t k = 0; k < Pool::planes; k++) {
              std::memset(p.pool + (k * p.N + blk) * p.chunk, turn, (size_t)p.chunk);
              std::memset(want.data() + (k * p.N + blk) * p.chunk, turn, (size_t)p.chunk);
            }
          cap.replay(g);
          if (kind == 0) moved(a, d);
          if (kind >= 2) moved(c, d);
          if (p.bytes() != want) die("bytes of a replay, kind", kind, turn);
          if (kind == 1 || kind == 3) {
            OK(kv_swap_in(p.h, 1, &id1, off, e.data(), KV_KEEP_STAGING, nullptr));
            moved(a, e);
          }
          OK(kv_move_blocks(p.h, 3, d.data(), b.data(), nullptr));
          moved(d, b);
          OK(kv_swap_out(p.h, 1, &id2, off, b.data(), &tok, nullptr));
          OK(kv_req_wait(p.h, id2));
          if (kv_req_poll(p.h, id2) != 1) die("a request that was waited for, kind", kind, turn);
          OK(kv_swap_in(p.h, 1, &id2, off, d.data(), 0, nullptr));
          moved(b, d);
          kv_stats st{};
          st.struct_size = sizeof(st);
          OK(kv_last_stats(p.h, &st));
          if (st.op != 3 || !(st.ms_total > 0)) die("statistics behind a captured call, kind", kind, turn);
          OK(kv_sync(p.h));
          if (p.bytes() != want) die("bytes behind a captured call, kind", kind, turn);
        }
      }
}

// kv_stats.scatter_order says how a scatter went, also where a pool whose planes collide decides it (61 MiB: such a scatter goes
// plane by plane from 60 MiB on).
void scatter_order() {
  const int n = 976, N = 1000;
  Pool p(N, n, KV_STAGING_DEVICE, 16384);
  const uint64_t id = 3;
  const int32_t off[2] = {0, n}, tok = n;
  std::vector<int32_t> ids(n);
  for (int i = 0; i < n; i++) ids[(size_t)i] = i * 17 % N;
  const std::vector<char> want = p.bytes();
  for (bool collide : {false, true})
    for (int knob = 0; knob < 3; knob++) {
      p.h->planes_collide = collide;
      OK(kv_pool_tune(p.h, KV_TUNE_SCATTER_ORDER, knob));
      kv_stats st{};
      st.struct_size = sizeof(st);
      OK(kv_swap_out(p.h, 1, &id, off, ids.data(), &tok, nullptr));
      OK(kv_last_stats(p.h, &st));
      if (st.scatter_order != -1) die("order of a gather", st.scatter_order, knob);
      for (int i = 0; i < n; i++) std::memset(p.pool + ids[(size_t)i] * p.chunk, 0, (size_t)p.chunk);
      OK(kv_swap_in(p.h, 1, &id, off, ids.data(), 0, nullptr));
      OK(kv_last_stats(p.h, &st));
      if (st.scatter_order != (knob == 2 || (collide && knob == 0) ? 1 : -1)) die("order of a scatter, knob", st.scatter_order, knob);
      if (p.bytes() != want) die("bytes of a swap, knob", collide, knob);
    }
}

// kv_stats.ms_kernel of an exchange is its kernels alone, without what the load has waited for, also where a launch does not
// time itself (a workgroup cap: kv_move_kernel).
void exchange_times() {
  for (int cap : {0, 4}) {
    const int n = 8;
    Pool p(40, 2 * n);
    OK(kv_pool_tune(p.h, KV_TUNE_MAX_WGS_DEVICE, cap));
    const uint64_t out = 1, in = 2;
    const int32_t off[2] = {0, n}, tok = n;
    int32_t a[n], b[n];
    for (int i = 0; i < n; i++) a[i] = i, b[i] = 20 + i;
    OK(kv_swap_out(p.h, 1, &in, off, b, &tok, nullptr));
    OK(kv_sync(p.h));
    mockhip::set_policy(mockhip::kLazy, nullptr);  // nothing runs before the host waits: the load waits for the eviction
    OK(kv_evict_and_load(p.h, 1, &out, off, a, &tok, 1, &in, off, a, 0, nullptr));
    kv_stats st{};
    st.struct_size = sizeof(st);
    OK(kv_last_stats(p.h, &st));
    if (st.op != 3 || st.launches != 1 || !(st.ms_kernel > 0)) die("statistics of an exchange's load", st.op, st.launches);
    if (cap ? st.ms_kernel >= st.ms_total : st.ms_kernel != st.ms_total) die("ms_kernel of an exchange's load, cap", cap, (long)(st.ms_kernel * 1e6));
    mockhip::set_policy(mockhip::kRandom, nullptr);
  }
}

// Allocation-free moves in a row while the evict stream is held back: from the upload buffers as long as one is free, then (none
// is free before the stream runs) inside the arguments of the move or of fill launches.
void uploads() {
  std::mt19937_64 rng(2);
  for (int64_t N : {2003, 66000})  // four buffers, and two
    for (size_t n : {60, 61, 448, 449, 897, 1000}) {
      Pool p(N);
      std::vector<char> want = p.bytes();
      mockhip::set_policy(mockhip::kLazy, nullptr);
      for (int turn = 0; turn < 2; turn++) {
        for (int k = 0; k < 7; k++) {
          const Moves m(rng, N, n - (size_t)(k % 3));  // lists that leave the end of an earlier, longer one behind theirs
          OK(m.run(p));
          m.apply(p, &want);
        }
        OK(kv_sync(p.h));
        if (p.bytes() != want) die("bytes of moves in a row: n, turn", (long)n, turn);
      }
      mockhip::set_policy(mockhip::kRandom, nullptr);
    }
}

// One swap out and in, and one exchange, on a handle; returns the waits for a number that were made.
long swap_and_exchange(Pool& p) {
  const int n = 4;
  const uint64_t id = 3, in = 8;
  const int32_t off[2] = {0, n}, tok = n, a[n] = {1, 2, 3, 4}, b[n] = {4, 5, 6, 7};
  mockhip::set_policy(mockhip::kLazy, nullptr);
  const long before = mockhip::value_waits();
  std::vector<char> want = p.bytes();
  auto move = [&](const int32_t* from, const int32_t* to) {
    const std::vector<char> was = want;
    for (int i = 0; i < n; i++)
      for (int64_t k = 0; k < Pool::planes; k++)
        std::memcpy(want.data() + (k * p.N + to[i]) * p.chunk, was.data() + (k * p.N + from[i]) * p.chunk, (size_t)p.chunk);
  };
  kv_stats st{};
  st.struct_size = sizeof(st);
  OK(kv_swap_out(p.h, 1, &id, off, a, &tok, nullptr));
  OK(kv_swap_in(p.h, 1, &id, off, b, 0, nullptr));
  move(a, b);
  OK(kv_last_stats(p.h, &st));
  if (!(st.ms_total > 0)) die("no time of a load");
  OK(kv_swap_out(p.h, 1, &in, off, b, &tok, nullptr));
  OK(kv_evict_and_load(p.h, 1, &id, off, a, &tok, 1, &in, off, a, 0, nullptr));
  move(b, a);
  OK(kv_last_stats(p.h, &st));
  if (!(st.ms_total > 0) || !(st.ms_kernel > 0)) die("no time of an exchange");
  OK(kv_req_release(p.h, id));
  OK(kv_sync(p.h));
  if (p.bytes() != want) die("bytes of a swap and an exchange");
  mockhip::set_policy(mockhip::kRandom, nullptr);
  return mockhip::value_waits() - before;
}

// Handles behind the first 128, which have no counters for launches with both ends in HBM, and behind the first 1024, whose job
// counters of the link are an allocation of their own.
void counters_used_up() {
  for (int others : {0, kLeaveSlots, kTicketSlots})
    for (uint32_t flags : {(uint32_t)KV_STAGING_DEVICE, (uint32_t)KV_PATH_ZEROCOPY}) {
      for (int s = 0; s < others; s++) g_ticket_taken[0][s >> 6] |= 1ull << (s & 63);  // as if that many handles were there
      {
        Pool p(9, 16, flags);
        const bool device = flags & KV_STAGING_DEVICE;
        if (p.h->ticket_slot != (others < kTicketSlots ? others : -1)) die("slot of a handle", p.h->ticket_slot, others);
        for (int turn = 0; turn < 3; turn++) {
          const long waits = swap_and_exchange(p);
          if (!waits != (device && others)) die("waits for a number: others, waits", others, waits);
        }
      }
      std::memset(g_ticket_taken[0], 0, sizeof(g_ticket_taken[0]));
    }
}

// More calls in flight than there are records of the clock: the others have start events.
void records_used_up() {
  Pool p(9);
  const uint64_t id = 3;
  const int32_t off[2] = {0, 2}, tok = 2, a[2] = {1, 2}, b[2] = {5, 6};
  const std::vector<char> before = p.bytes();
  mockhip::set_policy(mockhip::kLazy, nullptr);
  const int pairs = kStamps / 2 + 40;
  for (int i = 0; i < pairs; i++) {
    OK(kv_swap_out(p.h, 1, &id, off, i % 2 ? b : a, &tok, nullptr));
    OK(kv_swap_in(p.h, 1, &id, off, i % 2 ? a : b, 0, nullptr));
  }
  if (!p.h->stamp_free.empty() || p.h->calls.back().stamp || !p.h->calls.back().start) die("records left", (long)p.h->stamp_free.size());
  kv_stats st{};
  st.struct_size = sizeof(st);
  OK(kv_last_stats(p.h, &st));
  if (!(st.ms_total > 0)) die("no time of a call without a record");
  OK(kv_sync(p.h));
  std::vector<char> want = before;
  for (int i = 0; i < 2; i++)
    for (int64_t k = 0; k < Pool::planes; k++)
      std::memcpy(want.data() + (k * p.N + b[i]) * p.chunk, before.data() + (k * p.N + a[i]) * p.chunk, (size_t)p.chunk);
  if (p.bytes() != want) die("bytes of calls in flight");
  mockhip::set_policy(mockhip::kRandom, nullptr);
  swap_and_exchange(p);
  kv_io_stats io{};
  io.struct_size = sizeof(io);
  OK(kv_io_stats_get(p.h, &io));
  if (io.total_calls[0] + io.total_calls[1] < 2 * pairs || !(io.ewma_small_us[0] > 0 && io.ewma_small_us[1] > 0)) die("telemetry", io.total_calls[0], io.total_calls[1]);
  if (!p.h->calls.back().stamp || p.h->stamp_free.size() + p.h->calls.size() < (size_t)kStamps) die("records not given back", (long)p.h->stamp_free.size());
}

// A load drawn into a capture by what it waits for, a captured move of the blocks that it writes: it goes into the graph behind that, with
// nothing of the handle's that a replay would store to.
void drawn_into_a_capture() {
  const std::vector<int32_t> a{1, 2, 3}, b{4, 5, 6}, c{7, 8, 9};
  const int32_t off[2] = {0, 3}, tok = 3;
  const uint64_t id = 3;
  for (uint32_t flags : {(uint32_t)KV_STAGING_DEVICE, (uint32_t)KV_PATH_ZEROCOPY}) {
    Pool p(40, 16, flags);
    std::vector<char> want = p.bytes();
    std::mt19937_64 rng(8);
    Moves m(rng, p.N, 1);
    auto moved = [&](const std::vector<int32_t>& src, const std::vector<int32_t>& dst) {
      m.src = src, m.dst = dst;
      m.apply(p, &want);
    };
    OK(kv_swap_out(p.h, 1, &id, off, c.data(), &tok, nullptr));
    OK(kv_sync(p.h));
    const size_t records = p.h->stamp_free.size() + 1;  // (the newest call keeps its own)
    Captured cap(true);
    OK(kv_move_blocks(p.h, 3, a.data(), b.data(), cap.fork));
    OK(kv_swap_in(p.h, 1, &id, off, a.data(), KV_KEEP_STAGING, nullptr));
    hipStreamCaptureStatus on;
    (void)hipStreamIsCapturing(p.st[1], &on);
    if (on != hipStreamCaptureStatusActive) die("the load stream is not in the capture", flags);
    if (p.h->calls.back().stamp || p.h->calls.back().done || !p.h->calls.back().start) die("a captured load has a clock record or a number", flags);
    const mockhip::Graph g = cap.end({p.st[0], p.st[1]});
    for (int turn = 0; turn < 3; turn++) {
      OK(kv_move_blocks(p.h, 3, b.data(), c.data(), nullptr));
      moved(b, c);
      OK(kv_sync(p.h));
      const uint64_t *record = p.h->calls.back().stamp, was[2] = {record[0], record[1]};
      std::vector<char> slots(p.arena, p.arena + 3 * Pool::planes * p.chunk);
      cap.replay(g);
      moved(a, b);
      for (int i = 0; i < 3; i++)
        for (int64_t k = 0; k < Pool::planes; k++)
          std::memcpy(want.data() + (k * p.N + a[(size_t)i]) * p.chunk, slots.data() + (i * Pool::planes + k) * p.chunk, (size_t)p.chunk);
      if (p.bytes() != want) die("bytes of a replay, turn", turn, flags);
      if (record[0] != was[0] || record[1] != was[1]) die("a replay has stored to a record, turn", turn, flags);
    }
    if (p.h->stamp_free.size() + 1 != records) die("records", (long)p.h->stamp_free.size(), (long)records);
  }
}

// The clock at the end of a call may arrive behind the call's number: its record is not handed to another call before, and what is reported
// is what has arrived.
void late_clock() {
  Pool p(40);
  const int32_t a[2] = {1, 2}, b[2] = {5, 6}, c[2] = {9, 10};
  mockhip::set_policy(mockhip::kLazy, nullptr);
  OK(kv_move_blocks(p.h, 2, a, b, nullptr));
  (void)hipStreamSynchronize(p.st[0]);
  uint64_t* record = p.h->calls.back().stamp;
  const uint64_t end = __atomic_exchange_n(record + 1, 0, __ATOMIC_ACQ_REL);  // as if it were still on its way
  if (!end || p.h->calls.back().end) die("a move that times itself");
  std::atomic<bool> arrived{false};
  std::thread device([&] {
    const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(200);
    while (std::chrono::steady_clock::now() < until) {}
    arrived = true;
    __atomic_store_n(record + 1, end, __ATOMIC_RELEASE);
  });
  OK(kv_move_blocks(p.h, 2, b, c, nullptr));
  OK(kv_move_blocks(p.h, 2, c, a, nullptr));  // the first one's call goes
  if (p.h->calls.back().stamp == record && !arrived) die("a record that the device still stores to");
  device.join();
  if (!p.h->call_by_seq.count(3) || p.h->call_by_seq.count(1)) die("the calls of the handle");
  OK(kv_sync(p.h));
  kv_stats st{};
  st.struct_size = sizeof(st);
  OK(kv_last_stats(p.h, &st));
  if (!(st.ms_total > 0 && st.ms_total < 1000)) die("time of a move");
  mockhip::set_policy(mockhip::kRandom, nullptr);
}

// An allocation-free move that is still under way when its stream is drawn into a capture: calls of the load stream come behind it all the
// same, by its number or by the event recorded behind it, during the capture as well as after one that another such move has gone into.
void capture_behind_a_move() {
  const std::vector<int32_t> a{1, 2, 3}, b{4, 5, 6}, c{7, 8, 9}, d{10, 11, 12}, e{13, 14, 15};
  const int32_t off[2] = {0, 3}, tok = 3;
  const uint64_t id = 3;
  for (uint32_t flags : {(uint32_t)KV_STAGING_DEVICE, (uint32_t)KV_PATH_ZEROCOPY})
    for (int how = 0; how < 4; how++) {
      const bool number = how % 2 == 0, behind = how >= 2;
      Pool p(40, 16, flags);
      std::mt19937_64 rng(8);
      std::vector<char> want = p.bytes();
      Moves m(rng, p.N, 1);
      OK(kv_swap_out(p.h, 1, &id, off, c.data(), &tok, nullptr));
      OK(kv_sync(p.h));
      mockhip::set_policy(mockhip::kLazy, nullptr);
      p.h->by_number = number;
      OK(kv_move_blocks_noalloc(p.h, 3, a.data(), b.data(), nullptr));
      m.src = a, m.dst = b;
      m.apply(p, &want);
      const long values = mockhip::value_waits();
      {
        Captured cap(true);
        if (behind) OK(kv_move_blocks_noalloc(p.h, 3, d.data(), e.data(), cap.fork));
        (void)hipStreamWaitEvent(p.st[0], cap.fork, 0);
        if (!behind) OK(kv_swap_in(p.h, 1, &id, off, a.data(), 0, nullptr));  // into what the move reads
        (void)cap.end({p.st[0]});
        if (behind) OK(kv_swap_in(p.h, 1, &id, off, a.data(), 0, nullptr));
      }
      m.src = c, m.dst = a;
      m.apply(p, &want);
      if ((mockhip::value_waits() != values) != number) die("waits for a number", flags, how);
      mockhip::set_policy(mockhip::kStarve0, p.st[0]);  // the load goes first where nothing holds it back
      OK(kv_sync(p.h));
      if (p.bytes() != want) die("a load has not waited for a move", flags, how);
      if (mockhip::capture_errors()) die("calls that a capture does not allow", mockhip::capture_errors(), how);
      mockhip::set_policy(mockhip::kRandom, nullptr);
    }
}

// A wait for one call that finishes by number ends with that call, whatever its stream has been given since: here the rest of the stream is
// held back until the wait has returned.  The same for the statistics, and for a full ring of descriptors, which waits for the list that
// is in the way; and while the stream is being captured.
void waits_for_numbers() {
  std::mt19937_64 rng(5);
  const int n = 61;  // beyond what travels inside the arguments
  for (uint32_t flags : {(uint32_t)KV_STAGING_DEVICE, (uint32_t)KV_PATH_ZEROCOPY})
    for (int what = 0; what < 5; what++) {
      const bool host = flags & KV_PATH_ZEROCOPY;
      const int m = what == 3 && host ? kInlineDescMax + 1 : n;  // (over the link such a list has to be longer)
      Pool p(6 * m, 2 * m, flags);
      std::vector<char> want = p.bytes();
      std::vector<int32_t> blk[6];
      for (int i = 0; i < 6; i++)
        for (int k = 0; k < m; k++) blk[i].push_back(i * m + k);
      auto moved = [&](int from, int to) {
        Moves mv(rng, p.N, 1);
        mv.src = blk[from], mv.dst = blk[to];
        mv.apply(p, &want);
      };
      const int32_t off[2] = {0, m}, tok = m;
      const uint64_t id = 3;
      uint64_t gate = 0;
      auto hold = [&](int s) { (void)hipStreamWaitValue64(p.st[s], &gate, 1, hipStreamWaitValueGte, ~0ull); };
      mockhip::set_policy(mockhip::kLazy, nullptr);
      OK(kv_move_blocks(p.h, m, blk[0].data(), blk[1].data(), nullptr));
      moved(0, 1);
      const long waited = mockhip::host_waits();
      if (what == 3) {
        if (p.h->ring_head < (size_t)m) die("the list has not been uploaded", flags);
        p.h->ring_cap = 2 * (size_t)m;
        OK(kv_move_blocks(p.h, m, blk[1].data(), blk[2].data(), nullptr));
        moved(1, 2);
        hold(0);
        if (mockhip::host_waits() != waited) die("a wait with room in the ring", flags);
        OK(kv_move_blocks(p.h, m, blk[2].data(), blk[3].data(), nullptr));  // where the first list is, behind what is held back
        moved(2, 3);
      } else {
        OK(kv_swap_out(p.h, 1, &id, off, blk[1].data(), &tok, nullptr));
        if (p.h->calls.back().end || !p.h->calls.back().done) die("a swap-out behind a call has an end event", flags);
        hold(0);
        kv_stats st{};
        st.struct_size = sizeof(st);
        uint64_t ids[1];
        float ms[1];
        if (what == 0) {
          OK(kv_req_wait(p.h, id));
        } else if (what == 1) {
          OK(kv_last_stats(p.h, &st));
          if (st.op != 1 || !(st.ms_total > 0)) die("statistics", flags);
        } else if (what == 2) {
          if (kv_last_timeline(p.h, ids, ms, 1) != 1 || ids[0] != id || !(ms[0] > 0)) die("timeline", flags);
        } else {
          Captured cap(true);
          (void)hipStreamWaitEvent(p.st[0], cap.fork, 0);
          if (kv_req_poll(p.h, id) != 0) die("a request is complete before anything has run", flags);
          OK(kv_req_wait(p.h, id));
          OK(kv_last_stats(p.h, &st));
          (void)cap.end({p.st[0]});
          if (mockhip::capture_errors()) die("calls that a capture does not allow", mockhip::capture_errors(), flags);
        }
        if (kv_req_poll(p.h, id) != 1 || p.bytes() != want) die("a request that was waited for", what, flags);
      }
      if (mockhip::host_waits() == waited) die("no wait", what, flags);
      kv_io_stats io{};
      io.struct_size = sizeof(io);
      OK(kv_io_stats_get(p.h, &io));
      if (io.inflight_calls[0]) die("a finished call is in flight", what, flags);
      gate = 1;
      OK(kv_move_blocks(p.h, m, blk[3].data(), blk[4].data(), nullptr));
      moved(3, 4);
      if (p.h->calls.back().end) die("an end event behind a wait", what, flags);
      OK(kv_sync(p.h));
      if (p.bytes() != want) die("bytes", what, flags);
      mockhip::set_policy(mockhip::kRandom, nullptr);
    }
}

// Calls that store a number record no end event: not behind others, and not for a program that polls or waits for single
// requests.  What a wait, a poll and a hazard with the other stream need is there all the same.
void no_end_events() {
  std::mt19937_64 rng(3);
  for (uint32_t flags : {(uint32_t)KV_STAGING_DEVICE, (uint32_t)KV_PATH_ZEROCOPY}) {
    Pool p(40, 16, flags);
    std::vector<char> want = p.bytes();
    auto moved = [&](const std::vector<int32_t>& src, const std::vector<int32_t>& dst) {
      Moves m(rng, p.N, 1);
      m.src = src, m.dst = dst;
      m.apply(p, &want);
    };
    const std::vector<int32_t> a{1, 2, 3}, b{4, 5, 6}, c{7, 8, 9}, d{10, 11, 12};
    const int32_t off[2] = {0, 3}, tok = 3;
    const uint64_t id = 3, id2 = 4;
    auto last = [&]() -> Call& { return p.h->calls.back(); };
    mockhip::set_policy(mockhip::kLazy, nullptr);
    OK(kv_move_blocks(p.h, 3, a.data(), b.data(), nullptr));
    moved(a, b);
    if (last().end || !last().done) die("a short move has an end event", flags);
    OK(kv_swap_out(p.h, 1, &id, off, b.data(), &tok, nullptr));  // behind the move: the handle is busy
    if (last().end) die("a swap-out behind a call has an end event", flags);
    OK(kv_swap_in(p.h, 1, &id, off, a.data(), KV_KEEP_STAGING, nullptr));  // a's blocks: behind the move, which reads them
    moved(b, a);
    if (last().end) die("a swap-in has an end event", flags);
    if (kv_req_poll(p.h, id) != 0) die("a request is complete before anything has run", flags);
    OK(kv_move_blocks_noalloc(p.h, 3, a.data(), c.data(), nullptr));
    moved(a, c);
    if (!p.h->na_done) die("an allocation-free move has no number", flags);
    OK(kv_swap_out(p.h, 1, &id2, off, c.data(), &tok, nullptr));
    OK(kv_swap_in(p.h, 1, &id2, off, d.data(), 0, nullptr));
    moved(c, d);
    kv_stats st{};
    st.struct_size = sizeof(st);
    OK(kv_last_stats(p.h, &st));
    if (!(st.ms_total > 0) || st.op != 3) die("statistics of a call without an event", flags);
    if (p.bytes() != want) die("bytes of calls without events", flags);
    OK(kv_sync(p.h));
    OK(kv_swap_out(p.h, 1, &id2, off, d.data(), &tok, nullptr));
    if (!last().end) die("a swap-out on an idle handle has no end event", flags);
    OK(kv_swap_in(p.h, 1, &id2, off, b.data(), 0, nullptr));
    moved(d, b);
    if (last().end) die("a swap-in behind it has one", flags);
    OK(kv_req_wait(p.h, id2));
    if (kv_req_poll(p.h, id2) != 1 || p.bytes() != want) die("a request that was waited for", flags);
    OK(kv_move_blocks(p.h, 3, b.data(), c.data(), nullptr));
    moved(b, c);
    if (last().end) die("an end event for a program that waits for requests", flags);
    OK(kv_sync(p.h));
    if (p.bytes() != want) die("bytes", flags);
    mockhip::set_policy(mockhip::kRandom, nullptr);
  }
}

// Streams hand over by event, and not by number, where the number's wait might not end: as soon as a profiling tool has been loaded
// (argument of the section: a library that is one), and where threads of the runtime submit the streams' work.
void late_profiler(const char* tool) {
  const int n = 4;
  const int32_t off[2] = {0, n}, tok = n, a[n] = {1, 2, 3, 4}, b[n] = {4, 5, 6, 7};
  {
    setenv("AMD_DIRECT_DISPATCH", "0", 1);
    Pool p(9);
    if (swap_and_exchange(p)) die("a wait for a number where the runtime's threads submit");
    setenv("AMD_DIRECT_DISPATCH", "1", 1);
    Pool q(9);
    if (!swap_and_exchange(q)) die("no wait for a number");
    unsetenv("AMD_DIRECT_DISPATCH");
  }
  Pool p(9), q(9);
  if (swap_and_exchange(p) < 2) die("no wait for a number");
  mockhip::set_policy(mockhip::kLazy, nullptr);
  const uint64_t id2 = 5;  // enqueued with a number, waited for after the tool has come
  OK(kv_swap_out(q.h, 1, &id2, off, a, &tok, nullptr));
  if (!dlopen(tool, RTLD_NOW | RTLD_GLOBAL)) die("the tool cannot be loaded");
  const long before = mockhip::value_waits();
  OK(kv_swap_in(q.h, 1, &id2, off, b, 0, nullptr));
  OK(kv_sync(q.h));
  if (swap_and_exchange(p) || swap_and_exchange(q) || mockhip::value_waits() != before) die("a wait for a number under a tool that came late");
}

// A call without an end event that the other stream has to wait for after a tool has come: by an event recorded then, or, where the
// event would be a graph's, on the host.
void late_events(const char* tool) {
  const int n = 4;
  const int32_t off[2] = {0, n}, tok = n, a[n] = {1, 2, 3, 4}, b[n] = {5, 6, 7, 8}, c[n] = {9, 10, 11, 12};
  const uint64_t id = 5;
  Pool p(16), q(16);
  std::vector<char> want[2];
  uint64_t gate = 0;  // holds p's move back until it is p's turn
  for (Pool* r : {&p, &q}) {
    std::vector<char>& w = want[r == &q];
    w = r->bytes();
    std::mt19937_64 rng(6);
    Moves m(rng, r->N, 1);
    OK(kv_swap_out(r->h, 1, &id, off, a, &tok, nullptr));
    OK(kv_sync(r->h));
    mockhip::set_policy(mockhip::kLazy, nullptr);
    if (r == &p) (void)hipStreamWaitValue64(r->st[0], &gate, 1, hipStreamWaitValueGte, ~0ull);
    OK(kv_move_blocks(r->h, n, b, c, nullptr));
    if (r->h->calls.back().end) die("a short move has an end event");
    m.src.assign(a, a + n), m.dst.assign(c, c + n);  // the swap-in into c comes last
    m.apply(*r, &w);
  }
  if (!dlopen(tool, RTLD_NOW | RTLD_GLOBAL)) die("the tool cannot be loaded");
  for (Pool* r : {&q, &p}) {
    const long values = mockhip::value_waits(), waits = mockhip::host_waits();
    {
      Captured cap(true);
      if (r == &q) (void)hipStreamWaitEvent(r->st[0], cap.fork, 0);
      OK(kv_swap_in(r->h, 1, &id, off, c, 0, nullptr));
      (void)cap.end({cap.origin});
    }
    if (mockhip::value_waits() != values) die("a wait for a number under a tool that came late");
    if ((mockhip::host_waits() != waits) != (r == &q)) die("waits on the host", r == &q);
    gate = r == &p;
    mockhip::set_policy(mockhip::kStarve0, r->st[0]);  // the load goes first where nothing holds it back
    OK(kv_sync(r->h));
    mockhip::set_policy(mockhip::kLazy, nullptr);
    if (r->bytes() != want[r == &q]) die("a load has not waited for a move", r == &q);
  }
  if (mockhip::capture_errors()) die("calls that a capture does not allow", mockhip::capture_errors());
}

}  // namespace

int main(int argc, char** argv) {
  if (argc == 3) {
    !std::strcmp(argv[1], "late_profiler") ? late_profiler(argv[2]) : late_events(argv[2]);
    std::printf("%s ok\n", argv[1]);
    return 0;
  }
  const struct {
    const char* name;
    void (*run)();
  } sections[] = {{"capture", capture}, {"captured_calls", captured_calls}, {"capture_behind_a_move", capture_behind_a_move}, {"scatter_order", scatter_order}, {"exchange_times", exchange_times}, {"uploads", uploads},
                {"counters_used_up", counters_used_up}, {"records_used_up", records_used_up}, {"late_clock", late_clock}, {"drawn_into_a_capture", drawn_into_a_capture},
                {"no_end_events", no_end_events}, {"waits_for_numbers", waits_for_numbers}};
  for (const auto& s : sections)
    if (argc == 2 && !std::strcmp(argv[1], s.name)) {
      mockhip::reset(5);
      s.run();
      std::printf("%s ok\n", s.name);
      return 0;
    }
  die("no such section");
}
