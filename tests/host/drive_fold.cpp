// Host-logic checks of calls that sum their pulses on a grid, on the stand-in
// runtime of mock_hip.cpp (no GPU): the scratch that such a launch is given
// against what its kernels touch, over shapes, pulse counts, shared and
// per-pulse codes and gate lists, with contexts, zooms, learned zooms and the
// static scratch; and contexts whose max_pulses is far above what they are
// called with.  Exit status: the number of failed checks plus the stand-in
// runtime's errors.
#define launch_fused plain_fused
#define launch_zoom plain_zoom
#include "mock_hip.cpp"
#undef launch_fused
#undef launch_zoom

#include "ispl.h"

static int g_fail = 0;
static long g_folded = 0, g_packed = 0;
static std::set<std::pair<int, int>> g_plans;  // (waves, chunks) of folded launches
static int g_grid_len = 0, g_chunks = 0;       // of the last launch (0: direct)
#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      fprintf(stderr, "CHECK failed (line %d): %s  [%s]\n", __LINE__, #cond, \
              ispl_last_error());                                          \
      ++g_fail;                                                            \
    }                                                                      \
  } while (0)

namespace ispl {

static void check_bits(const uint32_t* bits, const int32_t* binary, int code_len, int per_pulse,
                       int P) {
  if (!bits) return;
  ++g_packed;
  const size_t rows = per_pulse ? size_t(P) : 1;
  check_range(bits, rows * (code_len > SUB ? SUB : 64) * 4, "grid bits");
  check_range(binary, rows * 4, "grid flags");
}

hipError_t launch_fused(const FusedArgs& a, hipStream_t st) {
  g_grid_len = a.grid_len;
  g_chunks = a.grid_chunks;
  if (a.grid_len == 0) return plain_fused(a, st);
  ++g_folded;
  g_plans.insert({a.grid_waves, a.grid_chunks});
  FusedArgs c = a;
  run_on(st, [c] {
    check_bits(c.grid_bits, c.grid_binary, c.code_len, c.tx_per_pulse, c.n_pulses);
    if (c.grid_rows < 1 || c.grid_chunks < 1) mock_fail("fold: empty plan");
    if (c.grid_len == c.n_fft) {
      if (c.grid_chunks > 1 || c.grid_defer)
        check_range(c.grid, size_t(c.grid_chunks) * c.n_gates * c.n_fft * 4, "grid partials");
      return;
    }
    const size_t sets = c.grid_chunks + (c.grid_len > 2 * SUB && c.grid_chunks > 1 ? 1 : 0);
    check_range(c.grid, sets * c.grid_rows * c.grid_len * sizeof(*c.grid), "grid sums");
    check_range(c.twiddle64, size_t(c.n_fft) * 16, "double twiddles");
    check_range(c.grid_gain, size_t(c.grid_len) * 8, "grid gains");
  });
  // the direct launch of gates that are not expanded, with few of them and with a full list
  for (int k : {1, a.grid_rows}) {
    if (a.grid_len == a.n_fft) break;
    run_on(st, [c, k] {
      check_range(c.redo_list, size_t(c.grid_rows) * 4, "redo list");
      check_range(c.redo_count, 4, "redo count");
      check_range(c.redo_early, size_t(c.grid_rows) * 4, "early flags");
      for (int i = 0; i < k; ++i) c.redo_list[i] = i;
      *c.redo_count = k;
      check_range(c.grid, size_t(c.redo_rows) * c.n_fft * 4, "redo partials");
    });
    FusedArgs d = a;
    d.grid_len = 0;
    d.gate_list = a.redo_list;
    d.gate_count = a.redo_count;
    d.adapt_partial = reinterpret_cast<float*>(a.grid);
    d.adapt_target = a.redo_target;
    d.adapt_max_chunks = a.redo_max_chunks;
    d.adapt_rows = a.redo_rows;
    (void)plain_fused(d, st);
  }
  return hipSuccess;
}

hipError_t launch_zoom(const ZoomArgs& a, hipStream_t st, bool prep) {
  if (a.grid_len == 0) return plain_zoom(a, st, prep);
  ++g_folded;
  ZoomArgs c = a;
  run_on(st, [c] {
    check_bits(c.grid_bits, c.grid_binary, c.code_len, c.tx_per_pulse, c.n_pulses);
    if (c.grid_rows < 1 || c.grid_chunks < 1) mock_fail("fold: empty plan");
    check_range(c.grid, size_t(c.grid_chunks) * c.grid_rows * c.grid_len * sizeof(*c.grid),
                "zoom grid sums");
    check_range(c.twiddle64, size_t(c.n_fft) * 16, "double twiddles");
    check_range(c.grid_gain, size_t(c.grid_len) * 8, "grid gains");
    check_range(c.redo_list, size_t(c.grid_rows) * 4, "redo list");
    check_range(c.redo_count, 4, "redo count");
    check_range(c.redo_early, size_t(c.grid_rows) * 4, "early flags");
  });
  ZoomArgs d = a;  // the products of gates that are not expanded
  d.grid_len = 0;
  return plain_zoom(d, st, true);
}

}  // namespace ispl

static std::vector<void*> g_bufs;
template <typename T>
static T* dev(size_t bytes) {
  void* p = nullptr;
  (void)hipMalloc(&p, bytes);
  memset(p, 0, bytes);
  g_bufs.push_back(p);
  return static_cast<T*>(p);
}
static void free_all() {
  for (void* p : g_bufs) (void)hipFree(p);
  g_bufs.clear();
}

static ispl_config config(int L, int N, int G, int P, int step = 3) {
  ispl_config c{};
  c.abi_version = ISPL_ABI_VERSION;
  c.code_len = L;
  c.fft_len = N;
  c.n_gates = G;
  c.gate_step = step;
  c.pulse_stride = int64_t(G - 1) * step + L;
  c.sample_type = ISPL_SAMPLES_CI16;
  c.max_pulses = P;
  return c;
}

static void folded_calls(int L, int N, int G, int P) {
  const ispl_config c = config(L, N, G, P);
  const void* x = dev<void>((size_t(P - 1) * c.pulse_stride + c.pulse_stride) * 4);
  const float* tx = dev<float>(size_t(P) * L * 8);
  float* out = dev<float>(size_t(G) * N * 4);
  int32_t* list = dev<int32_t>(size_t(G) * 4);
  int32_t* count = dev<int32_t>(4);
  for (int g = 0; g < G; ++g) list[g] = G - 1 - g;
  *count = (G + 1) / 2;
  ispl_ctx* ctx = nullptr;
  CHECK(ispl_create(&c, &ctx) == ISPL_OK);
  if (!ctx) return;
  for (int p : {P, 1, 2, 3, 4, 5, (P + 1) / 2})
    for (int per = 0; per < 2; ++per) {
      if (p > P) continue;
      CHECK(ispl_integrate_spectra(ctx, x, tx, per, p, out, per, nullptr) == ISPL_OK);
      CHECK(ispl_integrate_spectra_gates(ctx, x, tx, per, p, list, count, out, 0, nullptr) == ISPL_OK);
      CHECK(ispl_integrate_spectra_noalloc(&c, x, tx, per, p, out, per, nullptr) == ISPL_OK);
    }
  if (L <= 1024) {
    ispl_zoom* z = nullptr;
    CHECK(ispl_zoom_create(ctx, 256, ISPL_ZOOM_FP16X3, &z) == ISPL_OK);
    const int32_t* start = dev<int32_t>(size_t(G) * 4);
    float* win = dev<float>(size_t(G) * 256 * 4);
    for (int p : {P, 1, 4, (P + 1) / 2})
      for (int per = 0; per < 2 && z && p <= P; ++per) {
        CHECK(ispl_zoom_spectra(z, x, tx, per, p, start, win, per, nullptr) == ISPL_OK);
        CHECK(ispl_zoom_spectra_gates(z, x, tx, per, p, start, list, count, win, 0, nullptr) == ISPL_OK);
      }
    ispl_zoom_destroy(z);
    ispl_net* net = nullptr;
    CHECK(ispl_net_create(0, 4, &net) == ISPL_OK);
    ispl_lzoom* lz = nullptr;
    CHECK(ispl_lzoom_create(&c, net, 256, ISPL_ZOOM_FP16X3, 0.9f, &lz) == ISPL_OK);
    int32_t* peak = dev<int32_t>(size_t(G) * 4);
    for (int p : {P, 1, 4})
      if (lz && p <= P) CHECK(ispl_lzoom_peaks(lz, x, tx, 1, p, peak, nullptr, nullptr) == ISPL_OK);
    ispl_lzoom_destroy(lz);
    ispl_net_destroy(net);
  }
  ispl_destroy(ctx);
  free_all();
}

// What a call of this many pulses sums on: a grid of `len` points in at least `chunks` pulse chunks,
// or 0 for direct transforms.
static void plan_of(int L, int N, int G, int P, int len, int chunks) {
  const ispl_config c = config(L, N, G, P);
  const void* x = dev<void>(size_t(P) * c.pulse_stride * 4);
  const float* tx = dev<float>(size_t(P) * L * 8);
  float* out = dev<float>(size_t(G) * N * 4);
  ispl_ctx* ctx = nullptr;
  CHECK(ispl_create(&c, &ctx) == ISPL_OK);
  if (!ctx) return;
  g_grid_len = -1;
  CHECK(ispl_integrate_spectra(ctx, x, tx, 1, P, out, 0, nullptr) == ISPL_OK);
  if (g_grid_len != len || (len > 0 && g_chunks < chunks))
    fprintf(stderr, "L %d N %d G %d P %d: grid %d, %d chunks\n", L, N, G, P, g_grid_len, g_chunks);
  CHECK(g_grid_len == len && (len == 0 || g_chunks >= chunks));
  ispl_destroy(ctx);
  free_all();
}

// A context allocates for the pulses it may sum side by side, not for every
// pulse that a call may pass.
static void generous_max_pulses(int L, int N) {
  ispl_config c = config(L, N, 1, INT32_MAX);
  ispl_ctx* ctx = nullptr;
  size_t before = 0, after = 0;
  for (const auto& a : g_allocs) before += a.second;
  CHECK(ispl_create(&c, &ctx) == ISPL_OK);
  for (const auto& a : g_allocs) after += a.second;
  CHECK(after - before < (size_t{256} << 20));
  ispl_destroy(ctx);
}

// More codes than there are rows of sign bits: the call reads them as complex
// numbers; as many pulses with one shared code are packed.
static void more_codes_than_rows(int L, int N, int G, int P) {
  ispl_config c = config(L, N, G, P);
  ispl_ctx* ctx = nullptr;
  CHECK(ispl_create(&c, &ctx) == ISPL_OK);
  if (!ctx) return;
  const void* x = dev<void>(size_t(P) * c.pulse_stride * 4);
  const float* tx = dev<float>(size_t(P) * L * 8);
  float* out = dev<float>(size_t(G) * N * 4);
  const long folded = g_folded;
  long packed = g_packed;
  CHECK(ispl_integrate_spectra(ctx, x, tx, 1, P, out, 0, nullptr) == ISPL_OK);
  CHECK(g_folded == folded + 1 && g_packed == packed);
  CHECK(ispl_integrate_spectra(ctx, x, tx, 0, P, out, 0, nullptr) == ISPL_OK);
  CHECK(g_folded == folded + 2 && g_packed == packed + 1);
  ispl_destroy(ctx);
  free_all();
}

// The tuner's and a set plan's waves and chunks reach a mode that is summed on a grid.
static void tuned_modes() {
  const ispl_config c = config(300, 16384, 40, 400);
  ispl_batch* b = nullptr;
  CHECK(ispl_batch_create(&c, 1, &b) == ISPL_OK);
  if (!b) return;
  ispl_batch_io io{};
  io.samples = dev<void>(size_t(400) * c.pulse_stride * 4);
  io.tx_code = dev<float>(size_t(400) * c.code_len * 8);
  io.tx_per_pulse = 1;
  io.n_pulses = 400;
  io.spectra = dev<float>(size_t(c.n_gates) * c.fft_len * 4);
  auto waves = [] {
    std::set<int> w;
    for (const auto& p : g_plans) w.insert(p.first);
    return w;
  };
  ispl_batch_plan plan{};
  for (int w : {8, 16}) {
    g_plans.clear();
    CHECK(ispl_batch_get_plan(b, &plan) == ISPL_OK);
    plan.waves[0] = w;
    CHECK(ispl_batch_set_plan(b, &plan) == ISPL_OK);
    CHECK(ispl_batch_integrate(b, &io, 0, 0, nullptr) == ISPL_OK);
    CHECK(waves() == std::set<int>{w});
  }
  plan.waves[0] = 0;
  CHECK(ispl_batch_set_plan(b, &plan) == ISPL_OK);
  g_plans.clear();
  float ms = 0.f;
  CHECK(ispl_batch_tune(b, &io, 1, &plan, &ms) == ISPL_OK);
  CHECK((waves() == std::set<int>{8, 16}));
  CHECK(g_plans.size() > 2);  // and other chunk counts
  CHECK(ispl_batch_set_plan(b, &plan) == ISPL_OK);
  ispl_batch_destroy(b);
  free_all();
}

int main() {
  tuned_modes();
  const int shapes[][4] = {{16, 1024, 64, 700},   {256, 1024, 64, 100}, {300, 16384, 900, 60},
                           {600, 4096, 9000, 9},  {1000, 16384, 37, 90}, {1000, 65536, 2, 400},
                           {1024, 2048, 300, 40}, {33, 65536, 1, 64},    {128, 4096, 200, 500}};
  for (const auto& s : shapes) folded_calls(s[0], s[1], s[2], s[3]);
  const int longer[][4] = {{1025, 16384, 300, 64}, {2000, 32768, 600, 40}, {4096, 16384, 500, 20},
                           {8192, 65536, 1, 90},   {5000, 16384, 30, 30}};
  for (const auto& s : longer) folded_calls(s[0], s[1], s[2], s[3]);
  // the faster form as measured
  plan_of(256, 1024, 64, 100, 1024, 2);
  plan_of(524, 2048, 1143, 2, 0, 0);
  plan_of(999, 2048, 1061, 14, 0, 0);
  plan_of(114, 1024, 1254, 1, 0, 0);
  plan_of(595, 2048, 1, 150, 2048, 2);
  plan_of(3943, 16384, 162, 200, 8192, 2);
  plan_of(6611, 16384, 260, 656, 0, 0);
  plan_of(5525, 16384, 43, 13, 16384, 2);
  generous_max_pulses(16, 1024);
  generous_max_pulses(1000, 16384);
  generous_max_pulses(2000, 16384);
  more_codes_than_rows(1, 1024, 1, 300000);
  more_codes_than_rows(1030, 16384, 64, 17000);
  printf("folded launches: %ld, with packed codes: %ld\n", g_folded, g_packed);
  printf("checks failed: %d, runtime errors: %d\n", g_fail, mock_errors());
  return g_fail + mock_errors();
}
