// The library's host side on the CPU: mist_host.cpp itself, over a stand-in for the HIP runtime whose
// device memory is host memory and whose kernels only record what they were given.  Each scenario
// exercises what a healthy GPU run does not show (the order of reads, failing allocations and copies)
// and exits with 0, or prints what differs.  Built and run by test_host_harness.py.

#include "../paper_2503_19050_amd/csrc/mist_host.cpp"

#include <cstdlib>
#include <functional>

namespace {

struct Op {
  char kind;        // 's' stream synchronized, 'c' copy, 'k' kernel
  void* stream;
  int device;
};
std::vector<Op> g_log;
int g_device = 0;            // current device
long g_copies_left = -1;     // copies that succeed before one fails (-1: none does)
long g_mallocs_left = -1;    // device allocations that succeed before one fails (-1: none does)
int g_emit_count = 0;        // candidates that the candidate pass reports per tile
long g_news_left = -1;       // allocations that succeed before one throws (-1: none does)
bool g_news_stay = false;    // and whether every later one throws as well
std::vector<DevTile> g_emit_tiles;  // what the last candidate pass was given
uint64_t g_result_id = ~0ull;       // the id that the result kernels report

void log(char kind, void* st) {
  if (g_news_left < 0) g_log.push_back({kind, st, g_device});
}

hipError_t copy(void* dst, const void* src, size_t n, void* st) {
  log('c', st);
  if (g_copies_left >= 0 && g_copies_left-- == 0) return hipErrorUnknown;
  std::memcpy(dst, src, n);
  return hipSuccess;
}

}  // namespace

void* operator new(size_t n) {
  if (g_news_left >= 0 && g_news_left-- == 0) {
    if (g_news_stay) g_news_left = 0;
    throw std::bad_alloc();
  }
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return std::malloc(n ? n : 1); }
void operator delete(void* p, const std::nothrow_t&) noexcept { std::free(p); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (g_mallocs_left >= 0 && g_mallocs_left-- == 0) return hipErrorOutOfMemory;
  *p = std::malloc(n);
  std::memset(*p, 0x7E, n);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return copy(d, s, n, nullptr); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) { return copy(d, s, n, st); }
hipError_t hipStreamSynchronize(hipStream_t st) {
  log('s', st);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = g_device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  g_device = d;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 4;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorUnknown; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorUnknown; }
}

namespace mist {

int noalloc_scratch(void**) { return (int)hipErrorUnknown; }
int launch_pairs(const EvalArgs& a, void* st) {
  log('k', st);
  if (a.pool_count) *a.pool_count = 0;
  return 0;
}
int launch_eval(const EvalArgs&, int, int, void* st) { return log('k', st), 0; }
int eval_blocks_per_cu(int, int) { return 4; }
int search_blocks_per_cu(int, int) { return 4; }
int launch_search(const EvalArgs& a, int, int mode, void* st) {
  log('k', st);
  if (mode == kModeEmit) {
    g_emit_tiles.assign(a.tiles, a.tiles + a.n_tiles);
    for (int32_t t = 0; t < a.n_tiles; ++t) {
      a.cnt_tile[t] = g_emit_count;
      a.tile_drop[t] = 0;
      a.tile_live[t] = 0;
    }
  }
  return 0;
}
int launch_reduce(const ReduceArgs& r, void* st) {  // every group: its best and all buckets are configuration 0
  log('k', st);
  for (int64_t g = 0; g < r.n_groups; ++g) {
    r.best_id[g] = 0;
    r.frontier[g] = 1;
  }
  return 0;
}
int launch_eval_ids(const EvalArgs&, const uint64_t*, int64_t, double*, void* st) { return log('k', st), 0; }
int launch_filter(const EvalArgs&, const double*, const uint64_t*, FiltEntry*, void* st) { return log('k', st), 0; }
int launch_results(const EvalArgs&, const uint64_t*, const double*, const uint64_t*, int32_t, int64_t n, mist_result* out, void* st) {
  log('k', st);
  for (int64_t i = 0; i < n; ++i) {
    out[i] = mist_result{};
    out[i].id = g_result_id;
  }
  return 0;
}
int launch_points(const EvalArgs&, const uint64_t*, const uint64_t*, int32_t n_alpha, int64_t, int64_t n, PlanPoint* out, void* st) {
  log('k', st);
  for (int64_t i = 0; i < n * (1 + n_alpha); ++i) out[i] = PlanPoint{g_result_id, 1.0, 0.0};
  return 0;
}
int launch_rows(const uint64_t*, int32_t NB, int64_t n, uint64_t* out, void* st) {
  log('k', st);
  for (int64_t i = 0; i < n * NB; ++i) out[i] = 0;
  return 0;
}
int launch_prefilter(uint64_t*, double*, uint64_t*, const int64_t*, int64_t, int64_t*, void* st) { return log('k', st), 0; }
int exact_sort(const uint64_t*, uint64_t*, uint32_t*, uint64_t*, uint32_t*, int64_t, const int64_t*, const int64_t*, void* st) {
  return log('k', st), 0;
}
int launch_compact(const uint64_t*, const double*, const uint64_t*, const int64_t*, const int32_t*, const uint8_t*,
                   const int64_t*, int32_t, uint64_t*, double*, uint64_t*, void* st) {
  return log('k', st), 0;
}
int launch_pool_place(const uint64_t*, const double*, const uint64_t*, const int32_t*, const int32_t*, int64_t,
                      const uint8_t*, const int64_t*, uint64_t*, double*, uint64_t*, void* st) {
  return log('k', st), 0;
}
int launch_front_scan(const uint32_t*, const uint64_t*, const double*, const uint64_t*, const int64_t*, const int64_t*,
                      int64_t n_groups, uint64_t*, double*, uint64_t*, int64_t* cnt, void* st) {
  log('k', st);
  for (int64_t g = 0; g < n_groups; ++g) cnt[g] = 0;
  return 0;
}

}  // namespace mist

namespace {

int g_bad = 0;
void check(bool ok, const char* what) {
  if (!ok) {
    std::printf("differs: %s\n", what);
    g_bad = 1;
  }
}

mist_space* make_space(int64_t devices, int32_t n_buckets, int32_t n_alphas, int32_t n_ratios) {
  mist_model_desc m{};
  m.arch = MIST_ARCH_GPT;
  m.n_layers = 6;
  m.hidden = 512;
  m.heads = m.kv_heads = 8;
  m.ffn = 2048;
  m.seq = 256;
  m.vocab = 1000;
  m.bytes_w = 2;
  m.bytes_opt = 12;
  m.flash = 1;
  mist_hw_desc h{};
  h.flops = 1e14;
  h.mem_bytes = 1e10;
  h.pcie_bw = 3e10;
  h.link_bw = 1e11;
  h.eta_max = 0.75;
  h.n_half = 1024;
  for (auto& row : h.phi)
    for (double& v : row) v = 1.0;
  const int32_t mb[] = {1, 2};
  double r[MIST_MAX_RATIOS], al[] = {0.25, 0.75};
  for (int32_t i = 0; i < n_ratios; ++i) r[i] = (double)i / n_ratios;
  mist_space_desc s{};
  s.n_devices = devices;
  s.global_batch = 16 * devices;
  s.mb = mb;
  s.n_mb = 2;
  s.ratios = r;
  s.n_ratios = n_ratios;
  s.n_buckets = n_buckets;
  s.l_rule = MIST_L_FULL;
  s.n_alphas = n_alphas;
  s.alphas = al;
  mist_space* S = nullptr;
  const mist_status rc = mist_space_create(&m, &h, 1, &s, nullptr, &S);
  if (rc) std::printf("create: %d %s\n", rc, mist_last_error());
  return S;
}

struct Read {
  const char* name;
  std::function<mist_status(mist_space*)> call;
};

// Every call that reads results back.
std::vector<Read> reads(std::vector<mist_result>& out, std::vector<uint64_t>& ids) {
  out.resize(4096);
  ids.resize(1 << 16);
  return {
      {"best", [&](mist_space* S) { return mist_get_best(S, 0, 1, out.data()); }},
      {"alpha", [&](mist_space* S) { return mist_get_alpha(S, 0, 1, out.data()); }},
      {"plan", [&](mist_space* S) { static mist_plan p; return mist_plan_pipeline(S, 0, 0, &p); }},
      {"buckets", [&](mist_space* S) { return mist_get_buckets(S, 0, 1, ids.data(), nullptr, nullptr); }},
      {"masks", [&](mist_space* S) { return mist_get_buckets(S, 0, 1, nullptr, nullptr, ids.data()); }},
      {"pareto", [&](mist_space* S) { int32_t n = 0; return mist_get_pareto(S, 0, out.data(), 64, &n); }},
  };
}

// Results are read on the null stream of the space's device, after the evaluation's stream was waited
// for: whatever the caller queued on the null stream or a blocking stream since comes first.
void order_of_reads() {
  std::vector<mist_result> out;
  std::vector<uint64_t> ids;
  void* const side = (void*)0x1000;
  void* const other = (void*)0x2000;
  mist_space* S = make_space(2, 7, 2, 3);
  check(mist_eval_space(S, side) == MIST_OK, "evaluation");
  auto ordered = [&](const char* name, void* stream) {
    size_t i = 0;
    while (i < g_log.size() && !(g_log[i].kind == 's' && g_log[i].stream == stream)) check(g_log[i++].kind == 's', name);
    check(i < g_log.size(), name);
    bool any = false;
    for (; i < g_log.size(); ++i) {
      if (g_log[i].kind != 's') any = true;
      check(g_log[i].kind == 's' || (g_log[i].stream == nullptr && g_log[i].device == 0), name);
    }
    check(any, name);
    check(g_log.back().kind == 's' && g_log.back().stream == nullptr, name);
  };
  for (int device = 0; device < 2; ++device) {
    for (const Read& r : reads(out, ids)) {
      g_device = device;
      g_log.clear();
      check(r.call(S) == MIST_OK, r.name);
      ordered(r.name, side);
      check(g_device == device, r.name);
    }
    g_device = 0;
  }
  check(mist_eval_pareto_exact(S, other) == MIST_OK, "exact frontier");
  int64_t n = 0;
  g_log.clear();
  check(mist_get_pareto_exact(S, 0, out.data(), 64, &n) == MIST_OK && n == 0, "exact staircase");
  ordered("exact staircase", other);
  mist_space_destroy(S);
}

// Ids that no evaluation wrote are refused.
void ids_out_of_range() {
  std::vector<mist_result> out;
  std::vector<uint64_t> ids;
  mist_space* S = make_space(2, 7, 2, 3);
  check(mist_eval_space(S, nullptr) == MIST_OK, "evaluation");
  for (uint64_t id : {S->n_configs, (uint64_t)0x7F7F7F7F7F7F7F7F, (uint64_t)-2}) {
    g_result_id = id;
    for (const Read& r : reads(out, ids))
      if (std::strcmp(r.name, "buckets") && std::strcmp(r.name, "masks"))  // raw tables: copied as they are
        check(r.call(S) == MIST_E_RANGE, r.name);
  }
  for (uint64_t id : {(uint64_t)0, S->n_configs - 1, (uint64_t)-1}) {
    g_result_id = id;
    for (const Read& r : reads(out, ids)) check(r.call(S) == MIST_OK, r.name);
  }
  mist_space_destroy(S);
}

// The candidate tiles are whole or absent, whichever host allocation fails.
void candidate_tiles() {
  mist_space* S = make_space(4, 64, 0, 3);
  for (long k = 0;; ++k) {
    bool thrown = false;
    g_news_left = k;
    try {
      build_cand_tiles(S, 16);
    } catch (const std::bad_alloc&) {
      thrown = true;
    }
    g_news_left = -1;
    check(thrown ? S->cand_first.empty() && S->cand_tiles.empty()
                 : S->cand_first.size() == S->groups.size() + 1 && (size_t)S->cand_first.back() == S->cand_tiles.size(),
          "candidate tiles");
    if (!thrown) {
      check(k > 8, "allocations that can fail");
      break;
    }
  }
  mist_space_destroy(S);
}

// Whichever copy, device allocation or host allocation of the first exact frontier fails, the call reports
// it and the next one starts over with whole tables.
void exact_tables() {
  mist_space* R = make_space(4, 64, 0, 3);
  build_cand_tiles(R, resident_blocks(R, kModeEmit) * kWaves);
  long* const failing[] = {&g_copies_left, &g_mallocs_left, &g_news_left};
  const mist_status codes[] = {MIST_E_DEVICE, MIST_E_NOMEM, MIST_E_NOMEM};
  g_emit_count = 1;
  for (int f = 0; f < 3; ++f) {
    for (long k = 0;; ++k) {
      mist_space* S = make_space(4, 64, 0, 3);
      check(mist_eval_space(S, nullptr) == MIST_OK, "evaluation");
      *failing[f] = k;
      const mist_status rc = mist_eval_pareto_exact(S, nullptr);
      *failing[f] = -1;
      if (rc) {
        check(rc == codes[f], "status");
        int64_t n = 0;
        check(mist_get_pareto_exact(S, 0, nullptr, 0, &n) == MIST_E_STATE, "no frontier after a failed call");
      }
      for (int again = 0; again < 2; ++again) {
        g_emit_tiles.clear();
        check(mist_eval_pareto_exact(S, nullptr) == MIST_OK, "the next call");
        check(g_emit_tiles.size() == R->cand_tiles.size() &&
                  !std::memcmp(g_emit_tiles.data(), R->cand_tiles.data(), R->cand_tiles.size() * sizeof(DevTile)),
              "the tiles of the next call");
        check(S->cand_cap == (int64_t)R->cand_tiles.size() && S->d_front_obj, "the candidates of the next call");
      }
      mist_space_destroy(S);
      if (!rc) {
        check(k > (f == 1 ? 28 : 4), "calls that can fail");
        break;
      }
    }
  }
  mist_space_destroy(R);
}

// A call that runs out of host memory and finds none for its message either returns MIST_E_NOMEM.
void out_of_memory() {
  std::vector<mist_result> out;
  std::vector<uint64_t> ids;
  const auto calls = reads(out, ids);
  std::vector<mist_stage_point> pts;
  for (int32_t l = 1; l <= 6; ++l) pts.push_back({2, 1, 1, l, (uint64_t)l, 1.0 + l, 0.5});
  mist_plan plan;
  mist_space* S = make_space(4, 7, 2, 3);
  check(mist_eval_space(S, nullptr) == MIST_OK, "evaluation");
  const std::function<mist_status()> run[] = {[&] { return mist_eval_pareto_exact(S, nullptr); },
                                              [&] { return mist_plan_points(pts.data(), (int64_t)pts.size(), 6, 0, &plan); },
                                              [&] { return mist_plan_pipeline(S, 0, 0, &plan); },
                                              [&] { return mist_get_best(S, 0, 1, out.data()); }};
  for (const auto& f : run)
    for (long k = 0;; ++k) {
      g_news_stay = true;
      g_news_left = k;
      const mist_status rc = f();
      g_news_left = -1;
      check(rc == MIST_OK || rc == MIST_E_NOMEM, "status without memory");
      if (rc == MIST_OK) break;
    }
  mist_space_destroy(S);
}

// Which spaces are searched with bounds: the lines of use_bounds, from both sides.
void search_rule() {
  const struct {
    int64_t D;
    int32_t A;
    uint64_t n, groups;
    bool want;
  } rows[] = {
      {16, 0, 120000000, 1000, true},  {16, 0, 119999999, 1000, false}, {2, 0, 120000000, 1000, true},
      {16, 0, 120000000, 15000, true}, {16, 0, 120000000, 15001, false}, {16, 0, 0, 0, false},
      {8, 4, 450000000, 1000, true},   {8, 4, 449999999, 1000, false},  {5, 4, 450000000, 1000, true},
      {4, 4, 599999999, 1000, false},  {4, 4, 600000000, 1000, true},   {2, 1, 500000000, 100, false},
      {8, 4, 450000000, 15000, true},  {8, 4, 450000000, 15001, false}, {4, 4, 600000000, 20001, false}};
  for (const auto& r : rows) {
    mist_space S;
    S.D = r.D;
    S.A = r.A;
    S.n_configs = r.n;
    S.groups.resize(r.groups);
    check(use_bounds(&S) == r.want, "which spaces are searched");
  }
}

}  // namespace

int main(int argc, char** argv) {
  const struct {
    const char* name;
    void (*run)();
  } all[] = {{"order_of_reads", order_of_reads}, {"ids_out_of_range", ids_out_of_range},
             {"candidate_tiles", candidate_tiles}, {"exact_tables", exact_tables}, {"search_rule", search_rule}, {"out_of_memory", out_of_memory}};
  for (const auto& s : all)
    if (argc == 2 && !std::strcmp(argv[1], s.name)) {
      s.run();
      return g_bad;
    }
  std::printf("no such scenario\n");
  return 2;
}
