// Result extraction (gfx950): the results of an evaluation in the layout the caller receives, so that one
// copy to the host ends the call.  Forming them on the host took two copies back, the ids' copy
// forth, a third copy and a host loop over the groups: 2.95 ms for the 66,496 groups of
// llama42b-d128-hw64 (9.0 MB of results) against 0.71 now, of which the copy into pageable memory
// takes 0.53; 0.57 against 0.12 ms for llama13b-d64's 9,634 groups.  Its bucket tables (9.9 MB) took
// 2.3 ms through host vectors, 0.57 straight into the caller's arrays.

#include "mist_device.h"

namespace mist {
namespace {

// A thread per result: the configuration's values and digits.  Result i is configuration ids[i] with
// objective objs[i] (with n_alpha > 0 the value of weight sample i mod n_alpha); key (or nullptr)
// holds the bits of its memory.  pad receives 1 when the values formed here differ from those.  Bound
// by latency: a binary search over the groups and the pair level's integer divisions.
__global__ __launch_bounds__(256) void k_results(EvalArgs a, const uint64_t* __restrict__ ids,
                                                 const double* __restrict__ objs, const uint64_t* __restrict__ key,
                                                 int32_t n_alpha, int64_t n, mist_result* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  mist_result r = {};
  r.id = ids[i];
  r.obj = objs[i];
  if (r.id >= a.n_configs) {  // kNone, or no configuration (results never written): the host refuses it
    r.t = r.d = r.mem = __builtin_huge_val();
    r.bucket = -1;
    r.cfg.hw = -1;
  } else {
    const Digits x = decode_one(a, r.id);
    const OneVal v = eval_one(a, x);
    const DevGroup g = a.groups[x.group];
    const DevHw& hw = a.hws[g.hw];
    const DevPair pr = a.pairs[g.pair_begin + x.p];
    r.t = v.t;
    r.d = v.d;
    r.mem = v.mem;
    double want = v.obj;
    if (n_alpha > 0) {
      const int q = (int)(i % n_alpha);
      want = __builtin_fma(a.alpha[q] * (double)g.G, v.t, a.beta[q] * v.d);
    }
    r.pad = want == r.obj && (!key || (uint64_t)__double_as_longlong(v.mem) == key[i]) ? 0 : 1;
    // The bucket as the evaluation kernel finds it: floor(mem * kNB) or the one above.
    const int j0 = (int)__builtin_fmin(v.mem * hw.kNB, 64.0);
    const int j = j0 < MIST_MAX_BUCKETS ? j0 + (v.mem > hw.edge[j0] ? 1 : 0) : j0;
    r.bucket = j < a.NB ? j : -1;
    r.cfg.hw = g.hw;
    r.cfg.G = g.G;
    r.cfg.PP = g.PP;
    r.cfg.k = g.k;
    r.cfg.l = g.l;
    r.cfg.b = pr.b;
    r.cfg.tp = pr.tp;
    r.cfg.dp = pr.dp;
    r.cfg.zero = x.z;
    r.cfg.ckpt = x.c;
    r.cfg.wo_idx = x.iw;
    r.cfg.go_idx = x.ig;
    r.cfg.oo_idx = x.io;
    r.cfg.ao_idx = x.ia;
    r.cfg.wo = a.ratio[x.iw];
    r.cfg.go = a.ratio[x.ig];
    r.cfg.oo = a.ratio[x.io];
    r.cfg.ao = a.ratio[x.ia];
  }
  out[i] = r;
}

// The planner's points of groups [g0, g0 + n): the best configuration, then each weight sample's.
__global__ __launch_bounds__(256) void k_points(EvalArgs a, const uint64_t* __restrict__ best,
                                                const uint64_t* __restrict__ alpha, int32_t n_alpha, int64_t g0,
                                                int64_t n, PlanPoint* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * (1 + n_alpha)) return;
  const int64_t g = g0 + i / (1 + n_alpha);
  const int q = (int)(i % (1 + n_alpha));
  PlanPoint p{q == 0 ? best[g] : alpha[g * n_alpha + q - 1], 0.0, 0.0};
  if (p.id < a.n_configs) {  // else kNone, or an id that the host refuses
    const OneVal v = eval_one(a, p.id);
    p.t = v.t;
    p.d = v.d;
  }
  out[i] = p;
}

// Rows of 64 words cut to their first NB.
__global__ __launch_bounds__(256) void k_rows(const uint64_t* __restrict__ in, int32_t NB, int64_t n,
                                              uint64_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n * NB) out[i] = in[i / NB * 64 + i % NB];
}

unsigned blocks256(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

int launch_results(const EvalArgs& a, const uint64_t* ids, const double* objs, const uint64_t* key, int32_t n_alpha,
                   int64_t n, mist_result* out, void* stream) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(k_results, dim3(blocks256(n)), dim3(256), 0, (hipStream_t)stream, a, ids, objs, key, n_alpha, n, out);
  return (int)hipGetLastError();
}

int launch_points(const EvalArgs& a, const uint64_t* best, const uint64_t* alpha, int32_t n_alpha, int64_t g0, int64_t n,
                  PlanPoint* out, void* stream) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(k_points, dim3(blocks256(n * (1 + n_alpha))), dim3(256), 0, (hipStream_t)stream, a, best, alpha,
                     n_alpha, g0, n, out);
  return (int)hipGetLastError();
}

int launch_rows(const uint64_t* in, int32_t NB, int64_t n, uint64_t* out, void* stream) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(k_rows, dim3(blocks256(n * NB)), dim3(256), 0, (hipStream_t)stream, in, NB, n, out);
  return (int)hipGetLastError();
}

}  // namespace mist
