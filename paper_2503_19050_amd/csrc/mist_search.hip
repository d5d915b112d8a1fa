// The bounded search over large spaces, and the exact frontier's candidate pass (gfx950).

#include "mist_bounds.h"
#include "mist_device.h"

namespace mist {
namespace {

// Overflow pool of the exact frontier's candidate pass: each wave takes chunks of kPoolChunk
// slots; the slots of a chunk it leaves unused are marked (tile -1) so that the placement skips
// them.
constexpr int kPoolChunk = 256;

// Every lane of the wave calls this.
__device__ __forceinline__ void pool_holes(const EvalArgs& a, unsigned long long base, int used, int lane) {
  for (int i = used + lane; i < kPoolChunk; i += 64) {
    const unsigned long long pos = base + (unsigned long long)i;
    if (pos < (unsigned long long)a.pool_cap) a.pool_tile[pos] = -1;
  }
}

// ---------------------------------------------------------------------------------------
// K1.  Bounded search: the results are minima (per bucket) or a filtered set (exact frontier), so
// a part of the space whose lower bound on the objective is above what it would have to beat is
// decided without forming its times.  A tile's strips are visited top down:
//   - unit (pair, recomputed layers, ZeRO level; R^4 configurations), one lane each: bounds of the
//     unit's memory and objective over all its ratios; live units' constants go to LDS records;
//   - strip (weight and gradient ratio), one lane each, 64 at a time: the levels that the strip
//     fixes, and bounds of its peak without the activation terms over the optimizer ratios;
//   - column (activation ratio), the same for every lane: the memory range over the optimizer
//     ratios and two lower bounds on the objective, before and after forming the stable time;
//   - configuration (optimizer ratio): its own memory, bucket and bound, then, only when some lane
//     of the wave may still win, Algorithm 1 and the reduction step.
// Each test is wave-uniform (a ballot), so a level is skipped when it fails in every lane.
//
// The bounds.  Every slowdown factor is at least 1, so each stream's standalone time is progressed
// by at most the phase length in every phase of Algorithm 1: a time it returns is at least each of
// its streams' times.  With t >= tl and T1 >= T1l, obj = G t + (T1 - t) >= (G - 1) tl + T1l.  Host
// streams grow with every ratio, so a level's smallest ones come with the smallest ratios still
// open.  The memory without the activation terms is max(BF, BB), each a sum over the ratios of
// functions that are linear in one ratio, so over the open ratios BF and BB lie between the sums of
// their end values' minima and maxima, and the maximum of the two between the maximum of their lower
// and that of their upper bounds.  Rounding: all terms are non-negative and a value takes a few
// dozen operations of relative error 2^-53; the objective's bound is lowered by a relative 2^-30
// (hw.lbs; with factors above 2^16, where T1 - t may cancel beyond that, it is lowered to 0 and
// excludes nothing) and memory ranges are widened by a relative 2^-28.
//
// The thresholds.  In a bucket's minimum a configuration matters only if its objective is at most
// the smallest known for its bucket (equal: the lowest id wins), so the test compares its bound with
// the largest threshold among the buckets of its memory range (range_max).  A tile starts from its
// group's thresholds so far (thr, filled by the seed variant below and lowered by every tile of the
// group as it goes), each the objective of some configuration of that bucket: never below the
// final minimum, so the winner itself is never excluded, whatever the order of the tiles.  In the
// exact frontier's variant the threshold is pm, the least objective of the lower buckets, which
// does not increase with the bucket: the lowest bucket of the range decides.
// ---------------------------------------------------------------------------------------
// What a strip needs of its unit (pair, recomputed layers, ZeRO level).  Kept small: the wave's records,
// its queue and its tables decide how many blocks a CU holds.
struct UnitRec {
  double Pw, iD, Wb2;        // stage fp16 parameter bytes, 1 / DP, double-buffered fp16 unit
  double So, Obo;            // optimizer states, their part of the optimizer-step unit
  double Xd;                 // logits
  double A, KA, A2;          // microbatch activations, in-flight stash, offload buffers
  double C, gs, gf;          // compute, GPU-GPU stable and first microbatch
  int32_t unit, ckpt;        // unit index (its last two bits: the ZeRO level); whether layers are recomputed
};

constexpr int kQueue = 128;  // queue of columns: fewer than 64 left over, and one push of 64

constexpr int kRangeLevels = 7;  // range maxima over 1, 2, 4, .. 64 buckets

// Largest of the thresholds of buckets a..b (0 <= a <= b <= 63): level e of tab holds the maxima over
// [i, i + 2^e).
__device__ __forceinline__ double range_max(const float* __restrict__ tab, unsigned int a, unsigned int b) {
  const unsigned int e = 31u - (unsigned int)__builtin_clz(b - a + 1u);
  const float* row = tab + e * 64u;
  return (double)__builtin_fmaxf(row[a], row[b + 1u - (1u << e)]);
}

// Live unit records per wave: as many as four blocks per CU leave room for.
template <int MODE>
constexpr int unit_slots() { return MODE == kModeAlpha || MODE == kModeSeedAlpha ? 28 : 32; }

template <int R, int MODE>
__global__ __launch_bounds__(kBlock, 4) void k_search(EvalArgs a, const double* __restrict__ ratio,
                                                      const PairK* __restrict__ pk) {
  constexpr bool EX = MODE == kModeEmit;
  constexpr bool DM = MODE == kModeDump;
  constexpr bool SD = MODE == kModeSeed || MODE == kModeSeedAlpha;
  constexpr bool AL = MODE == kModeAlpha || MODE == kModeSeedAlpha;
  constexpr bool BK = MODE == kModeBuckets || SD || AL;
  constexpr bool QU = !SD;  // columns go through the queue
  constexpr int R2 = R * R;
  constexpr int kUnits = unit_slots<MODE>();
  __shared__ double s_tab[kWaves][16 * kLdsRow + 2 * kTab2];
  __shared__ BucketEntry s_bucket[kWaves][65];  // entries NB..64: sinks of infeasible configurations
  __shared__ UnitRec s_unit[kWaves][kUnits];
  __shared__ float s_range[BK ? kWaves : 1][BK ? kRangeLevels * 64 : 1];
  __shared__ double s_ratio[2 * R];
  __shared__ double s_qt[QU ? kWaves : 1][QU ? kQueue : 1];   // queued columns: their stable times
  __shared__ uint32_t s_qi[QU ? kWaves : 1][QU ? kQueue : 1];  // and what they are
  __shared__ FiltEntry s_filt[EX ? kWaves : 1][EX ? 64 : 1];
  __shared__ double2 s_ab[AL ? kWaves : 1][kMaxAlphas];      // alpha * G, 1 - alpha
  __shared__ AlphaEntry s_aent[AL ? kWaves : 1][kMaxAlphas];
  __shared__ double2 s_apq[AL ? kWaves : 1][kMaxAlphas];     // limits of d: P - Q t

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // The wave index is uniform across the wave: stated, so that the tile, group and hardware
  // values derived from it live in scalar registers (scalar loads) rather than in every lane.
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NB = a.NB;
  const double* __restrict__ rr = ratio;  // read-only and uniform: scalar loads
  const double* __restrict__ om = ratio + R;
  if (tid < 2 * R) s_ratio[tid] = ratio[tid];
  __syncthreads();
  const bool r0_zero = rr[0] == 0.0;
  const double ra0 = rr[0], ra1 = rr[R - 1], qa0 = om[0], qa1 = om[R - 1];  // the end ratios
  double* tab = s_tab[wave];
  BucketEntry* bucket = s_bucket[wave];
  float* range = s_range[BK ? wave : 0];
  UnitRec* units = s_unit[wave];
  const unsigned long long kEmpty = (unsigned long long)__double_as_longlong(__builtin_huge_val());

  // Tile schedule: wave w of the grid takes work item w.  Item n_waves + x + kClaimCounters
  // * c goes to the claim that draws number c from counter x (counters reset to 0 by K0); a
  // wave draws from the counter of its block's XCD and moves to the next counter when one
  // runs out, until all have.  When the grid has at least as many waves as there are items
  // no claim is made.  Item x is tile tile_order[x] (the host gives each XCD's items a
  // contiguous range of tiles), or tile tile_list[x] when a variant runs a list; the seed
  // variant's items are the groups.
  const bool listed = (EX || DM) && a.tile_list != nullptr;
  const int n_items = SD ? (int)a.n_groups : (listed ? a.n_list : a.n_tiles);
  const int n_waves = (int)gridDim.x * kWaves;
  const bool claims = n_items > n_waves;
  int counter = (int)(blockIdx.x % kClaimCounters);
  int exhausted = 0;
  int loaded_hw = -1;
  // Exact frontier: the wave's current chunk of overflow-pool slots (none yet: used = chunk).
  unsigned long long pool_base = 0;
  int pool_used = kPoolChunk;
  for (int x = (int)blockIdx.x * kWaves + wave; x < n_items;) {
    const int t = SD ? 0 : (listed ? load_uniform(a.tile_list + x) : (a.tile_order ? load_uniform(a.tile_order + x) : x));
    DevTile tile{x, 0, 0, 0};
    if constexpr (!SD) tile = load_uniform(a.tiles + t);
    const DevGroup g = load_uniform(a.groups + tile.group);
    const DevHw& hw = a.hws[g.hw];
    if (g.hw != loaded_hw) {  // the wave's LDS copy of the hardware tables
      for (int i = lane; i < 16 * kTabStride; i += 64)
        tab[(i / kTabStride) * kLdsRow + i % kTabStride] = (&hw.itab[0][0])[i];
      wave_sync();
      if (lane < 2 * kTab2) {  // the third round's rows of compute and one host stream, from the rows
        const int h = 2 + lane / kTab2, i = lane % kTab2;
        const int row = i < 4 ? (1 | (1 << h)) : 13;
        const int col = ((i & 1) ? h : 0) + (i >= 2 ? 4 : 0);  // phi[0], phi[h], psi[0], psi[h], psi[0], psi[h]
        tab[kTab2Off + lane] = tab[row * kLdsRow + col];
      }
      bucket[lane].edge = hw.edge[lane];
      loaded_hw = g.hw;
    }
    // Buckets 0..NB-1 start empty.  Entries NB..64 are sinks: they hold key 0 and local id
    // 0, which no configuration beats, so an infeasible configuration sent to one never
    // takes part.
    lds_store(&bucket[lane].key, lane < NB ? kEmpty : 0ull);
    lds_store(&bucket[lane].lid, lane < NB ? 0xFFFFFFFFu : 0u);
    if (lane == 0) {
      bucket[64].edge = __builtin_huge_val();
      bucket[64].key = 0ull;
      bucket[64].lid = 0u;
    }
    const double Gd = (double)g.G;
    const double Gm1 = Gd - 1.0;
    int64_t n_cand = 0;  // exact frontier: the next candidate's slot
    int64_t n_beg = 0;   // and the tile's window of slots
    int64_t n_end = 0;
    [[maybe_unused]] bool any_live = false;  // and whether some unit may hold one
    bool dropped = false;  // and whether a candidate of this lane found no place
    if constexpr (EX) {
      s_filt[wave][lane] = a.filt[(size_t)tile.group * 64 + lane];
      n_beg = load_uniform(a.win_begin + t);  // wave-uniform: scalar registers
      n_end = load_uniform(a.win_end + t);
      n_cand = n_beg;
    }
    if constexpr (AL) {
      if (lane < a.n_alpha) {
        s_ab[wave][lane] = make_double2(a.alpha[lane] * Gd, a.beta[lane]);
        lds_store(&s_aent[wave][lane].val, __builtin_huge_val());
        lds_store(&s_aent[wave][lane].key, order_key(__builtin_huge_val()));
        lds_store(&s_aent[wave][lane].lid, 0xFFFFFFFFu);
      }
    }
    wave_sync();

    const double iP = load_uniform(&hw.iP), kNB = load_uniform(&hw.kNB), M = load_uniform(&hw.M);
    const double lbs = load_uniform(&hw.lbs);
    [[maybe_unused]] const double slope0 = load_uniform(&hw.slope[0]), slope1 = load_uniform(&hw.slope[1]),
                                  slope2 = load_uniform(&hw.slope[2]);
    const double kLo = kNB * (1.0 - 0x1p-28), kHi = kNB * (1.0 + 0x1p-28), Mhi = M * (1.0 + 0x1p-28);
    const RowK RK{load_uniform(&hw.itab[15][2]), load_uniform(&hw.itab[15][3]), load_uniform(&hw.itab[15][6]),
                  load_uniform(&hw.itab[15][7]), load_uniform(&hw.itab[13][2]), load_uniform(&hw.itab[13][3])};
    const int l = g.l;
    const int64_t ke = g.k < g.G ? g.k : g.G;
    unsigned long long* const thr = a.thr ? a.thr + (size_t)tile.group * 64 : nullptr;
    unsigned long long* const athr = AL && a.athr ? a.athr + (size_t)tile.group * a.n_alpha : nullptr;

    bool changed = false;  // some threshold fell since the tables below were formed
    // The range maxima of the thresholds, each rounded up to the next float (at least the smallest
    // normal one): still an upper bound.
    auto build_range = [&](unsigned long long key) {
      const unsigned int up = __float_as_uint((float)__longlong_as_double((long long)key));
      unsigned int v = up >= 0x7F800000u ? 0x7F800000u : max(up + 1u, 0x00800000u);
#pragma unroll
      for (int e = 0; e < kRangeLevels; ++e) {
        range[e * 64 + lane] = __uint_as_float(v);
        v = max(v, (unsigned int)__shfl_down((int)v, 1u << e, 64));  // past lane 63: its own
      }
      wave_sync();
    };
    // Weight samples: with b = 1 - alpha > 0 a configuration matters to a sample only if
    // d <= (v - alpha G t) / b with v the sample's smallest value known, a limit P - Q t of d given t.
    // Q is lowered and P raised by a relative 2^-40 of their own magnitudes, far above the rounding
    // of the limit and of the weighted value, in which the two may cancel.
    [[maybe_unused]] auto build_alpha = [&]() {
      if (lane < a.n_alpha) {
        const double2 ab = s_ab[wave][lane];
        const double v = lds_load(&s_aent[wave][lane].val);
        const double ib = ab.y > 0.0 ? 1.0 / ab.y : 0.0;
        double P = v * ib;
        P = P + __builtin_fabs(P) * 0x1p-40;
        s_apq[wave][lane] = ab.y > 0.0 ? make_double2(P, ab.x * ib * (1.0 - 0x1p-40)) : make_double2(v, -1.0);
      }
      wave_sync();
    };
    // The largest d with which a configuration of stable time t may matter to some sample.
    [[maybe_unused]] auto d_limit = [&](double t) -> double {
      double lim = -__builtin_huge_val();
      for (int q = 0; q < a.n_alpha; ++q) {
        const double2 pq = s_apq[wave][q];
        if (pq.y < 0.0)  // alpha = 1: any d, if G t is small enough
          lim = Gd * t * (1.0 - 0x1p-40) <= pq.x ? __builtin_huge_val() : lim;
        else
          lim = __builtin_fmax(lim, __builtin_fma(-pq.y, t, pq.x));
      }
      return lbs > 0.0 ? lim : __builtin_huge_val();
    };
    // Exchanges thresholds with the group's other tiles.  An entry that another tile holds lower
    // takes that value with no local id: a configuration of this tile that reaches it later records
    // its own.
    auto exchange = [&](bool publish) {
      wave_sync();
      unsigned long long key = lds_load(&bucket[lane].key);
      if (thr && !SD && lane < NB) {
        const unsigned long long cur = __hip_atomic_load(thr + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur < key) {
          lds_store(&bucket[lane].key, cur);
          lds_store(&bucket[lane].lid, 0xFFFFFFFFu);
          key = cur;
        } else if (publish && key < cur) {
          __hip_atomic_fetch_min(thr + lane, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      build_range(key);
      if constexpr (AL) {
        if (lane < a.n_alpha) {
          AlphaEntry* const e = &s_aent[wave][lane];
          const unsigned long long mine = lds_load(&e->key);
          if (athr && !SD) {
            const unsigned long long cur = __hip_atomic_load(athr + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (cur < mine) {
              lds_store(&e->key, cur);
              lds_store(&e->val, order_value(cur));
              lds_store(&e->lid, 0xFFFFFFFFu);
            } else if (publish && mine < cur) {
              __hip_atomic_fetch_min(athr + lane, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
          }
        }
        build_alpha();
      }
    };
    // The tables formed from the thresholds, after some fell.
    auto refresh = [&]() {
      wave_sync();
      build_range(lds_load(&bucket[lane].key));
      if constexpr (AL) build_alpha();
      changed = false;
    };
    // A column's first-microbatch time T10 at the smallest optimizer ratio (host streams h0, d0), and the
    // slope sl by which it grows at least.  Another optimizer ratio's is that time with both host
    // streams longer by the same (r - r0) So / PCIe, and Algorithm 1's time is continuous and
    // piecewise linear in that length, with no slope below slope0 (slope1 when GPU-GPU finishes first at
    // the smallest ratio, slope2 when compute follows: as the host streams grow, it stays so).
    [[maybe_unused]] auto first_times = [&](const KnownRow& fr, double C, double gf, int ia, double h0, double d0, bool free,
                                            double& T10, double& sl) {
      int f0 = kFormGeneral;
      if (__builtin_amdgcn_ballot_w64((ia == 0) & !free))
        T10 = interference(C, gf, h0, d0, tab);
      else
        T10 = interference_known(fr, h0, d0, free, tab, RK, f0);
      sl = f0 == kFormGeneral ? slope0 : (f0 == kFormHostsLeft ? slope2 : slope1);
    };
    // The largest objective that a configuration in the memory range [lo, hi] may have to matter.
    auto limit = [&](double lo, double hi) -> double {
      const unsigned int ja = (unsigned int)__builtin_fmin(lo * kLo, 63.0);
      if constexpr (EX) {
        return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(s_filt[wave]) +
                                                __umul24(ja, (unsigned int)sizeof(FiltEntry)));
      } else if constexpr (BK) {
        const unsigned int jb = (unsigned int)__builtin_fmin(hi * kHi, 63.0);
        return range_max(range, ja, max(ja, jb));
      } else {
        return __builtin_huge_val();
      }
    };
    // Whether something of memory at least lo and objective bound lb can matter below limit th.
    auto alive = [&](double lo, double lb, double th) -> bool {
      if constexpr (DM) return true;
      if constexpr (EX) return (lo <= Mhi) & (lb * lbs < th);
      return (lo <= Mhi) & (lb * lbs <= th);
    };

    // Whether something with t >= tl and T1 >= T1l can matter to some weight sample: for
    // alpha G >= 1 - alpha the value (alpha G - (1 - alpha)) t + (1 - alpha) T1 grows with both, for
    // the others it needs t itself.
    [[maybe_unused]] auto sample_alive = [&](double tl, double T1l) -> bool {
      bool may = !(lbs > 0.0);
      for (int q = 0; q < a.n_alpha; ++q) {
        const double2 ab = s_ab[wave][q];
        const double v = lds_load(&s_aent[wave][q].val);
        may = may | (ab.x < ab.y) | (__builtin_fma(ab.x - ab.y, tl, ab.y * T1l) * lbs <= v);
      }
      return may;
    };

    // One strip: its unit's constants, weight and gradient ratios, and the levels they fix.
    struct Strip {
      OoIn I;
      double HW, A, KA, A2, C, gs, gf;
      int s;
      bool zero;  // weight and gradient ratios 0
    };
    auto load_strip = [&](const UnitRec& U, int rem2) -> Strip {
      const int iw = rem2 / R;
      const int ig = rem2 - iw * R;
      const double rw = s_ratio[iw], qw = s_ratio[R + iw], rg = s_ratio[ig], qg = s_ratio[R + ig];
      const int z = U.unit & 3;
      const double sw = z == 3 ? U.iD : 1.0, sg = z >= 2 ? U.iD : 1.0;
      const double Sw = U.Pw * sw, Sg = U.Pw * sg;
      Strip T;
      T.I.So = U.So;
      T.I.Swg = __builtin_fma(qg, Sg, qw * Sw);
      T.I.Obo = U.Obo;
      T.I.Og = rg * (U.Wb2 * sg);
      T.I.DG = rg * Sg;
      T.I.DW = rw * Sw;
      T.I.Wbuf = U.Wb2 * (1.0 - qw * sw);
      T.I.Gbuf = U.Wb2 * (1.0 - qg * sg);
      T.I.Rc = U.ckpt ? 0.5 * U.A2 : 0.0;  // one layer's activations: 2A / 2, exactly
      T.I.Xd = U.Xd;
      T.HW = rw * (2.0 * Sw);
      T.A = U.A;
      T.KA = U.KA;
      T.A2 = U.A2;
      T.C = U.C;
      T.gs = U.gs;
      T.gf = U.gf;
      T.s = U.unit * R2 + rem2;
      T.zero = r0_zero && rw == 0.0 && rg == 0.0;
      return T;
    };
    // A column's configurations: one optimizer ratio after the other, the lanes' columns side by side
    // (strip T, activation ratio ia, host streams hs and ds, stash SO, stable time tv of each lane).  A
    // lane takes part for the buckets (col) or the weight samples (acol).
    auto configs = [&](const Strip& T, bool col, bool acol, int ia, double hs, double ds, double SO, double tv, int fst) {
      const double C = T.C, gf = T.gf;
      const double T1c = __builtin_fmax(C, gf);
      const double Hx0 = __builtin_fma(ra0, T.I.So, T.I.DG) * iP, Dx0 = __builtin_fma(ra0, T.I.So, T.I.DW) * iP;
      const KnownRow fr = known_row(tab, gf > 0.0 ? 15 : 13, C, gf);
      const unsigned int lid_strip = (unsigned int)T.s * (unsigned int)R2;
      // Weight samples: the column's first-microbatch time at the smallest optimizer ratio, with the
      // slope by which it grows at least (first_times), and the limit of d.
      [[maybe_unused]] double T10 = 0.0, sl = 0.0, dl = 0.0;
      if constexpr (AL) {
        first_times(fr, C, gf, ia, hs + Hx0, ds + Dx0, !(col | acol), T10, sl);
        dl = d_limit(tv);
      }
#pragma unroll 1
      for (int io = 0; io < R; ++io) {
        const OoK O = oo_level(T.I, rr[io], om[io], iP);
        const double hf = hs + O.H2Dx, df = ds + O.D2Hx;
        const double mem = O.Bmax + SO;
        // Bucket j = min{j : mem <= E_j}: floor(mem * kNB) is j or j - 1 (kNB carries a
        // 2^-40 margin), so one comparison with E settles it.  An infeasible
        // configuration (Eq. 4: mem > M = E_{NB-1}) has floor(mem * kNB) >= NB - 1 and
        // lands on a sink: past NB - 1 the edges are +inf.  j0 = j - 1 needs mem within a
        // relative 2^-40 above an edge, or an infeasible mem just above M: rare, so only
        // entry j0's edge and key are read, and entry j0 + 1 (<= 64: entry 64's edge is
        // +inf) only by lanes whose mem exceeds E_j0.
        const int j0 = (int)__builtin_fmin(mem * kNB, 64.0);
        const unsigned int off0 = __umul24((unsigned int)j0, (unsigned int)sizeof(BucketEntry));
        char* const b0 = reinterpret_cast<char*>(bucket) + off0;
        wave_sync();  // read the entry after every earlier update of the wave
        const double e0 = reinterpret_cast<const BucketEntry*>(b0)->edge;
        const unsigned long long k_lo = lds_load(&reinterpret_cast<const BucketEntry*>(b0)->key);
        const bool up = mem > e0;
        // The configuration's own bound against its bucket (a lane in entry j0 + 1 is kept).
        bool may = col;
        double T1b = __builtin_fmax(T1c, __builtin_fmax(hf, df));
        if constexpr (AL) T1b = __builtin_fmax(T1b, __builtin_fma(sl, O.H2Dx - Hx0, T10));
        const double lb = __builtin_fma(Gm1, tv, T1b);
        [[maybe_unused]] bool amay = false;
        if constexpr (EX) {
          const double pm = *reinterpret_cast<const double*>(
              reinterpret_cast<const char*>(s_filt[wave]) + __umul24((unsigned int)min(j0, 63), (unsigned int)sizeof(FiltEntry)));
          may = may & (mem <= M) & (lb * lbs < pm);
        } else if constexpr (BK) {
          may = may & ((lb * lbs <= __longlong_as_double((long long)k_lo)) | up);
          if constexpr (AL) {
            amay = acol & (mem <= M) & (__builtin_fma(T1b, lbs, -tv) <= dl);
            may = may | amay;
          }
        }
        if (!__builtin_amdgcn_ballot_w64(may)) continue;
        [[maybe_unused]] int f1 = 0;
        const bool zero = (ia == 0) & (io == 0) & T.zero;
        double T1 = interference_known(fr, hf, df, !may | zero, tab, RK, f1);
        if (io == 0 && r0_zero) {  // a strip's all-zero configuration: no host streams
          const double T1z = interference_zero(C, gf, tab);
          T1 = zero ? T1z : T1;
        }
        const double d = T1 - tv;
        const double obj = __builtin_fma(Gd, tv, d);
        const unsigned int lid = lid_strip + (unsigned int)(io * R + ia);
        if constexpr (DM) {
          if (col) {
            double* o = a.dump + kDumpWords * (a.dump_off[x] + (int64_t)(T.s - tile.strip_begin) * R2 + io * R + ia);
            o[0] = tv;
            o[1] = d;
            o[2] = mem;
            o[3] = obj;
            o[4] = (double)(j0 + (up ? 1 : 0));
            o[5] = (double)((zero ? kFormZero : f1) + 8 * fst);
          }
          continue;
        }
        if constexpr (EX) {
          // Exact frontier candidates: feasible, below every lower bucket's minimum, and not
          // dominated by the bucket's winner (no more memory and no smaller objective, not
          // both equal).  Every frontier point passes; the scan after the sort decides.
          const int j = min(j0 + (up ? 1 : 0), 63);
          const FiltEntry f = s_filt[wave][j];
          const bool cand = may & (obj < f.pm) &
                            !(((obj > f.bobj) & (mem >= f.bmem)) | ((obj >= f.bobj) & (mem > f.bmem)));
          const unsigned long long m = __builtin_amdgcn_ballot_w64(cand);
          if (!m) continue;
          int64_t slot = 0;
          if (cand) {
            const unsigned int below = __builtin_amdgcn_mbcnt_hi(
                (unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
            slot = n_cand + below;
            if (slot < n_end) {
              a.cand_key[slot] = (unsigned long long)__double_as_longlong(mem);
              a.cand_obj[slot] = obj;
              a.cand_id[slot] = g.base + (uint64_t)lid;
            }
          }
          // Past the window: the overflow pool, in chunks of kPoolChunk slots per wave (one
          // device-wide atomic per chunk), else counted only and the tile is evaluated again.
          const bool over = cand && slot >= n_end;
          const unsigned long long mo = __builtin_amdgcn_ballot_w64(over);
          if (mo && a.pool_count) {
            const int k = __builtin_popcountll(mo);
            if (pool_used + k > kPoolChunk) {
              pool_holes(a, pool_base, pool_used, lane);
              const int leader = __builtin_ctzll(mo);
              unsigned long long b = 0;
              if (lane == leader) b = atomicAdd(a.pool_count, (unsigned long long)kPoolChunk);
              const unsigned long long bb = __shfl(b, leader, 64);
              pool_base = ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned int)(bb >> 32)) << 32) |
                          (unsigned long long)__builtin_amdgcn_readfirstlane((unsigned int)bb);
              pool_used = 0;
            }
            if (over) {
              const unsigned long long pos = pool_base + (unsigned long long)pool_used + __builtin_amdgcn_mbcnt_hi(
                  (unsigned int)(mo >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)mo, 0u));
              if (pos < (unsigned long long)a.pool_cap) {
                a.pool_key[pos] = (unsigned long long)__double_as_longlong(mem);
                a.pool_obj[pos] = obj;
                a.pool_id[pos] = g.base + (uint64_t)lid;
                a.pool_tile[pos] = t;
                a.pool_rank[pos] = (int32_t)(slot - n_beg);
              } else {
                dropped = true;
              }
            }
            pool_used += k;
          } else if (mo) {
            dropped = dropped | over;
          }
          n_cand += __builtin_popcountll(m);
          continue;
        }

        // Lexicographic (obj, id) minimum per bucket without a serial loop: the lanes
        // that beat their bucket's entry lower the objective bits with an LDS atomic
        // minimum; a lane that sees its bucket's objective drop clears the id, then the
        // lanes whose objective equals the new minimum lower the id.  The LDS operations
        // of a wave execute in program order and each step addresses the same words as
        // the one before, so each step sees the previous one's result.
        const unsigned long long key = (unsigned long long)__double_as_longlong(obj);
        if (__builtin_amdgcn_ballot_w64(may & ((key <= k_lo) | up))) {
          BucketEntry* const be = reinterpret_cast<BucketEntry*>(b0 + (up ? sizeof(BucketEntry) : 0));
          const unsigned long long k_old = up ? lds_load(&be->key) : k_lo;
          const unsigned int i_old = lds_load(&be->lid);
          const bool cand = may & ((key < k_old) | ((key == k_old) & (lid < i_old)));
          changed = changed | (__builtin_amdgcn_ballot_w64(cand) != 0ull);
          if (cand) atomicMin(&be->key, key);
          const unsigned long long k_new = cand ? lds_load(&be->key) : 0ull;
          if (cand && k_new < k_old) lds_store(&be->lid, 0xFFFFFFFFu);
          if (cand && key == k_new) atomicMin(&be->lid, lid);
        }
        if constexpr (AL) {
          // Eq. 4 for every weight sample, feasible configurations only: the samples some lane
          // may win, each with the same three-step sequence on its single entry (the value's
          // order key: weighted values may be negative).
          amay = amay & (d <= dl);
          if (__builtin_amdgcn_ballot_w64(amay)) {
#pragma unroll 1
            for (int q = 0; q < a.n_alpha; ++q) {
              const double2 ab = s_ab[wave][q];
              AlphaEntry* const e = &s_aent[wave][q];
              const double v = __builtin_fma(ab.x, tv, ab.y * d);
              const double cur = lds_load(&e->val);
              if (!__builtin_amdgcn_ballot_w64(amay & (v <= cur))) continue;
              const unsigned long long ak = order_key(v);
              const unsigned long long ak_old = lds_load(&e->key);
              const unsigned int ai_old = lds_load(&e->lid);
              const bool cand = amay & ((ak < ak_old) | ((ak == ak_old) & (lid < ai_old)));
              changed = changed | (__builtin_amdgcn_ballot_w64(cand) != 0ull);
              if (cand) atomicMin(&e->key, ak);
              const unsigned long long ak_new = cand ? lds_load(&e->key) : 0ull;
              if (cand && ak_new < ak_old) lds_store(&e->lid, 0xFFFFFFFFu);
              if (cand && ak == ak_new) {
                atomicMin(&e->lid, lid);
                lds_store(&e->val, v);
              }
              wave_sync();
            }
          }
        }
      }
    };
    // Queued columns, 64 at a time, a lane each: few lanes of a strip iteration reach this point (3 of 64
    // on llama42b-d128-hw64), and side by side they share the optimizer level and the rounds.
    int qn = 0;
    auto flush = [&](int n) {
      wave_sync();
      const bool on = lane < n;
      const uint32_t it = on ? s_qi[wave][qn - n + lane] : 0u;
      const double tv = on ? s_qt[wave][qn - n + lane] : 0.0;
      const int ia = (int)(it >> 13 & 15u);
      const Strip T = load_strip(units[it & 31u], (int)(it >> 5 & 255u));
      const double ra = s_ratio[ia], qa = s_ratio[R + ia];
      const double hs = __builtin_fma(ra, T.A, T.HW) * iP, ds = __builtin_fma(ra, T.A, T.I.DG) * iP;
      configs(T, on & ((it >> 17 & 1u) != 0u), on & ((it >> 18 & 1u) != 0u), ia, hs, ds,
              __builtin_fma(ra, T.A2, qa * T.KA), tv, DM ? (int)(it >> 19 & 7u) : 0);
      qn -= n;
      if (BK && changed) refresh();
    };

    const int nu = g.n_pairs * (l + 1) * 4;  // units of the group
    // The tile's units in chunks, one lane each.  A chunk takes one unit of each of kChunk equal
    // segments, so that the first ones sample the whole tile and the thresholds settle early; the
    // place within the segment turns with the lane, which mixes the ZeRO levels.  The first kUnits
    // live ones are visited, then the others' bounds are taken again (the exact frontier's thresholds
    // are final and few of its units live: it takes 64 at a time; with the buckets' a chunk of 64 tests
    // too many units against early thresholds: 0.96 against 0.90 ms on llama7b-d32).  The seed variant
    // samples one chunk over the whole group.
    const int u_beg = tile.strip_begin / R2;
    const int n_u = SD ? nu : (tile.strip_end > tile.strip_begin ? (tile.strip_end - 1) / R2 + 1 - u_beg : 0);
    constexpr int kChunk = EX ? 64 : kUnits;
    const int n_chunks = (n_u + kChunk - 1) / kChunk;
    for (int k = 0; k < (SD ? 1 : n_chunks); ++k) {
      const int at = (k + lane) % n_chunks + n_chunks * lane;
      const int u = u_beg + at;
      bool pending = lane < kChunk && at < n_u;
      bool again = k > 0;
      while (__builtin_amdgcn_ballot_w64(pending)) {
      if constexpr (BK) exchange(again);
      again = true;
      bool live = pending;
      UnitRec rec{};
      if (live) {
        const int uc = u >> 2, z = u & 3;
        const int p = uc / (l + 1);
        const int c = uc - p * (l + 1);
        const PairK P = pk[g.pk_begin + p];
        const CkptK K = ckpt_level(P, l, c, ke);
        const ZeroK Z = zero_level(P, z);
        rec = UnitRec{P.Pw, P.iD, P.Wb2, Z.So, Z.Obo, P.Xd, K.A, K.KA, P.A2, K.C, Z.G2Gs, Z.G2Gf, u, c > 0 ? 1 : 0};
        if constexpr (!DM && !SD) {
          // End values of each ratio's terms: weights (both peaks), gradients and optimizer states
          // (forward peak, backward peak), activations.
          const double w0 = qa0 * Z.Sw + P.Wb2 * (1.0 - qa0 * Z.sw), w1 = qa1 * Z.Sw + P.Wb2 * (1.0 - qa1 * Z.sw);
          const double gf0 = qa0 * Z.Sg + ra0 * Z.Obg, gf1 = qa1 * Z.Sg + ra1 * Z.Obg;
          const double gb0 = qa0 * Z.Sg + P.Wb2 * (1.0 - qa0 * Z.sg), gb1 = qa1 * Z.Sg + P.Wb2 * (1.0 - qa1 * Z.sg);
          const double of0 = qa0 * Z.So + ra0 * Z.Obo, of1 = qa1 * Z.So + ra1 * Z.Obo;
          const double ob0 = qa0 * Z.So, ob1 = qa1 * Z.So;
          const double s0 = ra0 * P.A2 + qa0 * K.KA, s1 = ra1 * P.A2 + qa1 * K.KA;
          const double wl = __builtin_fmin(w0, w1), wh = __builtin_fmax(w0, w1);
          const double lo = __builtin_fmax(wl + __builtin_fmin(gf0, gf1) + __builtin_fmin(of0, of1),
                                           wl + __builtin_fmin(gb0, gb1) + ob1 + K.Rc) + P.Xd + __builtin_fmin(s0, s1);
          const double hi = __builtin_fmax(wh + __builtin_fmax(gf0, gf1) + __builtin_fmax(of0, of1),
                                           wh + __builtin_fmax(gb0, gb1) + ob0 + K.Rc) + P.Xd + __builtin_fmax(s0, s1);
          const double hl = ra0 * (K.A + 2.0 * Z.Sw) * iP, dl = ra0 * (K.A + Z.Sg) * iP;
          const double tl = __builtin_fmax(__builtin_fmax(K.C, Z.G2Gs), __builtin_fmax(hl, dl));
          const double T1l = __builtin_fmax(__builtin_fmax(K.C, Z.G2Gf),
                                            __builtin_fmax(hl + ra0 * (Z.So + Z.Sg) * iP, dl + ra0 * (Z.So + Z.Sw) * iP));
          live = alive(lo, __builtin_fma(Gm1, tl, T1l), limit(lo, hi));
          if constexpr (AL) live = live | ((lo <= Mhi) & sample_alive(tl, T1l));
        }
      }
      const unsigned long long lm = __builtin_amdgcn_ballot_w64(live);
      const int rank = (int)__builtin_amdgcn_mbcnt_hi((unsigned int)(lm >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)lm, 0u));
      const int n_live = min(__builtin_popcountll(lm), kUnits);
      any_live = any_live | (n_live > 0);
      pending = live & (rank >= kUnits);
      wave_sync();  // the previous units' records are done with
      if (live & (rank < kUnits)) units[rank] = rec;
      wave_sync();

      // Strips of the live units, one lane each, 64 at a time, and whenever the queue holds 64 columns
      // (or at the end some) those: the strips' values are not kept across that but formed again, so
      // that neither part holds the other's registers.
      const int n_strips = SD ? 64 * kSeedIters : n_live * R2;
      int i0 = 0, ca = 0;  // strips done, columns done of the next ones
      while (i0 < n_strips || qn > 0) {
        if (QU && (qn >= 64 || i0 >= n_strips)) {
          flush(min(qn, 64));
          continue;
        }
        if (BK && changed) refresh();
        const int i = i0 + lane;
        int slot, rem2;
        bool on;
        if constexpr (SD) {  // two lanes per unit
          slot = lane >> 1;
          on = slot < n_live;
          rem2 = (lane & 1) ? (int)((unsigned int)(lane * 37 + (i0 >> 6) * 29) % (unsigned int)R2) : (i0 >> 6) % R2;
        } else {
          slot = i / R2;
          rem2 = i - slot * R2;
          on = i < n_strips;
        }
        slot = on ? slot : 0;
        const Strip T = load_strip(units[slot], rem2);
        if constexpr (!SD) on = on & (T.s >= tile.strip_begin) & (T.s < tile.strip_end);
        const double A = T.A, KA = T.KA, A2 = T.A2, C = T.C, gs = T.gs, gf = T.gf, HW = T.HW, DG = T.I.DG;
        // Peak without the activation terms over the optimizer ratios: between Blo and Bhi.
        double Blo, Bhi;
        {
          const OoIn& I = T.I;
          const double b0 = __builtin_fma(qa0, I.So, I.Swg) + I.Wbuf, b1 = __builtin_fma(qa1, I.So, I.Swg) + I.Wbuf;
          const double f0 = b0 + __builtin_fma(ra0, I.Obo, I.Og), f1 = b1 + __builtin_fma(ra1, I.Obo, I.Og);
          const double g0 = (b0 + I.Gbuf) + I.Rc, g1 = (b1 + I.Gbuf) + I.Rc;
          Blo = __builtin_fmax(__builtin_fmin(f0, f1), g1) + I.Xd;
          Bhi = __builtin_fmax(__builtin_fmax(f0, f1), g0) + I.Xd;
        }
        const double Hx0 = __builtin_fma(ra0, T.I.So, DG) * iP, Dx0 = __builtin_fma(ra0, T.I.So, T.I.DW) * iP;
        const double tc = __builtin_fmax(C, gs), T1c = __builtin_fmax(C, gf);
        // With a positive activation ratio both host streams run, so the stable microbatch's first
        // round has the pattern compute, both host streams, and GPU-GPU when it carries traffic; the
        // first microbatch's configurations with a non-zero offload ratio start likewise.
        const KnownRow sr = known_row(tab, gs > 0.0 ? 15 : 13, C, gs);
        // Weight samples: whether the strip may matter to one, the largest d with which it may, and
        // whether it may matter to a bucket (few strips do: the others' columns skip that test).
        [[maybe_unused]] bool smp = false, bkt = true;
        [[maybe_unused]] double dls = 0.0;
        if constexpr (AL) {
          const double hl = __builtin_fma(ra0, A, HW) * iP, dl = __builtin_fma(ra0, A, DG) * iP;
          const double tl = __builtin_fmax(tc, __builtin_fmax(hl, dl));
          const double T1l = __builtin_fmax(T1c, __builtin_fmax(hl + Hx0, dl + Dx0));
          const double s0 = __builtin_fma(ra0, A2, qa0 * KA), s1 = __builtin_fma(ra1, A2, qa1 * KA);
          const double lo = Blo + __builtin_fmin(s0, s1), hi = Bhi + __builtin_fmax(s0, s1);
          on = on & (lo <= Mhi);
          smp = sample_alive(tl, T1l);
          bkt = __builtin_amdgcn_ballot_w64(on & alive(lo, __builtin_fma(Gm1, tl, T1l), limit(lo, hi))) != 0ull;
          if (!bkt & !__builtin_amdgcn_ballot_w64(on & smp)) {  // nothing in these strips
            ca = 0;
            i0 += 64;
            continue;
          }
          dls = d_limit(tl * lbs);
        }

#pragma unroll 1
        for (; ca < R && qn < 64; ++ca) {
          const int ia = ca;
          const double ra = rr[ia], qa = om[ia];
          const double hs = __builtin_fma(ra, A, HW) * iP;
          const double ds = __builtin_fma(ra, A, DG) * iP;
          const double SO = __builtin_fma(ra, A2, qa * KA);  // stash + offload buffers
          const double T1l = __builtin_fmax(T1c, __builtin_fmax(hs + Hx0, ds + Dx0));
          bool col = false;  // matters to a bucket (or the exact frontier)
          double th = 0.0;
          if (!AL || bkt) {
            th = limit(Blo + SO, Bhi + SO);
            col = on & alive(Blo + SO, __builtin_fma(Gm1, __builtin_fmax(tc, __builtin_fmax(hs, ds)), T1l), th);
          }
          [[maybe_unused]] bool acol = false;  // matters to a weight sample
          if constexpr (AL) acol = on & (Blo + SO <= Mhi) & smp;
          if (!__builtin_amdgcn_ballot_w64(col | acol)) continue;
          // The stable time does not depend on the optimizer ratio.
          double tv;
          [[maybe_unused]] int fst = kFormGeneric;
          if (ia == 0 && r0_zero)
            tv = interference(C, gs, hs, ds, tab);
          else
            tv = interference_known(sr, hs, ds, !(col | acol), tab, RK, fst);
          col = col & alive(Blo + SO, __builtin_fma(Gm1, tv, T1l), th);
          if constexpr (AL) acol = acol & (__builtin_fma(T1l, lbs, -tv) <= dls);
          if (!__builtin_amdgcn_ballot_w64(col | acol)) continue;
          // Weight samples: the first-microbatch time at the smallest optimizer ratio bounds the column's.
          // (For the buckets alone it excludes too little for its cost: 6.4 against 5.7 ms on
          // llama42b-d128-hw64.)
          if constexpr (AL) {
            const KnownRow fr = known_row(tab, gf > 0.0 ? 15 : 13, C, gf);
            double T10, sl;
            const double h0 = hs + Hx0, d0 = ds + Dx0;
            first_times(fr, C, gf, ia, h0, d0, !(col | acol), T10, sl);
            const double T1m = __builtin_fmax(T1l, any_length(T10, sl, __builtin_fmax(h0, d0)));
            col = col & alive(Blo + SO, __builtin_fma(Gm1, tv, T1m), th);
            acol = acol & (__builtin_fma(T1m, lbs, -tv) <= dls);
            if (!__builtin_amdgcn_ballot_w64(col | acol)) continue;
            acol = acol & (__builtin_fma(T1m, lbs, -tv) <= d_limit(tv));
          }
          const unsigned long long m = __builtin_amdgcn_ballot_w64(col | acol);
          if (!m) continue;
          if constexpr (QU) {
            if (col | acol) {
              const int pos = qn + (int)__builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
              s_qt[wave][pos] = tv;
              s_qi[wave][pos] = (uint32_t)slot | (uint32_t)rem2 << 5 | (uint32_t)ia << 13 | (col ? 1u << 17 : 0u) | (acol ? 1u << 18 : 0u) |
                                 (DM ? (uint32_t)fst << 19 : 0u);
            }
            qn += __builtin_popcountll(m);
          } else {
            configs(T, col, acol, ia, hs, ds, SO, tv, fst);
          }
        }
        if (ca == R) {
          ca = 0;
          i0 += 64;
        }
      }
      }
    }
    if constexpr (SD) {
      // The group's first thresholds: objectives of configurations of each bucket.
      wave_sync();
      thr[lane] = lds_load(&bucket[lane].key);
      if constexpr (AL)
        if (lane < a.n_alpha) athr[lane] = lds_load(&s_aent[wave][lane].key);
    } else if constexpr (EX) {
      // Saturated at 2^31 - 1, which the host rejects (no tile of a space with fewer than
      // 2^32 candidates reaches it).
      if (lane == 0) a.tile_live[t] = any_live ? 1 : 0;
      if (lane == 0) a.cnt_tile[t] = (int32_t)min(n_cand - n_beg, (int64_t)0x7FFFFFFF);
      const unsigned long long md = __builtin_amdgcn_ballot_w64(dropped);
      if (lane == 0 && a.tile_drop) a.tile_drop[t] = md ? 1 : 0;
    } else if constexpr (!DM) {
      // The tile's partials: lane j = bucket j.  A bucket that no configuration of this tile
      // reached carries the threshold it did not beat (the tile's configurations of that bucket, if
      // any, have larger objectives) and no id.
      wave_sync();
      const unsigned long long key = lds_load(&bucket[lane].key);
      const unsigned int bl = lds_load(&bucket[lane].lid);
      if (thr && lane < NB && bl != 0xFFFFFFFFu)
        __hip_atomic_fetch_min(thr + lane, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      a.part_obj[(size_t)t * 64 + lane] = __longlong_as_double((long long)key);
      a.part_id[(size_t)t * 64 + lane] = bl == 0xFFFFFFFFu ? kNone : g.base + (uint64_t)bl;
      if constexpr (AL) {
        if (lane < a.n_alpha) {
          const unsigned long long ak = lds_load(&s_aent[wave][lane].key);
          const unsigned int al = lds_load(&s_aent[wave][lane].lid);
          if (athr && al != 0xFFFFFFFFu)
            __hip_atomic_fetch_min(athr + lane, ak, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          a.part_aobj[(size_t)t * a.n_alpha + lane] = order_value(ak);
          a.part_aid[(size_t)t * a.n_alpha + lane] = al == 0xFFFFFFFFu ? kNone : g.base + (uint64_t)al;
        }
      }
    }
    if (!claims) break;
    for (;;) {
      int c = 0;
      if (lane == 0) c = atomicAdd(a.work + counter * kCounterStride, 1);
      c = __builtin_amdgcn_readfirstlane(__shfl(c, 0, 64));
      const int64_t next = (int64_t)n_waves + counter + (int64_t)kClaimCounters * c;
      if (next < n_items) {
        x = (int)next;
        break;
      }
      if (++exhausted == kClaimCounters) {  // every counter has run out: no item is left
        x = n_items;
        break;
      }
      counter = counter + 1 == kClaimCounters ? 0 : counter + 1;
    }
  }
  if constexpr (EX) {
    if (a.pool_count) pool_holes(a, pool_base, pool_used, lane);
  }
}

int check_launch() {
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : (int)e;
}

#define MIST_FOR_EACH_R(X) \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

template <int R, int MODE>
void launch_rm(const EvalArgs& a, int blocks, hipStream_t st) {
  hipLaunchKernelGGL((k_search<R, MODE>), dim3(blocks), dim3(kBlock), 0, st, a, a.ratio, (const PairK*)a.pk);
}

template <int R>
void launch_r(const EvalArgs& a, int blocks, int mode, hipStream_t st) {
  switch (mode) {
    case kModeAlpha: launch_rm<R, kModeAlpha>(a, blocks, st); break;
    case kModeEmit: launch_rm<R, kModeEmit>(a, blocks, st); break;
    case kModeDump: launch_rm<R, kModeDump>(a, blocks, st); break;
    case kModeSeed: launch_rm<R, kModeSeed>(a, blocks, st); break;
    case kModeSeedAlpha: launch_rm<R, kModeSeedAlpha>(a, blocks, st); break;
    default: launch_rm<R, kModeBuckets>(a, blocks, st); break;
  }
}

template <int R, int MODE>
int blocks_per_cu_rm() {
  int n = 0;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_search<R, MODE>, kBlock, 0) == hipSuccess ? n : 1;
}

template <int R>
int blocks_per_cu_r(int mode) {
  switch (mode) {
    case kModeAlpha: return blocks_per_cu_rm<R, kModeAlpha>();
    case kModeEmit: return blocks_per_cu_rm<R, kModeEmit>();
    case kModeDump: return blocks_per_cu_rm<R, kModeDump>();
    default: return blocks_per_cu_rm<R, kModeBuckets>();
  }
}

}  // namespace

int search_blocks_per_cu(int R, int mode) {
  switch (R) {
#define MIST_CASE(n) \
  case n:            \
    return blocks_per_cu_r<n>(mode);
    MIST_FOR_EACH_R(MIST_CASE)
#undef MIST_CASE
    default:
      return 1;
  }
}

int launch_search(const EvalArgs& a, int blocks, int mode, void* stream) {
  if (mode < kModeBuckets || mode > kModeSeedAlpha) return (int)hipErrorInvalidValue;
  if (a.n_tiles <= 0) return 0;
  hipStream_t st = (hipStream_t)stream;
  switch (a.R) {
#define MIST_CASE(n)                  \
  case n:                             \
    launch_r<n>(a, blocks, mode, st); \
    break;
    MIST_FOR_EACH_R(MIST_CASE)
#undef MIST_CASE
    default:
      return (int)hipErrorInvalidValue;
  }
  return check_launch();
}

}  // namespace mist
