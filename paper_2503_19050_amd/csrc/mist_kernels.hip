// libmist kernels for gfx950: batched FP64 evaluation of Mist's per-stage cost model
// (Sec. 5.2-5.3, Eq. 4-6, Algorithm 1) over every configuration of a space, feasibility filter,
// per-bucket and per-group reductions.  Large spaces are searched with bounds instead
// (mist_search.hip).

#include "mist_device.h"

namespace mist {
namespace {

// Algorithm 1 for the first n of the N configurations of an activation-ratio block (host streams
// h[c], d[c]), one wave-uniform choice of form per configuration (measured fastest against one
// choice per block or half block: 0.81 against 1.16 and 1.02 ms on gpt2.7b-d16, equal on the
// Llama spaces).
template <int N>
__device__ __forceinline__ void interference_known_n(const KnownRow& r, const double (&h)[N], const double (&d)[N],
                                                     const bool (&free)[N], double (&out)[N], int (&form)[N], int n,
                                                     const double* __restrict__ tab, const RowK& K) {
#pragma unroll
  for (int c = 0; c < N; ++c) {
    if (c >= n) break;
    out[c] = interference_known(r, h[c], d[c], free[c], tab, K, form[c]);
  }
}

// K0: pair-level constants of every (group, pair).
__global__ __launch_bounds__(256) void k_pairs(EvalArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kClaimCounters) a.work[i * kCounterStride] = 0;  // the evaluation kernel's tile
                                                           // counters (it runs after this one)
  if (i == 0 && a.pool_count) *a.pool_count = 0ull;       // and its candidate overflow pool
  if (i >= a.n_pk) return;
  const DevGroup g = a.groups[a.pk_group[i]];
  const int p = i - g.pk_begin;
  a.pk[i] = pair_level(a.m, g.PP, g.k, g.l, a.pairs[g.pair_begin + p], a.hws[g.hw]);
}

// ---------------------------------------------------------------------------------------
// K1.  Persistent: every wave takes one tile (a range of strips of one group) by its index
// in the grid and claims further tiles from a device counter until none is left; each lane
// walks the tile's strips with stride 64.  A
// strip fixes (pair, c, z, wo, go) and holds the R x R (optimizer ratio, activation ratio)
// configurations:
//   - the stable time t does not depend on the optimizer ratio, so it is computed once per
//     activation ratio and reused across the optimizer ratios;
//   - the first microbatch's streams start in the same pattern for every configuration of
//     the strip (compute, GPU-GPU iff that stream carries traffic, and both host streams
//     iff any offload ratio is non-zero), except the one configuration whose four ratios
//     are all zero: its host streams are exactly +0, and its time is computed once per
//     strip in closed form (interference_zero).
// Each wave keeps an LDS table of the 64 bucket minima of its current tile and writes it
// as the tile's partials.
// ---------------------------------------------------------------------------------------
// Activation ratios per block of the strip loop: a block keeps its stable times and the
// per-ratio terms of its configurations in registers across the optimizer ratios.
// Weight samples take larger blocks for 7 <= R <= 10 (at R = 9, 79.5 against 85.2 ms for 8
// samples on the 64-hardware-sample Llama space).
template <int R, int MODE>
constexpr int ia_block() {
  return R <= 6 ? R : (MODE == kModeAlpha && R <= 10 ? (R + 1) / 2 : (R + 2) / 3);
}

// Waves per SIMD the register allocation aims at: four, 128 registers per lane (a few
// strip-level values spill; the occupancy is worth more).  Five would fit the LDS of the blocks,
// but at 96 registers the inner loop spills: 77 against 59 ms on the 64-sample Llama space.
constexpr int kEvalWaves = 4;

// MODE kModeBuckets: bucket minima; kModeAlpha: also the weight-sampled argmins of Eq. 4
// (a.n_alpha samples); kModeDump: per-configuration values of listed tiles.
template <int R, int MODE>
__global__ __launch_bounds__(kBlock, kEvalWaves) void k_eval(EvalArgs a, const double* __restrict__ ratio,
                                                                 const PairK* __restrict__ pk) {
  constexpr bool AL = MODE == kModeAlpha;
  constexpr bool DM = MODE == kModeDump;
  constexpr int R2 = R * R;
  constexpr int SU = 4 * R2;  // strips per (pair, c) unit
  constexpr int IB = ia_block<R, MODE>();
  __shared__ double s_tab[kWaves][16 * kLdsRow + 2 * kTab2];
  __shared__ BucketEntry s_bucket[kWaves][65];  // entries NB..64: sinks of infeasible configurations
  __shared__ OoIn s_oo[kBlock];         // per-lane strip constants of the optimizer level
  __shared__ double2 s_ab[AL ? kWaves : 1][kMaxAlphas];      // alpha * G, 1 - alpha
  __shared__ AlphaEntry s_aent[AL ? kWaves : 1][kMaxAlphas];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // The wave index is uniform across the wave: stated, so that the tile, group and hardware
  // values derived from it live in scalar registers (scalar loads) rather than in every lane.
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NB = a.NB;
  const double* __restrict__ rr = ratio;  // read-only and uniform: scalar loads
  const double* __restrict__ om = ratio + R;
  const bool r0_zero = rr[0] == 0.0;
  double* tab = s_tab[wave];
  BucketEntry* bucket = s_bucket[wave];
  const unsigned long long kEmpty = (unsigned long long)__double_as_longlong(__builtin_huge_val());

  // Tile schedule: wave w of the grid takes work item w.  Item n_waves + x + kClaimCounters
  // * c goes to the claim that draws number c from counter x (counters reset to 0 by K0); a
  // wave draws from the counter of its block's XCD and moves to the next counter when one
  // runs out, until all have.  When the grid has at least as many waves as there are items
  // no claim is made.  Item x is tile tile_order[x] (the host gives each XCD's items a
  // contiguous range of tiles), or tile tile_list[x] when a variant runs a list.
  const bool listed = DM && a.tile_list != nullptr;
  const int n_items = listed ? a.n_list : a.n_tiles;
  const int n_waves = (int)gridDim.x * kWaves;
  const bool claims = n_items > n_waves;
  int counter = (int)(blockIdx.x % kClaimCounters);
  int exhausted = 0;
  int loaded_hw = -1;
  for (int x = (int)blockIdx.x * kWaves + wave; x < n_items;) {
    const int t = listed ? load_uniform(a.tile_list + x) : (a.tile_order ? load_uniform(a.tile_order + x) : x);
    const DevTile tile = load_uniform(a.tiles + t);
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
    bucket[lane].key = lane < NB ? kEmpty : 0ull;
    bucket[lane].lid = lane < NB ? 0xFFFFFFFFu : 0u;
    if (lane == 0) {
      bucket[64].edge = __builtin_huge_val();
      bucket[64].key = 0ull;
      bucket[64].lid = 0u;
    }
    const double Gd = (double)g.G;
    if constexpr (AL) {
      if (lane < a.n_alpha) {
        s_ab[wave][lane] = make_double2(a.alpha[lane] * Gd, a.beta[lane]);
        s_aent[wave][lane].val = __builtin_huge_val();
        s_aent[wave][lane].key = order_key(__builtin_huge_val());
        s_aent[wave][lane].lid = 0xFFFFFFFFu;
      }
    }
    wave_sync();

    const double iP = load_uniform(&hw.iP), kNB = load_uniform(&hw.kNB), M = load_uniform(&hw.M);
    const RowK RK{load_uniform(&hw.itab[15][2]), load_uniform(&hw.itab[15][3]), load_uniform(&hw.itab[15][6]),
                  load_uniform(&hw.itab[15][7]), load_uniform(&hw.itab[13][2]), load_uniform(&hw.itab[13][3])};
    const int l = g.l;
    const int64_t ke = g.k < g.G ? g.k : g.G;

#pragma unroll 1
    for (int s = tile.strip_begin + lane; s < tile.strip_end; s += 64) {
      const int unit = s / SU;
      const int rem = s - unit * SU;
      const int z = rem / R2;
      const int rem2 = rem - z * R2;
      const int iw = rem2 / R;
      const int ig = rem2 - iw * R;
      const int p = unit / (l + 1);
      const int c = unit - p * (l + 1);
      const PairK P = pk[g.pk_begin + p];
      const CkptK K = ckpt_level(P, l, c, ke);
      const ZeroK Z = zero_level(P, z);
      const double rw = rr[iw], rg = rr[ig];
      const WoGoK W = wogo_levels(P, Z, rw, om[iw], rg, om[ig]);
      // First microbatch: every configuration of the strip with a non-zero offload ratio
      // starts with compute, both host streams and (if it carries traffic) GPU-GPU.
      const int pat1 = Z.G2Gf > 0.0 ? 15 : 13;
      const KnownRow fr = known_row(tab, pat1, K.C, Z.G2Gf);
      const bool zero_strip = r0_zero && rw == 0.0 && rg == 0.0;
      // First-microbatch time of the strip's all-zero configuration (no host streams).
      const double T1z = interference_zero(K.C, Z.G2Gf, tab);
      s_oo[tid] = oo_inputs(P, K, Z, W);
      const double A = K.A, KA = K.KA, A2 = P.A2, HW = W.HW, DG = W.DG;
      const unsigned int lid_strip = (unsigned int)s * (unsigned int)R2;
      // With a positive activation ratio both host streams run, so the stable microbatch's
      // first round has the pattern compute + both host streams (+ GPU-GPU when it carries
      // traffic).
      const int pats = Z.G2Gs > 0.0 ? 15 : 13;

      // Activation ratios in blocks of IB: the values a block keeps across the optimizer
      // ratios fit the registers, at the price of one more optimizer-level evaluation per
      // block.  A block's stable times, and per optimizer ratio its first-microbatch times, are
      // formed before its memory, objective and reduction steps, so that the interference rounds
      // of its configurations are straight-line code.
#pragma unroll
      for (int ib = 0; ib < R; ib += IB) {
        // Stable time per activation ratio (it does not depend on the optimizer ratio).
        const int nb = R - ib < IB ? R - ib : IB;  // configurations of the block
        const KnownRow sr = known_row(tab, pats, K.C, Z.G2Gs);
        double tt[IB];
        [[maybe_unused]] int fst[IB];  // dump variant: the form of each stable time
        {
          double hs[IB], ds[IB];
          bool fs[IB];
#pragma unroll
          for (int c = 0; c < IB; ++c) {
            const int ia = ib + c;
            if (ia >= R) break;
            hs[c] = __builtin_fma(rr[ia], K.A, W.HW) * iP;
            ds[c] = __builtin_fma(rr[ia], K.A, W.DG) * iP;
            fs[c] = ia == 0 && r0_zero;
          }
          interference_known_n<IB>(sr, hs, ds, fs, tt, fst, nb, tab, RK);
          // Activation ratio 0 leaves the host streams to the weights and gradients alone: the
          // first round's pattern is not known in advance.
          if (ib == 0 && r0_zero) {
            tt[0] = interference(K.C, Z.G2Gs, hs[0], ds[0], tab);
            fst[0] = kFormGeneric;
          }
        }
        // Weight samples: the block's smallest stable time, for the lower bound below.
        [[maybe_unused]] double t_min = tt[0];
        if constexpr (AL) {
#pragma unroll
          for (int c = 1; c < IB; ++c)
            if (ib + c < R) t_min = __builtin_fmin(t_min, tt[c]);
        }

#pragma unroll 1
        for (int io = 0; io < R; ++io) {
          const OoK O = oo_level(s_oo[tid], rr[io], om[io], iP);
          const bool zero_oo = zero_strip && io == 0;
          const unsigned int lid_oo = lid_strip + (unsigned int)(io * R);
          [[maybe_unused]] double dn_blk[AL ? IB : 1];  // weight samples: the block's deltas (NaN
                                                        // when infeasible)
          double T1b[IB];
          [[maybe_unused]] int f1b[IB];  // dump variant: the form of each first-microbatch time
          {
            double hf[IB], df[IB];
            bool fz[IB];
#pragma unroll
            for (int c = 0; c < IB; ++c) {
              const int ia = ib + c;
              if (ia >= R) break;
              hf[c] = __builtin_fma(rr[ia], A, HW) * iP + O.H2Dx;
              df[c] = __builtin_fma(rr[ia], A, DG) * iP + O.D2Hx;
              fz[c] = ia == 0 && zero_oo;
            }
            interference_known_n<IB>(fr, hf, df, fz, T1b, f1b, nb, tab, RK);
          }
#pragma unroll
          for (int c = 0; c < IB; ++c) {
            const int ia = ib + c;
            if (ia >= R) break;
            const double ra = rr[ia];
            const double SO = __builtin_fma(ra, A2, om[ia] * KA);  // stash + offload buffers
            const double mem = O.Bmax + SO;
            double T1 = T1b[c];
            if (ia == 0) T1 = zero_oo ? T1z : T1;
            const double tv = tt[c];
            const double d = T1 - tv;
            const double obj = __builtin_fma(Gd, tv, d);

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
            const unsigned long long k_lo = reinterpret_cast<const BucketEntry*>(b0)->key;
            if constexpr (DM) {
              double* o = a.dump + kDumpWords * (a.dump_off[x] + (int64_t)(s - tile.strip_begin) * R2 + io * R + ia);
              o[0] = tv;
              o[1] = d;
              o[2] = mem;
              o[3] = obj;
              o[4] = (double)(j0 + (mem > e0 ? 1 : 0));
              o[5] = (double)((ia == 0 && zero_oo ? kFormZero : f1b[c]) + 8 * fst[c]);
              continue;
            }
            const bool up = mem > e0;

            // Lexicographic (obj, id) minimum per bucket without a serial loop: the lanes
            // that beat their bucket's entry lower the objective bits with an LDS atomic
            // minimum; a lane that sees its bucket's objective drop clears the id, then the
            // lanes whose objective equals the new minimum lower the id.  The LDS operations
            // of a wave execute in program order and each step addresses the same words as
            // the one before, so each step sees the previous one's result.
            const unsigned long long key = (unsigned long long)__double_as_longlong(obj);
            // A candidate beats the entry: key < k_old, or an equal key with a lower id.  No
            // lane with key > k_old is one, so the exact test waits for a lane with key <= k_old
            // or a lane in entry j0 + 1 (combined as wave masks by the scalar ALU).
            const unsigned long long m_up = __builtin_amdgcn_ballot_w64(up);
            const unsigned long long m_lo = __builtin_amdgcn_ballot_w64(key <= k_lo);
            if (m_lo | m_up) {
              BucketEntry* const be = reinterpret_cast<BucketEntry*>(b0 + (up ? sizeof(BucketEntry) : 0));
              const unsigned long long k_old = up ? lds_load(&be->key) : k_lo;
              const unsigned int lid = lid_oo + (unsigned int)ia;
              const unsigned int i_old = lds_load(&be->lid);
              const bool cand = (key < k_old) | ((key == k_old) & (lid < i_old));
              if (cand) atomicMin(&be->key, key);
              const unsigned long long k_new = cand ? lds_load(&be->key) : 0ull;
              if (cand && k_new < k_old) lds_store(&be->lid, 0xFFFFFFFFu);
              if (cand && key == k_new) atomicMin(&be->lid, lid);
            }

            if constexpr (AL) dn_blk[c] = mem <= M ? d : __builtin_nan("");
          }

          if constexpr (AL) {
            // Eq. 4 for every weight sample, feasible configurations only: an infeasible one
            // carries a NaN delta, so each of its weighted values is NaN and compares false.
            // First the block's configurations against every sample's entry as it stands (no
            // lane can beat an entry it does not beat now: entries only decrease), each
            // sample's values read once for the block; the exact sequence only when some lane
            // of the wave may win.  All lanes address the sample's single entry; the same
            // three-step LDS sequence as the buckets' keeps the lexicographic minimum.
            //
            // Before that, one bound per sample and block: with a = alpha*G >= 0 and
            // b = 1 - alpha >= 0, fma(a, t, b*d) is non-decreasing in t and d under rounding to
            // nearest, so fma(a, t_min, b*d_min) over the block's smallest t and smallest
            // feasible d is at most every feasible configuration's value.  A sample whose bound
            // exceeds its entry on every lane cannot be won by the block, and its per-
            // configuration values are not formed (NaN deltas drop out of the minimum; a block
            // without a feasible configuration has a NaN bound, which compares false).
            wave_sync();
            double d_min = dn_blk[0];
#pragma unroll
            for (int c = 1; c < IB; ++c)
              if (ib + c < R) d_min = __builtin_fmin(d_min, dn_blk[c]);
            unsigned int qmask = 0;  // samples some lane of the wave may win
#pragma unroll 1
            for (int q = 0; q < a.n_alpha; ++q) {
              const double2 ab = s_ab[wave][q];
              const double cur = lds_load(&s_aent[wave][q].val);
              if (!__builtin_amdgcn_ballot_w64(__builtin_fma(ab.x, t_min, ab.y * d_min) <= cur)) continue;
              bool any = false;
#pragma unroll
              for (int c = 0; c < IB; ++c) {
                if (ib + c >= R) break;
                any = any | (__builtin_fma(ab.x, tt[c], ab.y * dn_blk[c]) <= cur);
              }
              if (__builtin_amdgcn_ballot_w64(any)) qmask |= 1u << q;
            }
            if (qmask) {
#pragma unroll 1
              for (unsigned int qs = qmask; qs; qs &= qs - 1) {
                const int q = __builtin_ctz(qs);
                const double2 ab = s_ab[wave][q];
                AlphaEntry* const e = &s_aent[wave][q];
#pragma unroll
                for (int c = 0; c < IB; ++c) {
                  const int ia = ib + c;
                  if (ia >= R) break;
                  const double v = __builtin_fma(ab.x, tt[c], ab.y * dn_blk[c]);
                  wave_sync();
                  const double cur = lds_load(&e->val);
                  if (__builtin_amdgcn_ballot_w64(v <= cur)) {
                    const unsigned int lid = lid_oo + (unsigned int)ia;
                    const unsigned long long ak = order_key(v);
                    const unsigned long long ak_old = lds_load(&e->key);
                    const unsigned int ai_old = lds_load(&e->lid);
                    const bool cand = (v <= cur) & ((ak < ak_old) | ((ak == ak_old) & (lid < ai_old)));
                    if (cand) atomicMin(&e->key, ak);
                    const unsigned long long ak_new = cand ? lds_load(&e->key) : 0ull;
                    if (cand && ak_new < ak_old) lds_store(&e->lid, 0xFFFFFFFFu);
                    if (cand && ak == ak_new) {
                      atomicMin(&e->lid, lid);
                      lds_store(&e->val, v);
                    }
                  }
                }
              }
            }
          }
        }
      }
    }
    // The tile's partials: lane j = bucket j.
    if constexpr (DM) {
    } else {
      wave_sync();
      const unsigned int bl = bucket[lane].lid;
      a.part_obj[(size_t)t * 64 + lane] = __longlong_as_double((long long)bucket[lane].key);
      a.part_id[(size_t)t * 64 + lane] = bl == 0xFFFFFFFFu ? kNone : g.base + (uint64_t)bl;
    }
    if constexpr (AL) {
      if (lane < a.n_alpha) {
        const AlphaEntry e = s_aent[wave][lane];
        a.part_aobj[(size_t)t * a.n_alpha + lane] = e.val;
        a.part_aid[(size_t)t * a.n_alpha + lane] = e.lid == 0xFFFFFFFFu ? kNone : g.base + (uint64_t)e.lid;
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
}

// ---------------------------------------------------------------------------------------
// K2: lane j owns bucket j.  With W = 4, a block of four waves per group: each wave takes
// the lexicographic minimum over every fourth tile of the group (its full-size ones, then its
// small ones), so the largest group's chain of dependent loads is a quarter as long, and the
// first wave combines the four in LDS; with W = 1 (spaces whose groups hold few tiles), a wave
// per group.  Then the group's best by a butterfly over the 64 lanes and the staircase by an
// exclusive prefix minimum over the buckets.
// ---------------------------------------------------------------------------------------
template <int kW>
__global__ __launch_bounds__(256) void k_reduce(ReduceArgs a) {
  __shared__ double s_o[kW][64];
  __shared__ uint64_t s_i[kW][64];
  __shared__ double s_ao[kW][kMaxAlphas];
  __shared__ uint64_t s_ai[kW][kMaxAlphas];
  const int lane = threadIdx.x & 63;
  // Wave-uniform (stated, so that the group record arrives by scalar loads and the tile loops
  // run on scalar registers).
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wave = kW > 1 ? wv : 0;  // the wave's share of the tiles
  const int64_t g = kW > 1 ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + wv;
  if (g >= a.n_groups) return;
  const DevGroup grp = load_uniform(a.groups + g);
  double obj = __builtin_huge_val();
  uint64_t id = kNone;
  if (lane < a.NB) {  // several tiles' loads in flight
#pragma unroll 4
    for (int t = grp.tile_begin + wave; t < grp.tile_begin + grp.n_tiles; t += kW) {
      const double o = __builtin_nontemporal_load(a.part_obj + (size_t)t * 64 + lane);  // read once
      const uint64_t i = __builtin_nontemporal_load(a.part_id + (size_t)t * 64 + lane);
      if (lex_less(o, i, obj, id)) {
        obj = o;
        id = i;
      }
    }
#pragma unroll 4
    for (int t = grp.tail_begin + wave; t < grp.tail_begin + grp.n_tail; t += kW) {
      const double o = __builtin_nontemporal_load(a.part_obj + (size_t)t * 64 + lane);
      const uint64_t i = __builtin_nontemporal_load(a.part_id + (size_t)t * 64 + lane);
      if (lex_less(o, i, obj, id)) {
        obj = o;
        id = i;
      }
    }
  }
  if constexpr (kW > 1) {
    s_o[wave][lane] = obj;
    s_i[wave][lane] = id;
  }
  double ao = __builtin_huge_val();
  uint64_t ai = kNone;
  if (lane < a.n_alpha) {  // lane a: weight sample a
    for (int t = grp.tile_begin + wave; t < grp.tile_begin + grp.n_tiles; t += kW) {
      const double o = a.part_aobj[(size_t)t * a.n_alpha + lane];
      const uint64_t i = a.part_aid[(size_t)t * a.n_alpha + lane];
      if (lex_less(o, i, ao, ai)) {
        ao = o;
        ai = i;
      }
    }
    for (int t = grp.tail_begin + wave; t < grp.tail_begin + grp.n_tail; t += kW) {
      const double o = a.part_aobj[(size_t)t * a.n_alpha + lane];
      const uint64_t i = a.part_aid[(size_t)t * a.n_alpha + lane];
      if (lex_less(o, i, ao, ai)) {
        ao = o;
        ai = i;
      }
    }
    if constexpr (kW > 1) {
      s_ao[wave][lane] = ao;
      s_ai[wave][lane] = ai;
    }
  }
  if constexpr (kW > 1) {
    __syncthreads();
    if (wave != 0) return;
    // The group's lexicographic minima over the waves' (order does not matter).
#pragma unroll
    for (int w = 1; w < kW; ++w)
      if (lex_less(s_o[w][lane], s_i[w][lane], obj, id)) {
        obj = s_o[w][lane];
        id = s_i[w][lane];
      }
  }
  a.bucket_obj[g * 64 + lane] = obj;
  a.bucket_id[g * 64 + lane] = id;

  double bo = obj;
  uint64_t bi = id;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(bo, off, 64);
    const uint64_t i = __shfl_xor(bi, off, 64);
    if (lex_less(o, i, bo, bi)) {
      bo = o;
      bi = i;
    }
  }
  double pm = obj;  // inclusive prefix minimum over buckets 0..lane
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_up(pm, off, 64);
    if (lane >= off) pm = __builtin_fmin(pm, o);
  }
  double below = __shfl_up(pm, 1, 64);
  if (lane == 0) below = __builtin_huge_val();
  const bool on = id != kNone && obj < below;
  const uint64_t mask = __ballot(on);
  if (lane == 0) {
    a.best_obj[g] = bo;
    a.best_id[g] = bi;
    a.frontier[g] = mask;
  }
  if (lane < a.n_alpha) {
#pragma unroll
    for (int w = 1; w < kW; ++w)
      if (lex_less(s_ao[w][lane], s_ai[w][lane], ao, ai)) {
        ao = s_ao[w][lane];
        ai = s_ai[w][lane];
      }
    a.alpha_obj[g * a.n_alpha + lane] = ao;
    a.alpha_id[g * a.n_alpha + lane] = ai;
  }
}

// Per-id evaluation (parity and listed configurations).
__global__ __launch_bounds__(256) void k_eval_ids(EvalArgs a, const uint64_t* __restrict__ ids,
                                                  int64_t n, double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const OneVal v = eval_one(a, ids[i]);
  out[4 * i + 0] = v.t;
  out[4 * i + 1] = v.d;
  out[4 * i + 2] = v.mem;
  out[4 * i + 3] = v.obj;
}

// Candidate filter of the exact frontier: one wave per group, lane j = bucket j.
__global__ __launch_bounds__(kReduceBlock) void k_filter(EvalArgs a, const double* __restrict__ bucket_obj,
                                                         const uint64_t* __restrict__ bucket_id,
                                                         FiltEntry* __restrict__ filt) {
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * (kReduceBlock / 64) + (threadIdx.x >> 6);
  if (g >= a.n_groups) return;
  const double obj = lane < a.NB ? bucket_obj[g * 64 + lane] : __builtin_huge_val();
  const uint64_t id = lane < a.NB ? bucket_id[g * 64 + lane] : kNone;
  double pm = obj;  // inclusive prefix minimum over buckets 0..lane
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_up(pm, off, 64);
    if (lane >= off) pm = __builtin_fmin(pm, o);
  }
  double below = __shfl_up(pm, 1, 64);
  if (lane == 0) below = __builtin_huge_val();
  FiltEntry f;
  f.pm = below;
  f.bobj = obj;
  f.bmem = id < a.n_configs ? eval_one(a, id).mem : __builtin_huge_val();  // kNone, or a table never written
  filt[g * 64 + lane] = f;
}

int check_launch() {
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : (int)e;
}

template <int R, int MODE>
void launch_eval_rm(const EvalArgs& a, int blocks, hipStream_t st) {
  hipLaunchKernelGGL((k_eval<R, MODE>), dim3(blocks), dim3(kBlock), 0, st, a, a.ratio, (const PairK*)a.pk);
}

template <int R>
void launch_eval_r(const EvalArgs& a, int blocks, int mode, hipStream_t st) {
  switch (mode) {
    case kModeAlpha: launch_eval_rm<R, kModeAlpha>(a, blocks, st); break;
    case kModeDump: launch_eval_rm<R, kModeDump>(a, blocks, st); break;
    default: launch_eval_rm<R, kModeBuckets>(a, blocks, st); break;
  }
}

template <int R, int MODE>
int blocks_per_cu_rm() {
  int n = 0;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_eval<R, MODE>, kBlock, 0) == hipSuccess ? n : 1;
}

template <int R>
int blocks_per_cu_r(int mode) {
  switch (mode) {
    case kModeAlpha: return blocks_per_cu_rm<R, kModeAlpha>();
    case kModeDump: return blocks_per_cu_rm<R, kModeDump>();
    default: return blocks_per_cu_rm<R, kModeBuckets>();
  }
}

#define MIST_FOR_EACH_R(X) \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

}  // namespace

int eval_blocks_per_cu(int R, int mode) {
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

int launch_eval(const EvalArgs& a, int blocks, int mode, void* stream) {
  if (mode != kModeBuckets && mode != kModeAlpha && mode != kModeDump) return (int)hipErrorInvalidValue;
  if (a.n_tiles <= 0) return 0;
  hipStream_t st = (hipStream_t)stream;
  switch (a.R) {
#define MIST_CASE(n)                       \
  case n:                                  \
    launch_eval_r<n>(a, blocks, mode, st); \
    break;
    MIST_FOR_EACH_R(MIST_CASE)
#undef MIST_CASE
    default:
      return (int)hipErrorInvalidValue;
  }
  return check_launch();
}

int launch_pairs(const EvalArgs& a, void* stream) {
  if (a.n_pk <= 0) return 0;
  hipLaunchKernelGGL(k_pairs, dim3((unsigned)((a.n_pk + 255) / 256)), dim3(256), 0, (hipStream_t)stream, a);
  return check_launch();
}

int launch_reduce(const ReduceArgs& a, void* stream) {
  if (a.n_groups <= 0) return 0;
  // Four waves per group pay off when some group's tiles make a long chain of loads and the
  // groups are few enough that the idle waves of small groups cost little (measured: 23 ->
  // 14 us on gpt2.7b-d16, 44 -> 31 us on llama13b-d64; 89 -> 93 us on llama42b-d128-hw64,
  // 66,496 groups, which keeps a wave per group).
  if (a.max_group_tiles >= 16 && a.n_groups <= 16384)
    hipLaunchKernelGGL(k_reduce<4>, dim3((unsigned)a.n_groups), dim3(256), 0, (hipStream_t)stream, a);
  else
    hipLaunchKernelGGL(k_reduce<1>, dim3((unsigned)((a.n_groups + 3) / 4)), dim3(256), 0, (hipStream_t)stream, a);
  return check_launch();
}

int launch_filter(const EvalArgs& a, const double* bucket_obj, const uint64_t* bucket_id, FiltEntry* filt,
                  void* stream) {
  if (a.n_groups <= 0) return 0;
  const int per = kReduceBlock / 64;
  const int64_t blocks = (a.n_groups + per - 1) / per;
  hipLaunchKernelGGL(k_filter, dim3((unsigned)blocks), dim3(kReduceBlock), 0, (hipStream_t)stream, a, bucket_obj,
                     bucket_id, filt);
  return check_launch();
}

int launch_eval_ids(const EvalArgs& a, const uint64_t* ids, int64_t n, double* out, void* stream) {
  if (n <= 0) return 0;
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(k_eval_ids, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, a, ids,
                     n, out);
  return check_launch();
}

}  // namespace mist
