// Device code that the evaluation kernels share: the cost model's levels (Sec. 5.2, Eq. 4-6), Algorithm 1
// in its wave-uniform forms, and the per-wave LDS tables of the reductions.
//
// Numerics: every floating-point operation of the cost model is an explicit IEEE binary64
// operation in a fixed order; the library is built with -ffp-contract=off and every fused
// multiply-add is an explicit __builtin_fma.  Reciprocals (1/F, 1/PCIe, 1/link, 1/DP,
// 1/eta(b), 1/phi) come from host divisions.  The results are therefore bit-reproducible
// and independent of the launch geometry.
#pragma once

#include <hip/hip_runtime.h>

#include "mist_internal.h"

namespace mist {
namespace {

constexpr uint64_t kNone = ~0ull;

__device__ __forceinline__ bool lex_less(double o1, uint64_t i1, double o2, uint64_t i2) {
  return o1 < o2 || (o1 == o2 && i1 < i2);
}

// ---------------------------------------------------------------------------------------
// Cost model, level by level.  Each level holds the quantities that depend on the digits
// fixed at that level: pair (b, TP, DP), recomputed layers c, ZeRO level z, then the
// weight, gradient, optimizer-state and activation offload ratios.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ PairK pair_level(const DevModel& m, int64_t PP, int64_t k, int64_t l,
                                            const DevPair& pr, const DevHw& hw) {
  const int64_t h = m.h, s = m.s, V = m.V, f = m.f, bw = m.bw, bo = m.bo;
  const int64_t b = pr.b, TP = pr.tp, DP = pr.dp;
  const int64_t first = (k == PP) ? 1 : 0;
  const int64_t last = (k == 1) ? 1 : 0;
  const int64_t dh = h / m.heads;
  const int64_t hkvr = (TP <= m.kv) ? (m.kv * dh) / TP : dh;  // KV heads replicated past kv
  const int64_t Pq = 2 * h * h;
  const int64_t Pm = (m.gpt ? 2 : 3) * h * f;
  const int64_t Prep = m.gpt ? 4 * h : 2 * h;
  const int64_t Psi = (Pq + Pm) / TP + 2 * h * hkvr + Prep;
  const int64_t Vr = (V + TP - 1) / TP;
  const int64_t Pe = Vr * h + (m.gpt ? s * h : 0);
  const int64_t Ph = Vr * h + (m.gpt ? 2 * h : h);
  const int64_t Pst = l * Psi + first * Pe + last * Ph;
  int64_t Pbuf = Psi;
  if (first * Pe > Pbuf) Pbuf = first * Pe;
  if (last * Ph > Pbuf) Pbuf = last * Ph;
  const int64_t mf = m.gpt ? 2 : 3;
  const int64_t atok = 4 * h + (2 * h + mf * f) / TP + 2 * hkvr + (m.flash ? 0 : m.heads * s / TP);
  const int64_t ftok = 2 * ((Pq + Pm) / TP + 2 * h * hkvr) + 4 * s * h / TP;
  const int64_t Fl = b * s * ftok;
  const int64_t Fh = last * 2 * b * s * h * Vr;
  const int64_t Xl = last * 4 * b * s * Vr;
  const int64_t p2pB = ((k > 1 ? 1 : 0) + (k < PP ? 1 : 0)) * b * s * h * bw;
  const int64_t arB = 2 * (TP - 1) * (b * s * h * bw / TP);
  const int64_t rB = (DP - 1) * bw * Pst;

  PairK P;
  P.afull = b * s * bw * atok;
  P.ack = b * s * bw * h;
  P.iD = pr.inv_dp;
  P.Pw = (double)(Pst * bw);
  P.Po = (double)(Pst * bo);
  P.Wb2 = (double)(2 * Pbuf * bw);
  P.Ob2o = (double)(2 * Pbuf * bo);
  P.A2 = (double)(2 * P.afull);
  P.AF = (double)P.afull;
  P.Xd = (double)Xl;
  P.Fld = (double)Fl;
  P.Fh3 = (double)(3 * Fh);
  P.r = ((double)rB * P.iD) * hw.iL;
  P.p2p = (double)p2pB * hw.iL;
  P.ar = (double)arB * hw.iL;
  P.FE = hw.iF * hw.ieta[pr.mb];
  return P;
}

struct CkptK {
  double A, KA, Rc, C;  // microbatch activations, in-flight stash, recompute unit, compute time
};

__device__ __forceinline__ CkptK ckpt_level(const PairK& P, int64_t l, int64_t c, int64_t ke) {
  const int64_t Amb = (l - c) * P.afull + c * P.ack;
  CkptK K;
  K.A = (double)Amb;
  K.KA = (double)(ke * Amb);
  K.Rc = c > 0 ? P.AF : 0.0;
  // fwd + 2 bwd per layer, one more fwd per recomputed layer, LM head fwd + bwd; serial TP
  // all-reduces: 2 fwd + 2 bwd per layer, 2 per recomputed layer.
  const double work = __builtin_fma((double)(3 * l + c), P.Fld, P.Fh3);
  K.C = __builtin_fma((double)(4 * l + 2 * c), P.ar, work * P.FE);
  return K;
}

struct ZeroK {
  double sw, sg;       // shard factors of weights and gradients
  double Sw, Sg, So;   // resident-if-kept bytes: weights, gradients, optimizer states
  double HWz;          // weight bytes fetched per microbatch (forward and backward)
  double G2Gs, G2Gf;   // GPU<->GPU stream: stable and first microbatch
  double Obo, Obg;     // optimizer-step unit parts
};

__device__ __forceinline__ ZeroK zero_level(const PairK& P, int z) {
  ZeroK Z;
  Z.sw = z == 3 ? P.iD : 1.0;
  Z.sg = z >= 2 ? P.iD : 1.0;
  const double so = z >= 1 ? P.iD : 1.0;
  Z.Sw = P.Pw * Z.sw;
  Z.Sg = P.Pw * Z.sg;
  Z.So = P.Po * so;
  Z.HWz = 2.0 * Z.Sw;
  const double ms = z == 2 ? 1.0 : (z == 3 ? 3.0 : 0.0);  // RS; AG + AG + RS
  const double mf = z == 3 ? 3.0 : 2.0;                   // first microbatch in total
  Z.G2Gs = __builtin_fma(ms, P.r, P.p2p);
  Z.G2Gf = __builtin_fma(mf, P.r, P.p2p);
  Z.Obo = P.Ob2o * so;
  Z.Obg = P.Wb2 * Z.sg;
  return Z;
}

// Weight and gradient offload levels (fixed within a strip).
struct WoGoK {
  double Swg;          // resident weight + gradient bytes
  double Wbuf, Gbuf;   // double-buffered fetched weights / gradient unit
  double HW;           // weight bytes fetched per microbatch (forward and backward)
  double DW;           // updated weight bytes written back after the step
  double DG;           // gradient bytes offloaded per microbatch
  double Og;           // gradient part of the optimizer-step unit
};

__device__ __forceinline__ WoGoK wogo_levels(const PairK& P, const ZeroK& Z, double rw, double qw,
                                             double rg, double qg) {
  WoGoK W;
  const double Sww = qw * Z.Sw;
  W.Wbuf = P.Wb2 * (1.0 - qw * Z.sw);
  W.HW = rw * Z.HWz;
  W.DW = rw * Z.Sw;
  W.Swg = __builtin_fma(qg, Z.Sg, Sww);
  W.Gbuf = P.Wb2 * (1.0 - qg * Z.sg);
  W.DG = rg * Z.Sg;
  W.Og = rg * Z.Obg;
  return W;
}

// Strip constants that the optimizer-state offload level reads, kept in a per-lane LDS
// record (registers are the scarce resource of the evaluation kernel).
struct OoIn {
  double So, Swg, Obo, Og, DG, DW, Wbuf, Gbuf, Rc, Xd;
};

// Optimizer-state offload level: everything of a configuration except its activation
// ratio's terms.
struct OoK {
  double Bmax;         // max(forward, backward) peak without the activation terms
  double H2Dx, D2Hx;   // seconds: first-microbatch extras
};

__device__ __forceinline__ OoIn oo_inputs(const PairK& P, const CkptK& K, const ZeroK& Z,
                                          const WoGoK& W) {
  return OoIn{Z.So, W.Swg, Z.Obo, W.Og, W.DG, W.DW, W.Wbuf, W.Gbuf, K.Rc, P.Xd};
}

__device__ __forceinline__ OoK oo_level(const OoIn& I, double ro, double qo, double iP) {
  const double S = __builtin_fma(qo, I.So, I.Swg);
  const double Obuf = __builtin_fma(ro, I.Obo, I.Og);
  const double HX = __builtin_fma(ro, I.So, I.DG);
  const double DX = __builtin_fma(ro, I.So, I.DW);
  const double base = S + I.Wbuf;
  const double BF = (base + Obuf) + I.Xd;
  const double BB = ((base + I.Gbuf) + I.Rc) + I.Xd;
  OoK O;
  // max(BF + x, BB + x) == max(BF, BB) + x: rounding to nearest is monotone.
  O.Bmax = __builtin_fmax(BF, BB);
  O.H2Dx = HX * iP;
  O.D2Hx = DX * iP;
  return O;
}

// ---------------------------------------------------------------------------------------
// Algorithm 1.
//
// Visiting n = 4..2 and updating when the non-zero pattern has exactly n streams is the
// same as updating while the pattern has at least two streams (each update stops at least
// one stream), so three fixed rounds suffice.  A round reads the row of the current
// pattern: rows of two or more streams scale members by phi, overlap the smallest scaled
// time, and leave members (scaled - overlap) * psi; non-members (time 0, or NaN from an
// earlier round) carry phi = +inf and become NaN, which min and max skip and "> 0"
// rejects.  Rows of at most one stream have phi = psi = 1; such a round always meets an
// exact zero (an unused stream, or the stream that finished last) so its overlap is 0 and
// nothing changes.  At the end at most one stream is positive and the others are 0 or NaN,
// so the oracle's final sum equals the running total plus the largest remaining time.
// ---------------------------------------------------------------------------------------
struct Streams {
  double x0, x1, x2, x3;
};

__device__ __forceinline__ double round_row(Streams& x, double f0, double f1, double f2, double f3,
                                            double p0, double p1, double p2, double p3) {
  const double s0 = x.x0 * f0, s1 = x.x1 * f1, s2 = x.x2 * f2, s3 = x.x3 * f3;
  const double ov = __builtin_fmin(__builtin_fmin(s0, s1), __builtin_fmin(s2, s3));
  x.x0 = (s0 - ov) * p0;
  x.x1 = (s1 - ov) * p1;
  x.x2 = (s2 - ov) * p2;
  x.x3 = (s3 - ov) * p3;
  return ov;
}

// Interference rows in LDS are padded to kLdsRow doubles so that lanes reading different
// rows spread over more banks.
constexpr int kLdsRow = 10;

template <int STRIDE>
__device__ __forceinline__ double round_lookup(Streams& x, const double* __restrict__ tab) {
  // Row of the non-zero pattern (bit i for stream i), as a pre-scaled offset.
  const int off = (x.x0 > 0.0 ? STRIDE : 0) + (x.x1 > 0.0 ? 2 * STRIDE : 0) +
                  (x.x2 > 0.0 ? 4 * STRIDE : 0) + (x.x3 > 0.0 ? 8 * STRIDE : 0);
  const double* e = tab + off;
  return round_row(x, e[0], e[1], e[2], e[3], e[4], e[5], e[6], e[7]);
}

__device__ __forceinline__ double remaining(const Streams& x) {
  return __builtin_fmax(__builtin_fmax(x.x0, x.x1), __builtin_fmax(x.x2, x.x3));
}

// Three rounds with per-lane rows (rows STRIDE doubles apart).
template <int STRIDE = kLdsRow>
__device__ __forceinline__ double interference(double c, double g, double h, double d,
                                               const double* __restrict__ tab) {
  Streams x{c, g, h, d};
  double T = round_lookup<STRIDE>(x, tab);
  T = T + round_lookup<STRIDE>(x, tab);
  T = T + round_lookup<STRIDE>(x, tab);
  return T + remaining(x);
}

// Calls whose first round uses a row known in advance: every configuration of a strip whose host
// streams both run (pattern 15, or 13 without GPU-GPU traffic), with compute c and GPU-GPU g fixed
// per strip.  The strip precomputes the scaled c and g and their minimum m01.
//
// After a round a member keeps running exactly when its scaled time exceeds the overlap
// (s_j - ov > 0, and (s_j - ov) * psi_j cannot round to zero: the host's input bounds keep every
// non-zero stream time and difference far above the subnormal range).  In the common case the
// GPU-GPU stream is a member and its scaled time s1 is below every other member's: the overlap is
// s1 itself, compute, host->device and device->host keep running, and the second round reads
// row 13 for every such configuration, with compute's second-round scaled time y0 fixed per
// strip.  The second-round scaled times y_j = ((s_j - s1) * psi15_j) * phi13_j have the sign of
// s_j - s1, so that case is y0 > 0 and y2, y3 > 0 (with pattern 13, s1 and y0 are NaN and the
// case never holds).
struct KnownRow {
  double s0, s1, m01;   // c * phi0, g * phi1 (NaN when GPU-GPU is no member), min of the two
  double y0;            // compute's scaled time in the second round (row 13) when s1 < s0
  const double* row;    // the first round's row
};

__device__ __forceinline__ KnownRow known_row(const double* __restrict__ tab, int pattern, double c, double g) {
  const double* e = tab + pattern * kLdsRow;
  KnownRow r;
  r.s0 = c * e[0];
  r.s1 = g * e[1];
  r.m01 = __builtin_fmin(r.s0, r.s1);
  r.row = e;
  r.y0 = ((r.s0 - r.s1) * e[4]) * tab[13 * kLdsRow + 0];
  return r;
}

// General rounds of such a call with host streams h, d > 0: the first with the known row, the
// others looked up by the lanes' patterns.
__device__ __forceinline__ double interference_general(const KnownRow& r, double h, double d,
                                                       const double* __restrict__ tab) {
  const double* e = r.row;
  const double s2 = h * e[2], s3 = d * e[3];
  const double ov = __builtin_fmin(r.m01, __builtin_fmin(s2, s3));
  Streams x{(r.s0 - ov) * e[4], (r.s1 - ov) * e[5], (s2 - ov) * e[6], (s3 - ov) * e[7]};
  double T = ov;
  T = T + round_lookup<kLdsRow>(x, tab);
  T = T + round_lookup<kLdsRow>(x, tab);
  return T + remaining(x);
}

// Rows of the third round when compute and one host stream are left after the second round
// (row 13's overlap ended the other host stream): for the stream h left (index 0: h = 2, row 5;
// index 1: h = 3, row 9) the kTab2 doubles phi[0], phi[h], psi[0], psi[h] of that row and psi[0],
// psi[h] of row 13, so that a lane reads its row from one per-lane offset.
constexpr int kTab2 = 6;
constexpr int kTab2Off = 16 * kLdsRow;  // after the sixteen pattern rows

// The factors every configuration's second-round scaled host times read: phi and psi of the host
// streams in row 15 and their phi in row 13.  Wave-uniform, loaded once per tile into scalar
// registers (as vector registers they crowd the strip loop into spilling).
struct RowK {
  double f2, f3;  // phi15[2], phi15[3]
  double p2, p3;  // psi15[2], psi15[3]
  double g2, g3;  // phi13[2], phi13[3]
};

// Algorithm 1 for one configuration of a strip with the strip's known first-round row.  Each form
// is chosen for the whole wave (lanes with free set, whose result the caller replaces or does
// not use, do not take part), so that every form is straight-line code:
//   - GPU-GPU finishes first (row 15) and the second round (row 13: compute, host->device,
//     device->host) ends the smaller host stream: compute and the larger host stream are left,
//     and each lane reads their row (5 or 9) at a per-lane offset and forms only their terms;
//   - GPU-GPU finishes first and compute ends the second round: both host streams are left, and
//     the third round's row (12) is the same for the wave;
//   - GPU-GPU finishes first otherwise (waves that mix the two cases above, ties): the third
//     round's row is looked up per lane from all three streams;
//   - else the general rounds (interference_general).
// Each form performs the same operations on the same operands as the general rounds: a stream
// that has finished carries NaN there (its time 0 times the row's +inf factor), which drops out
// of the minimum and the maximum that the special forms take over the streams left.  form
// receives the form taken (kForm*; read by the dump variant only).
constexpr int kFormHostLeft = 1;    // compute and the larger host stream left: per-lane row 5 or 9
constexpr int kFormHostsLeft = 2;   // compute finished in the second round: row 12
constexpr int kFormLookup = 3;      // GPU-GPU first, third row looked up per lane
constexpr int kFormGeneral = 4;     // the general rounds
constexpr int kFormZero = 5;        // the all-zero configuration's closed form (first microbatch)
constexpr int kFormGeneric = 6;     // three rounds from an unknown pattern (stable time, ratio 0)

__device__ __forceinline__ double interference_known(const KnownRow& r, double h, double d, bool free,
                                                     const double* __restrict__ tab, const RowK& K,
                                                     int& form) {
  const double* e13 = tab + 13 * kLdsRow;
  const double y0 = r.y0;
  const double y2 = ((h * K.f2 - r.s1) * K.p2) * K.g2;
  const double y3 = ((d * K.f3 - r.s1) * K.p3) * K.g3;
  const double m23 = __builtin_fmin(y2, y3);
  const double yh = __builtin_fmax(y2, y3);
  // Wave masks of plain compares (combined by the scalar unit).
  const unsigned long long ex = __builtin_amdgcn_read_exec();
  const unsigned long long fm = __builtin_amdgcn_ballot_w64(free);
  const unsigned long long g1 = __builtin_amdgcn_ballot_w64(m23 > 0.0);  // with y0 > 0: GPU-GPU first
  if (((__builtin_amdgcn_ballot_w64(y0 > m23) & g1 & __builtin_amdgcn_ballot_w64(yh > m23)) | fm) == ex) {
    // Compute and the larger host stream are left (row 5 or 9); the second round's overlap is
    // the smaller host time m23.
    const double* e = tab + kTab2Off + (y2 > y3 ? 0 : kTab2);
    const double z0 = (y0 - m23) * e[4];
    const double zh = (yh - m23) * e[5];
    const double w0 = z0 * e[0], wh = zh * e[1];
    const double ov3 = __builtin_fmin(w0, wh);
    const double rem = __builtin_fmax((w0 - ov3) * e[2], (wh - ov3) * e[3]);
    form = kFormHostLeft;
    return ((r.s1 + m23) + ov3) + rem;
  }
  const unsigned long long y0p = __builtin_amdgcn_ballot_w64(y0 > 0.0);
  if (((__builtin_amdgcn_ballot_w64(y0 < m23) & y0p) | fm) == ex) {
    // Compute finished in the second round (overlap y0); both host streams are left (row 12).
    const double* e12 = tab + 12 * kLdsRow;
    const double w2 = ((y2 - y0) * e13[6]) * e12[2];
    const double w3 = ((y3 - y0) * e13[7]) * e12[3];
    const double ov3 = __builtin_fmin(w2, w3);
    const double rem = __builtin_fmax((w2 - ov3) * e12[6], (w3 - ov3) * e12[7]);
    form = kFormHostsLeft;
    return ((r.s1 + y0) + ov3) + rem;
  }
  if (((y0p & g1) | fm) == ex) {
    const double ov2 = __builtin_fmin(y0, m23);
    const double T2 = r.s1 + ov2;
    // Third round: the row of the streams still running, those whose scaled time exceeds the
    // overlap.
    const bool q0 = y0 > ov2, q2 = y2 > ov2, q3 = y3 > ov2;
    const double z0 = (y0 - ov2) * e13[4], z2 = (y2 - ov2) * e13[6], z3 = (y3 - ov2) * e13[7];
    const double* e = tab + ((q0 ? 1 : 0) + (q2 ? 4 : 0) + (q3 ? 8 : 0)) * kLdsRow;
    const double w0 = z0 * e[0], w2 = z2 * e[2], w3 = z3 * e[3];
    const double ov3 = __builtin_fmin(__builtin_fmin(w0, w2), w3);
    const double rem = __builtin_fmax(__builtin_fmax((w0 - ov3) * e[4], (w2 - ov3) * e[6]), (w3 - ov3) * e[7]);
    form = kFormLookup;
    return (T2 + ov3) + rem;
  }
  form = kFormGeneral;
  return interference_general(r, h, d, tab);
}

// Algorithm 1 on (c, g, +0, +0), c > 0: the first round uses the row of pattern 3 (compute and
// GPU-GPU), after which at most one stream is positive and the other rounds leave the times
// unchanged and add +0; with g = 0 the only row met has one stream and the time is c.  This
// equals interference() on the same streams bit for bit.
__device__ __forceinline__ double interference_zero(double c, double g, const double* __restrict__ tab) {
  const double* e = tab + 3 * kLdsRow;
  const double s0 = c * e[0], s1 = g * e[1];
  const double ov = __builtin_fmin(s0, s1);
  const double t = ov + __builtin_fmax((s0 - ov) * e[4], (s1 - ov) * e[5]);
  return g > 0.0 ? t : c;
}

struct BucketEntry {
  double edge;             // the bucket's upper memory edge E_j (+inf past NB - 1): the edge
                           // and the key are adjacent, read together
  unsigned long long key;  // bits of the minimum objective (a non-negative double orders like
                           // its bit pattern)
  unsigned int lid;        // lowest local id (id - group base, < 2^32) reaching it; 0xFFFFFFFF:
                           // none of this tile
  unsigned int pad;
};
static_assert(sizeof(BucketEntry) == 24, "24-byte entries: the entry offset is one multiply-add");

// Weight-sampled argmin (Eq. 4 with sampled alpha) of the wave's current tile: the value
// (a double, for the fast comparison), its order key (for the LDS atomic minimum; weighted
// values may be negative) and the lowest local id reaching it.
struct AlphaEntry {
  double val;
  unsigned long long key;
  unsigned int lid;
  unsigned int pad;
};

// Reads a table entry at a wave-uniform index through the constant address space, so that it
// arrives in scalar registers (scalar loads; the tables are read-only during the kernel).
template <class T>
__device__ __forceinline__ T load_uniform(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole dwords");
  const __attribute__((address_space(4))) uint32_t* q = (const __attribute__((address_space(4))) uint32_t*)p;
  T v;
  uint32_t* d = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) d[i] = q[i];
  return v;
}

// A 64-bit key that orders like the double (neither -0 nor NaN occurs as a key).
__device__ __forceinline__ unsigned long long order_key(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// The double an order key stands for.
__device__ __forceinline__ double order_value(unsigned long long k) {
  return __longlong_as_double((long long)((k >> 63) ? k & 0x7FFFFFFFFFFFFFFFull : ~k));
}

// Orders this wave's LDS accesses for the compiler: a lane may read a word another lane of
// the same wave wrote (the hardware executes a wave's LDS operations in order), so no load
// may be moved across this point or answered from the lane's own earlier store.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Words that other lanes of the wave update with atomics are read and written with relaxed
// wavefront-scope atomics: a plain load after a lane's own atomic update could otherwise be
// answered from a value the compiler already holds (for an entry at a wave-uniform address the
// compiler combines the lanes' atomic minima into one update by one lane).
template <class T>
__device__ __forceinline__ T lds_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

template <class T>
__device__ __forceinline__ void lds_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// ---------------------------------------------------------------------------------------
// Per-id evaluation with the same level functions (parity, listed configurations and result
// extraction).
// ---------------------------------------------------------------------------------------
struct OneVal {
  double t, d, mem, obj;
};

// The digits of a configuration id: binary search of the group, mixed-radix decode.
struct Digits {
  int64_t group;
  int p, c, z, iw, ig, io, ia;
};

__device__ __forceinline__ Digits decode_one(const EvalArgs& a, uint64_t id) {
  int64_t lo = 0, hi = a.n_groups;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) / 2;
    if (a.groups[mid].base <= id) lo = mid;
    else hi = mid;
  }
  const DevGroup& g = a.groups[lo];
  const uint64_t R = (uint64_t)a.R;
  uint64_t v = id - g.base;
  Digits x;
  x.group = lo;
  x.ia = (int)(v % R);
  v /= R;
  x.io = (int)(v % R);
  v /= R;
  x.ig = (int)(v % R);
  v /= R;
  x.iw = (int)(v % R);
  v /= R;
  x.z = (int)(v % 4);
  v /= 4;
  x.c = (int)(v % (uint64_t)(g.l + 1));
  x.p = (int)(v / (uint64_t)(g.l + 1));
  return x;
}

__device__ OneVal eval_one(const EvalArgs& a, const Digits& x) {
  const DevGroup g = a.groups[x.group];
  const DevHw& hw = a.hws[g.hw];
  const double* r = a.ratio;
  const double* om = a.ratio + a.R;
  const int64_t ke = g.k < g.G ? g.k : g.G;
  const double* tab = &hw.itab[0][0];
  const PairK P = pair_level(a.m, g.PP, g.k, g.l, a.pairs[g.pair_begin + x.p], hw);
  const CkptK K = ckpt_level(P, g.l, x.c, ke);
  const ZeroK Z = zero_level(P, x.z);
  const WoGoK W = wogo_levels(P, Z, r[x.iw], om[x.iw], r[x.ig], om[x.ig]);
  const OoK O = oo_level(oo_inputs(P, K, Z, W), r[x.io], om[x.io], hw.iP);
  const double ra = r[x.ia];
  const double SO = __builtin_fma(ra, P.A2, om[x.ia] * K.KA);
  const double H2Ds = __builtin_fma(ra, K.A, W.HW) * hw.iP;
  const double D2Hs = __builtin_fma(ra, K.A, W.DG) * hw.iP;
  OneVal res;
  res.mem = O.Bmax + SO;
  res.t = interference<kTabStride>(K.C, Z.G2Gs, H2Ds, D2Hs, tab);
  const double T1 = interference<kTabStride>(K.C, Z.G2Gf, H2Ds + O.H2Dx, D2Hs + O.D2Hx, tab);
  res.d = T1 - res.t;
  res.obj = __builtin_fma((double)g.G, res.t, res.d);
  return res;
}

// One configuration by id.
__device__ __forceinline__ OneVal eval_one(const EvalArgs& a, uint64_t id) { return eval_one(a, decode_one(a, id)); }

}  // namespace
}  // namespace mist
