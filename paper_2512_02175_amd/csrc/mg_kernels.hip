// mg_kernels.hip -- gfx950 kernels of the timestep-splitting Euler-Maruyama
// particle step on metric graphs (Dwaraknath & Ying, Alg. 2 with Alg. 1's
// vertex rule), the particle initialisation and the per-edge histogram.
//
// One lane owns one particle for all steps of a launch; its edge record
// lives in registers and is reloaded only when a vertex hit changes the
// edge, so the common no-hit step touches no memory.  Random numbers are
// counter-based Philox4x32-10 (Salmon et al., SC'11) keyed by the seed with
// counter (particle, step word, stream word, graph tag):
//   main stream  (p, n>>2, 0, tag): two Box-Muller pairs drive the first
//                sub-steps of steps 4m..4m+3 (cos, sin of pair A; cos, sin
//                of pair B), so one Philox call serves four steps;
//   hit stream   (p, n, k, tag): after the k-th vertex hit of step n, word 0
//                draws the slot and the cosine of pair (word 1, word 2)
//                drives the next sub-step;
//   init stream  (p, 0xFFFFFFFF, 0xFFFFFFFF, tag).
// The FP32 path consumes the same integers as the FP64 path.
//
// Compiled with -ffp-contract=off: every fused multiply-add is explicit.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

#include "mg_internal.h"

namespace mg {
namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;

// Main-stream Philox groups (four steps each) run before the parked lanes
// of a window resolve their vertex hits.
#ifndef MG_WINDOW_GROUPS32
#define MG_WINDOW_GROUPS32 1
#endif
#ifndef MG_WINDOW_GROUPS64
#define MG_WINDOW_GROUPS64 2
#endif
constexpr int kWindowGroups32 = MG_WINDOW_GROUPS32;
constexpr int kWindowGroups64 = MG_WINDOW_GROUPS64;
constexpr uint64_t kFnvPrime = 0x100000001b3ull;

#include "mg_bm64.inc"

struct U4 {
  uint32_t x, y, z, w;
};

// Three-input exclusive or in one gfx950 instruction (v_bitop3_b32 with
// truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Philox4x32-10: ten rounds of two 32x32->64 products (v_mad_u64_u32) and
// three-way xors, the key bumped by the Weyl increments before every round
// but the first.
__device__ __forceinline__ U4 philox(uint32_t c0, uint32_t c1, uint32_t c2,
                                     uint32_t c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
    const uint32_t t0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t t2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = t0;
    c2 = t2;
  }
  return {c0, c1, c2, c3};
}

// Keys of a Philox call in an FP64 kernel.  The FP64 polynomial constants
// fill the scalar registers there, so the round keys, which the compiler
// computes once outside the loops, are spilled to lanes of a vector
// register and read back with a readlane (a vector issue slot) per round.
// Hiding the two keys from the optimiser at the call keeps each Weyl
// increment next to its round, as a scalar add.  FP32 kernels keep their
// round keys in scalar registers and are left as they are.
template <class real>
__device__ __forceinline__ void fresh_keys(uint32_t &k0, uint32_t &k1) {
  if constexpr (sizeof(real) == 8) asm volatile("" : "+s"(k0), "+s"(k1));
}

// Main-stream Philox with the particle's share computed once.  The counter
// (p, g, 0, tag) differs between a particle's groups only in its second
// word, and its third word is zero, so of the first three rounds' six
// products three depend on the particle alone: those of round one (p and
// zero), one of round two (of a word that holds p and the tag) and one of
// round three.  A lane keeps the four words that later rounds read from them
// and a call takes 16 products instead of 20 (19 after the compiler has
// folded the zero).
struct MainCtr {
  uint32_t lo1, lo2, hi3, lo3;
};
__device__ __forceinline__ MainCtr main_ctr(uint32_t pid, uint32_t tag, uint32_t k0,
                                            uint32_t k1) {
  const uint64_t p1 = (uint64_t)0xD2511F53u * (uint64_t)pid;
  const uint32_t c2 = xor3((uint32_t)(p1 >> 32), tag, k1);
  const uint64_t p2 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
  const uint32_t c0 = (uint32_t)(p2 >> 32) ^ (k0 + 0x9E3779B9u);
  const uint64_t p3 = (uint64_t)0xD2511F53u * (uint64_t)c0;
  return {(uint32_t)p1, (uint32_t)p2, (uint32_t)(p3 >> 32), (uint32_t)p3};
}
__device__ __forceinline__ U4 philox_main(const MainCtr &m, uint32_t g, uint32_t k0,
                                          uint32_t k1) {
  uint32_t c0 = g ^ k0;  // round one
  k0 += 0x9E3779B9u;
  k1 += 0xBB67AE85u;
  const uint64_t p2 = (uint64_t)0xD2511F53u * (uint64_t)c0;  // round two
  uint32_t c2 = xor3((uint32_t)(p2 >> 32), m.lo1, k1);
  k0 += 0x9E3779B9u;
  k1 += 0xBB67AE85u;
  const uint64_t p3 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;  // round three
  c0 = xor3((uint32_t)(p3 >> 32), m.lo2, k0);
  c2 = xor3(m.hi3, (uint32_t)p2, k1);
  uint32_t c1 = (uint32_t)p3, c3 = m.lo3;
#pragma unroll
  for (int r = 3; r < 10; ++r) {
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
    const uint32_t t0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t t2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = t0;
    c2 = t2;
  }
  return {c0, c1, c2, c3};
}

// Square root of x in [2^-767, 2^1023) (normal, positive, finite): the
// hardware reciprocal square root y refined in Markstein's coupled form
// (g ~ sqrt(x) and h ~ 1/(2 sqrt(x)) updated together, then two residual
// corrections of g).  These are the device library's steps without its
// scaling of tiny arguments and its zero, infinity and NaN checks, which
// leave such arguments unchanged, so the root is the library's.  The
// Box-Muller radius argument -2 ln u lies in [2.3e-10, 44.4].
__device__ __forceinline__ double sqrt_normal(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y;
  double h = y * 0.5;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  double d = fma(-g, g, x);
  h = fma(h, r, h);
  g = fma(d, h, g);
  d = fma(-g, g, x);
  return fma(d, h, g);
}

// The tables of the FP64 Box-Muller in a block's LDS: {c, -2 log(1/c)} by the
// mantissa's interval; {cos a, sin a} and a by the 128th of a turn.
struct alignas(16) BmLds {
  double2 lg[128];
  double2 cs[129];
  double a[129];
};
__device__ __forceinline__ void stage_bm(BmLds *t) {
  for (int32_t i = threadIdx.x; i < 129; i += blockDim.x) {
    if (i < 128) t->lg[i] = make_double2(kLogTab[i][0], kLogTab[i][1]);
    t->cs[i] = make_double2(kTurnTab[i][0], kTurnTab[i][1]);
    t->a[i] = kTurnTab[i][2];
  }
}

// -2 ln u of the Box-Muller uniform u = (a + 1/2) 2^-32: u = 2^k m with m in
// [45/64, 45/32), m's interval of 128 gives c ~ 1/m, z = m c - 1 (one
// rounding) lies in [-2^-8, 2^-7), and -2 ln u = -2 (k ln 2 + ln(1/c)) - 2
// log1p(z) (the table-driven reduction of P. T. P. Tang, ACM TOMS 16, 1990, with
// reciprocals of its own), with log1p(z) = z + z^2 q(z), q the degree-5 minimax
// polynomial (error below 2^-59 of log1p; minimax_fit.py beside this file) and
// ln 2 in two parts, whose first, times k, adds to the table's constant exactly.
// c = 1 and no constant in the two intervals at 1, so the relative error stays
// small where the logarithm vanishes.  Within 0.753 ulp of every u above 0.9
// (below, 0.55) and 0.29 ulp rms on 4e6 draws; the worst draws lie in the two
// binades of the result next to those intervals, where the constant's error and
// z's rounding weigh most (1.06 ulp with constants chosen there as elsewhere).
// 14 FP64 operations and a table read; the series of atanh with a division that
// it replaces took 30 (0.80 ulp, 0.30 rms).
__device__ __forceinline__ double neg2log_unit(uint32_t a, const BmLds *t) {
  const uint64_t bits = (uint64_t)__double_as_longlong(fma((double)a, 0x1p-32, 0x1p-33));
  const uint32_t h = (uint32_t)(bits >> 32), d = h - 0x3fe68000u;
  const double2 lg = t->lg[(d >> 13) & 127u];
  const double k = (double)((int32_t)d >> 20);
  const double m = __longlong_as_double(
      (long long)(((uint64_t)(h - (d & 0xfff00000u)) << 32) | (bits & 0xffffffffull)));
  const double z = fma(m, lg.x, -1.0);
  double q = 0.13996369133691272;  // highest degree first
  q = fma(q, z, -0.16665110133186214);
  q = fma(q, z, 0.20000004212836844);
  q = fma(q, z, -0.2500000003871666);
  q = fma(q, z, 0.3333333333332643);
  q = fma(q, z, -0.4999999999999981);
  double r = fma(z * z, q, z);
  r = fma(k, 1.9082149292705877e-10, r);
  return fma(-2.0, r, fma(k, -1.3862943607382476, lg.y));
}

// Cosine and sine of the Box-Muller angle t = 2 pi u, u = (b + 1/2) 2^-32,
// rounded to FP64 as it stands: the nearest 128th of a turn comes from the
// integer; the table has an angle a close to it whose cosine and sine are
// doubles to within 2^-62 (Gal's accurate tables), x = t - a is exact, and
// the addition theorem takes sin x = x + x^3 s(x^2) and cos x - 1 = x^2
// c(x^2), minimax polynomials of degree 2 (errors below 2^-64 for |x| <=
// pi/128).  The results are rounded almost correctly.  17 FP64 operations
// and two table reads where quarter turns and polynomials of degree 5 took
// 23 and eight selects.
__device__ __forceinline__ void sincos_turn(uint32_t b, const BmLds *t, double &s_out,
                                            double &c_out) {
  const uint32_t i = ((b >> 24) + 1u) >> 1;  // 0 .. 128
  const double2 cs = t->cs[i];
  const double x = kTwoPi * fma((double)b, 0x1p-32, 0x1p-33) - t->a[i];
  const double x2 = x * x;
  double p = -0.0001984095097329375;  // s, highest degree first
  p = fma(p, x2, 0.008333333332219878);
  p = fma(p, x2, -0.16666666666666655);
  const double sx = fma(x * x2, p, x);
  double c = -0.0013888601908199634;  // c, highest degree first
  c = fma(c, x2, 0.0416666666566456);
  c = fma(c, x2, -0.499999999999999);
  c = c * x2;
  c_out = cs.x + fma(-cs.y, sx, cs.x * c);
  s_out = cs.y + fma(cs.x, sx, cs.y * c);
}

// Box-Muller in FP64: R = sqrt(-2 ln u1), angle 2 pi u2, u = (bits + 1/2)
// 2^-32.  Against exact values on 6e6 draws a normal is off by 2.434e-16 rms
// and 2.80e-15 at most, nearly all of it the rounding of the angle (2.459e-16
// and 2.87e-15 with a series for the logarithm and polynomials on a quarter
// turn; 2.429e-16 and 2.80e-15 with glibc's functions, whose normals it
// equals in 97 % of draws, against 82 %).  In place of those the 64-edge
// star takes 24.5 ms instead of 30.1 for 2000 steps of 4e6 particles at dt
// 1e-2, 18.0 instead of 22.2 at 1e-3, and the vascular network 14.7 instead
// of 18.9 for 1000 steps of 1e7: a group of four steps 190 VALU instructions
// instead of 232, at the price of six LDS reads per lane.
__device__ __forceinline__ void box_muller64(uint32_t a, uint32_t b, const BmLds *t, double &wc,
                                             double &ws) {
  const double r = sqrt_normal(neg2log_unit(a, t));
  double s, c;
  sincos_turn(b, t, s, c);
  wc = r * c;
  ws = r * s;
}

__device__ __forceinline__ double box_muller64_cos(uint32_t a, uint32_t b, const BmLds *t) {
  double s, c;
  sincos_turn(b, t, s, c);
  return sqrt_normal(neg2log_unit(a, t)) * c;
}

// Box-Muller in FP32 on the transcendental unit: v_log_f32 is log2 and
// v_sin_f32 / v_cos_f32 take their argument in turns (sin(2 pi t)).
__device__ __forceinline__ void box_muller32(uint32_t a, uint32_t b, float &wc,
                                             float &ws) {
  const float u1 = fmaf((float)a, 0x1p-32f, 0x1p-33f);
  const float u2 = fmaf((float)b, 0x1p-32f, 0x1p-33f);
  const float r =
      __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));
  wc = r * __builtin_amdgcn_cosf(u2);
  ws = r * __builtin_amdgcn_sinf(u2);
}

__device__ __forceinline__ float box_muller32_cos(uint32_t a, uint32_t b) {
  const float u1 = fmaf((float)a, 0x1p-32f, 0x1p-33f);
  const float u2 = fmaf((float)b, 0x1p-32f, 0x1p-33f);
  return __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1)) *
         __builtin_amdgcn_cosf(u2);
}

// Smallest u in (0, 1] with C + B u + A u^2 = 0 (C >= 0), u = sqrt(alpha):
// Alg. 2's crossing equation in the frame of the distance to the hit
// vertex; cancellation-free quadratic formula q = -(B + sgn(B) sqrt(disc))/2
// with roots q/A and C/q; C = 0 (on the vertex) gives -B/A, A = 0 gives
// -C/B; clamped to [0, 1].  The three cases are computed as one pair of
// divisions whose operands are selected, so no lane branches; in FP64 the
// divisions are IEEE-exact, which keeps the result bit-equal to the plain
// case-by-case evaluation.
__device__ __forceinline__ double first_root64(double A, double B, double Cc) {
  double disc = B * B - 4.0 * A * Cc;
  disc = disc < 0.0 ? 0.0 : disc;
  const double sq = sqrt(disc);
  const double q = -0.5 * (B >= 0.0 ? B + sq : B - sq);
  const bool c0 = Cc == 0.0, a0 = A == 0.0;
  // general: q / A and C / q;  C = 0: -B / A;  A = 0: -C / B
  const double n1 = c0 ? -B : (a0 ? -Cc : q);
  const double d1 = a0 ? B : A;
  const double d2 = (c0 || a0) ? 1.0 : q;
  const double r1 = n1 / d1;
  const double r2 = Cc / d2;
  const double lo = r1 < r2 ? r1 : r2;
  const double hi = r1 < r2 ? r2 : r1;
  double ug = lo > 0.0 ? lo : hi;
  ug = ug > 0.0 ? ug : 1.0;
  double u = (c0 || a0) ? r1 : ug;
  u = (c0 && a0) ? 0.0 : u;
  u = u >= 0.0 ? u : 0.0;  // also maps NaN to 0
  return u > 1.0 ? 1.0 : u;
}

// The same in FP32 with one hardware reciprocal (about one ulp).  In the
// general case the sign of B tells which root is the smallest positive one,
// so only that division is made: with C > 0 and real roots, B < 0 gives
// q > 0 and the root C/q, which is the smaller of two positive roots (A > 0;
// q^2 >= AC) or the positive one (A < 0); B >= 0 gives q <= 0, so C/q <= 0
// and q/A is positive exactly when A < 0.  A negative discriminant (only
// after rounding, next to a double root) is clamped to 0 and gives the
// double root q/A.  No positive root gives the whole sub-step, u = 1.  The
// result equals that of taking both divisions and the smallest positive.
__device__ __forceinline__ float first_root32(float A, float B, float Cc) {
  const float disc0 = fmaf(B, B, -4.0f * A * Cc);
  const bool real2 = disc0 > 0.0f;
  const float sq = __builtin_amdgcn_sqrtf(real2 ? disc0 : 0.0f);
  const bool bneg = B < 0.0f;
  const float q = -0.5f * (bneg ? B - sq : B + sq);
  const bool c0 = Cc == 0.0f, a0 = A == 0.0f;
  const bool cq = bneg & real2;
  // C = 0: -B / A;  A = 0: -C / B;  else C / q or q / A
  const float num = c0 ? -B : (a0 ? -Cc : (cq ? Cc : q));
  const float den = c0 ? A : (a0 ? B : (cq ? q : A));
  const float r = num * __builtin_amdgcn_rcpf(den);
  float u = (c0 || a0) ? r : (r > 0.0f ? r : 1.0f);
  u = (c0 && a0) ? 0.0f : u;
  u = u >= 0.0f ? u : 0.0f;
  return u > 1.0f ? 1.0f : u;
}

__device__ __forceinline__ uint64_t fnv(uint64_t h, uint32_t w) {
  return (h ^ (uint64_t)w) * kFnvPrime;
}

// Event trace: a vertex hit of a chosen particle (ids ascending in S.ev_ids)
// appends its record (step, hit index, vertex, slot or -1 when the particle
// is removed there, u = sqrt(alpha) and the time left after the hit); the
// counter counts every event, records past the capacity are dropped.  Only
// sets with trace call it.
__device__ void trace_hit(const SetDev &S, uint32_t pid, uint32_t step, int32_t k, int32_t v,
                          int32_t slot, double u, double h_after) {
  if (!S.ev) return;
  int32_t lo = 0, hi = S.ev_nids;
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (S.ev_ids[mid] < pid)
      lo = mid + 1;
    else
      hi = mid;
  }
  if (lo == S.ev_nids || S.ev_ids[lo] != pid) return;
  const unsigned long long i = atomicAdd(S.ev_cnt, 1ull);
  if (i < (unsigned long long)S.ev_cap) {
    mg_event &r = S.ev[i];
    r.pid = pid;
    r.step = step;
    r.k = k;
    r.vertex = v;
    r.slot = slot;
    r.reserved = 0;
    r.u = u;
    r.h_after = h_after;
  }
}

// Vertex stream of a Wentzell visit: word 0 of Philox (p, n, 0x100 + k, tag)
// decides the killing at the visit of the k-th hit of step n (k = 0: the
// visit at the start of a step that begins on the vertex).  Hit streams use
// k <= 255 in that word, so the two never share a counter.
__device__ __forceinline__ uint32_t vertex_draw(uint32_t pid, uint32_t step, uint32_t k,
                                                const SetDev &S, const StepArgs &A) {
  return philox(pid, step, 0x100u + k, S.tag, A.key0, A.key1).x;
}

// One visit of a Wentzell vertex (general gluing condition, Sec. 2.2; the
// scheme charges each visit its local time l = o + lt_per_sqrt sqrt(h''),
// the overshoot o of the proposal that crossed the vertex plus the mean
// local time of the move of length h'' that leaves it).  With h left in
// the step, the particle first stays on the vertex for gamma l and then
// moves for h'', where h'' + gamma (o + lt_per_sqrt sqrt(h'')) = h, a
// quadratic in sqrt(h'') solved in cancellation-free form; when gamma o >= h
// it stays for all of h and owes gamma o - h more.  The visit kills with
// probability 1 - exp(-kappa l), decided by the vertex-stream word `bits`
// as a uniform (bits + 1/2) 2^-32.  Returns true if the particle is killed;
// otherwise hm is the move's length (0: it stays for the rest of the step)
// and owed the stay still owed after this step.  FP64 throughout (both
// precisions; visits are rare).
__device__ __forceinline__ bool wz_visit(const WzRec &w, double o, double h, uint32_t bits,
                                         double &hm, double &owed) {
  double lt;
  owed = 0.0;
  if (w.gamma == 0.0) {
    hm = h;
    lt = o + w.lt_per_sqrt * sqrt(h);
  } else if (w.gamma * o >= h) {
    hm = 0.0;
    lt = o;
    owed = w.gamma * o - h;
  } else {
    const double b = w.gamma * w.lt_per_sqrt, r = h - w.gamma * o;
    const double sq = 2.0 * r / (b + sqrt(b * b + 4.0 * r));
    hm = sq * sq;
    lt = o + w.lt_per_sqrt * sq;
  }
  return w.kappa > 0.0 && ((double)bits + 0.5) * 0x1p-32 < -expm1(-w.kappa * lt);
}

// Graph tables as the step kernels see them: global memory, or LDS when the
// block staged them.
struct GView {
  const VtxBlk *vtx;
  const SlotRec8 *slots;
  const int32_t *guide;
  const EdgeRec32 *e32;
  const EdgeRec64 *e64;
  const EdgeHi32 *hi32;   // the FP32 path's higher coefficient terms
  const WzRec *wz;        // global Wentzell table
  const TabRec64 *tab64;  // global tabulated-coefficient intervals
  const TabRec32 *tab32;
  const BmLds *bm;        // FP64: the Box-Muller tables in LDS
};

__device__ __forceinline__ GView global_view(const GraphDev &G) {
  return {G.vtx, G.slots, G.guide, G.e32, G.e64, G.hi32, G.wz, G.tab64, G.tab32, nullptr};
}

struct SlotPick {
  int32_t s;    // global slot id
  uint32_t eo;  // edge << 1 | orient (bit 31: saturated threshold)
};

__device__ __forceinline__ int32_t eo_edge(uint32_t eo) { return (int32_t)((eo & 0x7FFFFFFFu) >> 1); }

// First slot k of the vertex with r < T_k (the last slot takes the rest):
// inline thresholds for degree <= 3, else the guide bucket of r and a short
// scan of the slot table.
__device__ __forceinline__ SlotPick pick_slot(const GView &g, const VtxBlk &vb, uint32_t r) {
  if (vb.deg <= 3) {
    int32_t k = 0;
    uint32_t eo = vb.eo0;
    if (vb.deg > 1 && !(r < vb.t0 || (vb.eo0 & kSatBit))) {
      k = 1;
      eo = vb.eo1;
      if (vb.deg > 2 && !(r < vb.t1 || (vb.eo1 & kSatBit))) {
        k = 2;
        eo = vb.eo2;
      }
    }
    return {vb.first + k, eo};
  }
  int32_t k = g.guide[vb.t0 + (r >> vb.t1)];
  SlotRec8 sr = g.slots[vb.first + k];
  while (k < vb.deg - 1 && !(r < sr.t || (sr.eo & kSatBit))) {
    ++k;
    sr = g.slots[vb.first + k];
  }
  return {vb.first + k, sr.eo};
}

// Per-lane tallies reduced once per block.  A lane of the lane schedule
// holds one particle for a launch of at most 2^20 steps and M <= 255, so
// each field stays below 2^20 (M + 1) = 2^28; the block adds them into
// 64-bit LDS totals.  A lane of the wave pools serves any number of
// particles, so the pools drain their lanes' tallies into the block totals
// periodically (drain_tally).
struct Tally {
  uint32_t trunc, sub, hits, steps;
};

template <bool LDS>
__device__ __forceinline__ void count_exit(uint32_t *s_exit, uint64_t *g_exit,
                                           int32_t slot) {
  if (LDS)
    atomicAdd(&s_exit[slot], 1u);
  else
    atomicAdd((unsigned long long *)&g_exit[slot], 1ull);
}

// Bin of position x on an edge binned over [0, span], nb bins per edge: x
// times the FP64 inverse bin width nb / span, rounded down, clamped to
// [0, nb - 1] (the appendix histogram kernel, with x = span and anything
// beyond in the last bin).
__device__ __forceinline__ int32_t bin_at(double x, double inv, int32_t nb) {
  const double f = floor(x * inv);
  return f < 0.0 ? 0 : (f > (double)(nb - 1) ? nb - 1 : (int32_t)f);
}
__device__ __forceinline__ int32_t bin_of(double x, double span, int32_t nb) {
  return bin_at(x, (double)nb / span, nb);
}

// Streamed histogram.  A snapshot adds every alive particle's bin at each
// step counter value that is a multiple of S.obs_every (the state after
// that many steps).  next_snapshot(n) is the first such value after n; 0
// (never reached: counters after a step are >= 1) when there is none below
// 2^32 or streaming is off.
__device__ __forceinline__ uint32_t next_snapshot(uint32_t n, const SetDev &S) {
  if (!S.obs) return 0u;
  const uint64_t v = ((uint64_t)(n / S.obs_every) + 1u) * S.obs_every;
  return v > 0xFFFFFFFFull ? 0u : (uint32_t)v;
}

// The snapshot count after one: multiples of S.obs_every follow each other
// (0 when the next would pass 2^32 - 1).
__device__ __forceinline__ uint32_t snapshot_after(uint32_t snap, const SetDev &S) {
  const uint32_t v = snap + S.obs_every;
  return v < snap ? 0u : v;
}

// Where snapshots go: LDS bins of the block (lds != null) or the set's
// global counters.  Bins are taken in FP64 from the set's table of edge
// lengths and inverse bin widths, made when streaming starts, and the next
// snapshot count waits in a particle's home slot, so no count costs a
// division (1e6 particles: the tracer's 2000 steps, a snapshot every 100, 6.9
// -> 6.1 ms with its readback; the 5-edge linear star, 1000 steps, every 50,
// 13.3 -> 11.7).
struct ObsSink {
  uint32_t *lds;
};

__device__ __forceinline__ void observe_at(int32_t e, double x, double inv, const SetDev &S,
                                           const ObsSink &o) {
  const int32_t idx = e * S.obs_nb + bin_at(x, inv, S.obs_nb);
  if (o.lds)
    atomicAdd(&o.lds[idx], 1u);
  else
    atomicAdd((unsigned long long *)&S.obs[idx], 1ull);
}
template <typename P>
__device__ __forceinline__ void observe(const P &q, const SetDev &S, const ObsSink &o) {
  const double2 r = S.obs_edge[q.e];
  observe_at(q.e, q.pos64(r.x), r.y, S, o);
}

// {length, inverse bin width} of every edge for a set's streamed histogram.
__global__ void k_obs_edges(const EdgeRec64 *e64, int32_t n_edges, int32_t nb, double2 *out) {
  const int32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n_edges) out[e] = make_double2(e64[e].L, (double)nb / e64[e].span);
}

template <typename T, int N>
__device__ __forceinline__ T pickw(const T (&W)[N], uint32_t j) {
  T w = W[0];
#pragma unroll
  for (int i = 1; i < N; ++i) w = (j == (uint32_t)i) ? W[i] : w;
  return w;
}

// Step loop shared by both precisions.  P is a per-lane particle (FP64 or
// FP32) with
//   bool fast(W)                    first sub-step of a step (h = dt); true if
//                                   it stays inside the edge (then applied);
//   void resolve(step, W, ...)      the rest of a step whose first sub-step
//                                   reached a vertex: splits, edge draws,
//                                   further sub-steps, exit record.
// Hits are not resolved where they happen: within one group of four steps
// (one main-stream Philox block) every lane first runs the cheap first
// sub-steps; a lane that reaches a vertex parks there; the parked lanes then
// resolve together and finish their group from the cached normals.  Each
// particle's arithmetic and random numbers are those of the plain order;
// the split code runs once per round for all parked lanes instead of once
// per step for any lane that hit.
template <int NG, bool OBS, typename P>
__device__ __forceinline__ void step_loop(P &q, const SetDev &S, const StepArgs &A,
                                          uint32_t pid, Tally &t, const ObsSink &o) {
  constexpr uint32_t NW = 4 * NG;  // steps per window
  const uint32_t n_end = S.n0 + A.nsteps;
  uint32_t n = S.n0;
  uint32_t snap = OBS ? next_snapshot(n, S) : 0u;
  // after each completed step (and the group-end re-anchoring)
  auto snapshot = [&](uint32_t done) {
    if (OBS && done == snap) {
      observe(q, S, o);
      snap = next_snapshot(done, S);
    }
  };
  while (n < n_end && q.alive) {
    const uint32_t base = n & ~(NW - 1);
    typename P::real W[NW];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      uint32_t k0 = A.key0, k1 = A.key1;
      fresh_keys<typename P::real>(k0, k1);
      const U4 o = philox(pid, (base >> 2) + g, 0u, S.tag, k0, k1);
      P::box_muller(o.x, o.y, q.G.bm, W[4 * g + 0], W[4 * g + 1]);
      P::box_muller(o.z, o.w, q.G.bm, W[4 * g + 2], W[4 * g + 3]);
    }
    const uint32_t jb = n - base;
    const uint32_t je = min(NW, n_end - base);
    // FP32: the window's normals stay in registers (every access has a
    // compile-time index; the normal of a parked step travels in wp).
    // FP64: the continuation after a hit indexes them at run time, which
    // keeps the eight doubles out of registers (measured faster: one more
    // wave per SIMD).
    int32_t pj = -1;
    typename P::real wp = 0;
    q.prep_window(W, jb);
#pragma unroll
    for (uint32_t j = 0; j < NW; ++j) {
      if (j < jb || j >= je || pj >= 0) continue;
      if (!q.fast_first(W[j])) {
        pj = (int32_t)j;
        wp = W[j];
      } else {
        if ((j & 3u) == 3u) q.reanchor();
        snapshot(base + j + 1u);
      }
    }
    while (pj >= 0) {
      const uint32_t j0 = (uint32_t)pj;
      q.resolve(base + j0, wp, pid, S, A, t);
      if (q.alive) {
        if ((j0 & 3u) == 3u) q.reanchor();
        snapshot(base + j0 + 1u);
      }
      pj = -1;
      if constexpr (sizeof(typename P::real) == 8) {
        for (uint32_t j = j0 + 1; j < je && q.alive; ++j) {
          const typename P::real wj = pickw(W, j);
          if (!q.fast(wj)) {
            pj = (int32_t)j;
            wp = wj;
            break;
          }
          if ((j & 3u) == 3u) q.reanchor();
          snapshot(base + j + 1u);
        }
      } else {
#pragma unroll
        for (uint32_t j = 1; j < NW; ++j) {
          if (j <= j0 || j >= je || !q.alive || pj >= 0) continue;
          if (!q.fast(W[j])) {
            pj = (int32_t)j;
            wp = W[j];
          } else {
            if ((j & 3u) == 3u) q.reanchor();
            snapshot(base + j + 1u);
          }
        }
      }
    }
    n = base + je;
  }
  // every step taken has one first sub-step; resolve() counts the others
  const uint32_t taken = q.alive ? A.nsteps : q.death_step + 1u - S.n0;
  t.steps += taken;
  t.sub += taken;
}

// ------------------------------------------------------------ FP64 path --
// Resolution state of an FP64 step whose sub-step proposal reached a vertex:
// the remaining time, the pending sub-step's normal (as drawn; a sub-step
// from a vertex folds it into the edge), the crossings so far and the last
// slot drawn.
struct Hit64 {
  double h, w;
  int32_t k, last;
};

// The canonical step in FP64, operation for operation.
template <bool TRACE, bool LDS, int GEN>
struct Particle64 {
  using real = double;
  GView G;
  uint32_t *s_exit;
  int32_t e;
  double x;
  EdgeRec64 R;
  bool alive;
  uint64_t hash;
  uint32_t nhit;
  uint32_t death_step;

  __device__ static void box_muller(uint32_t a, uint32_t b, const BmLds *t, double &c,
                                    double &s) {
    box_muller64(a, b, t, c, s);
  }

  // FP64 positions are always measured from the initial vertex.
  __device__ __forceinline__ void reanchor() {}
  __device__ __forceinline__ bool fast_first(double w) { return fast(w); }
  __device__ __forceinline__ double pos64(double) const { return x; }

  // Window preparation of the step loop: only a window's first active step
  // can start on a vertex (every step that stays inside an edge ends
  // strictly inside it), where the normal points into the edge.
  template <int N>
  __device__ __forceinline__ void prep_window(double (&W)[N], uint32_t jb) const {
    if (x == 0.0 || x == R.L) {
      const bool init = x == 0.0;
#pragma unroll
      for (int i = 0; i < N; ++i)
        W[i] = (jb == (uint32_t)i) ? (init ? fabs(W[i]) : -fabs(W[i])) : W[i];
    }
  }

  // Drift and diffusion at x: affine and constant, or with GEN the cubics
  // by Horner's rule (with zero higher terms these equal the affine values
  // exactly).
  // A tabulated edge (GEN): its interval at x (the last one at x = L) and
  // the local coordinate t = x K / L - j.
  __device__ __forceinline__ const TabRec64 &interval(double at, double &t) const {
    const double s = at * R.inv_h;
    // (also a row of the edge for a lane that has run past its vertex)
    const double j = fmin(fmax(floor(s), 0.0), (double)(R.tab_k - 1));
    t = s - j;
    return G.tab64[R.tab0 + (int32_t)j];
  }
  __device__ __forceinline__ double drift(double at) const {
    if (!GEN) return fma(R.c, at, R.a);
    if (GEN == kGenFull && R.tab_k) {
      double t;
      const TabRec64 &T = interval(at, t);
      return fma(fma(fma(T.mu[3], t, T.mu[2]), t, T.mu[1]), t, T.mu[0]);
    }
    return fma(fma(fma(R.c3, at, R.c2), at, R.c), at, R.a);
  }
  __device__ __forceinline__ double diffusion(double at) const {
    if (!GEN) return R.sigma;
    if (GEN == kGenFull && R.tab_k) {
      double t;
      const TabRec64 &T = interval(at, t);
      return fma(fma(fma(T.sg[3], t, T.sg[2]), t, T.sg[1]), t, T.sg[0]);
    }
    return fma(fma(fma(R.s3, at, R.s2), at, R.s1), at, R.sigma);
  }

  // GEN: the particle sits on a Wentzell vertex (x <= 0 at the initial
  // end, x >= L at the terminal one; a particle that owes a stay there
  // holds -t or L + t).  Its step starts with a visit, in resolve().
  __device__ __forceinline__ bool on_wentzell() const {
    if constexpr (GEN != kGenFull) return false;
    return (x <= 0.0 && ((uint32_t)R.vinit & kWentzellEnd)) ||
           (x >= R.L && ((uint32_t)R.vterm & kWentzellEnd));
  }

  __device__ __forceinline__ void die(int32_t v, uint32_t step, const SetDev &S) {
    alive = false;
    death_step = step;
    atomicAdd((unsigned long long *)&S.absorbed[v], 1ull);
    if (TRACE) hash = fnv(fnv(hash, step), 0x80000000u | (uint32_t)v);
  }

  __device__ __forceinline__ bool fast(double w) {
    if (on_wentzell()) return false;
    if (x == 0.0)
      w = fabs(w);
    else if (x == R.L)
      w = -fabs(w);
    const double mu = drift(x);
    const double g = diffusion(x) * sqrt(dtv);
    const double xt = fma(g, w, fma(mu, dtv, x));
    if (xt > 0.0 && xt < R.L) {
      x = xt;
      return true;
    }
    return false;
  }

  double dtv;
  double sqdt;  // sqrt(dtv)

  // One vertex crossing of a step whose pending sub-step proposal (normal
  // H.w over the remaining time H.h; the step's first sub-step when
  // H.k == 0) reached a vertex: crossing time, edge draw, and the next
  // sub-step's proposal.  Returns true when the step is complete (inside an
  // edge, absorbed, out of time or at the split cap), false when the next
  // proposal reaches a vertex again.  resolve() loops over it; the wave
  // pools run one crossing per lane per pass.  A step that starts on a
  // Wentzell vertex begins here with its visit.
  __device__ bool cross(uint32_t step, Hit64 &H, uint32_t pid, const SetDev &S,
                        const StepArgs &A, Tally &t) {
    double h = H.h;
    bool left_visit = false;  // the move that leaves a start-of-step visit
    if (H.k == 0 && on_wentzell()) {
      // a step that starts on a Wentzell vertex: the stay owed there first,
      // then the visit that leaves it (its own local time only, o = 0); a
      // step spent on the vertex, or ended by the visit's killing, has no
      // move (its one sub-step is counted with the step)
      const bool init = x <= 0.0;
      const int32_t v = (init ? R.vinit : R.vterm) & kVertexMask;
      double owe = init ? -x : x - R.L;
      if (owe >= h) {
        owe = owe - h;
        x = init ? -owe : R.L + owe;
        return true;
      }
      h = h - owe;
      x = init ? 0.0 : R.L;
      double hm, owed;
      if (wz_visit(G.wz[G.vtx[v].wz - 1u], 0.0, h, vertex_draw(pid, step, 0u, S, A), hm, owed)) {
        die(v, step, S);
        return true;
      }
      if (hm == 0.0) {
        x = init ? -owed : R.L + owed;
        return true;
      }
      h = hm;
      H.h = h;
      left_visit = true;
    }
    // the pending proposal, recomputed as it was made
    double w = H.w;
    if (x == 0.0)
      w = fabs(w);
    else if (x == R.L)
      w = -fabs(w);
    const double mu = drift(x);
    const double g = diffusion(x) * sqrt(h);
    const double xt = fma(g, w, fma(mu, h, x));
    bool done = false;
    if (left_visit && xt > 0.0 && xt < R.L) {
      x = xt;
      return true;
    }
    const bool at_init = xt <= 0.0;
    const int32_t vr = at_init ? R.vinit : R.vterm;
    // reflecting leaf: the mirror image ends the step if it lies inside
    // the edge
    const double xr = at_init ? -xt : 2.0 * R.L - xt;
    if (vr < 0 && xr > 0.0 && xr < R.L) {
      x = xr;
      done = true;
    } else {
      const int32_t v = vr & kVertexMask;
      const double d = at_init ? x : R.L - x;
      const double qa = at_init ? mu * h : -(mu * h);
      const double qb = at_init ? g * w : -(g * w);
      const double u = first_root64(qa, qb, d);
      const double alpha = u * u;
      h = fma(-alpha, h, h);
      ++H.k;
      ++nhit;
      t.hits++;
      const VtxBlk vb = G.vtx[v];
      // (drawn while the vertex block loads, for a removed particle too)
      uint32_t k0 = A.key0, k1 = A.key1;
      fresh_keys<double>(k0, k1);
      const U4 hd = philox(pid, step, (uint32_t)H.k, S.tag, k0, k1);
      // a Wentzell vertex: the visit this hit starts, its overshoot being
      // how far past the vertex the proposal went
      double h_move = h, owed = 0.0;
      bool killed = false;
      if (GEN == kGenFull && vb.wz) {
        const double o = at_init ? -xt : xt - R.L;
        killed = wz_visit(G.wz[vb.wz - 1u], o, h, vertex_draw(pid, step, (uint32_t)H.k, S, A),
                          h_move, owed);
      }
      if (vb.deg < 0 || killed) {  // absorbing vertex, or killed at the visit
        if (TRACE) trace_hit(S, pid, step, H.k, v, -1, u, h);
        die(v, step, S);
        return true;
      }
      const SlotPick sp = pick_slot(G, vb, hd.x);
      e = eo_edge(sp.eo);
      R = G.e64[e];
      x = (sp.eo & 1u) ? R.L : 0.0;
      H.last = sp.s;
      if (TRACE) {
        hash = fnv(fnv(hash, step), (uint32_t)sp.s);
        trace_hit(S, pid, step, H.k, v, sp.s, u, h);
      }
      if (GEN == kGenFull && vb.wz) {
        h = h_move;
        if (h == 0.0) {  // stays on the vertex for the rest of the step
          x = (sp.eo & 1u) ? R.L + owed : -owed;
          done = true;
        }
      }
      if (!done) done = h == 0.0;
      if (!done && H.k == A.max_splits) {
        t.trunc++;
        done = true;
      }
      if (!done) {
        // the next sub-step, from the vertex (normal folded into the edge)
        H.w = box_muller64_cos(hd.y, hd.z, G.bm);
        H.h = h;
        const double w2 = (sp.eo & 1u) ? -fabs(H.w) : fabs(H.w);
        const double mu2 = drift(x);
        const double g2 = diffusion(x) * sqrt(h);
        const double xt2 = fma(g2, w2, fma(mu2, h, x));
        t.sub++;
        if (xt2 > 0.0 && xt2 < R.L) {
          x = xt2;
          done = true;
        }
      }
    }
    if (done && H.k > 0) count_exit<LDS>(s_exit, S.exit_cnt, H.last);
    return done;
  }

  __device__ void resolve(uint32_t step, double w, uint32_t pid, const SetDev &S,
                          const StepArgs &A, Tally &t) {
    Hit64 H{dtv, w, 0, -1};
    while (!cross(step, H, pid, S, A, t)) {
    }
  }
};

template <bool TRACE, bool LDS, bool OBS, int NG, int GEN>
__device__ void run64(const GView &G, int32_t n_edges, const SetDev &S, const StepArgs &A,
                      uint32_t pid, uint32_t *s_exit, Tally &t, const ObsSink &o) {
  const uint32_t ef = S.ef[pid];
  if (ef & kDeadBit) return;
  const int32_t e = (int32_t)(ef & kEdgeMask);
  if (e >= n_edges) {
    atomicOr(S.err, kErrEdge);
    return;
  }
  Particle64<TRACE, LDS, GEN> q{G, s_exit, e, S.x64[pid], G.e64[e], true,
                           TRACE ? S.seqhash[pid] : 0ull, TRACE ? S.hits[pid] : 0u,
                           0u, A.dt, sqrt(A.dt)};
  if (!((q.x >= 0.0 && q.x <= q.R.L) || q.on_wentzell())) {
    atomicOr(S.err, kErrPos);
    return;
  }
  step_loop<NG, OBS>(q, S, A, pid, t, o);
  S.ef[pid] = (uint32_t)q.e | (q.alive ? 0u : kDeadBit);
  S.x64[pid] = q.x;
  if (TRACE) {
    S.seqhash[pid] = q.hash;
    S.hits[pid] = q.nhit;
  }
}

// ------------------------------------------------------------ FP32 path --
// Same step; the position is y = distance from the reference end (bit 30
// of the state word).  The reference end is re-chosen as the nearer end
// after every step that closes a Philox group (step index = 3 mod 4, in
// every schedule alike), so points near a vertex keep full relative
// precision.  In that
// frame the drift is as + c y with as = a (from the initial end) or
// -(a + c L) (from the terminal end), and the normal's sign flips with the
// end.  The position is a compensated pair (y, yl): each move adds its
// increment, computed at the increment's own magnitude, with the rounding
// error of the sum carried in yl (Fast2Sum, Dekker), so positions do not
// collect one rounding of y per step.  The remaining time is a compensated
// pair (hh, hl) too; the crossing solve runs in FP64 when the particle is
// within 1e-6 L of the vertex but not on it (on it the root is one
// division).
struct Edge32 {
  float L, a, c, sigma, aL;
  int32_t vinit, vterm;
};

__device__ __forceinline__ Edge32 load_edge32(const EdgeRec32 *e32, int32_t e) {
  const EdgeRec32 r = e32[e];
  return {r.L, r.a, r.c, r.sigma, r.aL, r.vinit, r.vterm};
}

// Resolution state of an FP32 step whose sub-step reached a vertex:
// remaining time (compensated pair), the pending sub-step's normal, the
// crossings so far and the last slot drawn.
struct Hit32 {
  float hh, hl, w;
  int32_t k, last;
};

// GEN: the graph has a general method variant.  Higher coefficient terms
// (cubic drift or diffusion): the first sub-step evaluates them at the
// particle's position instead of using the per-frame affine constants.
// Wentzell vertices: a step that starts on one begins with a visit (in
// cross()), and a hit there is a visit too; a particle that owes a stay on
// the vertex holds y = -t in the frame of that end.
template <bool TRACE, bool LDS, int GEN = 0>
struct Particle32 {
  using real = float;
  GView G;
  uint32_t *s_exit;
  int32_t e;
  uint32_t side;
  float y, yl;    // distance from the reference end, compensation term
  Edge32 R;
  float as, g0;   // drift constant in the local frame, sigma sqrt(dt)
  float dt, sqdt;
  bool alive;
  uint64_t hash;
  uint32_t nhit;
  uint32_t death_step;
  // First sub-step constants of the current edge and frame: c dt, as dt and
  // g0 with the frame's sign, so that a first sub-step is
  // y + fma(gs, w, fma(cd, y, ad)) with no per-step sign select.
  float cd = 0.0f, ad = 0.0f, gs = 0.0f;
  // Higher terms of the current edge (GEN), x from the initial vertex:
  // drift + c2 x^2 + c3 x^3, diffusion + s1 x + s2 x^2 + s3 x^3.
  float c2 = 0.0f, c3 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
  // A tabulated edge (GEN): intervals per unit length and the first
  // interval's row (tab_k = 0: no table).
  float inv_h = 0.0f;
  int32_t tab0 = 0, tab_k = 0;

  // Sets as, g0 and the first sub-step constants for the current edge R and
  // side (after an edge load or a change of reference end).
  __device__ __forceinline__ void frame() {
    as = side ? -R.aL : R.a;
    g0 = R.sigma * sqdt;
    cd = R.c * dt;
    ad = as * dt;
    gs = side ? -g0 : g0;
    if constexpr (GEN) {
      const EdgeHi32 P = G.hi32[e];
      c2 = P.c2;
      c3 = P.c3;
      s1 = P.s1;
      s2 = P.s2;
      s3 = P.s3;
      if constexpr (GEN == kGenFull) {
        inv_h = P.inv_h;
        tab0 = P.tab0;
        tab_k = P.tab_k;
      }
    }
  }

  // A tabulated edge's interval at x from the initial vertex (the last one
  // at x = L) and the local coordinate t.
  __device__ __forceinline__ const TabRec32 &interval(float x, float &t) const {
    const float s = x * inv_h;
    const float j = fminf(fmaxf(floorf(s), 0.0f), (float)(tab_k - 1));
    t = s - j;
    return G.tab32[tab0 + (int32_t)j];
  }

  // Drift in the frame (sign of the reference end) and diffusion at
  // distance yy from the reference end.
  __device__ __forceinline__ float fdrift(float yy) const {
    if constexpr (!GEN) {
      return fmaf(R.c, yy, as);
    } else {
      const float x = side ? R.L - yy : yy;
      float m;
      if (GEN == kGenFull && tab_k) {
        float t;
        const TabRec32 &T = interval(x, t);
        m = fmaf(fmaf(fmaf(T.mu[3], t, T.mu[2]), t, T.mu[1]), t, T.mu[0]);
      } else {
        m = fmaf(fmaf(fmaf(c3, x, c2), x, R.c), x, R.a);
      }
      return side ? -m : m;
    }
  }
  __device__ __forceinline__ float fsigma(float yy) const {
    if constexpr (!GEN) {
      return R.sigma;
    } else {
      const float x = side ? R.L - yy : yy;
      if (GEN == kGenFull && tab_k) {
        float t;
        const TabRec32 &T = interval(x, t);
        return fmaf(fmaf(fmaf(T.sg[3], t, T.sg[2]), t, T.sg[1]), t, T.sg[0]);
      }
      return fmaf(fmaf(fmaf(s3, x, s2), x, s1), x, R.sigma);
    }
  }

  __device__ static void box_muller(uint32_t a, uint32_t b, const BmLds *, float &c, float &s) {
    box_muller32(a, b, c, s);
  }

  // y + s as a compensated sum (Fast2Sum: exact error when |y| >= |s|,
  // a bounded one otherwise, which happens only within one step of the
  // reference end): returns the rounded sum, err its error.
  __device__ __forceinline__ float add_comp(float s, float &err) const {
    const float yt = y + s;
    err = s - (yt - y);
    return yt;
  }

  // Position from the initial vertex in FP64, as the histogram reads it.
  __device__ __forceinline__ double pos64(double L) const {
    const double v = (double)y + (double)yl;
    return side ? L - v : v;
  }

  // Re-anchor to the nearer end: L - y is exact for y in [L/2, L)
  // (Sterbenz), so the move loses nothing; the compensation flips sign.
  __device__ __forceinline__ void reanchor() {
    reanchor_if(true);
  }
  __device__ __forceinline__ void reanchor_if(bool cond) {
    const bool flip = cond & (y > 0.5f * R.L);
    y = flip ? R.L - y : y;
    yl = flip ? -yl : yl;
    side ^= flip ? 1u : 0u;
    as = flip ? (side ? -R.aL : R.a) : as;
    ad = flip ? as * dt : ad;
    gs = flip ? -gs : gs;
  }

  // GEN: the particle sits on a Wentzell vertex, its reference end (y <= 0:
  // on the vertex, or owing a stay of -y there).
  __device__ __forceinline__ bool on_wentzell() const {
    if constexpr (GEN != kGenFull) return false;
    return y <= 0.0f && ((uint32_t)(side ? R.vterm : R.vinit) & kWentzellEnd);
  }
  // The particle stays on its reference end, a Wentzell vertex, owing a
  // further stay of t there (y = -t as a compensated pair).
  __device__ __forceinline__ void owe_stay(double t) {
    const double yd = -t;
    y = (float)yd;
    yl = (float)(yd - (double)y);
  }
  __device__ __forceinline__ void die(int32_t v, uint32_t step, const SetDev &S) {
    alive = false;
    death_step = step;
    atomicAdd((unsigned long long *)&S.absorbed[v], 1ull);
    if (TRACE) hash = fnv(fnv(hash, step), 0x80000000u | (uint32_t)v);
  }

  // The normal a first sub-step from y = 0 uses: a particle on a vertex
  // moves into its edge, so the noise term is g0 |w| (gs carries the frame's
  // sign, hence |w| with that sign).
  __device__ __forceinline__ float at_vertex(float w) const {
    return copysignf(fabsf(w), gs);
  }
  // A step's first sub-step over dt with normal w; w must already be
  // at_vertex(w) when y = 0.  Returns the proposal and its compensation.
  __device__ __forceinline__ float propose(float w, float &err) const {
    if constexpr (!GEN) {
      return add_comp(fmaf(gs, w, fmaf(cd, y, ad)) + yl, err);
    } else {
      const float sg = fsigma(y) * sqdt;
      return add_comp(fmaf(side ? -sg : sg, w, fdrift(y) * dt) + yl, err);
    }
  }

  // Window preparation of the step loop: the first active step of a window
  // is the only one that can start on a vertex.
  template <int N>
  __device__ __forceinline__ void prep_window(float (&W)[N], uint32_t jb) const {
    if (y == 0.0f) {
#pragma unroll
      for (int i = 0; i < N; ++i) W[i] = (jb == (uint32_t)i) ? at_vertex(W[i]) : W[i];
    }
  }
  // First sub-step of a window's first active step after prep_window.
  __device__ __forceinline__ bool fast_first(float w) {
    if (on_wentzell()) return false;
    float err;
    const float yt = propose(w, err);
    if (yt > 0.0f && yt < R.L) {
      y = yt;
      yl = err;
      return true;
    }
    return false;
  }

  __device__ __forceinline__ bool fast(float w) {
    if (on_wentzell()) return false;
    float err;
    const float yt = propose((y == 0.0f) ? at_vertex(w) : w, err);
    if (yt > 0.0f && yt < R.L) {
      y = yt;
      yl = err;
      return true;
    }
    return false;
  }

  // One vertex crossing of a step whose current sub-step proposal (normal
  // h.w over the remaining time h.hh + h.hl; the step's first sub-step when
  // h.k == 0) reached a vertex: crossing time, edge draw, and the next
  // sub-step's proposal.  Returns true when the step is complete (inside an
  // edge, absorbed, out of time or at the split cap), false when the next
  // proposal reaches a vertex again.  resolve() loops over it; the wave
  // pools run one crossing per lane per pass.
  __device__ bool cross(uint32_t step, Hit32 &h, uint32_t pid, const SetDev &S,
                        const StepArgs &A, Tally &t) {
    float hh = h.hh, hl = h.hl;
    // the pending sub-step is the step's first, over dt (else over hh + hl)
    bool first = h.k == 0;
    if (first && on_wentzell()) {
      // a step that starts on a Wentzell vertex: the stay owed there first,
      // then the visit that leaves it (o = 0); a step spent on the vertex,
      // or ended by the visit's killing, has no move
      const int32_t v = (side ? R.vterm : R.vinit) & kVertexMask;
      double hd = (double)hh + (double)hl;
      const double owe = -((double)y + (double)yl);
      if (owe >= hd) {
        owe_stay(owe - hd);
        return true;
      }
      hd = hd - owe;
      y = 0.0f;
      yl = 0.0f;
      double hm, owed;
      if (wz_visit(G.wz[G.vtx[v].wz - 1u], 0.0, hd, vertex_draw(pid, step, 0u, S, A), hm,
                   owed)) {
        die(v, step, S);
        return true;
      }
      if (hm == 0.0) {
        owe_stay(owed);
        return true;
      }
      hh = (float)hm;
      hl = (float)(hm - (double)hh);
      h.hh = hh;
      h.hl = hl;
      first = false;
    }
    // the pending proposal, recomputed as it was made
    // (the first sub-step's exactly as propose() made it: g0 we = gs w)
    const float we = (y == 0.0f) ? fabsf(h.w) : (side ? -h.w : h.w);
    const float mu = fdrift(y);
    const float g = first ? (GEN ? fsigma(y) * sqdt : g0)
                          : fsigma(y) * __builtin_amdgcn_sqrtf(hh);
    const float mdt = first ? (GEN ? mu * dt : fmaf(cd, y, ad)) : mu * hh;
    float err;
    const float yt = add_comp(fmaf(g, we, mdt) + yl, err);
    // the move that leaves a start-of-step visit need not reach a vertex
    if (GEN == kGenFull && h.k == 0 && !first && yt > 0.0f && yt < R.L) {
      y = yt;
      yl = err;
      return true;
    }
    const bool near = yt <= 0.0f;
    const bool at_term = near == (side != 0u);
    const int32_t vr = at_term ? R.vterm : R.vinit;
    // reflecting leaf: the mirror image, as a distance from the hit end
    // (-(yt + err) at the reference end; (yt - L) + err at the other, where
    // yt - L is exact for yt <= 2L), renormalised by TwoSum; it ends the
    // step when it lies inside the edge
    const float r0 = near ? -yt : yt - R.L;
    const float r1 = near ? -err : err;
    const float rs = r0 + r1;
    const float rb = rs - r0;
    const float re = (r0 - (rs - rb)) + (r1 - rb);
    bool done;
    if (vr < 0 && rs > 0.0f && rs < R.L) {
      y = rs;
      yl = re;
      if (!near) {
        side ^= 1u;
        frame();
      }
      done = true;
    } else {
      const int32_t v = vr & kVertexMask;
      const float dn = y + yl;
      const float d = fmaxf(near ? dn : (R.L - y) - yl, 0.0f);
      float u;
      if (d > 0.0f && d < G.e32[e].near) {
        // crossing solve in FP64 next to the vertex (on the vertex itself,
        // d = 0, the root is -B/A: one division, no cancellation)
        const double hd = (double)hh + (double)hl;
        const double mud = GEN ? (double)mu : fma((double)R.c, (double)y, (double)as);
        const double gd = (double)fsigma(y) * sqrt(hd);
        const double qa = near ? mud * hd : -(mud * hd);
        const double qb = near ? gd * (double)we : -(gd * (double)we);
        const double yd = (double)y + (double)yl;
        const double dd = fmax(near ? yd : (double)R.L - yd, 0.0);
        u = (float)first_root64(qa, qb, dd);
      } else {
        const float gw = g * we;
        u = first_root32(near ? mdt : -mdt, near ? gw : -gw, d);
      }
      // remaining time (1 - u^2)(hh + hl), compensated (TwoProduct by fma,
      // TwoSum, renormalised)
      {
        const float al = u * u;
        const float p = al * hh;
        const float pe = fmaf(al, hh, -p);
        const float s = hh - p;
        const float bb = s - hh;
        const float se = (hh - (s - bb)) + (-p - bb);
        const float lo = ((se - pe) + hl) - al * hl;
        hh = s + lo;
        hl = lo - (hh - s);
      }
      h.hh = hh;
      h.hl = hl;
      ++h.k;
      ++nhit;
      t.hits++;
      const VtxBlk vb = G.vtx[v];
      // (drawn while the vertex block loads, for a removed particle too)
      const U4 hd = philox(pid, step, (uint32_t)h.k, S.tag, A.key0, A.key1);
      // a Wentzell vertex: the visit this hit starts, with the proposal's
      // overshoot past the vertex
      double hm = 0.0, owed = 0.0;
      bool killed = false;
      if (GEN == kGenFull && vb.wz)
        killed = wz_visit(G.wz[vb.wz - 1u], (double)r0 + (double)r1,
                          (double)hh + (double)hl, vertex_draw(pid, step, (uint32_t)h.k, S, A),
                          hm, owed);
      if (vb.deg < 0 || killed) {
        if (TRACE) trace_hit(S, pid, step, h.k, v, -1, u, (double)hh + (double)hl);
        die(v, step, S);
        return true;
      }
      const SlotPick sp = pick_slot(G, vb, hd.x);
      e = eo_edge(sp.eo);
      R = load_edge32(G.e32, e);
      side = sp.eo & 1u;
      y = 0.0f;
      yl = 0.0f;
      frame();
      h.last = sp.s;
      if (TRACE) {
        hash = fnv(fnv(hash, step), (uint32_t)sp.s);
        trace_hit(S, pid, step, h.k, v, sp.s, u, (double)hh + (double)hl);
      }
      bool stays = false;
      if (GEN == kGenFull && vb.wz) {
        if (hm == 0.0) {  // stays on the vertex for the rest of the step
          owe_stay(owed);
          stays = true;
        } else {
          hh = (float)hm;
          hl = (float)(hm - (double)hh);
          h.hh = hh;
          h.hl = hl;
        }
      }
      done = stays || hh == 0.0f;
      if (!done && h.k == A.max_splits) {
        t.trunc++;
        done = true;
      }
      if (!done) {
        // the next sub-step, from the vertex (normal folded into the edge)
        h.w = box_muller32_cos(hd.y, hd.z);
        const float mu2 = fdrift(y);
        const float g2 = fsigma(y) * __builtin_amdgcn_sqrtf(hh);
        float err2;
        const float yt2 = add_comp(fmaf(g2, fabsf(h.w), mu2 * hh) + yl, err2);
        t.sub++;
        if (yt2 > 0.0f && yt2 < R.L) {
          y = yt2;
          yl = err2;
          done = true;
        }
      }
    }
    if (done && h.k > 0) count_exit<LDS>(s_exit, S.exit_cnt, h.last);
    return done;
  }

  __device__ void resolve(uint32_t step, float w, uint32_t pid, const SetDev &S,
                          const StepArgs &A, Tally &t) {
    Hit32 h{dt, 0.0f, w, 0, -1};
    while (!cross(step, h, pid, S, A, t)) {
    }
  }
};

template <bool TRACE, bool LDS, bool OBS, int NG, int GEN>
__device__ void run32(const GView &G, int32_t n_edges, const SetDev &S, const StepArgs &A,
                      uint32_t pid, uint32_t *s_exit, Tally &t, const ObsSink &o) {
  const uint32_t ef = S.ef[pid];
  if (ef & kDeadBit) return;
  const int32_t e = (int32_t)(ef & kEdgeMask);
  if (e >= n_edges) {
    atomicOr(S.err, kErrEdge);
    return;
  }
  const float sqdt = (float)sqrt(A.dt);
  const Edge32 R = load_edge32(G.e32, e);
  const uint32_t side = (ef & kSideBit) ? 1u : 0u;
  const float2 yy = S.y32[pid];
  Particle32<TRACE, LDS, GEN> q{G, s_exit, e, side, yy.x, yy.y, R,
                           side ? -R.aL : R.a, R.sigma * sqdt, (float)A.dt, sqdt, true,
                           TRACE ? S.seqhash[pid] : 0ull, TRACE ? S.hits[pid] : 0u, 0u};
  q.frame();
  if (!((q.y >= 0.0f && q.y <= R.L) || q.on_wentzell())) {
    atomicOr(S.err, kErrPos);
    return;
  }
  step_loop<NG, OBS>(q, S, A, pid, t, o);
  S.ef[pid] = (uint32_t)q.e | (q.side ? kSideBit : 0u) | (q.alive ? 0u : kDeadBit);
  S.y32[pid] = make_float2(q.y, q.yl);
  if (TRACE) {
    S.seqhash[pid] = q.hash;
    S.hits[pid] = q.nhit;
  }
}

// Block-level reduction of the lane tallies (into the 64-bit LDS totals,
// to which the wave pools' periodic drains have already added) and the LDS
// exit counters.
__device__ __forceinline__ void flush(const SetDev &S, const Tally &t,
                                      unsigned long long *s_tot, uint32_t *s_exit,
                                      int32_t nnz, bool lds) {
  if (t.trunc) atomicAdd(&s_tot[0], (unsigned long long)t.trunc);
  if (t.sub) atomicAdd(&s_tot[1], (unsigned long long)t.sub);
  if (t.hits) atomicAdd(&s_tot[2], (unsigned long long)t.hits);
  if (t.steps) atomicAdd(&s_tot[3], (unsigned long long)t.steps);
  __syncthreads();
  if (threadIdx.x < 4 && s_tot[threadIdx.x])
    atomicAdd((unsigned long long *)&S.totals[threadIdx.x], s_tot[threadIdx.x]);
  if (lds) {
    for (int32_t s = threadIdx.x; s < nnz; s += blockDim.x)
      if (s_exit[s]) atomicAdd((unsigned long long *)&S.exit_cnt[s],
                               (unsigned long long)s_exit[s]);
  }
}

// Adds a block's LDS snapshot bins to the set's counters (after the
// barrier in flush()).
__device__ __forceinline__ void flush_obs(const SetDev &S, const uint32_t *s_obs,
                                          int32_t nbins) {
  for (int32_t b = threadIdx.x; b < nbins; b += blockDim.x)
    if (s_obs[b]) atomicAdd((unsigned long long *)&S.obs[b], (unsigned long long)s_obs[b]);
}

__device__ __forceinline__ int32_t align16(int32_t v) { return (v + 15) & ~15; }

// Shared memory of a step block: [FP64: Box-Muller tables][exit counters
// (LDS)][staged tables][snapshot bins (LDS)].
// Staged tables keep their relative layout: vertex blocks, slot table and
// guide tables, then the edge records of the kernel's precision; on graphs of
// the general levels the higher terms and tabulated intervals follow, if the
// host found that all of them fit (each step evaluates them: from global
// memory a load of L2 latency per step and coefficient).  1000 steps, 8
// tabulated edges of 16 intervals, 1e4 particles 2.94 -> 1.67 ms in FP32 and
// 3.25 -> 1.64 in FP64, 2e5 3.37 -> 2.41 and 4.08 -> 2.87; 64 cubic edges,
// 1e4 particles in FP32 0.75 -> 0.51 (with the pools spread over more waves,
// which is most of it where the tables do not fit: 200 tabulated edges, 1e4
// particles in FP64 5.41 -> 2.84).
template <bool FP64, bool STAGED, int GEN>
__device__ __forceinline__ GView block_view(const GraphDev &G, char *smem) {
  if (!STAGED) return global_view(G);
  const int32_t x = GEN ? (FP64 ? G.x_bytes64 : G.x_bytes32) : 0;
  const int32_t bytes = (FP64 ? G.stage_bytes64 - G.x_bytes64 : G.stage_bytes32 - G.x_bytes32);
  const int32_t head = G.o_e32;
  const uint4 *src_head = (const uint4 *)G.tables;
  const uint4 *src_edge = (const uint4 *)(G.tables + (FP64 ? G.o_e64 : G.o_e32));
  uint4 *dst = (uint4 *)smem;
  for (int32_t i = threadIdx.x; i < head / 16; i += blockDim.x) dst[i] = src_head[i];
  for (int32_t i = threadIdx.x; i < (bytes - head) / 16; i += blockDim.x)
    dst[head / 16 + i] = src_edge[i];
  GView v;
  v.vtx = (const VtxBlk *)(smem + G.o_vtx);
  v.slots = (const SlotRec8 *)(smem + G.o_slots);
  v.guide = (const int32_t *)(smem + G.o_guide);
  v.e32 = (const EdgeRec32 *)(smem + head);
  v.e64 = (const EdgeRec64 *)(smem + head);
  v.hi32 = G.hi32;
  v.wz = G.wz;
  v.tab64 = G.tab64;
  v.tab32 = G.tab32;
  v.bm = nullptr;
  if (GEN && x) {
    const uint4 *src = FP64 ? (const uint4 *)G.tab64 : (const uint4 *)G.hi32;
    uint4 *to = dst + bytes / 16;
    for (int32_t i = threadIdx.x; i < x / 16; i += blockDim.x) to[i] = src[i];
    if (FP64) {
      v.tab64 = (const TabRec64 *)to;
    } else {
      v.hi32 = (const EdgeHi32 *)to;
      v.tab32 = (const TabRec32 *)((const EdgeHi32 *)to + G.E);
    }
  }
  return v;
}

__device__ __forceinline__ int32_t exit_bytes(int32_t nnz) { return ((nnz * 4) + 15) & ~15; }

template <bool FP64, bool TRACE, bool LDS, bool STAGED, bool OBS, int GEN>
__device__ __forceinline__ void step_block(const GraphDev &G, const SetDev &S,
                                           const StepArgs &A, uint32_t pid,
                                           unsigned long long *s_tot, char *smem) {
  BmLds *bm = (BmLds *)smem;
  if (FP64) {
    stage_bm(bm);
    smem += sizeof(BmLds);
  }
  uint32_t *s_exit = (uint32_t *)smem;
  if (threadIdx.x < 4) s_tot[threadIdx.x] = 0;
  if (LDS)
    for (int32_t s = threadIdx.x; s < G.nnz; s += blockDim.x) s_exit[s] = 0;
  const int32_t ex = LDS ? exit_bytes(G.nnz) : 0;
  GView view = block_view<FP64, STAGED, GEN>(G, smem + ex);
  if (FP64) view.bm = bm;
  ObsSink o{nullptr};
  if (OBS && A.obs_lds) {
    o.lds = (uint32_t *)(smem + align16(ex + (STAGED ? (FP64 ? G.stage_bytes64
                                                             : G.stage_bytes32) : 0)));
    for (int32_t b = threadIdx.x; b < A.obs_lds; b += blockDim.x) o.lds[b] = 0;
  }
  __syncthreads();
  Tally t{0, 0, 0, 0};
  if (pid < S.n) {
    if (FP64)
      run64<TRACE, LDS, OBS, kWindowGroups64, GEN>(view, G.E, S, A, pid, s_exit, t, o);
    else
      run32<TRACE, LDS, OBS, kWindowGroups32, GEN>(view, G.E, S, A, pid, s_exit, t, o);
  }
  flush(S, t, s_tot, s_exit, G.nnz, LDS);
  if (OBS && A.obs_lds) flush_obs(S, o.lds, A.obs_lds);
}

// GEN: the method-variant level of the graph (GraphDev::gen).
template <bool FP64, bool TRACE, bool LDS, bool STAGED, bool OBS, int GEN>
__global__ __launch_bounds__(kBlock) void k_step(GraphDev G, SetDev S, StepArgs A) {
  extern __shared__ uint4 smem4[];
  __shared__ unsigned long long s_tot[4];
  step_block<FP64, TRACE, LDS, STAGED, OBS, GEN>(G, S, A, blockIdx.x * kBlock + threadIdx.x,
                                                  s_tot, (char *)smem4);
}

template <bool FP64, bool TRACE, bool LDS, bool STAGED, bool OBS, int GEN>
__global__ __launch_bounds__(kBlock) void k_batch(const GraphDev *graphs,
                                                  const SetDev *sets,
                                                  const BatchItem *items,
                                                  StepArgs A) {
  extern __shared__ uint4 smem4[];
  __shared__ unsigned long long s_tot[4];
  const BatchItem it = items[blockIdx.x];
  SetDev S = sets[it.set];
  S.n0 += A.n0_offset;  // steps already taken by earlier launches of this call
  const GraphDev G = graphs[it.set];
  step_block<FP64, TRACE, LDS, STAGED, OBS, GEN>(G, S, A, it.first + threadIdx.x, s_tot,
                                                  (char *)smem4);
}

// ------------------------------------------------ FP32 wave-pool kernel --
// Each wave owns PW particles (128 or 256; fewer where the set is small): 64
// ride in the lanes, the others wait in the wave's private LDS home slots.
// The lanes run their particles' first sub-steps in groups of four (one
// main-stream Philox block) until enough of them wait for another particle;
// a particle whose sub-step reaches a vertex is parked: its state
// goes to its home slot and its slot id onto the wave's split queue, and the
// lane takes a ready particle instead.  When 64 particles are parked (or
// lanes would idle), one split pass takes them with every lane busy and
// resolves one vertex crossing each: crossing time, Philox hit stream, slot
// draw and the next sub-step's proposal.  A particle whose step is then
// complete goes back on the ready queue (with its exit record); one whose
// proposal reaches a vertex again goes back on the split queue, so a pass
// never waits for the lane with the most crossings.  Each particle still
// consumes exactly the random numbers of its own (step, hit) counters, so the
// results equal the plain per-particle order bit for bit.  Waves never wait
// for one another: the queues and their counters are private to a wave.
constexpr int kWavesPerBlock = kBlock / 64;
#ifndef MG_POOL_CLAIM_MIN
#define MG_POOL_CLAIM_MIN 16
#endif
constexpr int kClaimMin = MG_POOL_CLAIM_MIN;  // free home slots that start a claim
static_assert((kClaimMin & (kClaimMin - 1)) == 0 && kClaimMin <= 64, "claim granularity");
// A batch work item stands for kBatchGens pools' worth of one set's
// particles per wave of a block: the number of items of a set, and so the
// number of blocks that may work on it at once, grows with its size.
constexpr int kBatchGens = 8;

template <bool TRACE, int PW>
struct PoolTrace {
  uint32_t hits[PW];
  uint64_t hash[PW];
};
template <int PW>
struct PoolTrace<false, PW> {};

// A wave's pool in LDS: home slots of its particles, the resolution state
// of parked steps, and the ready and split queues (slot ids).
template <bool TRACE, int PW>
struct PoolLds32 : PoolTrace<TRACE, PW> {
  static_assert(PW % 64 == 0 && PW <= 256, "slot ids are bytes");
  uint32_t ef[PW];
  float y[PW];
  float yl[PW];
  uint32_t n[PW];   // next step (ready) or the step to resolve (parked)
  float w[PW];      // normal of a parked step's pending sub-step
  float hh[PW];     // remaining time of a parked step (when k > 0)
  float hl[PW];
  int32_t last[PW]; // last slot drawn in the parked step
  uint32_t pid[PW];   // particle held by each home slot
  uint8_t k[PW];    // crossings so far in the parked step, else 0
  uint8_t ready[PW];
  uint8_t split[PW];
  uint8_t freeq[PW];  // home slots without a particle
};

// The same for FP64 particles: position from the initial vertex, and the
// parked step's normal and remaining time in FP64.
template <bool TRACE, int PW>
struct PoolLds64 : PoolTrace<TRACE, PW> {
  static_assert(PW % 64 == 0 && PW <= 256, "slot ids are bytes");
  uint32_t ef[PW];
  uint32_t n[PW];
  double x[PW];
  double w[PW];
  double h[PW];
  int32_t last[PW];
  uint32_t pid[PW];
  uint8_t k[PW];
  uint8_t ready[PW];
  uint8_t split[PW];
  uint8_t freeq[PW];
};

// The lanes of the wave where c holds, and whether a lane is in a mask.  The
// wave pools keep their lane masks as 64-bit values, combined in the scalar
// unit: a ballot of a plain comparison is the comparison, whereas a
// combination of conditions, and HIP's __ballot of an int, go through a
// vector register and a second comparison.
__device__ __forceinline__ uint64_t ballot(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ bool in_mask(uint64_t m) {
  return __builtin_amdgcn_inverse_ballot_w64(m);
}

// A pool's LDS: with streaming, each home slot also keeps its particle's
// next snapshot count.
template <class Pool, int PW>
struct PoolObs : Pool {
  uint32_t snap[PW];
};
template <int PW, bool FP64, bool TRACE, bool OBS>
using PoolPlain = std::conditional_t<FP64, PoolLds64<TRACE, PW>, PoolLds32<TRACE, PW>>;
template <int PW, bool FP64, bool TRACE, bool OBS>
using PoolLds = std::conditional_t<OBS, PoolObs<PoolPlain<PW, FP64, TRACE, OBS>, PW>,
                                   PoolPlain<PW, FP64, TRACE, OBS>>;
template <int PW, bool FP64, bool TRACE>
size_t pool_lds_bytes(bool obs) {
  return obs ? sizeof(PoolLds<PW, FP64, TRACE, true>) : sizeof(PoolLds<PW, FP64, TRACE, false>);
}

__device__ __forceinline__ uint32_t lane_rank(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// A wave's LDS instructions execute in issue order, so lanes of one wave
// may exchange data through LDS without waiting; only the compiler must not
// move the accesses across each other.
__device__ __forceinline__ void wave_lds_fence() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

// Moving particles between registers, the pool's home slots and the set:
// one overload per precision.
template <bool TRACE, bool LDS, int GEN, int PW>
__device__ __forceinline__ void pool_load(Particle32<TRACE, LDS, GEN> &q,
                                          const PoolLds32<TRACE, PW> &P,
                                          uint32_t s) {
  const uint32_t ef = P.ef[s];
  q.e = (int32_t)(ef & kEdgeMask);
  q.side = (ef & kSideBit) ? 1u : 0u;
  q.y = P.y[s];
  q.yl = P.yl[s];
  q.R = load_edge32(q.G.e32, q.e);
  q.frame();
  q.alive = true;
  if constexpr (TRACE) {
    q.nhit = P.hits[s];
    q.hash = P.hash[s];
  }
}
template <bool TRACE, bool LDS, int GEN, int PW>
__device__ __forceinline__ void pool_load(Particle64<TRACE, LDS, GEN> &q,
                                          const PoolLds64<TRACE, PW> &P,
                                          uint32_t s) {
  q.e = (int32_t)(P.ef[s] & kEdgeMask);
  q.x = P.x[s];
  q.R = q.G.e64[q.e];
  q.alive = true;
  if constexpr (TRACE) {
    q.nhit = P.hits[s];
    q.hash = P.hash[s];
  }
}

template <bool TRACE, bool LDS, int GEN, int PW>
__device__ __forceinline__ void pool_store(const Particle32<TRACE, LDS, GEN> &q,
                                           PoolLds32<TRACE, PW> &P,
                                           uint32_t s, uint32_t n) {
  P.ef[s] = (uint32_t)q.e | (q.side ? kSideBit : 0u);
  P.y[s] = q.y;
  P.yl[s] = q.yl;
  P.n[s] = n;
  if constexpr (TRACE) {
    P.hits[s] = q.nhit;
    P.hash[s] = q.hash;
  }
}
template <bool TRACE, bool LDS, int GEN, int PW>
__device__ __forceinline__ void pool_store(const Particle64<TRACE, LDS, GEN> &q,
                                           PoolLds64<TRACE, PW> &P,
                                           uint32_t s, uint32_t n) {
  P.ef[s] = (uint32_t)q.e;
  P.x[s] = q.x;
  P.n[s] = n;
  if constexpr (TRACE) {
    P.hits[s] = q.nhit;
    P.hash[s] = q.hash;
  }
}

// A parked step's resolution state, to and from its home slot (a fresh
// park, k = 0, has the whole step left: dt, no slot drawn yet).
template <bool TRACE, int PW>
__device__ __forceinline__ Hit32 pool_hit(const PoolLds32<TRACE, PW> &P, uint32_t s,
                                          const StepArgs &A) {
  Hit32 h{(float)A.dt, 0.0f, P.w[s], (int32_t)P.k[s], -1};
  if (h.k > 0) {
    h.hh = P.hh[s];
    h.hl = P.hl[s];
    h.last = P.last[s];
  }
  return h;
}
template <bool TRACE, int PW>
__device__ __forceinline__ void pool_park(PoolLds32<TRACE, PW> &P, uint32_t s, const Hit32 &h) {
  P.w[s] = h.w;
  P.hh[s] = h.hh;
  P.hl[s] = h.hl;
  P.last[s] = h.last;
  P.k[s] = (uint8_t)h.k;
}
template <bool TRACE, int PW>
__device__ __forceinline__ Hit64 pool_hit(const PoolLds64<TRACE, PW> &P, uint32_t s,
                                          const StepArgs &A) {
  Hit64 h{A.dt, P.w[s], (int32_t)P.k[s], -1};
  if (h.k > 0) {
    h.h = P.h[s];
    h.last = P.last[s];
  }
  return h;
}
template <bool TRACE, int PW>
__device__ __forceinline__ void pool_park(PoolLds64<TRACE, PW> &P, uint32_t s, const Hit64 &h) {
  P.w[s] = h.w;
  P.h[s] = h.h;
  P.last[s] = h.last;
  P.k[s] = (uint8_t)h.k;
}

// Reads particle id from the set when a wave claims it: the state word
// and position go to home slot hs.  False for a removed particle, and for
// a corrupt state (the set's error word is raised).
template <bool TRACE, int PW, int GEN>
__device__ __forceinline__ bool pool_claim(const GView &G, const SetDev &S, int32_t n_edges,
                                           uint32_t id, PoolLds32<TRACE, PW> &P, uint32_t hs,
                                           bool mine) {
  bool ok = false;
  uint32_t ef = 0;
  float2 yy = make_float2(0.0f, 0.0f);
  if (mine) {
    ef = S.ef[id];
    yy = S.y32[id];
    const int32_t e = (int32_t)(ef & kEdgeMask);
    if (!(ef & kDeadBit)) {
      if (e >= n_edges) {
        atomicOr(S.err, kErrEdge);
      } else if (!((yy.x >= 0.0f && yy.x <= G.e32[e].L) ||
                   (GEN == kGenFull && yy.x < 0.0f &&
                    ((uint32_t)((ef & kSideBit) ? G.e32[e].vterm : G.e32[e].vinit) &
                     kWentzellEnd)))) {
        atomicOr(S.err, kErrPos);
      } else {
        ok = true;
      }
    }
  }
  if (ok) {
    P.ef[hs] = ef;
    P.y[hs] = yy.x;
    P.yl[hs] = yy.y;
  }
  return ok;
}
template <bool TRACE, int PW, int GEN>
__device__ __forceinline__ bool pool_claim(const GView &G, const SetDev &S, int32_t n_edges,
                                           uint32_t id, PoolLds64<TRACE, PW> &P, uint32_t hs,
                                           bool mine) {
  bool ok = false;
  uint32_t ef = 0;
  double x = 0.0;
  if (mine) {
    ef = S.ef[id];
    x = S.x64[id];
    const int32_t e = (int32_t)(ef & kEdgeMask);
    if (!(ef & kDeadBit)) {
      if (e >= n_edges) {
        atomicOr(S.err, kErrEdge);
      } else {
        const EdgeRec64 &r = G.e64[e];
        if (!((x >= 0.0 && x <= r.L) ||
              (GEN == kGenFull && ((x <= 0.0 && ((uint32_t)r.vinit & kWentzellEnd)) ||
                       (x >= r.L && ((uint32_t)r.vterm & kWentzellEnd)))))) {
          atomicOr(S.err, kErrPos);
        } else {
          ok = true;
        }
      }
    }
  }
  if (ok) {
    P.ef[hs] = ef;
    P.x[hs] = x;
  }
  return ok;
}

// Writes a particle back at the end of its launch and counts the steps it
// took (each has one first sub-step; resolve() counts the others).
template <bool TRACE, bool LDS, int GEN>
__device__ __forceinline__ void pool_finish(const Particle32<TRACE, LDS, GEN> &q, const SetDev &S,
                                            const StepArgs &A, uint32_t pid, Tally &t) {
  S.ef[pid] = (uint32_t)q.e | (q.side ? kSideBit : 0u) | (q.alive ? 0u : kDeadBit);
  S.y32[pid] = make_float2(q.y, q.yl);
  if (TRACE) {
    S.seqhash[pid] = q.hash;
    S.hits[pid] = q.nhit;
  }
  const uint32_t taken = q.alive ? A.nsteps : q.death_step + 1u - S.n0;
  t.steps += taken;
  t.sub += taken;
}
template <bool TRACE, bool LDS, int GEN>
__device__ __forceinline__ void pool_finish(const Particle64<TRACE, LDS, GEN> &q, const SetDev &S,
                                            const StepArgs &A, uint32_t pid, Tally &t) {
  S.ef[pid] = (uint32_t)q.e | (q.alive ? 0u : kDeadBit);
  S.x64[pid] = q.x;
  if (TRACE) {
    S.seqhash[pid] = q.hash;
    S.hits[pid] = q.nhit;
  }
  const uint32_t taken = q.alive ? A.nsteps : q.death_step + 1u - S.n0;
  t.steps += taken;
  t.sub += taken;
}

// A particle of the pool loop, before its first pickup: the graph view,
// exit counters and the launch's dt.
template <bool TRACE, bool LDS, int GEN>
__device__ __forceinline__ void pool_particle(Particle32<TRACE, LDS, GEN> &q, const GView &G,
                                              uint32_t *s_exit, const StepArgs &A) {
  q = Particle32<TRACE, LDS, GEN>{G, s_exit, 0, 0u, 0.0f, 0.0f, Edge32{}, 0.0f, 0.0f,
                                  (float)A.dt, (float)sqrt(A.dt), true, 0ull, 0u, 0u};
}
template <bool TRACE, bool LDS, int GEN>
__device__ __forceinline__ void pool_particle(Particle64<TRACE, LDS, GEN> &q, const GView &G,
                                              uint32_t *s_exit, const StepArgs &A) {
  q = Particle64<TRACE, LDS, GEN>{G, s_exit, 0, 0.0, EdgeRec64{}, true, 0ull, 0u, 0u,
                                  A.dt, sqrt(A.dt)};
}

// A lane's particle while it runs first sub-steps: what a window of steps
// needs, in registers, and no more.  Pos is the part that a step changes;
//   propose(p, w)   the position a first sub-step from p reaches;
//   inside(p)       the lanes where it lies strictly inside the edge;
//   fold(p, w)      the normal of a step from p as it enters the proposal
//                   (a particle on a vertex moves into its edge);
//   on_vertex(p)    the lanes where p is an end of the edge;
//   visits(p)       the step from p starts with a Wentzell visit (GEN);
//   reanchor(p, c)  the nearer reference end, where c (FP32).
struct Pos32 {
  float y, yl;
};
struct Pos64 {
  double x;
};
__device__ __forceinline__ Pos32 pick(bool c, const Pos32 &a, const Pos32 &b) {
  return {c ? a.y : b.y, c ? a.yl : b.yl};
}
__device__ __forceinline__ Pos64 pick(bool c, const Pos64 &a, const Pos64 &b) {
  return {c ? a.x : b.x};
}

// FP32.  Affine coefficients: the first sub-step is y + (fma(gs, w, fma(cd,
// y, ad)) + yl) with per-frame constants; adf is ad of the other reference
// end and the sign of gs is the end itself (negative: the terminal one), so
// a change of end is four selects.  GEN evaluates the coefficients at y.
template <bool TRACE, bool LDS, int GEN>
struct Lane32 {
  using real = float;
  using Pos = Pos32;
  using Q = Particle32<TRACE, LDS, GEN>;
  Pos32 p;
  int32_t e;
  float L, cd, ad, adf, gs;
  Q q;  // GEN only

  __device__ __forceinline__ void init(const GView &G, uint32_t *s_exit, const StepArgs &A) {
    pool_particle(q, G, s_exit, A);
    p = {0.0f, 0.0f};
    e = 0;
    L = cd = ad = adf = gs = 0.0f;
  }
  template <class Pool>
  __device__ __forceinline__ void load(const Pool &P, uint32_t s, const GView &G) {
    p = {P.y[s], P.yl[s]};
    if constexpr (GEN) {
      pool_load(q, P, s);
      e = q.e;
      L = q.R.L;
    } else {
      const uint32_t ef = P.ef[s];
      e = (int32_t)(ef & kEdgeMask);
      const EdgeRec32 r = G.e32[e];
      const bool side = (ef & kSideBit) != 0u;
      const float d0 = r.a * q.dt, d1 = -r.aL * q.dt, g0 = r.sigma * q.sqdt;
      L = r.L;
      cd = r.c * q.dt;
      ad = side ? d1 : d0;
      adf = side ? d0 : d1;
      gs = side ? -g0 : g0;
    }
  }
  __device__ __forceinline__ uint32_t side() const {
    if constexpr (GEN) return q.side;
    return __float_as_uint(gs) >> 31;
  }
  __device__ __forceinline__ uint32_t state() const {
    return (uint32_t)e | (side() ? kSideBit : 0u);
  }
  __device__ __forceinline__ Pos32 propose(const Pos32 &a, float w) {
    float s;
    if constexpr (GEN) {
      const float sg = q.fsigma(a.y) * q.sqdt;
      s = fmaf(q.side ? -sg : sg, w, q.fdrift(a.y) * q.dt) + a.yl;
    } else {
      s = fmaf(gs, w, fmaf(cd, a.y, ad)) + a.yl;
    }
    const float yt = a.y + s;  // Fast2Sum, as Particle32::add_comp
    return {yt, s - (yt - a.y)};
  }
  __device__ __forceinline__ uint64_t inside(const Pos32 &a) const {
    return ballot(a.y > 0.0f) & ballot(a.y < L);
  }
  __device__ __forceinline__ uint64_t on_vertex(const Pos32 &a) const {
    return ballot(a.y == 0.0f);
  }
  __device__ __forceinline__ float fold(const Pos32 &, float w) const {
    return copysignf(fabsf(w), GEN ? q.gs : gs);
  }
  __device__ __forceinline__ bool visits(const Pos32 &a) const {
    if constexpr (GEN != kGenFull) return false;
    return a.y <= 0.0f && ((uint32_t)(q.side ? q.R.vterm : q.R.vinit) & kWentzellEnd);
  }
  // y > L - y exactly when y > L/2: L - y is exact from L/2 on (Sterbenz)
  // and no smaller than L/2, so than y, below.
  __device__ __forceinline__ void reanchor(Pos32 &a, bool c) {
    if constexpr (GEN) {
      q.y = a.y;
      q.yl = a.yl;
      q.reanchor_if(c);
      a = {q.y, q.yl};
    } else {
      const float t = L - a.y;
      const bool flip = c & (a.y > t);
      a = {flip ? t : a.y, flip ? -a.yl : a.yl};
      gs = flip ? -gs : gs;
      const float o = ad;
      ad = flip ? adf : ad;
      adf = flip ? o : adf;
    }
  }
  template <class Pool>
  __device__ __forceinline__ void store(Pool &P, uint32_t s, const Pos32 &a) const {
    P.ef[s] = state();
    P.y[s] = a.y;
    P.yl[s] = a.yl;
  }
  __device__ __forceinline__ void write(const SetDev &S, uint32_t pid, const Pos32 &a,
                                        uint32_t state) const {
    S.ef[pid] = state;
    S.y32[pid] = make_float2(a.y, a.yl);
  }
  // position from the initial vertex in FP64, as the histogram reads it
  __device__ static double pos64(const Pos32 &a, uint32_t side, double L) {
    const double v = (double)a.y + (double)a.yl;
    return side ? L - v : v;
  }
};

// FP64: positions from the initial vertex, no reference end to change.
template <bool TRACE, bool LDS, int GEN>
struct Lane64 {
  using real = double;
  using Pos = Pos64;
  using Q = Particle64<TRACE, LDS, GEN>;
  Pos64 p;
  int32_t e;
  double L, a0, c0, gd;  // affine: drift a0 + c0 x, sigma sqrt(dt)
  Q q;                   // its dt; GEN: the edge record too

  __device__ __forceinline__ void init(const GView &G, uint32_t *s_exit, const StepArgs &A) {
    pool_particle(q, G, s_exit, A);
    p = {0.0};
    e = 0;
    L = a0 = c0 = gd = 0.0;
  }
  template <class Pool>
  __device__ __forceinline__ void load(const Pool &P, uint32_t s, const GView &G) {
    p = {P.x[s]};
    e = (int32_t)(P.ef[s] & kEdgeMask);
    if constexpr (GEN) {
      q.R = G.e64[e];
      L = q.R.L;
    } else {
      const EdgeRec64 &r = G.e64[e];
      L = r.L;
      a0 = r.a;
      c0 = r.c;
      gd = r.sigma * q.sqdt;
    }
  }
  __device__ __forceinline__ uint32_t side() const { return 0u; }
  __device__ __forceinline__ uint32_t state() const { return (uint32_t)e; }
  __device__ __forceinline__ Pos64 propose(const Pos64 &a, double w) const {
    if constexpr (GEN)
      return {fma(q.diffusion(a.x) * q.sqdt, w, fma(q.drift(a.x), q.dtv, a.x))};
    return {fma(gd, w, fma(fma(c0, a.x, a0), q.dtv, a.x))};
  }
  __device__ __forceinline__ uint64_t inside(const Pos64 &a) const {
    return ballot(a.x > 0.0) & ballot(a.x < L);
  }
  __device__ __forceinline__ uint64_t on_vertex(const Pos64 &a) const {
    return ballot(a.x == 0.0) | ballot(a.x == L);
  }
  __device__ __forceinline__ double fold(const Pos64 &a, double w) const {
    return a.x == 0.0 ? fabs(w) : -fabs(w);
  }
  __device__ __forceinline__ bool visits(const Pos64 &a) const {
    if constexpr (GEN != kGenFull) return false;
    return (a.x <= 0.0 && ((uint32_t)q.R.vinit & kWentzellEnd)) ||
           (a.x >= L && ((uint32_t)q.R.vterm & kWentzellEnd));
  }
  __device__ __forceinline__ void reanchor(Pos64 &, bool) {}
  template <class Pool>
  __device__ __forceinline__ void store(Pool &P, uint32_t s, const Pos64 &a) const {
    P.x[s] = a.x;  // the edge in the home slot is unchanged
  }
  __device__ __forceinline__ void write(const SetDev &S, uint32_t pid, const Pos64 &a,
                                        uint32_t state) const {
    S.ef[pid] = state;
    S.x64[pid] = a.x;
  }
  __device__ static double pos64(const Pos64 &a, uint32_t, double) { return a.x; }
};

// Adds a lane's tallies to the block's 64-bit totals and clears them.
__device__ __forceinline__ void drain_tally(Tally &t, unsigned long long *s_tot) {
  if (t.trunc) atomicAdd(&s_tot[0], (unsigned long long)t.trunc);
  if (t.sub) atomicAdd(&s_tot[1], (unsigned long long)t.sub);
  if (t.hits) atomicAdd(&s_tot[2], (unsigned long long)t.hits);
  if (t.steps) atomicAdd(&s_tot[3], (unsigned long long)t.steps);
  t = Tally{0, 0, 0, 0};
}

// Moves a block's u32 LDS counters into their 64-bit counters in the set
// (the lanes of one wave, each counter taken and cleared atomically, so
// counts other waves add meanwhile are kept).
__device__ __forceinline__ void drain_lds(uint32_t *lds, uint64_t *glob, int32_t n) {
  for (int32_t i = (int32_t)(threadIdx.x & 63u); i < n; i += 64) {
    const uint32_t v = atomicExch(&lds[i], 0u);
    if (v) atomicAdd((unsigned long long *)&glob[i], (unsigned long long)v);
  }
}

// A lane of a pool serves any number of particles in a launch, and a
// persistent block any number of particle-steps, so every wave drains its
// lanes' 32-bit tallies into the block's 64-bit totals every A.drain (at
// most kDrainMax = 1024) iterations of its pool loop, and the block's u32
// LDS exit and snapshot counters into the set's 64-bit ones every
// A.drain_lds (at most kLdsDrainMax = 2^20) groups of steps and split
// passes.  Bounds: one iteration finishes at most two particles on a lane
// (its own, and the one of its split-pass slot), each adding at most 2^20
// steps (a launch's cap), plus at most one crossing, so 1024 iterations add
// at most 2^31 + 1024 to a tally.  Between two drains of an LDS counter (by
// any wave), each of the block's four waves runs fewer than A.drain_lds +
// kMaxGroups + 1 groups and passes, each adding at most 64 x 4 snapshots, or
// 64 exit records and 64 snapshots: below 4 (2^20 + 65) x 256 < 2^31 per
// counter.  The LDS drains are rare because each is a round of
// device-scope atomics on the set's counters, which go past the XCD's L2.

// Where a wave's particles come from: the set's counter.  The grid stays
// resident; every wave reserves the next A.claim_chunk particle ids from the
// counter (one atomic) and moves them into its pool as its home slots free
// up, so pools stay nearly full until the set runs out and a launch ends
// with one short tail instead of one per block.  The reservation is larger
// for short launches (up to 1024 ids): the set's counter is one address
// that every wave of the grid updates, and with 16 ids per update a
// 100-step launch over 1e8 particles spent most of its time on it.  A wave
// that finds the set run out stops reserving, so every wave passes n by at
// most one reservation per set and launch (a batched launch lets a block
// join a set only while its counter is below n, so this holds there too);
// the host bounds the reservation so that the counter cannot wrap.
// In a launch that is the set's own (not a batch) a wave's first reservation is
// its place in the grid, and the counter starts behind those of all waves
// (own_claims): a set spread over many small pools (set_pool) otherwise updated
// the one address twice per wave, and a short launch waited for that (1 / 8 / 31
// steps of 3e4 FP32 particles on the 64-edge star 29 / 40 / 67 -> 14 / 26 / 52
// us; with full pools 18 / 32 / 61).
// Q: the particle type (Particle32 or Particle64, each with its pool type
// in LDS).
template <bool BATCH, bool TRACE, bool LDS, bool OBS, int PW, int GEN, class Ln, class Pool>
__device__ void run_pool(const GView &G, int32_t n_edges, const SetDev &S,
                         const StepArgs &A, Pool &P, uint32_t *s_exit, Tally &t,
                         unsigned long long *s_tot, int32_t nnz, const ObsSink &sink) {
  using Q = typename Ln::Q;
  using Pos = typename Ln::Pos;
  using real = typename Ln::real;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t n_end = S.n0 + A.nsteps;
  const uint32_t g_last = (n_end - 1u) >> 2, part = n_end & 3u;
  Ln ln;
  ln.init(G, s_exit, A);
  MainCtr ctr{0u, 0u, 0u, 0u};
  uint64_t m_has = 0ull;             // lanes with a particle
  uint32_t slot = 0, g = 0, jb = 0;  // the lane's home slot, next group, first step in it
  uint32_t snap = 0;  // next snapshot count of the lane's particle
  const uint32_t snap0 = OBS ? next_snapshot(S.n0, S) : 0u;
  // Ready, split and free queues: FIFO rings over the pool's slot ids, with
  // wave-uniform head and tail counters.  FIFO keeps the particles of a pool
  // advancing together, so a launch ends without a long tail of stragglers.
  constexpr uint32_t K = (uint32_t)PW;
  uint32_t r_head = 0, r_tail = 0, s_head = 0, s_tail = 0;
  uint32_t f_head = 0, f_tail = A.pool_cap;
  for (uint32_t i = lane; i < A.pool_cap; i += 64u) P.freeq[i] = (uint8_t)i;
  const int32_t lanes = min((int32_t)A.pool_cap, 64);  // lanes that a full pool keeps busy
  const uint32_t lim = S.n;
  bool exhausted = false;   // the reservation is used up and the set has run out
  bool last_chunk = false;  // the set ran out with the current reservation
  uint32_t res_next = 0, res_end = 0;  // the wave's reserved ids [res_next, res_end)
  if (!BATCH && lane == 0u) {
    // The first reservation, and whether no more follow, wait in a home slot that
    // is empty until then: carried in scalar registers to their use they cost
    // the loop 40 spills (64-edge star, dt 10^-2, 153 -> 185 ms in one form).
    P.pid[0] = (blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6)) * A.claim_chunk;
    P.n[0] = gridDim.x * kWavesPerBlock * A.claim_chunk >= lim;
  }
  uint32_t iter = 0, iter_lds = 0;
  wave_lds_fence();

  for (;;) {
    if (++iter >= A.drain) {
      iter = 0;
      drain_tally(t, s_tot);
    }
    if (iter_lds >= A.drain_lds) {
      iter_lds = 0;
      if (LDS) drain_lds(s_exit, S.exit_cnt, nnz);
      if (OBS && sink.lds) drain_lds(sink.lds, S.obs, A.obs_lds);
    }
    // Claim more particles: a wave takes as many ids as it has free home
    // slots, in multiples of kClaimMin up to 64, from its reservation, so a
    // pool refills while its first particles finish rather than after half
    // of them have.  Reservations and claims stay multiples of kClaimMin
    // (but for the last ids below n), so every claim starts at a multiple
    // of it: a claim's 128-byte lines of positions belong to one wave (its
    // state words share a line with one neighbouring claim).
    while (!exhausted && f_tail - f_head >= (uint32_t)kClaimMin) {
      if (res_next == res_end) {
        if (last_chunk) {
          exhausted = true;
          break;
        }
        uint32_t v = BATCH ? 0u : P.pid[0], all = BATCH ? 0u : P.n[0];
        if (lane == 0u && (BATCH || f_head != 0u)) {
          v = atomicAdd(S.work, A.claim_chunk);
          all = 0u;
        }
        all = __builtin_amdgcn_readfirstlane(all);
        const uint32_t b = __builtin_amdgcn_readfirstlane(v);
        if (b >= lim) {
          exhausted = true;
          break;
        }
        last_chunk = all != 0u || lim - b <= A.claim_chunk;
        res_next = b;
        res_end = min(b + A.claim_chunk, lim);
      }
      const uint32_t want =
          min(min(64u, f_tail - f_head) & ~((uint32_t)kClaimMin - 1u), res_end - res_next);
      const uint32_t id = res_next + lane;
      res_next += want;
      const bool mine = lane < want;
      const uint32_t hs = mine ? P.freeq[(f_head + lane) % K] : 0u;
      const bool ok = pool_claim<TRACE, PW, GEN>(G, S, n_edges, id, P, hs, mine && id < lim);
      f_head += want;
      const uint64_t m_ok = ballot(ok);
      const uint64_t m_back = ballot(mine & !ok);
      if (ok) {
        P.n[hs] = S.n0;
        P.pid[hs] = id;
        P.k[hs] = 0;
        if constexpr (OBS) P.snap[hs] = snap0;
        if constexpr (TRACE) {
          P.hits[hs] = S.hits[id];
          P.hash[hs] = S.seqhash[id];
        }
        P.ready[(r_tail + lane_rank(m_ok)) % K] = (uint8_t)hs;
      } else if (mine) {
        P.freeq[(f_tail + lane_rank(m_back)) % K] = (uint8_t)hs;
      }
      r_tail += (uint32_t)__popcll(m_ok);
      f_tail += (uint32_t)__popcll(m_back);
      wave_lds_fence();
    }
    // lanes without a particle take ready ones
    {
      const uint32_t ready_cnt = r_tail - r_head;
      const uint32_t r = lane_rank(~m_has);
      const uint64_t m_take = ~m_has & ballot(r < ready_cnt);
      if (m_take != 0ull) {
        if (in_mask(m_take)) {
          slot = P.ready[(r_head + r) % K];
          const uint32_t n = P.n[slot];
          ln.load(P, slot, G);
          ctr = main_ctr(P.pid[slot], S.tag, A.key0, A.key1);
          g = n >> 2;
          jb = n & 3u;
          if constexpr (OBS) snap = P.snap[slot];
        }
        r_head += (uint32_t)__popcll(m_take);
        m_has |= m_take;
      }
    }
    bool do_split = false;
    if (m_has == 0ull) {
      if (s_tail == s_head) {
        if (exhausted) break;
        continue;  // every particle claimed so far was dead: claim more
      }
      do_split = true;
    } else {
      // Groups of four first sub-steps (one main-stream Philox block) until
      // enough lanes wait for another particle.  Every lane runs the same
      // straight-line code from the positions H[0] to H[4], past a vertex
      // too; the lane masks of the proposals that stayed inside tell
      // afterwards where a lane stopped, so a step carries no select, and a
      // lane's state is taken back from H only if some lane of the wave
      // stopped.  The first group after a pickup may start inside (jb > 0).
      //
      // Bound by VALU issue: a group of 64 lanes takes 97 VALU instructions
      // without a hit (16 of them 64-bit products at half rate, 8
      // transcendentals at a quarter), 24 a step, where windows of eight steps with a
      // select per step took 39; what a hit adds (parking, the refill and
      // its shorter first group, the split pass, lanes that wait for them) is
      // 650 lane slots at 7.7 % hits a step and 1080 at 2.2 %.
      // FP32, 1000 steps of 3e7 particles on the vascular network (0.35 %
      // hits a step) 23.0 -> 19.3 ms, 2000 steps of 1e7 on the 64-edge star
      // 21.1 -> 20.4 ms (2.1 % hits), 30.7 -> 30.7 (7.1 %); FP64, 1e7 on the
      // network 19.9 -> 18.9 ms.  More waves change nothing (five a SIMD run
      // the network as fast as seven).
      // How many lanes without a particle end the window: A.refill if there
      // is (or can be claimed) a particle for them; as many as would fill a
      // split pass, or leave A.idle lanes idle while particles are parked.
      // (Only parking and finishing empty a lane, so no more than the newly
      // empty lanes have joined the split queue.)
      const int32_t ready0 = (int32_t)(r_tail - r_head), split0 = (int32_t)(s_tail - s_head);
      const int32_t empty0 = lanes - (int32_t)__popcll(m_has);
      const bool more = ready0 > 0 || (!exhausted && f_tail - f_head >= (uint32_t)kClaimMin);
      const int32_t full = lanes - split0 + empty0;
      const int32_t leave = min(min(more ? A.refill : ready0 + A.idle, full), lanes);
      bool fresh = true;
      int32_t groups = 0;
      for (;;) {
        uint32_t k0 = A.key0, k1 = A.key1;
        fresh_keys<real>(k0, k1);
        const U4 o = philox_main(ctr, g, k0, k1);
        real W[4];
        Q::box_muller(o.x, o.y, G.bm, W[0], W[1]);
        Q::box_muller(o.z, o.w, G.bm, W[2], W[3]);
        Pos H[5];
        H[0] = ln.p;
        uint64_t m_visit = 0ull;
        if (fresh) {
          const uint64_t m_fold = m_has & ln.on_vertex(ln.p);
          if (m_fold != 0ull) {
            if (in_mask(m_fold)) {
#pragma unroll
              for (uint32_t j = 0; j < 4; ++j) W[j] = jb == j ? ln.fold(ln.p, W[j]) : W[j];
            }
          }
          if constexpr (GEN == kGenFull) m_visit = ballot(ln.visits(ln.p));
        }
        uint64_t in[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
          H[j + 1] = ln.propose(H[j], W[j]);
          in[j] = ln.inside(H[j + 1]);
          if (GEN == kGenFull && fresh) in[j] &= ~m_visit;
          if (j < 3 && fresh) {
            const uint64_t m_skip = ballot(jb > j);
            H[j + 1] = pick(in_mask(m_skip), H[0], H[j + 1]);
            in[j] |= m_skip;
          }
        }
        // the launch's last group may end inside (part = 1 .. 3 steps of it)
        const uint64_t m_last = ballot(g == g_last);
        if (part) {
          if (part < 2u) in[1] |= m_last;
          if (part < 3u) in[2] |= m_last;
          in[3] |= m_last;
        }
        const uint64_t stay = in[0] & in[1] & in[2] & in[3];
        const uint64_t m_park = m_has & ~stay;
        const uint64_t m_fin = m_has & stay & m_last;
        // snapshots of the group's steps: the lanes that completed step m - 1
        // and are at the snapshot count after it (after the fourth step, with
        // the new reference end)
        auto snapshot = [&](uint32_t m, uint64_t completed, const Pos &a) {
          const uint64_t due = completed & ballot(snap == 4u * g + m);
          if (due != 0ull) {
            if (in_mask(due)) {
              const double2 r = S.obs_edge[ln.e];
              observe_at(ln.e, Ln::pos64(a, ln.side(), r.x), r.y, S, sink);
              snap = snapshot_after(snap, S);
            }
          }
        };
        const bool any_snap = OBS && (m_has & ballot(snap - 4u * g - 1u < 4u)) != 0ull;
        if (OBS && any_snap) {
          uint64_t c = m_has;
#pragma unroll
          for (uint32_t m = 1; m < 4; ++m) {
            c &= in[m - 1];
            if (part != 0u && m > part) c &= ~m_last;
            snapshot(m, c, H[m]);
          }
        }
        if (m_park != 0ull) {
          // back to where the lane stopped: step j from H[j] with normal W[j]
          if (in_mask(m_park)) {
            uint32_t j = in_mask(in[2]) ? 3u : 2u;
            Pos a = pick(in_mask(in[2]), H[3], H[2]);
            real w = in_mask(in[2]) ? W[3] : W[2];
            j = in_mask(in[1]) ? j : 1u;
            a = pick(in_mask(in[1]), a, H[1]);
            w = in_mask(in[1]) ? w : W[1];
            j = in_mask(in[0]) ? j : 0u;
            a = pick(in_mask(in[0]), a, H[0]);
            w = in_mask(in[0]) ? w : W[0];
            ln.store(P, slot, a);
            P.n[slot] = 4u * g + j;
            P.w[slot] = w;
            if constexpr (OBS) P.snap[slot] = snap;
            P.split[(s_tail + lane_rank(m_park)) % K] = (uint8_t)slot;
          }
          s_tail += (uint32_t)__popcll(m_park);
        }
        ln.p = H[4];
        if (part) {
          const bool cut = in_mask(m_fin);
          ln.p = pick(cut, pick(part == 1u, H[1], pick(part == 2u, H[2], H[3])), ln.p);
          ln.reanchor(ln.p, !cut);
        } else {
          ln.reanchor(ln.p, true);
        }
        if (OBS && any_snap) snapshot(4u, m_has & stay & (part ? ~m_last : ~0ull), ln.p);
        if (m_fin != 0ull) {
          if (in_mask(m_fin)) {
            const uint32_t id = P.pid[slot];
            ln.write(S, id, ln.p, ln.state());
            if constexpr (TRACE) {
              S.seqhash[id] = P.hash[slot];
              S.hits[id] = P.hits[slot];
            }
            t.steps += A.nsteps;
            t.sub += A.nsteps;
            P.freeq[(f_tail + lane_rank(m_fin)) % K] = (uint8_t)slot;
          }
          f_tail += (uint32_t)__popcll(m_fin);
        }
        m_has &= stay & ~m_last;
        ++g;
        jb = 0;
        fresh = false;
        ++groups;
        wave_lds_fence();
        if (lanes - (int32_t)__popcll(m_has) >= leave || groups == kMaxGroups) break;
      }
      const int32_t split_cnt = (int32_t)(s_tail - s_head);
      const int32_t idle = lanes - (int32_t)__popcll(m_has) - (int32_t)(r_tail - r_head);
      do_split = split_cnt >= lanes || (split_cnt > 0 && idle >= A.idle);
      iter_lds += (uint32_t)groups;
    }
    if (do_split) {
      ++iter_lds;
      // Up to 64 parked particles, one per lane, one crossing each.  The
      // lanes' own particles stay in registers meanwhile.
      const uint32_t B = min(s_tail - s_head, 64u);
      const uint32_t s_base = s_head;
      s_head += B;
      wave_lds_fence();
      bool back = false, again = false, freed = false;
      uint32_t s2 = 0;
      if (lane < B) {
        s2 = P.split[(s_base + lane) % K];
        Q q2;
        pool_particle(q2, G, s_exit, A);
        pool_load(q2, P, s2);
        const uint32_t step = P.n[s2];
        const uint32_t pid2 = P.pid[s2];
        auto h = pool_hit(P, s2, A);
        if (!q2.cross(step, h, pid2, S, A, t)) {
          // reached a vertex again: back on the split queue for a later pass
          pool_store(q2, P, s2, step);
          pool_park(P, s2, h);
          again = true;
        } else {
          if (q2.alive) {
            if ((step & 3u) == 3u) q2.reanchor();
            if constexpr (OBS) {
              const uint32_t at = P.snap[s2];
              if (step + 1u == at) {
                observe(q2, S, sink);
                P.snap[s2] = snapshot_after(at, S);
              }
            }
          }
          const uint32_t n2 = step + 1u;
          if (!q2.alive || n2 == n_end) {
            pool_finish(q2, S, A, pid2, t);
            freed = true;
          } else {
            pool_store(q2, P, s2, n2);
            P.k[s2] = 0;
            back = true;
          }
        }
      }
      const uint64_t m_freed = ballot(freed);
      if (freed) P.freeq[(f_tail + lane_rank(m_freed)) % K] = (uint8_t)s2;
      f_tail += (uint32_t)__popcll(m_freed);
      const uint64_t m_again = ballot(again);
      if (again) P.split[(s_tail + lane_rank(m_again)) % K] = (uint8_t)s2;
      s_tail += (uint32_t)__popcll(m_again);
      const uint64_t m_back = ballot(back);
      if (back) P.ready[(r_tail + lane_rank(m_back)) % K] = (uint8_t)s2;
      r_tail += (uint32_t)__popcll(m_back);
      wave_lds_fence();
    }
  }
}

// Shared memory of a pool block: [FP64: Box-Muller tables][exit counters]
// [staged tables][pools][snapshot bins].  Stages the set's tables, runs its particles until the
// set's counter has run out and the block's pools are empty, and adds the
// block's counts to the set's counters.

// BATCH: one of the blocks that work on the set at a time; else the whole grid
// does.
template <bool BATCH, bool FP64, bool TRACE, bool LDS, bool STAGED, bool OBS, int PW, int GEN>
__device__ __forceinline__ void pool_block(const GraphDev &G, const SetDev &S,
                                           const StepArgs &A, unsigned long long *s_tot,
                                           char *smem) {
  using Pool = PoolLds<PW, FP64, TRACE, OBS>;
  using Ln = std::conditional_t<FP64, Lane64<TRACE, LDS, GEN>, Lane32<TRACE, LDS, GEN>>;
  BmLds *bm = (BmLds *)smem;
  if (FP64) {
    stage_bm(bm);
    smem += sizeof(BmLds);
  }
  uint32_t *s_exit = (uint32_t *)smem;
  if (threadIdx.x < 4) s_tot[threadIdx.x] = 0;
  if (LDS)
    for (int32_t s = threadIdx.x; s < G.nnz; s += blockDim.x) s_exit[s] = 0;
  const int32_t ex = LDS ? exit_bytes(G.nnz) : 0;
  GView view = block_view<FP64, STAGED, GEN>(G, smem + ex);
  if (FP64) view.bm = bm;
  const int32_t o_pools =
      align16(ex + (STAGED ? (FP64 ? G.stage_bytes64 : G.stage_bytes32) : 0));
  Pool *pools = (Pool *)(smem + o_pools);
  ObsSink o{nullptr};
  if (OBS && A.obs_lds) {
    o.lds = (uint32_t *)(smem + o_pools + (int32_t)sizeof(Pool) * kWavesPerBlock);
    for (int32_t b = threadIdx.x; b < A.obs_lds; b += blockDim.x) o.lds[b] = 0;
  }
  __syncthreads();
  Tally t{0, 0, 0, 0};
  const uint32_t wave = threadIdx.x >> 6;
  run_pool<BATCH, TRACE, LDS, OBS, PW, GEN, Ln>(view, G.E, S, A, pools[wave], s_exit, t, s_tot,
                                                G.nnz, o);
  flush(S, t, s_tot, s_exit, G.nnz, LDS);
  if (OBS && A.obs_lds) flush_obs(S, o.lds, A.obs_lds);
}

#ifndef MG_POOL_WAVES_PER_EU
#define MG_POOL_WAVES_PER_EU 6
#endif

// The general levels (GEN) are built for pools of 128 only.  The full one takes
// 117 to 128 registers: four waves a SIMD.  At six it spilled 53 to 118 of them
// (2e6 particles on the Wentzell star, 60 steps of 10^-3: 2.32 ms, streaming
// 2.74, in a batch of six sets of 2e5, 100 steps, 5.5; at five 1.35, 1.77, 3.7; at
// four 1.32, 1.49, 3.1; 2e6 with 200 tabulated edges 1.32 / 1.17 / 1.16; 200
// steps of 3e6 on the Wentzell star, streaming, 16.3 against 6.9 at four).
template <bool TRACE, bool LDS, bool STAGED, bool OBS, int PW, int GEN = 0>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(GEN == kGenFull ? 4 : MG_POOL_WAVES_PER_EU)))
void k_pool32(GraphDev G, SetDev S, StepArgs A) {
  extern __shared__ uint4 smem4[];
  __shared__ unsigned long long s_tot[4];
  pool_block<false, false, TRACE, LDS, STAGED, OBS, PW, GEN>(G, S, A, s_tot, (char *)smem4);
}

// FP64 wave pools: the same schedule over FP64 particles (pools of 128).  Two
// FP64 particles per lane take more registers: four waves per SIMD, three at
// the full general level, whose 160 registers would spill (three, four and
// five waves run the affine level alike: it is bound by VALU issue).
#ifndef MG_POOL64_WAVES_PER_EU
#define MG_POOL64_WAVES_PER_EU 4
#endif
template <bool TRACE, bool LDS, bool STAGED, bool OBS, int GEN>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(GEN == kGenFull ? 3 : MG_POOL64_WAVES_PER_EU)))
void k_pool64(GraphDev G, SetDev S, StepArgs A) {
  extern __shared__ uint4 smem4[];
  __shared__ unsigned long long s_tot[4];
  pool_block<false, true, TRACE, LDS, STAGED, OBS, kPoolSmall, GEN>(G, S, A, s_tot, (char *)smem4);
}

// Batched form of the wave pools: a resident grid whose blocks take work
// items (a set index each; A.batch_items of them, largest sets first) from
// the counter A.batch_claim, and for each runs the set's particles with the
// single-set pool code: the block's waves claim ids from the set's own
// counter, alongside every other block working on that set, until it has
// run out.  An item of a set that has run out is passed over at the cost
// of one load.  Both counters are cleared by k_batch_reset before each
// launch.
template <bool TRACE, bool LDS, bool STAGED, bool OBS, int PW, int GEN = 0>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(GEN == kGenFull ? 4 : MG_POOL_WAVES_PER_EU)))
void k_pool32_batch(const GraphDev *graphs, const SetDev *sets, const BatchItem *items,
                    StepArgs A) {
  extern __shared__ uint4 smem4[];
  __shared__ unsigned long long s_tot[4];
  __shared__ int32_t s_set;
  for (;;) {
    if (threadIdx.x == 0) {
      const uint32_t i = atomicAdd(A.batch_claim, 1u);
      int32_t set = -1;  // -1: no items left
      if (i < A.batch_items) {
        set = items[i].set;
        const SetDev &Si = sets[set];
        if (__hip_atomic_load(Si.work, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= Si.n)
          set = -2;  // that set has run out
      }
      s_set = set;
    }
    __syncthreads();
    const int32_t set = s_set;
    __syncthreads();  // every thread has read s_set before thread 0 writes it again
    if (set == -1) break;
    if (set < 0) continue;
    SetDev S = sets[set];
    S.n0 += A.n0_offset;  // steps already taken by earlier launches of this call
    const GraphDev G = graphs[set];
    pool_block<true, false, TRACE, LDS, STAGED, OBS, PW, GEN>(G, S, A, s_tot, (char *)smem4);
  }
}

// The same over FP64 sets: FP64 wave pools (128 per wave).
template <bool TRACE, bool LDS, bool STAGED, bool OBS, int GEN = 0>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(GEN == kGenFull ? 3 : MG_POOL64_WAVES_PER_EU)))
void k_pool64_batch(const GraphDev *graphs, const SetDev *sets, const BatchItem *items,
                    StepArgs A) {
  extern __shared__ uint4 smem4[];
  __shared__ unsigned long long s_tot[4];
  __shared__ int32_t s_set;
  for (;;) {
    if (threadIdx.x == 0) {
      const uint32_t i = atomicAdd(A.batch_claim, 1u);
      int32_t set = -1;  // -1: no items left
      if (i < A.batch_items) {
        set = items[i].set;
        const SetDev &Si = sets[set];
        if (__hip_atomic_load(Si.work, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= Si.n)
          set = -2;  // that set has run out
      }
      s_set = set;
    }
    __syncthreads();
    const int32_t set = s_set;
    __syncthreads();  // every thread has read s_set before thread 0 writes it again
    if (set == -1) break;
    if (set < 0) continue;
    SetDev S = sets[set];
    S.n0 += A.n0_offset;
    const GraphDev G = graphs[set];
    pool_block<true, true, TRACE, LDS, STAGED, OBS, kPoolSmall, GEN>(G, S, A, s_tot,
                                                                  (char *)smem4);
  }
}

// Clears the particle counters of a batch's sets and its groups' item
// counters before the launches of k_pool32_batch or k_pool64_batch (a kernel,
// so that the launches can be a HIP graph of kernel nodes).
__global__ void k_batch_reset(const SetDev *sets, int32_t n_sets, uint32_t *claim,
                              int32_t n_claims) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_sets) *sets[i].work = 0u;
  if (i < n_claims) claim[i] = 0u;
}

// Autotuning probes: the FP32 step kernels under names of their own, so a
// profile tells the probes apart from the launches they tune.
template <bool LDS, bool STAGED, int PW>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(MG_POOL_WAVES_PER_EU)))
void k_pool32_probe(GraphDev G, SetDev S, StepArgs A) {
  extern __shared__ uint4 smem4[];
  __shared__ unsigned long long s_tot[4];
  pool_block<false, false, false, LDS, STAGED, false, PW, 0>(G, S, A, s_tot, (char *)smem4);
}

template <bool LDS, bool STAGED>
__global__ __launch_bounds__(kBlock) void k_step32_probe(GraphDev G, SetDev S, StepArgs A) {
  extern __shared__ uint4 smem4[];
  __shared__ unsigned long long s_tot[4];
  step_block<false, false, LDS, STAGED, false, false>(G, S, A, blockIdx.x * kBlock + threadIdx.x,
                                               s_tot, (char *)smem4);
}

// Sets the particle counter of a persistent pool launch (a kernel rather than
// a memset, so that launch chains can be captured in HIP graphs).
__global__ void k_set_word(uint32_t *w, uint32_t v) {
  if (threadIdx.x == 0) *w = v;
}

// Blocks of a persistent launch: as many as stay resident at once (CUs x
// blocks per CU for this kernel and LDS size), fewer if the set is small.
uint32_t resident_blocks(const void *func, size_t shm, uint32_t need) {
  // blocks per CU of (device, kernel, LDS bytes) times the device's CU
  // count, queried once and kept: the occupancy query costs microseconds,
  // which short launches would pay on every call
  struct Entry {
    int dev;
    const void *func;
    size_t shm;
    uint32_t blocks;
  };
  static std::mutex mu;
  static std::vector<Entry> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = -1;
  uint32_t r = 0;
  {
    std::lock_guard<std::mutex> lock(mu);
    for (const Entry &e : cache)
      if (e.dev == dev && e.func == func && e.shm == shm) {
        r = e.blocks;
        break;
      }
  }
  if (r == 0) {
    int cus = 0;
    if (dev < 0 ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, func, kBlock, shm) != hipSuccess ||
        per_cu <= 0)
      per_cu = 1;
    r = (uint32_t)cus * (uint32_t)per_cu;
    if (r > kMaxPersistBlocks) r = kMaxPersistBlocks;  // bounds the claim counter
    std::lock_guard<std::mutex> lock(mu);
    if (cache.size() < 4096) cache.push_back({dev, func, shm, r});
  }
  return need < r ? need : r;
}

// ---------------------------------------------------------------- init --
template <bool FP64>
__global__ __launch_bounds__(kBlock) void k_init(GraphDev G, SetDev S, int mode,
                                                 int32_t vertex, uint32_t k0,
                                                 uint32_t k1, const int32_t *edge_in,
                                                 const double *pos_in, InitSources src) {
  const uint32_t pid = blockIdx.x * kBlock + threadIdx.x;
  if (pid >= S.n) return;
  int32_t e;
  double x;
  if (mode == 0) {
    e = edge_in[pid];
    x = pos_in[pid];
  } else {
    const U4 o = philox(pid, 0xFFFFFFFFu, 0xFFFFFFFFu, S.tag, k0, k1);
    if (mode == 1 || mode == 3) {
      uint32_t r = o.x;
      if (mode == 3) {
        // source: first j with word 0 < T_j (T nondecreasing, last 2^32)
        int32_t lo = 0, hi = src.n - 1;
        while (lo < hi) {
          const int32_t mid = (lo + hi) >> 1;
          if ((uint64_t)o.x < src.thr[mid])
            hi = mid;
          else
            lo = mid + 1;
        }
        vertex = src.vtx[lo];
        r = o.y;
      }
      const SlotPick sp = pick_slot(global_view(G), G.vtx[vertex], r);
      e = eo_edge(sp.eo);
      x = (sp.eo & 1u) ? G.e64[e].L : 0.0;
    } else {
      // first e with r < T_e (thresholds nondecreasing; T_{E-1} = 2^32),
      // between the first edges of the draw's bucket and of the next: a
      // search over all 26000 edges of the vascular network took 15
      // dependent loads (1e8 particles 3.63 ms, now 1.50)
      const uint32_t b = G.len_bits ? o.x >> (32 - G.len_bits) : 0u;
      int32_t lo = G.len_guide[b], hi = G.len_guide[b + 1];
      while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if ((uint64_t)o.x < G.len_thr[mid])
          hi = mid;
        else
          lo = mid + 1;
      }
      e = lo;
      x = G.e64[e].L * (((double)o.y + 0.5) * 0x1p-32);
    }
  }
  const double L = G.e64[e].L;
  if (FP64) {
    S.ef[pid] = (uint32_t)e;
    S.x64[pid] = x;
  } else {
    const bool side = x > 0.5 * L;
    const double yd = side ? L - x : x;
    const float yh = (float)yd;
    S.ef[pid] = (uint32_t)e | (side ? kSideBit : 0u);
    S.y32[pid] = make_float2(yh, (float)(yd - (double)yh));
  }
  if (S.seqhash) S.seqhash[pid] = 0xcbf29ce484222325ull;
  if (S.hits) S.hits[pid] = 0;
}

// ----------------------------------------------------------- histogram --
// The four particles 4 i .. 4 i + 3 of a set (those below n): state words and
// positions in one wide load each.
template <bool FP64>
struct Quad {
  uint32_t ef[4];
  double2 x[2];   // FP64
  float4 y[2];    // FP32
  __device__ __forceinline__ void load(const SetDev &S, uint32_t i) {
    const uint4 e = ((const uint4 *)S.ef)[i];
    ef[0] = e.x, ef[1] = e.y, ef[2] = e.z, ef[3] = e.w;
    if (FP64) {
      x[0] = ((const double2 *)S.x64)[2 * i];
      x[1] = ((const double2 *)S.x64)[2 * i + 1];
    } else {
      y[0] = ((const float4 *)S.y32)[2 * i];
      y[1] = ((const float4 *)S.y32)[2 * i + 1];
    }
  }
  __device__ __forceinline__ void load_tail(const SetDev &S, uint32_t first) {
    for (uint32_t k = 0; k < 4; ++k) {
      const uint32_t id = first + k;
      ef[k] = id < S.n ? S.ef[id] : kDeadBit;
      const uint32_t at = id < S.n ? id : first;
      if (FP64) {
        const double v = S.x64[at];
        (k & 1u ? x[k >> 1].y : x[k >> 1].x) = v;
      } else {
        const float2 v = S.y32[at];
        if (k & 1u)
          y[k >> 1].z = v.x, y[k >> 1].w = v.y;
        else
          y[k >> 1].x = v.x, y[k >> 1].y = v.y;
      }
    }
  }
  // position of particle k from the initial vertex of its edge of length L
  __device__ __forceinline__ double pos(uint32_t k, double L) const {
    if (FP64) return k & 1u ? x[k >> 1].y : x[k >> 1].x;
    const float4 &v = y[k >> 1];
    const double d = k & 1u ? (double)v.z + (double)v.w : (double)v.x + (double)v.y;
    return (ef[k] & kSideBit) ? L - d : d;
  }
};

// Calls f(quad, k) for every alive particle of the set, four per thread and
// turn, over the whole grid.
template <bool FP64, typename F>
__device__ __forceinline__ void for_alive(const SetDev &S, F &&f) {
  const uint32_t quads = S.n / 4u, stride = gridDim.x * blockDim.x;
  Quad<FP64> q;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < quads; i += stride) {
    q.load(S, i);
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
      if (!(q.ef[k] & kDeadBit)) f(q, k);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && (S.n & 3u)) {
    q.load_tail(S, 4u * quads);
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
      if (!(q.ef[k] & kDeadBit)) f(q, k);
  }
}

// Adds a block's LDS bins to the u64 counters.
__device__ __forceinline__ void merge_bins(const uint32_t *s_bin, int32_t nbins, uint64_t *out) {
  for (int32_t b = threadIdx.x; b < nbins; b += blockDim.x)
    if (s_bin[b]) atomicAdd((unsigned long long *)&out[b], (unsigned long long)s_bin[b]);
}

// Uniform bins in LDS: [the edges' {length, inverse bin width}][bins].  Bound
// by the latency of its loads (few blocks fit beside a copy of the bins), so
// 16 waves share a copy and a thread takes four particles per turn, and the
// inverse widths are made once per block: 1e7 particles on 64 edges of 256
// bins 34 us, where one particle per turn in blocks of four waves took 111;
// 1e6 particles 57 -> 10 us.
template <bool FP64>
__global__ __launch_bounds__(kHistBlock) void k_hist_lds(GraphDev G, SetDev S, int32_t nb,
                                                         int32_t edges, uint64_t *out) {
  extern __shared__ uint4 smem4[];
  const int32_t nbins = G.E * nb;
  double2 *s_edge = (double2 *)smem4;   // edges = G.E, or 0: from the records
  uint32_t *s_bin = (uint32_t *)(s_edge + edges);
  for (int32_t b = threadIdx.x; b < nbins; b += blockDim.x) s_bin[b] = 0;
  for (int32_t e = threadIdx.x; e < edges; e += blockDim.x)
    s_edge[e] = make_double2(G.e64[e].L, (double)nb / G.e64[e].span);
  __syncthreads();
  for_alive<FP64>(S, [&](const Quad<FP64> &q, uint32_t k) {
    const int32_t e = (int32_t)(q.ef[k] & kEdgeMask);
    const double2 r = edges ? s_edge[e]
                            : make_double2(G.e64[e].L, (double)nb / G.e64[e].span);
    atomicAdd(&s_bin[e * nb + bin_at(q.pos(k, r.x), r.y, nb)], 1u);
  });
  __syncthreads();
  merge_bins(s_bin, nbins, out);
}

// Uniform bins too many for LDS: 64-bit global atomics, about 2.2e10 a second
// whatever the number of bins beyond 32768, but one after another (12 ns) where
// many particles share a bin.  So a block first counts in a table of recent
// bins in LDS, buckets of two by the bin's hash: a bin that finds an entry of
// its own, or an empty one, counts there, any other in global memory; every
// kHotTurns turns the entries go to the counters and the table starts anew, so
// that bins of a part of the set are found too; lanes left to global memory add
// up within the wave.  1e7 FP32 particles, by atomics alone and with the table:
// 76800 bins, even 455 -> 453 us, all in one bin 120021 -> 105, in ten bins 12048
// -> 102, the second half in one bin 60064 -> 340 (703 where the table is kept
// for 8 turns), in 1000 bins 459 -> 307; 1.7e6 bins, even 478 -> 480, at the
// vascular network's inlets 1228 -> 521; 1e8 particles on the network 4.65 ->
// 4.55 ms.  (A pass per range of edges whose bins fit in LDS takes 250 us for
// 76800 bins and 2.5 ms for 1.7e6 where the particles gather, and more than the
// atomics where they do not.)
constexpr uint32_t kHotBuckets = 256, kHotTurns = 2, kNoBin = 0xFFFFFFFFu;
template <bool FP64>
__global__ __launch_bounds__(kBlock) void k_hist_global(GraphDev G, SetDev S, int32_t nb,
                                                            uint64_t *out) {
  __shared__ alignas(8) uint32_t s_bin[2 * kHotBuckets];
  __shared__ uint32_t s_cnt[2 * kHotBuckets];
  auto add = [&](uint32_t bin, uint32_t n) {
    atomicAdd((unsigned long long *)&out[bin], (unsigned long long)n);
  };
  // the active lanes' bins, one addition for lanes of one bin while that saves
  // at least three
  auto add_together = [&](uint32_t bin) {
    for (;;) {
      const uint32_t b = __builtin_amdgcn_readfirstlane(bin);
      const uint64_t same = ballot(bin == b);
      const uint32_t n = (uint32_t)__popcll(same);
      if (n < 4u) {
        add(bin, 1u);
        return;
      }
      if (bin == b) {
        if (lane_rank(same) == 0u) add(b, n);
        return;
      }
    }
  };
  auto bin_of_particle = [&](const Quad<FP64> &q, uint32_t k) {
    const int32_t e = (int32_t)(q.ef[k] & kEdgeMask);
    const EdgeRec64 &r = G.e64[e];
    return (uint32_t)(e * nb + bin_of(q.pos(k, r.L), r.span, nb));
  };
  for (uint32_t i = threadIdx.x; i < 2 * kHotBuckets; i += kBlock)
    s_bin[i] = kNoBin, s_cnt[i] = 0;
  __syncthreads();
  auto flush_table = [&]() {
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < 2 * kHotBuckets; i += kBlock) {
      if (s_cnt[i]) add(s_bin[i], s_cnt[i]);
      s_bin[i] = kNoBin, s_cnt[i] = 0;
    }
    __syncthreads();
  };
  // whether `bin` has (or now has) entry i, which held `held` when last read
  auto owns = [&](uint32_t i, uint32_t held, uint32_t bin) {
    if (held == kNoBin) held = atomicCAS(&s_bin[i], kNoBin, bin);
    return held == bin || held == kNoBin;
  };
  const uint32_t quads = S.n / 4u, stride = gridDim.x * kBlock;
  uint32_t turns = 0;
  Quad<FP64> q;
  for (uint32_t first = blockIdx.x * kBlock; first < quads; first += stride) {
    const uint32_t id = first + threadIdx.x;
    if (id < quads) {
      q.load(S, id);
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        if (q.ef[k] & kDeadBit) continue;
        const uint32_t bin = bin_of_particle(q, k);
        const uint32_t i = 2u * ((bin * 2654435769u) >> 24);  // 256 buckets
        const volatile uint32_t *held = &s_bin[i];
        const uint32_t h0 = held[0], h1 = held[1];
        if (h0 == bin || (h1 != bin && owns(i, h0, bin)))
          atomicAdd(&s_cnt[i], 1u);
        else if (h1 == bin || owns(i + 1u, h1, bin))
          atomicAdd(&s_cnt[i + 1u], 1u);
        else
          add_together(bin);
      }
    }
    if (++turns == kHotTurns) {
      turns = 0;
      flush_table();
    }
  }
  flush_table();
  if (blockIdx.x == 0 && threadIdx.x == 0 && (S.n & 3u)) {
    q.load_tail(S, 4u * quads);
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
      if (!(q.ef[k] & kDeadBit)) add(bin_of_particle(q, k), 1u);
  }
}

// Histogram over per-edge bins of any widths (the appendix's general
// histogram kernel): the bins of edge e are off[e] .. off[e+1]-1 with upper
// boundaries up[] (FP64, strictly increasing along the edge).  A particle at
// x takes the first bin whose upper boundary is >= x (binary search), or the
// edge's last bin.
template <bool FP64, bool LDS>
__global__ __launch_bounds__(kHistBlock) void k_hist_csr(GraphDev G, SetDev S,
                                                         const int32_t *off, const double *up,
                                                         int32_t nbins, uint64_t *out) {
  extern __shared__ uint4 smem4[];
  uint32_t *s_bin = (uint32_t *)smem4;
  if (LDS) {
    for (int32_t b = threadIdx.x; b < nbins; b += blockDim.x) s_bin[b] = 0;
    __syncthreads();
  }
  for_alive<FP64>(S, [&](const Quad<FP64> &q, uint32_t k) {
    const int32_t e = (int32_t)(q.ef[k] & kEdgeMask);
    const double x = q.pos(k, FP64 ? 0.0 : G.e64[e].L);
    int32_t lo = off[e], hi = off[e + 1] - 1;  // the answer lies in [lo, hi]
    while (lo < hi) {
      const int32_t mid = (lo + hi) >> 1;
      if (x <= up[mid])
        hi = mid;
      else
        lo = mid + 1;
    }
    if (LDS)
      atomicAdd(&s_bin[lo], 1u);
    else
      atomicAdd((unsigned long long *)&out[lo], 1ull);
  });
  if (LDS) {
    __syncthreads();
    merge_bins(s_bin, nbins, out);
  }
}

// ------------------------------------------------------------ readback --
// Writes go straight to pinned host memory: one launch and one wait where
// separate copies into pageable memory each took a wait of their own.
__global__ __launch_bounds__(kBlock) void k_copy_out(CopyOut c) {
  const int32_t s = (int32_t)blockIdx.y;
  const uint32_t words = c.words[s], quads = words / 4u, stride = gridDim.x * kBlock;
  const uint32_t i0 = blockIdx.x * kBlock + threadIdx.x;
  for (uint32_t i = i0; i < quads; i += stride) ((uint4 *)c.dst[s])[i] = ((const uint4 *)c.src[s])[i];
  if (i0 < (words & 3u))
    ((uint32_t *)c.dst[s])[4u * quads + i0] = ((const uint32_t *)c.src[s])[4u * quads + i0];
}

template <bool FP64>
__global__ __launch_bounds__(kBlock) void k_read(GraphDev G, SetDev S, uint32_t first,
                                                 uint32_t count, int32_t *edge, double *pos,
                                                 uint8_t *alive, uint64_t *hash,
                                                 uint32_t *hits) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count) return;
  const uint32_t id = first + i, ef = S.ef[id];
  const int32_t e = (int32_t)(ef & kEdgeMask);
  if (edge) edge[i] = e;
  if (alive) alive[i] = (ef & kDeadBit) ? 0 : 1;
  if (pos) {
    if (FP64) {
      pos[i] = S.x64[id];
    } else {
      const float2 yy = S.y32[id];
      const double y = (double)yy.x + (double)yy.y;
      pos[i] = (ef & kSideBit) ? (e < G.E ? G.e64[e].L : 0.0) - y : y;
    }
  }
  if (hash) hash[i] = S.seqhash[id];
  if (hits) hits[i] = S.hits[id];
}

// Calls f(std::bool_constant<x>...) for the run-time flags, so one launch
// site covers every compiled variant.
template <typename F>
void with_flags(F &&f) {
  f();
}
template <typename F, typename... Rest>
void with_flags(F &&f, bool x, Rest... rest) {
  if (x)
    with_flags([&](auto... v) { f(std::true_type{}, v...); }, rest...);
  else
    with_flags([&](auto... v) { f(std::false_type{}, v...); }, rest...);
}

// The graph's method-variant level as a compile-time constant: 0 affine
// coefficients, kGenCubic cubic ones, kGenFull tables or Wentzell vertices.
template <typename F>
void with_gen(int32_t level, F &&f) {
  if (level == kGenFull)
    f(std::integral_constant<int, kGenFull>{});
  else if (level == kGenCubic)
    f(std::integral_constant<int, kGenCubic>{});
  else
    f(std::integral_constant<int, 0>{});
}

// Particles per wave of an FP32 wave-pool schedule (StepArgs::kernel 1, 2, 3).
template <typename F>
void with_pool(int32_t kernel, F &&f) {
  if (kernel == 2)
    f(std::integral_constant<int, kPoolLarge>{});
  else
    f(std::integral_constant<int, kPoolSmall>{});
}

// LDS layout of a step block, shared by the host launchers and the
// kernels' offsets: [FP64: Box-Muller tables][exit counters][staged
// tables][pools][snapshot bins].
// Within kLdsBlockMax bytes, exit counters come first (they take an atomic
// per hit-step), staged tables next, snapshot bins last.  What a block keeps
// beside those (the Box-Muller tables, the snapshot counts of its home slots)
// comes on top: counters that leave LDS cost an atomic on the set's own at
// every hit, one at a time where few slots take the exits.  50 steps of 3e5
// particles that leave a star's centre by 4 of its edges, exits counted in LDS
// against beyond: FP64 pools with 9600 slots 0.53 against 3.9 ms, FP64 lanes
// with 15200 0.45 against 4.1, FP32 pools with streaming and 10800 1.4 against
// 4.1 (all slots taking their share: 0.43 against 0.24, 0.34 against 0.23, 0.5
// against 0.25).
struct LdsPlan {
  bool lds_exit;
  bool staged;
  int32_t obs_lds;  // snapshot bins in LDS, 0: global counters
  size_t shm;
};

// pools: bytes of the block's pools; beside: of them and of the tables, those
// on top of kLdsBlockMax (beside_bytes).
LdsPlan plan_lds(bool fp64, int32_t nnz, int32_t stage, size_t pools, size_t beside,
                 const SetDev *obs_set, int32_t n_edges) {
  const size_t most = (size_t)kLdsBlockMax + beside;
  LdsPlan p{};
  p.lds_exit = nnz <= kLdsExitMax;
  p.staged = stage > 0;
  auto size = [&]() {
    const int32_t ex = p.lds_exit ? ((nnz * 4 + 15) & ~15) : 0;
    const size_t b = (fp64 ? sizeof(BmLds) : 0) +
                     (size_t)((ex + (p.staged ? stage : 0) + 15) & ~15) + pools;
    return (b + 15) & ~(size_t)15;
  };
  if (size() > most) p.staged = false;
  if (size() > most) p.lds_exit = false;
  const size_t base = size();
  p.shm = base;
  if (obs_set && obs_set->obs) {
    const int64_t nbins = (int64_t)n_edges * obs_set->obs_nb;
    if (nbins <= kLdsObsMax && base + (size_t)nbins * 4 <= most) {
      p.obs_lds = (int32_t)nbins;
      p.shm = base + (size_t)nbins * 4;
    }
  }
  return p;
}

// The bytes that a block's LDS holds on top of kLdsBlockMax: the FP64 tables
// and, in pools of PW (0: the lane schedule), the snapshot counts.
template <int PW, bool FP64, bool TRACE>
size_t beside_bytes(bool obs) {
  size_t b = FP64 ? sizeof(BmLds) : 0;
  if constexpr (PW > 0)
    b += (pool_lds_bytes<PW, FP64, TRACE>(obs) - pool_lds_bytes<PW, FP64, TRACE>(false)) *
         kWavesPerBlock;
  return b;
}

// Lanes without a particle that end a wave pool's window of groups while there
// are others for them.  A refill costs about 70 VALU instructions whatever the
// number of lanes it serves, a group of steps 97: at 1 / 8 / 16 / 24 lanes 2000
// steps of 1e7 FP32 particles on the 64-edge star take 32.4 / 32.3 / 31.2 /
// 31.3 ms at 7.1 % hits a step, 23.1 / 21.2 / 20.7 / 21.9 at 2.1 %, and 1000
// steps of 3e7 on the vascular network (0.35 %) 19.3 / 18.6 / 19.2 / 20.4.
// Hence 16 lanes where the launch stages its tables in LDS (FP64, 16 against 8:
// 55.2 against 56.2 ms for 2000 steps of 1e7 on the 64-edge star).  An FP32
// refill that reads them from global memory waits for loads that the other
// lanes' steps hide: it pays earlier where hits are few, later where they are
// many.  1e7 particles, 300 steps, at 8 / 16 lanes by the hits that diffusion
// makes: vascular network 0.2 % 1.89 / 1.95 ms; tree of 2000 edges 0.2 % 2.52 /
// 2.56, 0.4 % 2.71 / 2.74, 1.0 % 3.30 / 3.27, 1.4 % 3.81 / 3.55; star of 2000
// 0.8 % 3.12 / 3.11, 1.1 % 3.43 / 3.35, 2.5 % 4.77 / 4.44; Langevin star of 1000
// 0.9 % 2.86 / 2.91, 1.8 % 3.47 / 3.44, 2.9 % 4.48 / 4.02; star of 4000, 500
// steps, 2.5 % 8.30 / 7.59.  Hence 16 there from 1 % on, and 8 below.
// In a batch 16 in every group: 64 uneven sets, 1000 steps, 18.1 against 18.8 ms
// with 8 in the groups that read from global memory; four trees of 600 to 2500
// edges, 8e6 particles, 300 steps of 10^-2, 5.0 against 5.4.
int32_t refill_lanes(int32_t kernel, bool fp64, bool late, int32_t far) {
  return kernel != 3 ? 8 : fp64 || late ? 16 : far;
}

// Compute units of the current device, looked up once.
uint32_t device_cus() {
  static std::mutex mu;
  static int cus[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  std::lock_guard<std::mutex> lock(mu);
  if (cus[dev] <= 0 &&
      (hipDeviceGetAttribute(&cus[dev], hipDeviceAttributeMultiprocessorCount, dev) !=
           hipSuccess ||
       cus[dev] <= 0))
    cus[dev] = 256;
  return (uint32_t)cus[dev];
}

// Particles that a wave of a pool launch holds at a time, and the blocks
// that the set then fills.  A full pool (two particles per lane) pays once
// the set fills the chip's waves; below that a launch takes as long as one
// wave needs for its share, so the set is spread over more waves: 16 or 32
// particles each while that leaves at most one wave per SIMD, 64 (a particle
// per lane) while it leaves at most two.  1000 steps, us, at 128 / 64 / 32 /
// 16 particles a wave: 1e4 particles on the 3-edge star in FP64 1076 / 710 /
// 669 / 658, on the 64-edge star in FP32 930 / 716 / 699 / 655; 3e4 (1114 /
// 788 / 735 / 900, 939 / 729 / 711 / 735); 1e5 (1144 / 1006 / 1452 / 2090,
// 964 / 822 / 1078 / 1465); 3e5 (1986 / 1914 / 3135 / -, 1266 / 1298 / 2065
// / -).  The lanes that stand idle before a refill or a partial split pass
// shrink with the pool.
//
// The reservations of a launch of 32 steps or more also leave every SIMD
// eight of them (or a pool's worth each), and in FP32 64 particles a wave last
// up to the six waves a SIMD that are resident, four at the full general level
// (3e5 particles with 8 tabulated edges, streaming, 200 steps 760 us at 64,
// 660 at 128; FP64 has three or four: 2e5 particles with tabulated
// coefficients 3.7 ms at 128, 4.1 at 64).  A reservation is one wave's serial
// work, and the 240 ids
// that keep the counter's updates cheap at 500 steps left 3e5 particles to
// 1250 waves.  FP32, 500 steps of 1.5e5 / 3e5 / 1e6 / 3e6 particles on the
// 64-edge star 0.80 / 0.90 / 1.46 / 2.51 -> 0.47 / 0.63 / 1.18 / 2.51 ms, 50
// steps 0.14 / 0.22 / 0.46 / 0.60 -> 0.12 / 0.17 / 0.29 / 0.44; on the 5-edge
// star with 2 hits a step 12.4 / 13.8 / 21.3 / 41.3 -> 4.6 / 6.2 / 14.9 / 41.6.
// Shorter launches are bound by the updates and keep the large reservations.
// From 96 steps on it is sixteen: the waves start together on their places in
// the grid, and with eight a SIMD, for its five or six waves, a third of them
// took a second turn while the others stood idle, by which of them came first.
// 2e6 FP32 particles, counter alone / places with eight / with sixteen: 400
// steps on the 64-edge star with trace 1520 / 1580 / 1457 us, streaming 1920 /
// 1880 to 2560 / 1690, on the star of 4000 edges, streaming, 3475 / 3680 / 3430;
// 100 steps on the 5-edge star with drifts 2200 / 2110 to 2690 / 2110.  At 60
// steps eight are the faster (the network 238 against 308 us).  (Reservations
// of one turn for all, where there are fewer than two, lose up to 26 %: 1000
// steps of 1e6 on that 5-edge star.)
uint32_t set_pool(StepArgs &a, uint32_t n, int32_t pool, bool fp64, bool full) {
  const uint32_t simds = 4u * device_cus();
  uint32_t cap = (uint32_t)pool;
  if (n <= 16u * simds)
    cap = 16;
  else if (n <= 32u * simds)
    cap = 32;
  else if (n <= (a.nsteps < 32u || fp64 ? 2u : full ? 4u : 6u) * 64u * simds)
    cap = 64;
  const int32_t lanes = (int32_t)std::min<uint32_t>(cap, 64u);
  a.pool_cap = cap;
  a.idle = std::max(1, a.idle * lanes / 64);
  a.refill = std::max(1, a.refill * lanes / 64);
  if (cap < (uint32_t)pool) a.claim_chunk = std::min(a.claim_chunk, cap);
  if (a.nsteps >= 32u)
    a.claim_chunk = std::min(a.claim_chunk,
                             std::max(cap, (n / ((a.nsteps < 96u ? 8u : 16u) * simds)) & ~15u));
  const uint32_t per_block = cap * kWavesPerBlock;
  return (n + per_block - 1) / per_block;
}

// The blocks of a set's own pool launch, whose waves take their places in the
// grid as first reservations; its counter is set behind them.
uint32_t own_claims(const void *func, size_t shm, uint32_t need, const SetDev &s,
                    const StepArgs &a, hipStream_t st) {
  const uint32_t blocks = resident_blocks(func, shm, need);
  hipLaunchKernelGGL(k_set_word, dim3(1), dim3(64), 0, st, s.work,
                     blocks * kWavesPerBlock * a.claim_chunk);
  return blocks;
}

template <bool FP64, bool TRACE>
hipError_t launch_step_t(const GraphDev &g, const SetDev &s, const StepArgs &a0,
                         hipStream_t st) {
  StepArgs a = a0;
  const bool obs = s.obs != nullptr;
  if constexpr (FP64) {
    if (a.kernel == 3) {
      // FP64 wave pools (128 per wave) on a resident grid
      const LdsPlan lp = plan_lds(true, g.nnz, g.stage_bytes64,
                                  pool_lds_bytes<kPoolSmall, true, TRACE>(obs) * kWavesPerBlock,
                                  beside_bytes<kPoolSmall, true, TRACE>(obs), &s, g.E);
      a.obs_lds = lp.obs_lds;
      a.refill = refill_lanes(a.kernel, true, lp.staged, a.refill);
      const uint32_t need = set_pool(a, s.n, kPoolSmall, true, g.gen == kGenFull);
      with_gen(g.gen, [&](auto Gn) {
        constexpr int gn = decltype(Gn)::value;
        with_flags([&](auto L, auto T, auto O) {
          constexpr bool l = decltype(L)::value, t = decltype(T)::value,
                         o = decltype(O)::value;
          const void *f = (const void *)k_pool64<TRACE, l, t, o, gn>;
          const uint32_t blocks = own_claims(f, lp.shm, need, s, a, st);
          hipLaunchKernelGGL((k_pool64<TRACE, l, t, o, gn>),
                             dim3(blocks), dim3(kBlock), lp.shm, st,
                             g, s, a);
        }, lp.lds_exit, lp.staged, obs);
      });
      return hipGetLastError();
    }
  }
  if (!FP64 && a.kernel >= 1 && (!g.gen || a.kernel == 3)) {
    with_pool(a.kernel, [&](auto PWc) {
      constexpr int PW = decltype(PWc)::value;
      const int32_t stage = g.stage_bytes32;
      const LdsPlan lp = plan_lds(false, g.nnz, stage,
                                  pool_lds_bytes<PW, false, TRACE>(obs) * kWavesPerBlock,
                                  beside_bytes<PW, false, TRACE>(obs), &s, g.E);
      a.obs_lds = lp.obs_lds;
      a.refill = refill_lanes(a.kernel, false, lp.staged, a.refill);
      const uint32_t need = set_pool(a, s.n, PW, false, g.gen == kGenFull);
      if (!TRACE && !obs && a.probe) {
        with_flags([&](auto L, auto T) {
          const void *f =
              (const void *)k_pool32_probe<decltype(L)::value, decltype(T)::value, PW>;
          const uint32_t blocks = own_claims(f, lp.shm, need, s, a, st);
          hipLaunchKernelGGL((k_pool32_probe<decltype(L)::value, decltype(T)::value, PW>),
                             dim3(blocks), dim3(kBlock), lp.shm, st,
                             g, s, a);
        }, lp.lds_exit, lp.staged);
        return;
      }
      if constexpr (PW == kPoolSmall) {
        if (g.gen) {
          with_gen(g.gen, [&](auto Gn) {
            constexpr int gn = decltype(Gn)::value;
            if constexpr (gn != 0)
              with_flags([&](auto L, auto T, auto O) {
                const void *f =
                    (const void *)k_pool32<TRACE, decltype(L)::value, decltype(T)::value,
                                           decltype(O)::value, PW, gn>;
                const uint32_t blocks = own_claims(f, lp.shm, need, s, a, st);
                hipLaunchKernelGGL((k_pool32<TRACE, decltype(L)::value, decltype(T)::value,
                                             decltype(O)::value, PW, gn>),
                                   dim3(blocks), dim3(kBlock),
                                   lp.shm, st, g, s, a);
              }, lp.lds_exit, lp.staged, obs);
          });
          return;
        }
      }
      with_flags([&](auto L, auto T, auto O) {
        const void *f = (const void *)k_pool32<TRACE, decltype(L)::value, decltype(T)::value,
                                               decltype(O)::value, PW>;
        const uint32_t blocks = own_claims(f, lp.shm, need, s, a, st);
        hipLaunchKernelGGL((k_pool32<TRACE, decltype(L)::value, decltype(T)::value,
                                     decltype(O)::value, PW>),
                           dim3(blocks), dim3(kBlock), lp.shm, st,
                           g, s, a);
      }, lp.lds_exit, lp.staged, obs);
    });
    return hipGetLastError();
  }
  const int32_t stage = FP64 ? g.stage_bytes64 : g.stage_bytes32;
  const LdsPlan lp =
      plan_lds(FP64, g.nnz, stage, 0, beside_bytes<0, FP64, TRACE>(obs), &s, g.E);
  a.obs_lds = lp.obs_lds;
  const uint32_t blocks = (s.n + kBlock - 1) / kBlock;
  if (!FP64 && !TRACE && !obs && a.probe) {
    with_flags([&](auto L, auto T) {
      hipLaunchKernelGGL((k_step32_probe<decltype(L)::value, decltype(T)::value>),
                         dim3(blocks), dim3(kBlock), lp.shm, st, g, s, a);
    }, lp.lds_exit, lp.staged);
    return hipGetLastError();
  }
  with_gen(g.gen, [&](auto Gn) {
    constexpr int gn = decltype(Gn)::value;
    with_flags([&](auto L, auto T, auto O) {
      hipLaunchKernelGGL((k_step<FP64, TRACE, decltype(L)::value, decltype(T)::value,
                                 decltype(O)::value, gn>),
                         dim3(blocks), dim3(kBlock), lp.shm, st, g, s, a);
    }, lp.lds_exit, lp.staged, obs);
  });
  return hipGetLastError();
}

// Batched launches keep snapshot bins in global memory (the sets differ).
template <bool FP64, bool TRACE>
KernelLaunch batch_launch_t(int32_t n_items, int32_t max_nnz, int32_t max_stage,
                            const StepArgs &a, bool obs, int32_t gen) {
  KernelLaunch k{};
  k.grid = dim3(n_items);
  k.block = dim3(kBlock);
  k.persistent = false;
  // FP32: the wave pools of the set's schedule (only MG_SCHED_POOLS_W8 for
  // the general levels); FP64: its wave pools
  const bool pools = FP64 ? a.kernel == 3 : (a.kernel >= 1 && (!gen || a.kernel == 3));
  with_pool(a.kernel, [&](auto PWc) {
    constexpr int PW = decltype(PWc)::value;
    constexpr int P = FP64 ? kPoolSmall : PW;
    const size_t pool_bytes = pool_lds_bytes<P, FP64, TRACE>(obs) * kWavesPerBlock;
    const LdsPlan lp = plan_lds(FP64, max_nnz, max_stage, pools ? pool_bytes : 0,
                                pools ? beside_bytes<P, FP64, TRACE>(obs)
                                      : beside_bytes<0, FP64, TRACE>(obs), nullptr, 0);
    k.shm = lp.shm;
    k.refill = refill_lanes(a.kernel, FP64, true, a.refill);
    with_gen(gen, [&](auto Gn) {
      constexpr int gn = decltype(Gn)::value;
      with_flags([&](auto L, auto T, auto O) {
        constexpr bool l = decltype(L)::value, t = decltype(T)::value, o = decltype(O)::value;
        if (pools) {
          if constexpr (FP64) {
            k.func = (const void *)k_pool64_batch<TRACE, l, t, o, gn>;
          } else {
            k.func = (const void *)k_pool32_batch<TRACE, l, t, o, PW>;
            if constexpr (PW == kPoolSmall && gn != 0)
              k.func = (const void *)k_pool32_batch<TRACE, l, t, o, PW, gn>;
          }
          // a resident grid takes the items from the batch's counter
          k.persistent = true;
          k.grid = dim3(resident_blocks(k.func, k.shm, (uint32_t)n_items));
          return;
        }
        k.func = (const void *)k_batch<FP64, TRACE, l, t, o, gn>;
      }, lp.lds_exit, lp.staged, obs);
    });
  });
  return k;
}

}  // namespace

hipError_t launch_init(const GraphDev &g, const SetDev &s, int mode, int32_t vertex,
                       uint32_t key0, uint32_t key1, const int32_t *edge_in,
                       const double *pos_in, const InitSources &src, bool fp64,
                       hipStream_t st) {
  const uint32_t blocks = (s.n + kBlock - 1) / kBlock;
  if (fp64)
    hipLaunchKernelGGL(k_init<true>, dim3(blocks), dim3(kBlock), 0, st, g, s, mode,
                       vertex, key0, key1, edge_in, pos_in, src);
  else
    hipLaunchKernelGGL(k_init<false>, dim3(blocks), dim3(kBlock), 0, st, g, s, mode,
                       vertex, key0, key1, edge_in, pos_in, src);
  return hipGetLastError();
}

hipError_t launch_step(const GraphDev &g, const SetDev &s, const StepArgs &a,
                       bool fp64, bool trace, hipStream_t st) {
  if (fp64) return trace ? launch_step_t<true, true>(g, s, a, st)
                         : launch_step_t<true, false>(g, s, a, st);
  return trace ? launch_step_t<false, true>(g, s, a, st)
               : launch_step_t<false, false>(g, s, a, st);
}

int32_t far_refill(double hits) { return hits >= 0.01 ? 16 : 8; }

int32_t pool_refill(const GraphDev &g, int32_t kernel, int32_t far) {
  bool staged = false;
  with_pool(kernel, [&](auto PWc) {
    const size_t pools = pool_lds_bytes<decltype(PWc)::value, false, false>(false);
    staged =
        plan_lds(false, g.nnz, g.stage_bytes32, pools * kWavesPerBlock, 0, nullptr, 0).staged;
  });
  return refill_lanes(kernel, false, staged, far);
}

const void *batch_reset_kernel() { return (const void *)k_batch_reset; }

int32_t batch_blocks_per_cu(int32_t max_nnz, int32_t max_stage, const StepArgs &a, bool fp64,
                            bool trace, int32_t gen, bool *staged) {
  const KernelLaunch k = batch_launch(1, max_nnz, max_stage, a, fp64, trace, false, gen);
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k.func, kBlock, k.shm) !=
          hipSuccess ||
      per_cu <= 0)
    per_cu = 1;
  if (staged) {
    // the plan stages the tables when their bytes are part of its LDS
    const KernelLaunch k0 = batch_launch(1, max_nnz, 0, a, fp64, trace, false, gen);
    *staged = max_stage > 0 && k.shm > k0.shm;
  }
  return per_cu;
}

int32_t batch_tile(bool fp64, int32_t kernel) {
  const bool pools = fp64 ? kernel == 3 : kernel >= 1;
  return pools ? pool_per_wave(kernel) * kWavesPerBlock * kBatchGens : kBlock;
}

KernelLaunch batch_launch(int32_t n_items, int32_t max_nnz, int32_t max_stage,
                          const StepArgs &a, bool fp64, bool trace, bool obs, int32_t gen) {
  if (fp64)
    return trace ? batch_launch_t<true, true>(n_items, max_nnz, max_stage, a, obs, gen)
                 : batch_launch_t<true, false>(n_items, max_nnz, max_stage, a, obs, gen);
  return trace ? batch_launch_t<false, true>(n_items, max_nnz, max_stage, a, obs, gen)
               : batch_launch_t<false, false>(n_items, max_nnz, max_stage, a, obs, gen);
}

// Blocks of an LDS histogram: reading falls with their number, merging their
// copies into the counters grows with it, so the best number goes with the
// square root of particles per bin (16384 bins: 64 blocks for 1e6 particles
// 10 us, 16 blocks 15, 512 blocks 27; 128 for 1e7 34 us, 16 blocks 148, 512
// blocks 68).
static uint32_t lds_hist_blocks(uint32_t n, int64_t nbins) {
  const double best = 5.0 * std::sqrt((double)n / (double)std::max<int64_t>(nbins, 1));
  const uint32_t most = std::min((n + 4095u) / 4096u, 512u);
  return std::max(1u, std::min((uint32_t)best, most));
}

hipError_t launch_histogram_csr(const GraphDev &g, const SetDev &s, const int32_t *off,
                                const double *up, int32_t nbins, uint64_t *out, bool fp64,
                                hipStream_t st) {
  const bool lds = nbins <= kLdsHistMax;
  const size_t shm = lds ? (size_t)nbins * 4 : 0;
  // (a particle's search takes longer than a uniform bin, so a block per CU
  // pays before the copies' merging does: 1e6 / 1e7 FP32 particles on 16384 bins
  // with 64 / 123 blocks 148 / 385 us, with 256 97 / 281, with 512 97 / 316; all
  // on 64 of the bins 156 / 365, 68 / 210, 68 / 214)
  const uint32_t blocks =
      lds ? std::max(lds_hist_blocks(s.n, nbins), std::min((s.n + 1023u) / 1024u, 256u))
          : std::min((s.n + 4095u) / 4096u, 2048u);
  with_flags([&](auto F, auto L) {
    hipLaunchKernelGGL((k_hist_csr<decltype(F)::value, decltype(L)::value>), dim3(blocks),
                       dim3(kHistBlock), shm, st, g, s, off, up, nbins, out);
  }, fp64, lds);
  return hipGetLastError();
}

// Clears n 64-bit words (a kernel rather than a memset, so that callers
// may capture the work in a HIP graph).
__global__ __launch_bounds__(kBlock) void k_fill_zero_u64(uint64_t *p, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) p[i] = 0ull;
}

hipError_t launch_fill_zero_u64(uint64_t *p, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + kBlock - 1) / kBlock;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_zero_u64, dim3((uint32_t)blocks), dim3(kBlock), 0, st, p, n);
  return hipGetLastError();
}

hipError_t launch_copy_out(const CopyOut &c, hipStream_t st) {
  uint32_t most = 1;
  for (int32_t i = 0; i < c.n; ++i) most = std::max(most, c.words[i]);
  const uint32_t blocks = std::min((most / 4u + kBlock) / kBlock, 256u);
  hipLaunchKernelGGL(k_copy_out, dim3(blocks, (uint32_t)c.n), dim3(kBlock), 0, st, c);
  return hipGetLastError();
}

hipError_t launch_read(const GraphDev &g, const SetDev &s, uint32_t first, uint32_t count,
                       int32_t *edge, double *pos, uint8_t *alive, uint64_t *hash,
                       uint32_t *hits, bool fp64, hipStream_t st) {
  const dim3 blocks((count + kBlock - 1) / kBlock);
  with_flags([&](auto F) {
    hipLaunchKernelGGL(k_read<decltype(F)::value>, blocks, dim3(kBlock), 0, st, g, s, first,
                       count, edge, pos, alive, hash, hits);
  }, fp64);
  return hipGetLastError();
}

hipError_t launch_obs_edges(const GraphDev &g, int32_t nb, double2 *out, hipStream_t st) {
  hipLaunchKernelGGL(k_obs_edges, dim3((g.E + kBlock - 1) / kBlock), dim3(kBlock), 0, st, g.e64,
                     g.E, nb, out);
  return hipGetLastError();
}

hipError_t launch_histogram(const GraphDev &g, const SetDev &s, int32_t nb,
                            uint64_t *out, bool fp64, hipStream_t st) {
  const int64_t nbins = (int64_t)g.E * nb;
  if (nbins <= kLdsHistMax) {
    const int32_t edges = g.E <= kLdsHistEdges ? g.E : 0;
    const size_t shm = (size_t)nbins * 4 + (size_t)edges * 16;
    with_flags([&](auto F) {
      hipLaunchKernelGGL((k_hist_lds<decltype(F)::value>), dim3(lds_hist_blocks(s.n, nbins)),
                         dim3(kHistBlock), shm, st, g, s, nb, edges, out);
    }, fp64);
    return hipGetLastError();
  }
  const uint32_t blocks = std::min((s.n + 4 * kBlock - 1) / (4 * kBlock), 2048u);
  with_flags([&](auto F) {
    hipLaunchKernelGGL((k_hist_global<decltype(F)::value>), dim3(blocks), dim3(kBlock), 0, st, g,
                       s, nb, out);
  }, fp64);
  return hipGetLastError();
}

}  // namespace mg

// Fixed workspace of the allocation-free entry points: one copy per GPU,
// created when the library's code object is loaded on that GPU and held
// until the process ends.  Host code must not take this array's address
// (in host code the name is a host-side stand-in, not a device address):
// it uses the per-device address that hipGetSymbolAddress returns.
static __device__ __align__(256) unsigned char scratch[mg::kNoAllocScratchBytes];

namespace mg {

hipError_t noalloc_scratch(int device, char **base) {
  static std::mutex mu;
  static char *addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    int cur = 0;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != device) {
      const hipError_t e2 = hipSetDevice(cur);
      if (e == hipSuccess) e = e2;
    }
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    addr[device] = (char *)ptr;
  }
  *base = addr[device];
  return hipSuccess;
}

}  // namespace mg

