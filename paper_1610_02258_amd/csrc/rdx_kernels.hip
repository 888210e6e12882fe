// rdx_kernels.hip -- gfx950 kernels of the operator-splitting reaction-diffusion
// window ("Parallel STEPS", Algorithm 1), one lane per tetrahedron.
//
// Per window and tet, in the paper's order:
//   1. load the tet's counts (species-major SoA, coalesced over tets);
//   2. the reaction SSA operator: propensities of the tet's reactions, exact
//      SSA events until the next one would fall outside the window, reaction
//      selection by composition-rejection (Slepoy, Thompson & Plimpton 2008),
//      FP64 time, occupancy O_S += N_S (dt - t_S) for every species an event
//      changes, finalised at the window end;
//   3. the diffusion operator for each diffusive species: mean occupancy
//      Nbar = O_S / tau, leavers Bin(round(Nbar), tau D_S G) (stochastic
//      rounding, at most the post-reaction count), each leaver sent to a face
//      with probability g_k / G (per-molecule draws for small counts);
//   4. integer adds of the remainder and of the face moves into the next
//      count buffer -- the single-GPU form of the paper's local application
//      plus remote change buffers; integer addition makes the result
//      independent of order.
// Random numbers are Philox4x32-10 (Salmon et al., SC'11) with the counter
// (draw call, stream, tet, window); stream 0 is the tet's SSA, stream 1+s the
// diffusion of species s.  The logarithm and the binomial use only correctly
// rounded IEEE-754 binary64 operations in a fixed order (no fp contraction),
// so results are reproducible bit for bit on any IEEE implementation of the
// same operation sequence.
#include <hip/hip_runtime.h>

#include <array>
#include <atomic>
#include <cstdint>
#include <type_traits>

#include "rdx_internal.hpp"
#include "rdx_kernels.hpp"

#pragma clang fp contract(off)

namespace rdx {
namespace {

constexpr int kBlock = 256;

// ---------------------------------------------------------------- Philox ----
// a ^ b ^ k in one VALU instruction, k wave-uniform (an SGPR operand):
// gfx950's three-input bitwise op with truth table 0x96 (odd parity); the
// compiler would split the three-way xor into two v_xor_b32.
__device__ __forceinline__ uint32_t xor3_sk(uint32_t a, uint32_t b, uint32_t k) {
  uint32_t r;
  asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "s"(k));
  return r;
}

// The key (the run's seed) must be the same on every lane of the wave.
__device__ __forceinline__ void philox4x32_10(uint32_t& x0, uint32_t& x1, uint32_t& x2,
                                              uint32_t& x3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    // one 32x32->64 multiply each (v_mad_u64_u32)
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)x0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)x2;
    const uint32_t y0 = xor3_sk((uint32_t)(p1 >> 32), x1, k0);
    const uint32_t y2 = xor3_sk((uint32_t)(p0 >> 32), x3, k1);
    x0 = y0;
    x1 = (uint32_t)p1;
    x2 = y2;
    x3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// SSA stream: 53-bit uniforms x 2^-53, x = w_hi << 21 | w_lo >> 11, two per
// Philox call (words 0-1, then 2-3); both terms and their sum are exact.
__device__ __forceinline__ double u53_co(uint32_t hi, uint32_t lo) {  // [0, 1)
  return (double)hi * 0x1p-32 + (double)(lo >> 11) * 0x1p-53;
}
__device__ __forceinline__ double u53_oc(uint32_t hi, uint32_t lo) { return u53_co(hi, lo) + 0x1p-53; }  // (0, 1]

// Species stream: 32-bit uniforms in [0, 1), four per Philox call.
struct Draw32 {
  uint32_t k0, k1, sid, tet, win, call;
  uint32_t w0, w1, w2, w3;  // the call's words, the next one first
  int pos;
  __device__ Draw32(uint32_t key0, uint32_t key1, uint32_t stream, uint32_t t, uint32_t w)
      : k0(key0), k1(key1), sid(stream), tet(t), win(w), call(0), w0(0), w1(0), w2(0), w3(0),
        pos(4) {}
  // The stream's next Philox call (all four words unused).
  __device__ __forceinline__ void refill() {
    w0 = call;
    w1 = sid;
    w2 = tet;
    w3 = win;
    philox4x32_10(w0, w1, w2, w3, k0, k1);
    ++call;
    pos = 0;
  }
  // The next 32-bit word of the stream, and the uniform w 2^-32 it stands for.
  __device__ __forceinline__ uint32_t word() {
    if (pos == 4) refill();
    const uint32_t w = w0;  // the words move up: a choice by pos is a branch per word
    w0 = w1;
    w1 = w2;
    w2 = w3;
    ++pos;
    return w;
  }
  __device__ __forceinline__ double u() { return (double)word() * 0x1p-32; }
};

// ------------------------------------------------------------------ ln ----
// x = m 2^e, m in [sqrt(1/2), sqrt(2)); ln m = 2 atanh(s) with s = (m-1)/(m+1)
// summed to s^21; e ln 2 added through the Cody-Waite split of ln 2.
__device__ __forceinline__ double ln_basic(double x) {
  const long long bits = __double_as_longlong(x);
  int e = (int)((bits >> 52) & 0x7ff) - 1022;
  double m = __longlong_as_double((bits & 0x000fffffffffffffLL) | 0x3fe0000000000000LL);
  if (m < 0.70710678118654752440) {
    m = m + m;
    e = e - 1;
  }
  const double s = (m - 1.0) / (m + 1.0);
  const double z = s * s;
  double p = 1.0 / 21.0;
  p = p * z + 1.0 / 19.0;
  p = p * z + 1.0 / 17.0;
  p = p * z + 1.0 / 15.0;
  p = p * z + 1.0 / 13.0;
  p = p * z + 1.0 / 11.0;
  p = p * z + 1.0 / 9.0;
  p = p * z + 1.0 / 7.0;
  p = p * z + 1.0 / 5.0;
  p = p * z + 1.0 / 3.0;
  p = p * z + 1.0;
  const double lnm = (s + s) * p;
  const double de = (double)e;
  const double ln2_hi = 6.93147180369123816490e-01;  // 0x3fe62e42fee00000
  const double ln2_lo = 1.90821492927058770002e-10;  // 0x3dea39ef35793c76
  return de * ln2_hi + (de * ln2_lo + lnm);
}

// ------------------------------------------------------------ binomial ----
// Sequential-search inversion, one uniform per chunk of <= 1000 trials
// (q^c >= 2^-1000 stays normal), complement for p > 1/2.
__device__ __forceinline__ double pow_int(double q, int c) {
  // the wave steps together to its largest exponent's last bit (a lane past
  // its own last bit multiplies nothing in), without a branch per lane and bit
  double result = 1.0, base = q;
  for (;;) {
    const double next = result * base;
    result = (c & 1) ? next : result;
    c >>= 1;
    if (__ballot(c != 0) == 0ull) break;
    base = base * base;
  }
  return result;
}

// Reciprocals 1/(k + 1) for k < 1000 (every step of a chunk's search),
// rounded once, at compile time, as the division rounds them.  The search's
// step counter is the same on every lane of a wave (the lanes step together),
// so the table is read with scalar loads that do not depend on the running
// pmf value, instead of a double division on the search's dependent chain.
struct ReciprocalTable {
  double v[1000];
  constexpr ReciprocalTable() : v() {
    for (int k = 0; k < 1000; ++k) v[k] = 1.0 / (double)(k + 1);
  }
};
__constant__ constexpr ReciprocalTable kRecip{};

// Steps of the search per pass of its loop.  A step taken alone waits for its
// own scalar load of the reciprocal (one load and one wait per pmf term) and
// tests for the end; eight share one 64-byte scalar load, one wait and one
// test.  Running past the end is harmless: the cdf does not fall (terms past
// k = c are zero), so the answer is the number of cdf values that u reaches,
// counted term by term and capped at c.  Against single steps: a window of the
// 112k-tet dendrite (counts near 1000, about 100 terms a search) 915 -> 608 us,
// of the 1M-tet one (counts near 110) 258 -> 247 us.
constexpr int kSearchSteps = 8;
static_assert(1000 % kSearchSteps == 0, "a pass never reads past the reciprocals");

template <typename I>
__device__ __forceinline__ I binom_core(I m, double p, Draw32& st) {
  const double q = 1.0 - p;
  const double r = p / q;
  I total = 0;
  while (m > 0) {
    const int c = m < 1000 ? (int)m : 1000;
    const double u = st.u();
    double f = pow_int(q, c);
    double F = f;
    int k = 0;
    double left = (double)c;  // c - k of the next term
    for (int j = 0; u >= F && j < c; j += kSearchSteps) {
#pragma unroll
      for (int s = 0; s < kSearchSteps; ++s) {
        k += u >= F ? 1 : 0;
        f = ((f * r) * left) * kRecip.v[j + s];
        left = left - 1.0;
        F = F + f;
      }
    }
    // a pass that reached c counted the steps past it too when u stayed above
    // the whole sum, and not the last comparison otherwise: both end at c
    total += k < c ? k : c;
    m -= c;
  }
  return total;
}

// One code path for both sides of 1/2 (the complement is taken by flipping),
// so that lanes of a wave with different p do not run two copies.
template <typename I>
__device__ __forceinline__ I binom(I m, double p, Draw32& st) {
  if (m <= 0 || !(p > 0.0)) return 0;
  if (p >= 1.0) return m;
  const bool flip = p > 0.5;
  const I k = binom_core<I>(m, flip ? 1.0 - p : p, st);
  return flip ? m - k : k;
}

// ---------------------------------------------------------- propensity ----
__device__ __forceinline__ int exp_field(double a) {
  return (int)((__double_as_longlong(a) >> 52) & 0x7ff);
}

// a_r = c_r h_r(N) with c = k N_A V[L] (order 0), k (order 1), k / (N_A V[L])
// (order 2) and h = 1, N_A, N_A N_B or N_A (N_A - 1) / 2, in a branch-free
// form whose products are those of the case-by-case definition: h = (x y) w
// with x = N_A (1 for order 0), y = N_B, N_A - 1 (A + A) or 1, w = 1/2 for
// A + A, and c = k f with f = N_A V, 1 or 1 / (N_A V).  Values below 2^-1000
// are taken as zero.
__device__ __forceinline__ double propensity(double c, int x, int y, double w) {
  const double v = c * (((double)x * (double)y) * w);
  return v >= 0x1p-1000 ? v : 0.0;
}

// The sum over the wave, on lane 63 (row shifts, then row broadcasts; lanes
// without a source add 0).
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
  auto add = [&](uint32_t lo, uint32_t hi) { v += ((unsigned long long)hi << 32) | lo; };
#define RDX_STEP(ctrl, rows)                                                     \
  add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, ctrl, rows, 0xf, false), \
      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), ctrl, rows, 0xf, false))
  RDX_STEP(0x111, 0xf);  // row_shr:1
  RDX_STEP(0x112, 0xf);  // row_shr:2
  RDX_STEP(0x114, 0xf);  // row_shr:4
  RDX_STEP(0x118, 0xf);  // row_shr:8
  RDX_STEP(0x142, 0xa);  // row_bcast:15
  RDX_STEP(0x143, 0xc);  // row_bcast:31
#undef RDX_STEP
  return v;
}

// The sum of v over the lanes up to the own one.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v) {
#define RDX_STEP(ctrl, rows) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false)
  RDX_STEP(0x111, 0xf);  // row_shr:1
  RDX_STEP(0x112, 0xf);  // row_shr:2
  RDX_STEP(0x114, 0xf);  // row_shr:4
  RDX_STEP(0x118, 0xf);  // row_shr:8
  RDX_STEP(0x142, 0xa);  // row_bcast:15
  RDX_STEP(0x143, 0xc);  // row_bcast:31
#undef RDX_STEP
  return v;
}

// -------------------------------------------------------- window kernel ----
// A window of a batch is one launch of window_main_kernel: persistent blocks of
// one wave (64 lanes), one lane per tet, a tile of 64, 32 or 16 tets at a time
// (a tile belongs to one run).  Per tile:
//
// Listing: a0 from regrouped coefficients and the tet's first SSA uniform.
// A tet whose first event may fall inside the window is listed.
//
// Reaction operator: the listed tets run their SSA window
// (composition-rejection, occupancy), each on a group of 4, 8 or 16 lanes, as
// many at a time as the wave has groups.
//
// Diffusion items: every (tet, species) pair with something to sample becomes
// an item; they are packed into LDS and sampled in rounds of 64, one per lane.
// Moves into the tile's own tets accumulate in LDS and are flushed once,
// coalesced; the rest are integer atomics into the next count buffer.
//
// What the one launch replaces: a listing launch over all tiles, which wrote
// queues of listed tets, and event blocks beside the diffusion blocks, which
// read the tets again and ran them in chunks.  The chain queue counters ->
// queue -> listed tets -> counts took 7 us before a chunk's first propensity, a
// chunk could hold one run only, and the event blocks ended last wherever
// tiles are few or runs small.  Here the tet is read once, listed, stepped and
// diffused by the wave that holds it.  Per window, two launches against one:
// 480,000 tets, 10 species, 2 molecules a tet 42.4 -> 35.1 us; a million
// molecules in 60,000 tets of it 47.2 -> 21.0 us; 112,000 tets of the calcium
// model with events crowded in one region 915 -> 220 us (by the binomial
// search alone 608); a million tets of it 258 -> 223 us; 48 runs of 200 to
// 1,500 tets 60 -> 19 us.  Also where every tet has events (4 molecules a
// species, 0.9 and 15 events a tet and window): 480,000 tets of 3 species 266 ->
// 133 and 1,119 -> 707 us, of 10 species 654 -> 323 and 2,512 -> 1,810, of 16
// species 2,433 -> 552 and 17,107 -> 3,789.
//
// What bounds a tile: the chain of a lone wave (a load, the propensities and a
// Philox call, the item list, the items' draws), 9 us where tets hold two
// molecules against 0.4 us of memory traffic at the copy rate, and VALU issue
// where they hold hundreds (69% of the issue slots at the million-tet calcium
// dendrite, 6,200 instructions a tile; 32% at two molecules, 1,119).  Hence
// waves per SIMD: four for up to 12 species, three above.
constexpr int kWave = 64;

// Tables the window kernel only reads -- the run table, the tile map, the
// reaction tables, the step word and tile count -- are read through the
// constant address space: nothing writes what is read while a kernel runs (of
// the two step words it writes the other one, which the next kernel reads), and
// a uniform address can then be served by a scalar load, whose wait does not
// hold up the vector loads in flight.
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;

template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p) {
  return (cptr<T>)p;
}

// Element j of a read-only int4 / double2 array through the constant address
// space (the HIP vector types cannot be copied out of it directly).
typedef int int4_v __attribute__((ext_vector_type(4)));
typedef double double2_v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int4 ld_int4(const int4* p, uint32_t j) {
  const int4_v v = ((cptr<int4_v>)p)[j];
  return make_int4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ double2 ld_double2(const double2* p, uint32_t j) {
  const double2_v v = ((cptr<double2_v>)p)[j];
  return make_double2(v.x, v.y);
}

// Every block of the window kernel is a single wave: its lanes execute in
// lockstep and its LDS operations complete in issue order, so handing LDS
// data from lane to lane only needs the compiler to keep the accesses in
// program order (a wavefront-scope fence), not a workgroup barrier, whose
// fence would also wait for every global load and atomic in flight.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The values as new ones to the compiler, so that what is computed from them
// in a loop stays there.  Left alone it computes every mask, address and item
// word of a tile's species ahead of the loop and keeps them, several hundred
// bytes a lane and most of that in scratch memory.
template <int SMAX, typename NV>
__device__ __forceinline__ void renew(NV& N) {
#pragma unroll
  for (int s = 0; s < SMAX; ++s) {
    int n = N[s];
    asm volatile("" : "+v"(n));
    N[s] = n;
  }
}
__device__ __forceinline__ void renew(int& v) { asm volatile("" : "+v"(v)); }
// Scalars.
__device__ __forceinline__ void renew_s(int& v) { asm volatile("" : "+s"(v)); }
__device__ __forceinline__ void renew_s(uint32_t& a, uint32_t& b) { asm volatile("" : "+s"(a), "+s"(b)); }

// Diffusion items.  An item is one (tet, species) pair of a window: m trials
// of leaving, m = nbar stochastically rounded (a draw only when nbar is
// fractional).  With m <= 16 every molecule draws one 32-bit uniform u and
// leaves when u < p, to the first face k before the last face present with
// u < p cum_k, else to the last face; once npost molecules have left the
// rest stay.  With m > 16 the faces in order take successive binomials of
// the molecules not yet placed (face k: Bin(rest, p s_k / (1 - p cum_{k-1})),
// s_k the face's share of the couplings) and the rest stay; should more than
// npost leave, npost leave instead, split afresh by the shares.  Both are
// exact samplers of binomial leavers split among the faces in proportion to
// the face couplings.
//
// The per-molecule draws of an item (m <= 16) are the words w0, w0 + 1, ...
// of its species stream, w0 the words the rounding used (0 or 1; a rounding
// word is counted with the others and taken back); word j is word j mod 4 of
// Philox call j / 4, so an item takes at most five calls, which its own lane
// makes, testing the words against the item's probabilities.  (With m > npost the cap can bind in the middle of the
// walk; such an item -- only a species changed in the window can have one --
// is walked word by word in stream order.)
constexpr int kSmallM = 16;

// Leavers by face.
struct Faces {
  int o0, o1, o2, o3;
};

__device__ __forceinline__ int last_face(int4 nb) {
  return nb.w >= 0 ? 3 : (nb.z >= 0 ? 2 : (nb.y >= 0 ? 1 : 0));
}

// What a lane's item draws against: the leave probability min(1, tau_k D_s G)
// and the cumulative shares of faces 0, 1, 2, with kAllFaces from the last
// face present on.
constexpr double kAllFaces = 2.0;
struct ItemGeo {
  double p;
  double c0, c1, c2;
};

// A draw w leaves when w 2^-32 < p, i.e. (scaling by a power of two is exact)
// w < p 2^32 as doubles, to the first face k < last with w < p 2^32 cum_k,
// else to the last.  The thresholds rise with k; those of the faces from
// `last` on are p's own, and none is above it, so the draws below threshold k
// are the leavers to the faces up to k: counting each threshold's draws (a
// compare and an add-with-carry each) gives the face counts as differences,
// with no choice of a face per draw.
struct DrawCounts {
  double t0, t1, t2, ts;
  int n0, n1, n2, ns;
  __device__ __forceinline__ explicit DrawCounts(const ItemGeo& g) : n0(0), n1(0), n2(0), ns(0) {
    ts = g.p * 0x1p32;
    t0 = fmin(ts * g.c0, ts);
    t1 = fmin(ts * g.c1, ts);
    t2 = fmin(ts * g.c2, ts);
  }
  __device__ __forceinline__ void add(double u) {
    n0 += u < t0 ? 1 : 0;
    n1 += u < t1 ? 1 : 0;
    n2 += u < t2 ? 1 : 0;
    ns += u < ts ? 1 : 0;
  }
  __device__ __forceinline__ void take_back(double u) {
    n0 -= u < t0 ? 1 : 0;
    n1 -= u < t1 ? 1 : 0;
    n2 -= u < t2 ? 1 : 0;
    ns -= u < ts ? 1 : 0;
  }
  __device__ __forceinline__ Faces faces() const { return Faces{n0, n1 - n0, n2 - n1, ns - n2}; }
};

// The first m draws of the item's stream, made on its lane.
__device__ __forceinline__ void count_draws(uint32_t key0, uint32_t key1, uint32_t window, uint32_t tet, int sp,
                                            int m, DrawCounts& c) {
  renew_s(key0, key1);  // the round keys are made here, not kept over the tile
  for (int call = 0, left = m; left > 0; ++call, left -= 4) {
    uint32_t x0 = (uint32_t)call, x1 = 1u + (uint32_t)sp, x2 = tet, x3 = window;
    philox4x32_10(x0, x1, x2, x3, key0, key1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t w = q == 0 ? x0 : (q == 1 ? x1 : (q == 2 ? x2 : x3));
      const double u = (double)w;  // past the last draw: 2^33 or more, below no threshold
      c.add(__hiloint2double(left > q ? __double2hiint(u) : 0x42000000, __double2loint(u)));
    }
  }
}

// The part of an item before its plain draws: rounding draw, binomial faces
// (into `split`), a walk under the cap (into c); leaves m, the draws still to
// count.
__device__ __forceinline__ void item_general(uint32_t key0, uint32_t key1, uint32_t window, uint32_t tet, int sp,
                                             double nbar, int npost, const ItemGeo& g, DrawCounts& c, Faces& split,
                                             int& m) {
  renew_s(key0, key1);
  Draw32 st(key0, key1, 1u + (uint32_t)sp, tet, window);
  const double fl = floor(nbar);
  const double frac = nbar - fl;
  m = (int)fl;  // counts are int32
  uint32_t rounding = 0;  // the stream's first word, if it went there
  if (frac > 0.0) {
    rounding = st.word();
    if ((double)rounding * 0x1p-32 < frac) m += 1;
  }
  if (!(g.p > 0.0)) m = 0;
  if (m > kSmallM) {
    // the multinomial over the faces and staying, one binomial per stage
    // from one call site, in stream order on this lane: stage k <= last
    // gives face k Bin(rest, p s_k / (1 - p cum_{k-1})) of the molecules
    // not yet placed (s_k the face's share, the last face present taking
    // all that remains of p), the rest stay.  Should more leave than
    // the post-reaction count (only after reactions), stages
    // last + 1 .. 2 last split that count afresh by the shares (face k
    // Bin(rest, s_k / (1 - cum_{k-1})), the last face the rest).
    const int last = g.c0 == kAllFaces ? 0 : (g.c1 == kAllFaces ? 1 : (g.c2 == kAllFaces ? 2 : 3));
    int rest = m, n = 0;
    double prev = 0.0;
    bool capped = false;
    int end = last;
#pragma unroll 1
    for (int stage = 0; stage <= end; ++stage) {
      const int f = capped ? stage - last - 1 : stage;
      const double cum = (!capped && f == last) ? 1.0 : (f == 0 ? g.c0 : (f == 1 ? g.c1 : g.c2));
      double qq;
      if (!capped) {
        // den is 0 only for p = 1 with the shares before face f summing to 1
        const double den = 1.0 - g.p * prev;
        qq = den > 0.0 ? (g.p * (cum - prev)) / den : (f == last ? 1.0 : 0.0);
      } else {
        qq = (cum - prev) / (1.0 - prev);
      }
      const int k = binom<int>(rest, qq, st);
      split.o0 = f == 0 ? k : split.o0;
      split.o1 = f == 1 ? k : split.o1;
      split.o2 = f == 2 ? k : split.o2;
      split.o3 = f == 3 ? k : split.o3;
      rest -= k;
      prev = cum;
      if (!capped) {
        n += k;
        if (f == last && n > npost) {
          capped = true;
          end = last + last;
          rest = npost;
          prev = 0.0;
        }
      }
    }
    if (capped) {
      split.o0 = last == 0 ? rest : split.o0;
      split.o1 = last == 1 ? rest : split.o1;
      split.o2 = last == 2 ? rest : split.o2;
      split.o3 = last == 3 ? rest : split.o3;
    }
    m = 0;
  } else if (m > npost) {  // the cap may bind mid-walk: in stream order
    for (int j = 0; j < m; ++j) {
      const double u = (double)st.word();
      if (u < c.ts && c.ns < npost) c.add(u);
    }
    m = 0;
  } else if (frac > 0.0 && m > 0) {
    // the face draws start at the second word
    c.take_back((double)rounding);
    m += 1;
  }
}

// Tile schedule of a persistent block: the blocks are dispatched round-robin
// over the 8 XCDs, so XCD x (= block % 8) owns one contiguous range of tiles
// (its L2 then sees neighbouring tets), shared round-robin by its blocks.
// The schedule is static: per-tile work is balanced by the grid size (every
// block gets the same number of tiles, to within one).
struct TileRange {
  int first, end, stride;
};

__device__ __forceinline__ TileRange tile_range(int b, int G, int n_tiles) {
  if (G < 8 || n_tiles < 8) return TileRange{b, n_tiles, G};
  const int x = b & 7, j = b >> 3;
  const int Gx = (G - x + 7) >> 3;  // blocks with block % 8 == x
  const int lo = (int)(((long long)n_tiles * x) >> 3);
  const int hi = (int)(((long long)n_tiles * (x + 1)) >> 3);
  return TileRange{lo + j, hi, Gx};
}

// The run a tile belongs to and its first tet there; what the step is for the
// run is read from its descriptor where it is used (scalar loads), so that a
// tile in flight holds few registers.
struct TileAt {
  cptr<RunDesc> rd;
  int base;
};

__device__ __forceinline__ TileAt tile_at(const StepArgs& A, int tile) {
  // with one run the tile map is (0, 64 t): no load on the chain to the counts
  const cptr<int> map = as_const(reinterpret_cast<const int*>(A.tile_map));
  const int cut = 6 - A.tile_shift, t = tile >> cut, part = (tile & ((1 << cut) - 1)) << A.tile_shift;
  const int run = A.single_run ? 0 : map[2 * t];
  const int first = A.single_run ? t * kWave : map[2 * t + 1];
  return TileAt{as_const(A.runs) + run, first + part};
}

__device__ __forceinline__ bool run_active(cptr<RunDesc> rd, int k) { return k < rd->n_steps; }
__device__ __forceinline__ uint32_t run_window(cptr<RunDesc> rd, int k) { return rd->window0 + (uint32_t)k; }
__device__ __forceinline__ double run_tau(cptr<RunDesc> rd, int k) { return k < rd->n_full ? rd->tau : rd->tau_last; }
// The counts window `window` of the run reads (0) and adds into (1).
__device__ __forceinline__ int32_t* run_counts(cptr<RunDesc> rd, uint32_t window, uint32_t which) {
  return rd->cnt[(window + which) & 1u];
}

// Everything one lane reads from global memory for its tet.
template <int SMAX>
struct TetData {
  int N[SMAX];
  double nav;
  int reg;
};
struct TetGeo {
  int4 nb;
  double2 ga, gb;  // (G, cum0), (cum1, cum2)
};

// Row pointers are uniform (scalar registers) and end at the tile's first tet;
// the lane's 32-bit offset is the only vector part of an address.
template <int SMAX>
__device__ __forceinline__ void load_tet(const TileAt& at, int k, int S, int width, int lane, TetData<SMAX>& d) {
  const cptr<RunDesc> rd = at.rd;
  const int T = rd->T;
  const bool active = run_active(rd, k) && lane < width && lane < T - at.base;
  renew_s(S);
#pragma unroll
  for (int s = 0; s < SMAX; ++s) d.N[s] = 0;
  d.nav = 1.0;
  d.reg = 0;
  if (active) {
    const uint32_t l = (uint32_t)lane;
    const int32_t* row = run_counts(rd, run_window(rd, k), 0u) + at.base;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
      if (s < S) d.N[s] = row[l];
      row += T;
    }
    d.nav = as_const(rd->nav + at.base)[l];
    if (rd->region) d.reg = as_const(rd->region + at.base)[l];
  }
}
__device__ __forceinline__ void load_geo(cptr<RunDesc> rd, int base, int lane, bool active, TetGeo& d) {
  d.nb = make_int4(-1, -1, -1, -1);
  d.ga = make_double2(0.0, 0.0);
  d.gb = make_double2(0.0, 0.0);
  if (active) {
    const uint32_t l = (uint32_t)lane;
    d.nb = ld_int4(reinterpret_cast<const int4*>(rd->nbr) + base, l);
    const double2* geo = reinterpret_cast<const double2*>(rd->geo) + 2 * (size_t)base;
    d.ga = ld_double2(geo, 2u * l);
    d.gb = ld_double2(geo, 2u * l + 1u);
  }
}

// Waits for the loads into d: without it the first use of the prefetched tile,
// a tile later, waits for every atomic issued since (one counter holds loads
// and atomics in order).
template <int SMAX>
__device__ __forceinline__ void settle(TetData<SMAX>& d) {
  renew<SMAX>(d.N);
  asm volatile("" : "+v"(d.nav), "+v"(d.reg));
}

// tau_k D_s of the run.
template <int SMAX>
__device__ __forceinline__ void set_run(double (&tauD)[SMAX], cptr<RunDesc> rd, double d, int k, int S, int lane) {
  asm volatile("" : "+v"(d));  // waited for on every path
  if (lane < SMAX) tauD[lane] = run_tau(rd, k) * (lane < S ? d : 0.0);
}

__device__ __forceinline__ unsigned long long* tally_slot(cptr<RunDesc> rd) {
  return rd->tally + kTallyWords * (blockIdx.x & (kTallySlots - 1));
}

// a_0 of one tet from the regrouped listing coefficients of a region (scalar
// loads).  The terms are those of the reaction-by-reaction sum, so the result
// agrees with it to within a few roundings (relative 1e-14 at most; fused
// multiply-adds are fine here); it is only used with a margin far above that.
template <int SMAX, typename NV>
__device__ __forceinline__ double listing_rate(const StepArgs& A, cptr<double> lc, const NV& N, double nav) {
  // beta_s is zero for s >= S, and so are the counts there
  double lin = nav * lc[0];
#pragma unroll
  for (int s = 0; s < SMAX; ++s) lin = __builtin_fma(lc[1 + s], (double)N[s], lin);
  asm volatile("" : "+v"(lin));  // its coefficients are not held over the pairs
  double quad = 0.0;
  // four pairs to a round of scalar loads (gamma is zero past the last pair)
#pragma unroll 1
  for (int p = 0; p < A.n_pairs; p += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int pr = A.pairs[p + q];
      const int a = pr & 0xff, b = (pr >> 8) & 0xff;
      const int x = a < SMAX ? N[a] : 0;
      const int y = (b < SMAX ? N[b] : 0) - ((pr >> 16) & 1);
      quad = __builtin_fma(lc[17 + p + q], (double)x * (double)y, quad);
    }
  }
  double r = __builtin_amdgcn_rcp(nav);  // one Newton step: to a few ulp
  r = r * (2.0 - nav * r);
  return __builtin_fma(quad, r, lin);
}

// Lanes that run the reaction operator of one tet: one per species, and one
// per reaction or two.
template <int SMAX, int RMAX>
constexpr int ssa_lanes() {
  return SMAX <= 4 && RMAX <= 8 ? 4 : (SMAX <= 8 && RMAX <= 16 ? 8 : 16);
}

// A lane's reaction, as the propensity takes it (unpacked from the reaction
// table once per block): lanes of the reactants in the group, what stands in
// for an absent one, A + A.
struct LaneReaction {
  uint32_t info;  // s0 | s1 << 8 | order << 16, 0xff000000 if there is none
  __device__ __forceinline__ void set(uint32_t i, bool any) {
    info = any ? ((i >> 8) & 0xffffu) | ((i & 0xffu) << 16) : 0xff000000u;
  }
};

// Items of changed species a tile holds at a time: a chunk of listed tets adds
// up to 64 to what waits.
template <int SMAX, int RMAX>
constexpr int drawn_items() {
  return SMAX > 12 && RMAX > 24 ? 88 : 96;
}

// LDS of a block: this part, of one size in an instance ...
template <int SMAX, int RMAX>
struct TileLds {
  // items of the species events changed: mean occupancy, post-reaction count,
  // lane << 4 | species
  static constexpr int kDrawn = drawn_items<SMAX, RMAX>();
  double nbar[kDrawn];
  int npost[SMAX <= 12 ? kDrawn : 1];  // (above 12 species at the end of tile_rows)
  uint16_t drawn[kDrawn];
  int ctr, sub_lo, sub_hi;  // the block's claim counter (index) and sub-range
  int8_t delta[RMAX][16];  // net changes by reaction and species
  double tauD[SMAX];       // tau_k D_s of the current run
  int4 nbr[kWave];        // neighbours, counted from the tile's first tet
  double2 geo[2][kWave];  // (G, cum0), (cum1, cum2), kAllFaces from the last face on
};

// ... and what its size follows from the model's species count S, behind it:
// the next counts of the tile's own tets, [S][64], and a space that holds first,
// while listed tets run, a row of propensities per tet (and before them the
// counts on the way to their lanes), then the items, count << 10 | lane << 4 |
// species, [S * 64] at most.  By S and not SMAX, for the blocks a CU holds.
extern __shared__ __attribute__((aligned(16))) uint32_t tile_rows[];
// Two bytes an item for up to 12 species, so that 16 blocks fit a CU (the
// counts that do not fit the word's six bits are read again); four above,
// where registers hold a CU to 12 blocks.
template <int SMAX>
using ItemWord = std::conditional_t<(SMAX <= 12), uint16_t, uint32_t>;

template <int SMAX, int RMAX>
constexpr int ssa_row_bytes() {
  return kWave / ssa_lanes<SMAX, RMAX>() * RMAX * (int)sizeof(double);
}
template <int SMAX, int RMAX>
__host__ __device__ constexpr int tile_row_bytes(int S) {
  constexpr int ssa = ssa_row_bytes<SMAX, RMAX>() > kWave * (int)sizeof(int) ? ssa_row_bytes<SMAX, RMAX>()
                                                                             : kWave * (int)sizeof(int);
  constexpr int least = ssa + (SMAX <= 12 ? 0 : drawn_items<SMAX, RMAX>() * (int)sizeof(int));
  const int items = S * kWave * (int)sizeof(ItemWord<SMAX>);
  return S * kWave * (int)sizeof(int) + (items > least ? items : least);
}

// The LDS of a compute unit is handed out in granules of 1,280 bytes, of which
// it has 128: twelve blocks of 16 species fit in ten granules each, and four
// bytes more leave room for eleven.  (The occupancy query does not know: at 11
// granules it says twelve, and the blocks that then wait for a place ran as a
// last round of their own: 375,000 tets of 16 species, 20 molecules of each in a
// tet, 334 us a window so, in ten granules 243.)
constexpr int kLdsGranule = 1280, kLdsGranules = 128;
template <int SMAX, int RMAX>
constexpr int lds_blocks(int S) {
  return kLdsGranules /
         ((int)((sizeof(TileLds<SMAX, RMAX>) + tile_row_bytes<SMAX, RMAX>(S) + kLdsGranule - 1) / kLdsGranule));
}
static_assert(lds_blocks<4, 4>(4) >= 16 && lds_blocks<8, 8>(8) >= 16 && lds_blocks<12, 12>(12) >= 16 &&
                  lds_blocks<16, 24>(16) >= 12 && lds_blocks<16, 32>(16) >= 12,
              "room for the waves that the registers allow");

// The largest of the GL lanes' values, on all of them (butterfly within rows of
// 16 lanes).
template <int GL>
__device__ __forceinline__ int group_max(int v) {
  auto up = [&](int o) { v = o > v ? o : v; };
  up(__builtin_amdgcn_mov_dpp(v, 0xb1, 0xf, 0xf, true));                  // quad_perm 1,0,3,2
  up(__builtin_amdgcn_mov_dpp(v, 0x4e, 0xf, 0xf, true));                  // quad_perm 2,3,0,1
  if (GL >= 8) up(__builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true));    // row_half_mirror
  if (GL >= 16) up(__builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true));   // row_mirror
  return v;
}

// The next GL calls of a listed tet's SSA stream, one a lane: -ln u and the
// two uniforms.
struct LaneDraws {
  uint32_t first;  // the group's first call in hand
  double mln, u01, u23;
  __device__ __forceinline__ void refill(int j, uint32_t key0, uint32_t key1, uint32_t window, uint32_t tet,
                                         uint32_t call) {
    first = call;
    renew_s(key0, key1);
    uint32_t x0 = call + (uint32_t)j, x1 = 0u, x2 = tet, x3 = window;
    philox4x32_10(x0, x1, x2, x3, key0, key1);
    mln = -ln_basic(u53_oc(x0, x1));
    u01 = u53_co(x0, x1);
    u23 = u53_co(x2, x3);
  }
};

__device__ __forceinline__ double lane_read(double v, int from) {
  return __hiloint2double(__builtin_amdgcn_ds_bpermute(4 * from, __double2hiint(v)),
                          __builtin_amdgcn_ds_bpermute(4 * from, __double2loint(v)));
}

// The reaction operator of up to 64 / GL tets over [0, tau], a tet to each
// group of GL lanes (`run`: this lane's group has one): lane j of the group
// holds species j (its count N, and as events change it its occupancy O, the
// time t of the last change, and `touched`) and reactions j, j + GL.  Per
// event: the waiting time and the composition draw come from one Philox call,
// then one call per rejection attempt.  Returns the group's events.
//
// A tile lists a tet or two as a rule, and a step of one tet on one lane is a
// chain of over a thousand instructions (every propensity, four scans of
// them, the logarithm, a Philox call for each pair of draws).  Here the group
// computes the propensities at once, and the next GL calls of the stream with
// their logarithms; what has to go in reaction order, a_0 and a group's total,
// are adds alone, of values read back from LDS.  A step of up to 4 tets (16
// species and lanes a tet) is 2 us, with one tet on each lane of a wave it was
// 5 us with the tables in LDS, and more with them spilled from registers.
//
// Composition: groups of reactions with equal binary exponent, visited from
// the largest exponent down, picked with probability proportional to their
// totals; rejection: a uniform member is accepted with probability a / 2^g.
// Group totals are summed in reaction order.
template <int SMAX, int RMAX>
__device__ __forceinline__ unsigned int ssa_window(TileLds<SMAX, RMAX>& L, double* rows, bool run, uint32_t key0, uint32_t key1,
                                                   uint32_t window, uint32_t tet, double tau, double nav, const double (&kc)[2],
                                                   const LaneReaction (&lr_in)[2], int& N, double& O, double& t,
                                                   bool& touched, int& err) {
  constexpr int GL = ssa_lanes<SMAX, RMAX>();
  constexpr int RPL = (RMAX + GL - 1) / GL;  // reactions of a lane
  static_assert(RPL <= 2 && GL >= SMAX && GL <= 16, "a lane per species, at most two reactions a lane");
  int lane = threadIdx.x;
  renew(lane);  // (what follows from it is not kept over the tile)
  const int j = lane & (GL - 1), g0 = lane - j;
  constexpr uint32_t group = (1u << GL) - 1u;
  LaneReaction lr[2] = {lr_in[0], lr_in[1]};
  asm volatile("" : "+v"(lr[0].info), "+v"(lr[1].info));
  double* const a = rows + (size_t)(g0 / GL) * RMAX;
  unsigned int events = 0;
  if (run) {
    double c[RPL];
    const double inv_nav = 1.0 / nav;
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
      const int r = j + q * GL, order = (int)(lr[q].info >> 16);
      const double f = order == 0 ? nav : (order == 1 ? 1.0 : inv_nav);
      c[q] = order <= 2 && r < RMAX ? kc[q] * f : 0.0;
    }
    LaneDraws draws;
    uint32_t call = 0;  // the next call
    draws.refill(j, key0, key1, window, tet, call);
    double dt = 0.0;
    for (;;) {
      double v[RPL];
#pragma unroll
      for (int q = 0; q < RPL; ++q) {
        const int r = j + q * GL;
        const int s0 = (int)(lr[q].info & 0xffu), s1 = (int)((lr[q].info >> 8) & 0xffu);
        const int order = (int)(lr[q].info >> 16);
        const bool same = order == 2 && s0 == s1;
        const int xs = __builtin_amdgcn_ds_bpermute(4 * (g0 + (s0 & (GL - 1))), N);
        const int ys = __builtin_amdgcn_ds_bpermute(4 * (g0 + (s1 & (GL - 1))), N);
        v[q] = propensity(c[q], order == 0 ? 1 : xs, order == 2 ? ys - (same ? 1 : 0) : 1, same ? 0.5 : 1.0);
        if (r < RMAX) a[r] = v[q];
      }
      if (call - draws.first >= (uint32_t)GL) draws.refill(j, key0, key1, window, tet, call);
      const int at = g0 + (int)(call - draws.first);
      const double mln = lane_read(draws.mln, at), u23 = lane_read(draws.u23, at);
      wave_sync();
      double a0 = 0.0;
#pragma unroll
      for (int r = 0; r < RMAX; ++r) a0 = a0 + a[r];
      if (!(a0 > 0.0)) break;
      const double t_reac = mln / a0;
      if (dt + t_reac > tau) break;
      ++call;
      double left = u23 * a0;
      int g = 0x800;  // exponent field of the group, at first above any (0x7ff: infinite propensities)
      uint32_t members = 0;
      for (;;) {  // the groups from the largest exponent down
        int e = 0;
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
          const int eq = exp_field(v[q]);
          e = eq < g && eq > e ? eq : e;
        }
        e = group_max<GL>(e);
        if (e == 0) break;  // none below: what is left falls to the last group
        g = e;
        members = 0;
#pragma unroll
        for (int q = 0; q < RPL; ++q)
          members |= ((uint32_t)(__ballot(exp_field(v[q]) == g) >> g0) & group) << (q * GL);
        double sum = 0.0;
        for (uint32_t m = members; m != 0u; m &= m - 1u) sum = sum + a[__builtin_ctz(m)];
        if (left < sum) break;
        left = left - sum;
      }
      const double n = (double)__popc(members);
      // u < a / 2^(g - 1022), both sides halved (which is exact): the bound of
      // the largest finite group would be infinite, and no attempt accepted.
      // An infinite propensity is accepted at once.
      const double half = g == 0x7ff ? 0.0 : __longlong_as_double((long long)g << 52);
      int rn = 0;
      for (;;) {  // the attempts of all calls in hand at once; the first accepted one counts
        int q = (int)(draws.u01 * n);
        if ((double)q >= n) q = (int)n - 1;
        uint32_t m = members;
        for (; q > 0; --q) m &= m - 1u;
        const int r = __builtin_ctz(m);
        const bool accept = draws.first + (uint32_t)j >= call && draws.u23 * half < 0.5 * a[r];
        const uint32_t acc = (uint32_t)(__ballot(accept) >> g0) & group;
        if (acc != 0u) {
          const int w = __builtin_ctz(acc);
          rn = __builtin_amdgcn_ds_bpermute(4 * (g0 + w), r);
          call = draws.first + (uint32_t)w + 1u;
          break;
        }
        call = draws.first + (uint32_t)GL;
        draws.refill(j, key0, key1, window, tet, call);
      }
      dt = dt + t_reac;
      const int d = (int)L.delta[rn][j];
      int bad = 0;
      if (d != 0) {
        O = O + (double)N * (dt - t);
        t = dt;
        touched = true;
        N += d;
        if (N > kCountCap) bad |= kErrOverflow;
      }
      ++events;
      if (events >= (unsigned int)kEventCap) bad |= kErrEvents;
      err |= bad;
      if (((uint32_t)(__ballot(bad != 0) >> g0) & group) != 0u) break;
      wave_sync();
    }
  }
  return events;
}

// Four waves per SIMD for up to 12 species, three above: the tiles are chains
// of a lone wave and need the others to fill its gaps.  At three, 480,000 tets
// of 10 species are 3 rounds of tiles and 46.1 us a window, at four 2 rounds
// and 36.7 us.  For 16 species four waves take 48 bytes of scratch a lane and
// items of two bytes, and gain nothing: a million tets of the calcium model
// 224 us a window, and at three 223.
template <int SMAX, int RMAX>
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(SMAX <= 12 ? 4 : 3)))
window_main_kernel(const StepArgs A) {
  __shared__ TileLds<SMAX, RMAX> L;
  int* const acc = reinterpret_cast<int*>(tile_rows);
  typedef ItemWord<SMAX> item_t;
  constexpr int kPackedCount = 1 << (8 * (int)sizeof(item_t) - 10);  // counts from here on do not fit an item
  item_t* const items = reinterpret_cast<item_t*>(tile_rows + A.S * kWave);
  int* const moved_n = reinterpret_cast<int*>(items);
  // The post-reaction counts of changed items, from the last one of this space
  // back.  Above 12 species they lie at the end of the items': that has a word
  // for each (tet, species) pair, and a changed one is not in the list that
  // fills it from its start (nor do the rows of the reaction operator, there
  // meanwhile, reach it).
  constexpr int kDrawn = TileLds<SMAX, RMAX>::kDrawn;
  int* const npost = SMAX <= 12 ? &L.npost[SMAX <= 12 ? kDrawn - 1 : 0]
                                : reinterpret_cast<int*>(tile_rows) + tile_row_bytes<SMAX, RMAX>(A.S) / (int)sizeof(int) - 1;
  // The first tile's counts are at the end of a chain of loads (arguments,
  // step and run, rows) that a block of two or three tiles feels: what of it
  // is known by now is read at once, a word of each cache line, so that later
  // reads find it in the scalar cache.
  const int step_word = as_const(A.step_words)[A.parity];
  const int width = 1 << A.tile_shift;  // tets of a tile
  const int n_tiles = *as_const(A.n_tiles) << (6 - A.tile_shift);
  asm volatile("" ::"s"(step_word), "s"(n_tiles), "s"(A.S), "s"(A.n_pairs), "s"(A.pairs[8]), "s"(A.pairs[24]),
               "s"(A.tile_claim));
  const int k = A.step >= 0 ? A.step : step_word;
  const int b = blockIdx.x, G = gridDim.x;
  if (b == 0) {
    // the next window's step index and claim counters (nothing in this window
    // reads the words of the other parity)
    if (threadIdx.x == 0) A.step_words[(k + 1) & 1] = k + 1;
    A.tile_ctr[((size_t)((k + 1) & 1) * 8 * kClaimSubs + (size_t)threadIdx.x) * kCtrStride] = 0;
  }
  const TileRange tr = tile_range(b, G, n_tiles);
  // Run-time claiming (a launch-shape setting, for workloads whose tiles
  // differ in cost): the block's first tile is its static one, lo + j; the
  // tiles from lo + Gx on are cut into kClaimSubs sub-ranges (fewer if the
  // XCD has fewer blocks), each handed out in order by a counter of its own
  // to the blocks with j mod kClaimSubs equal to its index.
  // Eight counters per XCD keep the claims at a window's start from queueing
  // on one address.  A block stops at its first claim past its sub-range,
  // so every block ends, and the slowest finishes within about one tile of
  // the others.
  const bool claim = A.tile_claim != 0 && G >= 8 && n_tiles >= 8;
  if (claim) {
    const int dyn0 = tr.first - (b >> 3) + tr.stride;  // lo + Gx
    const int n_claim = tr.end > dyn0 ? tr.end - dyn0 : 0;  // at most 2^22 (64 tets a tile, an eighth of them)
    const bool all = tr.stride >= kClaimSubs;
    const int nsub = all ? kClaimSubs : (tr.stride > 0 ? tr.stride : 1);
    const int sub = all ? (b >> 3) % kClaimSubs : (b >> 3) % nsub;
    L.ctr = ((A.parity * 8 + (b & 7)) * kClaimSubs + sub) * kCtrStride;
    L.sub_lo = dyn0 + (all ? n_claim * sub / kClaimSubs : n_claim * sub / nsub);
    L.sub_hi = dyn0 + (all ? n_claim * (sub + 1) / kClaimSubs : n_claim * (sub + 1) / nsub);
  }
  constexpr int GL = ssa_lanes<SMAX, RMAX>();
  int raw = 0;  // lane 0: the counter value of the claim in flight
  // (At an address known to be uniform the compiler would add for the wave and
  // wait for the result at once.)
  auto claim_next = [&] {
    if (claim && threadIdx.x == 0) {
      int at = L.ctr;
      renew(at);
      raw = atomicAdd(A.tile_ctr + at, 1);
    }
  };
  cptr<RunDesc> cached = nullptr;  // the run whose tables are in LDS
  unsigned long long n_ev = 0, n_moved = 0;
  uint32_t n_faces = 0;

  TileAt here{nullptr, 0}, there{nullptr, 0};  // this tile, the next one
  TetData<SMAX> cur, nxt;
  double first_d = 0.0;
  if (tr.first < tr.end) {
    here = tile_at(A, tr.first);
    asm volatile("" ::"s"(here.rd->cnt[0]), "s"(here.rd->n_steps), "s"(here.rd->tau), "s"(here.rd->D[4]),
                 "s"(here.rd->D[12]));
    load_tet<SMAX>(here, k, A.S, width, threadIdx.x, cur);
    first_d = here.rd->D[threadIdx.x & 15];
  }
  // the tables, in flight beside the first tile
  LaneReaction lr[2];
  {
    constexpr int kWords = RMAX * 4, kPer = (kWords + kWave - 1) / kWave;
    const cptr<uint32_t> mw = as_const(reinterpret_cast<const uint32_t*>(A.model));
    const int t = (int)threadIdx.x, j = t & (GL - 1);
    uint32_t dw[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) dw[q] = mw[offsetof(DevModel, delta) / 4 + (kWave * q + t) % kWords];
    const uint32_t i0 = mw[offsetof(DevModel, info) / 4 + j], i1 = mw[offsetof(DevModel, info) / 4 + j + GL];
    lr[0].set(i0, j < A.R);
    lr[1].set(i1, j + GL < A.R);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (kWave * q + t < kWords) reinterpret_cast<uint32_t*>(L.delta)[kWave * q + t] = dw[q];
    }
  }
  if (tr.first < tr.end) {
    if (run_active(here.rd, k)) {
      cached = here.rd;
      set_run(L.tauD, here.rd, first_d, k, A.S, threadIdx.x);
    }
    settle<SMAX>(cur);
  }
  for (int tile = tr.first; tile < tr.end;) {
    int lane = threadIdx.x, S = A.S;
    asm volatile("" : "+v"(lane), "+s"(S));
    const unsigned long long below = (1ull << lane) - 1ull;
    const cptr<RunDesc> rd = here.rd;
    const int base = __builtin_amdgcn_readfirstlane(here.base);
    const int T = rd->T;
    const bool stepping = run_active(rd, k);  // else the tile only forwards the prefetch
    const uint32_t window = run_window(rd, k);
    const double tau = run_tau(rd, k);
    const int i = base + lane;
    const bool active = stepping && lane < width && i < T;
    if (stepping && rd != cached) {
      if (cached != nullptr) {  // tallies are kept per run
        const unsigned long long ev = wave_sum(n_ev), mv = wave_sum(n_moved), fm = wave_sum(n_faces);
        if (lane == kWave - 1) {
          if (ev) atomicAdd(tally_slot(cached), ev);
          if (mv) atomicAdd(tally_slot(cached) + 1, mv);
          if (fm) atomicAdd(tally_slot(cached) + 2, fm);
        }
        n_ev = n_moved = 0;
        n_faces = 0;
      }
      set_run(L.tauD, rd, rd->D[lane & 15], k, S, lane);
      cached = rd;
    }
    TetGeo tg;  // in flight until the listing is done
    load_geo(rd, base, lane, active, tg);
    const uint32_t key0 = rd->key0, key1 = rd->key1, dmask = rd->dmask;
    const double nav = cur.nav;
    const int reg = cur.reg;
    int N[SMAX];
#pragma unroll
    for (int s = 0; s < SMAX; ++s) N[s] = cur.N[s];
    int errbits = 0;
    uint32_t most = 0u;  // (a count that wrapped past 2^31 is above the cap, too)
#pragma unroll
    for (int s = 0; s < SMAX; ++s) most = (uint32_t)N[s] > most ? (uint32_t)N[s] : most;
    if (most > (uint32_t)kCountCap) errbits |= kErrOverflow;
    const bool any_wide = __ballot(most >= (uint32_t)kPackedCount) != 0ull;

    // ---- listing ----
    // The window's first SSA event falls inside [0, tau_k] only if
    // t_reac = -ln(u) / a0 <= tau_k, and -ln(u) >= 1 - u; so a tet whose first
    // uniform u of the window has 1 - u above a0 tau_k (with a relative
    // margin of 1e-6, far above the rounding of a0, of ln and of the
    // division) has no event, and every other tet with a0 > 0 is listed, or
    // whose a0 is indefinite (constants that sum to infinity, of an absent
    // species).  A listed tet without an event is harmless: its SSA ends at the
    // first draw and its items are those of an unlisted tet.
    bool event = false;
    double a0 = 0.0;
    if (active) {
      // the counts as one vector value, so that a uniform (run-time) species
      // index selects a register rather than spilling the array to memory
      int __attribute__((ext_vector_type(SMAX))) NV;
#pragma unroll
      for (int s = 0; s < SMAX; ++s) NV[s] = N[s];
      if (rd->region == nullptr) {
        a0 = listing_rate<SMAX>(A, as_const(rd->lcoef), NV, nav);
      } else {
        // One region of the tile at a time, its coefficients by scalar loads,
        // where there are one or two (neighbouring tets mostly share one); else
        // each tet with loads of its own.  A window of 480,000 tets of 8 species
        // and 8 reactions, labels drawn at random from 2, 3, 4 and 8 regions: a
        // pass for each 37.3, 40.0, 51.5, 52.9 us, by this rule 36.2, 36.5, 37.6,
        // 36.4; with one region 35.3.
        const unsigned long long all = __ballot(true);
        const int q0 = __builtin_amdgcn_readlane(reg, __builtin_ctzll(all));
        unsigned long long left = __ballot(reg != q0);
        const int q1 = __builtin_amdgcn_readlane(reg, __builtin_ctzll(left != 0ull ? left : all));
        left = __ballot(reg != q0 && reg != q1);
        if (left == 0ull) {
          for (int q = q0;; q = q1) {
            const double r = listing_rate<SMAX>(A, as_const(rd->lcoef) + q * kLStride, NV, nav);
            if (reg == q) a0 = r;
            if (q == q1) break;
          }
        } else {
          a0 = listing_rate<SMAX>(A, as_const(rd->lcoef) + reg * kLStride, NV, nav);
        }
      }
    }
    // The claim of the next tile, its latency behind the rest of the listing.
    // Where many tets will have events it waits until their SSA is done: a
    // tile claimed and held meanwhile is the branch's next crowded one, which
    // then runs after this one instead of beside it (branch 281 us a window
    // with claims a tile ahead, 225 so; dendrite 241 and 233).
    const bool early = (int)__popcll(__ballot(tau * a0 > 0.5)) <= 2 * (kWave / GL);
    if (early) claim_next();
    {
      if (!(a0 <= 0.0)) {
        uint32_t w0 = 0u, w1 = 0u, w2 = (uint32_t)i, w3 = window;
        philox4x32_10(w0, w1, w2, w3, key0, key1);
        event = !(1.0 - u53_oc(w0, w1) > (tau * a0) * 1.000001);
      }
    }

    const int last_f = last_face(tg.nb);
    L.nbr[lane] = make_int4(tg.nb.x - base, tg.nb.y - base, tg.nb.z - base, tg.nb.w - base);
    L.geo[0][lane] = make_double2(tg.ga.x, last_f > 0 ? tg.ga.y : kAllFaces);
    L.geo[1][lane] = make_double2(last_f > 1 ? tg.gb.x : kAllFaces, last_f > 2 ? tg.gb.y : kAllFaces);
    const bool coupled = tg.ga.x > 0.0;

    // ---- diffusion operator ----
    // The accumulator starts with what cannot leave: immobile species and tets
    // without a neighbour.  (A listed tet's come after its events.)  From here
    // on N holds what becomes an item.
    const unsigned long long listed = __ballot(event);
    const int n_listed = (int)__popcll(listed);
    const bool apart = active && !coupled;
    if (__ballot(apart) == 0ull) {
#pragma unroll
      for (int s = 0; s < SMAX; ++s)
        if (s < S) acc[s * kWave + lane] = ((dmask >> s) & 1u) || event ? 0 : N[s];
    } else {
#pragma unroll
      for (int s = 0; s < SMAX; ++s) {
        if (s < S) acc[s * kWave + lane] = (((dmask >> s) & 1u) && !apart) || event ? 0 : N[s];
        if (apart && !event) N[s] = 0;
      }
    }

    // Rounds: the reaction operator of the listed tets, a few at a time; the
    // items of the species their events changed wait for the tile's others,
    // unless they are too many.
    int c0 = 0, n_drawn = 0;
    uint32_t kept = apart && !event ? 0u : ~0u;  // species whose count is still the tet's item
    for (;;) {
      if (c0 > 0) {  // after a flush of changed items: the counts again
        const int32_t* row = run_counts(rd, window, 0u) + base;
        int n[SMAX];
#pragma unroll
        for (int s = 0; s < SMAX; ++s) {
          n[s] = 0;
          if (s < S && active) n[s] = row[(uint32_t)lane];
          row += T;
        }
#pragma unroll
        for (int s = 0; s < SMAX; ++s) N[s] = (kept >> s) & 1u ? n[s] : 0;
      }
      while (c0 < n_listed && n_drawn <= kDrawn - kWave) {
        // ---- reaction SSA operator over [0, tau_k] ----
        const int rank = (int)__popcll(listed & below) - c0;
        const bool mine = event && (unsigned)rank < (unsigned)(kWave / GL);
        // the tets' counts go to their groups' lanes
        int ln = lane;
        renew(ln);
        const int j = ln & (GL - 1), grp = ln / GL;
        if (mine) {
#pragma unroll
          for (int s = 0; s < SMAX; ++s) moved_n[rank * GL + s] = N[s];
          npost[-(n_drawn + rank)] = lane;  // space not yet in use
        }
        wave_sync();
        const bool run = c0 + grp < n_listed;
        const int Lt = run ? npost[-(n_drawn + grp)] : 0;
        int Nj = run && j < SMAX ? moved_n[ln] : 0;
        const double nav_t = lane_read(nav, Lt);
        const int reg_t = __builtin_amdgcn_ds_bpermute(4 * Lt, reg);
        const cptr<double> kw = as_const(rd->kcst) + reg_t * 32;
        double kc[2] = {j < RMAX ? kw[j] : 0.0, j + GL < RMAX ? kw[j + GL] : 0.0};
        // (a load that some path leaves unread has every later write of its
        // register wait for all memory operations)
        asm volatile("" : "+v"(kc[0]), "+v"(kc[1]));
        double O = 0.0, t = 0.0;
        bool touched = false;
        int err = 0;
        const unsigned int events =
            ssa_window<SMAX, RMAX>(L, reinterpret_cast<double*>(items), run, key0, key1, window, (uint32_t)(base + Lt), tau, nav_t, kc, lr, Nj,
                                   O, t, touched, err);
        errbits |= err;
        if (j == 0) n_ev += events;
        const unsigned long long bt = __ballot(touched);
        const bool item = touched && ((dmask >> j) & 1u) && L.geo[0][Lt].x > 0.0;
        const unsigned long long bi = __ballot(item);
        wave_sync();
        if (item) {
          const int at = n_drawn + (int)__popcll(bi & below);
          L.drawn[at] = (uint16_t)((Lt << 4) | j);
          npost[-at] = Nj;
          L.nbar[at] = (O + (double)Nj * (tau - t)) / tau;
        } else if (touched && Nj != 0) {
          atomicAdd(acc + (j * kWave + Lt), Nj);
        }
        if (mine) {  // what is left of the tet: the species no event changed
          const uint32_t changed = (uint32_t)(bt >> (rank * GL)) & ((1u << SMAX) - 1u);
          int mobile = (int)dmask;
          renew_s(mobile);
#pragma unroll
          for (int s = 0; s < SMAX; ++s) {
            const bool gone = (changed >> s) & 1u;
            if (!gone && (((mobile >> s) & 1) == 0 || apart) && N[s] != 0) atomicAdd(acc + (s * kWave + lane), N[s]);
            if (gone || apart) N[s] = 0;
          }
          kept = apart ? 0u : kept & ~changed;
        }
        n_drawn += (int)__popcll(bi);
        c0 += kWave / GL;
        wave_sync();
      }
      const bool last = c0 >= n_listed;
      int n_item = 0;
      if (last) {
        // the next tile's loads are in flight while the items are listed
        __builtin_amdgcn_sched_barrier(0);
        if (claim) {
          if (!early) claim_next();
          tile = __builtin_amdgcn_readfirstlane(L.sub_lo) + __builtin_amdgcn_readfirstlane(raw);
          if (tile >= __builtin_amdgcn_readfirstlane(L.sub_hi)) tile = tr.end;
        } else {
          tile += tr.stride;
        }
        if (tile < tr.end) {
          there = tile_at(A, tile);
          load_tet<SMAX>(there, k, S, width, lane, nxt);
        }
        __builtin_amdgcn_sched_barrier(0);
        // Items in five classes: more than 16 molecules (binomial face counts),
        // species-major, so that few rounds wait on a binomial and one that
        // does has binomials of like length; then those of four, three, two
        // and one Philox calls (13 to 16, ... 1 to 4 molecules), tet-major.  A
        // round's lanes step through as many calls as its longest item has:
        // with 5 to 16 molecules in one class the dendrite made 18.8 calls a
        // tile, of which its items need 12.  Where no tet has more than four
        // of any species there is one class.  (Found by a loop over classes
        // and the species of each, the list took 5.9 us of the dendrite's 35
        // a tile; by prefix sums of the lanes' class counts the window is 4%
        // shorter, 6% at 480,000 tets with 20 molecules each.)
        renew<SMAX>(N);
        renew(lane);
        int mobile = (int)dmask;
        renew_s(mobile);
        if (__ballot(most > 4u) == 0ull) {
#pragma unroll
          for (int s = 0; s < SMAX; ++s) {
            const bool has = N[s] > 0 && ((mobile >> s) & 1);
            const unsigned long long bs = __ballot(has);
            if (has) items[n_item + (int)__popcll(bs & below)] = (item_t)((N[s] << 10) | (lane << 4) | s);
            n_item += (int)__popcll(bs);
          }
        } else {
          // the lane's items by class, eight bits each, from one call up
          uint32_t held = 0u;
#pragma unroll
          for (int s = 0; s < SMAX; ++s) {
            if (((mobile >> s) & 1) == 0) N[s] = 0;
            const bool wide = N[s] > kSmallM;
            const unsigned long long bs = __ballot(wide);
            if (bs != 0ull) {
              if (wide)
                items[n_item + (int)__popcll(bs & below)] =
                    (item_t)(((N[s] < kPackedCount ? N[s] : 0) << 10) | (lane << 4) | s);
              n_item += (int)__popcll(bs);
            }
            const uint32_t u = (uint32_t)N[s] - 1u;
            held += (u < (uint32_t)kSmallM ? 1u : 0u) << ((u << 1) & 24u);
          }
          // prefix sums over the lanes, sixteen bits a class
          const uint32_t even = held & 0x00ff00ffu, odd = (held >> 8) & 0x00ff00ffu;
          const uint32_t even_to = wave_prefix(even), odd_to = wave_prefix(odd);
          const uint32_t even_all = (uint32_t)__builtin_amdgcn_readlane((int)even_to, kWave - 1);
          const uint32_t odd_all = (uint32_t)__builtin_amdgcn_readlane((int)odd_to, kWave - 1);
          const uint32_t at3 = (uint32_t)n_item, at2 = at3 + (odd_all >> 16), at1 = at2 + (even_all >> 16);
          const uint32_t at0 = at1 + (odd_all & 0xffffu);
          n_item = (int)(at0 + (even_all & 0xffffu));
          const uint32_t e = even_to - even + (at0 | (at2 << 16)), o = odd_to - odd + (at1 | (at3 << 16));
          unsigned long long next = (unsigned long long)((e & 0xffffu) | (o << 16)) |
                                    ((unsigned long long)((e >> 16) | (o & 0xffff0000u)) << 32);
#pragma unroll
          for (int s = 0; s < SMAX; ++s) {
            const uint32_t u = (uint32_t)N[s] - 1u;
            if (u < (uint32_t)kSmallM) {
              const uint32_t sh = (u << 2) & 48u;
              items[(uint32_t)(next >> sh) & 0xffffu] = (item_t)((N[s] << 10) | (lane << 4) | s);
              next += 1ull << sh;
            }
          }
        }
        settle<SMAX>(nxt);
      }
      wave_sync();
      const int total = n_drawn + n_item;
      int32_t* const out = run_counts(rd, window, 1u);
      for (int r0 = 0; r0 < total; r0 += kWave) {
        const int at = r0 + lane;
        const bool valid = at < total;
        int Ln = 0, sp = 0, m = 0;
        double nb = 0.0;
        bool general = false;  // uniform
        if (r0 < n_drawn) {    // a round with items of changed species
          general = true;
          if (valid) {
            const uint32_t itw = at < n_drawn ? (uint32_t)L.drawn[at] : (uint32_t)items[at - n_drawn];
            Ln = (int)((itw >> 4) & 63);
            sp = (int)(itw & 15);
            m = at < n_drawn ? npost[-at] : (int)(itw >> 10);
            nb = at < n_drawn ? L.nbar[at] : 0.0;
          }
        } else if (valid) {
          const uint32_t itw = (uint32_t)items[at - n_drawn];
          Ln = (int)((itw >> 4) & 63);
          sp = (int)(itw & 15);
          m = (int)(itw >> 10);
        }
        const bool plain = valid && at >= n_drawn;
        if (any_wide) {  // a count that does not fit its field is read from the count buffer
          if (plain && m == 0) {
            m = run_counts(rd, window, 0u)[(size_t)sp * T + base + Ln];
            renew(m);  // the other rounds do not wait for memory
          }
        }
        if (plain) nb = (double)m;
        general = general || __ballot(m > kSmallM) != 0ull;
        if (valid) {
          const int4 tnb = L.nbr[Ln];
          const double2 g0 = L.geo[0][Ln], g1 = L.geo[1][Ln];
          // 0 x infinity (no leaving) is not 1: zero is the larger of it and zero
          const ItemGeo geo{fmin(fmax(L.tauD[sp] * g0.x, 0.0), 1.0), g0.y, g1.x, g1.y};
          const uint32_t tet = (uint32_t)(base + Ln);
          int draws = m;
          DrawCounts c(geo);
          Faces o{0, 0, 0, 0};
          if (general) item_general(key0, key1, window, tet, sp, nb, m, geo, c, o, draws);
          count_draws(key0, key1, window, tet, sp, draws, c);
          const Faces d = c.faces();
          if (general) o = Faces{o.o0 + d.o0, o.o1 + d.o1, o.o2 + d.o2, o.o3 + d.o3};
          else o = d;
          // own remainder and moves to the tile's own tets go to LDS, the
          // rest to the next count buffer
          const int n = o.o0 + o.o1 + o.o2 + o.o3;
          int* const own = acc + sp * kWave;
          int32_t* const row = out + ((size_t)sp * T + base);
          if (m != n) atomicAdd(own + Ln, m - n);
#define RDX_DEPOSIT(t, v)                                              \
          if (v) {                                                     \
            if ((unsigned)(t) < (unsigned)width) atomicAdd(own + (t), (v)); \
            else atomicAdd(row + (t), (v));                            \
            ++n_faces;                                                 \
          }
          RDX_DEPOSIT(tnb.x, o.o0)
          RDX_DEPOSIT(tnb.y, o.o1)
          RDX_DEPOSIT(tnb.z, o.o2)
          RDX_DEPOSIT(tnb.w, o.o3)
#undef RDX_DEPOSIT
          n_moved += (unsigned long long)n;
        }
        wave_sync();
      }
      n_drawn = 0;
      if (last) break;
      // the counts are read again above: they are not held over the rounds
#pragma unroll
      for (int s = 0; s < SMAX; ++s) {
        int n;
        asm volatile("" : "=v"(n));
        N[s] = n;
      }
    }
    if (stepping) {
      // coalesced flush of the tile's own tets (other tiles add into them too);
      // the counts read are cleared for the window after next
      renew_s(S);
      if (active) {
        const uint32_t l = (uint32_t)lane;
        int32_t *in = run_counts(rd, window, 0u) + base, *out = run_counts(rd, window, 1u) + base;
#pragma unroll
        for (int s = 0; s < SMAX; ++s) {
          if (s < S) {
            const int v = acc[s * kWave + lane];
            if (v != 0) atomicAdd(out + l, v);
            in[l] = 0;
          }
          in += T;
          out += T;
        }
      }
      if (errbits) atomicOr(rd->err, errbits);
    }
    wave_sync();  // LDS is rebuilt for the next tile
    here = there;
    cur = nxt;
  }

  const unsigned long long ev = wave_sum(n_ev), mv = wave_sum(n_moved), fm = wave_sum(n_faces);
  if (threadIdx.x == kWave - 1 && cached != nullptr) {
    if (ev) atomicAdd(tally_slot(cached), ev);
    if (mv) atomicAdd(tally_slot(cached) + 1, mv);
    if (fm) atomicAdd(tally_slot(cached) + 2, fm);
  }
}

// Batched reset: one block per chunk.
__global__ void __launch_bounds__(kBlock) reset_chunks_kernel(const ResetChunk* chunks) {
  const ResetChunk c = chunks[blockIdx.x];
  for (int64_t j = c.begin + threadIdx.x; j < c.end; j += kBlock) {
    c.dst[j] = c.src[j];
    c.other[j] = 0;
  }
  if (c.begin == 0) {
    if (threadIdx.x < kTallyWords * kTallySlots) c.tally[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) *c.err = 0;
  }
}
__global__ void set_step_kernel(int32_t* word, int32_t value) { *word = value; }

// ----------------------------------------------------------- self-tests ----
// One vector per wave (block j of 64 lanes), so that its key is wave-uniform
// as in the window kernels; lane 0 writes.
__global__ void __launch_bounds__(kWave) selftest_philox_kernel(const uint32_t* in, uint32_t* out) {
  const int64_t j = blockIdx.x;
  const cptr<uint32_t> v = as_const(in) + 6 * j;
  uint32_t x0 = v[0], x1 = v[1], x2 = v[2], x3 = v[3];
  philox4x32_10(x0, x1, x2, x3, v[4], v[5]);
  if (threadIdx.x == 0) {
    out[4 * j] = x0;
    out[4 * j + 1] = x1;
    out[4 * j + 2] = x2;
    out[4 * j + 3] = x3;
  }
}

__global__ void selftest_ln_kernel(const double* x, double* y, int64_t n) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) y[j] = ln_basic(x[j]);
}

__global__ void selftest_binom_kernel(uint32_t key0, uint32_t key1, uint32_t stream_id,
                                      uint32_t window, long long m, double p, int64_t n,
                                      long long* out) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  Draw32 st(key0, key1, stream_id, (uint32_t)j, window);
  out[j] = binom<long long>(m, p, st);
}

__global__ void copy_kernel(const int4* __restrict__ src, int4* __restrict__ dst, int64_t n16) {
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n16;
       j += (int64_t)gridDim.x * blockDim.x)
    dst[j] = src[j];
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

// Blocks of a window kernel the device holds at once (occupancy x CUs), by the
// model's species count.
template <int SMAX, int RMAX>
int window_resident(int S) {
  static std::array<std::atomic<int>, SMAX + 1> known{};  // 0: not asked yet
  int n = known[S].load(std::memory_order_relaxed);
  if (n == 0) {
    int dev = 0, n_cu = 0, per_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void*>(&window_main_kernel<SMAX, RMAX>), kWave, tile_row_bytes<SMAX, RMAX>(S));
    per_cu = per_cu < lds_blocks<SMAX, RMAX>(S) ? per_cu : lds_blocks<SMAX, RMAX>(S);
    n = n_cu > 0 && per_cu > 0 ? n_cu * per_cu : 2048;
    known[S].store(n, std::memory_order_relaxed);
  }
  return n;
}

template <int SMAX, int RMAX>
hipError_t launch_one(const StepArgs& a, hipStream_t stream, hipEvent_t* marks) {
  if (marks) (void)hipEventRecord(marks[0], stream);
  hipLaunchKernelGGL((window_main_kernel<SMAX, RMAX>), dim3((unsigned)a.grid), dim3(kWave),
                     (tile_row_bytes<SMAX, RMAX>(a.S)), stream, a);
  if (marks) (void)hipEventRecord(marks[1], stream);
  return hipGetLastError();
}

int grid_resident(int S, int R) {
  if (S <= 4 && R <= 4) return window_resident<4, 4>(S);
  if (S <= 8 && R <= 8) return window_resident<8, 8>(S);
  if (S <= 12 && R <= 12) return window_resident<12, 12>(S);
  if (S <= 16 && R <= 24) return window_resident<16, 24>(S);
  return window_resident<16, 32>(S);
}

hipError_t launch_window(const StepArgs& a, hipStream_t stream, hipEvent_t* marks) {
  if (a.S <= 4 && a.R <= 4) return launch_one<4, 4>(a, stream, marks);
  if (a.S <= 8 && a.R <= 8) return launch_one<8, 8>(a, stream, marks);
  if (a.S <= 12 && a.R <= 12) return launch_one<12, 12>(a, stream, marks);
  if (a.S <= 16 && a.R <= 24) return launch_one<16, 24>(a, stream, marks);
  return launch_one<16, 32>(a, stream, marks);
}

hipError_t launch_set_step(int32_t* words, int32_t step, hipStream_t stream) {
  hipLaunchKernelGGL(set_step_kernel, dim3(1), dim3(1), 0, stream, words + (step & 1), step);
  return hipGetLastError();
}

hipError_t launch_reset_chunks(const ResetChunk* chunks, int64_t n_chunks, hipStream_t stream) {
  if (n_chunks <= 0) return hipSuccess;
  hipLaunchKernelGGL(reset_chunks_kernel, dim3((unsigned)n_chunks), dim3(kBlock), 0, stream, chunks);
  return hipGetLastError();
}

hipError_t launch_selftest_philox(const uint32_t* in, uint32_t* out, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(selftest_philox_kernel, dim3((unsigned)n), dim3(kWave), 0, s, in, out);
  return hipGetLastError();
}

hipError_t launch_selftest_ln(const double* x, double* y, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(selftest_ln_kernel, dim3(grid_for(n)), dim3(kBlock), 0, s, x, y, n);
  return hipGetLastError();
}

hipError_t launch_copy(const int4* src, int4* dst, int64_t n16, hipStream_t s) {
  hipLaunchKernelGGL(copy_kernel, dim3(256 * 16), dim3(kBlock), 0, s, src, dst, n16);
  return hipGetLastError();
}

hipError_t launch_selftest_binom(uint64_t seed, uint32_t stream_id, uint32_t window, int64_t m,
                                 double p, int64_t n, long long* out, hipStream_t s) {
  hipLaunchKernelGGL(selftest_binom_kernel, dim3(grid_for(n)), dim3(kBlock), 0, s,
                     (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32), stream_id, window,
                     (long long)m, p, n, out);
  return hipGetLastError();
}

}  // namespace rdx
