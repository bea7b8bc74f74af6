// Binomial Options region (Cox-Ross-Rubinstein tree, American or European
// call and put) with the paper's techniques.  The paper's Binomial Options
// benchmark has a whole group of threads price one option, so its decisions
// are taken per option by that group (section 4.1); here that group is one
// wavefront:
//
//   * one wave prices one option: a European price is the FP64 sum over the
//     leaves, an American one a backward induction over the live nodes of
//     the tree, ceil(nodes / 64) per lane in registers, a node's other
//     neighbour one lane away (a wavefront shift, no barrier and no LDS);
//   * a wave is the decision unit ("logical lane") of the techniques: unit u
//     of L = 64 ceil(ceil(n/IPT)/64) units processes options u + kL,
//     k < IPT, and decides alone for each (the thread level of section
//     3.1.2, the unit being the wave);
//   * iACT: the unit's table (tSize <= 64 entries of 5 inputs and 2 outputs)
//     is spread over the lanes, lane e holding entry e; distances are taken
//     in parallel with the oracle's FP32 rounding sequence, the minimum and
//     the lowest arg-min slot by a wave reduction and a ballot; a unit that
//     computed writes its entry round-robin;
//   * TAF: the unit's window of its last h accurate outputs, FP64 RSD test,
//     pSize approximate options after a passing test;
//   * perforation: herded over the unit's option loop (small, large, ini,
//     fini); a skipped option is neither read nor written.
//
// Bound by VALU issue.  65,536 American options on 512 steps: 2772 us when
// every step updated all 64 x 9 node slots of both values (9 instructions a
// node), 481 us with the triangle of nodes, two instructions a node and the
// European one of the two prices summed (6,435 VALU instructions per wave
// against 43,000, 2.6 clocks each); 1023 steps 9694 -> 1494 us, 127 steps
// 204 -> 94, 30 steps 68 -> 37; European 512 steps 1262 -> 98 us.
#include "launch_binomial.hpp"
#include <type_traits>
#include "wave.hpp"

namespace hpac {

namespace {

template <int N>
__device__ __forceinline__ float bo_dist2(const float (&x)[N], const float (&e)[N]) {
#pragma clang fp contract(off)
  float t = x[0] - e[0];
  float acc = t * t;
#pragma unroll
  for (int j = 1; j < N; ++j) {
    const float u = x[j] - e[j];
    acc = __builtin_fmaf(u, u, acc);
  }
  return acc;
}

// value of the next / previous lane, by a wavefront shift in the VALU (no LDS
// round trip on the step loop's dependence chain); lane 63 / lane 0, which
// have none, read 0 and never need it
__device__ __forceinline__ float from_next_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));  // wave_shl:1
}
__device__ __forceinline__ float from_prev_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));  // wave_shr:1
}

// Lane l's value of v, the same for every lane.
__device__ __forceinline__ double read_lane(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Inclusive prefix sum over the lanes (lane 63 ends with the wave's sum):
// row shifts scan each row of 16 lanes, row broadcasts carry the rows on; a
// lane with no source adds zero.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xf, true);
  return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_scan_add(double v) {
  v = dpp_add<0x111, 0xf>(v);  // row_shr:1
  v = dpp_add<0x112, 0xf>(v);  // row_shr:2
  v = dpp_add<0x114, 0xf>(v);  // row_shr:4
  v = dpp_add<0x118, 0xf>(v);  // row_shr:8
  v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
}

constexpr double kLog2eD = 1.4426950408889634074, kLn2D = 0.69314718055994530942;

// 2^x as m 2^e, m in [2^-1/2, 2^1/2], whatever the size of x: m by the Taylor
// series of e^t, |t| <= ln 2 / 2, to t^13 / 13! (the next term is below 5e-18).
struct Power2 {
  double m;
  int e;
  __device__ __forceinline__ explicit Power2(double x) {
    const double n = rint(x), t = (x - n) * kLn2D;
    double s = 1.0 / 6227020800.0;
    constexpr double kFact[13] = {1.0, 1.0, 2.0, 6.0, 24.0, 120.0, 720.0, 5040.0, 40320.0, 362880.0, 3628800.0,
                                  39916800.0, 479001600.0};
#pragma unroll
    for (int k = 12; k >= 0; --k) {
      double c = 1.0 / kFact[k];
      asm("" : "+s"(c));  // an operand in scalar registers, not moved to vector ones first
      s = __builtin_fma(s, t, c);
    }
    m = s;
    e = (int)n;
  }
};

struct BoOut {
  float call, put;
};

typedef __attribute__((address_space(3))) float LdsFloat;

__device__ __forceinline__ bool uniform(bool b) { return __builtin_amdgcn_readfirstlane((int)b) != 0; }

// What the FP64 part of a price hands on: the tree's FP32 parameters and the
// prices that need no induction.  16 dwords, the most that a function returns
// in registers: a 17th sends it through scratch memory, and 65,536 American
// options on 8 steps take 62 us instead of 33.
struct BoHead {
  double u, d, l2u;  // up and down factors, log2 u
  double pu, pd;     // discounted probabilities
  double X;          // spot at the lane's first leaf: S u^(2 j - N), j = lane ceil((N + 1) / 64)
  float call, put;   // European prices, where `sums` says so
  int sums;          // bit 0: the call is final, bit 1: the put is
  int regular;       // 0 < p < 1, prices positive and finite
};
static_assert(sizeof(BoHead) <= 64, "returned in registers");

// The tree's parameters and, with `sums`, its European call and put as what
// they are: the discounted expectation of the payoff over the leaves, whose
// up-move counts are binomially distributed.  N + 1 terms in FP64 instead of
// N^2 / 2 nodes: lane l takes C consecutive leaves; the first one's weight
// comes from a wave scan of log2 of the lanes' coefficient ratios, the
// others from w_{j+1} / w_j = (N - j) / (j + 1) p / (1 - p).
//
// Early exercise on this tree (no dividends): holding from a node with the
// exercise values X u - K and X d - K above it is worth at least
// pu (X u - K) + pd (X d - K) = X - K / a, so for r >= 0 a call is never
// exercised before its expiry, and with the signs turned a put never for
// r <= 0: such a price is the European one.  Irregular parameters (p outside
// (0, 1), prices that are not positive and finite, u above e^{300 / C}) leave
// both values to the induction.
//
// A function of its own: inlined, the FP64 constants and temporaries are kept
// in registers across the caller's option loop (over 200 VGPRs).
__device__ __attribute__((noinline)) BoHead bo_head(float Sf, float Kf, float T, float r, float v, int N,
                                                    bool american, bool sums) {
  const int lane = lane_id();
  const double dt = (double)T / N, su = (double)v * sqrt(dt), rdt = (double)r * dt;
  // the four exponentials of the tree in one evaluation, a lane each
  const double ex = exp(lane == 0 ? su : lane == 1 ? -su : lane == 2 ? rdt : -rdt);
  const double u = read_lane(ex, 0), d = read_lane(ex, 1), a = read_lane(ex, 2), disc = read_lane(ex, 3);
  const double p = (a - d) / (u - d), q = 1.0 - p, l2u = su * kLog2eD;
  const int C = (N + 64) >> 6;
  const int j0 = lane * C;
  const Power2 x((double)(2 * j0 - N) * l2u);  // the lane's first spot, over S
  BoHead h{u, d, l2u, p * disc, q * disc, ldexp((double)Sf * x.m, x.e), 0.0f, 0.0f, 0, 0};
  // the last one: a lane's weights and spots, of at most 16 leaves, do not run
  // from zero or infinity to a value that counts
  h.regular = uniform(p > 0.0 && q > 0.0 && Sf > 0.0f && Kf > 0.0f && Sf < INFINITY && Kf < INFINITY &&
                      fabs((double)C * su) < 300.0);
  if (sums) {
    if (h.regular)
      h.sums = (uniform(!american || r >= 0.0f) ? 1 : 0) | (uniform(!american || r <= 0.0f) ? 2 : 0);
    if (h.sums) {
      double num = 1.0, den = 1.0;
#pragma unroll 1
      for (int c = 0; c < C; ++c) {
        const int j = j0 + c;
        if (j < N) {
          num *= (double)(N - j);
          den *= (double)(j + 1);
        }
      }
      const double own = log2(num / den);
      const double before = wave_scan_add(own) - own;
      const double l2 = log2(lane == 0 ? p : q);
      const double l2p = read_lane(l2, 0), l2q = read_lane(l2, 1);
      const Power2 f(before + (double)j0 * l2p + (double)(N - j0) * l2q - (double)N * rdt * kLog2eD);
      double w = ldexp(f.m, f.e);
      const double u2 = u * u, K = (double)Kf, pq = p / q;
      double call = 0.0, put = 0.0;
      // far: the spots leave FP64's range, and their products with the weights,
      // which do not, take their place (a multiplication more per leaf: with
      // it throughout, 65,536 European options on 512 steps take 103 us, not 99)
      auto leaves = [&](auto far_tag) {
        constexpr bool kFar = decltype(far_tag)::value;
        double X = kFar ? ldexp((double)Sf * (f.m * x.m), f.e + x.e) : h.X;
#pragma unroll 1
        for (int c = 0; c < C; ++c) {
          const int j = j0 + c;
          if (j <= N) {
            call += kFar ? fmax(X - K * w, 0.0) : w * fmax(X - K, 0.0);
            put += kFar ? fmax(K * w - X, 0.0) : w * fmax(K - X, 0.0);
          }
          const double next = pq * ((double)(N - j) / (double)(j + 1));
          w *= next;
          X *= kFar ? next * u2 : u2;
        }
      };
      if (uniform(fabs((double)N * su) < 500.0))
        leaves(std::false_type{});
      else
        leaves(std::true_type{});
      h.call = (float)read_lane(wave_scan_add(call), 63);
      h.put = (float)read_lane(wave_scan_add(put), 63);
      if (american) {  // never below the exercise value, rounding included
        h.call = fmaxf(h.call, Sf - Kf);
        h.put = fmaxf(h.put, Kf - Sf);
      }
    }
  }
  return h;
}

// Backward induction of NV value arrays of one option over the 64 lanes of the
// calling wave; every lane returns the values at the root.
//
// Positions: after 2m steps node i sits at position i + m, and so it does one
// step later.  Position p then holds the spot S u^(2p-N) after an even
// number of steps and S u^(2p-N+1) after an odd one, whatever the step: what
// a node needs of its spot is one of two constant arrays (E0 even, E1 odd;
// no per-step spot update and no drift).  Even to odd steps take a node's
// upper neighbour, odd to even ones its lower.  Two steps shrink the live
// positions m .. N-m by one at either end, and as soon as they fit c - 1
// positions per lane instead of c they are dealt out anew through LDS, so
// the wave works on the triangle of nodes and not on its bounding rectangle.
// Positions outside the live range hold values that no live node reads.
// node(v, e, up, dn): value v of a node from the two it leads to; NE: constant
// arrays, one for every value or one of each.
template <int CM, int NV, int NE, class Node>
__device__ __forceinline__ void bo_walk(int N, int lane, LdsFloat *lds, float (&V)[NV][CM], float (&E0)[NE][CM],
                                        float (&E1)[NE][CM], const Node &node, float (&root)[NV]) {
  const int need = (N + 64) >> 6;
  int base = 0, m = 0;
  // one phase: c positions per lane, from base
  auto phase = [&](auto c_tag) {
    constexpr int c = decltype(c_tag)::value;
    if (c > need) return;
    if (c < need) {  // from c + 1 positions per lane: deal the live ones out from m
      // at most 33: a phase starts with at most 64 (c + 1) live positions and
      // ends with at least 64 c - 1, so every read below is inside 64 (c + 1)
      const int from = m - base;
      int ln = lane;
      asm volatile("" : "+v"(ln));  // addresses are formed here, not kept in registers throughout
      auto deal = [&](float (&a)[CM]) {
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < (c < CM ? c + 1 : c); ++k) lds[ln * (c + 1) + k] = a[k];
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < c; ++k) a[k] = lds[from + ln * c + k];
      };
#pragma unroll
      for (int v = 0; v < NV; ++v) deal(V[v]);
#pragma unroll
      for (int v = 0; v < NE; ++v) {
        deal(E0[v]);
        deal(E1[v]);
      }
      base = m;
    }
    const int stop = c > 1 ? 64 * (c - 1) : 2;  // live positions at which the phase ends
    for (; N - 2 * m + 1 > stop; ++m) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {  // even to odd
        const float up = from_next_lane(V[v][0]);
#pragma unroll
        for (int k = 0; k < c; ++k) V[v][k] = node(v, E1[v % NE][k], k + 1 < c ? V[v][k + 1 < c ? k + 1 : k] : up, V[v][k]);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {  // odd to even
        const float dn = from_prev_lane(V[v][c - 1]);
#pragma unroll
        for (int k = c - 1; k >= 0; --k) V[v][k] = node(v, E0[v % NE][k], V[v][k], k ? V[v][k ? k - 1 : 0] : dn);
      }
    }
  };
  auto phases = [&](auto self, auto c_tag) -> void {
    constexpr int c = decltype(c_tag)::value;
    phase(c_tag);
    if constexpr (c > 1) self(self, std::integral_constant<int, c - 1>{});
  };
  phases(phases, std::integral_constant<int, CM>{});
  // m = floor(N / 2); an odd N has one step, even to odd, left
  const int at = m - base;  // < 64: the live positions fit one per lane
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const float last = node(v, E1[v % NE][0], from_next_lane(V[v][0]), V[v][0]);
    root[v] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int((N & 1) ? last : V[v][0]), at));
  }
}

// Lane index for an induction's first positions: opaque, so that what depends
// on it is formed there and not kept in registers across the option loop.
__device__ __forceinline__ int fresh_lane() {
  int lane = lane_id();
  asm volatile("" : "+v"(lane));
  return lane;
}

// American prices by their early-exercise premium, for regular parameters
// and N >= 1.  With the exercise value e = max(sgn (X - K), 0) of a node and
// A = V - e >= 0, V = max(continuation, e) becomes
//   A = max(pu A_up + pd A_dn + D, 0),  D = pu e_up + pd e_dn - e,
// with A = 0 on the leaves.  D depends on the position alone and is formed
// once, in FP64.  Scaled by a power of two not below A's largest value the
// maximum is the clamp of the second multiply-add, so a node costs two
// instructions; max itself would be a third, and one that issues at half the
// rate of a multiply-add.  That value is at most K for a call, which is worth
// at most its spot at any rate, and for a put at r >= 0; at r < 0 a put is
// worth up to K e^{|r| T}, and its scale is larger by that (put_exp).  The
// rounding errors are those of the premium, not of the price, and D is an
// exact zero where the option is out of the money.  NV = 2: call (value 0) and
// put; NV = 1, longer trees: the one whose European price is not its own, so a
// put at r > 0 only.
template <int CM, int NV>
__device__ __forceinline__ void bo_premium(const BoHead &q, float Sf, float Kf, int N, float sgn, int put_exp,
                                           LdsFloat *lds, float (&price)[NV]) {
  const int lane = fresh_lane();
  const int need = (N + 64) >> 6;
  const int kexp = __builtin_amdgcn_frexp_expf(Kf);  // K <= 2^kexp
  float A[NV][CM], D0[NV][CM], D1[NV][CM];
  const double K = (double)Kf, u2 = q.u * q.u;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double sg = NV == 2 ? (v == 0 ? 1.0 : -1.0) : (double)sgn;
    const int ks = kexp + (NV == 2 && v == 1 ? put_exp : 0);
    auto ex = [&](double x) { return fmax(sg * (x - K), 0.0); };
    double X = q.X;
    double below = ex(X * q.d), e = ex(X);  // at the odd position below, at this even position
#pragma unroll
    for (int c = 0; c < CM; ++c) {
      A[v][c] = D0[v][c] = D1[v][c] = 0.0f;
      if (c < need) {
        const double odd = ex(X * q.u);
        X *= u2;
        const double up = ex(X);
        D0[v][c] = ldexpf((float)(q.pu * odd + q.pd * below - e), -ks);
        D1[v][c] = ldexpf((float)(q.pu * up + q.pd * e - odd), -ks);
        below = odd;
        e = up;
      }
      // one position after the other: side by side, their FP64 temporaries
      // would take over a hundred registers more
      asm volatile("" : "+v"(D0[v][c]), "+v"(D1[v][c]));
    }
  }
  const float pu = (float)q.pu, pd = (float)q.pd;
  auto node = [&](int, float d, float up, float dn) {
    const float t = __builtin_fmaf(pu, up, __builtin_fmaf(pd, dn, d));
    return __builtin_amdgcn_fmed3f(t, 0.0f, 1.0f);  // the clamp modifier
  };
  float root[NV];
  bo_walk<CM, NV, NV>(N, lane, lds, A, D0, D1, node, root);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const float sg = NV == 2 ? (v == 0 ? 1.0f : -1.0f) : sgn;
    price[v] = ldexpf(root[v], kexp + (NV == 2 && v == 1 ? put_exp : 0)) + fmaxf(sg * (Sf - Kf), 0.0f);
  }
}

// The induction on the prices themselves, for any parameters (NV = 2: call
// and put; NV = 1: the one of sign sgn): a node is its continuation or, where
// american, its exercise value if that is larger.
template <int CM, int NV>
__device__ __forceinline__ void bo_values(const BoHead &q, float S, float K, int N, bool american, float sgn,
                                          LdsFloat *lds, float (&price)[NV]) {
  const int lane = fresh_lane();
  const int need = (N + 64) >> 6;
  const float pu = (float)q.pu, pd = (float)q.pd;
  const float l2u = (float)q.l2u, l2ul = (float)(q.l2u - (double)l2u);
  float V[NV][CM], E0[1][CM], E1[1][CM];  // exercise values, NaN (no exercise) for European options
  // S u^k, the exponent's rounding error e carried into the result; where the
  // exponent is infinite e is NaN, and some number takes its place
  auto spot = [&](int k) {
    const float f = (float)k, h = f * l2u;
    const float e = __builtin_amdgcn_fmed3f(__builtin_fmaf(f, l2ul, __builtin_fmaf(f, l2u, -h)), -1.0f, 1.0f);
    return S * (__builtin_amdgcn_exp2f(h) * __builtin_fmaf(e, 0.693147180559945309f, 1.0f));
  };
#pragma unroll
  for (int c = 0; c < CM; ++c) {
    const int p = lane * need + c;
    const float x0 = sgn * (spot(2 * p - N) - K), x1 = sgn * (spot(2 * p - N + 1) - K);
#pragma unroll
    for (int v = 0; v < NV; ++v) V[v][c] = fmaxf(v ? -x0 : x0, 0.0f);
    E0[0][c] = american ? x0 : __builtin_nanf("");
    E1[0][c] = american ? x1 : __builtin_nanf("");
    asm volatile("" : "+v"(E0[0][c]), "+v"(E1[0][c]));  // one position after the other, as above
  }
  // max(cont, e) as the instruction itself: fmaxf would first quiet e, a
  // register from outside the loop, with a second one.  Like fmaxf it returns
  // the other operand when one is NaN, and NaN when both are.
  auto node = [&](int v, float e, float up, float dn) {
    const float cont = __builtin_fmaf(pu, up, pd * dn);
    float x;
    if (v)
      asm("v_max_f32_e64 %0, %1, -%2" : "=v"(x) : "v"(cont), "v"(e));
    else
      asm("v_max_f32_e32 %0, %1, %2" : "=v"(x) : "v"(cont), "v"(e));
    return x;
  };
  bo_walk<CM, NV, 1>(N, lane, lds, V, E0, E1, node, price);
}

// Longer trees with irregular parameters; rare, and a function of its own so
// that each kernel does not carry a copy.
template <int CM>
__device__ __attribute__((noinline)) BoOut bo_irregular(const BoHead q, float S, float K, int N, bool american,
                                                        LdsFloat *lds) {
  BoOut o{0.0f, 0.0f};
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {
    float p[1];
    bo_values<CM, 1>(q, S, K, N, american, side == 0 ? 1.0f : -1.0f, lds, p);
    (side == 0 ? o.call : o.put) = p[0];
  }
  return o;
}

// Call and put of one option on the N-step tree, computed by the calling wave.
// From 64 steps (European) or 128 (American) on, a European price comes from
// the leaf sum and only the other one, if any, goes through an induction.
template <int CM>
__device__ __forceinline__ BoOut bo_price(float S, float K, float T, float r, float v, int N, bool american,
                                          LdsFloat *lds) {
  const BoHead q = bo_head(S, K, T, r, v, N, american, CM > 2 || (!american && N >= 64));
  const int sums = __builtin_amdgcn_readfirstlane(q.sums);
  const bool regular = __builtin_amdgcn_readfirstlane(q.regular) != 0;
  BoOut o{q.call, q.put};
  if (sums == 3) return o;
  if constexpr (CM <= 2) {
    float p[2];
    if (american && regular) {
      int put_exp = 0;  // 2^put_exp is at least e^{-r T}
      if (uniform(r < 0.0f)) put_exp = (int)ceil(fmin(-(double)r * (double)T * kLog2eD, 4096.0));
      bo_premium<CM, 2>(q, S, K, N, -1.0f, put_exp, lds, p);
    } else {
      bo_values<CM, 2>(q, S, K, N, american, 1.0f, lds, p);
    }
    o = BoOut{p[0], p[1]};
  } else {
    if (!regular) return bo_irregular<CM>(q, S, K, N, american, lds);
    float p[1];
    bo_premium<CM, 1>(q, S, K, N, sums == 1 ? -1.0f : 1.0f, 0, lds, p);
    (sums == 1 ? o.put : o.call) = p[0];
  }
  return o;
}

// Division-free FP64 RSD test over the h window slots (slot h-1 newest):
// var < theta^2 mu^2  <=>  D < h theta^2 s^2, D == 0 passes iff theta > 0.
template <int H>
__device__ __forceinline__ bool bo_rsd_below(const float (&w)[H][2], double th2, bool th_pos) {
  bool ok = true;
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < H; ++q) s += (double)w[q][o];
    double D = 0.0;
#pragma unroll
    for (int q = 0; q < H; ++q) {
      const double dd = (double)H * (double)w[q][o] - s;
      D = __builtin_fma(dd, dd, D);
    }
    ok = ok && (D == 0.0 ? th_pos : D < (double)H * th2 * (s * s));
  }
  return ok;
}

// per-block counters: lane 0 of each wave adds into LDS, thread 0 publishes
struct BoStats {
  unsigned long long *g, *s;
  __device__ void begin() {
    if (!g) return;
    if (threadIdx.x < 4) s[threadIdx.x] = 0;
    __syncthreads();
  }
  __device__ void end(unsigned long long visited, unsigned long long approx) {
    if (!g) return;
    if (lane_id() == 0) {
      atomicAdd(&s[0], visited);
      atomicAdd(&s[1], approx);
      atomicAdd(&s[2], approx);
      atomicAdd(&s[3], visited);
    }
    __syncthreads();
    if (threadIdx.x < 4 && s[threadIdx.x]) atomicAdd(&g[threadIdx.x], s[threadIdx.x]);
  }
};

__device__ __forceinline__ uint32_t bo_trace_word(bool approx, bool voted, bool crit) {
  return 0x80000000u | (crit ? 1u : 0u) | ((approx ? 1u : 0u) << 8) | ((approx ? 1u : 0u) << 24) |
         ((voted ? 1u : 0u) << 25);
}

}  // namespace

// TECH: 0 exact, 1 iACT, 2 TAF, 3 perforation, 4 dense small/large
// perforation.  H: TAF history (1..8).
//
// Dense perforation (no trace or counters): the region keeps no state, so
// the options a herded small/large pattern keeps -- whole steps k, i.e. the
// option ranges [kL, (k+1)L) -- can be priced by any wavefronts: one option
// per wavefront over the kept ranges only, so every SIMD gets the same share
// of trees whatever the options per unit.  The outputs are those of TECH 3.
template <int CM, int TECH, int H>
__global__ void __launch_bounds__(256) k_binomial(BoArgs a) {
  __shared__ unsigned long long sums[4];
  __shared__ float deal[4][64 * CM];  // per wave: positions changing lanes
  LdsFloat *const lds = (LdsFloat *)deal[threadIdx.x >> 6];
  const int lane = lane_id();
  const int64_t unit = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (TECH == 4) {
    // wavefront -> r-th kept step; kept steps repeat with period M: small
    // keeps every position of a period but `special`, large only `special`
    const int64_t r = unit / a.L;
    const int64_t P = r / a.kept_per_period;
    const int rem = (int)(r - P * a.kept_per_period);
    const int pos = a.kind == 1 ? a.special : (rem < a.special ? rem : rem + 1);
    const int64_t i = (P * a.param + pos) * a.L + (unit - r * a.L);
    if (i < a.n) {
      float x[5];
#pragma unroll
      for (int j = 0; j < 5; ++j) x[j] = a.in[j][i];
      const BoOut y = bo_price<CM>(x[0], x[1], x[2], x[3], x[4], a.steps, a.american, lds);
      if (lane == 0) {
        a.out[0][i] = y.call;
        a.out[1][i] = y.put;
      }
    }
    return;
  }
  BoStats stats{a.counters, sums};
  stats.begin();
  unsigned long long visited = 0, approxd = 0;
  // iACT: lane e holds entry e
  float ex[5] = {0, 0, 0, 0, 0}, ey[2] = {0, 0};
  int cnt = 0, ins = 0;
  const float thr2 = a.threshold * a.threshold;
  // TAF
  float win[H][2];
#pragma unroll
  for (int q = 0; q < H; ++q) win[q][0] = win[q][1] = 0.0f;
  int fill = 0, rho = 0;
  const double th = (double)a.threshold;

  for (int k = 0; k < a.ipt && unit < a.L; ++k) {
    const int64_t i = unit + (int64_t)k * a.L;
    if (i >= a.n) break;
    visited += 1;
    if (TECH == 3) {
      bool skip = false;
      const int M = a.param;
      if (M > 0) {
        switch (a.kind) {
          case 0: skip = (int)(((int64_t)k + a.offset) % M) == M - 1; break;
          case 1: skip = (int)(((int64_t)k + a.offset) % M) != 0; break;
          case 2: skip = i < (int64_t)M * a.n / 100; break;
          default: skip = i >= a.n - (int64_t)M * a.n / 100; break;
        }
      }
      if (skip) {
        approxd += 1;
        if (a.trace && lane == 0) a.trace[unit * a.ipt + k] = bo_trace_word(true, false, false);
        continue;
      }
    }
    if (TECH == 2 && rho > 0) {
      rho -= 1;
      approxd += 1;
      if (lane == 0) {
        a.out[0][i] = win[H - 1][0];
        a.out[1][i] = win[H - 1][1];
        if (a.trace) a.trace[unit * a.ipt + k] = bo_trace_word(true, false, false);
      }
      continue;
    }
    float x[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) x[j] = a.in[j][i];
    if (TECH == 1 && cnt > 0) {
      const float d2 = lane < cnt ? bo_dist2<5>(x, ex) : INFINITY;
      const float md2 = -wave_max(-d2);
      if (md2 < thr2) {
        const int arg = lowest_lane(ballot(lane < cnt && d2 == md2));
        const float yc = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ey[0]), arg));
        const float yp = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ey[1]), arg));
        approxd += 1;
        if (lane == 0) {
          a.out[0][i] = yc;
          a.out[1][i] = yp;
          if (a.trace) a.trace[unit * a.ipt + k] = bo_trace_word(true, true, true);
        }
        continue;
      }
    }
    const BoOut y = bo_price<CM>(x[0], x[1], x[2], x[3], x[4], a.steps, a.american, lds);
    if (lane == 0) {
      a.out[0][i] = y.call;
      a.out[1][i] = y.put;
    }
    bool voted = false, crit = false;
    if (TECH == 1) {
      const int slot = ins % a.tsize;
      if (lane == slot) {
#pragma unroll
        for (int j = 0; j < 5; ++j) ex[j] = x[j];
        ey[0] = y.call;
        ey[1] = y.put;
      }
      cnt = cnt < a.tsize ? cnt + 1 : a.tsize;
      ins += 1;
      voted = true;
    }
    if (TECH == 2) {
#pragma unroll
      for (int q = 0; q + 1 < H; ++q) {
        win[q][0] = win[q + 1][0];
        win[q][1] = win[q + 1][1];
      }
      win[H - 1][0] = y.call;
      win[H - 1][1] = y.put;
      fill = fill < H ? fill + 1 : H;
      if (fill == H) {
        voted = true;
        crit = bo_rsd_below<H>(win, th * th, th > 0.0);
        if (crit) rho = a.psize;
      }
    }
    if (a.trace && lane == 0) a.trace[unit * a.ipt + k] = bo_trace_word(false, voted, crit);
  }
  stats.end(visited, approxd);
}

// --------------------------------------------------------------- launchers

int64_t bo_units(int64_t n, int ipt) { return 64 * (((n + ipt - 1) / ipt + 63) / 64); }

// Most positions per lane a kernel is instantiated for: a tree of N steps
// starts with ceil((N+1)/64) of them; N is at most 1023.
int bo_positions_per_lane(int steps) {
  const int need = (steps + 64) / 64;
  for (int c : {2, 4, 8, 12, 16})
    if (need <= c) return c;
  return 0;
}

template <int C, int TECH>
static void bo_go_h(const BoArgs &a, int block, hipStream_t s) {
  if (TECH == 3 && !a.trace && !a.counters && a.param > 0) {
    if (a.kind == 0 || a.kind == 1) {
      // small / large: the kept steps below the last one that holds options
      const int M = a.param;
      const int off = (int)(a.offset % M);
      BoArgs b = a;
      b.special = a.kind == 0 ? ((M - 1 - off) % M + M) % M : ((M - off) % M + M) % M;
      b.kept_per_period = a.kind == 0 ? M - 1 : 1;
      if (b.kept_per_period == 0) return;  // small with M = 1 drops every step
      const int64_t steps = (a.n + a.L - 1) / a.L;
      int64_t kept = (steps / M) * b.kept_per_period;
      for (int64_t st = (steps / M) * M; st < steps; ++st) {
        const int pos = (int)(st % M);
        kept += a.kind == 0 ? pos != b.special : pos == b.special;
      }
      if (kept == 0) return;
      if (kept * a.L * 64 > 0xFFFFFFFFll) {  // beyond a 32-bit grid: one unit per lane group, as traced
        hipLaunchKernelGGL((k_binomial<C, TECH, 1>), dim3((unsigned)(a.L * 64 / block)), dim3(block), 0, s, a);
        return;
      }
      hipLaunchKernelGGL((k_binomial<C, 4, 1>), dim3((unsigned)(kept * a.L * 64 / block)), dim3(block), 0, s, b);
      return;
    }
    // ini / fini: the kept options are one contiguous range, one per unit
    const int64_t cut = ((int64_t)a.param * a.n) / 100;
    const int64_t lo = a.kind == 2 ? cut : 0;
    BoArgs b = a;
    b.n = a.n - cut;
    if (b.n == 0) return;
    b.ipt = 1;
    b.L = bo_units(b.n, 1);
    if (b.L * 64 > 0xFFFFFFFFll) {  // beyond a 32-bit grid: the caller's units, as traced
      hipLaunchKernelGGL((k_binomial<C, TECH, 1>), dim3((unsigned)(a.L * 64 / block)), dim3(block), 0, s, a);
      return;
    }
    for (int j = 0; j < 5; ++j) b.in[j] = a.in[j] + lo;
    for (int o = 0; o < 2; ++o) b.out[o] = a.out[o] + lo;
    hipLaunchKernelGGL((k_binomial<C, 0, 1>), dim3((unsigned)(b.L * 64 / block)), dim3(block), 0, s, b);
    return;
  }
  const dim3 grid((unsigned)(a.L * 64 / block));
  if (TECH != 2) {
    hipLaunchKernelGGL((k_binomial<C, TECH, 1>), grid, dim3(block), 0, s, a);
    return;
  }
  switch (a.hsize) {
    case 1: hipLaunchKernelGGL((k_binomial<C, 2, 1>), grid, dim3(block), 0, s, a); break;
    case 2: hipLaunchKernelGGL((k_binomial<C, 2, 2>), grid, dim3(block), 0, s, a); break;
    case 3: hipLaunchKernelGGL((k_binomial<C, 2, 3>), grid, dim3(block), 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_binomial<C, 2, 4>), grid, dim3(block), 0, s, a); break;
    case 5: hipLaunchKernelGGL((k_binomial<C, 2, 5>), grid, dim3(block), 0, s, a); break;
    case 6: hipLaunchKernelGGL((k_binomial<C, 2, 6>), grid, dim3(block), 0, s, a); break;
    case 7: hipLaunchKernelGGL((k_binomial<C, 2, 7>), grid, dim3(block), 0, s, a); break;
    default: hipLaunchKernelGGL((k_binomial<C, 2, 8>), grid, dim3(block), 0, s, a); break;
  }
}

template <int C>
static void bo_go_c(const BoArgs &a, int tech, int block, hipStream_t s) {
  switch (tech) {
    case 0: bo_go_h<C, 0>(a, block, s); break;
    case 1: bo_go_h<C, 1>(a, block, s); break;
    case 2: bo_go_h<C, 2>(a, block, s); break;
    default: bo_go_h<C, 3>(a, block, s); break;
  }
}

hipError_t launch_binomial(const BoArgs &a, int tech, int block, hipStream_t s) {
  switch (bo_positions_per_lane(a.steps)) {
    case 2: bo_go_c<2>(a, tech, block, s); break;
    case 4: bo_go_c<4>(a, tech, block, s); break;
    case 8: bo_go_c<8>(a, tech, block, s); break;
    case 12: bo_go_c<12>(a, tech, block, s); break;
    case 16: bo_go_c<16>(a, tech, block, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace hpac
