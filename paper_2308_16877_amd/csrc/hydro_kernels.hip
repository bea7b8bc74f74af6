// Lagrangian hydrodynamics on a structured hexahedral mesh (a Sedov point
// blast) with the paper's techniques applied across timesteps to two
// per-element regions: the hourglass-force region (TAF or herded
// perforation) and the EOS region (TAF).  The paper approximates the
// hourglass computation of its hydrodynamics proxy and reports the final
// origin energy as quantity of interest (section 4, Table 1 and 4.1).
//
// Scheme (our own, from published methods; FP32 state, FP64 time step):
//   n^3 elements on [0, side]^3, (n+1)^3 nodes, symmetry planes x=0, y=0,
//   z=0, free outer faces.  Element (i,j,k), corner a + 2b + 4c is node
//   (i+a, j+b, k+c); reference coordinates s = (2a-1, 2b-1, 2c-1).
//   k_hydro_force  per element: volume V and its gradient B = dV/dx in
//                  closed form (exact for a trilinear hexahedron);
//                  corner forces (p + q) B + hourglass forces (viscous
//                  Flanagan-Belytschko form); the element's FP64 time-step
//                  bound, reduced per workgroup.
//   k_hydro_dt     dt = min(growth * previous dt, all bounds); time += dt.
//   k_hydro_node   per node: gather of the adjacent corner forces in corner
//                  order (no atomics), u' = u + dt F / M, zero normal
//                  velocity on the symmetry planes, x += dt (u + u') / 2.
//   k_hydro_eos    per element: compatible energy update m de = -dt
//                  sum F . (u + u')/2 (Caramana et al. 1998), ideal-gas
//                  pressure, von Neumann-Richtmyer viscosity from the
//                  volume rate sum B(x') . (u + u')/2, sound speed.
// One element per lane, so a wave is 64 consecutive elements and a TAF
// "step" is a timestep: windows live in HBM.  At wave level the countdown
// and push count of each wave are one int each, read by the whole wave and
// written by its first lane; at thread level every element has its own.
// An approximate EOS step reads only the countdown; an approximate
// hourglass step adds the last accurate hourglass forces -- the newest slot
// of its window -- instead of computing them.  A perforated hourglass
// iteration adds nothing.
//
// The kernels are bound by memory, by its latency on small meshes: every
// kernel issues all of its loads before it waits for the first and before its
// first store (with the node gather's corners loaded one branch after the
// other the node kernel took 6.9 us on 24^3 elements, now 4.0, and 17.0 on
// 90^3, now 16.2).
#include "launch_hydro.hpp"
#include "wave.hpp"

#include <mutex>
#include <type_traits>

namespace hpac {

namespace {

constexpr float sgnf(int c, int d) { return ((c >> d) & 1) ? 1.0f : -1.0f; }

// Hourglass base vectors: products of reference coordinates.
constexpr float gamma_base(int a, int k) {
  return a == 0 ? sgnf(k, 1) * sgnf(k, 2)
       : a == 1 ? sgnf(k, 0) * sgnf(k, 2)
       : a == 2 ? sgnf(k, 0) * sgnf(k, 1)
                : sgnf(k, 0) * sgnf(k, 1) * sgnf(k, 2);
}

// Volume and, with kGrad, B = dV/dx of the trilinear hexahedron, in closed
// form.  Writing the map in the Walsh-Hadamard basis of the corner signs,
// x(xi) = a0 + a1 xi + a2 eta + a3 zeta + a4 xi eta + a5 xi zeta + a6 eta zeta
// + a7 xi eta zeta with a_k = 1/8 sum_c h_k(c) x_c, and integrating det J
// over the reference cube, the odd monomials vanish and
//   V = 8 [a1, a2, a3] + 8/3 ([a1, a4, a5] + [a4, a2, a6] + [a5, a6, a3]),
// [x, y, z] = x . (y cross z); a0 and a7 drop out.  Then dV/da_k = g_k (cross
// products of the others) and B_c = 1/8 sum_k g_k h_k(c): two 8-point
// Hadamard transforms and twelve cross products, about a quarter of the
// Gauss-point work, and the same values (the Gauss rule is exact here).
// The transform is taken of x_c - x_0, differences that neighbouring FP32
// coordinates give almost exactly, since the coordinates themselves far
// exceed an element's size.
__device__ __forceinline__ void cross3(const float (&u)[3], const float (&v)[3], float (&w)[3]) {
  w[0] = __builtin_fmaf(u[1], v[2], -u[2] * v[1]);
  w[1] = __builtin_fmaf(u[2], v[0], -u[0] * v[2]);
  w[2] = __builtin_fmaf(u[0], v[1], -u[1] * v[0]);
}
__device__ __forceinline__ float dot3(const float (&u)[3], const float (&v)[3]) {
  return __builtin_fmaf(u[0], v[0], __builtin_fmaf(u[1], v[1], u[2] * v[2]));
}

template <bool kGrad>
__device__ __forceinline__ float hex_volume(const float (&x)[8][3], float (&B)[8][3]) {
  // A[m] = 8 a_m: Hadamard transform of the corner offsets; bit 0 of m is
  // the xi factor, bit 1 eta, bit 2 zeta (a1 = A[1], a2 = A[2], a3 = A[4],
  // a4 = A[3], a5 = A[5], a6 = A[6])
  float A[8][3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    float d[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) d[c] = c ? x[c][i] - x[0][i] : 0.0f;
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (!((c >> j) & 1)) {
          const float lo = d[c], hi = d[c | (1 << j)];
          d[c] = lo + hi;
          d[c | (1 << j)] = hi - lo;
        }
#pragma unroll
    for (int m = 0; m < 8; ++m) A[m][i] = d[m];
  }
  const float(&A1)[3] = A[1], (&A2)[3] = A[2], (&A3)[3] = A[4], (&A4)[3] = A[3], (&A5)[3] = A[5],
               (&A6)[3] = A[6];
  constexpr float kThird = 1.0f / 3.0f;
  float x23[3], x45[3], x26[3], x63[3];
  cross3(A2, A3, x23);
  cross3(A4, A5, x45);
  cross3(A2, A6, x26);
  cross3(A6, A3, x63);
  // G1 = A2 x A3 + (A4 x A5) / 3 = 64 dV/dA1 (times 8 a1 . G1 it gives the leading terms)
  float G1[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) G1[i] = __builtin_fmaf(x45[i], kThird, x23[i]);
  const float V = (dot3(A1, G1) + (dot3(A4, x26) + dot3(A5, x63)) * kThird) * (1.0f / 64.0f);
  if (kGrad) {
    float x31[3], x64[3], x12[3], x56[3], x51[3], x14[3], x42[3], x35[3];
    cross3(A3, A1, x31);
    cross3(A6, A4, x64);
    cross3(A1, A2, x12);
    cross3(A5, A6, x56);
    cross3(A5, A1, x51);
    cross3(A1, A4, x14);
    cross3(A4, A2, x42);
    cross3(A3, A5, x35);
    // E[m] = 64 dV/dA_m at the Hadamard position m, then the inverse transform
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      float E[8];
      E[0] = 0.0f;
      E[7] = 0.0f;
      E[1] = G1[i];
      E[2] = __builtin_fmaf(x64[i], kThird, x31[i]);
      E[4] = __builtin_fmaf(x56[i], kThird, x12[i]);
      E[3] = (x51[i] + x26[i]) * kThird;
      E[5] = (x14[i] + x63[i]) * kThird;
      E[6] = (x42[i] + x35[i]) * kThird;
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int m = 0; m < 8; ++m)
          if (!((m >> j) & 1)) {
            const float u = E[m], v = E[m | (1 << j)];
            E[m] = u - v;
            E[m | (1 << j)] = u + v;
          }
#pragma unroll
      for (int c = 0; c < 8; ++c) B[c][i] = E[c] * (1.0f / 64.0f);
    }
  }
  return V;
}

__device__ __forceinline__ void hourglass(const float (&x)[8][3], const float (&u)[8][3], const float (&B)[8][3],
                                          float V, float rho, float c, float khg, float (&f)[8][3]) {
  const float inv_v = 1.0f / V;
  float h[4][3];
  float gam[4][8];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    float gx[3];
    // both sums vanish on constants (the base vectors and the hourglass
    // vectors sum to zero), so they are taken relative to corner 0
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      float s = 0.0f;
#pragma unroll
      for (int k = 1; k < 8; ++k) s = __builtin_fmaf(gamma_base(a, k), x[k][i] - x[0][i], s);
      gx[i] = s * inv_v;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      gam[a][k] = gamma_base(a, k) - (gx[0] * B[k][0] + gx[1] * B[k][1] + gx[2] * B[k][2]);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      float s = 0.0f;
#pragma unroll
      for (int k = 1; k < 8; ++k) s = __builtin_fmaf(gam[a][k], u[k][i] - u[0][i], s);
      h[a][i] = s;
    }
  }
  const float cv = cbrtf(V);
  const float coef = -(khg * 0.125f) * rho * c * (cv * cv);
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      float s = 0.0f;
#pragma unroll
      for (int a = 0; a < 4; ++a) s = __builtin_fmaf(gam[a][k], h[a][i], s);
      f[k][i] = coef * s;
    }
}

// Element and node arrays hold at most 1001^3 floats, so a byte offset into
// one fits 32 bits: a load or store takes the array's base from scalar
// registers and one 32-bit offset, the same for every array of its kind,
// instead of a 64-bit address formed per access.  The fused kernel goes from
// 200 to 161 registers (three waves per SIMD instead of two) and from 37.4 to
// 30.4 us at 90^3, the EOS alone from 22.5 to 18.6, the force from 23.0 to 21.2.
template <class T>
__device__ __forceinline__ T &at(T *base, uint32_t off) {
  using Byte = std::conditional_t<std::is_const_v<T>, const char, char>;
  return *(T *)((Byte *)base + (uint64_t)off);
}

// The 24 planes of the corner forces in order: the current plane's base in
// scalar registers, opaque so that the planes' bases are not all formed (and
// held, in vector registers too) beforehand.
template <class T>
struct Planes {
  T *base;
  uint64_t off = 0;
  __device__ __forceinline__ T *next(int64_t E) {
    using Byte = std::conditional_t<std::is_const_v<T>, const char, char>;
    T *p = (T *)((Byte *)base + off);
    off += 4 * (uint64_t)E;
    asm volatile("" : "+s"(off));
    return p;
  }
};

struct ElemIdx {
  uint32_t z;        // byte offset of the element
  uint32_t node[4];  // byte offsets of the nodes of corners 0, 2, 4 and 6; the odd ones follow them
  __device__ ElemIdx(int64_t z_, const DivBy &dn) {
    const uint32_t n = dn.d, m = n + 1, ze = (uint32_t)z_;
    const uint32_t t = dn.quo(ze), k = dn.quo(t);
    const uint32_t i = ze - t * n, j = t - k * n;
    z = 4 * ze;
    node[0] = 4 * (i + m * (j + m * k));
    node[1] = node[0] + 4 * m;
    node[2] = node[0] + 4 * m * m;
    node[3] = node[2] + 4 * m;
  }
};

// The second of two neighbouring nodes is a load of its own: its offset is a
// 32-bit sum, which the compiler cannot merge into one 8-byte load at a
// 4-byte-aligned address (merged, the fused kernel took 33.5 us).
__device__ __forceinline__ void gather3(const float *const *src, const ElemIdx &e, float (&v)[8][3]) {
#pragma unroll
  for (int c = 0; c < 8; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) v[c][d] = at(src[d], e.node[c >> 1] + (c & 1 ? 4u : 0u));
}

// Whether the RSD of every output over the h window slots is below theta.
// The value y in slot `fresh`, just pushed by this thread, is read back as
// a pivot.  With the deviations d_q = w_q - y of the other slots (exact in
// FP64 for FP32 data), s' = sum d_q and Q = sum d_q^2, the two-pass
// statistic is
//   D = sum_q (h w_q - s)^2 = h (h Q - s'^2),   s = sum_q w_q = h y + s',
// shifted by a sample so that it does not cancel (h Q >= s'^2 by
// Cauchy-Schwarz, so D >= 0).  Division-free test D < h theta^2 s^2, and D
// == 0 (a constant window) passes whenever theta > 0, as in the
// Black-Scholes TAF.  Outputs go in groups of G, a slot of a whole group per
// memory round trip; the first failing group decides.
template <int NO, int G>
__device__ __forceinline__ bool window_rsd_below(const float *win, int64_t E, int64_t z, int h, int fresh,
                                                 double th2, bool th_pos) {
  static_assert(NO % G == 0, "outputs come in whole groups");
  for (int o0 = 0; o0 < NO; o0 += G) {
    double y[G], s1[G], Q[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      y[g] = (double)win[((int64_t)fresh * NO + o0 + g) * E + z];
      s1[g] = 0.0;
      Q[g] = 0.0;
    }
    for (int q = 0; q < h; ++q) {
      if (q == fresh) continue;
      float wq[G];
#pragma unroll
      for (int g = 0; g < G; ++g) wq[g] = win[((int64_t)q * NO + o0 + g) * E + z];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const double d = (double)wq[g] - y[g];
        s1[g] += d;
        Q[g] = __builtin_fma(d, d, Q[g]);
      }
    }
    bool ok = true;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double D = (double)h * __builtin_fma((double)h, Q[g], -(s1[g] * s1[g]));
      const double sum = __builtin_fma((double)h, y[g], s1[g]);
      ok = ok && (D == 0.0 ? th_pos : D < (double)h * th2 * (sum * sum));
    }
    if (!ok) return false;
  }
  return true;
}

// Workgroups are dispatched to the 8 XCDs in turn (workgroup b to XCD b mod
// 8).  Renumbered this way, XCD x runs one contiguous stretch of the range,
// so neighbouring planes of the mesh, which share nodes, meet in the same L2.
// A bijection of [0, nb): XCD x takes nb/8 workgroups, one more if x < nb mod 8.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb) {
  const int64_t x = b & 7, j = b >> 3, q = nb >> 3, r = nb & 7;
  return x * q + (x < r ? x : r) + j;
}

__device__ __forceinline__ double block_min(double v, double *red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  return red[0];
}

// Doubles as unsigned integers of the same order, for integer atomics.
__device__ __forceinline__ unsigned long long ordered_key(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  return u >> 63 ? ~u : u | 0x8000000000000000ull;
}
__device__ __forceinline__ double key_value(unsigned long long k) {
  return __builtin_bit_cast(double, k >> 63 ? k ^ 0x8000000000000000ull : ~k);
}

}  // namespace

// ------------------------------------------------------------------ init

__global__ void __launch_bounds__(256) k_hydro_init_elem(HydroArgs a, double e_origin) {
  const int64_t z = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (z >= a.E) return;
  const int64_t n = a.n;
  const uint32_t t = a.dn.quo((uint32_t)z), kk = a.dn.quo(t);
  const int64_t i = z - (int64_t)t * n, j = (int64_t)t - (int64_t)kk * n, k = kk;
  float x[8][3], B[8][3];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    x[c][0] = a.h * (float)(i + (c & 1));
    x[c][1] = a.h * (float)(j + ((c >> 1) & 1));
    x[c][2] = a.h * (float)(k + ((c >> 2) & 1));
  }
  const float V = hex_volume<false>(x, B);
  const float rho0 = 1.0f;
  a.vol[z] = V;
  a.mass[z] = rho0 * V;
  const float e = z == 0 ? (float)e_origin : 0.0f;
  const float p = (a.gamma - 1.0f) * rho0 * e;
  a.e[z] = e;
  a.p[z] = p;
  a.q[z] = 0.0f;
  a.c[z] = sqrtf(a.gamma * fmaxf(p, 0.0f) / rho0);
}

__global__ void __launch_bounds__(256) k_hydro_init_node(HydroArgs a) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= a.Nn) return;
  const int n = a.n;
  const int64_t m = n + 1;
  const uint32_t t = a.dm.quo((uint32_t)v), kk = a.dm.quo(t);
  const int64_t i = v - (int64_t)t * m, j = (int64_t)t - (int64_t)kk * m, k = kk;
  a.x[0][v] = a.h * (float)i;
  a.x[1][v] = a.h * (float)j;
  a.x[2][v] = a.h * (float)k;
  float M = 0.0f;
  for (int c = 0; c < 8; ++c) {
    const int64_t ei = i - (c & 1), ej = j - ((c >> 1) & 1), ek = k - ((c >> 2) & 1);
    if (ei < 0 || ej < 0 || ek < 0 || ei >= n || ej >= n || ek >= n) continue;
    M += a.mass[ei + n * (ej + (int64_t)n * ek)] * 0.125f;
  }
  a.mnode[v] = M;
  for (int d = 0; d < 3; ++d) {
    a.u[d][v] = 0.0f;
    a.un[d][v] = 0.0f;
  }
}

// TAF decision-group state, over one entry per element (the largest grouping)
__global__ void __launch_bounds__(256) k_hydro_init_groups(HydroArgs a, double dt0) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g == 0) {
    a.clock[0] = 0.0;
    a.clock[1] = dt0;
    *a.status = 0;
  }
  if (g >= a.E) return;
  if (a.rho_eos) a.rho_eos[g] = 0, a.z_eos[g] = 0;
  if (a.rho_hg) a.rho_hg[g] = 0, a.z_hg[g] = 0;
}

// ------------------------------------------------------------------ force

// Corner forces (p + q) B + f of one element, f = NULL for none.
__device__ __forceinline__ void store_forces(float *force, int64_t E, const ElemIdx &ei, float pq,
                                             const float (&B)[8][3], const float (*f)[3]) {
  Planes<float> plane{force};
#pragma unroll
  for (int c = 0; c < 8; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d)
      at(plane.next(E), ei.z) = f ? __builtin_fmaf(pq, B[c][d], f[c][d]) : pq * B[c][d];
}

// Volume rate sum B . u (B sums to zero, so relative to corner 0).
__device__ __forceinline__ float volume_rate(const float (&B)[8][3], const float (&u)[8][3]) {
  float vdot = 0.0f;
#pragma unroll
  for (int c = 1; c < 8; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) vdot = __builtin_fmaf(B[c][d], u[c][d] - u[0][d], vdot);
  return vdot;
}

// The element's time-step bound in FP64.
__device__ __forceinline__ double time_bound(const HydroArgs &a, float V, float mass, float pq, float vdot) {
  const double Vd = (double)V, rd = (double)mass / Vd;
  const double ceff2 = a.gamma_d * fmax((double)pq, 0.0) / rd;
  double b = ceff2 > 0.0 ? a.cfl * cbrt(Vd) / sqrt(ceff2) : INFINITY;
  if (vdot != 0.0f) b = fmin(b, a.dvmax * Vd / fabs((double)vdot));
  return b;
}

template <int HG>
__global__ void __launch_bounds__(256) k_hydro_force(HydroArgs a) {
  __shared__ double red[256];
  const int64_t E = a.E;
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);  // element block: the block-level group
  const int64_t l = blk * blockDim.x + threadIdx.x;
  const int lane = lane_id();
  constexpr bool kTaf = HG == kHgTafWave || HG == kHgTafThread || HG == kHgTafBlock;
  __shared__ int tally[3];  // block level: active elements, votes to approximate, waves that voted
  if (HG == kHgTafBlock) {
    if (threadIdx.x < 3) tally[threadIdx.x] = 0;
    __syncthreads();
  }
  double bound = INFINITY;
  for (int k = 0; k < a.hg_ipt; ++k) {
    const int64_t z = l + (int64_t)k * a.hg_L;
    const bool active = z < E;
    const int64_t w = l >> 6;  // TAF: one element per lane
    bool compute_hg = HG != kHgNone;
    int rho = 0, pushes = 0;
    if (HG == kHgPerfo) {
      const int M = a.perfo_param;
      if (M > 0) {
        switch (a.perfo_kind) {
          case 0: compute_hg = (int)(((int64_t)k + a.step) % M) != M - 1; break;
          case 1: compute_hg = (int)(((int64_t)k + a.step) % M) == 0; break;
          case 2: compute_hg = z >= (int64_t)M * E / 100; break;
          default: compute_hg = z < E - (int64_t)M * E / 100; break;
        }
      }
    }
    if (HG == kHgTafWave && w < a.W) {
      rho = a.rho_hg[w];
      pushes = a.z_hg[w];
      compute_hg = rho <= 0;
    }
    if (HG == kHgTafThread && active) {
      rho = a.rho_hg[z];
      pushes = a.z_hg[z];
      compute_hg = rho <= 0;
    }
    if (HG == kHgTafBlock) {
      rho = a.rho_hg[blk];
      pushes = a.z_hg[blk];
      compute_hg = rho <= 0;
    }
    bool crit = false, voted = false;
    if (active) {
      const ElemIdx ei(z, a.dn);
      float x[8][3], u[8][3], B[8][3];
      // every load before the first store: a store could alias a later load,
      // which would then wait for a memory latency of its own
      gather3(a.x, ei, x);
      gather3(a.u, ei, u);
      const float pq = at(a.p, ei.z) + at(a.q, ei.z), mass = at(a.mass, ei.z), cs = at(a.c, ei.z);
      const float V = hex_volume<true>(x, B);
      at(a.vol, ei.z) = V;
      if (!(V > 0.0f)) atomicOr(a.status, kHydroBadVolume);  // tangled (or NaN) element
      const float vdot = volume_rate(B, u);
      if (compute_hg) {
        float f[8][3];
        hourglass(x, u, B, V, mass / V, cs, a.khg, f);
        store_forces(a.force, E, ei, pq, B, f);
        if (kTaf) {  // push the accurate forces
          const int slot = pushes % a.hg_h;
#pragma unroll
          for (int o = 0; o < 24; ++o) a.whg[((int64_t)slot * 24 + o) * E + z] = f[o / 3][o % 3];
        }
      } else if (kTaf) {
        // TAF's approximate path: the newest window slot holds the last
        // accurate forces (a countdown is only set after a push)
        const int slot = (pushes - 1) % a.hg_h;
        float f[8][3];
#pragma unroll
        for (int o = 0; o < 24; ++o) f[o / 3][o % 3] = a.whg[((int64_t)slot * 24 + o) * E + z];
        store_forces(a.force, E, ei, pq, B, f);
      } else {
        store_forces(a.force, E, ei, pq, B, nullptr);  // perforated: no hourglass force
      }
      bound = fmin(bound, time_bound(a, V, mass, pq, vdot));
      if (kTaf && compute_hg && pushes + 1 >= a.hg_h) {  // the window is full: vote
        voted = true;
        const double th = (double)a.hg_theta;
        crit = window_rsd_below<24, 8>(a.whg, E, z, a.hg_h, pushes % a.hg_h, th * th, th > 0.0);
      }
    }
    if (HG == kHgTafThread && active) {
      if (!compute_hg) {
        a.rho_hg[z] = rho - 1;
      } else {
        a.z_hg[z] = pushes + 1;
        if (crit) a.rho_hg[z] = a.hg_p;
      }
      if (a.dec_hg) a.dec_hg[z] = compute_hg ? 0 : 1;
    }
    if (HG == kHgTafWave && w < a.W) {
      const uint64_t amask = ballot(active);
      const uint64_t vmask = ballot(crit);
      const bool any_vote = ballot(voted) != 0;
      if (lane == 0) {
        if (!compute_hg) {
          a.rho_hg[w] = rho - 1;
        } else {
          a.z_hg[w] = pushes + 1;
          if (any_vote && majority(popc(vmask), popc(amask))) a.rho_hg[w] = a.hg_p;
        }
        if (a.dec_hg) a.dec_hg[w] = compute_hg ? 0 : 1;
      }
    }
    if (HG == kHgTafBlock) {  // every lane of the workgroup reaches the barrier
      const uint64_t amask = ballot(active);
      const uint64_t vmask = ballot(crit);
      const bool any_vote = ballot(voted) != 0;
      if (lane == 0 && compute_hg) {
        atomicAdd(&tally[0], popc(amask));
        atomicAdd(&tally[1], popc(vmask));
        if (any_vote) atomicAdd(&tally[2], 1);
      }
      __syncthreads();
      if (threadIdx.x == 0 && blk * blockDim.x < E) {
        if (!compute_hg) {
          a.rho_hg[blk] = rho - 1;
        } else {
          a.z_hg[blk] = pushes + 1;
          if (tally[2] > 0 && majority(tally[1], tally[0])) a.rho_hg[blk] = a.hg_p;
        }
        if (a.dec_hg) a.dec_hg[blk] = compute_hg ? 0 : 1;
      }
    }
  }
  const double m = block_min(bound, red);
  if (threadIdx.x == 0) a.dt_partials[blockIdx.x] = m;
}

// ------------------------------------------------------------------ dt

__global__ void __launch_bounds__(256) k_hydro_dt(HydroArgs a, int64_t parts, HydroLoop lp) {
  __shared__ double red[256];
  // sixteen independent loads per thread in flight at once: the partials
  // were just written by every XCD, so each round trip is a memory latency
  constexpr int kU = 16;
  double m = INFINITY;
  for (int64_t b0 = threadIdx.x; b0 < parts; b0 += (int64_t)blockDim.x * kU) {
    double v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t b = b0 + (int64_t)u * blockDim.x;
      v[u] = b < parts ? a.dt_partials[b] : INFINITY;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) m = fmin(m, v[u]);
  }
  m = block_min(m, red);
  // every partial has been read: their space becomes a loop's slots
  if ((int)threadIdx.x < lp.slots) lp.bounds_next[threadIdx.x] = ordered_key(INFINITY);
  if (threadIdx.x == 0) {
    const double dt = fmin(m, a.growth * a.clock[1]);
    if (!(dt > 0.0) || !isfinite(dt)) atomicOr(a.status, kHydroBadDt);
    a.clock[0] += dt;
    a.clock[1] = dt;
  }
}

// ------------------------------------------------------------------ nodes

// kLoop: within a loop of steps there is no time-step kernel before this one;
// every wave takes the minimum of the slots itself, and the first thread of
// the grid keeps the clock (nobody else reads what it writes).
template <bool kLoop>
__global__ void __launch_bounds__(256) k_hydro_node(HydroArgs a, HydroLoop lp) {
  const int64_t v = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
  unsigned long long key = ~0ull;
  double prev = 0.0;
  if (kLoop) {
    const int lane = lane_id();
    if (lane < lp.slots) key = lp.bounds[lane];
    prev = *lp.dt_prev;
  } else if (v >= a.Nn) {
    return;
  }
  const int n = a.n, m = n + 1;
  const int64_t E = a.E;
  const uint32_t t = a.dm.quo((uint32_t)v), kk = a.dm.quo(t);
  const int i = (int)((uint32_t)v - t * m), j = (int)(t - kk * m), k = (int)kk;
  // every load is issued at once, a corner outside the mesh reading the element
  // next to it instead (a load per branch would wait for eight latencies in turn)
  float f[8][3], u0[3], x0[3];
  bool in[8];
  uint32_t zx[2], zy[2], zz[2];  // byte offsets of the two adjacent elements of each direction
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    auto clip = [&](int q) { return (uint32_t)(q < 0 ? 0 : q < n ? q : n - 1); };
    zx[s] = 4 * clip(i - s);
    zy[s] = 4 * clip(j - s) * (uint32_t)n;
    zz[s] = 4 * clip(k - s) * (uint32_t)n * (uint32_t)n;
  }
  Planes<const float> plane{a.force};
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int ei = i - (c & 1), ej = j - ((c >> 1) & 1), ek = k - ((c >> 2) & 1);
    in[c] = ei >= 0 && ej >= 0 && ek >= 0 && ei < n && ej < n && ek < n;  // a thread past the last node has k > n
    const uint32_t z = zx[c & 1] + zy[(c >> 1) & 1] + zz[(c >> 2) & 1];
#pragma unroll
    for (int d = 0; d < 3; ++d) f[c][d] = at(plane.next(E), z);
  }
  const uint32_t vl = 4 * (uint32_t)(v < a.Nn ? v : a.Nn - 1);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    u0[d] = at(a.u[d], vl);
    x0[d] = at(a.x[d], vl);
  }
  const float mn = at(a.mnode, vl);
  double dtd;
  if (kLoop) {
#pragma unroll
    for (int m2 = 1; m2 < 64; m2 <<= 1) {
      const unsigned long long o = __shfl_xor(key, m2, 64);
      key = o < key ? o : key;
    }
    dtd = fmin(key_value(key), a.growth * prev);
    if (blockIdx.x == 0) {
      if ((int)threadIdx.x < lp.slots) lp.bounds_next[threadIdx.x] = ordered_key(INFINITY);
      if (threadIdx.x == 0) {
        if (!(dtd > 0.0) || !isfinite(dtd)) atomicOr(a.status, kHydroBadDt);
        a.clock[0] += dtd;
        *lp.dt = dtd;
      }
    }
    if (v >= a.Nn) return;
  } else {
    dtd = a.clock[1];
  }
  const float dt = (float)dtd;
  const float inv_m = 1.0f / mn;
  float F[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int c = 0; c < 8; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) F[d] += in[c] ? f[c][d] : 0.0f;
  const int idx[3] = {i, j, k};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    float u1 = __builtin_fmaf(dt, F[d] * inv_m, u0[d]);
    if (idx[d] == 0) u1 = 0.0f;
    at(a.un[d], vl) = u1;
    at(a.x[d], vl) = __builtin_fmaf(dt, 0.5f * (u0[d] + u1), x0[d]);
  }
}

// ------------------------------------------------------------------ EOS

// NEXT (within a loop of steps): the next step's forces, kHgExact or kHgNone,
// follow in the same kernel.  Both sides are functions of the element's new
// positions and velocities, so the gathers, the volume and its gradient are
// formed once, and pressure, viscosity and sound speed stay in registers; the
// next step's time-step bound goes to one of lp.slots minima by an integer
// atomic.  kNoNext: the EOS alone.  A step on 90^3 elements takes 47.5 us
// (30.2 this kernel, 16.6 the nodes: 186 and 109 MB counted, 6.2 and 6.6 TB/s)
// against 61 in four launches, one on 24^3 with EOS TAF 11.1 against 17.  With
// EOS TAF at 90^3 this kernel takes 35.0 us at thread level, 28.8 at wave level.
// Registers for three waves per SIMD, four where there are no hourglass
// forces; with what the compiler takes by itself (172, two waves) EOS TAF at
// 90^3 measured 12% slower.
template <int EOS, int NEXT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NEXT == kNoNext || NEXT == kHgNone ? 4 : 3))) k_hydro_eos(HydroArgs a, HydroLoop lp) {
  constexpr bool kTaf = EOS != kEosExact, kFused = NEXT != kNoNext;
  static_assert(!kFused || EOS != kEosTafBlock, "block level steps one kernel at a time");
  const int64_t E = a.E;
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);  // element block: the block-level group
  const int64_t z = blk * blockDim.x + threadIdx.x;
  const int64_t w = z >> 6;
  // whole waves past the last element leave, except where every lane of the
  // workgroup must reach barriers
  if (EOS != kEosTafBlock && !kFused && w >= a.W) return;
  const int lane = lane_id();
  const bool active = z < E;
  // the end of a loop: the last step's time step goes where single steps keep it
  if (!kFused && z == 0 && lp.dt != &a.clock[1]) a.clock[1] = *lp.dt;
  bool approx = false;  // the element keeps its EOS outputs
  int pushes = 0;
  __shared__ int tally[3];  // block level: active elements, votes to approximate, waves that voted
  if (EOS == kEosTafBlock) {
    const int rho = a.rho_eos[blk];
    if (rho > 0) {  // the same for the whole workgroup
      if (threadIdx.x == 0) {
        a.rho_eos[blk] = rho - 1;
        if (a.dec_eos) a.dec_eos[blk] = 1;
      }
      return;
    }
    pushes = a.z_eos[blk];
    if (threadIdx.x < 3) tally[threadIdx.x] = 0;
    __syncthreads();
  }
  if (EOS == kEosTafWave && (!kFused || w < a.W)) {
    const int rho = a.rho_eos[w];
    if (rho > 0) {
      if (lane == 0) {
        a.rho_eos[w] = rho - 1;
        if (a.dec_eos) a.dec_eos[w] = 1;
      }
      approx = true;
      if (!kFused) return;
    }
    pushes = a.z_eos[w];
  }
  if (EOS == kEosTafThread) {
    if (!kFused && !active) return;
    if (active) {
      const int rho = a.rho_eos[z];
      if (rho > 0) {
        a.rho_eos[z] = rho - 1;
        if (a.dec_eos) a.dec_eos[z] = 1;
        approx = true;
        if (!kFused) return;
      }
      pushes = a.z_eos[z];
    }
  }
  bool crit = false, voted = false;
  double bound = INFINITY;
  if (active) {
    const ElemIdx ei(z, a.dn);
    float x[8][3], u1[8][3], B[8][3];
    // every load before the atomic and the stores, as in the force kernel
    gather3(a.x, ei, x);
    gather3(a.un, ei, u1);
    const float m = at(a.mass, ei.z);
    float p1 = 0.0f, q1 = 0.0f, c1 = 0.0f;
    if (kFused && approx) {
      p1 = at(a.p, ei.z);
      q1 = at(a.q, ei.z);
      c1 = at(a.c, ei.z);
    }
    float V1;
    if (!kTaf || !approx) {
      float u0[8][3];
      gather3(a.u, ei, u0);
      const float dt = (float)*lp.dt, e0 = at(a.e, ei.z), c0 = at(a.c, ei.z);
      float W = 0.0f;
      Planes<const float> plane{a.force};
#pragma unroll
      for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int d = 0; d < 3; ++d) W = __builtin_fmaf(at(plane.next(E), ei.z), 0.5f * (u0[c][d] + u1[c][d]), W);
      // the work, the volume and its rate one after the other: interleaved, they
      // hold more in registers at once and measured 1.4% slower per step
      __builtin_amdgcn_sched_barrier(0);
      V1 = hex_volume<true>(x, B);
      if (!(V1 > 0.0f)) atomicOr(a.status, kHydroBadVolume);
      __builtin_amdgcn_sched_barrier(0);
      // volume rate sum B . u (B sums to zero, so relative to corner 0)
      float vdot = 0.0f;
#pragma unroll
      for (int c = 1; c < 8; ++c)
#pragma unroll
        for (int d = 0; d < 3; ++d)
          vdot = __builtin_fmaf(B[c][d], 0.5f * (u0[c][d] + u1[c][d]) - 0.5f * (u0[0][d] + u1[0][d]), vdot);
      const float e1 = e0 - dt * W / m;
      const float rho1 = m / V1;
      const float cv = cbrtf(V1);
      const float du = vdot / (cv * cv);
      q1 = du < 0.0f ? rho1 * (a.cq * du * du + a.cl * c0 * fabsf(du)) : 0.0f;
      p1 = (a.gamma - 1.0f) * rho1 * e1;
      c1 = sqrtf(a.gamma * fmaxf(p1, 0.0f) / rho1);
      at(a.e, ei.z) = e1;
      if (!kFused || kTaf) {  // else the loop's last EOS writes them
        at(a.p, ei.z) = p1;
        at(a.q, ei.z) = q1;
      }
      at(a.c, ei.z) = c1;
      if (kTaf) {
        const int slot = pushes % a.eos_h;
        const float y[4] = {e1, p1, q1, c1};
#pragma unroll
        for (int o = 0; o < 4; ++o) a.weos[((int64_t)slot * 4 + o) * E + z] = y[o];
        if (pushes + 1 >= a.eos_h) {
          voted = true;
          const double th = (double)a.eos_theta;
          crit = window_rsd_below<4, 4>(a.weos, E, z, a.eos_h, slot, th * th, th > 0.0);
        }
      }
    } else {
      V1 = hex_volume<true>(x, B);
      if (!(V1 > 0.0f)) atomicOr(a.status, kHydroBadVolume);
    }
    if (kFused) {
      if (lp.store_vol) at(a.vol, ei.z) = V1;
      const float pq = p1 + q1;
      const float vdot = volume_rate(B, u1);
      if (NEXT == kHgExact) {
        float f[8][3];
        hourglass(x, u1, B, V1, m / V1, c1, a.khg, f);
        store_forces(a.force, E, ei, pq, B, f);
      } else {
        store_forces(a.force, E, ei, pq, B, nullptr);
      }
      bound = fmin(bound, time_bound(a, V1, m, pq, vdot));
    }
  }
  if (EOS == kEosTafThread && active && !approx) {
    a.z_eos[z] = pushes + 1;
    if (crit) a.rho_eos[z] = a.eos_p;
    if (a.dec_eos) a.dec_eos[z] = 0;
  }
  if (EOS == kEosTafWave && !approx) {
    const uint64_t amask = ballot(active);
    const uint64_t vmask = ballot(crit);
    const bool any_vote = ballot(voted) != 0;
    if (lane == 0 && w < a.W) {
      a.z_eos[w] = pushes + 1;
      if (any_vote && majority(popc(vmask), popc(amask))) a.rho_eos[w] = a.eos_p;
      if (a.dec_eos) a.dec_eos[w] = 0;
    }
  }
  if (EOS == kEosTafBlock) {
    const uint64_t amask = ballot(active);
    const uint64_t vmask = ballot(crit);
    const bool any_vote = ballot(voted) != 0;
    if (lane == 0) {
      atomicAdd(&tally[0], popc(amask));
      atomicAdd(&tally[1], popc(vmask));
      if (any_vote) atomicAdd(&tally[2], 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      a.z_eos[blk] = pushes + 1;
      if (tally[2] > 0 && majority(tally[1], tally[0])) a.rho_eos[blk] = a.eos_p;
      if (a.dec_eos) a.dec_eos[blk] = 0;
    }
  }
  if (kFused) {
    __shared__ double mins[4];
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) bound = fmin(bound, __shfl_xor(bound, s, 64));
    // every lane holds its wave's minimum; a workgroup of one wave fills all slots
    if (lane < (blockDim.x == 64 ? 4 : 1)) mins[(threadIdx.x >> 6) + lane] = bound;
    __syncthreads();
    if (threadIdx.x == 0)
      atomicMin(&lp.bounds[blockIdx.x % lp.slots], ordered_key(fmin(fmin(mins[0], mins[1]), fmin(mins[2], mins[3]))));
  }
}

// --------------------------------------------------------------- launchers

int64_t hydro_lanes(int64_t E, int ipt) { return 64 * (((E + ipt - 1) / ipt + 63) / 64); }

int64_t hydro_partials(int64_t E) { return (hydro_lanes(E, 1) + 255) / 256; }

// Partial time-step minima of the allocation-free step: one double per
// workgroup of the force kernel, held in a file-scope device array rather
// than a caller buffer.  Every GPU the library runs on holds its own copy,
// at its own address, until the process ends.  In host code `scratch` names
// a host-side stand-in, never passed to a kernel: its device address is
// looked up once per device, with that device current, and kept.
static __device__ __align__(256) double scratch[kHydroScratchPartials];

hipError_t hydro_scratch(hipStream_t stream, double **ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static double *addr[kMaxDevices] = {};
  int cur = 0, dev = 0;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  dev = cur;
  if (stream && (e = hipStreamGetDevice(stream, &dev)) != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    if (dev != cur && (e = hipSetDevice(dev)) != hipSuccess) return e;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (dev != cur) {
      const hipError_t r = hipSetDevice(cur);
      if (e == hipSuccess) e = r;
    }
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = (double *)p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_hydro_init(const HydroArgs &a, double e_origin, double dt0, hipStream_t s) {
  hipLaunchKernelGGL(k_hydro_init_elem, dim3((unsigned)((a.E + 255) / 256)), dim3(256), 0, s, a, e_origin);
  hipLaunchKernelGGL(k_hydro_init_node, dim3((unsigned)((a.Nn + 255) / 256)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_hydro_init_groups, dim3((unsigned)((a.E + 255) / 256)), dim3(256), 0, s, a, dt0);
  return hipGetLastError();
}

// The force mode of step a.step: with one item per lane the herded rule keeps
// or drops the whole step.
static int step_hg_mode(const HydroArgs &a, int hg_mode) {
  if (hg_mode == kHgPerfo && a.hg_ipt == 1 && a.perfo_param > 0 && (a.perfo_kind == 0 || a.perfo_kind == 1)) {
    const int r = (int)((int64_t)a.step % a.perfo_param);
    const bool keep = a.perfo_kind == 0 ? r != a.perfo_param - 1 : r == 0;
    return keep ? kHgExact : kHgNone;
  }
  return hg_mode;
}

static void go_force(const HydroArgs &a, int hg_mode, unsigned blocks, hipStream_t s) {
  switch (hg_mode) {
    case kHgExact: hipLaunchKernelGGL(k_hydro_force<kHgExact>, dim3(blocks), dim3(256), 0, s, a); break;
    case kHgTafWave: hipLaunchKernelGGL(k_hydro_force<kHgTafWave>, dim3(blocks), dim3(256), 0, s, a); break;
    case kHgTafThread: hipLaunchKernelGGL(k_hydro_force<kHgTafThread>, dim3(blocks), dim3(256), 0, s, a); break;
    case kHgTafBlock: hipLaunchKernelGGL(k_hydro_force<kHgTafBlock>, dim3(blocks), dim3(256), 0, s, a); break;
    case kHgNone: hipLaunchKernelGGL(k_hydro_force<kHgNone>, dim3(blocks), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL(k_hydro_force<kHgPerfo>, dim3(blocks), dim3(256), 0, s, a); break;
  }
}

// Meshes of at most one wave per CU take a workgroup per wave, so that no two
// waves share a CU's load path while others idle (EOS with the next forces:
// 16^3 elements 6.3 -> 5.8 us, 24^3 6.45 -> 6.15); larger ones keep four waves
// per workgroup, whose minimum is one atomic instead of four (40^3 7.25 us
// against 8.6, 90^3 30 against 40).
constexpr int64_t kSmallMesh = 256 * 64;
static unsigned mesh_block(const HydroArgs &a) { return a.E <= kSmallMesh ? 64 : 256; }

template <int NEXT>
static void go_eos(const HydroArgs &a, const HydroLoop &lp, int eos_mode, hipStream_t s) {
  const unsigned block = eos_mode == kEosTafBlock ? 256 : mesh_block(a);
  const dim3 g((unsigned)((hydro_lanes(a.E, 1) + block - 1) / block)), b(block);
  switch (eos_mode) {
    case kEosExact: hipLaunchKernelGGL((k_hydro_eos<kEosExact, NEXT>), g, b, 0, s, a, lp); break;
    case kEosTafWave: hipLaunchKernelGGL((k_hydro_eos<kEosTafWave, NEXT>), g, b, 0, s, a, lp); break;
    case kEosTafThread: hipLaunchKernelGGL((k_hydro_eos<kEosTafThread, NEXT>), g, b, 0, s, a, lp); break;
    default:
      if constexpr (NEXT == kNoNext) hipLaunchKernelGGL((k_hydro_eos<kEosTafBlock, NEXT>), g, b, 0, s, a, lp);
      break;
  }
}

hipError_t launch_hydro_step(const HydroArgs &a, int hg_mode, int eos_mode, hipStream_t s) {
  const unsigned fblocks = (unsigned)((a.hg_L + 255) / 256), nblocks = (unsigned)((a.Nn + mesh_block(a) - 1) / mesh_block(a));
  HydroLoop lp = {};
  lp.dt = &a.clock[1];
  go_force(a, step_hg_mode(a, hg_mode), fblocks, s);
  hipLaunchKernelGGL(k_hydro_dt, dim3(1), dim3(256), 0, s, a, (int64_t)fblocks, lp);
  hipLaunchKernelGGL(k_hydro_node<false>, dim3(nblocks), dim3(mesh_block(a)), 0, s, a, lp);
  go_eos<kNoNext>(a, lp, eos_mode, s);
  return hipGetLastError();
}

// A loop of steps.  Where the EOS and the next step's forces can share a
// kernel (no hourglass TAF, no perforation within a step, EOS decisions of a
// thread or wave), a step is two launches instead of four: the node kernel,
// which also forms the time step, and the EOS with the next step's forces.
// The time-step bounds live in the caller's partial array: two sets of `slots`
// minima, used by steps in turn (the node kernel that reads one clears the
// other), and the time steps of odd steps; even ones are in clock[1].
// Same values as single steps.
hipError_t launch_hydro_run(HydroArgs a, int hg_mode, int eos_mode, int steps, hipStream_t s) {
  const int64_t parts = hydro_partials(a.E);
  const bool whole = hg_mode == kHgExact || step_hg_mode(a, hg_mode) != kHgPerfo;
  const bool fused = steps > 1 && parts >= 3 && eos_mode != kEosTafBlock && whole && hg_mode != kHgTafWave &&
                     hg_mode != kHgTafThread && hg_mode != kHgTafBlock;
  auto swap_u = [&] {  // the new velocities are the next step's old ones
    for (int d = 0; d < 3; ++d) {
      float *t = a.u[d];
      a.u[d] = a.un[d];
      a.un[d] = t;
    }
  };
  if (!fused) {
    for (int k = 0; k < steps; ++k) {
      const hipError_t e = launch_hydro_step(a, hg_mode, eos_mode, s);
      if (e != hipSuccess) return e;
      a.step += 1;
      swap_u();
    }
    return hipSuccess;
  }
  const unsigned fblocks = (unsigned)((a.hg_L + 255) / 256), nblocks = (unsigned)((a.Nn + mesh_block(a) - 1) / mesh_block(a));
  const int slots = (int)((parts - 1) / 2 < 64 ? (parts - 1) / 2 : 64);
  unsigned long long *const set[2] = {(unsigned long long *)a.dt_partials, (unsigned long long *)a.dt_partials + slots};
  double *const cell[2] = {&a.clock[1], a.dt_partials + 2 * slots};
  HydroLoop lp = {};
  lp.slots = slots;
  lp.dt = cell[0];
  lp.bounds_next = set[1];
  go_force(a, step_hg_mode(a, hg_mode), fblocks, s);
  hipLaunchKernelGGL(k_hydro_dt, dim3(1), dim3(256), 0, s, a, (int64_t)fblocks, lp);
  hipLaunchKernelGGL(k_hydro_node<false>, dim3(nblocks), dim3(mesh_block(a)), 0, s, a, lp);
  for (int k = 0; k + 1 < steps; ++k) {
    // step k's EOS and step k + 1's forces
    lp.dt = cell[k & 1];
    lp.bounds = set[(k + 1) & 1];
    lp.store_vol = k + 2 == steps;
    a.step += 1;
    if (step_hg_mode(a, hg_mode) == kHgNone)
      go_eos<kHgNone>(a, lp, eos_mode, s);
    else
      go_eos<kHgExact>(a, lp, eos_mode, s);
    swap_u();
    // step k + 1's nodes
    lp.dt_prev = cell[k & 1];
    lp.dt = cell[(k + 1) & 1];
    lp.bounds_next = set[k & 1];
    hipLaunchKernelGGL(k_hydro_node<true>, dim3(nblocks), dim3(mesh_block(a)), 0, s, a, lp);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  go_eos<kNoNext>(a, lp, eos_mode, s);
  return hipGetLastError();
}

}  // namespace hpac
