// MLP surrogate of the Black-Scholes region (5 -> 64 -> 64 -> 2, GELU in the
// tanh form), used as a further approximation technique: items inside the
// training box are priced by the network, the others by the exact region.
//
//  k_mlp_infer   BF16 MFMA inference with FP32 accumulation.  Every layer is
//                computed transposed (units x items), so the accumulator
//                layout of one layer is, after GELU and conversion, the B
//                operand of the next: the order of the reduction index inside
//                each 32-wide chunk is permuted, and the weights are loaded
//                in the same permuted order.  Items outside the box are
//                ballot-compacted per wave, listed in a queue and priced by
//                the exact region.
//  k_mlp_grad    training: forward (FP32 activations, BF16-rounded weights)
//                and backward for 64 items per workgroup, its products on
//                FP32 MFMA; weight-gradient partial sums per workgroup
//                (deterministic, no atomics).
//  k_mlp_adam    sums the partials and applies one Adam step to the FP32
//                master weights.
#include "launch_mlp.hpp"
#include "region_bs.hpp"
#include "wave.hpp"

namespace hpac {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kNH = 64;
constexpr int kOffB1 = 64 * 5, kOffW2 = kOffB1 + 64, kOffB2 = kOffW2 + 64 * 64, kOffW3 = kOffB2 + 64,
              kOffB3 = kOffW3 + 2 * 64, kNumParams = kOffB3 + 2;

// GELU, tanh form: x/2 (1 + tanh(u)) = x / (1 + exp(-2u)),
// u = sqrt(2/pi) (x + 0.044715 x^3); the exponent is formed in base 2.
constexpr float kGeluA = -2.0f * 0.797884560802865356f * 1.44269504088896341f;
constexpr float kGeluB = kGeluA * 0.044715f;
__device__ __forceinline__ float gelu(float x) {
  const float t = x * __builtin_fmaf(x * x, kGeluB, kGeluA);
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}
// the same and its derivative s + x s (1 - s) (-t'), s = 1/(1 + e^{t}), t' = dt/dx
__device__ __forceinline__ float gelu_both(float x, float &d) {
  const float x2 = x * x;
  const float t = x * __builtin_fmaf(x2, kGeluB, kGeluA);
  const float s = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
  const float dt = __builtin_fmaf(3.0f * kGeluB, x2, kGeluA) * 0.693147180559945309f;
  d = s - x * s * (1.0f - s) * dt;
  return x * s;
}

__device__ __forceinline__ float round_bf16(float v) { return (float)(__bf16)v; }

// Output o of the network's normalised output yh: the affine map back, then
// exp(v) - shift where the network models log(y + shift).
__device__ __forceinline__ float out_map(const MlpArgs &a, int o, float yh) {
  const float v = __builtin_fmaf(yh, a.out_scale[o], a.out_mean[o]);
  return a.out_shift[o] > 0.0f ? expf(v) - a.out_shift[o] : v;
}

// Training target o in the network's output space.
__device__ __forceinline__ float target_map(const MlpGradArgs &a, int o, float t) {
  return a.out_shift[o] > 0.0f ? logf(t + a.out_shift[o]) : t;
}

// ------------------------------------------------------------------ infer

// permuted position of reduction slot (lane group g, slot j) in chunk c:
// the accumulator rows a lane holds in the two 16-unit tiles of the chunk
__device__ __forceinline__ int kperm(int c, int g, int j) { return 32 * c + (j < 4 ? 4 * g + j : 16 + 4 * g + j - 4); }

// Out-of-box items are staged per wave in LDS (index and inputs) and dealt with
// kQueueStage at a time: their indices are appended to the global queue with
// one atomic per flush, not one per 64 items (a single counter hit by every
// wave serialises them), and the exact region prices them with every lane
// busy, from the inputs the wave has already read (a second kernel over the
// queue read and wrote most of the columns' lines again: 77 us at 2^24 items,
// 5% of them out of the box).
constexpr int kQueueStage = 256;
struct OutOfBox {
  int32_t index[kQueueStage];
  float x[5][kQueueStage];
};

__device__ __forceinline__ void out_of_box_flush(const MlpArgs &a, const OutOfBox &st, int count, int lane) {
  int base = 0;
  if (lane == 0) base = atomicAdd(a.queue_count, count);
  base = __builtin_amdgcn_readfirstlane(base);
  for (int q = lane; q < count; q += 64) {
    const int32_t i = st.index[q];
    a.queue[base + q] = i;
    float x[5], y[2];
#pragma unroll
    for (int j = 0; j < 5; ++j) x[j] = st.x[j][q];
    RegionBSPrice::eval(x, y);
    a.out[0][i] = y[0];
    a.out[1][i] = y[1];
  }
}

// Persistent: each wave walks 64-item chunks (chunk = wave id + k * waves in
// the grid).  The parameters are fetched once per workgroup, coalesced, into
// LDS and from there into MFMA operand layout; the first two layers' weights
// stay in registers, the biases and the last layer's weights are read from
// LDS where a tile starts, as accumulators and operands: that keeps the kernel
// within the registers of WAVES waves per SIMD.
//
// Bound by VALU issue: the 128 GELUs per item take about 35 clocks each per
// wave, 16 of them the two transcendentals, which hold the SIMD (480 of the
// 680 us at 2^24 items); the MFMAs are nearly hidden (659 us without them),
// and three or five waves per SIMD measured 699 and 690 us.  2^24 items, 5%
// out of the box: 766 us with every weight and bias in registers and a
// second pass for the out-of-box items, 680 us here.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) k_mlp_infer(MlpArgs a) {
  // per wave: the BF16 normalised inputs of its 64 items in the B-operand
  // layout of layer 1 (slots 5..7 zero), and a zero row 64 for lane groups
  // 1..3; the network's normalised outputs; the staged out-of-box items
  struct Wave {
    bf16x8 xs[65];
    float ys[64][2];
    OutOfBox oob;
  };
  __shared__ union {
    float params[kNumParams];  // before the loop
    Wave wave[4];
  } sh;
  __shared__ bf16x8 w3s[2][64];             // last layer's weights in operand layout
  __shared__ floatx4 b1s[16], b2s[16], b3s[4];  // biases by accumulator row groups of four
  const int lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // chunk numbers and column bases in scalar registers
  const int g = lane >> 4, r = lane & 15;
  Wave &wv = sh.wave[w];

  for (int p = threadIdx.x; p < kNumParams; p += 256) sh.params[p] = a.params[p];
  const int64_t chunks = (a.n + 63) >> 6;
  const int64_t waves = (int64_t)gridDim.x * 4;
  // inputs of the wave's next chunk, loaded one chunk ahead
  float xn[5];
  auto load = [&](int64_t first) {  // the columns of the chunk that starts at item `first`
    const bool have = lane < a.n - first;
#pragma unroll
    for (int j = 0; j < 5; ++j) xn[j] = have ? (a.in[j] + first)[lane] : 0.0f;
  };
  load(((int64_t)blockIdx.x * 4 + w) * 64);
  __syncthreads();
  // weights in MFMA A layout (lane holds row r of a 16-row tile, reduction
  // slots 8g..8g+7), rounded to BF16
  bf16x8 W1[4], W2[4][2];
#pragma unroll
  for (int tm = 0; tm < 4; ++tm)
#pragma unroll
    for (int j = 0; j < 8; ++j) W1[tm][j] = (__bf16)(g == 0 && j < 5 ? sh.params[(16 * tm + r) * 5 + j] : 0.0f);
#pragma unroll
  for (int tm = 0; tm < 4; ++tm)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int j = 0; j < 8; ++j) W2[tm][c][j] = (__bf16)sh.params[kOffW2 + (16 * tm + r) * kNH + kperm(c, g, j)];
  if (w < 2) {
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (__bf16)(r < 2 ? sh.params[kOffW3 + r * kNH + kperm(w, g, j)] : 0.0f);
    w3s[w][lane] = v;
  } else if (lane < 36) {
    const int q = lane & 15;
    floatx4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      v[j] = lane < 32 ? sh.params[(lane < 16 ? kOffB1 : kOffB2) + 4 * q + j]
                       : (lane == 32 && j < 2 ? sh.params[kOffB3 + j] : 0.0f);
    if (w == 2) (lane < 16 ? b1s[q] : lane < 32 ? b2s[q] : b3s[lane - 32]) = v;
  }
  __syncthreads();  // the parameters' space becomes the waves' own

  if (lane == 0) {
    bf16x8 z;
#pragma unroll
    for (int j = 0; j < 8; ++j) z[j] = (__bf16)0.0f;
    wv.xs[64] = z;
  }
  int staged = 0;  // wave-uniform
#pragma unroll 1
  for (int64_t ch = (int64_t)blockIdx.x * 4 + w; ch < chunks; ch += waves) {
    const int64_t first = ch * 64;
    const bool active = lane < a.n - first;
    // box test, then the loads of the next chunk go out while this one computes
    float x[5];
    bool inside = active;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      x[j] = xn[j];
      inside = inside && x[j] >= a.box_lo[j] && x[j] <= a.box_hi[j];
    }
    if (ch + waves < chunks) load(first + waves * 64);  // wave-uniform
    const uint64_t out_mask = ballot(active && !inside);
    // the previous chunk's LDS reads are done before anything is rewritten
    wave_lds_fence();
    if (out_mask) {
      const int cnt = popc(out_mask);
      if (staged + cnt > kQueueStage) {
        out_of_box_flush(a, wv.oob, staged, lane);
        staged = 0;
        wave_lds_fence();
      }
      if (active && !inside) {
        const int q = staged + popc(out_mask & ((1ull << lane) - 1));
        wv.oob.index[q] = (int32_t)first + lane;
#pragma unroll
        for (int j = 0; j < 5; ++j) wv.oob.x[j][q] = x[j];
      }
      staged += cnt;
    }
    {
      bf16x8 v;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = (__bf16)(j < 5 ? (x[j < 5 ? j : 0] - a.in_center[j < 5 ? j : 0]) * a.in_scale[j < 5 ? j : 0] : 0.0f);
      wv.xs[lane] = v;
    }
    wave_lds_fence();

#pragma unroll 1
    for (int tn = 0; tn < 4; ++tn) {
      // B operand of layer 1: inputs of item 16 tn + r in slots 0..7 of lane
      // group 0, zeros elsewhere
      const bf16x8 xb = wv.xs[g == 0 ? 16 * tn + r : 64];
      // opaque: the biases and the last layer's weights are read here, not
      // kept in registers across the loops
      int gt = g, lt = lane;
      asm volatile("" : "+v"(gt), "+v"(lt));
      floatx4 D1[4];
#pragma unroll
      for (int tm = 0; tm < 4; ++tm)
        D1[tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W1[tm], xb, b1s[4 * tm + gt], 0, 0, 0);
      // GELU, BF16, and the permuted B operand of layer 2: chunk c, slot j
      bf16x8 h1[2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int j = 0; j < 8; ++j) h1[c][j] = (__bf16)gelu(D1[2 * c + (j >> 2)][j & 3]);
      floatx4 D2[4];
#pragma unroll
      for (int tm = 0; tm < 4; ++tm) {
        D2[tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W2[tm][0], h1[0], b2s[4 * tm + gt], 0, 0, 0);
        D2[tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W2[tm][1], h1[1], D2[tm], 0, 0, 0);
      }
      bf16x8 h2[2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int j = 0; j < 8; ++j) h2[c][j] = (__bf16)gelu(D2[2 * c + (j >> 2)][j & 3]);
      floatx4 D3 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w3s[0][lt], h2[0], b3s[gt], 0, 0, 0);
      D3 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w3s[1][lt], h2[1], D3, 0, 0, 0);
      // rows 0 and 1 (the two outputs) live in lanes 0..15, slots 0 and 1
      if (g == 0) {
        wv.ys[16 * tn + r][0] = D3[0];
        wv.ys[16 * tn + r][1] = D3[1];
      }
    }
    wave_lds_fence();
    if (active && inside) {
      // the output map once per item, each lane on its own item
      (a.out[0] + first)[lane] = out_map(a, 0, wv.ys[lane][0]);
      (a.out[1] + first)[lane] = out_map(a, 1, wv.ys[lane][1]);
    }
  }
  if (staged > 0) {
    wave_lds_fence();
    out_of_box_flush(a, wv.oob, staged, lane);
  }
}

__global__ void k_zero_int(int32_t *p) { *p = 0; }

// ------------------------------------------------------------------ train

// 64 items per workgroup of 16 waves.  The three 64 x 64 x 64 products (second
// layer forward, its backward, its weight gradient) and the thin ones run on
// v_mfma_f32_16x16x4_f32: FP32 operands, FP32 accumulation.  Wave w holds
// tile (w / 4, w % 4) of each 64 x 64 result, so every GELU is evaluated once,
// by the lane whose accumulator holds its argument, and with its derivative.
// Matrices lie in LDS with rows of 65 words: a row's columns and a column's
// rows are both read without bank conflicts (an operand is read along rows
// in one product and along columns in the next).
//
// Bound by latency: a batch of 8,192 items is 128 workgroups, one per CU on
// half the chip, going through six barriers; the matrix cores are busy about
// 3 us of it.  8,192 items: 31.9 us with scalar multiply-adds over four
// waves per workgroup, 12.2 us here.
constexpr int kLd = kNH + 1;
constexpr int kGradWaves = 16;

// a tile of A B, K = 64: A[row][k] = a[row * ars + k * aks], B[k][col] = b[k * bks + col * bcs]
__device__ __forceinline__ floatx4 tile_product(const float *a, int ars, int aks, const float *b, int bks, int bcs,
                                                floatx4 acc, int lane) {
  const int r = lane & 15, k0 = lane >> 4;
#pragma unroll
  for (int s = 0; s < kNH / 4; ++s) {
    const int k = 4 * s + k0;
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r * ars + k * aks], b[k * bks + r * bcs], acc, 0, 0, 0);
  }
  return acc;
}

__global__ void __launch_bounds__(64 * kGradWaves) k_mlp_grad(MlpGradArgs a) {
  // BF16-rounded weights, FP32 biases; the first layer's bias is the weight
  // of a sixth input that is always one
  __shared__ float W1[kNH * 9], W2[kNH * kLd], B2[kNH], W3[2 * kNH], B3[2];
  __shared__ float xs[8 * kNH];  // [input][item], rows 6 and 7 zero
  __shared__ float ths[2 * kNH], yparts[4 * 2 * kNH], dys[2 * kNH], errs[kNH];
  __shared__ float h1s[kNH * kLd], h2s[kNH * kLd], dz2s[kNH * kLd], dz1s[kNH * kLd];  // [unit][item]
  const int T = threadIdx.x, lane = lane_id();
  const int w = T >> 6, to = w >> 2, ti = w & 3;
  const int row0 = 16 * to + 4 * (lane >> 4), col = 16 * ti + (lane & 15);  // the lane's accumulator elements
  for (int p = T; p < kNumParams; p += 64 * kGradWaves) {
    const float v = a.params[p], vr = round_bf16(v);
    if (p < kOffB1) W1[p / 5 * 9 + p % 5] = vr;
    else if (p < kOffW2) W1[(p - kOffB1) * 9 + 5] = v;
    else if (p < kOffB2) W2[((p - kOffW2) >> 6) * kLd + ((p - kOffW2) & 63)] = vr;
    else if (p < kOffW3) B2[p - kOffB2] = v;
    else if (p < kOffB3) W3[p - kOffW3] = vr;
    else B3[p - kOffB3] = v;
  }
  const int64_t i0 = (int64_t)blockIdx.x * kNH;
  if (T < 8 * kNH) {  // input j of item t
    const int j = T >> 6, t = T & 63;
    const bool active = i0 + t < a.n;
    float v = j == 5 ? 1.0f : 0.0f;
    if (j < 5 && active) v = (a.x[j][i0 + t] - a.in_center[j]) * a.in_scale[j];
    xs[j * kNH + t] = v;
    if (j >= 6) W1[t * 9 + j] = 0.0f;
  } else if (T < 10 * kNH) {  // target o of item t
    const int o = (T >> 6) - 8, t = T & 63;
    ths[o * kNH + t] = i0 + t < a.n ? (target_map(a, o, a.t[o][i0 + t]) - a.out_mean[o]) / a.out_scale[o] : 0.0f;
  }
  __syncthreads();
  // layer 1
  float d1[4];
  {
    floatx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int k = 4 * s + (lane >> 4);
      z = __builtin_amdgcn_mfma_f32_16x16x4f32(W1[(16 * to + (lane & 15)) * 9 + k], xs[k * kNH + col], z, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) h1s[(row0 + i) * kLd + col] = gelu_both(z[i], d1[i]);
  }
  __syncthreads();
  // layer 2, and the tile's share of layer 3
  float d2[4];
  {
    floatx4 z;
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = B2[row0 + i];
    z = tile_product(W2 + 16 * to * kLd, kLd, 1, h1s + 16 * ti, kLd, 1, z, lane);
    float y0 = 0.0f, y1 = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float h = gelu_both(z[i], d2[i]);
      h2s[(row0 + i) * kLd + col] = h;
      y0 = __builtin_fmaf(W3[row0 + i], h, y0);
      y1 = __builtin_fmaf(W3[kNH + row0 + i], h, y1);
    }
#pragma unroll
    for (int m = 16; m < 64; m <<= 1) {
      y0 += __shfl_xor(y0, m, 64);
      y1 += __shfl_xor(y1, m, 64);
    }
    if (lane < 16) {
      yparts[(2 * to) * kNH + col] = y0;
      yparts[(2 * to + 1) * kNH + col] = y1;
    }
  }
  __syncthreads();
  // loss 1/(2N) sum (yh - th)^2 over the N training items and both outputs;
  // backward through layer 3 and the second GELU
  {
    float yh0 = B3[0], yh1 = B3[1];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      yh0 += yparts[2 * q * kNH + col];
      yh1 += yparts[(2 * q + 1) * kNH + col];
    }
    const bool active = i0 + col < a.n;
    const float e0 = active ? yh0 - ths[col] : 0.0f, e1 = active ? yh1 - ths[kNH + col] : 0.0f;
    const float dy0 = e0 * a.inv_count, dy1 = e1 * a.inv_count;
    if (to == 0 && lane < 16) {
      dys[col] = dy0;
      dys[kNH + col] = dy1;
      errs[col] = e0 * e0 + e1 * e1;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float dh = W3[row0 + i] * dy0 + W3[kNH + row0 + i] * dy1;
      dz2s[(row0 + i) * kLd + col] = dh * d2[i];
    }
  }
  __syncthreads();
  float *part = a.grad_partials + (int64_t)blockIdx.x * kNumParams;
  const floatx4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  // through layer 2 and the first GELU
  {
    const floatx4 dh = tile_product(W2 + 16 * to, 1, kLd, dz2s + 16 * ti, kLd, 1, zero, lane);
#pragma unroll
    for (int i = 0; i < 4; ++i) dz1s[(row0 + i) * kLd + col] = dh[i] * d1[i];
  }
  // the second layer's weights: tile (to, ti) of dz2 h1^T
  {
    const floatx4 g = tile_product(dz2s + 16 * to * kLd, kLd, 1, h1s + 16 * ti * kLd, 1, kLd, zero, lane);
#pragma unroll
    for (int i = 0; i < 4; ++i) part[kOffW2 + (row0 + i) * kNH + col] = g[i];
  }
  __syncthreads();
  // the thin gradients, 16 units per wave: columns of the second operand are
  // the inputs and the one (layer 1), the output errors (layer 3), ones (second bias)
  const int c = lane & 15, u0 = 16 * ti + 4 * (lane >> 4);
  if (to < 3) {
    const float *src = to == 0 ? dz1s : to == 1 ? h2s : dz2s;
    const float *rhs = to == 0 ? xs : dys;
    const int cols = to == 0 ? 8 : to == 1 ? 2 : 0;
    floatx4 g = zero;
#pragma unroll
    for (int s = 0; s < kNH / 4; ++s) {
      const int k = 4 * s + (lane >> 4);
      const float bv = to == 2 ? 1.0f : c < cols ? rhs[c * kNH + k] : 0.0f;
      g = __builtin_amdgcn_mfma_f32_16x16x4f32(src[(16 * ti + c) * kLd + k], bv, g, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = u0 + i;
      if (to == 0 && c < 5) part[u * 5 + c] = g[i];
      if (to == 0 && c == 5) part[kOffB1 + u] = g[i];
      if (to == 1 && c < 2) part[kOffW3 + c * kNH + u] = g[i];
      if (to == 2 && c == 0) part[kOffB2 + u] = g[i];
    }
  } else if (ti < 3) {  // the third bias and the loss
    float s = ti < 2 ? dys[ti * kNH + lane] : errs[lane];
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) s += __shfl_xor(s, m, 64);
    if (lane == 0) (ti < 2 ? part[kOffB3 + ti] : a.loss_partials[blockIdx.x]) = s;
  }
}

// One workgroup per 64 parameters: wave w sums every kAdamWaves-th partial,
// eight loads in flight, the waves' sums meet in LDS in wave order and the
// first wave applies the step.  Bound by memory latency: 128 partials
// (8,192 items) took 8.7 us summed by one thread per parameter, 3.2 us here.
constexpr int kAdamWaves = 16;
__global__ void __launch_bounds__(64 * kAdamWaves) k_mlp_adam(AdamArgs a) {
  __shared__ float sums[kAdamWaves][64];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + lane;
  constexpr int kU = 8;
  float g = 0.0f;
  if (p < kNumParams) {
    for (int64_t b0 = w; b0 < a.blocks; b0 += kU * kAdamWaves) {
      float v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t b = b0 + u * kAdamWaves;
        v[u] = b < a.blocks ? a.grad_partials[b * kNumParams + p] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) g += v[u];
    }
  }
  sums[w][lane] = g;
  __syncthreads();
  if (w != 0 || p >= kNumParams) return;
#pragma unroll
  for (int q = 1; q < kAdamWaves; ++q) g += sums[q][lane];
  const float m = a.beta1 * a.m[p] + (1.0f - a.beta1) * g;
  const float v = a.beta2 * a.v[p] + (1.0f - a.beta2) * g * g;
  a.m[p] = m;
  a.v[p] = v;
  const float mh = m / a.bc1, vh = v / a.bc2;
  a.params[p] -= a.lr * mh / (sqrtf(vh) + a.eps);
}

// --------------------------------------------------------------- launchers

int mlp_num_params() { return kNumParams; }

hipError_t launch_mlp_infer(const MlpArgs &a, hipStream_t stream) {
  // one resident wave per SIMD slot the kernel's register use allows
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_infer, 256, 0);
  if (e != hipSuccess) return e;
  const int64_t want = (a.n + 255) / 256;
  const int64_t resident = (int64_t)(cus > 0 ? cus : 1) * (per_cu > 0 ? per_cu : 1);
  const unsigned grid = (unsigned)(want < resident ? (want < 1 ? 1 : want) : resident);
  hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, stream, a.queue_count);
  hipLaunchKernelGGL(k_mlp_infer, dim3(grid), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpGradArgs &a, hipStream_t stream) {
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)((a.n + 63) / 64)), dim3(64 * kGradWaves), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(const AdamArgs &a, hipStream_t stream) {
  hipLaunchKernelGGL(k_mlp_adam, dim3((kNumParams + 63) / 64), dim3(64 * kAdamWaves), 0, stream, a);
  return hipGetLastError();
}

}  // namespace hpac
