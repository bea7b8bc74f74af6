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
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));  // at any float

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

// Out-of-box items are staged per wave in LDS (index and inputs).  The exact
// region prices them 64 at a time with every lane busy, from the inputs the
// wave has already read and while the lines around their outputs are still in
// the L2 (a second kernel over the queue read and wrote most of the columns'
// lines again: 77 us at 2^24 items, 5% of them out of the box; all of a wave's
// at its end, 12 us).  Their indices are appended to the global queue when
// the stage is full and, by the whole workgroup, at the end: every append is
// an atomic on one counter, 7.6 ns each, and one per wave at the end cost 30
// us on a full chip.
constexpr int kQueueStage = 256;
struct OutOfBox {
  int32_t index[kQueueStage];
  float x[5][kQueueStage];
};

__device__ __forceinline__ void out_of_box_price(const MlpArgs &a, const OutOfBox &st, int from, int count, int lane) {
  for (int q = from + lane; q < count; q += 64) {
    const int32_t i = st.index[q];
    float x[5], y[2];
#pragma unroll
    for (int j = 0; j < 5; ++j) x[j] = st.x[j][q];
    RegionBSPrice::eval(x, y);
    a.out[0][i] = y[0];
    a.out[1][i] = y[1];
  }
}

__device__ __forceinline__ void out_of_box_list(const MlpArgs &a, const OutOfBox &st, int count, int base, int lane) {
  for (int q = lane; q < count; q += 64) a.queue[base + q] = st.index[q];
}

// Persistent: each wave walks chunks of TILES 16-item tiles (chunk = wave id +
// k * waves in the grid).  The first two layers' weights stay in registers,
// the biases and the last layer's weights are read from LDS where a tile
// starts, as accumulators and operands: that keeps the kernel within the
// registers of four waves per SIMD.
//
// Bound by VALU issue: the 128 GELUs per item take about 35 clocks each per
// wave, 16 of them the two transcendentals, which hold the SIMD (480 of the
// 677 us at 2^24 items); the MFMAs are nearly hidden (22 us less without them),
// and three or five waves per SIMD measured 18 and 9 us more.  2^24 items, 5%
// out of the box: 766 us with every weight and bias in registers and a second
// pass for the out-of-box items, 677 us here; 250,000 items 54 -> 22 us.
template <int TILES>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) k_mlp_infer(MlpArgs a) {
  constexpr int kItems = 16 * TILES;
  // per wave: the BF16 normalised inputs of its items in the B-operand
  // layout of layer 1 (slots 5..7 zero), and a zero row 64 for lane groups
  // 1..3; the network's normalised outputs; the staged out-of-box items
  struct Wave {
    bf16x8 xs[65];
    float ys[64][2];
    OutOfBox oob;
  };
  __shared__ Wave wave[4];
  __shared__ int32_t left[4], queue_base;
  __shared__ bf16x8 w3s[2][64];             // last layer's weights in operand layout
  __shared__ floatx4 b1s[16], b2s[16], b3s[4];  // biases by accumulator row groups of four
  const int lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // chunk numbers and column bases in scalar registers
  const int g = lane >> 4, r = lane & 15;
  Wave &wv = wave[w];

  const int64_t chunks = (a.n + kItems - 1) / kItems;
  const int64_t waves = (int64_t)gridDim.x * 4;
  // inputs of the wave's next chunk, loaded one chunk ahead
  float xn[5];
  auto load = [&](int64_t first) {  // the columns of the chunk that starts at item `first`
    const bool have = lane < kItems && lane < a.n - first;
#pragma unroll
    for (int j = 0; j < 5; ++j) xn[j] = have ? (a.in[j] + first)[lane] : 0.0f;
  };
  load(((int64_t)blockIdx.x * 4 + w) * kItems);
  // weights in MFMA A layout (lane holds row r of a 16-row tile, reduction
  // slots 8g..8g+7), rounded to BF16; every load is issued before the first
  // conversion, so the prologue waits for one memory latency
  float w1[4][5];
  float4u w2[4][2][2], w3[2], bv;
#pragma unroll
  for (int tm = 0; tm < 4; ++tm)
#pragma unroll
    for (int j = 0; j < 5; ++j) w1[tm][j] = a.params[(16 * tm + r) * 5 + j];
#pragma unroll
  for (int tm = 0; tm < 4; ++tm)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        w2[tm][c][h] = *(const float4u *)&a.params[kOffW2 + (16 * tm + r) * kNH + kperm(c, g, 4 * h)];
#pragma unroll
  for (int h = 0; h < 2; ++h) w3[h] = *(const float4u *)&a.params[kOffW3 + (r & 1) * kNH + kperm(w & 1, g, 4 * h)];
  bv = *(const float4u *)&a.params[(lane < 16 ? kOffB1 : kOffB2) + 4 * r];
  const float b30 = a.params[kOffB3], b31 = a.params[kOffB3 + 1];
  bf16x8 W1[4], W2[4][2];
#pragma unroll
  for (int tm = 0; tm < 4; ++tm)
#pragma unroll
    for (int j = 0; j < 8; ++j) W1[tm][j] = (__bf16)(g == 0 && j < 5 ? w1[tm][j < 5 ? j : 0] : 0.0f);
#pragma unroll
  for (int tm = 0; tm < 4; ++tm)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int j = 0; j < 8; ++j) W2[tm][c][j] = (__bf16)w2[tm][c][j >> 2][j & 3];
  if (w < 2) {
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (__bf16)(r < 2 ? w3[j >> 2][j & 3] : 0.0f);
    w3s[w][lane] = v;
  } else if (w == 2 && lane < 32) {
    (lane < 16 ? b1s[r] : b2s[r]) = floatx4{bv[0], bv[1], bv[2], bv[3]};
  } else if (w == 3 && lane < 4) {
    b3s[lane] = lane == 0 ? floatx4{b30, b31, 0.0f, 0.0f} : floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  __syncthreads();

  if (lane == 0) {
    bf16x8 z;
#pragma unroll
    for (int j = 0; j < 8; ++j) z[j] = (__bf16)0.0f;
    wv.xs[64] = z;
  }
  int staged = 0, priced = 0;  // wave-uniform
#pragma unroll 1
  for (int64_t ch = (int64_t)blockIdx.x * 4 + w; ch < chunks; ch += waves) {
    const int64_t first = ch * kItems;
    const bool active = lane < kItems && lane < a.n - first;
    // box test, then the loads of the next chunk go out while this one computes
    float x[5];
    bool inside = active;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      x[j] = xn[j];
      inside = inside && x[j] >= a.box_lo[j] && x[j] <= a.box_hi[j];
    }
    if (ch + waves < chunks) load(first + waves * kItems);  // wave-uniform
    const uint64_t out_mask = ballot(active && !inside);
    // the previous chunk's LDS reads are done before anything is rewritten
    wave_lds_fence();
    if (out_mask) {
      const int cnt = popc(out_mask);
      if (staged + cnt > kQueueStage) {
        int base = 0;
        if (lane == 0) base = atomicAdd(a.queue_count, staged);
        out_of_box_price(a, wv.oob, priced, staged, lane);
        out_of_box_list(a, wv.oob, staged, __builtin_amdgcn_readfirstlane(base), lane);
        staged = priced = 0;
        wave_lds_fence();
      }
      if (active && !inside) {
        const int q = staged + popc(out_mask & ((1ull << lane) - 1));
        wv.oob.index[q] = (int32_t)first + lane;
#pragma unroll
        for (int j = 0; j < 5; ++j) wv.oob.x[j][q] = x[j];
      }
      staged += cnt;
      if (staged - priced >= 64) {
        wave_lds_fence();
        out_of_box_price(a, wv.oob, priced, priced + 64, lane);
        priced += 64;
      }
    }
    {
      bf16x8 v;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = (__bf16)(j < 5 ? (x[j < 5 ? j : 0] - a.in_center[j < 5 ? j : 0]) * a.in_scale[j < 5 ? j : 0] : 0.0f);
      wv.xs[lane] = v;
    }
    wave_lds_fence();

#pragma unroll 1
    for (int tn = 0; tn < TILES; ++tn) {
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
  // the rest of the staged items: one atomic for the workgroup, in flight while
  // the waves price theirs
  if (lane == 0) left[w] = staged;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    before += q < w ? left[q] : 0;
    total += left[q];
  }
  if (total == 0) return;
  if (threadIdx.x == 0) queue_base = atomicAdd(a.queue_count, total);
  out_of_box_price(a, wv.oob, priced, staged, lane);
  __syncthreads();
  out_of_box_list(a, wv.oob, staged, queue_base + before, lane);
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
// waves per workgroup, 11.2 us here.
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
  const int64_t i0 = (int64_t)blockIdx.x * kNH;
  // every load of the workgroup in flight at once
  constexpr int kLoads = (kNumParams + 64 * kGradWaves - 1) / (64 * kGradWaves);
  float pv[kLoads], iv = 0.0f;
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    const int p = T + 64 * kGradWaves * q;
    pv[q] = a.params[p < kNumParams ? p : kNumParams - 1];
  }
  const int row = w, t = lane;  // waves 0..4 input `row` of item t, waves 8 and 9 target row - 8
  const bool have = i0 + t < a.n;
  if (have && (row < 5 || row == 8 || row == 9)) iv = (row < 5 ? a.x[row] : a.t[row - 8])[i0 + t];
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    const int p = T + 64 * kGradWaves * q;
    const float v = pv[q], vr = round_bf16(v);
    if (p < kOffB1) W1[p / 5 * 9 + p % 5] = vr;
    else if (p < kOffW2) W1[(p - kOffB1) * 9 + 5] = v;
    else if (p < kOffB2) W2[((p - kOffW2) >> 6) * kLd + ((p - kOffW2) & 63)] = vr;
    else if (p < kOffW3) B2[p - kOffB2] = v;
    else if (p < kOffB3) W3[p - kOffW3] = vr;
    else if (p < kNumParams) B3[p - kOffB3] = v;
  }
  if (row < 8) {
    xs[row * kNH + t] = row < 5 ? (have ? (iv - a.in_center[row]) * a.in_scale[row] : 0.0f) : row == 5 ? 1.0f : 0.0f;
    if (row >= 6) W1[t * 9 + row] = 0.0f;
  } else if (row < 10) {
    const int o = row - 8;
    ths[o * kNH + t] = have ? (target_map(a, o, iv) - a.out_mean[o]) / a.out_scale[o] : 0.0f;
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

template <int TILES>
static hipError_t infer_go(const MlpArgs &a, int64_t resident, hipStream_t stream) {
  const int64_t want = (a.n + 64 * TILES - 1) / (64 * TILES);
  hipLaunchKernelGGL(k_mlp_infer<TILES>, dim3((unsigned)(want < resident ? want : resident)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_mlp_infer(const MlpArgs &a, hipStream_t stream) {
  // one resident wave per SIMD slot the kernel's register use allows; a batch
  // of at most one workgroup per CU is resident whatever that is
  int dev = 0, cus = 0, per_cu = 1;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (cus < 1) cus = 1;
  if (e == hipSuccess && a.n > (int64_t)cus * 256)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_infer<4>, 256, 0);
  if (e != hipSuccess) return e;
  const int64_t resident = (int64_t)cus * (per_cu > 0 ? per_cu : 1);
  hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, stream, a.queue_count);
  // one tile per wave while that is at most one workgroup per CU: four tiles in
  // a row are then latency no other wave hides (12,000 items: 8.8 us against
  // 10.0); beyond, the workgroups' prologues cost more (60,000: 18.2 against 12.0)
  return a.n <= (int64_t)cus * 64 ? infer_go<1>(a, resident, stream) : infer_go<4>(a, resident, stream);
}

// A dispatch's grid size is a 32-bit count of lanes: with 1024 of them per 64
// items, larger batches (from 2^28 items, whose partials are 81 GB) take
// several launches.
constexpr int64_t kGradBlocks = 0xFFFFFFFFll / (64 * kGradWaves);

hipError_t launch_mlp_grad(const MlpGradArgs &a, hipStream_t stream) {
  for (int64_t b0 = 0; b0 * kNH < a.n; b0 += kGradBlocks) {
    MlpGradArgs part = a;
    part.n = a.n - b0 * kNH < kGradBlocks * kNH ? a.n - b0 * kNH : kGradBlocks * kNH;
    for (int j = 0; j < 5; ++j) part.x[j] += b0 * kNH;
    for (int o = 0; o < 2; ++o) part.t[o] += b0 * kNH;
    part.grad_partials += b0 * kNumParams;
    part.loss_partials += b0;
    hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)((part.n + kNH - 1) / kNH)), dim3(64 * kGradWaves), 0, stream, part);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_mlp_adam(const AdamArgs &a, hipStream_t stream) {
  hipLaunchKernelGGL(k_mlp_adam, dim3((kNumParams + 63) / 64), dim3(64 * kAdamWaves), 0, stream, a);
  return hipGetLastError();
}

}  // namespace hpac
