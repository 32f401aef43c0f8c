// Attention-based initial context (Initial Context Strategies, item 4):
// head-averaged attention maps of the extra forward passes and the Attention
// Rollout (Abnar and Zuidema, 2020) flow into the masked positions.
//
// attention_map: A[i, j] = (1 / H) sum_h softmax_j(scale q_h,i . k_h,j), heads in
//   ascending order, from Q, K and the row maxima and sums attention leaves.
// rollout: v <- (A_l^T v + v) / 2 from the last layer to the first.
#include "kernels.h"

namespace dlmc {
namespace {

constexpr int MT = 64;  // a block's tile of a map: 64 queries x 64 keys

// A wave computes S^T = K Q^T for 32 queries x 32 keys of one head after the
// other, so a lane holds 16 keys of one query and needs one (max, sum) pair per
// head; the probabilities stay in registers until the last head and a map is
// written once.  Fragments come straight from global memory (a row is read by
// one lane pair, L1 and L2 serve the other waves), the next head's while this
// one's are multiplied: that latency, H times, bounds short chunks.
//
// One product and one softmax launch per head with the scores in between took
// 12.8 us a head at T = 1024 (12 heads of dim 64): 154 us a layer, against 14.7.
template <int DH>
__global__ void __launch_bounds__(256)
attention_map_bf16_kernel(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
                          const float2* __restrict__ ml, float* __restrict__ A, int H, int T, int Tp,
                          int ld, float scale_log2, float w) {
  constexpr int NS = DH / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, lg = lane >> 5;
  const int q0 = blockIdx.y * MT + (wave >> 1) * 32, k0 = blockIdx.x * MT + (wave & 1) * 32;
  const int q = q0 + lr;
  // Tp is a multiple of 128: rows at or beyond T are inside the buffers, finite,
  // and not stored (queries) or stored as 0 (keys)
  const bf16_t* qp = Q + (size_t)q * DH + lg * 8;
  const bf16_t* kp = K + (size_t)(k0 + lr) * DH + lg * 8;
  const float2* mp = ml + min(q, T - 1);
  const size_t hs = (size_t)Tp * DH;
  bf16x8 qf[2][NS], kf[2][NS];
  float2 st[2];
  f32x16 a;
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.0f;
  auto load = [&](int h, bf16x8(&qd)[NS], bf16x8(&kd)[NS], float2& sd) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      qd[s] = *reinterpret_cast<const bf16x8*>(qp + h * hs + s * 16);
      kd[s] = *reinterpret_cast<const bf16x8*>(kp + h * hs + s * 16);
    }
    sd = mp[(size_t)h * Tp];
  };
  auto head = [&](const bf16x8(&qd)[NS], const bf16x8(&kd)[NS], float2 sd) {
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
    for (int i = 0; i < NS; ++i) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kd[i], qd[i], s, 0, 0, 0);
    const float n = w / sd.y;
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] += __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2, -sd.x)) * n;
  };
  load(0, qf[0], kf[0], st[0]);
  for (int h = 0; h < H; h += 2) {
    if (h + 1 < H) load(h + 1, qf[1], kf[1], st[1]);
    head(qf[0], kf[0], st[0]);
    if (h + 2 < H) load(h + 2, qf[0], kf[0], st[0]);
    if (h + 1 < H) head(qf[1], kf[1], st[1]);
  }
  // register r: key 8 (r / 4) + 4 lg + r % 4 of the wave's 32; ld is a multiple of MT
  if (q < T)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int k = k0 + 8 * g + 4 * lg;
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = k + e < T ? a[4 * g + e] : 0.0f;
      *reinterpret_cast<f32x4*>(A + (size_t)q * ld + k) = v;
    }
}

// fp32: the same on v_mfma_f32_16x16x4_f32, a wave on 16 queries x 64 keys (a
// lane holds keys 4 g + r of each group of 16, g = lane / 16; step e of a
// 16-dim group takes dims 4 g + e, as in attention).
template <int DH>
__global__ void __launch_bounds__(256)
attention_map_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                         const float2* __restrict__ ml, float* __restrict__ A, int H, int T, int Tp,
                         int ld, float scale, float w) {
  constexpr int ND = DH / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lg = lane >> 4;
  const int q = blockIdx.y * MT + wave * 16 + lr, k0 = blockIdx.x * MT;
  const float* qp = Q + (size_t)q * DH + lg * 4;
  const float* kp = K + (size_t)(k0 + lr) * DH + lg * 4;
  const size_t hs = (size_t)Tp * DH;
  f32x4 a[MT / 16];
#pragma unroll
  for (int t = 0; t < MT / 16; ++t) a[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  for (int h = 0; h < H; ++h) {
    const float2 sd = ml[(size_t)h * Tp + min(q, T - 1)];
    f32x4 s[MT / 16];
#pragma unroll
    for (int t = 0; t < MT / 16; ++t) s[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const f32x4 qf = *reinterpret_cast<const f32x4*>(qp + h * hs + 16 * i);
      f32x4 kf[MT / 16];
#pragma unroll
      for (int t = 0; t < MT / 16; ++t)
        kf[t] = *reinterpret_cast<const f32x4*>(kp + h * hs + (size_t)(16 * t) * DH + 16 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < MT / 16; ++t)
          s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][e], qf[e], s[t], 0, 0, 0);
    }
    const float n = w / sd.y;
#pragma unroll
    for (int t = 0; t < MT / 16; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) a[t][r] += expf(s[t][r] * scale - sd.x) * n;
  }
  if (q < T)
#pragma unroll
    for (int t = 0; t < MT / 16; ++t) {
      const int k = k0 + 16 * t + 4 * lg;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e >= T) a[t][e] = 0.0f;
      *reinterpret_cast<f32x4*>(A + (size_t)q * ld + k) = a[t];
    }
}

// One rollout step in partial sums: vectors are kept as `n` rows of pitch ld
// whose column sums, in row order, are the vector.  Block (x, y) takes R rows
// of A from y R on and 256 columns from 256 x on, and writes row y of the
// result: half the rows' product, plus half of v where its columns are its own
// rows.  Rows are split because a thread per column with all of A's rows in a
// chain, T / 256 blocks in all, took 269 us at T = 1024, against 5.7.
constexpr int RC = 256;

__global__ void __launch_bounds__(256)
rollout_step_kernel(const float* __restrict__ A, const float* __restrict__ in, int n_in,
                    float* __restrict__ out, int T, int ld, int R) {
  __shared__ float vs[256];
  __shared__ float part[256];
  __shared__ f32x4 red[4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r0 = blockIdx.y * R, c = blockIdx.x * RC + lane * 4;
  // v of this block's rows: 256 / R threads a row (R is a power of two, 16 .. 128)
  {
    const int row = tid & (R - 1), r = r0 + row;
    float s = 0.0f;
    if (r < T)
      for (int p = tid / R; p < n_in; p += 256 / R) s += in[(size_t)p * ld + r];
    part[tid] = s;
    __syncthreads();
    if (tid < R) {
      float t = part[tid];
      for (int p = 1; p < 256 / R; ++p) t += part[tid + p * R];
      vs[tid] = t;
    }
    __syncthreads();
  }
  f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  if (c < ld) {
    const int per = R / 4, i0 = wave * per, n = min(per, T - r0 - i0);
#pragma unroll 8
    for (int i = 0; i < n; ++i) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(A + (size_t)(r0 + i0 + i) * ld + c);
      const float v = vs[i0 + i];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += v * x[e];
    }
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && c < ld) {
    f32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      y[e] = 0.5f * ((red[0][lane][e] + red[1][lane][e]) + (red[2][lane][e] + red[3][lane][e]));
      const int j = c + e - r0;
      if (j >= 0 && j < R) y[e] += 0.5f * vs[j];
    }
    *reinterpret_cast<f32x4*>(out + (size_t)blockIdx.y * ld + c) = y;
  }
}

__global__ void __launch_bounds__(256)
rollout_sum_kernel(const float* __restrict__ in, int n_in, float* __restrict__ out, int T, int ld) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= T) return;
  float s = 0.0f;
#pragma unroll 8
  for (int p = 0; p < n_in; ++p) s += in[(size_t)p * ld + j];
  out[j] = s;
}

// rows of A per block: at most ROLLOUT_PARTS partial rows, so that reading them
// stays well below reading A (R x 256 floats a block against n_in x R)
int rollout_rows(int T) {
  int R = 16;
  while (ceil_div(T, R) > ROLLOUT_PARTS) R *= 2;
  return R;
}

}  // namespace

void attention_map(hipStream_t st, const void* q, const void* k, const float2* ml, float* A, bool bf16,
                   int H, int T, int Tp, int dh, int ld) {
  if (T <= 0 || H <= 0) return;
  DLMC_CHECK(ld % MT == 0 && ld >= T && Tp % 128 == 0 && Tp >= T, DLMC_E_INVAL, "attention map: bad pitch");
  const dim3 grid(ceil_div(T, MT), ceil_div(T, MT)), block(256);
  const float scale = 1.0f / sqrtf((float)dh), w = 1.0f / (float)H;
  auto run = [&](auto kernel, auto* qq, auto* kk, float s) {
    kernel<<<grid, block, 0, st>>>(qq, kk, ml, A, H, T, Tp, ld, s, w);
    DLMC_HIP(hipGetLastError());
  };
  if (bf16) {
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)dh);  // the units of attention's maxima
    DLMC_CHECK(dh == 64 || dh == 128, DLMC_E_INVAL, "bf16 attention supports head dims 64 and 128");
    run(dh == 64 ? attention_map_bf16_kernel<64> : attention_map_bf16_kernel<128>, (const bf16_t*)q,
        (const bf16_t*)k, scale_log2);
    return;
  }
  const float *qf = (const float*)q, *kf = (const float*)k;
  switch (dh) {
    case 16: run(attention_map_f32_kernel<16>, qf, kf, scale); break;
    case 32: run(attention_map_f32_kernel<32>, qf, kf, scale); break;
    case 64: run(attention_map_f32_kernel<64>, qf, kf, scale); break;
    case 128: run(attention_map_f32_kernel<128>, qf, kf, scale); break;
    default: throw Error(DLMC_E_INVAL, "fp32 attention supports head dims 16, 32, 64, 128");
  }
}

void rollout(hipStream_t st, const float* maps, int L, const float* v, float* ws, float* out, int T,
             int ld) {
  if (T <= 0) return;
  DLMC_CHECK(ld % MT == 0 && ld >= T, DLMC_E_INVAL, "rollout: bad pitch");
  const int R = rollout_rows(T), parts = ceil_div(T, R);
  const float* in = v;
  int n_in = 1;
  float* dst = ws;
  for (int l = L - 1; l >= 0; --l) {
    rollout_step_kernel<<<dim3(ceil_div(ld, RC), parts), 256, 0, st>>>(maps + (size_t)l * T * ld, in, n_in,
                                                                      dst, T, ld, R);
    DLMC_HIP(hipGetLastError());
    in = dst;
    n_in = parts;
    dst = dst == ws ? ws + (size_t)ROLLOUT_PARTS * ld : ws;
  }
  rollout_sum_kernel<<<ceil_div(T, 256), 256, 0, st>>>(in, n_in, out, T, ld);
  DLMC_HIP(hipGetLastError());
}

}  // namespace dlmc
