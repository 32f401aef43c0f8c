// Softmax statistics of logit rows for the entropy of the commitment
// schedule (Symbol Commitment Schedules, item 3: H = -sum p log p over the
// predicted distribution), in one fixed partition shared by the LM head's
// epilogue and the standalone statistics kernel, so both give the same bits.
//
// A row of V logits is cut into groups of 128 columns.  The statistics of a
// group are its max m first, then Z and A as binary-tree sums over its columns
// in order ((c0 + c1) + (c2 + c3), ...), which one thread can evaluate from a
// staged tile and 32 lanes of a wave from coalesced loads, with the same bits.
// A row's groups are merged by one wave: lane l folds groups l, l + 64, ... in
// order, then the wave merges with butterflies over lane distances 1 .. 32.
//
// Statistics of a set of logits relative to its max m: Z = sum e^(l - m),
// A = sum e^(l - m) (l - m); then H (nats) = ln Z - A / Z.  Columns past V
// and -inf logits carry nothing.  A NaN logit makes its group's Z and A NaN, and
// with them the row's entropy, also in a group with nothing above -inf.
#pragma once

#include "common.h"

namespace dlmc {

struct RowStat {
  float m, Z, A;
};

constexpr int STAT_GROUP = 128;  // columns per group

__host__ __device__ constexpr int stat_groups(int V) { return (V + STAT_GROUP - 1) / STAT_GROUP; }

// e^t for t <= 0 on the hardware 2^x (a few ulps of fp32)
__device__ __forceinline__ float stat_exp(float t) {
  return __builtin_amdgcn_exp2f(t * 1.4426950408889634f);
}

__device__ __forceinline__ RowStat stat_merge(RowStat x, RowStat y) {
  if (y.Z == 0.0f) return x;
  if (x.Z == 0.0f) return y;
  const float m = fmaxf(x.m, y.m);
  const float cx = stat_exp(x.m - m), cy = stat_exp(y.m - m);
  RowStat r;
  r.m = m;
  r.Z = cx * x.Z + cy * y.Z;
  r.A = cx * (x.A + (x.m - m) * x.Z) + cy * (y.A + (y.m - m) * y.Z);
  return r;
}

// Z and A of four columns relative to the group's max m: the two lowest levels
// of the tree.  A -inf logit contributes 0 to both (its t is made finite, so that
// 0 t is 0); a NaN logit makes e, and with it both sums, NaN.
__device__ __forceinline__ void stat_quad(f32x4 v, float m, float& z, float& a) {
  float e[4], w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float t = v[i] - m;
    e[i] = stat_exp(t);
    w[i] = e[i] * fmaxf(t, -3.0e38f);
  }
  z = (e[0] + e[1]) + (e[2] + e[3]);
  a = (w[0] + w[1]) + (w[2] + w[3]);
}

// NaN if one of four columns is, else 0
__device__ __forceinline__ float stat_quad_nan(f32x4 v) {
  const bool nan = v.x != v.x || v.y != v.y || v.z != v.z || v.w != v.w;
  return nan ? __builtin_nanf("") : 0.0f;
}

// N quads of a group, evaluated depth first, so that few partial sums are live
template <int N, typename Quad>
__device__ __forceinline__ void stat_tree(const Quad& quad, int q0, float m, float& z, float& a) {
  if constexpr (N == 1) {
    stat_quad(quad(q0), m, z, a);
  } else {
    float z1, a1;
    stat_tree<N / 2>(quad, q0, m, z, a);
    stat_tree<N / 2>(quad, q0 + N / 2, m, z1, a1);
    z += z1;
    a += a1;
  }
}

// The statistics of the n <= 128 logits p[0 .. n) of one group by one thread, in
// LDS, 16-byte aligned and with room for a whole group: the columns past n are
// overwritten with -inf, so that one straight tree serves every n.  (With a
// second tree of conditional loads for a row's last group the LM head's kernel
// spilled 108 registers: 65536 x 32768 x 768 took 4513 us without statistics and
// 5319 with them, against 4343 and 5024.)
__device__ __forceinline__ RowStat group_stat(float* p, int n) {
#pragma unroll 1
  for (int c = n; c < STAT_GROUP; ++c) p[c] = -INFINITY;
  auto quad = [&](int q) { return *reinterpret_cast<const f32x4*>(p + 4 * q); };
  float m = -INFINITY;
#pragma unroll 8
  for (int q = 0; q < STAT_GROUP / 4; ++q) {
    const f32x4 v = quad(q);
    m = fmaxf(m, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
  }
  RowStat s{m, 0.0f, 0.0f};
  if (m != -INFINITY) {
    stat_tree<STAT_GROUP / 4>(quad, 0, m, s.Z, s.A);
  } else {  // the max passes over NaN: an empty group, unless it holds one
#pragma unroll 1
    for (int q = 0; q < STAT_GROUP / 4; ++q) s.Z = s.A = s.Z + stat_quad_nan(quad(q));
  }
  return s;
}

// Lane i's value of lane i ^ 1, i ^ 2, 7 - i (within 8 lanes) or 15 - i (within 16)
// by a DPP move: a few cycles, where a shuffle goes through the LDS.
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
#else
  return x;
#endif
}
// Reduction over each half of a wave (32 lanes), the binary tree over lane
// distances 1, 2, 4, 8, 16: after two levels the lanes of a quad agree, so the
// mirrors pair quads, then groups of eight, as distances 4 and 8 would.
template <typename Op>
__device__ __forceinline__ float half_wave_reduce(float x, Op op) {
  x = op(x, dpp_move<DPP_XOR1>(x));
  x = op(x, dpp_move<DPP_XOR2>(x));
  x = op(x, dpp_move<DPP_HALF_MIRROR>(x));
  x = op(x, dpp_move<DPP_MIRROR>(x));
  return op(x, __shfl_xor(x, 16));
}

// The same by the 32 lanes of half a wave: lane i (0 .. 31) holds columns 4 i ..
// 4 i + 3 (-inf past the row's end); every lane returns the group's statistics.
__device__ __forceinline__ RowStat group_stat_lanes(f32x4 v) {
  RowStat s{fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)), 0.0f, 0.0f};
  s.m = half_wave_reduce(s.m, [](float x, float y) { return fmaxf(x, y); });
  stat_quad(v, s.m, s.Z, s.A);
  s.Z = half_wave_reduce(s.Z, [](float x, float y) { return x + y; });
  s.A = half_wave_reduce(s.A, [](float x, float y) { return x + y; });
  if (!(s.m > -INFINITY)) {  // nothing above -inf: an empty group, unless it holds a NaN
    s.m = -INFINITY;
    s.Z = s.A = half_wave_reduce(stat_quad_nan(v), [](float x, float y) { return x + y; });
  }
  return s;
}

// merge over lanes at xor distances 1 .. W/2
template <int W>
__device__ __forceinline__ RowStat stat_butterfly(RowStat s) {
#pragma unroll
  for (int o = 1; o < W; o <<= 1) {
    RowStat t{__shfl_xor(s.m, o), __shfl_xor(s.Z, o), __shfl_xor(s.A, o)};
    s = stat_merge(s, t);
  }
  return s;
}

// entropy in bits of a merged row statistic
__device__ __forceinline__ float stat_entropy_bits(RowStat r) {
  return (logf(r.Z) - r.A / r.Z) * 1.4426950408889634f;
}

}  // namespace dlmc
