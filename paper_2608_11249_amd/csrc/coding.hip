// Coding stages of one masked-diffusion step: masked-row compaction,
// per-position entropy, the entropy-based commitment schedule, integer CDF
// quantisation, the decoders' symbol search (decode) and the reveal of
// committed symbols.
//
// All reductions use fixed trees (wave butterflies, then wave totals in order)
// and the CDF is integer arithmetic after one expf per entry, so encode and
// decode compute bit-identical selections and CDFs.
#include <climits>

#include "kernels.h"
#include "rowstats.h"

namespace dlmc {
namespace {

// ---------------------------------------------------------------- compaction
// One block; positions are taken 65536 at a time, up to 1024 words of 64, split
// evenly over the 16 waves: a wave ballots its words from coalesced loads, 16 in
// flight, lane i keeping its i-th word's ballot, one block scan of the word
// counts gives every word its first output row, and the ballots in LDS place
// each row and the chunk boundaries without reading anything back.  65536
// positions: 18 us, bound by one CU's loads (75 with a barrier per 1024 positions
// and binary searches over the row list in memory); 4096: 4.7 us (7.6).
__global__ void __launch_bounds__(1024)
compact_kernel(const int32_t* __restrict__ state, int B, int T, int mask_id,
               int32_t* __restrict__ rows, int32_t* __restrict__ n_rows,
               int32_t* __restrict__ chunk_off, int32_t* __restrict__ chunk_cnt) {
  constexpr int WORDS = 1024, SPAN = WORDS * 64, LF = 16;
  __shared__ uint64_t word[WORDS];
  __shared__ int first[WORDS];
  __shared__ int wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int total = B * T;
  int carry = 0;
  for (int base = 0; base < total; base += SPAN) {
    const int span = min(SPAN, total - base);
    const int n_words = (span + 63) / 64, wpw = (n_words + 15) / 16;  // words in all, per wave (<= 64)
    const int w0 = wave * wpw;
    uint64_t mine = 0;
    for (int i0 = 0; i0 < wpw; i0 += LF) {
      int32_t v[LF];
#pragma unroll
      for (int i = 0; i < LF; ++i) v[i] = state[min(base + (w0 + i0 + i) * 64 + lane, total - 1)];
#pragma unroll
      for (int i = 0; i < LF; ++i) {
        const bool in = i0 + i < wpw && base + (w0 + i0 + i) * 64 + lane < total;
        const uint64_t bal = __ballot(in && v[i] == mask_id);
        mine = i0 + i == lane ? bal : mine;
      }
    }
    const int cnt = __popcll(mine);
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = carry, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      before += w < wave ? wsum[w] : 0;
      all += wsum[w];
    }
    if (lane < wpw && w0 + lane < WORDS) {
      word[w0 + lane] = mine;
      first[w0 + lane] = before + incl - cnt;
    }
    __syncthreads();
#pragma unroll 4
    for (int w = w0; w < min(w0 + wpw, n_words); ++w) {
      const uint64_t bal = word[w];
      if (bal >> lane & 1) rows[first[w] + __popcll(bal & ((1ull << lane) - 1ull))] = base + w * 64 + lane;
    }
    // first rows of the chunks that start in this span
    for (int b = (base + T - 1) / T + tid; b < B && b * T < base + span; b += 1024) {
      const int p = b * T - base;
      chunk_off[b] = first[p >> 6] + __popcll(word[p >> 6] & ((1ull << (p & 63)) - 1ull));
    }
    carry += all;
    __syncthreads();
  }
  if (tid == 0) n_rows[0] = carry;
  for (int b = tid; b < B; b += 1024) chunk_cnt[b] = (b + 1 < B ? chunk_off[b + 1] : carry) - chunk_off[b];
}

// ---------------------------------------------------------------- entropy
// Row statistics in the fixed partition of rowstats.h: the LM head's epilogue
// writes the statistics of every 128-column group (stats_merge_kernel merges
// them); from stored logits half a wave computes a group from one coalesced
// 16-byte load per lane.  row_stats_kernel does a whole row per block, merging
// in the same order; with few rows, group_stats_kernel spreads the groups over
// the chip into a scratch row per logit row, for stats_merge_kernel.  512 rows of
// 32768: 15 us, 24 when a thread read a whole group, 128 columns apart from the
// next thread's.

// columns 4 i .. 4 i + 3 (i = lane % 32) of group g of a row, -inf past V
__device__ __forceinline__ f32x4 group_quad(const float* lg, int g, int i, int V, bool aligned) {
  const int c = g * STAT_GROUP + 4 * i;
  if (aligned && c + 4 <= V) return *reinterpret_cast<const f32x4*>(lg + c);
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = c + e < V ? lg[c + e] : -INFINITY;
  return v;
}

// One row per block of NT threads, 256 groups at a time into LDS; lane l of
// wave 0 folds groups 256 c + l, + 64, + 128, + 192 into its running statistic
// -- the fold order of stats_merge_kernel.
template <int NT>
__global__ void __launch_bounds__(NT)
row_stats_kernel(const float* __restrict__ logits, const int32_t* __restrict__ n_dev, int V,
                 float* __restrict__ H, float* __restrict__ mx) {
  __shared__ RowStat part[256];
  const int row = blockIdx.x;
  if (n_dev && row >= *n_dev) return;
  const float* lg = logits + (size_t)row * V;
  const int tid = threadIdx.x, half = tid >> 5, i = tid & 31;
  const int G = stat_groups(V);
  const bool aligned = (V & 3) == 0 && ((uintptr_t)logits & 15) == 0;
  RowStat acc{-INFINITY, 0.0f, 0.0f};
  for (int g0 = 0; g0 < G; g0 += 256) {
    const int gn = min(256, G - g0);
#pragma unroll 2
    for (int g = half; g < gn; g += NT / 32) {
      const RowStat s = group_stat_lanes(group_quad(lg, g0 + g, i, V, aligned));
      if (i == 0) part[g] = s;
    }
    __syncthreads();
    if (tid < 64)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (g0 + tid + 64 * k < G) acc = stat_merge(acc, part[tid + 64 * k]);
    __syncthreads();
  }
  if (tid < 64) {
    acc = stat_butterfly<64>(acc);
    if (tid == 0) {
      H[row] = stat_entropy_bits(acc);
      mx[row] = acc.m;
    }
  }
}

// GPB groups per block: group statistics of row blockIdx.y into its scratch
// row (ld RowStats apart in 4-byte words)
constexpr int GROUPS_PER_BLOCK = 32;

__global__ void __launch_bounds__(256)
group_stats_kernel(const float* __restrict__ logits, int V, float* __restrict__ scratch, size_t ld) {
  const int row = blockIdx.y, half = threadIdx.x >> 5, i = threadIdx.x & 31;
  const float* lg = logits + (size_t)row * V;
  const bool aligned = (V & 3) == 0 && ((uintptr_t)logits & 15) == 0;
  const int G = stat_groups(V), g0 = blockIdx.x * GROUPS_PER_BLOCK;
  f32x4 v[GROUPS_PER_BLOCK / 8];
#pragma unroll
  for (int k = 0; k < GROUPS_PER_BLOCK / 8; ++k)
    if (g0 + half + 8 * k < G) v[k] = group_quad(lg, g0 + half + 8 * k, i, V, aligned);
#pragma unroll
  for (int k = 0; k < GROUPS_PER_BLOCK / 8; ++k) {
    const int g = g0 + half + 8 * k;
    if (g >= G) break;
    const RowStat s = group_stat_lanes(v[k]);
    if (i < 3) scratch[row * ld + 3 * (size_t)g + i] = i == 0 ? s.m : i == 1 ? s.Z : s.A;
  }
}

// Merge of the group statistics of a row, g < G at words row * ld + 3 g, one
// wave per row.
__global__ void __launch_bounds__(256)
stats_merge_kernel(const float* __restrict__ stats, size_t ld, int G, const int32_t* __restrict__ n_dev,
                   int n_max, float* __restrict__ H, float* __restrict__ mx) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n = n_dev ? min(*n_dev, n_max) : n_max;
  if (row >= n) return;
  const float* s = stats + (size_t)row * ld;
  RowStat acc{-INFINITY, 0.0f, 0.0f};
  for (int g0 = lane; g0 < G; g0 += 64 * 16) {
    RowStat r[16];  // 16 groups in flight per lane
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int g = g0 + 64 * k;
      r[k] = g < G ? RowStat{s[3 * g], s[3 * g + 1], s[3 * g + 2]} : RowStat{-INFINITY, 0.0f, 0.0f};
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) acc = stat_merge(acc, r[k]);
  }
  acc = stat_butterfly<64>(acc);
  if (lane == 0) {
    H[row] = stat_entropy_bits(acc);
    mx[row] = acc.m;
  }
}

// ---------------------------------------------------------------- selection
__device__ __forceinline__ uint32_t order_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int SEL_MAX_T = 8192;
constexpr int SEL_MAX_M = 1024;

// number of the ascending rows[0 .. n) below x: a wave probes the ends of 64 even
// stretches of the bracket at a time (65536 rows: three rounds of one load)
__device__ __forceinline__ int rows_below(const int32_t* __restrict__ rows, int n, int x) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = n;
  while (lo < hi) {
    const int step = (hi - lo + 63) / 64;
    const uint64_t below = __ballot(rows[min(lo + (lane + 1) * step, hi) - 1] < x);
    // probes past hi repeat its last row: whole stretches below x, or all of it
    const int full = min(lo + __popcll(below) * step, hi);
    hi = min(full + step - 1, hi);
    lo = full;
  }
  return lo;
}

// One workgroup per chunk: commit the n = min(|M|, max(m_min, min(m_max, #{H <=
// tau}))) masked positions that come first by (entropy, position), in
// ascending position order.  The n-th smallest entropy is found by a radix
// search, two bits a round: a thread keeps its keys (position order within each
// NT) in registers, ballots count the digits of the keys that still match the
// prefix, and the waves add their counts to one LDS word per digit.  The search
// ends when every key that still matches is to be committed.  Everything below
// the entropy found is committed, and the lowest positions among its equals;
// prefix counts over the ballots place them.  A round costs a barrier and an
// LDS round trip, so chunks that fit 8 keys per thread use 256 threads.  32
// chunks of 1024 masked positions: 13 us (35 with a bitonic sort of the keys).
template <int NT, int KPT>
__global__ void __launch_bounds__(NT)
select_kernel(const float* __restrict__ H, const int32_t* __restrict__ rows,
              const int32_t* __restrict__ chunk_off, const int32_t* __restrict__ chunk_cnt, int T,
              float tau, int m_min, int m_max, int32_t* __restrict__ sel_pos,
              int32_t* __restrict__ sel_row, int32_t* __restrict__ n_sel, int32_t* __restrict__ err,
              int n_rows) {
  constexpr int NW = NT / 64;
  __shared__ int digits[64];  // of round r: 4 r + digit
  __shared__ int wsum[KPT][NW], esum[KPT][NW];
  __shared__ int n_thr, n_bad;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int off, cnt;
  if (chunk_off) {
    off = chunk_off[b];
    cnt = chunk_cnt[b];
  } else {
    off = b == 0 ? 0 : rows_below(rows, n_rows, b * T);
    cnt = rows_below(rows, n_rows, (b + 1) * T) - off;
  }
  cnt = min(max(cnt, 0), NT * KPT);  // rows are distinct: at most T <= NT KPT of a chunk
  const int nr = (cnt + NT - 1) / NT;  // groups of NT keys in use
  if (tid < 64) digits[tid] = 0;
  if (tid == 0) n_thr = n_bad = 0;
  uint32_t key[KPT];
  int thr = 0, bad = 0;
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const int i = r * NT + tid;
    key[r] = 0;
    if (r < nr && i < cnt) {
      const float h = H[off + i];
      bad |= !(h == h) || isinf(h);
      thr += h <= tau;
      key[r] = order_bits(h);
    }
  }
  __syncthreads();
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) thr += __shfl_xor(thr, o);
  if (lane == 0 && thr) atomicAdd(&n_thr, thr);
  if (__any(bad) && lane == 0) n_bad = 1;
  __syncthreads();
  if (tid == 0 && n_bad) err[0] = 1;
  const int n = min(cnt, max(m_min, min(m_max, n_thr)));
  // key of the n-th smallest (1-based); `need` of its equals are committed
  // (with fewer bits in mask: of the keys that match the prefix, all)
  uint32_t prefix = 0, mask = 0;
  int need = n, match = cnt;
  if (n < cnt) {
#pragma unroll 1
    for (int round = 0; round < 16 && need < match; ++round) {
      const int sh = 30 - 2 * round;
      int c[3] = {0, 0, 0};
#pragma unroll
      for (int r = 0; r < KPT; ++r) {
        if (r >= nr) break;
        const bool in = r * NT + tid < cnt && (key[r] & mask) == prefix;
        const uint32_t d = key[r] >> sh & 3u;
#pragma unroll
        for (int k = 0; k < 3; ++k) c[k] += __popcll(__ballot(in && d == (uint32_t)k));
      }
      if (lane < 3) {
        const int v = lane == 0 ? c[0] : lane == 1 ? c[1] : c[2];
        if (v) atomicAdd(&digits[4 * round + lane], v);
      }
      __syncthreads();
      // keys with a digit below 1, 2 and 3 among those that match the prefix
      const int u1 = digits[4 * round], u2 = u1 + digits[4 * round + 1], u3 = u2 + digits[4 * round + 2];
      const uint32_t d = need > u3 ? 3u : need > u2 ? 2u : need > u1 ? 1u : 0u;
      const int below = need > u3 ? u3 : need > u2 ? u2 : need > u1 ? u1 : 0;
      prefix |= d << sh;
      mask |= 3u << sh;
      need -= below;
      match = d == 0 ? u1 : d == 1 ? u2 - u1 : d == 2 ? u3 - u2 : match - u3;
    }
  }
  int ls[KPT], le[KPT];  // committed-below and equal keys before this lane, in its wave
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    if (r >= nr) break;
    const bool valid = r * NT + tid < cnt;
    const uint64_t lt = __ballot(valid && (key[r] & mask) < prefix);
    const uint64_t eq = __ballot(valid && (key[r] & mask) == prefix);
    const uint64_t lower = (1ull << lane) - 1ull;
    ls[r] = __popcll(lt & lower);
    le[r] = __popcll(eq & lower);
    if (lane == 0) {
      wsum[r][wave] = __popcll(lt);
      esum[r][wave] = __popcll(eq);
    }
  }
  __syncthreads();
  int s0 = 0, e0 = 0;
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    if (r >= nr) break;
    int sw = s0, ew = e0, st = 0, et = 0;
    for (int w = 0; w < NW; ++w) {
      st += wsum[r][w];
      et += esum[r][w];
      if (w < wave) {
        sw += wsum[r][w];
        ew += esum[r][w];
      }
    }
    const int i = r * NT + tid;
    const bool valid = i < cnt, lt = valid && (key[r] & mask) < prefix;
    const bool eq = valid && (key[r] & mask) == prefix && ew + le[r] < need;
    if (lt || eq) {
      const int j = sw + ls[r] + min(ew + le[r], need);  // committed keys before this one
      sel_pos[b * m_max + j] = rows[off + i] - b * T;
      sel_row[b * m_max + j] = off + i;
    }
    s0 += st;
    e0 += et;
  }
  if (tid == 0) n_sel[b] = n;
}

// ---------------------------------------------------------------- CDF
__device__ __forceinline__ uint32_t gval(float l, float m) {
  return (uint32_t)(expf(l - m) * 16777216.0f);  // floor(e * 2^24), e in [0, 1]
}

template <typename U>
__device__ __forceinline__ U block_sum_int(U v, U* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// Integer CDF of the committed rows:
//   g_v = floor(exp(l_v - max) 2^24), G = sum g, f_v = 1 + floor(g_v (2^P - V) / G),
//   the remainder 2^P - sum f goes to the lowest index of maximal g,
//   cdf[0] = 0, cdf[v+1] = cdf[v] + f_v.
// Every sum is an integer, so no split of the work changes a single bit.  Two
// forms: one block per row with the row in registers (cdf_row_kernel), and,
// for few long rows, CDF_SEG-entry segments over three passes that park g, then
// f, in the CDF row itself: A: g, per-segment sum of g and lowest index with
// g = 2^24; B: f and per-segment sum of f; C: segment offset + in-segment scan.
constexpr int CDF_SEG = 4096;

struct CdfArgs {
  const float* logits;
  const float* mx;
  const int32_t* sel_row;
  const int32_t* n_sel;
  int m_max, V, P, S;
  uint32_t* cdf;
  uint32_t* g_out;
  uint64_t* segG;
  uint64_t* segF;
  int32_t* segA;
};

// whether slot holds a committed row, and which
__device__ __forceinline__ bool cdf_live(const CdfArgs& c, int slot) {
  if (!c.n_sel) return true;
  const int b = slot / c.m_max;
  return slot - b * c.m_max < c.n_sel[b];
}
// The slot of block i of a launch of one block per slot, and whether it holds a
// committed row.  A chunk's committed rows are its first few slots, m_max apart:
// with m_max a multiple of the 8 XCDs the rows of all chunks ran on one of them.
// There each run of 8 slots is turned round by its chunk's number (64 chunks, one
// row of 32768 each, m_max 32: 182 -> 30 us; 25 with the j-th slots of all chunks
// one after another, which made launches with every slot live 4 to 8% slower).
__device__ __forceinline__ bool cdf_block_slot(const CdfArgs& c, int i, int& slot) {
  slot = i;
  if (!c.n_sel || (c.m_max & 7)) return cdf_live(c, i);
  const int b = i / c.m_max;  // a run lies in one chunk
  slot = (i & ~7) | ((i + b) & 7);
  return slot - b * c.m_max < c.n_sel[b];
}
__device__ __forceinline__ int cdf_row_of(const CdfArgs& c, int slot) {
  return c.sel_row ? c.sel_row[slot] : slot;
}

// floor(g cst / G) for g <= 2^24, cst < 2^31, G < 2^53, by one double product:
// cst / G and the product are each rounded once, so t is off by less than 2^31
// x 2^-51 = 2^-20, and its floor is the quotient unless t lies within that of an
// integer, where it can be off by one and the remainder decides (once in about
// 2^17 entries).  A 64-bit division per entry took most of the time of passes B
// and C.
struct Quot {
  uint64_t cst, G;
  double c;
  __device__ Quot(uint64_t cst_, uint64_t G_) : cst(cst_), G(G_), c((double)cst_ / (double)G_) {}
  __device__ __forceinline__ uint32_t operator()(uint32_t g) const {
    const double t = (double)g * c;
    uint32_t q = (uint32_t)t;
    const double frac = t - (double)q;
    if (g != 0 && (frac < 0x1p-18 || frac > 1.0 - 0x1p-18)) {
      const int64_t r = (int64_t)((uint64_t)g * cst - (uint64_t)q * G);
      q += r < 0 ? -1 : r >= (int64_t)G ? 1 : 0;
    }
    return q;
  }
};

// G of a row.  A finite row maximum gives G >= 2^24; a row of non-finite
// logits (reported as E_NUMERIC before its CDF is used) can give 0, which is
// raised to 1 so that the quotients stay defined.
__device__ __forceinline__ uint64_t nonzero(uint64_t G) { return G > 0 ? G : 1; }

template <typename U>
__device__ __forceinline__ U wave_sum(U v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}

// inclusive prefix sum over the 64 lanes of a wave: row shifts, then the last
// lane of each 16-lane row broadcast into the next rows
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
#endif
  return x;
}

// One row per block: wave w holds entries 64 (w E + e) + lane, e < E, in
// registers (V <= NT E), so a logit is read once and a CDF entry written once.
template <int NT, int E>
__global__ void __launch_bounds__(NT) cdf_row_kernel(CdfArgs c) {
  constexpr int NW = NT / 64;
  __shared__ uint64_t wG[NW];
  __shared__ int wA[NW];
  __shared__ uint32_t wF[NW];
  int slot;
  if (!cdf_block_slot(c, blockIdx.x, slot)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = cdf_row_of(c, slot), V = c.V;
  const float* lg = c.logits + (size_t)row * V;
  const float m = c.mx[row];
  const int v0 = wave * 64 * E + lane;
  uint32_t f[E];
  uint64_t G = 0;
  int a = INT_MAX;
  constexpr int EB = E < 16 ? E : 16;  // loads in flight
#pragma unroll
  for (int e0 = 0; e0 < E; e0 += EB) {
    float l[EB];
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int v = v0 + 64 * (e0 + e);
      l[e] = v < V ? lg[v] : -INFINITY;
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int v = v0 + 64 * (e0 + e);
      const uint32_t g = v < V ? gval(l[e], m) : 0u;
      f[e0 + e] = g;
      G += g;
      if (g == (1u << 24)) a = min(a, v);
      if (c.g_out && v < V) c.g_out[(size_t)slot * V + v] = g;
    }
    __builtin_amdgcn_sched_barrier(0);  // else every load is hoisted, past the registers
  }
  G = wave_sum(G);
  a = wave_min(a);
  if (lane == 0) {
    wG[wave] = G;
    wA[wave] = a;
  }
  __syncthreads();
  G = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    G += wG[w];
    a = min(a, wA[w]);
  }
  const Quot quot((1ull << c.P) - (uint64_t)V, nonzero(G));
  uint32_t run = 0;  // entries of this wave before the current 64
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t inc = wave_scan(v0 + 64 * e < V ? 1u + quot(f[e]) : 0u);
    f[e] = run + inc;
    run += __builtin_amdgcn_readlane(inc, 63);
    if (e % 16 == 15) __builtin_amdgcn_sched_barrier(0);
  }
  if (lane == 0) wF[wave] = run;
  __syncthreads();
  uint32_t before = 0, F = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    before += w < wave ? wF[w] : 0u;
    F += wF[w];
  }
  const uint32_t R = (uint32_t)(1ull << c.P) - F;
  uint32_t* out = c.cdf + (size_t)slot * ((size_t)V + 1);
  if (tid == 0) out[0] = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int v = v0 + 64 * e;
    if (v < V) out[v + 1] = before + f[e] + (v >= a ? R : 0u);
  }
}

// where the passes keep the g of slot `slot`
__device__ __forceinline__ uint32_t* parked_g(const CdfArgs& c, int slot) {
  return c.g_out ? c.g_out + (size_t)slot * c.V : c.cdf + (size_t)slot * ((size_t)c.V + 1) + 1;
}

__global__ void __launch_bounds__(256) cdf_pass_a(CdfArgs c) {
  __shared__ uint64_t red64[4];
  __shared__ int redi[4];
  const int seg = blockIdx.x, slot = blockIdx.y;
  if (!cdf_live(c, slot)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = cdf_row_of(c, slot);
  const float* lg = c.logits + (size_t)row * c.V;
  uint32_t* park = parked_g(c, slot);
  const float m = c.mx[row];
  const int v0 = seg * CDF_SEG, v1 = min(c.V, v0 + CDF_SEG);
  uint64_t G = 0;
  int a = INT_MAX;
#pragma unroll 8
  for (int v = v0 + tid; v < v1; v += 256) {
    const uint32_t g = gval(lg[v], m);
    G += g;
    if (g == (1u << 24)) a = min(a, v);
    park[v] = g;
  }
  G = block_sum_int<uint64_t>(G, red64);
  a = wave_min(a);
  if (lane == 0) redi[wave] = a;
  __syncthreads();
  if (tid == 0) {
    c.segG[(size_t)slot * c.S + seg] = G;
    c.segA[(size_t)slot * c.S + seg] = min(min(redi[0], redi[1]), min(redi[2], redi[3]));
  }
}

__global__ void __launch_bounds__(256) cdf_pass_b(CdfArgs c) {
  __shared__ uint64_t red64[4];
  const int seg = blockIdx.x, slot = blockIdx.y;
  if (!cdf_live(c, slot)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  uint64_t G = 0;
  for (int s = lane; s < c.S; s += 64) G += c.segG[(size_t)slot * c.S + s];
  const Quot quot((1ull << c.P) - (uint64_t)c.V, nonzero(wave_sum(G)));
  const uint32_t* park = parked_g(c, slot);
  const int v0 = seg * CDF_SEG, v1 = min(c.V, v0 + CDF_SEG);
  uint64_t F = 0;
#pragma unroll 8
  for (int v = v0 + tid; v < v1; v += 256) F += 1u + quot(park[v]);
  F = block_sum_int<uint64_t>(F, red64);
  if (tid == 0) c.segF[(size_t)slot * c.S + seg] = F;
}

__global__ void __launch_bounds__(256) cdf_pass_c(CdfArgs c) {
  constexpr int PT = CDF_SEG / 256;  // consecutive entries per thread in the scan
  __shared__ uint32_t buf[CDF_SEG + CDF_SEG / PT];  // one word of padding per thread
  __shared__ uint32_t wtot[4];
  const int seg = blockIdx.x, slot = blockIdx.y;
  if (!cdf_live(c, slot)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint64_t F = 0, G = 0, before = 0;
  int a = INT_MAX;
  for (int s = lane; s < c.S; s += 64) {
    const uint64_t f = c.segF[(size_t)slot * c.S + s];
    G += c.segG[(size_t)slot * c.S + s];
    F += f;
    before += s < seg ? f : 0;
    a = min(a, c.segA[(size_t)slot * c.S + s]);
  }
  F = wave_sum(F);
  before = wave_sum(before);
  const Quot quot((1ull << c.P) - (uint64_t)c.V, nonzero(wave_sum(G)));
  a = wave_min(a);
  const uint32_t R = (uint32_t)((1ull << c.P) - F);
  uint32_t* out = c.cdf + (size_t)slot * ((size_t)c.V + 1);
  if (seg == 0 && tid == 0) out[0] = 0;
  const uint32_t* park = parked_g(c, slot);
  const int v0 = seg * CDF_SEG, v1 = min(c.V, v0 + CDF_SEG);
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int k = i * 256 + tid;
    buf[k + k / PT] = v0 + k < v1 ? 1u + quot(park[v0 + k]) : 0u;
  }
  __syncthreads();
  uint32_t f[PT], loc = 0;
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    loc += buf[tid * (PT + 1) + i];
    f[i] = loc;
  }
  const uint32_t inc = wave_scan(loc);
  if (lane == 63) wtot[wave] = inc;
  __syncthreads();
  uint32_t base = (uint32_t)before + inc - loc;
  for (int w = 0; w < wave; ++w) base += wtot[w];
#pragma unroll
  for (int i = 0; i < PT; ++i) buf[tid * (PT + 1) + i] = base + f[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int k = i * 256 + tid, v = v0 + k;
    if (v < v1) out[v + 1] = buf[k + k / PT] + (v >= a ? R : 0u);
  }
}

// a quiet NaN in element 0 of the first head input row, if any row exists
__global__ void poison_kernel(void* __restrict__ rows, int bf16, const int32_t* __restrict__ n_dev) {
  if (threadIdx.x == 0 && n_dev[0] > 0) {
    if (bf16)
      *(bf16_t*)rows = 0x7FC0u;
    else
      *(float*)rows = __builtin_nanf("");
  }
}

// ---------------------------------------------------------------- reveal
__global__ void gather_reveal_kernel(const uint32_t* __restrict__ cdf, const int32_t* __restrict__ sel_pos,
                                     const int32_t* __restrict__ n_sel, const int32_t* __restrict__ tokens,
                                     const int64_t* __restrict__ slot_base, int32_t* __restrict__ state,
                                     int T, int m_max, int V, uint32_t* __restrict__ sym) {
  const int b = blockIdx.x;
  for (int j = threadIdx.x; j < n_sel[b]; j += blockDim.x) {
    const int slot = b * m_max + j, pos = sel_pos[slot];
    const int s = tokens[slot_base[b] + pos];
    const uint32_t* c = cdf + (size_t)slot * (V + 1);
    sym[2 * slot] = c[s];
    sym[2 * slot + 1] = c[s + 1] - c[s];
    state[(size_t)b * T + pos] = s;
  }
}

__global__ void reveal_kernel(const int32_t* __restrict__ sel_pos, const int32_t* __restrict__ n_sel,
                              const int32_t* __restrict__ dec, int32_t* __restrict__ state, int T,
                              int m_max) {
  const int b = blockIdx.x;
  for (int j = threadIdx.x; j < n_sel[b]; j += blockDim.x) {
    const int slot = b * m_max + j;
    state[(size_t)b * T + sel_pos[slot]] = dec[slot];
  }
}

// ---------------------------------------------------------------- host exchange
// A pass hands the host a few short arrays (and a block schedule hands some to
// the device).  Each as a copy of its own was a launch of 2 us and a gap of its
// own, four to six a pass, where the data is a few hundred words; one kernel
// reads or writes the pinned buffers for all (4 KiB round trip of the tiny model,
// 128 passes: 24.7 -> 24.0 ms).
struct WordCopies {
  WordCopy c[MAX_WORD_COPIES];
};
__global__ void __launch_bounds__(256) copy_words_kernel(WordCopies k) {
  const size_t i0 = (size_t)blockIdx.x * 256 + threadIdx.x, step = (size_t)gridDim.x * 256;
#pragma unroll
  for (int j = 0; j < MAX_WORD_COPIES; ++j)
    for (size_t i = i0; i < k.c[j].words; i += step) ((uint32_t*)k.c[j].dst)[i] = ((const uint32_t*)k.c[j].src)[i];
}

// ---------------------------------------------------------------- decoding
// One wave per slot.  Every lane keeps the same decoder state; the lanes only
// split the search for the symbol, the largest s with row[s] <= t (row[0] = 0
// <= t < 2^P = row[V]): each round probes 64 evenly spaced entries of the
// bracket [lo, hi) and keeps the stretch after the last probe that is <= t,
// so V + 1 = 126465 entries take three rounds of one load per lane.
__global__ void __launch_bounds__(64)
decode_symbols_kernel(const uint32_t* __restrict__ cdf, const int32_t* __restrict__ n_sel, int m_max,
                      int V, int P, int W, int rans, uint64_t rans_lo, const uint8_t* __restrict__ payload,
                      DecSlot* __restrict__ slots, int32_t* __restrict__ dec, uint32_t* __restrict__ iv,
                      int32_t* __restrict__ err) {
  const int b = blockIdx.x, lane = threadIdx.x;
  DecSlot d = slots[b];
  if (!d.live) return;
  const int ns = min(n_sel[b], m_max);
  const uint8_t* data = payload + d.off;
  const uint64_t total = 1ull << P;
  bool bad = false;
  for (int j = 0; j < ns; ++j) {
    const int slot = b * m_max + j;
    const uint32_t* row = cdf + (size_t)slot * ((size_t)V + 1);
    uint64_t r = 0, t;
    if (rans) {
      t = d.x & (total - 1);
    } else {
      r = d.range >> P;
      if (r == 0) {
        bad = true;
        break;
      }
      t = d.x / r;
      if (t >= total) {
        bad = true;
        break;
      }
    }
    int lo = 0, hi = V;
    for (int round = 0; round < 8 && hi - lo > 1; ++round) {
      const int step = (hi - lo + 63) / 64;
      const int idx = lo + lane * step;
      const uint64_t le = __ballot(idx < hi && (uint64_t)row[idx] <= t);
      if (!le) break;  // row[lo] > t: not a CDF row; caught below
      lo += (63 - __clzll(le)) * step;
      hi = min(lo + step, hi);
    }
    const uint32_t c0 = row[lo], c1 = row[lo + 1];
    if (hi - lo != 1 || c0 > t || c1 <= t) {
      bad = true;
      break;
    }
    const uint64_t f = c1 - c0;
    if (rans) {
      d.x = f * (d.x >> P) + t - c0;
      while (d.x < rans_lo) {
        if (d.pos + 4 > d.len) {
          bad = true;
          break;
        }
        const uint8_t* w = data + d.pos;
        d.x = (d.x << 32) | ((uint64_t)w[0] | (uint64_t)w[1] << 8 | (uint64_t)w[2] << 16 | (uint64_t)w[3] << 24);
        d.pos += 4;
      }
      if (bad) break;
    } else {
      d.x -= r * c0;
      d.range = r * f;
      const uint64_t lim = 1ull << (W - 8);
      while (d.range < lim) {
        d.x = (d.x << 8) | (d.pos < d.len ? data[d.pos] : 0u);
        ++d.pos;
        d.range <<= 8;
      }
    }
    if (lane == 0) {
      dec[slot] = lo;
      iv[2 * slot] = c0;
      iv[2 * slot + 1] = (uint32_t)f;
    }
  }
  if (lane == 0) {
    if (bad) {
      d.live = 0;
      atomicCAS(err, 0, 2);
    }
    slots[b] = d;
  }
}

}  // namespace

void compact_masked(hipStream_t st, const int32_t* state, int B, int T, int mask_id,
                    int32_t* rows, int32_t* n_rows, int32_t* chunk_off, int32_t* chunk_cnt) {
  compact_kernel<<<1, 1024, 0, st>>>(state, B, T, mask_id, rows, n_rows, chunk_off, chunk_cnt);
  DLMC_HIP(hipGetLastError());
}

void entropy_rows(hipStream_t st, const float* logits, int n_max, const int32_t* n_dev, int V,
                  float* H, float* mx, void* scratch, size_t scratch_ld) {
  if (n_max <= 0) return;
  // Few long rows: a block per row would leave most CUs idle (64 rows of 126464:
  // 37 us; spread over the chip 12 + 5).  From about one row per CU on, and for rows
  // of a few groups, the single kernel is faster.
  const int G = stat_groups(V);
  if (scratch && !n_dev && n_max < 256 && G >= 2 * GROUPS_PER_BLOCK && scratch_ld >= (size_t)3 * G) {
    group_stats_kernel<<<dim3(ceil_div(G, GROUPS_PER_BLOCK), n_max), 256, 0, st>>>(logits, V, (float*)scratch,
                                                                                   scratch_ld);
    stats_merge_kernel<<<ceil_div(n_max, 4), 256, 0, st>>>((const float*)scratch, scratch_ld, G, nullptr,
                                                            n_max, H, mx);
  } else if (G > 32) {
    row_stats_kernel<1024><<<n_max, 1024, 0, st>>>(logits, n_dev, V, H, mx);
  } else {
    row_stats_kernel<64><<<n_max, 64, 0, st>>>(logits, n_dev, V, H, mx);
  }
  DLMC_HIP(hipGetLastError());
}

void entropy_merge(hipStream_t st, const void* stats, int ld, int V, int n_max, const int32_t* n_dev,
                   float* H, float* mx) {
  if (n_max <= 0) return;
  stats_merge_kernel<<<ceil_div(n_max, 4), 256, 0, st>>>((const float*)stats, (size_t)3 * ld, stat_groups(V),
                                                          n_dev, n_max, H, mx);
  DLMC_HIP(hipGetLastError());
}

void select_positions(hipStream_t st, const float* H, const int32_t* rows,
                      const int32_t* chunk_off, const int32_t* chunk_cnt, int B, int T,
                      float tau, int m_min, int m_max, int32_t* sel_pos, int32_t* sel_row,
                      int32_t* n_sel, int32_t* err_flag, int n_rows) {
  DLMC_CHECK(T <= SEL_MAX_T, DLMC_E_INVAL, "chunk length above 8192 is not supported");
  DLMC_CHECK(m_min >= 1 && m_max >= m_min && m_max <= SEL_MAX_M, DLMC_E_INVAL,
             "need 1 <= m_min <= m_max <= 1024");
  if (B <= 0) return;
  if (T <= 2048)
    select_kernel<256, 8><<<B, 256, 0, st>>>(H, rows, chunk_off, chunk_cnt, T, tau, m_min, m_max, sel_pos,
                                             sel_row, n_sel, err_flag, n_rows);
  else
    select_kernel<1024, SEL_MAX_T / 1024><<<B, 1024, 0, st>>>(H, rows, chunk_off, chunk_cnt, T, tau, m_min,
                                                              m_max, sel_pos, sel_row, n_sel, err_flag, n_rows);
  DLMC_HIP(hipGetLastError());
}

int cdf_segments(int V) { return ceil_div(V, CDF_SEG); }

// One block per row while a row fits in a block's registers and either the rows
// fill at least half the CUs or a row is a single segment; else in segments.
// 512 rows of 32768 with g: 61 us by rows, 122 in segments with a 64-bit division
// per entry; 64 rows of 126464 in segments: 43 us (59).  How many slots hold a
// committed row is known on the device only.  With up to 64 of 32768 entries, rows
// take 23 to 36 us however many slots there are; segments 16 to 35 up to 1024 slots,
// 25 to 43 at 2048 and 46 to 60 at 4096, most of it for blocks without a row.
bool cdf_by_rows(size_t slots, int V) { return V <= 32768 && (slots >= 128 || V <= CDF_SEG); }

void cdf_rows(hipStream_t st, const float* logits, const float* mx, const int32_t* sel_row,
              const int32_t* n_sel, int B, int m_max, int V, int P, uint32_t* cdf,
              uint32_t* g_out, void* seg_ws) {
  if (B <= 0) return;
  DLMC_CHECK(P <= 31 && (1ll << P) > V, DLMC_E_INVAL, "CDF precision must exceed the alphabet");
  DLMC_CHECK((int64_t)B * m_max <= 65535, DLMC_E_INVAL, "too many CDF rows per launch");
  CdfArgs c;
  c.logits = logits;
  c.mx = mx;
  c.sel_row = sel_row;
  c.n_sel = n_sel;
  c.m_max = m_max;
  c.V = V;
  c.P = P;
  c.S = cdf_segments(V);
  c.cdf = cdf;
  c.g_out = g_out;
  const size_t n = (size_t)B * m_max * c.S;
  c.segG = (uint64_t*)seg_ws;
  c.segF = c.segG + n;
  c.segA = (int32_t*)(c.segF + n);
  const int n_slots = B * m_max;
  if (cdf_by_rows((size_t)n_slots, V)) {
    if (V <= 1024) cdf_row_kernel<256, 4><<<n_slots, 256, 0, st>>>(c);
    else if (V <= 4096) cdf_row_kernel<256, 16><<<n_slots, 256, 0, st>>>(c);
    else if (V <= 16384) cdf_row_kernel<512, 32><<<n_slots, 512, 0, st>>>(c);
    else cdf_row_kernel<512, 64><<<n_slots, 512, 0, st>>>(c);
  } else {
    const dim3 grid(c.S, n_slots);
    cdf_pass_a<<<grid, 256, 0, st>>>(c);
    cdf_pass_b<<<grid, 256, 0, st>>>(c);
    cdf_pass_c<<<grid, 256, 0, st>>>(c);
  }
  DLMC_HIP(hipGetLastError());
}

void poison_head_input(hipStream_t st, void* rows, int bf16, const int32_t* n_dev) {
  poison_kernel<<<1, 64, 0, st>>>(rows, bf16, n_dev);
  DLMC_HIP(hipGetLastError());
}

void gather_reveal(hipStream_t st, const uint32_t* cdf, const int32_t* sel_pos,
                   const int32_t* n_sel, const int32_t* tokens, const int64_t* slot_base,
                   int32_t* state, int B, int T, int m_max, int V, uint32_t* sym) {
  if (B <= 0) return;
  gather_reveal_kernel<<<B, 256, 0, st>>>(cdf, sel_pos, n_sel, tokens, slot_base, state, T,
                                          m_max, V, sym);
  DLMC_HIP(hipGetLastError());
}

void reveal(hipStream_t st, const int32_t* sel_pos, const int32_t* n_sel, const int32_t* dec,
            int32_t* state, int B, int T, int m_max) {
  if (B <= 0) return;
  reveal_kernel<<<B, 256, 0, st>>>(sel_pos, n_sel, dec, state, T, m_max);
  DLMC_HIP(hipGetLastError());
}

void decode_symbols(hipStream_t st, const uint32_t* cdf, const int32_t* n_sel, int B, int m_max,
                    int V, int P, int W, bool rans, uint64_t rans_lo, const uint8_t* payload,
                    DecSlot* slots, int32_t* dec, uint32_t* iv, int32_t* err) {
  if (B <= 0) return;
  DLMC_CHECK(V >= 1 && P >= 1 && P <= 31 && (rans || (W >= 16 && W <= 64 && P <= W - 16)), DLMC_E_INVAL,
             "decode_symbols: bad coder parameters");
  decode_symbols_kernel<<<B, 64, 0, st>>>(cdf, n_sel, m_max, V, P, W, rans ? 1 : 0, rans_lo, payload,
                                          slots, dec, iv, err);
  DLMC_HIP(hipGetLastError());
}

void copy_words(hipStream_t st, const WordCopy* c, int n) {
  DLMC_CHECK(n >= 0 && n <= MAX_WORD_COPIES, DLMC_E_INVAL, "copy_words: too many copies");
  WordCopies k{};
  size_t top = 0;
  for (int j = 0; j < n; ++j) {
    k.c[j] = c[j];
    top = std::max(top, c[j].words);
  }
  if (top == 0) return;
  copy_words_kernel<<<(int)std::min<size_t>((top + 255) / 256, 256), 256, 0, st>>>(k);
  DLMC_HIP(hipGetLastError());
}

}  // namespace dlmc
