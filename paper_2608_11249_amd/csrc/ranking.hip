// Symbol ranking on the GPU (Definition of Symbol Ranking): the rank of a
// symbol is its index in the list of all symbols ordered by non-increasing
// probability, equal probabilities by token id.  Probability order is logit
// order, so both kernels compare 32-bit keys of the fp32 logits that sort
// ascending in rank order (larger logits first; -0 counts as +0).
//
// Encode: rank = #{v : (key_v, v) < (key_s, s)} -- one read of the row.
// Decode: the symbol of rank r.  The row's logits are binned by value, 2048 even
// bins from the row's maximum down (a monotone map, so rank order is bin order),
// the bin that holds rank r is found from the counts, and the few candidates in
// it are collected and ranked exactly by (key, id): three coalesced reads of
// the row, and counting that spreads over the bins.  Rows that this cannot
// split -- non-finite logits, more than CAP candidates in the bin (one logit far
// from the others leaves those in a few bins) -- take a radix selection over the
// keys: 11 bits a pass, as many counts as bins, until no more than CAP keys match,
// and where more are equal, a prefix count in id order.  A call over 512 rows of
// 32768 takes 54 us by bins and, by radix as well, 99 (an infinity in each row),
// 148 (a logit of 1e4) to 253 us (all equal), where four 8-bit passes and the count
// alone took 248, 261 and 465, and behind the bins 206, 225 and 417; 64 rows of
// 126464 with a logit of 1e4 take 194 us, against 332 alone and 373 behind the bins.
// Both kernels also reveal the symbol in the state.
#include "kernels.h"

namespace dlmc {
namespace {

constexpr int RT = 1024;  // threads per row

__device__ __forceinline__ uint32_t rank_key(float l) {
  uint32_t u = __float_as_uint(l);
  if (u == 0x80000000u) u = 0u;
  const uint32_t asc = (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // ascending in l
  return ~asc;
}

// exclusive prefix sum over the RT threads of a block; returns the block total in *total
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* lds, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) lds[wave] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t run = 0;
    for (int w = 0; w < RT / 64; ++w) {
      const uint32_t t = lds[w];
      lds[w] = run;
      run += t;
    }
    lds[RT / 64] = run;
  }
  __syncthreads();
  const uint32_t ex = lds[wave] + incl - x;
  *total = lds[RT / 64];
  __syncthreads();
  return ex;
}

// Row and slot tables of a launch.  With sel_row NULL every row is its own slot
// (row = slot = blockIdx.x, always live, nothing to reveal).
struct RankArgs {
  const float* logits;
  const int32_t* sel_row;
  const int32_t* sel_pos;
  const int32_t* n_sel;
  int T, m_max, V;
  int32_t* state;
};
__device__ __forceinline__ bool rank_slot(const RankArgs& a, int& slot, const float*& row) {
  slot = blockIdx.x;
  if (a.sel_row) {
    const int b = slot / a.m_max;
    if (slot - b * a.m_max >= a.n_sel[b]) return false;
  }
  row = a.logits + (size_t)(a.sel_row ? a.sel_row[slot] : slot) * a.V;
  return true;
}
__device__ __forceinline__ void rank_reveal(const RankArgs& a, int slot, int s) {
  if (a.sel_row) a.state[(size_t)(slot / a.m_max) * a.T + a.sel_pos[slot]] = s;
}

__global__ void __launch_bounds__(RT)
rank_kernel(RankArgs a, const int32_t* __restrict__ tokens, const int64_t* __restrict__ slot_base,
            uint32_t* __restrict__ out) {
  __shared__ uint32_t lds[RT / 64 + 1];
  int slot;
  const float* row;
  if (!rank_slot(a, slot, row)) return;
  const int V = a.V;
  const int s = a.sel_row ? tokens[slot_base[slot / a.m_max] + a.sel_pos[slot]] : tokens[slot];
  const uint32_t ks = rank_key(row[s]);
  uint32_t cnt = 0;
#pragma unroll 8
  for (int v = threadIdx.x; v < V; v += RT) {
    const uint32_t kv = rank_key(row[v]);
    cnt += (kv < ks) || (kv == ks && v < s);
  }
  uint32_t total;
  (void)block_exclusive_scan(cnt, lds, &total);
  if (threadIdx.x == 0) {
    if (a.sel_row) {
      out[2 * slot] = total;
      out[2 * slot + 1] = (uint32_t)s;
    } else {
      out[slot] = total;
    }
    rank_reveal(a, slot, s);
  }
}

// CAP: comparing n candidates with one another takes n^2 / 128 LDS reads, which 2048
// of them made dearer than another pass over a row (512 rows of 4099, two values
// in a bin each: 158 us a call, 79 with 1280)
constexpr int BINS = 2048, CAP = 1280;

// bin of a logit of a row with maximum hi (monotone in l: larger logits first)
__device__ __forceinline__ int rank_bin(float l, float hi, float scale) {
  return min((int)((hi - l) * scale), BINS - 1);
}

// The bin (count) that holds rank r: sh[0] = the bin, sh[1] = the rank inside it,
// sh[3] = its count.
__device__ __forceinline__ void pick_bin(const uint32_t* hist, uint32_t r, uint32_t* lds, uint32_t* sh) {
  static_assert(BINS == 2 * RT, "two bins per thread");
  const uint32_t h0 = hist[2 * threadIdx.x], h1 = hist[2 * threadIdx.x + 1];
  uint32_t total;
  const uint32_t base = block_exclusive_scan(h0 + h1, lds, &total);
  if (r >= base && r < base + h0 + h1) {
    const int second = r >= base + h0;
    sh[0] = 2 * threadIdx.x + second;
    sh[1] = r - base - (second ? h0 : 0u);
    sh[3] = second ? h1 : h0;
  }
  __syncthreads();
}

// *found = the id of the candidate of rank r among n candidates (key, id); cand has
// one more entry, all ones, if n is odd
__device__ __forceinline__ void rank_candidates(const uint64_t* cand, int n, uint32_t r, int32_t* found) {
  for (int i = threadIdx.x; i < n; i += RT) {
    const uint64_t me = cand[i];
    uint32_t before = 0;
#pragma unroll 4
    for (int k = 0; k < n; k += 2) {
      const ulonglong2 c = *reinterpret_cast<const ulonglong2*>(cand + k);
      before += (c.x < me) + (c.y < me);
    }
    if (before == r) *found = (int32_t)(uint32_t)me;
  }
}

// the general selection: see the head of the file
__device__ void radix_select(const float* __restrict__ row, int V, uint32_t rest, uint32_t* hist,
                             uint64_t* cand, uint32_t* lds, uint32_t* sh, int32_t* found) {
  uint32_t prefix = 0, mask = 0;
#pragma unroll 1
  for (int shift = 21; shift >= 0; shift -= shift > 10 ? 11 : shift > 0 ? shift : 1) {
    const uint32_t digit = shift > 0 ? 2047u : 1023u;  // bits 21 .. 31, 10 .. 20, 0 .. 9
    for (int d = threadIdx.x; d < BINS; d += RT) hist[d] = 0;
    if (threadIdx.x == 0) sh[2] = 0;
    __syncthreads();
#pragma unroll 8
    for (int v = threadIdx.x; v < V; v += RT) {
      const uint32_t k = rank_key(row[v]);
      if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & digit], 1u);
    }
    __syncthreads();
    pick_bin(hist, rest, lds, sh);
    prefix |= sh[0] << shift;
    rest = sh[1];
    mask |= digit << shift;
    if (sh[3] <= (uint32_t)CAP) {
      if (threadIdx.x == 0) cand[sh[3]] = ~0ull;
#pragma unroll 8
      for (int v = threadIdx.x; v < V; v += RT) {
        const uint32_t k = rank_key(row[v]);
        if ((k & mask) == prefix) cand[atomicAdd(&sh[2], 1u)] = (uint64_t)k << 32 | (uint32_t)v;
      }
      __syncthreads();
      rank_candidates(cand, (int)sh[2], rest, found);
      return;
    }
  }
  // the rest-th id (in id order) among the symbols whose key is `prefix`
  const int per = (V + RT - 1) / RT, lo = threadIdx.x * per, hi = min(lo + per, V);
  uint32_t c = 0;
  for (int v = lo; v < hi; ++v) c += rank_key(row[v]) == prefix;
  uint32_t total;
  uint32_t base = block_exclusive_scan(c, lds, &total);
  if (rest >= base && rest < base + c) {
    for (int v = lo; v < hi; ++v) {
      if (rank_key(row[v]) != prefix) continue;
      if (base == rest) {
        *found = v;
        break;
      }
      ++base;
    }
  }
}

// *err = 1 if one of n ranks lies outside the alphabet (one block)
__global__ void __launch_bounds__(RT)
check_ranks_kernel(const int32_t* __restrict__ rank, int n, int V, int32_t* __restrict__ err) {
  bool out = false;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += RT) out |= rank[i] < 0 || rank[i] >= V;
  if (__syncthreads_or(out) && threadIdx.x == 0) *err = 1;
}

// rank[slot] -> sym[slot] (the two may be the same array).  A rank outside the
// alphabet sets *err and leaves its row alone, or, with n_check, every row: each
// block looks at all of rank[0 .. n_check), where another may have put a symbol, in
// the alphabet like the rank it stands for.  Nothing is done if *refuse is set.
__global__ void __launch_bounds__(RT)
select_rank_kernel(RankArgs a, const int32_t* rank, int32_t* sym, int32_t* err, int n_check,
                   const int32_t* refuse) {
  __shared__ uint32_t hist[BINS];
  __shared__ __attribute__((aligned(16))) uint64_t cand[CAP + 2];
  __shared__ uint32_t lds[RT / 64 + 1];
  __shared__ float red[2][RT / 64];
  __shared__ int wave_out[RT / 64];
  __shared__ uint32_t sh[4];  // bin, rank inside it, candidates, their count
  __shared__ int32_t found;
  int slot;
  const float* row;
  if ((refuse && *refuse) || !rank_slot(a, slot, row)) return;
  const int V = a.V, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t want = rank[slot];
  bool out = want < 0 || want >= V;
  for (int i = tid; i < n_check; i += RT) out |= rank[i] < 0 || rank[i] >= V;
  float mx = -INFINITY, mn = INFINITY;
  bool odd = false;  // a NaN or an infinity
#pragma unroll 8
  for (int v = tid; v < V; v += RT) {
    const float l = row[v];
    mx = fmaxf(mx, l);
    mn = fminf(mn, l);
    odd |= !(fabsf(l) <= 3.0e38f);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    mx = fmaxf(mx, __shfl_xor(mx, o));
    mn = fminf(mn, __shfl_xor(mn, o));
  }
  out = __any(out);
  if (lane == 0) {
    red[0][wave] = mx;
    red[1][wave] = mn;
    wave_out[wave] = out;
  }
  for (int d = tid; d < BINS; d += RT) hist[d] = 0;
  if (tid == 0) sh[2] = 0;
  odd = __syncthreads_or(odd);
#pragma unroll
  for (int w = 0; w < RT / 64; ++w) {
    mx = fmaxf(mx, red[0][w]);
    mn = fminf(mn, red[1][w]);
    out |= wave_out[w] != 0;
  }
  if (out) {
    if (tid == 0) *err = 1;
    return;
  }
  // (BINS - 1/2 of the range: rounding cannot push the minimum past the last bin
  // by more than the clamp takes back)
  const float scale = ((float)BINS - 0.5f) / (mx - mn);
  bool general = odd || !(mx - mn <= 3.0e38f) || !(scale <= 3.0e38f);
  if (!general) {
#pragma unroll 8
    for (int v = tid; v < V; v += RT) atomicAdd(&hist[rank_bin(row[v], mx, scale)], 1u);
    __syncthreads();
    pick_bin(hist, (uint32_t)want, lds, sh);
    const int bin = (int)sh[0];
    general = sh[3] > (uint32_t)CAP;
    if (!general) {
      if (tid == 0) cand[sh[3]] = ~0ull;
#pragma unroll 8
      for (int v = tid; v < V; v += RT) {
        const float l = row[v];
        if (rank_bin(l, mx, scale) == bin)
          cand[atomicAdd(&sh[2], 1u)] = (uint64_t)rank_key(l) << 32 | (uint32_t)v;
      }
      __syncthreads();
      rank_candidates(cand, (int)sh[2], sh[1], &found);
    }
  }
  if (general) radix_select(row, V, (uint32_t)want, hist, cand, lds, sh, &found);
  __syncthreads();
  if (tid == 0) {
    sym[slot] = found;
    rank_reveal(a, slot, found);
  }
}

}  // namespace

void rank_symbols(hipStream_t st, const float* logits, const int32_t* sel_row,
                  const int32_t* sel_pos, const int32_t* n_sel, const int32_t* tokens,
                  const int64_t* slot_base, int32_t* state, int B, int T, int m_max, int V,
                  uint32_t* out) {
  if (B <= 0 || m_max <= 0) return;
  DLMC_CHECK(m_max <= 65535 && B <= 65535, DLMC_E_INVAL, "too many rank rows per launch");
  const RankArgs a{logits, sel_row, sel_pos, n_sel, T, m_max, V, state};
  rank_kernel<<<B * m_max, RT, 0, st>>>(a, tokens, slot_base, out);
  DLMC_HIP(hipGetLastError());
}

void select_by_rank(hipStream_t st, const float* logits, const int32_t* sel_row,
                    const int32_t* sel_pos, const int32_t* n_sel, const int32_t* rank, int32_t* sym,
                    int32_t* state, int B, int T, int m_max, int V, int32_t* err) {
  if (B <= 0 || m_max <= 0) return;
  DLMC_CHECK(m_max <= 65535 && B <= 65535, DLMC_E_INVAL, "too many rank rows per launch");
  const RankArgs a{logits, sel_row, sel_pos, n_sel, T, m_max, V, state};
  // Without slots a bad rank refuses the call.  Every block checks up to 4096 ranks,
  // four a thread, behind its other loads; a launch of its own before that took 5 us.
  const int n = sel_row ? 0 : B;
  const bool apart = n > 4096;
  if (apart) check_ranks_kernel<<<1, RT, 0, st>>>(rank, n, V, err);
  select_rank_kernel<<<B * m_max, RT, 0, st>>>(a, rank, sym, err, apart ? 0 : n, apart ? err : nullptr);
  DLMC_HIP(hipGetLastError());
}

}  // namespace dlmc
