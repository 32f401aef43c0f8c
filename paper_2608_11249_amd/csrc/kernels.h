// Host-side launchers of the HIP kernels of the masked-diffusion step.
#pragma once

#include "common.h"

namespace dlmc {

// ---------------------------------------------------------------- GEMMs
// Epilogues fused into C = A * B^T (A [M, K] activations, B [N, K] weights).
enum EpiKind : int {
  EPI_STORE_F32 = 0,  // out_f32[row * ldo + col] = acc                 (LM head logits)
  EPI_RESIDUAL = 1,   // x[row * ldo + col] += acc                      (O-proj, FFN out)
  EPI_QKV_ROPE = 2,   // Q, K with rotary embedding, V transposed       (QKV projection)
  EPI_GELU = 3,       // out_bf16[row * ldo + col] = gelu(acc)          (FFN in, GELU)
  EPI_SWIGLU = 4,     // out_bf16[row * ldo + col/2..] = silu(g) * u     (FFN gate/up pairs)
};

struct EpiArgs {
  void* out = nullptr;  // float* or bf16_t* depending on the epilogue
  int ldo = 0;
  // EPI_QKV_ROPE: Q, K are [B, H, Tp, dh]; Vt is [B, H, dh, Tp]
  void* q = nullptr;
  void* k = nullptr;
  void* vt = nullptr;
  const float* rope_cos = nullptr;  // [T, dh/2]
  const float* rope_sin = nullptr;
  int T = 0, Tp = 0, H = 0, dh = 0, d = 0;
  float inv_T = 0.0f;  // 1 / T
  // row / T for rows below 2^22: row + 0.5 is exact, its product with 1 / T is off
  // by less than 2^-23 of itself, and at least 0.5 / T from a whole number (an
  // integer division by T is some forty issue slots, more than a QKV tile's
  // rotary arithmetic: 32768 x 2304 x 768 161 -> 148 us, 2048 x 12288 x 4096 198 -> 191)
  __device__ __forceinline__ int chunk_of(int row) const { return (int)(((float)row + 0.5f) * inv_T); }
  // EPI_STORE_F32 (optional): softmax statistics of every 128-column group of
  // every stored row, RowStat [rows, stat_ld] (rowstats.h)
  void* stats = nullptr;
  int stat_ld = 0;
};

// Tile shape of a bf16 GEMM (the choice never changes the result):
// 128 x 128 or 192 x 128 tiles two blocks per CU; the 4-wave kernel with
// columns [0, split) on 256 x 256 tiles and [split, N) on 256 x 128 tiles; or,
// for launches with few tiles, the ring kernel on 64 x 64, 128 x 64 or
// (one block per CU) 128 x 128 tiles.  deep: more LDS stages, fewer blocks per CU.
enum GemmTileKind {
  GEMM_TILES_128x128 = 0,
  GEMM_TILES_192x128 = 1,
  GEMM_TILES_4WAVE = 2,
  GEMM_TILES_64x64 = 3,
  GEMM_TILES_128x64 = 4,
  GEMM_TILES_128x128_DEEP = 5
};
struct GemmTiles {
  int kind, split, deep;
};
// the choice gemm_bf16 makes for these sizes (d: the QKV epilogue's model
// width); host only
GemmTiles gemm_bf16_tiles(int M, int N, int K, EpiKind epi, int d, int rows_hint);
// M_dev (optional): device int holding the live row count (<= M); rows at or
// beyond it are neither computed (whole tiles) nor stored.  rows_hint: the
// live row count if the host knows it (tile selection only), else -1.
void gemm_bf16(hipStream_t st, const bf16_t* A, const bf16_t* B, int M, int N, int K,
               const int* M_dev, EpiKind epi, const EpiArgs& ea, int rows_hint = -1);
void gemm_f32(hipStream_t st, const float* A, const float* B, int M, int N, int K,
              const int* M_dev, EpiKind epi, const EpiArgs& ea);

// whether gemm_f32 takes EPI_QKV_ROPE at this width and head dim
bool gemm_f32_fuses_rope(int d, int dh);

// fp32 path helpers (fused into GEMM epilogues elsewhere): rotary for widths
// gemm_f32 does not fuse, and SwiGLU
void qkv_rope_f32(hipStream_t st, const float* qkv, int M, const EpiArgs& ea);
void swiglu_f32(hipStream_t st, const float* in, float* out, int M, int F);

// ---------------------------------------------------------------- attention
// Non-causal softmax(Q K^T / sqrt(dh)) V over all T keys of each chunk.
// out is [B*T, H*dh] row-major.  ml, if given, takes each row's (m, l) at
// [b, h, t] with pitch Tp: a probability is e^(s - m) / l of the scaled score s
// (bf16: 2^(s log2(e) - m) / l).
void attention_bf16(hipStream_t st, const bf16_t* q, const bf16_t* k, const bf16_t* vt,
                    bf16_t* out, int B, int H, int T, int Tp, int dh, float2* ml = nullptr);
void attention_f32(hipStream_t st, const float* q, const float* k, const float* vt, float* out,
                   int B, int H, int T, int Tp, int dh, float2* ml = nullptr);

// ---------------------------------------------------------------- elementwise
// Row layout of an initialised weight tensor inside its device buffer.
enum RowMap : int {
  MAP_IDENTITY = 0,  // device row = canonical row + offset
  MAP_QK_PAIRS = 1,  // rotate-half pairs (i, i + dh/2) moved to adjacent 32-row blocks
  MAP_GLU_PAIRS = 2, // gate/up features interleaved in 32-row blocks (up: offset 32)
};
void init_weights(hipStream_t st, void* dst, int dtype, uint64_t seed, int tensor_id, int rows,
                  int cols, int exp, RowMap map, int row_offset, int dh);
void embed(hipStream_t st, const int32_t* state, const void* table, int dtype, float* x,
           int n_rows, int d, int max_id);
// gather_rows (optional): output row i normalises x[gather_rows[i]]; n_dev
// (optional) holds the live row count.
void norm_rows(hipStream_t st, const float* x, void* out, int out_dtype, int n_rows, int d,
               int norm_kind, float eps, const int32_t* gather_rows, const int32_t* n_dev);
void fill_i32(hipStream_t st, int32_t* p, int32_t v, size_t n);
// dst[b*m_max + j] = src[sel_row[b*m_max + j]] (rows of d bf16) and
// dst_mx[b*m_max + j] = mx[sel_row[b*m_max + j]] for j < n_sel[b], else zeros
void gather_slot_rows(hipStream_t st, const bf16_t* src, const float* mx, const int32_t* sel_row,
                      const int32_t* n_sel, int B, int m_max, int d, bf16_t* dst, float* dst_mx);

// ---------------------------------------------------------------- coding stages
// rows[] = flat indices b*T+t with state == mask_id (ascending), n_rows[0],
// chunk_off[b] / chunk_cnt[b] = the segment of chunk b inside rows[].
void compact_masked(hipStream_t st, const int32_t* state, int B, int T, int mask_id,
                    int32_t* rows, int32_t* n_rows, int32_t* chunk_off, int32_t* chunk_cnt);
// per row of logits[n, V]: entropy in bits and row max (n from n_dev when given).
// scratch (optional): rows of scratch_ld 4-byte words for the group statistics
// of each row, overwritten; lets few long rows use the whole chip
void entropy_rows(hipStream_t st, const float* logits, int n_max, const int32_t* n_dev, int V,
                  float* H, float* mx, void* scratch = nullptr, size_t scratch_ld = 0);
// the same from the 128-column group statistics the LM head's epilogue
// wrote (stats: RowStat [n, ld]); bit-identical to entropy_rows
void entropy_merge(hipStream_t st, const void* stats, int ld, int V, int n_max, const int32_t* n_dev,
                   float* H, float* mx);
// commitment schedule, one workgroup per chunk.  chunk_off / chunk_cnt NULL: the
// chunks' segments are found in the ascending rows[n_rows]
void select_positions(hipStream_t st, const float* H, const int32_t* rows,
                      const int32_t* chunk_off, const int32_t* chunk_cnt, int B, int T,
                      float tau, int m_min, int m_max, int32_t* sel_pos, int32_t* sel_row,
                      int32_t* n_sel, int32_t* err_flag, int n_rows = 0);
// integer CDF of row sel_row[b*m_max+j] of logits (for j < n_sel[b]) into
// cdf[(b*m_max+j)*(V+1) ..]; g_out (optional) receives the g values.
// sel_row and n_sel NULL (m_max 1): slot i is row i.
// seg_ws: device workspace of cdf_workspace_bytes(B * m_max, V) bytes; unused
// (may be NULL) where cdf_by_rows(B * m_max, V).
bool cdf_by_rows(size_t slots, int V);
int cdf_segments(int V);
inline size_t cdf_workspace_bytes(size_t slots, int V) {
  return slots * (size_t)cdf_segments(V) * (8 + 8 + 4);
}
void cdf_rows(hipStream_t st, const float* logits, const float* mx, const int32_t* sel_row,
              const int32_t* n_sel, int B, int m_max, int V, int P, uint32_t* cdf,
              uint32_t* g_out, void* seg_ws);
// ---------------------------------------------------------------- static scratch
// Bytes of the static device scratch used by the allocation-free entry point.
constexpr size_t SCRATCH_BYTES = DLMC_SCRATCH_BYTES;
// Device address of `device`'s copy of the scratch (looked up on first use,
// with that device current; each GPU holds its own copy).
void* scratch_address(int device);

// test hook: a NaN into element 0 of the head's input rows (bf16 or fp32)
// when n_dev[0] > 0, which makes the first head row non-finite
void poison_head_input(hipStream_t st, void* rows, int bf16, const int32_t* n_dev);
// encode: (start, freq) of the true symbol of every committed position and reveal it
void gather_reveal(hipStream_t st, const uint32_t* cdf, const int32_t* sel_pos,
                   const int32_t* n_sel, const int32_t* tokens, const int64_t* slot_base,
                   int32_t* state, int B, int T, int m_max, int V, uint32_t* sym);
// decode: reveal decoded symbols
void reveal(hipStream_t st, const int32_t* sel_pos, const int32_t* n_sel, const int32_t* dec,
            int32_t* state, int B, int T, int m_max);
// decode: the entropy decoder of one batch slot, kept in device memory between
// passes.  Range coder: x = code - low and range; rANS: x = the state.  pos /
// len: read position and length (bytes) of the slot's stream, which starts at
// byte off of the payload buffer.  Slots with live = 0 decode nothing.
struct DecSlot {
  uint64_t x, range, pos, len, off;
  uint32_t live, pad;
};
// decode: one wave per live slot b decodes the slot's n_sel[b] committed
// symbols of the pass, in slot order, from CDF rows b * m_max + j (V + 1 words
// each) with the arithmetic of the host decoders (W-bit range coder, or rANS
// with lower bound rans_lo when `rans`); writes dec[slot] = symbol and
// iv[2 slot], iv[2 slot + 1] = (start, freq), and the slot's new state.  A
// corrupt stream stops its slot and sets *err to 2 if it was 0.
void decode_symbols(hipStream_t st, const uint32_t* cdf, const int32_t* n_sel, int B, int m_max,
                    int V, int P, int W, bool rans, uint64_t rans_lo, const uint8_t* payload,
                    DecSlot* slots, int32_t* dec, uint32_t* iv, int32_t* err);
// Up to MAX_WORD_COPIES copies of 32-bit words in one launch, between device
// memory and pinned host memory (visible on the other side as a copy's would be:
// to the host once the stream is synchronised).
struct WordCopy {
  const void* src;
  void* dst;
  size_t words;
};
constexpr int MAX_WORD_COPIES = 6;
void copy_words(hipStream_t st, const WordCopy* c, int n);
// attention-based context: the head-averaged map A [T, T] (pitch ld, a multiple
// of 64) of one chunk's Q and K [H, Tp, dh] and attention's (m, l), and the rollout
// out = v through maps L - 1 .. 0 (each T rows of pitch ld); v has ld entries, ws
// 2 ROLLOUT_PARTS ld
constexpr int ROLLOUT_PARTS = 64;
void attention_map(hipStream_t st, const void* q, const void* k, const float2* ml, float* A, bool bf16,
                   int H, int T, int Tp, int dh, int ld);
void rollout(hipStream_t st, const float* maps, int L, const float* v, float* ws, float* out, int T,
             int ld);
// symbol ranking: encode writes (rank, symbol) pairs to out[2 * slot], decode
// turns rank[slot] into sym[slot] (may be the same array; *err = 1 for a rank
// outside the alphabet); both reveal the symbols in state.  With sel_row NULL
// (B rows, m_max 1) slot i is row i, nothing is revealed, tokens[i] is row i's
// symbol and its rank goes to out[i]; a rank outside the alphabet (*err, 0 before the
// call) then leaves all of sym alone.
void rank_symbols(hipStream_t st, const float* logits, const int32_t* sel_row,
                  const int32_t* sel_pos, const int32_t* n_sel, const int32_t* tokens,
                  const int64_t* slot_base, int32_t* state, int B, int T, int m_max, int V,
                  uint32_t* out);
void select_by_rank(hipStream_t st, const float* logits, const int32_t* sel_row,
                    const int32_t* sel_pos, const int32_t* n_sel, const int32_t* rank, int32_t* sym,
                    int32_t* state, int B, int T, int m_max, int V, int32_t* err);

}  // namespace dlmc
