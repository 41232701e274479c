// Kernel argument blocks and launchers (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pd {

constexpr int kNumCu = 256;

// Gathered KV rows of one decode shard whose cache-row codes fit the kernel's
// LDS table; the host raises the shard count until every shard fits.
constexpr int kDecodeTableRows = 2048;

// Query rows of a bf16 prefill workgroup, and of a decode one when it has four
// waves.
constexpr int kBf16Rows = 128;

// Stage (a).  Element pointers are bf16 bit patterns (uint16_t) or fp32.
struct PrefillArgs {
  const uint16_t *q_pre, *k_pre, *v_pre, *q_qm, *k_qm, *v_qm;
  uint16_t *o, *k_cache, *v_cache;
  float* part_i;   // [B][N][Hq][C]  per-head mass of content row j on the query columns
  float* lse_q;    // [B][N][Hq][Lq] log2-domain LSE of the query rows
  float* qm_mass;  // [B][N][Hq][Lq+Lm] mass of each q/m row on the C content columns, or nullptr
  float* km_part;  // bf16: [B][N][Hkv][n_qt*G][d] content-key sums of each cache-writing workgroup
  int B, N, C, Lq, Lm, Hq, Hkv, G, Sc;
  int n_qt, n_kvt, total;
  int qm_per_chunk;
  int out_f32;       // o is fp32 instead of the input element type
  float scale_log2;  // softmax scale * log2(e)
};

struct EscoreArgs {
  const uint16_t *q_qm, *k_cache;
  const float* lse_q;
  float* part_io;    // per-head sums [B][N][Hq][C], updated in place
  int B, N, C, Lq, Lm, Hq, Hkv, G, n_cb, qm_per_chunk;
  int q2c;           // 1: only the query rows' mass on the token (query-to-chunk score)
  float scale_log2;
};

// Stage (c).
struct DecodeArgs {
  const uint16_t *q_dec, *k_dec, *v_dec, *k_cache, *v_cache, *k_static, *v_static;
  const int32_t *chunk_idx, *tok_slot;
  void* o_dec;       // element type of the call
  float* lse_dec;    // natural-log LSE or nullptr (only when S == 1)
  float* o_part;     // [S][B][Hq][Ld][D] shard outputs (normalised), S > 1
  float* lse_part;   // [S][B][Hq][Ld] log2-domain shard LSE, S > 1
  int B, N, C, Hq, Hkv, G, Ld, Ls, K, Bt, n_static, S;
  int n_sel;         // prefix rows per (sequence, KV head): K*(1+Bt) gathered, or the compact count
  int compact;       // 1: prefix rows j < n_sel are rows of k_cache/v_cache laid out [B][Hkv][n_sel][D]
  int n_qt, total;
  int out_f32;       // o_dec is fp32 instead of the input element type
  float scale_log2;
};

// n workgroups, block_id() < n, rounded up to whole rows of the grid.
inline dim3 grid_xy(long long n) {
  const long long x = n < (1 << 20) ? n : 1 << 20;
  return dim3((unsigned)x, (unsigned)((n + x - 1) / x));
}

// Query rows of an fp32 workgroup: 32 (four waves, half the K/V reads per product; at
// d = 128 one workgroup fills a CU's registers) when tiles of 32 rows give 512
// workgroups, two rounds of the CUs, or more, else 16 (eight waves, which split the
// keys further).  Steps at d = 128: 2048 workgroups of 32 rows over 643 keys 342 us, 4096
// of 16 rows 412; a prefill of 32 chunks of 577 rows, 8 heads, 779 against 934; below
// the line 36 of 32 rows over 499 keys 37.1, 72 of 16 rows 26.5; 128 of 32 rows over
// 451 keys 38.2, 256 of 16 rows 27.9.  (A single chunk of 4161 rows and one head, 131 tiles of 32 rows,
// would take 217 us instead of 294.)  units: workgroups per row tile.
inline int f32_rows(long long units, long long rows) { return units * ((rows + 31) / 32) >= 512 ? 32 : 16; }
inline long long f32_groups(long long units, long long rows) {
  const int r = f32_rows(units, rows);
  return units * ((rows + r - 1) / r);
}
// Content keys of an fp32 token-score workgroup.
constexpr int kF32ScoreKeys = 16;

// Whether a decode of `units` (sequence, KV head) pairs of `rows` query rows over `tiles`
// KV tiles in S shards takes workgroups of eight waves and 256 rows instead of four and
// 128 (d = 128).  Eight win by the traffic they save, where their workgroups fill the
// CUs in whole rounds and a sweep is long against its start: step of 8 x 32K (512
// workgroups of 27 tiles) 139.7 us against 145.3 with four waves, four steps of 4 x 32K
// 287 against 300.  With 320 workgroups of 19 tiles (joint pass of 2 x 1156 rows), two
// rounds for 1.25 of work, they take 112 against 98 us, with 4 tiles (8K, 5 shards)
// 35.5 against 33.1 us.
// Their second half of rows has to be there: with 128 rows or fewer in the last tile
// four waves need half the places (units of 23, 64, 125 rows in 2 shards of 17 tiles:
// 56.5, 65, 84-90 us against 65, 76, 92; 260, 300, 384 rows over 26 to 29 tiles: 101,
// 108, 124 against 112, 117, 131; but 160, 200 rows 105, 118 against 102, 117, and 400,
// 450 rows 138, 150-159 against 135, 148).  Only where the four-wave workgroups have a CU each
// anyway, eight keep more tiles in flight: 256 units of 23, 100, 128 rows over 17 to
// 26 tiles, keys not in cache, 40.1, 48, 61.5 us against 41.7, 49.9, 64.0.
inline bool prefers_eight_waves(long long units, int rows, int tiles, int S) {
  const long long groups = units * ((rows + 255) / 256) * S, rounds = (groups + kNumCu - 1) / kNumCu;
  const bool full = (rows - 1) % 256 >= 128 || units * ((rows + 127) / 128) * S <= kNumCu;
  return full && tiles >= 16 * S && 10 * groups >= 9 * kNumCu * rounds;
}

hipError_t launch_prefill_bf16(const PrefillArgs& a, int head_dim, hipStream_t s);
hipError_t launch_escore_bf16(const EscoreArgs& a, int head_dim, hipStream_t s);
hipError_t launch_decode_bf16(const DecodeArgs& a, int head_dim, hipStream_t s);

// Also writes the chunk cache and the key means.
hipError_t launch_prefill_f32(const PrefillArgs& a, float* key_mean, int head_dim, hipStream_t s);
hipError_t launch_escore_f32(const EscoreArgs& a, int head_dim, hipStream_t s);
hipError_t launch_decode_f32(const DecodeArgs& a, int head_dim, hipStream_t s);

// Generic (both element types).
hipError_t launch_merge(const float* o_part, const float* lse_part, void* o_dec, float* lse_dec,
                        int S, int B, int Hq, int Ld, int head_dim, bool bf16, hipStream_t s);

// Stage (b).
struct SelectArgs {
  const void* q_dec;
  const float* key_mean;
  const int32_t* tok_rank;
  float* partial;   // [B][N][Hq*NS] workspace: per (head, row split) chunk-score terms
  float* chunk_score;  // [B][N] or nullptr
  int32_t *chunk_idx, *tok_slot;
  int B, N, C, Hq, Hkv, G, Ld, D, K, Bt, NS;
  int q_rows, q_row0, q_bstride;   // rows averaged into the mean query: rows q_row0.. of q_bstride per sequence
  bool bf16;
  float scale;
};
hipError_t launch_score_select(const SelectArgs& a, hipStream_t s);
hipError_t launch_gather_selected(const void* k_cache, const void* v_cache, const int32_t* chunk_idx,
                                  const int32_t* tok_slot, void* k_sel, void* v_sel, int B, int N, int C, int Hkv,
                                  int K, int Bt, int row_bytes, hipStream_t s);
hipError_t launch_mfma_rate(int n_workgroups, int iters, float* sink, hipStream_t s);

// Full-mask cache construction: joint rows [kept rows ; query rows] per sequence.
struct JointArgs {
  const void *q_pre, *k_cache, *v_cache, *q_qm, *k_qm, *v_qm;
  const int32_t *chunk_idx, *tok_slot;
  void *q_joint, *k_joint, *v_joint;
  void *k_pref, *v_pref;   // optional [B][Hkv][Lj][d] copies of K, V (NULL: skipped)
  int B, N, C, Lq, Lm, Hq, Hkv, G, D, K, Bt, Lj, qm_per_chunk, elem_bytes;
  double rope_base;   // 0: no rotation
};
hipError_t launch_gather_joint(const JointArgs& a, hipStream_t s);
// The end of the prefill: e = sum over the H_q heads of the per-head sums (fixed
// order) and the ranks; the key means from the partial sums of the cache-writing
// workgroups (key_mean NULL: none); the chunk scores (chunk_score NULL: none).
struct RankArgs {
  const float* per_head;   // [B][N][Hq][C]
  float* tok_score;
  int32_t* tok_rank;
  const float* km_part;    // [B][N][Hkv][km_slots][D]
  float* key_mean;
  const float* qm_mass;    // [B][N][Hq][Lq+Lm]
  float* chunk_score;
  int B, N, C, Hq, Hkv, D, km_slots, Lq, Lm;
};
hipError_t launch_head_sum_rank(const RankArgs& a, hipStream_t s);
hipError_t launch_select_ranked(const float* chunk_score, int lowest, const int32_t* tok_rank, int32_t* chunk_idx,
                                int32_t* tok_slot, int B, int N, int C, int K, int Bt, hipStream_t s);
int select_row_splits(int Ld);

}  // namespace pd
