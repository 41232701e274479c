// Stage (b): per-step chunk scores, top-K chunks and the kept tokens of each
// kept chunk, plus the once-per-layer token ranking of stage (a).
//
//   head_sum_rank: grid (b, n; part) -- Eq. 5 scores summed over the heads and the
//                                  token ranks (score desc, index asc), by counting in
//                                  one workgroup per 64 tokens where there are few
//                                  chunks, else by a bitonic sort in one per chunk;
//                                  in workgroups of their own the key means and, from
//                                  the content mass of the q/m rows, the prefill-time
//                                  chunk score;
//   qscore:     grid (b, h, sp) -- by linearity the chunk score splits into
//                                  terms scale * <(1/L_d) sum_{r in sp} q_r, kbar_n>
//                                  over heads and row splits: one workgroup sums
//                                  its rows of one head, then dots with all N
//                                  key means of that head's KV group;
//   gather:     grid (rows)     -- static-selection mode: kept rows copied once
//                                  into a contiguous per-(sequence, KV head) buffer;
//   select:     grid (b, n), up to 64 chunks, or (b, k) -- sums the terms of every
//                                  chunk in a fixed order, ranks the N scores (by
//                                  counting, from 256 chunks on by a bitonic sort in
//                                  LDS) and writes the tokens of its chunk, n if
//                                  kept or the k-th kept one in ascending order, with
//                                  rank < B_tok in ascending slot order (block scan).
// All reductions run in a fixed order, so results are bitwise reproducible.
#include "pd_common.h"
#include "pd_kernels.h"

namespace pd {

// 16 bytes of elements as floats: 8 bf16 or 4 fp32.
template <bool BF16>
struct Vec16 {
  static constexpr int E = BF16 ? 8 : 4;
  __device__ static void load(const void* base, size_t elem_off, float (&v)[E]) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(
        reinterpret_cast<const char*>(base) + elem_off * (BF16 ? 2 : 4));
    if constexpr (BF16) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(w[i]);
    }
  }
};

// Sums in ascending order with many loads in flight before the first add, also where
// fewer terms are left: an unrolled loop would wait for each load of its remainder in
// turn (selection at 8K, 8 terms a thread: 5.3 -> 4.0 us; end of the 16K prefill, 28
// heads and 77 partial key means: 13.9 -> 10.2 us).
// Of p[first], p[first + step], ... below n:
__device__ __forceinline__ float sum_terms(const float* p, int first, int step, int n) {
  constexpr int U = 16;
  float sum = 0.f;
  for (int i = first; i < n; i += U * step) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[min(i + u * step, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) sum += i + u * step < n ? v[u] : 0.f;
  }
  return sum;
}
// Of column `at` of n rows (p, stride and n uniform):
template <int U>
__device__ __forceinline__ float add_rows(float sum, const float* p, uint32_t at, int stride, int first, int n) {
  float v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = (p + (size_t)stride * min(first + u, n - 1))[at];
#pragma unroll
  for (int u = 0; u < U; ++u) sum += first + u < n ? v[u] : 0.f;
  return sum;
}
__device__ __forceinline__ float sum_rows(const float* p, uint32_t at, int stride, int n) {
  float sum = 0.f;
  for (int i = 0; i < n; i += 32)
    sum = n - i > 16 ? add_rows<32>(sum, p, at, stride, i, n) : add_rows<16>(sum, p, at, stride, i, n);
  return sum;
}

__device__ __forceinline__ uint64_t rank_key(float score, int idx) {
  return ((uint64_t)(~float_order_key(score)) << 32) | (uint32_t)idx;
}

// Ascending bitonic sort of P (power of two) keys in LDS, 256 threads.
__device__ void bitonic_sort(uint64_t* keys, int P) {
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < P; i += 256) {
        const int ixj = i ^ j;
        if (ixj > i) {
          const uint64_t a = keys[i], c = keys[ixj];
          const bool up = (i & k) == 0;
          if ((a > c) == up) {
            keys[i] = c;
            keys[ixj] = a;
          }
        }
      }
      __syncthreads();
    }
  }
}

static int next_pow2(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

// Bitonic sort of P = 2^x <= 1024 E keys by 1024 threads; thread t holds keys
// e * 1024 + t, e < E.  Exchanges over less than a wave go by lane shuffles, those
// over 1024 and more stay in the thread, and only the others (10 of the 55 stages at
// 1024 keys) go through LDS, in two buffers of 1024 E keys in turn, so that each
// needs one barrier.
constexpr int kRankThreads = 1024;
template <int E>
__device__ __forceinline__ void sort_keys(uint64_t (&key)[E], uint64_t* lds, int P) {
  const int t = threadIdx.x;
  int buf = 0;
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      uint64_t other[E];
      if (j >= kRankThreads) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          other[e] = key[e];
#pragma unroll
          for (int x = 0; x < E; ++x)
            if (x == (e ^ (j / kRankThreads))) other[e] = key[x];
        }
      } else if (j >= 64) {
        uint64_t* const at = lds + buf * (E * kRankThreads);
        buf ^= 1;
#pragma unroll
        for (int e = 0; e < E; ++e) at[e * kRankThreads + t] = key[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) other[e] = at[e * kRankThreads + (t ^ j)];
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const uint32_t lo = __shfl_xor((uint32_t)key[e], j), hi = __shfl_xor((uint32_t)(key[e] >> 32), j);
          other[e] = ((uint64_t)hi << 32) | lo;
        }
      }
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = e * kRankThreads + t;
        const bool small = ((i & j) == 0) == ((i & k) == 0);   // this place takes the smaller key
        key[e] = (other[e] < key[e]) == small ? other[e] : key[e];
      }
    }
  }
}

// e of one chunk = sum over the H_q heads of the per-head sums (heads in ascending
// order), written out, then every token's rank.
template <int E>
__device__ __forceinline__ void head_sum_rank(const float* ph, float* tok_score, int32_t* tok_rank, int Hq, int C,
                                              int Cpad, uint64_t* lds) {
  uint64_t key[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int j = e * kRankThreads + threadIdx.x;
    key[e] = ~0ull;
    if (j < C) {
      const float x = sum_rows(ph, j, C, Hq);
      tok_score[j] = x;
      key[e] = rank_key(x, j);
    }
  }
  sort_keys<E>(key, lds, Cpad);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * kRankThreads + threadIdx.x;
    if (i < C) tok_rank[(uint32_t)key[e]] = i;
  }
}

// The same for the 64 tokens of one of several slices of a chunk, by counting: a
// token's rank is the number of tokens that come before it.  Every slice sums the
// scores of all tokens; lane l of each wave counts for token l of the slice over
// segments of 64 tokens, whose keys all lanes read together.  Equal scores rank by
// index, so a whole segment below the slice also counts its equal keys and one
// above does not.
constexpr int kSlice = 64;
template <int E>
__device__ __forceinline__ void head_sum_count(const float* ph, float* tok_score, int32_t* tok_rank, int Hq, int C,
                                               int slice, uint32_t* key) {
  const int t = threadIdx.x, lane = t & 63;
  int* const cnt = reinterpret_cast<int*>(key + E * kRankThreads);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int j = e * kRankThreads + t;
    uint32_t k = ~0u;
    if (j < C) {
      const float x = sum_rows(ph, j, C, Hq);
      if (j / kSlice == slice) tok_score[j] = x;
      k = (uint32_t)(rank_key(x, 0) >> 32);
    }
    key[j] = k;
  }
  if (t < kSlice) cnt[t] = 0;
  __syncthreads();
  const uint32_t me = key[slice * kSlice + lane];
  int n = 0;
  for (int seg = __builtin_amdgcn_readfirstlane(t / 64); seg * 64 < C; seg += kRankThreads / 64) {
    const u32x4* const at = reinterpret_cast<const u32x4*>(key + seg * 64);
    if (seg < slice) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const u32x4 k = at[i];
#pragma unroll
        for (int q = 0; q < 4; ++q) n += k[q] <= me;
      }
    } else if (seg > slice) {   // the padding counts nowhere: no key is above it
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const u32x4 k = at[i];
#pragma unroll
        for (int q = 0; q < 4; ++q) n += k[q] < me;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const u32x4 k = at[i];
#pragma unroll
        for (int q = 0; q < 4; ++q) n += k[q] < me || (k[q] == me && 4 * i + q < lane);
      }
    }
  }
  atomicAdd(&cnt[lane], n);
  __syncthreads();
  if (t < kSlice && slice * kSlice + t < C) tok_rank[slice * kSlice + t] = cnt[t];
}

// Prefill-time chunk score of one (b, n) from the per-head content masses of its
// L_q + L_m query and pseudo-label rows: a(r) = (1/H_q) sum_h mass[h][r],
// s = -(1/L_q) sum_{r < L_q} ln a(r) - (1/L_m) sum_{r >= L_q} ln a(r) (the
// second term only when L_m > 0).  Thread t takes rows t, t + 1024, ...; both
// sums are reduced by a fixed tree, so the result is reproducible.
__device__ __forceinline__ void chunk_score_sum(const float* m, float* chunk_score, int Hq, int Lq, int Lm,
                                                float* red) {
  const int R = Lq + Lm, t = threadIdx.x;
  float si = 0.f, sp = 0.f;
  for (int r = t; r < R; r += kRankThreads) {
    const float a = sum_rows(m, r, R, Hq);
    const float nl = -logf(a / Hq);
    if (r < Lq) si += nl;
    else sp += nl;
  }
  red[t] = si;
  red[kRankThreads + t] = sp;
  __syncthreads();
  for (int w = kRankThreads / 2; w > 0; w >>= 1) {
    if (t < w) {
      red[t] += red[t + w];
      red[kRankThreads + t] += red[kRankThreads + t + w];
    }
    __syncthreads();
  }
  if (t == 0) *chunk_score = red[0] / Lq + (Lm > 0 ? red[kRankThreads] / Lm : 0.f);
}

// The end of the prefill, one chunk per blockIdx.x.  The first `slices` of
// blockIdx.y: token scores and ranks (SORT: one, which sorts).  Then one for
// the chunk score, if asked for.  The others, at most 64: the key means
// k-bar[g][d] = (1/C) * the sum of the km_slots partial sums of the cache-writing
// workgroups (fixed order), 1024 of the H_kv*d values at a time.  With every sort
// stage in LDS behind a barrier and the chunk score in a launch of its own, one load
// after the other, the two took 20 and 21 us at 16K; this way the whole prefill of
// 16K went from 539 to 512 us, of 2 x 5 chunks of 777 from 78.5 to 73.2 us.
template <int E, bool SORT>
__global__ __launch_bounds__(kRankThreads) void head_sum_rank_kernel(RankArgs a, int Cpad, int slices) {
  extern __shared__ __attribute__((aligned(16))) uint64_t lds[];
  const size_t bn = (size_t)blockIdx.z * gridDim.x + blockIdx.x;
  if (bn >= (size_t)a.B * a.N) return;   // the grid's last row
  const int first_km = slices + (a.chunk_score ? 1 : 0);
  if ((int)blockIdx.y >= first_km) {
    const int HD = a.Hkv * a.D, n_km = gridDim.y - first_km;
    for (int i = (blockIdx.y - first_km) * kRankThreads + threadIdx.x; i < HD; i += n_km * kRankThreads) {
      const int g = i / a.D, d = i % a.D;
      const float* src = a.km_part + bn * a.Hkv * (size_t)a.km_slots * a.D;
      const float sum = sum_rows(src, (uint32_t)g * a.km_slots * a.D + d, a.D, a.km_slots);
      a.key_mean[bn * HD + i] = sum * (1.0f / a.C);
    }
  } else if ((int)blockIdx.y >= slices) {
    chunk_score_sum(a.qm_mass + bn * a.Hq * (a.Lq + a.Lm), a.chunk_score + bn, a.Hq, a.Lq, a.Lm,
                    reinterpret_cast<float*>(lds));
  } else if constexpr (!SORT) {
    head_sum_count<E>(a.per_head + bn * a.Hq * a.C, a.tok_score + bn * a.C, a.tok_rank + bn * a.C, a.Hq, a.C,
                      blockIdx.y, reinterpret_cast<uint32_t*>(lds));
  } else {
    head_sum_rank<E>(a.per_head + bn * a.Hq * a.C, a.tok_score + bn * a.C, a.tok_rank + bn * a.C, a.Hq, a.C, Cpad,
                     lds);
  }
}

// Counting takes ceil(C / 64) workgroups a chunk where sorting takes one, which
// leaves the chip idle with few chunks and is a chain of 55 stages: 8 chunks of 1024
// 11.5 -> 6.2 us, 10 of 777 12.3 -> 6.9, 4 of 128 5.7 -> 4.7.  Every slice sums all
// heads again, so 256 chunks of 1024 (4096 slices, 8 rounds of the chip's 512) sort:
// 27 us.
constexpr int kCountGroups = 512;
template <int E>
static void launch_head_sum_rank_e(const RankArgs& a, int Cpad, hipStream_t s) {
  const int n_km = a.key_mean ? std::min(64, (a.Hkv * a.D + kRankThreads - 1) / kRankThreads) : 0;
  const int slices = (a.C + kSlice - 1) / kSlice, other = (a.chunk_score ? 1 : 0) + n_km;
  const dim3 bn = grid_xy((long long)a.B * a.N);
  if ((long long)a.B * a.N * slices <= kCountGroups) {
    const size_t bytes = std::max(4 * (E * kRankThreads + kSlice), 8 * kRankThreads);   // keys and counts, or two sums a thread
    hipLaunchKernelGGL((head_sum_rank_kernel<E, false>), dim3(bn.x, slices + other, bn.y), dim3(kRankThreads), bytes, s, a, Cpad, slices);
  } else {
    const size_t bytes = 2 * 8 * E * kRankThreads;   // two buffers of the sort
    hipLaunchKernelGGL((head_sum_rank_kernel<E, true>), dim3(bn.x, 1 + other, bn.y), dim3(kRankThreads), bytes, s, a, Cpad, 1);
  }
}

hipError_t launch_head_sum_rank(const RankArgs& a, hipStream_t s) {
  const int Cpad = next_pow2(a.C);
  if (Cpad <= 1024) launch_head_sum_rank_e<1>(a, Cpad, s);
  else if (Cpad <= 2048) launch_head_sum_rank_e<2>(a, Cpad, s);
  else launch_head_sum_rank_e<4>(a, Cpad, s);
  return hipGetLastError();
}

// Decode rows per score workgroup.
constexpr int kScoreRows = 128;
int select_row_splits(int Ld) { return (Ld + kScoreRows - 1) / kScoreRows; }

// Chunk-score terms of one (b, h, row split): scale * <(1/L_d) sum_r q_r, kbar[b][n][h/G]> for all n.
// Latency-bound (a few KB per workgroup), so every load of a thread is issued
// before the first use: the key means of the first 32 chunks, then the thread's
// share of the rows (fully unrolled).  The row sums are reduced through LDS in
// a fixed order; the dot products run 8 lanes per chunk (D/8 dimensions each),
// reduced by a fixed xor butterfly.  Workgroup id: heads fastest, then row
// split, then sequence.
template <bool BF16, int D>
__device__ __forceinline__ void qscore_terms(const SelectArgs& a, int bid) {
  constexpr int SL = D / 8;
  constexpr int E = Vec16<BF16>::E;
  constexpr int TPR = D / E, NG = 256 / TPR, IT = kScoreRows / NG;
  __shared__ float red[NG * D];
  __shared__ float qp[D];
  const int N = a.N, Hq = a.Hq, NS = a.NS;
  const int h = bid % Hq;
  const int sp = (bid / Hq) % NS;
  const int b = bid / (Hq * NS);
  const int t = threadIdx.x;
  const int r0 = sp * kScoreRows, nr = min(a.q_rows, r0 + kScoreRows) - r0;
  const float* kb = a.key_mean + ((size_t)b * N * a.Hkv + h / a.G) * D;
  const int j = t & 7;
  f32x4 kv[SL / 4];
  {
    const int n = t >> 3;
    if (n < N) {
      const f32x4* kr = reinterpret_cast<const f32x4*>(kb + (size_t)n * a.Hkv * D + j * SL);
#pragma unroll
      for (int i = 0; i < SL / 4; ++i) kv[i] = kr[i];
    }
  }
  const int c = t % TPR, rg = t / TPR;
  const size_t base = (((size_t)b * a.q_bstride + a.q_row0 + r0) * Hq + h) * D + c * E;
  u32x4 w[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int r = rg + it * NG;
    w[it] = r < nr ? *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(a.q_dec) +
                                                      (base + (size_t)r * Hq * D) * (BF16 ? 2 : 4))
                   : u32x4{0u, 0u, 0u, 0u};
  }
  float acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.f;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    if constexpr (BF16) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[2 * i] += __uint_as_float(w[it][i] << 16);
        acc[2 * i + 1] += __uint_as_float(w[it][i] & 0xffff0000u);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] += __uint_as_float(w[it][i]);
    }
  }
#pragma unroll
  for (int e = 0; e < E; ++e) red[rg * D + c * E + e] = acc[e];
  __syncthreads();
  if (t < D) {
    float sum = 0.f;
#pragma unroll
    for (int g = 0; g < NG; ++g) sum += red[g * D + t];
    qp[t] = sum * (1.0f / a.q_rows);
  }
  __syncthreads();
  float q[SL];
#pragma unroll
  for (int i = 0; i < SL; ++i) q[i] = qp[j * SL + i];
  for (int n0 = 0; n0 < N; n0 += 32) {
    const int n = n0 + (t >> 3);
    if (n0 > 0 && n < N) {
      const f32x4* kr = reinterpret_cast<const f32x4*>(kb + (size_t)n * a.Hkv * D + j * SL);
#pragma unroll
      for (int i = 0; i < SL / 4; ++i) kv[i] = kr[i];
    }
    float acc2 = 0.f;
    if (n < N) {
#pragma unroll
      for (int i = 0; i < SL / 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc2 = fmaf(q[4 * i + e], kv[i][e], acc2);
    }
    acc2 += __shfl_xor(acc2, 1);
    acc2 += __shfl_xor(acc2, 2);
    acc2 += __shfl_xor(acc2, 4);
    if (j == 0 && n < N) a.partial[((size_t)b * N + n) * Hq * NS + (size_t)h * NS + sp] = acc2 * a.scale;
  }
}

template <bool BF16, int D>
__global__ __launch_bounds__(256) void qscore_kernel(SelectArgs a) {
  qscore_terms<BF16, D>(a, blockIdx.x);
}

// Chunk scores of sequence b: the T terms of each chunk summed 8 lanes per
// chunk (lane j sums terms j, j+8, ...), then a fixed xor butterfly over the 8
// lanes; keys[n] = rank key of the score (negated when neg), keys past N =
// max.  Writes chunk_score[b][n] when `out` is given.
__device__ void chunk_keys(const float* partial, int b, int N, int T, int Npad, int neg, uint64_t* keys,
                           float* out) {
  const int t = threadIdx.x;
  for (int n = t; n < Npad; n += 256) keys[n] = ~0ull;
  __syncthreads();
  const int j = t & 7;
  for (int n0 = 0; n0 < N; n0 += 32) {
    const int n = n0 + (t >> 3);
    float s = 0.f;
    if (n < N) {
      const float* pr = partial + ((size_t)b * N + n) * T;
      s = sum_terms(pr, j, 8, T);
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    if (j == 0 && n < N) {
      keys[n] = rank_key(neg ? -s : s, n);
      if (out) out[(size_t)b * N + n] = s;
    }
  }
  __syncthreads();
}

// Sum of the values of all lower threads of 256 (within each wave by shuffles, then
// across the 4 waves through wsum).
__device__ __forceinline__ int block_exclusive_sum(int x, int* wsum) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  int pos = inc - x;
  for (int w = 0; w < wv; ++w) pos += wsum[w];
  return pos;
}

// Kept tokens (rank < Bt) of one chunk in ascending order: counts over
// contiguous segments, an exclusive scan, then each segment writes its slots
// (token + 1).  The ranks of a segment are loaded 16 at a time, all in flight
// before the first compare (a plain loop waits for each load in turn).
__device__ void list_tokens(const int32_t* rk, int C, int Bt, int32_t* out, int* wsum) {
  constexpr int U = 16;
  const int t = threadIdx.x;
  const int seg = (C + 255) / 256;
  const int j0 = min(C, t * seg), j1 = min(C, j0 + seg);
  int cnt = 0;
  for (int base = j0; base < j1; base += U) {
    int r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = base + u < j1 ? rk[base + u] : Bt;
#pragma unroll
    for (int u = 0; u < U; ++u) cnt += r[u] < Bt;
  }
  int pos = block_exclusive_sum(cnt, wsum);
  for (int base = j0; base < j1; base += U) {
    int r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = base + u < j1 ? rk[base + u] : Bt;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r[u] < Bt) out[pos++] = base + u + 1;
  }
}

// The same for at most 64 chunks: one workgroup per (sequence, chunk n) loads the
// ranks of its own chunk while it waits for the scores, finds out whether the chunk
// is kept and where, and lists its tokens: one dependent trip to memory less than
// when the chunk is known first (steps: 8K 30.2 -> 29.8 us, 16K 30.4 -> 29.3, 32-row
// block 27.8 -> 26.7).  More chunks: every workgroup sums all scores, so K of them do.
constexpr int kSelectAll = 64;
__global__ __launch_bounds__(256) void select_all_kernel(const float* partial, const int32_t* tok_rank,
                                                          float* chunk_score, int32_t* chunk_idx, int32_t* tok_slot,
                                                          int N, int C, int K, int Bt, int T, int neg) {
  constexpr int U = 16;   // tokens of a thread: C <= 4096
  __shared__ uint64_t keys[kSelectAll];
  __shared__ int wsum[4];
  __shared__ int my_pos;
  const int b = blockIdx.x / N, n = blockIdx.x % N;
  const int t = threadIdx.x;
  const int32_t* rk = tok_rank + ((size_t)b * N + n) * C;
  const int seg = (C + 255) / 256;
  const int j0 = min(C, t * seg), j1 = min(C, j0 + seg);
  int r[U];
#pragma unroll
  for (int u = 0; u < U; ++u) r[u] = j0 + u < j1 ? rk[j0 + u] : Bt;
  chunk_keys(partial, b, N, T, kSelectAll, neg, keys, n == 0 ? chunk_score : nullptr);
  if (t < 64) {
    const uint64_t me = keys[t];
    int rank = 0;
    for (int i = 0; i < N; ++i) rank += keys[i] < me;
    const uint64_t kept = __ballot(t < N && rank < K);
    if (t == n) my_pos = (kept >> n) & 1 ? __popcll(kept & ((1ull << n) - 1)) : -1;
  }
  __syncthreads();
  const int k = my_pos;
  if (k < 0) return;
  if (t == 0) chunk_idx[(size_t)b * K + k] = n;
  int cnt = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) cnt += r[u] < Bt;
  int pos = block_exclusive_sum(cnt, wsum);
  int32_t* out = tok_slot + ((size_t)b * K + k) * Bt;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (r[u] < Bt) out[pos++] = j0 + u + 1;
}

// neg = 1 keeps the K lowest scores instead of the K highest.  One workgroup
// per (sequence, kept chunk k): all compute the chunk ranking, workgroup k then
// lists the kept tokens of the k-th kept chunk.
__global__ __launch_bounds__(256) void select_kernel(const float* partial, const int32_t* tok_rank,
                                                      float* chunk_score, int32_t* chunk_idx, int32_t* tok_slot,
                                                      int N, int C, int K, int Bt, int T, int Npad, int neg) {
  extern __shared__ __attribute__((aligned(16))) uint64_t keys[];
  __shared__ int rankv[256];
  __shared__ int wsum[4];
  __shared__ int my_chunk;
  const int b = blockIdx.x / K, k = blockIdx.x % K;
  const int t = threadIdx.x;
  chunk_keys(partial, b, N, T, Npad, neg, keys, k == 0 ? chunk_score : nullptr);
  if (N <= 256) {
    if (t < N) {
      const uint64_t me = keys[t];
      int r = 0;
      for (int i = 0; i < N; ++i) r += keys[i] < me;
      rankv[t] = r;
    }
    __syncthreads();
    if (t < N && rankv[t] < K) {
      int pos = 0;
      for (int i = 0; i < t; ++i) pos += rankv[i] < K;
      if (pos == k) my_chunk = t;
      if (k == 0) chunk_idx[(size_t)b * K + pos] = t;
    }
  } else {
    bitonic_sort(keys, Npad);
    for (int i = t; i < K; i += 256) {
      const int x = (int)(uint32_t)keys[i];
      int pos = 0;
      for (int j = 0; j < K; ++j) pos += (int)(uint32_t)keys[j] < x;
      if (pos == k) my_chunk = x;
      if (k == 0) chunk_idx[(size_t)b * K + pos] = x;
    }
  }
  __syncthreads();
  list_tokens(tok_rank + ((size_t)b * N + my_chunk) * C, C, Bt, tok_slot + ((size_t)b * K + k) * Bt, wsum);
}

// Selection from T score terms per chunk.
static hipError_t launch_select(const float* partial, const int32_t* tok_rank, float* chunk_score, int32_t* chunk_idx,
                                int32_t* tok_slot, int B, int N, int C, int K, int Bt, int T, int neg,
                                hipStream_t s) {
  // 2^24 workgroups of 256 threads are too many for one dimension.
  if (N <= kSelectAll && (long long)B * N < (1 << 24)) {
    hipLaunchKernelGGL(select_all_kernel, dim3(B * N), dim3(256), 0, s, partial, tok_rank, chunk_score, chunk_idx,
                       tok_slot, N, C, K, Bt, T, neg);
  } else {
    const int Npad = next_pow2(N);
    hipLaunchKernelGGL(select_kernel, dim3(B * K), dim3(256), (size_t)Npad * 8, s, partial, tok_rank, chunk_score,
                       chunk_idx, tok_slot, N, C, K, Bt, T, Npad, neg);
  }
  return hipGetLastError();
}

hipError_t launch_score_select(const SelectArgs& a, hipStream_t s) {
  const dim3 g1(a.B * a.Hq * a.NS);
#define PD_QSCORE(BF, DD) hipLaunchKernelGGL((qscore_kernel<BF, DD>), g1, dim3(256), 0, s, a)
  if (a.D == 128) {
    if (a.bf16) PD_QSCORE(true, 128); else PD_QSCORE(false, 128);
  } else {
    if (a.bf16) PD_QSCORE(true, 64); else PD_QSCORE(false, 64);
  }
#undef PD_QSCORE
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  return launch_select(a.partial, a.tok_rank, a.chunk_score, a.chunk_idx, a.tok_slot, a.B, a.N, a.C, a.K, a.Bt,
                       a.Hq * a.NS, 0, s);
}

// Selection from scores the caller supplies (one term per chunk).
hipError_t launch_select_ranked(const float* chunk_score, int lowest, const int32_t* tok_rank, int32_t* chunk_idx,
                                int32_t* tok_slot, int B, int N, int C, int K, int Bt, hipStream_t s) {
  return launch_select(chunk_score, tok_rank, nullptr, chunk_idx, tok_slot, B, N, C, K, Bt, 1, lowest, s);
}

// Static-selection mode: copy the kept rows of every (sequence, KV head) into a
// contiguous buffer [B][Hkv][K*(1+Bt)][row]: per kept chunk (ascending), its BOS
// row (slot 0) and then its kept slots.  16 bytes per thread.
__global__ __launch_bounds__(256) void gather_selected_kernel(const u32x4* k_cache, const u32x4* v_cache,
                                                               const int32_t* chunk_idx, const int32_t* tok_slot,
                                                               u32x4* k_sel, u32x4* v_sel, size_t total, int N,
                                                               int C1, int Hkv, int K, int Bt, int cpr) {
  const size_t gid = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (gid >= total) return;
  const int n_sel = K * (1 + Bt);
  const int c = (int)(gid % cpr);
  size_t r = gid / cpr;
  const int j = (int)(r % n_sel);
  r /= n_sel;
  const int g = (int)(r % Hkv);
  const int b = (int)(r / Hkv);
  const int kk = j / (1 + Bt), sl = j - kk * (1 + Bt);
  int slot = sl == 0 ? 0 : tok_slot[((size_t)b * K + kk) * Bt + sl - 1];
  int chunk = chunk_idx[(size_t)b * K + kk];
  const bool bad = kCheckIndices && !kept_row_ok(chunk, slot, sl == 0, N, C1 - 1);
  if (bad) chunk = slot = 0;
  const size_t src = ((((size_t)b * N + chunk) * Hkv + g) * C1 + slot) * cpr + c;
  const u32x4 nan4 = {kNanWord, kNanWord, kNanWord, kNanWord};
  k_sel[gid] = bad ? nan4 : k_cache[src];
  v_sel[gid] = bad ? nan4 : v_cache[src];
}

hipError_t launch_gather_selected(const void* k_cache, const void* v_cache, const int32_t* chunk_idx,
                                  const int32_t* tok_slot, void* k_sel, void* v_sel, int B, int N, int C, int Hkv,
                                  int K, int Bt, int row_bytes, hipStream_t s) {
  const int cpr = row_bytes / 16;
  const size_t total = (size_t)B * Hkv * K * (1 + Bt) * cpr;
  const dim3 grid((unsigned)((total + 255) / 256));
  hipLaunchKernelGGL(gather_selected_kernel, grid, dim3(256), 0, s, (const u32x4*)k_cache, (const u32x4*)v_cache,
                     chunk_idx, tok_slot, (u32x4*)k_sel, (u32x4*)v_sel, total, N, C + 1, Hkv, K, Bt, cpr);
  return hipGetLastError();
}

// Full-mask cache construction: the joint rows [kept rows ; L_q query rows] of
// every sequence in the decode layout [B][Lj][H][d], Q and K moved to the
// joint positions by the rotate-half rotary rotation, V copied.  Kept chunk k
// (ascending) moves by k*(C+1), the query rows by (K-1)*(C+1); element i < d/2
// pairs with i + d/2 at frequency base^(-2i/d).  The rotation runs in double
// and is rounded once to the element type.  K and V also go, when asked, to
// the compact prefix layout [B][Hkv][Lj][d] that the decoding steps read.
// One workgroup per joint row: its d/2 cosines and sines (one shift) are
// computed once into LDS, then the threads stream (tensor and head, pair of
// 16-byte chunks c and c + d/2 elements) tasks through them.
template <bool BF16>
__global__ __launch_bounds__(256) void gather_joint_kernel(JointArgs a) {
  constexpr int EPC = BF16 ? 8 : 4;   // elements per 16-byte chunk
  __shared__ double cs_tab[64], sn_tab[64];
  const size_t jrow = blockIdx.x;     // b * Lj + j
  const int j = (int)(jrow % a.Lj), b = (int)(jrow / a.Lj);
  const int C1 = a.C + 1, n_sel = a.K * (1 + a.Bt);
  const bool kept = j < n_sel;
  int kk = a.K - 1, slot = 0;
  size_t n = 0, qm_row = 0;
  bool bad = false;
  if (kept) {
    kk = j / (1 + a.Bt);
    const int sl = j - kk * (1 + a.Bt);
    slot = sl == 0 ? 0 : a.tok_slot[((size_t)b * a.K + kk) * a.Bt + sl - 1];
    int chunk = a.chunk_idx[(size_t)b * a.K + kk];
    bad = kCheckIndices && !kept_row_ok(chunk, slot, sl == 0, a.N, a.C);
    if (bad) chunk = slot = 0;
    n = (size_t)b * a.N + chunk;
  } else {
    qm_row = (a.qm_per_chunk ? (size_t)b * a.N : (size_t)b) * (size_t)(a.Lq + a.Lm) + (j - n_sel);
  }
  const bool rot = a.rope_base > 0.0;
  if (rot) {
    const double delta = (double)kk * C1;
    for (int i = threadIdx.x; i < a.D / 2; i += 256) {
      double sn, cs;
      sincos(delta * pow(a.rope_base, -2.0 * i / a.D), &sn, &cs);
      cs_tab[i] = cs;
      sn_tab[i] = sn;
    }
    __syncthreads();
  }
  const int CP = a.D / EPC / 2;       // chunk pairs per row
  const int tasks = (a.Hq + 2 * a.Hkv) * CP;
  for (int task = threadIdx.x; task < tasks; task += 256) {
    const int cp = task % CP, th = task / CP;
    const int tensor = th < a.Hq ? 0 : (th < a.Hq + a.Hkv ? 1 : 2);   // Q, K, V
    const int head = tensor == 0 ? th : (tensor == 1 ? th - a.Hq : th - a.Hq - a.Hkv);
    const int H = tensor == 0 ? a.Hq : a.Hkv;
    size_t src_el;
    const void* src;
    if (kept) {
      if (tensor == 0) {
        src = a.q_pre;
        src_el = ((n * C1 + slot) * a.Hq + head) * a.D;
      } else {
        src = tensor == 1 ? a.k_cache : a.v_cache;
        src_el = ((n * a.Hkv + head) * C1 + slot) * a.D;
      }
    } else {
      src = tensor == 0 ? a.q_qm : (tensor == 1 ? a.k_qm : a.v_qm);
      src_el = (qm_row * H + head) * a.D;
    }
    void* dst = tensor == 0 ? a.q_joint : (tensor == 1 ? a.k_joint : a.v_joint);
    const size_t dst_el = (jrow * H + head) * a.D;
    const u32x4* s4 = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(src) + src_el * a.elem_bytes);
    u32x4* d4 = reinterpret_cast<u32x4*>(reinterpret_cast<char*>(dst) + dst_el * a.elem_bytes);
    u32x4 lo = s4[cp], hi = s4[cp + CP];
    if (tensor < 2 && rot) {
      float x[2][EPC];
      Vec16<BF16>::load(s4 + cp, 0, x[0]);
      Vec16<BF16>::load(s4 + cp + CP, 0, x[1]);
#pragma unroll
      for (int e = 0; e < EPC; ++e) {
        const int i = cp * EPC + e;   // pair index, 0 .. d/2 - 1
        const double cs = cs_tab[i], sn = sn_tab[i];
        const double p0 = x[0][e], p1 = x[1][e];
        x[0][e] = (float)(p0 * cs - p1 * sn);
        x[1][e] = (float)(p1 * cs + p0 * sn);
      }
      if constexpr (BF16) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          lo[q] = pack_bf16x2(x[0][2 * q], x[0][2 * q + 1]);
          hi[q] = pack_bf16x2(x[1][2 * q], x[1][2 * q + 1]);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          lo[q] = __float_as_uint(x[0][q]);
          hi[q] = __float_as_uint(x[1][q]);
        }
      }
    }
    if (bad) lo = hi = u32x4{kNanWord, kNanWord, kNanWord, kNanWord};
    d4[cp] = lo;
    d4[cp + CP] = hi;
    void* pref = tensor == 1 ? a.k_pref : (tensor == 2 ? a.v_pref : nullptr);
    if (pref) {
      const size_t p_el = (((size_t)b * a.Hkv + head) * a.Lj + j) * a.D;
      u32x4* p4 = reinterpret_cast<u32x4*>(reinterpret_cast<char*>(pref) + p_el * a.elem_bytes);
      p4[cp] = lo;
      p4[cp + CP] = hi;
    }
  }
}

hipError_t launch_gather_joint(const JointArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)((size_t)a.B * a.Lj));
  if (a.elem_bytes == 2) hipLaunchKernelGGL(gather_joint_kernel<true>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(gather_joint_kernel<false>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Split-S merge: O = sum_s 2^(lse_s - M) O_s / sum_s 2^(lse_s - M), in ascending shard
// order.  U > 0: at most U shards, whose LSE and rows are all loaded before the first
// use: one trip to memory (17 shards of 1024 rows 5.8 -> 4.2 us, 4 shards of 8192 rows
// 4.8 -> 4.5).  U = 0: any number, first the LSE, then the rows, 8 at a time.
template <bool BF16, int U>
__global__ __launch_bounds__(256) void merge_kernel(const float* o_part, const float* lse_part, void* o_dec,
                                                     float* lse_dec, int S, int B, int Hq, int Ld, int D) {
  const int TPR = D / 4;
  const size_t gid = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t rows = (size_t)B * Hq * Ld;
  const size_t row = gid / TPR;
  if (row >= rows) return;
  const int c = gid % TPR;
  constexpr int V = U > 0 ? U : 8;
  float l[V];
  f32x4 v[V];
  auto load_lse = [&](int s0) {
#pragma unroll
    for (int u = 0; u < V; ++u) l[u] = lse_part[min(s0 + u, S - 1) * rows + row];
  };
  auto load_rows = [&](int s0) {
#pragma unroll
    for (int u = 0; u < V; ++u) v[u] = *reinterpret_cast<const f32x4*>(o_part + (min(s0 + u, S - 1) * rows + row) * D + 4 * c);
  };
  float M = -INFINITY, W = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  auto maximum = [&]() {
#pragma unroll
    for (int u = 0; u < V; ++u) M = fmaxf(M, l[u]);
  };
  auto add = [&](int s0) {
#pragma unroll
    for (int u = 0; u < V; ++u) {
      if (s0 + u < S) {
        const float w = fast_exp2(l[u] - M);
        W += w;
        acc += w * v[u];
      }
    }
  };
  if constexpr (U > 0) {
    load_lse(0);
    load_rows(0);
    // Issued here: the compiler would sink each load to its use.
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < V; ++u) asm volatile("" ::"v"(v[u]));
    maximum();
    add(0);
  } else {
    for (int s0 = 0; s0 < S; s0 += V) {
      load_lse(s0);
      maximum();
    }
    for (int s0 = 0; s0 < S; s0 += V) {
      load_lse(s0);
      load_rows(s0);
      add(s0);
    }
  }
  const float inv = 1.0f / W;
  // row = (b*Hq + h)*Ld + r  ->  o_dec[b][r][h][:]
  const int r = row % Ld;
  const size_t bh = row / Ld;
  const int h = bh % Hq;
  const size_t b = bh / Hq;
  const size_t out = ((b * Ld + r) * Hq + h) * D + 4 * c;
  if constexpr (BF16) {
    u32x2 v = {pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv)};
    *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(o_dec) + out) = v;
  } else {
    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(o_dec) + out) = acc * inv;
  }
  if (lse_dec && c == 0) lse_dec[row] = (M + __log2f(W)) * kLn2;
}

hipError_t launch_merge(const float* o_part, const float* lse_part, void* o_dec, float* lse_dec, int S, int B,
                        int Hq, int Ld, int head_dim, bool bf16, hipStream_t s) {
  const size_t threads = (size_t)B * Hq * Ld * (head_dim / 4);
  const dim3 grid((unsigned)((threads + 255) / 256));
#define PD_MERGE(BF, U) \
  hipLaunchKernelGGL((merge_kernel<BF, U>), grid, dim3(256), 0, s, o_part, lse_part, o_dec, lse_dec, S, B, Hq, Ld, head_dim)
#define PD_MERGE_UP_TO(U) \
  if (S <= U || U == 0) {   \
    if (bf16) PD_MERGE(true, U); else PD_MERGE(false, U); \
    return hipGetLastError(); \
  }
  PD_MERGE_UP_TO(4)
  PD_MERGE_UP_TO(8)
  PD_MERGE_UP_TO(16)
  PD_MERGE_UP_TO(24)
  PD_MERGE_UP_TO(0)
#undef PD_MERGE_UP_TO
#undef PD_MERGE
  return hipGetLastError();
}

}  // namespace pd
