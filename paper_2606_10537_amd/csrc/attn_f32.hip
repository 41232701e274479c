// fp32 attention kernels (stage a prefill, Eq. 5 first sum, stage c decode).
//
// The products run on v_mfma_f32_16x16x4_f32 (fp32 operands, products and sums):
// 256 FLOP per clock and CU, twice what unpacked VALU FMAs reach, and a wave's
// operands fit its registers.  (One thread per query row with q and the output
// row in registers, the layout before, spilled at d = 128 and left most CUs
// idle: 964 us for a 16-head decode of 72 x 499 rows, 125 us for the prefill of
// four chunks of 177 rows, d = 64.)
//
// fp32 calls are small, so what counts is the depth of one workgroup: its waves
// share 16 QB query rows and split the keys, 32 at a time and wave; every wave
// keeps its own online softmax, and the partial rows are merged through LDS at
// the end, in a fixed order.  No key is read by two waves of a workgroup, so K and
// V go from memory straight to registers: the next K block while this one's
// softmax and P*V run, the next V block during the next S.  QB = 2 halves the
// K/V traffic per product and is taken when it still fills the CUs; QB = 1 with
// twice the waves otherwise.
//
// Operand layouts of 16x16x4 (lane q = lane % 16, g = lane / 16): A holds row q,
// B column q, both at k = g; element r of the result is row 4 g + r of column q.
//   S^T = K Q^T: four k steps share one 16-byte read of either operand: step e of
//     group s takes d = 16 s + 4 g + e.  The result is keys 4 g + r of query q.
//   O^T += V^T P^T: step r takes keys 4 g + r, so P^T is the result of S^T as it
//     stands.  The A rows of d block (c, e) are d = 64 c + 4 q + e: one 16-byte
//     read of a V row serves four blocks, and o[4 c + e][r] is d = 64 c + 16 g +
//     4 r + e, four neighbours over e.
#include "pd_common.h"
#include "pd_kernels.h"

namespace pd {

constexpr int kF32Table = 512;   // key rows whose addresses are resident at a time

__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 mfma16x16x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Lanes q, q + 16, q + 32, q + 48 hold the same query.
__device__ __forceinline__ float max_over_groups(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float sum_over_groups(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

template <int D, int QB, int NW>
struct F32Lds {
  static constexpr int R = 16 * QB, P = D + 4;   // rows of a workgroup; padded row of partial outputs
  const float *k[kF32Table], *v[kF32Table];
  float o[NW][R][P];
  float m[NW][R], l[NW][R], mass[NW][R];
};

// Attention of the workgroup's R query rows over keys [j0, j1).  qrow(i) is the
// pointer of row i or NULL (zeros), key(j, k, v) gives the K and V rows of key j,
// range(i, lo, hi) the keys whose mass is counted for row i (MASS).  Then
// out(i, d, l, x) receives four merged output values, times the weight sum l, of row i
// from d on, and row(i, m, l, mass) its log2-domain maximum, weight sum and mass.
template <int D, int QB, int NW, bool MASS, class QRow, class Key, class Range, class Out, class Row>
__device__ __forceinline__ void attend_f32(F32Lds<D, QB, NW>& lds, int j0, int j1, float scale_log2, QRow&& qrow,
                                           Key&& key, Range&& range, Out&& out, Row&& row) {
  constexpr int KS = D / 16, DC = D / 64, R = 16 * QB;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane & 15, g = lane >> 4;
  f32x4 qf[QB][KS], o[QB][4 * DC];
  float m[QB], l[QB], mass[QB];
  int lo[QB], hi[QB];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const float* src = qrow(16 * b + q);
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[b][s] = src ? ld4(src + 16 * s + 4 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4 * DC; ++i) o[b][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    m[b] = kNoMax;
    l[b] = mass[b] = 0.f;
    if constexpr (MASS) range(16 * b + q, lo[b], hi[b]);
  }
  for (int c0 = j0; c0 < j1; c0 += kF32Table) {
    const int nk = min(kF32Table, j1 - c0);
    if (c0 > j0) __syncthreads();   // the previous addresses are no longer read
    for (int i = tid; i < kF32Table; i += 64 * NW) {
      const float *kp = nullptr, *vp = nullptr;
      if (i < nk) key(c0 + i, kp, vp);
      lds.k[i] = kp;
      lds.v[i] = vp;
    }
    __syncthreads();
    // 32 keys i0 .. i0+31 of the table; rows past the end have no address and are zero.
    f32x4 kf[2][KS], vf[2][4][DC];
    auto load_k = [&](int i0) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float* p = lds.k[i0 + 16 * h + q];
#pragma unroll
        for (int s = 0; s < KS; ++s) kf[h][s] = p ? ld4(p + 16 * s + 4 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    };
    auto load_v = [&](int i0) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float* p = lds.v[i0 + 16 * h + 4 * g + r];
#pragma unroll
          for (int c = 0; c < DC; ++c) vf[h][r][c] = p ? ld4(p + 64 * c + 4 * q) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    int i0 = 32 * wave;
    if (i0 < nk) {
      load_k(i0);
      load_v(i0);
    }
    for (; i0 < nk; i0 += 32 * NW) {
      f32x4 s[2][QB];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int b = 0; b < QB; ++b) s[h][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int b = 0; b < QB; ++b) s[h][b] = mfma16x16x4(kf[h][ks][e], qf[b][ks][e], s[h][b]);
      const int next = i0 + 32 * NW;
      if (next < nk) load_k(next);
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        float mt = -INFINITY;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            s[h][b][r] = i0 + 16 * h + 4 * g + r < nk ? s[h][b][r] * scale_log2 : -INFINITY;
            mt = fmaxf(mt, s[h][b][r]);
          }
        mt = max_over_groups(mt);
        if (__ballot(mt > m[b])) {
          const float mn = fmaxf(m[b], mt), a = fast_exp2(m[b] - mn);
          m[b] = mn;
          l[b] *= a;
          mass[b] *= a;
#pragma unroll
          for (int i = 0; i < 4 * DC; ++i) o[b][i] *= a;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float p = fast_exp2(s[h][b][r] - m[b]);
            s[h][b][r] = p;
            l[b] += p;
            if constexpr (MASS) {
              const int j = c0 + i0 + 16 * h + 4 * g + r;
              mass[b] += j >= lo[b] && j < hi[b] ? p : 0.f;
            }
          }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < DC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int b = 0; b < QB; ++b) o[b][4 * c + e] = mfma16x16x4(vf[h][r][c][e], s[h][b][r], o[b][4 * c + e]);
      if (next < nk) load_v(next);
    }
  }
  // Merge the waves' partial rows: O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w.
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const int i = 16 * b + q;
    const float lt = sum_over_groups(l[b]), mst = sum_over_groups(mass[b]);
    if (g == 0) {
      lds.m[wave][i] = m[b];
      lds.l[wave][i] = lt;
      lds.mass[wave][i] = mst;
    }
#pragma unroll
    for (int c = 0; c < DC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(&lds.o[wave][i][64 * c + 16 * g + 4 * r]) =
            f32x4{o[b][4 * c][r], o[b][4 * c + 1][r], o[b][4 * c + 2][r], o[b][4 * c + 3][r]};
  }
  __syncthreads();
  for (int u = tid; u < R * (D / 4); u += 64 * NW) {
    const int i = u / (D / 4), d = 4 * (u % (D / 4));
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, lds.m[w][i]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float L = 0.f, ms = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      // A wave without keys, or with scores of -inf only, has no weight, whatever M is.
      const float a = lds.l[w][i] == 0.f ? 0.f : fast_exp2(lds.m[w][i] - M);
      acc += a * *reinterpret_cast<const f32x4*>(&lds.o[w][i][d]);
      L += a * lds.l[w][i];
      ms += a * lds.mass[w][i];
    }
    out(i, d, L, acc);
    if (d == 0) row(i, M, L, ms);
  }
}

// ---------------------------------------------------------------------------
// Prefill.  Workgroups [0, total): (b, n, h, tile of 16 QB rows).  The others,
// one per (b, n, kv head): the chunk's cache rows and, summed in a fixed order,
// its key mean.
template <int D, int QB, int NW>
__global__ __launch_bounds__(64 * NW) void prefill_f32_kernel(PrefillArgs p, float* key_mean) {
  __shared__ __attribute__((aligned(16))) F32Lds<D, QB, NW> lds;
  const float* q_pre = reinterpret_cast<const float*>(p.q_pre);
  const float* k_pre = reinterpret_cast<const float*>(p.k_pre);
  const float* v_pre = reinterpret_cast<const float*>(p.v_pre);
  const int C1 = p.C + 1, tid = threadIdx.x;
  const uint32_t bid = block_id(), total = p.total;
  if (bid >= total) {
    if (bid - total >= (uint32_t)(p.B * p.N * p.Hkv)) return;   // the grid's last row
    constexpr int CH = D / 4, NG = 64 * NW / CH;   // 16-byte chunks of a row; rows in flight
    const size_t bng = bid - total, chunk = bng / p.Hkv;
    const int g = (int)(bng % p.Hkv), c = tid % CH, rg = tid / CH;
    float* kc = reinterpret_cast<float*>(p.k_cache) + bng * C1 * D + 4 * c;
    float* vc = reinterpret_cast<float*>(p.v_cache) + bng * C1 * D + 4 * c;
    const size_t src = (chunk * C1 * p.Hkv + g) * D + 4 * c;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int r = rg; r < C1; r += NG) {
      const size_t at = src + (size_t)r * p.Hkv * D;
      const f32x4 k = ld4(k_pre + at);
      *reinterpret_cast<f32x4*>(kc + (size_t)r * D) = k;
      *reinterpret_cast<f32x4*>(vc + (size_t)r * D) = ld4(v_pre + at);
      if (r >= 1) sum += k;   // content rows only
    }
    *reinterpret_cast<f32x4*>(&lds.o[0][0][0] + rg * D + 4 * c) = sum;
    static_assert(NG * D <= NW * 16 * QB * (D + 4), "partial sums fit");
    __syncthreads();
    if (tid < D) {
      float s = 0.f;
      for (int r = 0; r < NG; ++r) s += (&lds.o[0][0][0])[r * D + tid];
      key_mean[bng * D + tid] = s * (1.0f / p.C);
    }
    return;
  }
  const float* q_qm = reinterpret_cast<const float*>(p.q_qm);
  const float* k_qm = reinterpret_cast<const float*>(p.k_qm);
  const float* v_qm = reinterpret_cast<const float*>(p.v_qm);
  float* o = reinterpret_cast<float*>(p.o);
  int lid = xcd_remap(bid, p.total);
  const int rb = lid % p.n_qt;
  lid /= p.n_qt;
  const int h = lid % p.Hq;
  lid /= p.Hq;
  const int n = lid % p.N;
  const int b = lid / p.N;
  const int g = h / p.G;
  const size_t chunk = (size_t)b * p.N + n;
  const size_t qm_base = (p.qm_per_chunk ? chunk : (size_t)b) * (size_t)(p.Lq + p.Lm);
  const size_t hb = chunk * p.Hq + h;
  const int row0 = rb * 16 * QB;
  const int qc_lo = C1, qc_hi = C1 + p.Lq;
  attend_f32<D, QB, NW, true>(
      lds, 0, p.Sc, p.scale_log2,
      [&](int i) -> const float* {
        const int row = row0 + i;
        if (row < C1) return q_pre + ((chunk * C1 + row) * p.Hq + h) * D;
        return row < p.Sc ? q_qm + ((qm_base + (row - C1)) * p.Hq + h) * D : nullptr;
      },
      [&](int j, const float*& k, const float*& v) {
        const bool own = j < C1;
        const size_t at = own ? ((chunk * C1 + j) * p.Hkv + g) * D : ((qm_base + (j - C1)) * p.Hkv + g) * D;
        k = (own ? k_pre : k_qm) + at;
        v = (own ? v_pre : v_qm) + at;
      },
      // The query columns for the BOS and content rows (second sum of Eq. 5), the content columns for the
      // query and pseudo-label rows when the chunk score is asked for.
      [&](int i, int& lo, int& hi) {
        lo = row0 + i < C1 ? qc_lo : 1;
        hi = row0 + i < C1 ? qc_hi : (p.qm_mass ? C1 : 1);
      },
      [&](int i, int d, float l, f32x4 x) {
        if (row0 + i < p.Sc) *reinterpret_cast<f32x4*>(o + ((chunk * p.Sc + row0 + i) * p.Hq + h) * D + d) = x * (1.0f / l);
      },
      [&](int i, float m, float l, float mass) {
        const int row = row0 + i;
        if (row >= p.Sc) return;
        if (row >= 1 && row < C1) p.part_i[hb * p.C + (row - 1)] = mass * (1.0f / l);
        if (row >= qc_lo && row < qc_hi) p.lse_q[hb * p.Lq + (row - qc_lo)] = m + __log2f(l);
        if (p.qm_mass && row >= C1) p.qm_mass[hb * (p.Lq + p.Lm) + (row - C1)] = mass * (1.0f / l);
      });
}

// ---------------------------------------------------------------------------
// Eq. 5, first sum: one wave per (b, n, h, 16 content keys).  S = Q_q K_c^T with
// the query rows as A (16 per step) and the keys as B, so a lane holds one key and
// four query rows; each key's mass exp2(S*scale - lse2(row)) is summed over the
// rows and added to the head's second sum (or replaces it for the query-to-chunk
// score); head_sum_rank_kernel sums the heads.
template <int D>
__global__ __launch_bounds__(64) void escore_f32_kernel(EscoreArgs p) {
  constexpr int KS = D / 16;
  const float* q_qm = reinterpret_cast<const float*>(p.q_qm);
  const float* k_cache = reinterpret_cast<const float*>(p.k_cache);
  const int lane = threadIdx.x, q = lane & 15, g = lane >> 4;
  const uint32_t bid = block_id();
  if (bid >= (uint32_t)(p.B * p.N * p.Hq * p.n_cb)) return;   // the grid's last row
  const size_t bnh = bid / p.n_cb;   // (b * N + n) * Hq + h
  const int cb = bid % p.n_cb, h = (int)(bnh % p.Hq);
  const size_t bn = bnh / p.Hq;
  const int b = (int)(bn / p.N);
  const size_t qm_base = (p.qm_per_chunk ? bn : (size_t)b) * (size_t)(p.Lq + p.Lm);
  const float* lse = p.lse_q + bnh * p.Lq;
  const int j = cb * kF32ScoreKeys + q;
  const float* kp = j < p.C ? k_cache + ((bn * p.Hkv + h / p.G) * (p.C + 1) + 1 + j) * D : nullptr;
  f32x4 kf[KS], qa[KS], qn[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) kf[s] = kp ? ld4(kp + 16 * s + 4 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
  float ln[4], lc[4];
  auto load = [&](int r0, f32x4 (&x)[KS], float (&le)[4]) {
    const float* src = r0 + q < p.Lq ? q_qm + ((qm_base + r0 + q) * p.Hq + h) * D : nullptr;
#pragma unroll
    for (int s = 0; s < KS; ++s) x[s] = src ? ld4(src + 16 * s + 4 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 4; ++r) le[r] = r0 + 4 * g + r < p.Lq ? lse[r0 + 4 * g + r] : INFINITY;
  };
  load(0, qn, ln);
  float acc = 0.f;
  for (int r0 = 0; r0 < p.Lq; r0 += 16) {
#pragma unroll
    for (int s = 0; s < KS; ++s) qa[s] = qn[s];
#pragma unroll
    for (int r = 0; r < 4; ++r) lc[r] = ln[r];
    if (r0 + 16 < p.Lq) load(r0 + 16, qn, ln);
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;   // two chains
#pragma unroll
    for (int s = 0; s < KS; s += 2)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s0 = mfma16x16x4(qa[s][e], kf[s][e], s0);
        s1 = mfma16x16x4(qa[s + 1][e], kf[s + 1][e], s1);
      }
#pragma unroll
    for (int r = 0; r < 4; ++r) acc += fast_exp2((s0[r] + s1[r]) * p.scale_log2 - lc[r]);
  }
  acc = sum_over_groups(acc);
  float* ph = p.part_io + bnh * p.C;
  if (g == 0 && j < p.C) ph[j] = p.q2c ? acc : ph[j] + acc;
}

// ---------------------------------------------------------------------------
// Decode.  Workgroup = (b, kv head, tile of 16 QB of the group's G L_d query
// rows, KV shard); query row rho of the group is head g*G + rho / L_d, decode row
// rho % L_d.  Shards are cut at multiples of 32 keys.
template <int D, int QB, int NW>
__global__ __launch_bounds__(64 * NW) void decode_f32_kernel(DecodeArgs p) {
  __shared__ __attribute__((aligned(16))) F32Lds<D, QB, NW> lds;
  __shared__ int bad_index;   // checking build: some kept row of this shard was out of range
  const float* q_dec = reinterpret_cast<const float*>(p.q_dec);
  const float* k_dec = reinterpret_cast<const float*>(p.k_dec);
  const float* v_dec = reinterpret_cast<const float*>(p.v_dec);
  const float* k_cache = reinterpret_cast<const float*>(p.k_cache);
  const float* v_cache = reinterpret_cast<const float*>(p.v_cache);
  const float* k_static = reinterpret_cast<const float*>(p.k_static);
  const float* v_static = reinterpret_cast<const float*>(p.v_static);

  if (block_id() >= (uint32_t)p.total) return;   // the grid's last row
  int lid = xcd_remap(block_id(), p.total);
  const int sp = lid % p.S;
  lid /= p.S;
  const int rb = lid % p.n_qt;
  lid /= p.n_qt;
  const int g = lid % p.Hkv;
  const int b = lid / p.Hkv;
  const int C1 = p.C + 1, GL = p.G * p.Ld;
  const int n_sel = p.n_sel;
  const int L_kv = n_sel + p.n_static + p.Ld;
  const int n_kvt = (L_kv + 31) / 32;
  const int j0 = 32 * (int)(((long long)n_kvt * sp) / p.S);
  const int j1 = min(L_kv, 32 * (int)(((long long)n_kvt * (sp + 1)) / p.S));
  const size_t cache_bg = ((size_t)b * p.N * p.Hkv + g) * C1;
  const int32_t* cidx = p.chunk_idx + (size_t)b * p.K;
  const int32_t* tslot = p.tok_slot + (size_t)b * p.K * p.Bt;
  if (kCheckIndices && threadIdx.x == 0) bad_index = 0;
  if (kCheckIndices) __syncthreads();
  const int row0 = rb * 16 * QB;
  auto where = [&](int i, int& hq, int& r) {
    hq = g * p.G + (row0 + i) / p.Ld;
    r = (row0 + i) % p.Ld;
  };
  attend_f32<D, QB, NW, false>(
      lds, j0, j1, p.scale_log2,
      [&](int i) -> const float* {
        if (row0 + i >= GL) return nullptr;
        int hq, r;
        where(i, hq, r);
        return q_dec + (((size_t)b * p.Ld + r) * p.Hq + hq) * D;
      },
      [&](int j, const float*& k, const float*& v) {
        if (j < n_sel && p.compact) {
          const size_t at = (((size_t)b * p.Hkv + g) * n_sel + j) * D;
          k = k_cache + at;
          v = v_cache + at;
        } else if (j < n_sel) {
          const int c = j / (1 + p.Bt), s = j - c * (1 + p.Bt);
          int slot = s == 0 ? 0 : tslot[c * p.Bt + s - 1];
          int chunk = cidx[c];
          if (kCheckIndices && !kept_row_ok(chunk, slot, s == 0, p.N, p.C)) {
            chunk = 0;
            slot = 0;
            bad_index = 1;
          }
          const size_t at = (cache_bg + (size_t)chunk * p.Hkv * C1 + slot) * D;
          k = k_cache + at;
          v = v_cache + at;
        } else {
          const bool stat = j < n_sel + p.n_static;
          const size_t at = stat ? (((size_t)b * p.Ls + (j - n_sel)) * p.Hkv + g) * D
                                 : (((size_t)b * p.Ld + (j - n_sel - p.n_static)) * p.Hkv + g) * D;
          // Both values before one is selected: the compiler would select among the
          // captures' addresses, which puts them into scratch memory.
          const float *ks = uniform(k_static), *kd = uniform(k_dec), *vs = uniform(v_static), *vd = uniform(v_dec);
          k = (stat ? ks : kd) + at;
          v = (stat ? vs : vd) + at;
        }
      },
      [](int, int&, int&) {},
      [&](int i, int d, float l, f32x4 x) {
        if (row0 + i >= GL) return;
        int hq, r;
        where(i, hq, r);
        // No weight in this shard (every score -inf): zeros of weight zero in the merge.
        x *= p.S > 1 && l == 0.f ? 0.f : 1.0f / l;
        if (kCheckIndices && bad_index) x = f32x4{1.f, 1.f, 1.f, 1.f} * __uint_as_float(kNanWord);
        float* dst = p.S == 1 ? reinterpret_cast<float*>(p.o_dec) + (((size_t)b * p.Ld + r) * p.Hq + hq) * D
                              : p.o_part + ((((size_t)sp * p.B + b) * p.Hq + hq) * p.Ld + r) * D;
        *reinterpret_cast<f32x4*>(dst + d) = x;
      },
      [&](int i, float m, float l, float) {
        if (row0 + i >= GL) return;
        int hq, r;
        where(i, hq, r);
        float lse2 = m + __log2f(l);
        if (kCheckIndices && bad_index) lse2 = __uint_as_float(kNanWord);
        if (p.S == 1) {
          if (p.lse_dec) p.lse_dec[((size_t)b * p.Hq + hq) * p.Ld + r] = lse2 * kLn2;
        } else {
          p.lse_part[(((size_t)sp * p.B + b) * p.Hq + hq) * p.Ld + r] = lse2;
        }
      });
}

// ---------------------------------------------------------------------------
template <int D>
static hipError_t prefill_f32_d(PrefillArgs a, float* key_mean, hipStream_t s) {
  const int units = a.B * a.N * a.Hq, copies = a.B * a.N * a.Hkv;   // the host has bounded the grid
  const bool wide = f32_rows(units, a.Sc) == 32;
  a.n_qt = wide ? (a.Sc + 31) / 32 : (a.Sc + 15) / 16;
  a.total = units * a.n_qt;
  if (wide) hipLaunchKernelGGL((prefill_f32_kernel<D, 2, 4>), grid_xy((long long)a.total + copies), dim3(256), 0, s, a, key_mean);
  else hipLaunchKernelGGL((prefill_f32_kernel<D, 1, 8>), grid_xy((long long)a.total + copies), dim3(512), 0, s, a, key_mean);
  return hipGetLastError();
}
hipError_t launch_prefill_f32(const PrefillArgs& a, float* key_mean, int head_dim, hipStream_t s) {
  return head_dim == 128 ? prefill_f32_d<128>(a, key_mean, s) : prefill_f32_d<64>(a, key_mean, s);
}

hipError_t launch_escore_f32(const EscoreArgs& a, int head_dim, hipStream_t s) {
  EscoreArgs e = a;
  e.n_cb = (a.C + kF32ScoreKeys - 1) / kF32ScoreKeys;
  const dim3 grid = grid_xy((long long)a.B * a.N * a.Hq * e.n_cb);
  if (head_dim == 128) hipLaunchKernelGGL(escore_f32_kernel<128>, grid, dim3(64), 0, s, e);
  else hipLaunchKernelGGL(escore_f32_kernel<64>, grid, dim3(64), 0, s, e);
  return hipGetLastError();
}

template <int D>
static hipError_t decode_f32_d(DecodeArgs a, hipStream_t s) {
  const int units = a.B * a.Hkv, rows = a.G * a.Ld;
  const bool wide = f32_rows((long long)units * a.S, rows) == 32;
  a.n_qt = wide ? (rows + 31) / 32 : (rows + 15) / 16;
  a.total = units * a.n_qt * a.S;
  if (wide) hipLaunchKernelGGL((decode_f32_kernel<D, 2, 4>), grid_xy(a.total), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((decode_f32_kernel<D, 1, 8>), grid_xy(a.total), dim3(512), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_decode_f32(const DecodeArgs& a, int head_dim, hipStream_t s) {
  return head_dim == 128 ? decode_f32_d<128>(a, s) : decode_f32_d<64>(a, s);
}

}  // namespace pd
