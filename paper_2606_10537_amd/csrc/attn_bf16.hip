// bf16 attention kernels for gfx950: chunk prefill (stage a) and sparse decode
// attention (stage c).
//
//   * a wave takes 32 query rows, d = 64 or 128, for the whole sweep over its KV
//     tiles of 64 rows; Q stays in registers;
//   * K/V tiles go from HBM straight into LDS with global_load_lds_dwordx4 (no
//     register staging), the next ones while one is multiplied, each DMA issued
//     between two MFMAs;
//   * both tiles are stored in 64-byte chunk groups with an XOR swizzle
//     (tile_off), so that the K fragment reads (ds_read_b128) and the
//     transposing V reads (ds_read_b64_tr_b16) are free of bank conflicts and
//     every fragment address is a per-lane base plus an immediate offset;
//   * S^T = K Q^T and O^T += V^T P^T run on v_mfma_f32_32x32x16_bf16 with
//     fp32 accumulation;
//   * online softmax in the log2 domain, lazy rescaling of the running output
//     (only when a row maximum grows by more than 2^8), P rounded to bf16.
//
// What bounds it.  A tile costs a wave 1088 matrix cycles and about 650 vector
// cycles (32 exponentials at 8, 100 others at 4-5), so the two waves of a SIMD
// have to be in different parts of their tiles.  Two sweeps do that.  sweep_pair:
// two workgroups of four waves on a CU, one wave of each on a SIMD, drift apart by
// themselves, and one's start and end cost nothing while the other computes.
// sweep_pingpong: one workgroup of eight waves whose halves run half a tile apart,
// held there by barriers; each tile in LDS serves twice the rows (half the
// traffic from L2), but the start, 8 us, and the end of a workgroup are bare.  The
// matrix cores are busy 42 % (decode of 8 x 32K) and 47 % (prefill) of the cycles;
// the waves issue 34 and 39 % of their time, wait 36 and 39 % for an issue slot and 29
// and 21 % for a barrier, a DMA or LDS data.  By the cycle counters the clock is
// 2.2 GHz in that decode and 1.6 in that prefill, of 2.4.  Against
// one workgroup of eight waves with one barrier a tile (before): prefill of 8 x
// 32K 14.67 -> 14.05 ms, of 16K 595 -> 539 us, joint pass of 2 x 1156 rows 86 ->
// 67 us, step of 8 x 32K 142.7 -> 139.7 us.
//
// Computing S transposed makes the MFMA output layout (each lane: one query,
// 16 keys) directly usable as the B operand of the P*V product.  The matching
// V^T operand (each lane: one d column, 8 keys) is produced from row-major V
// by ds_read_b64_tr_b16: within a group of 16 lanes, lane j receives element
// m of the 4 elements read by lane 4m + j/4, element j % 4.  If lane k of the
// group points at V[key0 + k/4][d0 + 4(k%4)], lane j therefore receives
// V[key0 + m][d0 + j], m = 0..3: four consecutive keys of one column.
#include <algorithm>
#include <utility>

#include "pd_common.h"
#include "pd_kernels.h"

namespace pd {

// f(0), f(1), ... f(N-1) with compile-time arguments.
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>());
}

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
#define PD_LDS __attribute__((address_space(3)))
#define PD_INLINE __attribute__((always_inline))   // of a lambda: a call would put its captures into scratch memory

// NW: waves per workgroup.  4: two workgroups per CU, two K/V tiles resident in
// each; 8: one workgroup per CU, four tiles resident.
template <int D, int NW_ = 4>
struct Tile {
  static constexpr int NW = NW_;
  static constexpr int BM = 32 * NW;         // query rows per workgroup
  static constexpr int BN = 64;              // key rows per KV tile
  static constexpr int NT = 64 * NW;         // threads per workgroup
  static constexpr int S = NW == 8 ? 4 : 2;  // resident K/V tiles
  static constexpr int CH = D / 8;           // 16-byte chunks per row
  static constexpr int BPW = CH / NW;        // 1 KB DMA blocks (16 rows x 64 B) per wave and tile, K and V
  static constexpr int KS = D / 16;          // MFMA k-steps along d
  static constexpr int DB = D / 32;          // 32-row blocks of O^T
  static constexpr int NF = D / 8;           // 32x32x16 fragments of one K or V tile
  static constexpr int VP = NF / 2;          // V fragments read ahead of their use (from the softmax on)
  static constexpr int KP = NF / 2;          // K fragments read ahead of their use
  static constexpr int TILE = BN * D;        // elements of one K or V tile
  static_assert(NW == 4 || NW == 8, "4 or 8 waves");
  static_assert(BPW >= 1, "unsupported head dim");
};

// LDS layout of a 64-row K or V tile, in elements: logical 16-byte chunk c of
// row r sits at (c / 4) * 2048 + r * 32 + 8 * ((c % 4) ^ ((r / 4) % 4)), i.e.
// 64-byte chunk groups of all 64 rows one after the other, with the chunks of
// a group XOR-swizzled by bits 2-3 of the row.  LDS has 64 banks (256 bytes per
// bank row); ds_read_b128 serves 16 lanes per pass and ds_read_b64 32 lanes,
// and a pass is conflict-free when its lanes cover a whole bank row.  A K
// fragment pass reads one chunk of 16 consecutive rows (rows r % 4 and r / 4 %
// 4 pick 16 distinct 16-byte bank groups); a transposing V pass reads 4 chunks
// of 4 consecutive rows (again 16 distinct groups).  A 1 KB DMA block is 16
// rows of one chunk group.
__device__ __forceinline__ int tile_off(int r, int c) { return (c >> 2) * 2048 + r * 32 + 8 * ((c & 3) ^ ((r >> 2) & 3)); }

__device__ __forceinline__ u32x4 ld16(const uint16_t* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ void st16(uint16_t* p, u32x4 v) { *reinterpret_cast<u32x4*>(p) = v; }

__device__ __forceinline__ i16x4 ld_tr16(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((PD_LDS i16x4*)(p));
}

// x, as a value the compiler knows nothing about: what a rare branch derives from
// it is computed there, instead of in registers kept over the whole sweep.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ const char* ubytes(const uint16_t* p) { return reinterpret_cast<const char*>(uniform(p)); }

// 16 bytes from global memory into LDS slot `lane` of the 1 KB block at byte
// address lds (global_load_lds_dwordx4 with the block's LDS address in M0), from
// a uniform base plus a per-lane byte offset; inactive lanes load nothing.  Issued
// as inline assembly: when the compiler sees an LDS DMA in flight it can no
// longer count LDS reads precisely and waits for all of them (lgkmcnt(0)) before
// every fragment use.  Completion is tracked by hand (wait_dma); loads the
// compiler does not see only make its own vmcnt waits stricter.  The s_nop holds the
// wait states that the compiler would insert between its own instructions: one
// between a write of M0 and the DMA that reads it, and five between a vector
// instruction that writes a scalar register and the DMA that reads that.  FRESH: the base
// may come straight from such an instruction (readfirstlane).
template <bool FRESH = false>
__device__ __forceinline__ void dma16(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop %3\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(uniform(base)), "s"(uniform((int)lds)), "n"(FRESH ? 3 : 0) : "memory", "m0");
}
// The same from an address per lane.
__device__ __forceinline__ void dma16(const char* at, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(at), "s"(uniform((int)lds)) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(const uint16_t* p) { return (uint32_t)(uintptr_t)(PD_LDS const void*)(p); }

// Engine state of the 32 query rows of a wave.
template <int D>
struct WaveState {
  bf16x8 qf[Tile<D>::KS];
  f32x16 o[Tile<D>::DB];
  float m;      // running row max (log2 domain), shared by lanes l and l^32
  f32x4 l;      // sums of the bf16-rounded weights that multiply V: [0] of query lane % 16, [1] of query lane % 16 + 16
  float lx;     // this lane's partial sum of the unrounded weights (prefill only)
  float qmass;  // this lane's partial mass on its counted key range (prefill only)
};

// Keys counted into qmass (prefill only), tile-relative: a lane whose query row
// lies below `split` (row index within the wave) counts [lo0, hi0), the other lanes
// [lo1, hi1).  The prefill
// counts the query columns for the BOS and content rows (Eq. 5, first sum)
// and the content columns for the query and pseudo-label rows (the
// prefill-time chunk score).
struct MassRange {
  int split, lo0, hi0, lo1, hi1;
};

// Lane-constant parts of the LDS fragment addresses (elements).  Everything
// else (k-step, key block, d block, tile buffer) is an immediate offset.
struct FragAddr {
  int k[2];   // K fragment, row l32 (+ 32 kb), chunk 2 ks + grp: base for ks % 2, + (ks / 2) * 2048 + kb * 1024
  int v[2];   // V transposing read: base for r2, + db * 2048 + (16 kk + 8 r2) * 32
  uint32_t ones;   // row-sum operand
  __device__ FragAddr(int lane) {
    const int sel = (lane >> 4) & 1;
    ones = (lane & 3) == sel ? 0x3f803f80u : 0u;
    const int l32 = lane & 31, grp = lane >> 5;
#pragma unroll
    for (int j = 0; j < 2; ++j) k[j] = tile_off(l32, 2 * j + grp);
    // Group q = lane / 16 of 16 lanes, kq = lane % 16: this lane points at
    // V[4 grp + kq/4 + 16 kk + 8 r2][32 db + 16 (q % 2) + 4 (kq % 4)], 4 elements.
    const int kq = lane & 15, dh = (lane >> 4) & 1;
    const int row = 4 * grp + (kq >> 2), c = 2 * dh + ((kq & 3) >> 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) v[j] = tile_off(row + 8 * j, c) - 8 * 32 * j + 4 * (kq & 1);
  }
};

// One KV tile for one wave, in the functions that follow: S^T = K Q^T (s_phase), online
// softmax producing the bf16 weights P (softmax_phase), O^T += V^T P^T (pv_phase).
// KEYS: keys that are computed, 64 or kShortTile.  kv_valid: number of valid keys
// among them (KEYS except in a ragged last tile).  mr: keys counted into qmass.
// EXACT: also keep the unrounded row sum and the counted mass (prefill).  O is
// normalised by the sum of the same bf16-rounded weights that multiply V, so rounding
// P perturbs a convex combination instead of scaling O.

// Fragment i of a K tile: k-step i / 2, 32-key block i % 2.
template <int D>
__device__ __forceinline__ bf16x8 k_frag(const uint16_t* Ks, const FragAddr& fa, int i) {
  const int ks = i >> 1, kb = i & 1;
  return __builtin_bit_cast(bf16x8, ld16(Ks + fa.k[ks & 1] + (ks >> 1) * 2048 + kb * 1024));
}

// Fragment i of a V^T tile (two transposing reads): key step i / DB, d block i % DB.
template <int D>
__device__ __forceinline__ bf16x8 v_frag(const uint16_t* Vs, const FragAddr& fa, int i) {
  const int kk = i / Tile<D>::DB, db = i % Tile<D>::DB;
  const uint16_t* vb = Vs + db * 2048 + 16 * kk * 32;
  const i16x4 lo = ld_tr16(vb + fa.v[0]);
  const i16x4 hi = ld_tr16(vb + fa.v[1] + 8 * 32);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The largest of three, NaN if one of them is: v_maximum3_f32 (v_max3_f32 would drop a
// NaN, and fmaxf also canonicalises each MFMA output first).  Not inline assembly, for
// which the compiler does not count the wait states after an MFMA that writes a or b.
__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

// Max of this lane's value and the value of lane l ^ 32 (v_permlane32_swap
// exchanges the two halves of the wave without going through LDS).
__device__ __forceinline__ float max_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = __uint_as_float(r[1]);
  return max3(__uint_as_float(r[0]), y, y);
}

// Softmax, part 1: mask, row max, lazy rescale of the running output.  Returns
// -m (log2 domain) for the exponent FMA.  Key of s[kb][r]: 32*kb + 8*(r/4) +
// 4*grp + r%4.  The max is taken on raw scores (the scale is positive) and the
// scale is folded into one FMA: p = exp2(s * scale_log2 - m).
// A row with a NaN or +inf score has no softmax: its sums and outputs turn NaN here,
// and its weights are zero from the tile on, because the product that sums the
// weights takes queries q and q + 16 in one column, one of them times zero.
template <int D, bool EXACT, int KEYS>
__device__ __forceinline__ float softmax_max(WaveState<D>& st, f32x16 (&s)[2], int grp, float scale_log2,
                                             int kv_valid) {
  using T = Tile<D>;
  if (KEYS < 64 || __builtin_expect(kv_valid < 64, 0)) {
    const int valid = kv_valid - 4 * opaque(grp);
#pragma unroll
    for (int e = 0; e < KEYS / 2; ++e) {
      const int kb = e >> 4, r = e & 15;
      s[kb][r] = 32 * kb + 8 * (r >> 2) + (r & 3) < valid ? s[kb][r] : -INFINITY;
    }
  }
  float mx = -INFINITY;
#pragma unroll
  for (int e = 0; e < KEYS / 2; e += 2) mx = max3(mx, s[e >> 4][e & 15], s[e >> 4][(e & 15) + 1]);
  mx = max_across_halves(mx) * scale_log2;
  if (__builtin_expect(__ballot(!(mx <= st.m + 8.0f)) != 0, 0)) {
    const bool bad = !(mx < INFINITY), upd = !bad && mx > st.m + 8.0f;
    const float mnew = upd ? mx : st.m;
    const float alpha = bad ? __uint_as_float(kNanWord) : fast_exp2(st.m - mnew);
    st.m = mnew;
    if (__ballot(bad)) {
#pragma unroll
      for (int e = 0; e < KEYS / 2; ++e) s[e >> 4][e & 15] = bad ? -INFINITY : s[e >> 4][e & 15];
    }
    const int q16 = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) & 15;
    st.l[0] *= __shfl(alpha, q16);
    st.l[1] *= __shfl(alpha, q16 + 16);
    if constexpr (EXACT) {
      st.lx *= alpha;
      st.qmass *= alpha;
    }
#pragma unroll
    for (int db = 0; db < T::DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
  }
  return -st.m;
}

// Part 2: weights p, packed to bf16 in pk; with EXACT the tile's exact sum is
// returned.  COUNT: cnt receives the sum over keys [qlo, qhi).  The first VP
// fragments of the tile's V are read on the way: they land behind the
// exponentials and wait in registers for the P*V of the next phase.
template <int D, bool EXACT, bool COUNT, int KEYS>
__device__ __forceinline__ float softmax_exp(const f32x16 (&s)[2], uint32_t (&pk)[16], bf16x8 (&vf)[Tile<D>::NF],
                                             const uint16_t* Vs, const FragAddr& fa, float nm, float scale_log2,
                                             int grp, int qlo, int qhi, float& cnt) {
  constexpr int Q = Tile<D>::VP / 2;
  float lsum = 0.f;
  if constexpr (COUNT) {
    const int first = 4 * opaque(grp);
    qlo -= first;
    qhi -= first;
  }
#pragma unroll
  for (int g = 0; g < KEYS / 16; ++g) {
    if (g < 2) {
#pragma unroll
      for (int i = 0; i < Q; ++i) vf[g * Q + i] = v_frag<D>(Vs, fa, g * Q + i);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 8 * g; e < 8 * g + 8; e += 2) {
      const int kb = e >> 4, r = e & 15;
      const float p0 = fast_exp2(fmaf(s[kb][r], scale_log2, nm));
      const float p1 = fast_exp2(fmaf(s[kb][r + 1], scale_log2, nm));
      if constexpr (EXACT) lsum += p0 + p1;
      if constexpr (COUNT) {
        const int key = 32 * kb + 8 * (r >> 2) + (r & 3);   // less 4 grp
        cnt += (key >= qlo && key < qhi) ? p0 : 0.f;
        cnt += (key + 1 >= qlo && key + 1 < qhi) ? p1 : 0.f;
      }
      pk[e >> 1] = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)p0, (__bf16)p1});
    }
    // Computed here: the compiler would sink the exponentials past the barrier to their use.
#pragma unroll
    for (int e = 4 * g; e < 4 * g + 4; ++e) asm volatile("" : "+v"(pk[e]));
    __builtin_amdgcn_sched_barrier(0);
  }
  return lsum;
}

// The vector phase of one tile: softmax, with the first V fragments read and
// (EXACT) the row sum and the mass of the lane's counted keys kept.  A range that
// covers the whole tile takes the tile's exact row sum; the per-key test runs
// only in tiles where some lane's range is partial.
template <int D, bool EXACT, int KEYS>
__device__ __forceinline__ void softmax_phase(WaveState<D>& st, f32x16 (&s)[2], uint32_t (&pk)[16],
                                              bf16x8 (&vf)[Tile<D>::NF], const uint16_t* Vs, const FragAddr& fa,
                                              int grp, int lane32, float scale_log2, int kv_valid,
                                              const MassRange& mr) {
  const float nm = softmax_max<D, EXACT, KEYS>(st, s, grp, scale_log2, kv_valid);
  float cnt = 0.f;
  if constexpr (!EXACT) {
    softmax_exp<D, false, false, KEYS>(s, pk, vf, Vs, fa, nm, scale_log2, grp, 0, 0, cnt);
  } else {
    const bool none = mr.lo0 >= mr.hi0 && mr.lo1 >= mr.hi1;   // wave-uniform: nothing counted in this tile
    const bool first = lane32 < mr.split;
    const int qlo = first ? mr.lo0 : mr.lo1, qhi = first ? mr.hi0 : mr.hi1;
    const bool any = qlo < qhi;
    if (!none && __ballot(any && (qlo > 0 || qhi < 64))) {
      st.lx += softmax_exp<D, true, true, KEYS>(s, pk, vf, Vs, fa, nm, scale_log2, grp, qlo, qhi, cnt);
      st.qmass += cnt;
    } else {
      const float lsum = softmax_exp<D, true, false, KEYS>(s, pk, vf, Vs, fa, nm, scale_log2, grp, 0, 0, cnt);
      st.lx += lsum;
      st.qmass += any ? lsum : 0.f;
    }
  }
}

// The matrix phase: O += V^T P^T of the previous tile (weights pk), then S^T of
// the next one.  LDS feeds the MFMAs at the rate at which it can: a 32-row wave
// reads 1 KB per MFMA, four waves of a group 128 bytes per clock and CU.  So the
// reads are spread over both phases: the first VP V fragments come from the
// vector phase, the others are read VP products ahead of their use, and then, in
// the second half of P*V and the first of S, the K fragments KP ahead of theirs.
// P^T operand of key step kk: keys 16kk + 4grp + {0..3} then 16kk + 8 + 4grp +
// {0..3} (pk[4kk .. 4kk+3]); the two transposing reads deliver V^T in that order.
// The row sums of the rounded weights are one more product, ones * P^T, on the
// 16x16x32 MFMA: its columns are 16 queries and its four 8-key blocks the lane
// quarters, so row 0 (mod 4) takes the two quarters that hold queries 0..15 and
// row 1 those of queries 16..31.  (v_dot2_f32_bf16 would do it on the vector
// side, but waits for the matrix core: 69 cycles each beside another wave's
// MFMAs, 5 alone.)
// NEXT: the second half also reads the first KP fragments of the next K tile.
template <int D, bool NEXT, int KEYS>
__device__ __forceinline__ void pv_phase(WaveState<D>& st, const uint32_t (&pk)[16], bf16x8 (&vf)[Tile<D>::NF],
                                         bf16x8 (&kf)[Tile<D>::NF], const uint16_t* Vs, const uint16_t* Ks_next,
                                         const FragAddr& fa) {
  using T = Tile<D>;
  constexpr int NI = T::NF * KEYS / 64;
  const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{fa.ones, fa.ones, fa.ones, fa.ones});
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int kk = i / T::DB, db = i % T::DB;
    const bf16x8 pf = __builtin_bit_cast(bf16x8, u32x4{pk[4 * kk], pk[4 * kk + 1], pk[4 * kk + 2], pk[4 * kk + 3]});
    if (i + T::VP < NI) vf[i + T::VP] = v_frag<D>(Vs, fa, i + T::VP);
    if (NEXT && i + T::KP >= T::NF) kf[i + T::KP - T::NF] = k_frag<D>(Ks_next, fa, i + T::KP - T::NF);
    st.o[db] = mfma32x32x16(vf[i], pf, st.o[db]);
    if (db == 0) st.l = mfma16x16x32(ones, pf, st.l);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The first KP fragments of a K tile.
template <int D, int KEYS = 64>
__device__ __forceinline__ void k_first(bf16x8 (&kf)[Tile<D>::NF], const uint16_t* Ks, const FragAddr& fa) {
#pragma unroll
  for (int i = 0; i < Tile<D>::KP; i += KEYS > 32 ? 1 : 2) kf[i] = k_frag<D>(Ks, fa, i);
}

// S^T of a tile whose first KP fragments are in kf.  issue(n), n < N, issues the
// wave's n-th DMA of a coming tile: one between every few MFMAs, where a wave
// otherwise only waits for the matrix core.
template <int D, int N, int KEYS, class Issue>
__device__ __forceinline__ void s_phase(const WaveState<D>& st, f32x16 (&s)[2], bf16x8 (&kf)[Tile<D>::NF],
                                        const uint16_t* Ks, const FragAddr& fa, Issue&& issue) {
  using T = Tile<D>;
  constexpr int STEP = T::NF / N;
  s[0] = s[1] = f32x16{0};
  static_for<T::NF>([&](auto i) PD_INLINE {
    if constexpr (KEYS > 32 || i % 2 == 0) {
      if constexpr (i + T::KP < T::NF) kf[i + T::KP] = k_frag<D>(Ks, fa, i + T::KP);
      s[i & 1] = mfma32x32x16(kf[i], st.qf[i >> 1], s[i & 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (i % STEP == 1) {
      issue(std::integral_constant<int, i / STEP>());
      __builtin_amdgcn_sched_barrier(0);
    }
  });
}

// Completes the loads of the Q fragments here, before the sweep.  The compiler
// does not see the tile DMAs (inline assembly): a Q load it still counted as
// pending would make it wait for every load in flight (s_waitcnt vmcnt(0)),
// tile DMAs included, at the fragment's first use in every tile.  Consuming
// the registers in an empty asm statement puts that one wait here instead.
template <int D>
__device__ __forceinline__ void q_landed(const WaveState<D>& st) {
#pragma unroll
  for (int ks = 0; ks < Tile<D>::KS; ++ks) asm volatile("" ::"v"(st.qf[ks]));
}

template <int D>
__device__ __forceinline__ void wave_init(WaveState<D>& st) {
#pragma unroll
  for (int db = 0; db < Tile<D>::DB; ++db) st.o[db] = f32x16{0};
  st.m = kNoMax;
  st.l = f32x4{0.f, 0.f, 0.f, 0.f};
  st.lx = 0.f;
  st.qmass = 0.f;
}

// Normalised O^T of this lane (query l32) for d = 32*db + 8*i + 4*grp + j is
// st.o[db][4*i+j] * inv; store one row of D bf16 values.
template <int D>
__device__ __forceinline__ void store_row_bf16(uint16_t* dst, const WaveState<D>& st, float inv, int grp) {
#pragma unroll
  for (int db = 0; db < Tile<D>::DB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      u32x2 v = {pack_bf16x2(st.o[db][4 * i] * inv, st.o[db][4 * i + 1] * inv),
                 pack_bf16x2(st.o[db][4 * i + 2] * inv, st.o[db][4 * i + 3] * inv)};
      *reinterpret_cast<u32x2*>(dst + 32 * db + 8 * i + 4 * grp) = v;
    }
}

template <int D>
__device__ __forceinline__ void store_row_f32(float* dst, const WaveState<D>& st, float inv, int grp) {
#pragma unroll
  for (int db = 0; db < Tile<D>::DB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 v = {st.o[db][4 * i] * inv, st.o[db][4 * i + 1] * inv, st.o[db][4 * i + 2] * inv,
                 st.o[db][4 * i + 3] * inv};
      *reinterpret_cast<f32x4*>(dst + 32 * db + 8 * i + 4 * grp) = v;
    }
}

// This wave's share of the DMA of one K or V tile: BPW blocks of 1 KB.  Block b
// holds rows 16 (b % 4) .. +15 of chunk group b / 4; a lane takes row 16 (b % 4)
// + lane / 4 (dma_row) and loads the logical chunk that tile_off places in its
// 16-byte slot (dma_chunk, the same for all blocks of a wave).
template <class T>
__device__ __forceinline__ int dma_row(int wave, int lane, int j) {
  return ((wave * T::BPW + j) & 3) * 16 + (lane >> 2);
}
template <class T>
__device__ __forceinline__ int dma_chunk(int wave, int lane) {
  return 4 * ((wave * T::BPW) >> 2) + ((lane & 3) ^ ((lane >> 4) & 3));
}

// Where the wave's rows of one tile come from.  plain: all rows of the tile lie
// at uniform bases k, v plus a byte offset per lane (from the row table if table,
// else that of consecutive rows); otherwise (a tile that crosses from one buffer to
// the next, or past the last row) mixed() issues the DMA.  In the decode every lane
// has an address of its own there: in short sweeps most tiles are of that kind, and with
// one masked DMA per buffer a step of 65 rows over 2 tiles took 16.0 us, now 15.6, one
// of 128 rows over 7 tiles 22.4, now 20.9.  The prefill, which has two such tiles in 15
// to 27 and two buffers, keeps one masked DMA per buffer (8 x 32K 14.36 ms, 14.44 with an
// address per lane).  The next `run` tiles continue this one, each `step` bytes further.
struct TileSrc {
  const char *k, *v;
  long long step;
  int run;
  bool plain, table;
};

// Wait until at most n DMAs of this wave are in flight, n = m * BPW.  DMAs are
// loads and complete in issue order, so all but the newest n have landed (stores
// issued in between can only make the wait longer).
template <class T>
__device__ __forceinline__ void wait_dma(int m) {
  constexpr int B = T::BPW;
  if (m >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * B) : "memory");
  else if (m == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(B) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Workgroup barrier without a memory fence.  __syncthreads() would also wait
// for every LDS DMA still in flight (they count as outstanding LDS writes),
// draining the pipeline; here the tile in use is covered by the wait for its DMA, and
// every LDS read of older tiles has been consumed before a wave gets here.  The
// memory clobber keeps the compiler from moving memory accesses across it.
__device__ __forceinline__ void tile_barrier() { asm volatile("s_barrier" ::: "memory"); }

// A last tile of at most this many keys takes one key step of P*V and one key block
// of S instead of four and two, and a quarter of the exponentials.  Most sweeps end
// in one: the BOS rows put 1 to 4 rows on top of sizes that are whole tiles (1345 rows
// are 21 tiles and a row).  Prefill of 8K 328.6 -> 324.1 us, of 16K 520.5 -> 515.9, of
// 8 x 32K 14.53 -> 14.39 ms, 8K step 29.5 -> 28.9 us, step of 8 x 32K 145.6 -> 143.9.
constexpr int kShortTile = 16;

// Sweep over KV tiles [t_begin, t_end), at least one, by one of two workgroups of
// four waves on a CU, which are not synchronised: one's start, end and softmax run
// beside the other's MFMAs.  Tile t lives in buffer (t - t_begin) % 2.  One barrier per tile: before it every wave
// has waited for its own share of tile t's DMA and has used all it read of tile
// t-1, whose buffer then takes tile t+1.  tile(t) gives a tile's rows, peek(t,
// code) reads the row table of a tile and off(ts, code, j) makes a lane's byte
// offsets from that; mixed(V, r, c, lds) is the DMA of chunk byte c of row r (a K
// or V row) in a tile that is not plain; hook(t, Ks, Vs) sees the landed tile
// (the prefill writes its cache share there); softmax(t, last, s, pk, vf, Vs) is
// the vector part.  tail: keys from the last tile's first row to the end of the
// sequence.  ACTIVE: false for the waves without query rows, which only move tiles.
template <int D, bool ACTIVE, class Peek, class Off, class Src, class Mixed, class Hook, class Softmax>
__device__ __forceinline__ void sweep_pair(WaveState<D>& st, uint16_t* Kb, uint16_t* Vb, const FragAddr& fa, int wave,
                                         int lane, int t_begin, int t_end, int tail, Peek&& peek, Off&& off,
                                         Src&& tile, Mixed&& mixed, Hook&& hook, Softmax&& softmax) {
  using T = Tile<D, 4>;
  // LDS byte address of this wave's first block in buffer 0.
  const uint32_t ka = lds_addr(Kb) + wave * T::BPW * 1024, va = lds_addr(Vb) + wave * T::BPW * 1024;
  TileSrc src;   // the tile whose DMA is issued next; code: the row table of that tile
  unsigned code[T::BPW], at[T::BPW];
  auto dma = [&](int t, int buf) PD_INLINE {
    const uint32_t ko = ka + buf * (T::TILE * 2), vo = va + buf * (T::TILE * 2);
#pragma unroll
    for (int j = 0; j < T::BPW; ++j) {
      if (src.plain) {
        dma16(src.k, at[j], ko + j * 1024);
        dma16(src.v, at[j], vo + j * 1024);
      } else {
        const int ln = opaque(lane), r = t * T::BN + dma_row<T>(wave, ln, j);
        mixed(std::false_type(), r, 16u * dma_chunk<T>(wave, ln), ko + j * 1024);
        mixed(std::true_type(), r, 16u * dma_chunk<T>(wave, ln), vo + j * 1024);
      }
    }
  };
  auto offsets = [&]() PD_INLINE {
#pragma unroll
    for (int j = 0; j < T::BPW; ++j) at[j] = off(src, code, j);
  };
  peek(t_begin, code);
  src = tile(t_begin);
  offsets();
  dma(t_begin, 0);
  peek(t_begin + 1, code);
  f32x16 s[2];
  uint32_t pk[16];
  bf16x8 vf[T::NF], kf[T::NF];
  int buf = 0;   // buffer of tile t
  auto step = [&](int t, auto last, auto keys) PD_INLINE {
    constexpr bool LAST = decltype(last)::value;
    constexpr int KEYS = decltype(keys)::value;
    const uint16_t *Ks = Kb + buf * T::TILE, *Vs = Vb + buf * T::TILE;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    tile_barrier();
    if constexpr (!LAST) {
      if (__builtin_expect(src.run > 0, 1)) {
        src.k += src.step;
        src.v += src.step;
        --src.run;
      } else {
        src = tile(t + 1);
      }
      offsets();
      const uint32_t ko = ka + (buf ^ 1) * (T::TILE * 2), vo = va + (buf ^ 1) * (T::TILE * 2);
      if (ACTIVE && __builtin_expect(src.plain, 1)) {
        k_first<D>(kf, Ks, fa);
        s_phase<D, 2 * T::BPW, 64>(st, s, kf, Ks, fa, [&](auto n) PD_INLINE {
          if constexpr (n < T::BPW) dma16(src.k, at[n], ko + n * 1024);
          else dma16(src.v, at[n - T::BPW], vo + (n - T::BPW) * 1024);
        });
      } else {
        dma(t + 1, buf ^ 1);
        if constexpr (ACTIVE) {
          k_first<D>(kf, Ks, fa);
          s_phase<D, 2 * T::BPW, 64>(st, s, kf, Ks, fa, [](auto) PD_INLINE {});
        }
      }
      peek(t + 2, code);
    } else if constexpr (ACTIVE) {
      k_first<D, KEYS>(kf, Ks, fa);
      s_phase<D, 2 * T::BPW, KEYS>(st, s, kf, Ks, fa, [](auto) PD_INLINE {});
    }
    hook(t, Ks, Vs);
    if constexpr (ACTIVE) {
      softmax(t, last, keys, s, pk, vf, Vs);
      pv_phase<D, false, KEYS>(st, pk, vf, kf, Vs, Ks, fa);
    }
    buf ^= 1;
  };
  for (int t = t_begin; t + 1 < t_end; ++t) step(t, std::false_type(), std::integral_constant<int, 64>());
  if (tail > kShortTile) step(t_end - 1, std::true_type(), std::integral_constant<int, 64>());
  else step(t_end - 1, std::true_type(), std::integral_constant<int, kShortTile>());
}

// The same sweep by the one workgroup of eight waves on a CU.  Tile t lives in
// buffer (t - t_begin) % S.  Every wave alternates a matrix phase M(t) (P*V of tile
// t-1, S of tile t) and a vector phase V(t) (softmax of t), one barrier after
// each; the two wave groups of a workgroup (one wave of each per SIMD) run half
// a period apart, so that on every SIMD one wave's MFMAs run beside the other's
// VALU work:
//   phase 2i     group 0: M(i)   group 1: V(i-1)
//   phase 2i+1   group 0: V(i)   group 1: M(i)
// K(i) is read in phases 2i and 2i+1 and V(i) in phases 2i+1 to 2i+3, at the
// latest by M(i+1), which uses what it reads.  M(i) issues the DMAs of K(i+3),
// over K(i-1), last read in phase 2i-1, and of V(i+2), over V(i-2), last read in
// phase 2i-1.  A wave's DMAs are thus issued in the order
// K(b) K(b+1) V(b) K(b+2) V(b+1) | K(b+3) V(b+2) | K(b+4) V(b+3) ...  K(i) must
// have landed before phase 2i and V(i) before phase 2i+1: at the end of V(i)
// every wave waits for all of its DMAs but those of M(i), so for V(i+1) and
// K(i+2), one phase or more ahead of need.
// The other arguments are those of sweep_pair (there is no hook).
template <int D, bool ACTIVE, class Peek, class Off, class Src, class Mixed, class Softmax>
__device__ __forceinline__ void sweep_pingpong(WaveState<D>& st, uint16_t* Kb, uint16_t* Vb, const FragAddr& fa, int wave,
                                         int lane, int t_begin, int t_end, int tail, Peek&& peek,
                                         Off&& off, Src&& tile, Mixed&& mixed, Softmax&& softmax) {
  using T = Tile<D, 8>;
  constexpr int S = T::S;
  const int group = wave / (T::NW / 2);
  // LDS byte address of this wave's first block in buffer 0.
  const uint32_t ka = lds_addr(Kb) + wave * T::BPW * 1024, va = lds_addr(Vb) + wave * T::BPW * 1024;
  // One tile's K (V = 0) or V (V = 1) into buffer buf.
  auto dma = [&](auto V, const TileSrc& ts, const unsigned (&o)[T::BPW], int t, int buf) PD_INLINE {
#pragma unroll
    for (int j = 0; j < T::BPW; ++j) {
      const uint32_t dst = (V ? va : ka) + buf * (T::TILE * 2) + j * 1024;
      if (ts.plain) {
        dma16(V ? ts.v : ts.k, o[j], dst);
      } else {
        const int ln = opaque(lane);
        mixed(V, t * T::BN + dma_row<T>(wave, ln, j), 16u * dma_chunk<T>(wave, ln), dst);
      }
    }
  };
  constexpr std::false_type K_;
  constexpr std::true_type V_;
  f32x16 s[2];
  uint32_t pk[16];
  bf16x8 vf[T::NF], kf[T::NF];
  // The tiles whose V and K the next M issues; code: the row table of the one after.
  TileSrc src_v, src_k;
  unsigned off_v[T::BPW], off_k[T::BPW], code[T::BPW];
  auto advance = [&](int t, const unsigned (&code)[T::BPW]) PD_INLINE {   // src_k: tile t, from tile t-1
    src_v = src_k;
#pragma unroll
    for (int j = 0; j < T::BPW; ++j) off_v[j] = off_k[j];
    if (__builtin_expect(src_k.run > 0, 1)) {
      src_k.k += src_k.step;
      src_k.v += src_k.step;
      --src_k.run;
    } else {
      src_k = tile(t);
    }
#pragma unroll
    for (int j = 0; j < T::BPW; ++j) off_k[j] = off(src_k, code, j);
  };
  unsigned first[S][T::BPW];   // row table of the first tiles, read together
#pragma unroll
  for (int i = 0; i < S; ++i) peek(t_begin + i, first[i]);
  src_k = tile(t_begin);
#pragma unroll
  for (int j = 0; j < T::BPW; ++j) off_k[j] = off(src_k, first[0], j);
  dma(K_, src_k, off_k, t_begin, 0);
#pragma unroll
  for (int i = 1; i < S - 1; ++i) {   // K(b+i), V(b+i-1)
    advance(t_begin + i, first[i]);
    if (t_begin + i < t_end) dma(K_, src_k, off_k, t_begin + i, i);
    if (t_begin + i - 1 < t_end) dma(V_, src_v, off_v, t_begin + i - 1, i - 1);
  }
#pragma unroll
  for (int j = 0; j < T::BPW; ++j) code[j] = first[S - 1][j];
  wait_dma<T>(t_begin + 2 < t_end ? 2 : (t_begin + 1 < t_end ? 1 : 0));
  tile_barrier();
  if (group) tile_barrier();
  if constexpr (ACTIVE) k_first<D>(kf, Kb, fa);
  int buf = 0;   // buffer of tile t
  // S of tile t and the DMAs of M(t).  HOT: tiles t .. t+3 exist.
  auto scores = [&](int t, auto hot, auto keys) PD_INLINE {
    constexpr bool HOT = decltype(hot)::value;
    constexpr int KEYS = decltype(keys)::value;
    const int buf2 = (buf + 2) & (S - 1), buf3 = (buf + 3) & (S - 1);
    advance(t + 3, code);
    peek(t + 4, code);
    if (ACTIVE && KEYS == 64 && __builtin_expect((HOT || t + 3 < t_end) && src_v.plain && src_k.plain, 1)) {
      s_phase<D, 2 * T::BPW, 64>(st, s, kf, Kb + buf * T::TILE, fa, [&](auto n) PD_INLINE {
        if constexpr (n < T::BPW) dma16(src_k.k, off_k[n], ka + buf3 * (T::TILE * 2) + n * 1024);
        else dma16(src_v.v, off_v[n - T::BPW], va + buf2 * (T::TILE * 2) + (n - T::BPW) * 1024);
      });
    } else {
      if (HOT || t + 3 < t_end) dma(K_, src_k, off_k, t + 3, buf3);
      if (HOT || t + 2 < t_end) dma(V_, src_v, off_v, t + 2, buf2);
      if constexpr (ACTIVE) s_phase<D, 2 * T::BPW, KEYS>(st, s, kf, Kb + buf * T::TILE, fa, [](auto) PD_INLINE {});
    }
  };
  // V(t).  HOT: tiles t .. t+3 exist, so tile t is whole.
  auto vector = [&](int t, auto hot, auto keys) PD_INLINE {
    constexpr bool HOT = decltype(hot)::value;
    if constexpr (ACTIVE) softmax(t, std::bool_constant<!HOT>(), keys, s, pk, vf, Vb + buf * T::TILE);
    wait_dma<T>(HOT || t + 3 < t_end ? 2 : (t + 2 < t_end ? 1 : 0));
  };
  auto product = [&](auto keys) PD_INLINE {   // P*V of tile t; buf moves on to tile t+1
    const int vbuf = buf;
    buf = (buf + 1) & (S - 1);
    // After the last tile the K fragments read here are an older tile's, and unused.
    if constexpr (ACTIVE) pv_phase<D, decltype(keys)::value == 64, decltype(keys)::value>(st, pk, vf, kf, Vb + vbuf * T::TILE, Kb + buf * T::TILE, fa);
  };
  constexpr std::integral_constant<int, 64> whole;
  constexpr std::integral_constant<int, kShortTile> few;
  int t = t_begin;
  scores(t, std::false_type(), whole);
  tile_barrier();
  for (; t + 4 < t_end; ++t) {
    vector(t, std::true_type(), whole);
    tile_barrier();
    product(whole);
    scores(t + 1, std::true_type(), whole);
    tile_barrier();
  }
  for (; t + 1 < t_end; ++t) {
    vector(t, std::false_type(), whole);
    tile_barrier();
    product(whole);
    if (t + 2 == t_end && tail <= kShortTile) scores(t + 1, std::false_type(), few);
    else scores(t + 1, std::false_type(), whole);
    tile_barrier();
  }
  if (tail > kShortTile) {
    vector(t, std::false_type(), whole);
    tile_barrier();
    product(whole);
  } else {
    vector(t, std::false_type(), few);
    tile_barrier();
    product(few);
  }
  if (!group) tile_barrier();
}

// ---------------------------------------------------------------------------
// Stage (a): chunk prefill.  Workgroup = (b, n, h, 128-row query tile).
// Also writes the chunk KV cache (each KV tile by exactly one workgroup of the
// (b, n, kv-head) group), the per-head query-column mass of the content rows,
// the log2-domain LSE of the query rows and, when asked, the per-head
// content mass of the query and pseudo-label rows.
template <int D>
__global__ __launch_bounds__(Tile<D>::NT, 2) void prefill_bf16_kernel(PrefillArgs p) {
  using T = Tile<D>;
  __shared__ __attribute__((aligned(1024))) uint16_t Kb[T::S * T::TILE], Vb[T::S * T::TILE];
  __shared__ __attribute__((aligned(16))) float kacc[T::NT / T::CH * D];   // content-key sums, one slot per thread

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, grp = lane >> 5;
  int lid = xcd_remap(blockIdx.x, p.total);
  const int qt = uniform(lid % p.n_qt);
  lid /= p.n_qt;
  const int h = uniform(lid % p.Hq);
  lid /= p.Hq;
  const int n = uniform(lid % p.N);
  const int b = uniform(lid / p.N);
  const int g = uniform(h / p.G);
  const int C1 = p.C + 1;
  const size_t chunk = (size_t)b * p.N + n;
  const size_t qm_base = (p.qm_per_chunk ? chunk : (size_t)b) * (size_t)(p.Lq + p.Lm);

  // Q fragments of this lane's query row.
  WaveState<D> st;
  const bool wave_active = qt * T::BM + wave * 32 < p.Sc;
  const int qrow = qt * T::BM + wave * 32 + l32;
  {
    const uint16_t* src = nullptr;
    if (qrow < C1) src = p.q_pre + ((chunk * C1 + qrow) * p.Hq + h) * D;
    else if (qrow < p.Sc) src = p.q_qm + ((qm_base + (qrow - C1)) * p.Hq + h) * D;
#pragma unroll
    for (int ks = 0; ks < T::KS; ++ks)
      st.qf[ks] = src ? __builtin_bit_cast(bf16x8, ld16(src + 16 * ks + 8 * grp)) : bf16x8{0};
    wave_init(st);
  }
  q_landed(st);
  const FragAddr fa(lane);

  // Row r of the chunk sequence lives at base + r*HD (HD = H_kv*d elements), with
  // base the chunk's rows for r <= C and the shared query/pseudo-label rows after.
  // Rows past the end are clamped to the last row: their keys are masked out of
  // the softmax and their (finite) values get probability 0.
  const int HD = p.Hkv * D;
  const uint16_t* k_lo = p.k_pre + (chunk * C1 * p.Hkv + g) * D;
  const uint16_t* v_lo = p.v_pre + (chunk * C1 * p.Hkv + g) * D;
  const uint16_t* k_hi = p.k_qm + (qm_base * p.Hkv + g) * D - (size_t)C1 * HD;
  const uint16_t* v_hi = p.v_qm + (qm_base * p.Hkv + g) * D - (size_t)C1 * HD;
  unsigned own_off[T::BPW];   // byte offset of this lane's rows within a tile of consecutive rows
#pragma unroll
  for (int j = 0; j < T::BPW; ++j) own_off[j] = 2u * dma_row<T>(wave, lane, j) * HD + 16u * dma_chunk<T>(wave, lane);
  auto peek = [](int, unsigned (&)[T::BPW]) PD_INLINE {};
  auto off = [=](const TileSrc&, const unsigned (&)[T::BPW], int j) PD_INLINE { return own_off[j]; };
  auto tile = [=](int t) PD_INLINE {
    const int r0 = t * T::BN, end = r0 < C1 ? C1 : p.Sc;   // rows up to end lie in one buffer
    const char *kl = ubytes(k_lo), *kh = ubytes(k_hi), *vl = ubytes(v_lo), *vh = ubytes(v_hi);
    const size_t at = (size_t)r0 * HD * 2;
    return TileSrc{(r0 < C1 ? kl : kh) + at, (r0 < C1 ? vl : vh) + at, (long long)T::BN * HD * 2, (end - r0) / T::BN - 1, r0 + T::BN <= end, false};
  };
  auto mixed = [=](auto V, int r, unsigned c, uint32_t lds) PD_INLINE {
    r = min(r, p.Sc - 1);
    const unsigned at = 2u * HD * r + c;
    if (r < C1) dma16<true>(ubytes(V ? v_lo : k_lo), at, lds);
    else dma16<true>(ubytes(V ? v_hi : k_hi), at, lds);
  };
  // Each KV tile of the (b, n, kv head) group is written to the cache by exactly
  // one workgroup of that group (query tile t % n_qt of head g*G + (t / n_qt) % G),
  // from the landed LDS tile: thread tid copies logical chunks tid + NT i.
  // Thread tid always handles 16-byte chunk tid % CH of the rows it copies, so
  // its content-key sums live in its own LDS slot kacc[tid / CH][8 (tid % CH) ..]
  // (no other thread touches it until the reduction after the sweep).
#pragma unroll
  for (int e = 0; e < 8; ++e) kacc[(tid / T::CH) * D + 8 * (tid % T::CH) + e] = 0.f;
  const size_t cache_base = (chunk * p.Hkv + g) * C1;
  const int w_step = p.n_qt * p.G;
  int w_next = qt + p.n_qt * (h % p.G);   // the next tile to write
  auto write_cache = [&](int t, const uint16_t* Ks, const uint16_t* Vs) PD_INLINE {
    if (__builtin_expect(t != w_next, 1)) return;
    w_next += w_step;
    const int tid = opaque(threadIdx.x);
    float* const kslot = kacc + (tid / T::CH) * D + 8 * (tid % T::CH);
    float ksum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < T::BN * T::CH / T::NT; ++i) {
      const int u = tid + T::NT * i;
      const int r = u / T::CH, c = u % T::CH;
      const int row = t * T::BN + r;
      if (row < C1) {
        const u32x4 kv = ld16(Ks + tile_off(r, c));
        st16(p.k_cache + (cache_base + row) * D + 8 * c, kv);
        st16(p.v_cache + (cache_base + row) * D + 8 * c, ld16(Vs + tile_off(r, c)));
        if (row >= 1) {   // content rows only (the BOS row is not part of the key mean)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            ksum[2 * q] += __uint_as_float(kv[q] << 16);
            ksum[2 * q + 1] += __uint_as_float(kv[q] & 0xffff0000u);
          }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) kslot[e] += ksum[e];
  };

  const int qc_lo = C1, qc_hi = C1 + p.Lq;   // query columns counted by Eq. 5
  const int cm_hi = p.qm_mass ? C1 : 1;       // content columns counted for the chunk score (if asked)
  const int split = C1 - (qt * T::BM + wave * 32);
  auto softmax = [&](int t, auto last, auto keys, f32x16 (&s)[2], uint32_t (&pk)[16], bf16x8 (&vf)[T::NF], const uint16_t* vs) PD_INLINE {
    const int t0 = t * T::BN;
    const int kv_valid = decltype(last)::value ? p.Sc - t0 : T::BN;
    const MassRange mr{split, max(qc_lo - t0, 0), min(qc_hi - t0, T::BN), max(1 - t0, 0), min(cm_hi - t0, T::BN)};
    softmax_phase<D, true, decltype(keys)::value>(st, s, pk, vf, vs, fa, grp, l32, p.scale_log2, kv_valid, mr);
  };
  if (wave_active)
    sweep_pair<D, true>(st, Kb, Vb, fa, wave, lane, 0, p.n_kvt, p.Sc - (p.n_kvt - 1) * T::BN, peek, off, tile, mixed, write_cache, softmax);
  else
    sweep_pair<D, false>(st, Kb, Vb, fa, wave, lane, 0, p.n_kvt, p.Sc - (p.n_kvt - 1) * T::BN, peek, off, tile, mixed, write_cache, softmax);
  // This workgroup's content-key sums: the thread slots summed in a fixed
  // order, one vector per (b, n, kv head, writer slot qt*G + h%G).
  __syncthreads();
  if (tid < D) {
    float sum = 0.f;
    for (int r = 0; r < T::NT / T::CH; ++r) sum += kacc[r * D + tid];
    p.km_part[((chunk * p.Hkv + g) * (size_t)(p.n_qt * p.G) + qt * p.G + h % p.G) * D + tid] = sum;
  }
  if (!wave_active) return;

  const float ltot = (lane & 16) ? st.l[1] : st.l[0];
  const float lxtot = st.lx + __shfl_xor(st.lx, 32);
  const float qtot = st.qmass + __shfl_xor(st.qmass, 32);
  const float inv = 1.0f / ltot;
  if (qrow < p.Sc) {
    const size_t orow = ((chunk * p.Sc + qrow) * p.Hq + h) * D;
    if (p.out_f32) store_row_f32<D>(reinterpret_cast<float*>(p.o) + orow, st, inv, grp);
    else store_row_bf16<D>(p.o + orow, st, inv, grp);
    if (grp == 0) {
      const size_t hb = chunk * p.Hq + h;
      if (qrow >= 1 && qrow < C1) p.part_i[hb * p.C + (qrow - 1)] = qtot / lxtot;
      if (qrow >= qc_lo && qrow < qc_hi) p.lse_q[hb * p.Lq + (qrow - qc_lo)] = st.m + __log2f(lxtot);
      if (p.qm_mass && qrow >= C1) p.qm_mass[hb * (p.Lq + p.Lm) + (qrow - C1)] = qtot / lxtot;
    }
  }
}

// ---------------------------------------------------------------------------
// Stage (c): sparse decode attention.  Workgroup = (b, kv head g, tile of 32 rows a
// wave of the G*L_d query rows of that group, KV shard).  Query row rho of the group
// is head g*G + rho / L_d, decode row rho % L_d.  KV row j of the shard walks:
// [kept chunks: BOS + kept slots] ; [static rows] ; [own rows].
template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 2) void decode_bf16_kernel(DecodeArgs p) {
  using T = Tile<D, NW>;
  __shared__ __attribute__((aligned(1024))) uint16_t Kb[T::S * T::TILE], Vb[T::S * T::TILE];
  __shared__ __attribute__((aligned(16))) unsigned rowtab[kDecodeTableRows];   // byte offset of each gathered row

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, grp = lane >> 5;
  int lid = xcd_remap(blockIdx.x, p.total);
  const int sp = uniform(lid % p.S);
  lid /= p.S;
  const int qt = uniform(lid % p.n_qt);
  lid /= p.n_qt;
  const int g = uniform(lid % p.Hkv);
  const int b = uniform(lid / p.Hkv);
  const int GL = p.G * p.Ld;
  const int C1 = p.C + 1;
  const int n_sel = p.n_sel;
  const int L_kv = n_sel + p.n_static + p.Ld;

  WaveState<D> st;
  const bool wave_active = qt * T::BM + wave * 32 < GL;
  const int rho = qt * T::BM + wave * 32 + l32;
  {
    const int hq = g * p.G + (rho < GL ? rho / p.Ld : 0);
    const int rr = rho < GL ? rho % p.Ld : 0;
    const uint16_t* src = rho < GL ? p.q_dec + (((size_t)b * p.Ld + rr) * p.Hq + hq) * D : nullptr;
#pragma unroll
    for (int ks = 0; ks < T::KS; ++ks)
      st.qf[ks] = src ? __builtin_bit_cast(bf16x8, ld16(src + 16 * ks + 8 * grp)) : bf16x8{0};
    wave_init(st);
  }
  const FragAddr fa(lane);

  // This shard's tiles.
  const int n_kvt = (L_kv + T::BN - 1) / T::BN;
  const int t_begin = uniform((int)(((long long)n_kvt * sp) / p.S));
  const int t_end = uniform((int)(((long long)n_kvt * (sp + 1)) / p.S));

  // Prefix rows of (b, g): gathered from the chunk cache (row n*Hkv*C1 + slot
  // from this base), or, in compact mode, row j of the contiguous buffer.
  const size_t cache_bg = p.compact ? ((size_t)b * p.Hkv + g) * n_sel : ((size_t)b * p.N * p.Hkv + g) * C1;
  // Prefix rows of this shard: byte offsets into LDS once (the host keeps
  // every shard within kDecodeTableRows rows), so tile loads need no index fetch.
  const int j_lo = t_begin * T::BN;
  const int j_hi = min(t_end * T::BN, n_sel);
  __shared__ int bad_index;   // checking build: some kept row of this shard was out of range
  if (kCheckIndices && tid == 0) bad_index = 0;
  if (kCheckIndices) __syncthreads();
  if (p.compact) {
    for (int j = j_lo + tid; j < j_hi; j += T::NT) rowtab[j - j_lo] = 2u * D * j;
  } else {
    const int32_t* cidx = p.chunk_idx + (size_t)b * p.K;
    const int32_t* tslot = p.tok_slot + (size_t)b * p.K * p.Bt;
    for (int j = j_lo + tid; j < j_hi; j += T::NT) {
      const int kk = j / (1 + p.Bt), s = j - kk * (1 + p.Bt);
      int slot = s == 0 ? 0 : tslot[kk * p.Bt + s - 1];
      int chunk = cidx[kk];
      if (kCheckIndices && !kept_row_ok(chunk, slot, s == 0, p.N, p.C)) {
        chunk = 0;
        slot = 0;
        bad_index = 1;
      }
      rowtab[j - j_lo] = 2u * D * (unsigned)(chunk * p.Hkv * C1 + slot);
    }
  }
  __syncthreads();
  // Row j of the shard: gathered cache rows (offset from the LDS table), then
  // static rows, then own rows, each at base + row*HD for the latter two.  Rows
  // past L_kv are clamped to the last row (masked out of the softmax).
  const int HD = p.Hkv * D;
  const uint16_t* kc = p.k_cache + cache_bg * D;
  const uint16_t* vc = p.v_cache + cache_bg * D;
  const size_t sb = ((size_t)b * p.Ls * p.Hkv + g) * D - (size_t)n_sel * HD;
  const size_t db = ((size_t)b * p.Ld * p.Hkv + g) * D - (size_t)(n_sel + p.n_static) * HD;
  const uint16_t* ks_ = p.k_static ? p.k_static + sb : p.k_dec + db;
  const uint16_t* vs_ = p.v_static ? p.v_static + sb : p.v_dec + db;
  const uint16_t* kd_ = p.k_dec + db;
  const uint16_t* vd_ = p.v_dec + db;
  const int n_static = p.n_static;
  const unsigned* const rowtab_p = rowtab;
  unsigned own_off[T::BPW];   // byte offset of this lane's rows within a tile of consecutive rows
#pragma unroll
  for (int j = 0; j < T::BPW; ++j) own_off[j] = 2u * dma_row<T>(wave, lane, j) * HD + 16u * dma_chunk<T>(wave, lane);
  const unsigned chunk_off = 16u * dma_chunk<T>(wave, lane);
  // Row offsets of a gathered tile (for other tiles whatever the table holds,
  // unused): read one tile ahead, so that issuing a DMA waits for no LDS read.
  auto peek = [=](int t, unsigned (&o)[T::BPW]) PD_INLINE {
    const unsigned* tab = rowtab_p + min(t * T::BN - j_lo, kDecodeTableRows - T::BN);
#pragma unroll
    for (int j = 0; j < T::BPW; ++j) o[j] = tab[dma_row<T>(wave, lane, j)];
  };
  auto off = [=](const TileSrc& ts, const unsigned (&o)[T::BPW], int j) PD_INLINE {
    return ts.table ? o[j] + chunk_off : own_off[j];
  };
  auto tile = [=](int t) PD_INLINE {
    const int r0 = t * T::BN, n_stat = n_sel + n_static;
    const bool gath = r0 < n_sel, stat = r0 < n_stat;
    const int end = gath ? n_sel : (stat ? n_stat : L_kv);   // rows up to end lie in one buffer
    // ubytes() of all before any is selected: the compiler would select among the
    // captures' addresses, which puts them into scratch memory.
    const char *kg = ubytes(kc), *ks = ubytes(ks_), *kd = ubytes(kd_);
    const char *vg = ubytes(vc), *vs = ubytes(vs_), *vd = ubytes(vd_);
    const size_t at = gath ? 0 : (size_t)r0 * HD * 2;
    return TileSrc{(gath ? kg : (stat ? ks : kd)) + at, (gath ? vg : (stat ? vs : vd)) + at, gath ? 0 : (long long)T::BN * HD * 2, (end - r0) / T::BN - 1,
                   r0 + T::BN <= end, gath};
  };
  auto mixed = [=](auto V, int r, unsigned c, uint32_t lds) PD_INLINE {
    r = min(r, L_kv - 1);
    const bool gath = r < n_sel;
    const unsigned tab = rowtab_p[gath ? r - j_lo : 0], at = gath ? tab : 2u * HD * r;
    const char *cg = ubytes(V ? vc : kc), *st = ubytes(V ? vs_ : ks_), *dc = ubytes(V ? vd_ : kd_);
    dma16((gath ? cg : (r < n_sel + n_static ? st : dc)) + at + c, lds);
  };
  // The Q loads overlap the row-table loads above; both have landed here.
  q_landed(st);
  auto softmax = [&](int t, auto last, auto keys, f32x16 (&s)[2], uint32_t (&pk)[16], bf16x8 (&vf)[T::NF], const uint16_t* vs) PD_INLINE {
    const int kv_valid = decltype(last)::value ? min(T::BN, L_kv - t * T::BN) : T::BN;
    softmax_phase<D, false, decltype(keys)::value>(st, s, pk, vf, vs, fa, grp, l32, p.scale_log2, kv_valid, MassRange{0, 0, 0, 0, 0});
  };
  if constexpr (NW == 8) {
    if (wave_active)
      sweep_pingpong<D, true>(st, Kb, Vb, fa, wave, lane, t_begin, t_end, L_kv - (t_end - 1) * T::BN, peek, off, tile, mixed, softmax);
    else
      sweep_pingpong<D, false>(st, Kb, Vb, fa, wave, lane, t_begin, t_end, L_kv - (t_end - 1) * T::BN, peek, off, tile, mixed, softmax);
  } else {
    auto no_hook = [](int, const uint16_t*, const uint16_t*) {};
    if (wave_active)
      sweep_pair<D, true>(st, Kb, Vb, fa, wave, lane, t_begin, t_end, L_kv - (t_end - 1) * T::BN, peek, off, tile, mixed, no_hook, softmax);
    else
      sweep_pair<D, false>(st, Kb, Vb, fa, wave, lane, t_begin, t_end, L_kv - (t_end - 1) * T::BN, peek, off, tile, mixed, no_hook, softmax);
  }
  if (!wave_active) return;

  if (rho >= GL) return;
  const int hq = g * p.G + rho / p.Ld;
  const int rr = rho % p.Ld;
  const float ltot = (lane & 16) ? st.l[1] : st.l[0];
  // No weight in this shard (every score -inf): zeros of weight zero in the merge.
  float inv = p.S > 1 && ltot == 0.f ? 0.f : 1.0f / ltot;
  float lse2 = st.m + __log2f(ltot);
  if (kCheckIndices && bad_index) inv = lse2 = __uint_as_float(kNanWord);
  if (p.S == 1) {
    const size_t orow = (((size_t)b * p.Ld + rr) * p.Hq + hq) * D;
    if (p.out_f32) store_row_f32<D>(reinterpret_cast<float*>(p.o_dec) + orow, st, inv, grp);
    else store_row_bf16<D>(reinterpret_cast<uint16_t*>(p.o_dec) + orow, st, inv, grp);
    if (p.lse_dec && grp == 0) p.lse_dec[((size_t)b * p.Hq + hq) * p.Ld + rr] = lse2 * kLn2;
  } else {
    const size_t row = (((size_t)sp * p.B + b) * p.Hq + hq) * p.Ld + rr;
    store_row_f32<D>(p.o_part + row * D, st, inv, grp);
    if (grp == 0) p.lse_part[row] = lse2;
  }
}

// ---------------------------------------------------------------------------
// Eq. 5, first sum, blockIdx.x = (b, n, h): the query rows of head h and
// their final LSE are staged in LDS (up to 128 rows per pass), and the 4 waves
// of each of gridDim.y workgroups split the C content keys in 32-key blocks, so every
// key row is read from HBM once.  S = Q_q K_c^T on MFMA (A: query rows from LDS, B: key rows from
// global memory, the next block's prefetched), each key's mass exp2(S*scale -
// lse2(row)) summed in the lane that holds the key.  The head's sum is added
// in place to its per-head second sum (written by the prefill), or replaces
// it for the query-to-chunk score; head_sum_rank_kernel then sums the heads.
// Query row r's 16-byte chunk c sits at chunk c ^ (r % CH) of its LDS row, so
// that the 16 lanes of a ds_read_b128 pass (16 rows, one chunk) hit 16
// different bank groups.
template <int D>
__global__ __launch_bounds__(256) void escore2_bf16_kernel(EscoreArgs p) {
  constexpr int KS = D / 16, CH = D / 8, QB = 128;
  __shared__ __attribute__((aligned(16))) uint16_t qs[QB * D];
  __shared__ __attribute__((aligned(16))) float ls[QB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, grp = lane >> 5;
  const size_t bnh = blockIdx.x;   // (b * N + n) * Hq + h
  const int h = (int)(bnh % p.Hq);
  const size_t bn = bnh / p.Hq;
  const int b = (int)(bn / p.N);
  const int g = h / p.G, C1 = p.C + 1;
  const size_t qm_base = (p.qm_per_chunk ? bn : (size_t)b) * (size_t)(p.Lq + p.Lm);
  const uint16_t* kbase = p.k_cache + ((bn * p.Hkv + g) * C1 + 1) * D;   // content row j at kbase + j*D
  const float* lse = p.lse_q + bnh * p.Lq;
  float* ph = p.part_io + bnh * p.C;
  const int nkb = (p.C + 31) / 32;
  auto load_k = [&](int kb, bf16x8 (&kf)[KS]) {
    const int j = kb * 32 + l32;
    const uint16_t* src = j < p.C ? kbase + (size_t)j * D : nullptr;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[ks] = src ? __builtin_bit_cast(bf16x8, ld16(src + 16 * ks + 8 * grp)) : bf16x8{0};
  };
  for (int r0 = 0; r0 < p.Lq; r0 += QB) {
    const int nr = min(QB, p.Lq - r0);
    if (r0 > 0) __syncthreads();   // the previous pass is done with qs, ls
    for (int u = tid; u < QB * CH; u += 256) {
      const int r = u / CH, c = u % CH;
      const u32x4 v = r < nr ? ld16(p.q_qm + ((qm_base + r0 + r) * p.Hq + h) * D + 8 * c) : u32x4{0u, 0u, 0u, 0u};
      st16(qs + r * D + 8 * (c ^ (r % CH)), v);
    }
    for (int r = tid; r < QB; r += 256) ls[r] = r < nr ? lse[r0 + r] : INFINITY;
    __syncthreads();
    bf16x8 kf[KS], kn[KS];
    const int kb0 = blockIdx.y * 4 + wave, step = 4 * gridDim.y;
    if (kb0 < nkb) load_k(kb0, kf);
    for (int kb = kb0; kb < nkb; kb += step) {
      if (kb + step < nkb) load_k(kb + step, kn);
      float colsum = 0.f;
#pragma unroll
      for (int qb = 0; qb < QB / 32; ++qb) {
        if (qb * 32 >= nr) break;
        const int row = qb * 32 + l32;
        f32x16 sacc = f32x16{0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8 qa = __builtin_bit_cast(bf16x8, ld16(qs + row * D + 8 * ((2 * ks + grp) ^ (row % CH))));
          sacc = mfma32x32x16(qa, kf[ks], sacc);
        }
        // Row (query) of element r: qb*32 + 8*(r/4) + 4*grp + r%4.
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 l4 = *reinterpret_cast<const f32x4*>(ls + qb * 32 + 8 * i + 4 * grp);
#pragma unroll
          for (int e = 0; e < 4; ++e) colsum += fast_exp2(sacc[4 * i + e] * p.scale_log2 - l4[e]);
        }
      }
      const float v = colsum + __shfl_xor(colsum, 32);
      const int j = kb * 32 + l32;
      if (grp == 0 && j < p.C) ph[j] = (p.q2c && r0 == 0) ? v : ph[j] + v;
      if (kb + step < nkb) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[ks] = kn[ks];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Host-side launchers.
template <int D>
static hipError_t launch_prefill_d(const PrefillArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(prefill_bf16_kernel<D>, dim3(a.total), dim3(Tile<D>::NT), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_prefill_bf16(const PrefillArgs& a, int head_dim, hipStream_t s) {
  return head_dim == 128 ? launch_prefill_d<128>(a, s) : launch_prefill_d<64>(a, s);
}

// Which sweep decodes: prefers_eight_waves (its rule and figures are there) where the
// kernel has one, d = 128.
template <int D, int NW>
static hipError_t launch_decode_w(DecodeArgs a, hipStream_t s) {
  a.n_qt = (a.G * a.Ld + Tile<D, NW>::BM - 1) / Tile<D, NW>::BM;
  a.total = a.B * a.Hkv * a.n_qt * a.S;
  hipLaunchKernelGGL((decode_bf16_kernel<D, NW>), dim3(a.total), dim3(Tile<D, NW>::NT), 0, s, a);
  return hipGetLastError();
}
template <int D>
static hipError_t launch_decode_d(const DecodeArgs& a, hipStream_t s) {
  if constexpr (D == 128) {
    const int tiles = (a.n_sel + a.n_static + a.Ld + 63) / 64;
    if (prefers_eight_waves((long long)a.B * a.Hkv, a.G * a.Ld, tiles, a.S)) return launch_decode_w<D, 8>(a, s);
  }
  return launch_decode_w<D, 4>(a, s);
}
hipError_t launch_decode_bf16(const DecodeArgs& a, int head_dim, hipStream_t s) {
  return head_dim == 128 ? launch_decode_d<128>(a, s) : launch_decode_d<64>(a, s);
}

// Workgroups up to which the keys of a head are split in the token scores.  With
// one workgroup a head few chunks leave each SIMD one wave, which waits for its own
// keys, MFMAs and exponentials in turn: 120 heads of d = 64 take 13.0 us in one piece
// and 7.6 in seven, 256 of d = 128 22 and 19 in four, 448 27 and 26 in two.  Every
// workgroup stages the query rows again, so up to 2048 of them cost more (22 us for
// 256 heads, 28 for 448).
constexpr int kEscoreGroups = 1024;
template <int D>
static hipError_t launch_escore_d(const EscoreArgs& a, hipStream_t s) {
  const long long heads = (long long)a.B * a.N * a.Hq;
  const int splits = (int)std::max(1LL, std::min<long long>(((a.C + 31) / 32 + 3) / 4, kEscoreGroups / heads));
  hipLaunchKernelGGL(escore2_bf16_kernel<D>, dim3((unsigned)heads, splits), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_escore_bf16(const EscoreArgs& a, int head_dim, hipStream_t s) {
  return head_dim == 128 ? launch_escore_d<128>(a, s) : launch_escore_d<64>(a, s);
}

}  // namespace pd
