// The attention tile engine shared by the stand-alone attention kernels and the fused selection +
// attention kernel (paper Sec. 4.2, eq. fac_output): 16 cached rows at a time, both products of a tile on the
// matrix cores, a running softmax per query head of the GQA group.  bf16 caches:
//
//   logits  C[row][head] = K_tile (16 rows x 128 dims) . Q^T: four v_mfma_f32_16x16x32_bf16; lane
//           (lo = lane mod 16, hi = lane / 16) supplies chunks hi, hi+4, hi+8, hi+12 (16 bytes each) of
//           K row lo and receives the logits of rows 4hi .. 4hi+3 for query head lo;
//   output  O[head][dim] += P (16 heads x 16 rows) . V_tile (16 rows x 128 dims): the lane's four
//           weights are already where the A operand wants them (head lo, rows 4hi .. 4hi+3).  The B
//           operand wants, per lane, the same four rows at ONE head dim: lane (lo, hi) loads 16 bytes
//           (dims 8lo .. 8lo+7) of V rows 4hi .. 4hi+3, and MFMA j of eight takes dim 8lo + j of each:
//           two byte permutes per MFMA.  Its result column lo is head dim 8lo + j, its rows 4hi .. 4hi+3
//           are query heads 4hi .. 4hi+3.
// The weights are float32 numbers in [0, 1]; the matrix cores take bf16.  Each weight goes in as
// hi + lo, hi = its top 16 bits, lo = the top 16 bits of the exact remainder: k-slots 0-3 of the 32-deep
// MFMA carry the hi parts, slots 4-7 the lo parts, against the same four V values twice.  What is
// dropped is below 2^-16 of the weight; V is bf16 already, products are exact, sums float32.
//
// float32 caches: v_mfma_f32_16x16x4_f32, float32 throughout, 32 for each product.
//   logits  lane (lo, hi) supplies chunks hi, hi+4, .., hi+28 (16 bytes each) of K row lo; MFMA (i, j) takes float
//           j of chunk hi + 4i from all lanes: head dims 4 (hi + 4i) + j in k-slot hi.
//   output  k-slot hi of MFMA (e, j) is row 4hi + e: the lane's own weight of it (head lo) as the A operand, and head
//           dim 8lo + j of it as the B operand: the lane's 32 bytes of V row 4hi + e.  Nothing is permuted.
// One tile is 64 MFMAs of 32 cycles; a CU's four matrix cores keep up with 75 KB per us, more than a CU loads.
#pragma once

#include <type_traits>

#include "attend_common.h"

namespace fasa {

// 2^x on the hardware's own instruction: results below 2^-126 become 0 (the library function scales around
// that at five instructions more).  Softmax weights are at most 1 and are summed with one that is 1.
__device__ __forceinline__ float exp2_weight(float x) { return __builtin_amdgcn_exp2f(x); }

// One lane's share of a tile: the chunks hi, hi + 4, .. of K row lo and head dims 8lo .. 8lo+7 of V rows 4hi .. 4hi+3.
// load_k: row lo of K, from its chunk hi on; load_v: V row 4hi + e, from its head dim 8lo on.
template <typename ET> struct TileKV;
template <> struct TileKV<uint16_t> {
  static constexpr int kPieces = 1;      // 16-byte pieces of a lane's share of a V row
  uint4 kc[4], vr[4];
  template <bool STREAM = false>
  __device__ __forceinline__ void load_k(const uint16_t* p) {
#pragma unroll
    for (int i = 0; i < 4; ++i) kc[i] = load_u128<STREAM>(p + 32 * i);
  }
  template <bool STREAM = false>
  __device__ __forceinline__ void load_v(int e, const uint16_t* p) { vr[e] = load_u128<STREAM>(p); }
  __device__ __forceinline__ uint4 v_piece(int e, int) const { return vr[e]; }
};
template <> struct TileKV<float> {
  static constexpr int kPieces = 2;
  f32x4_t kc[8], vr[4][2];
  __device__ __forceinline__ void load_k(const float* p) {
#pragma unroll
    for (int i = 0; i < 8; ++i) kc[i] = *reinterpret_cast<const f32x4_t*>(p + 16 * i);
  }
  __device__ __forceinline__ void load_v(int e, const float* p) {
    vr[e][0] = *reinterpret_cast<const f32x4_t*>(p);
    vr[e][1] = *reinterpret_cast<const f32x4_t*>(p + 4);
  }
  __device__ __forceinline__ uint4 v_piece(int e, int i) const { return __builtin_bit_cast(uint4, vr[e][i]); }
};
// K rows of a bf16 tile that were loaded as V's are (lane (lo, hi): chunk lo of rows 4hi .. 4hi + 3), as the matrix cores want them: through 4 KB of LDS of the wave's
// own.  Row r's chunk c goes to place c ^ r, so that writes and reads touch all banks evenly.  A load of the latter kind is half a line of each of 16 rows, and
// lines are what a compute unit's request rate is in: 128 rows take one 1.45 us that way, 1.0 as whole rows; 256 of K and V 3.35, 2.8 (256 compute units at
// once: 4.45, 4.3).  Rows next to each other gain nothing: full KV of 8 rows of 32768 23.3 -> 23.7, and 24.3 with K read non-temporal.
constexpr int kTurnWords = 16 * kHeadDim / 8;                 // uint4s
__device__ __forceinline__ void turn_k(uint4 (&kc)[4], uint4* lds, int lo, int hi) {
#pragma unroll
  for (int i = 0; i < 4; ++i) lds[(4 * hi + i) * 16 + (lo ^ (4 * hi + i))] = kc[i];
  // (the wave's LDS operations complete in order; the fences only keep the compiler from moving them)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int i = 0; i < 4; ++i) kc[i] = lds[lo * 16 + ((hi + 4 * i) ^ lo)];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
template <typename ET> constexpr int kChunk = 16 / (int)sizeof(ET);   // head dims per chunk of a K row

// G: most query heads per KV head (1 .. 8; the tile is padded to 16 heads, whose results nobody reads); kernels
// with one instance for all group sizes pass the actual number as `heads` (<= G)
template <int G, typename ET = uint16_t>
struct MfmaTile {
  static constexpr bool F32 = sizeof(ET) == 4;
  using QT = typename std::conditional<F32, f32x4_t, bf16x8_t>::type;
  using KV = TileKV<ET>;
  QT qb[F32 ? 8 : 4];    // B operands of the logits: Q^T, column lo, chunks hi + 4i
  f32x4_t oc[8];         // oc[j][e]: weighted V of query head 4hi + e at head dim 8lo + j
  float m_run, l_run;    // of query head lo (log2 domain); l_run over this lane's rows only until finish()

  // The group's queries.  Lanes beyond the group take its last head again, whose results nobody reads: no load stands
  // under a test, because the compiler may wait for it where the branches meet, and did: the first rows were only
  // requested when the queries were there (2 x 8 rows, 1250 of 20011 tokens selected: 8.33 us, like this 8.00).
  __device__ __forceinline__ void load_q(const ET* q_group /* [G][128] */, int lo, int hi) {
    const ET* p = q_group + (size_t)min(lo, G - 1) * kHeadDim + kChunk<ET> * hi;
#pragma unroll
    for (int i = 0; i < (F32 ? 8 : 4); ++i) qb[i] = __builtin_bit_cast(QT, *reinterpret_cast<const uint4*>(p + 4 * i * kChunk<ET>));
  }
  // With a run-time group size: only the lanes that have a head load, the others carry zeros.  The kernels that use this
  // have 8 or 16 waves on a compute unit at it, whose requests for the copies take as long as the wait
  // (decode step in one launch, 8 rows of 1531, 192 selected: 9.27 us, with copies 9.30; of 6000, 250: 11.95 / 11.98).
  __device__ __forceinline__ void load_q(const ET* q_group /* [heads][128] */, int lo, int hi, int heads) {
#pragma unroll
    for (int i = 0; i < (F32 ? 8 : 4); ++i) {
      uint4 x = make_uint4(0, 0, 0, 0);
      if (lo < heads) x = *reinterpret_cast<const uint4*>(q_group + (size_t)lo * kHeadDim + kChunk<ET> * (hi + 4 * i));
      qb[i] = __builtin_bit_cast(QT, x);
    }
  }
  __device__ __forceinline__ void reset() {
#pragma unroll
    for (int j = 0; j < 8; ++j) oc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    m_run = kNegBig;
    l_run = 0.f;
  }
  // scaled logits (log2 domain) of rows 4hi .. 4hi+3 of the tile for query head lo
  __device__ __forceinline__ void logits(const KV& kv, float scale_log2e, float (&sv)[4]) const {
    // The scaled logit is rounded once and that rounded value is what the running maximum and the
    // exponent see: the scaling is never fused into the subtraction of the maximum (the weight of
    // the maximal row must be exactly 1).
#pragma clang fp contract(off)
    f32x4_t c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};   // two chains of two: half the latency
    if constexpr (F32) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv.kc[i][0], qb[i][0], c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv.kc[i][1], qb[i][1], c1, 0, 0, 0);
        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv.kc[i][2], qb[i][2], c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv.kc[i][3], qb[i][3], c1, 0, 0, 0);
      }
    } else {
      c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kv.kc[0]), qb[0], c0, 0, 0, 0);
      c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kv.kc[1]), qb[1], c1, 0, 0, 0);
      c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kv.kc[2]), qb[2], c0, 0, 0, 0);
      c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kv.kc[3]), qb[3], c1, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) sv[e] = (c0[e] + c1[e]) * scale_log2e;
  }
  // Folds the tile into the running softmax: rows with valid[e] false get weight 0.  scs_wave: 16 floats
  // of LDS owned by this wave.
  __device__ __forceinline__ void accumulate(const KV& kv, const float (&sv)[4], const bool (&valid)[4],
                                             float* scs_wave, int lo, int hi) {
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = valid[e] ? sv[e] : -INFINITY;   // weight exp2(-inf) = 0
    accumulate_full(kv, x, scs_wave, lo, hi);
  }
  // a tile whose 16 rows all count (a logit of -inf: weight 0)
  __device__ __forceinline__ void accumulate_full(const KV& kv, const float (&sv)[4], float* scs_wave, int lo, int hi) {
#pragma clang fp contract(off)
    float mx = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
    mx = xor32_max(xor16_max(mx));
    const float m_new = fmaxf(m_run, mx);
    const float sc = exp2_weight(m_run - m_new);
    m_run = m_new;
    float pv[4];
    uint32_t ph[4], pl[4];
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      pv[e] = exp2_weight(sv[e] - m_new);
      psum += pv[e];
      ph[e] = __float_as_uint(pv[e]) & 0xffff0000u;
      pl[e] = __float_as_uint(pv[e] - __uint_as_float(ph[e]));   // exact; its own top 16 bits go in
    }
    l_run = fmaf(l_run, sc, psum);
    // A operand: k-slots (hi, 0..3) = hi parts of rows 4hi .. 4hi+3, (hi, 4..7) = lo parts
    const uint4 aw = make_uint4(__builtin_amdgcn_perm(ph[1], ph[0], 0x07060302u), __builtin_amdgcn_perm(ph[3], ph[2], 0x07060302u),
                                __builtin_amdgcn_perm(pl[1], pl[0], 0x07060302u), __builtin_amdgcn_perm(pl[3], pl[2], 0x07060302u));
    const bf16x8_t pa = __builtin_bit_cast(bf16x8_t, aw);
    // The running sums only need rescaling when some head's maximum moved in this tile - after the first
    // few tiles of a list that is rare, and the whole exchange (the factor of head lo has to reach the
    // lanes that hold head lo's sums, through LDS) and 32 multiplies are skipped: a wave-uniform test.
    if (__ballot(sc != 1.0f) != 0ull) {
      if (hi == 0) scs_wave[lo] = sc;
      // same wave writes and reads: LDS operations of a wave complete in order; the fences only keep the
      // compiler from moving the accesses across
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const float4 s4 = *reinterpret_cast<const float4*>(scs_wave + 4 * hi);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();   // read before the next tile overwrites it
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        oc[j][0] *= s4.x; oc[j][1] *= s4.y; oc[j][2] *= s4.z; oc[j][3] *= s4.w;
      }
    }
    if constexpr (F32) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          oc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[e], kv.vr[e][j >> 2][j & 3], oc[j], 0, 0, 0);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;   // which half of word j / 2
        const uint32_t w0 = j < 2 ? kv.vr[0].x : j < 4 ? kv.vr[0].y : j < 6 ? kv.vr[0].z : kv.vr[0].w;
        const uint32_t w1 = j < 2 ? kv.vr[1].x : j < 4 ? kv.vr[1].y : j < 6 ? kv.vr[1].z : kv.vr[1].w;
        const uint32_t w2 = j < 2 ? kv.vr[2].x : j < 4 ? kv.vr[2].y : j < 6 ? kv.vr[2].z : kv.vr[2].w;
        const uint32_t w3 = j < 2 ? kv.vr[3].x : j < 4 ? kv.vr[3].y : j < 6 ? kv.vr[3].z : kv.vr[3].w;
        const uint32_t b01 = __builtin_amdgcn_perm(w1, w0, sel), b23 = __builtin_amdgcn_perm(w3, w2, sel);
        const bf16x8_t vb = __builtin_bit_cast(bf16x8_t, make_uint4(b01, b23, b01, b23));
        oc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, vb, oc[j], 0, 0, 0);
      }
    }
  }
  // The wave's totals to LDS: sm_m_wave, sm_l_wave [G]; sm_o_wave [G][128].  (A block barrier must follow
  // before another wave reads them.)
  __device__ __forceinline__ void finish(float* sm_m_wave, float* sm_l_wave, float* sm_o_wave, int lo, int hi, int heads = G) {
    l_run = xor32_sum(xor16_sum(l_run));
    if (hi == 0 && lo < heads) { sm_m_wave[lo] = m_run; sm_l_wave[lo] = l_run; }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int g = 4 * hi + e;
      if (g < heads) {
        float4* dst = reinterpret_cast<float4*>(sm_o_wave + g * kHeadDim + 8 * lo);
        dst[0] = make_float4(oc[0][e], oc[1][e], oc[2][e], oc[3][e]);
        dst[1] = make_float4(oc[4][e], oc[5][e], oc[6][e], oc[7][e]);
      }
    }
  }
};

// Workgroup totals from the waves' finish() output, for thread (query head g, 4 head dims d4):
// max, sum of weights at that max, weighted V.  sm_m, sm_l: [NWV][G]; sm_o: [NWV][G][128].
template <int G, int NWV = 4>
__device__ __forceinline__ void tile_wg_totals(const float* sm_m, const float* sm_l, const float* sm_o, int g, int d4,
                                               float& mn, float& ls, float4& a) {
  mn = sm_m[g];
#pragma unroll
  for (int w = 1; w < NWV; ++w) mn = fmaxf(mn, sm_m[w * G + g]);
  ls = 0.f;
  a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int w = 0; w < NWV; ++w) {
    const float sc = exp2f(sm_m[w * G + g] - mn);
    ls = fmaf(sm_l[w * G + g], sc, ls);
    const float4 sw = *reinterpret_cast<const float4*>(sm_o + ((size_t)(w * G + g)) * kHeadDim + 4 * d4);
    a.x = fmaf(sw.x, sc, a.x); a.y = fmaf(sw.y, sc, a.y);
    a.z = fmaf(sw.z, sc, a.z); a.w = fmaf(sw.w, sc, a.w);
  }
}

}  // namespace fasa
