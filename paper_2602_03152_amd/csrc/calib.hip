// Offline calibration (paper Sec. 3.3 eq. ca_k and Alg. 1): contextual agreement of every single
// frequency chunk with the full head, for one query.  Kp_all holds all d/2 FCs, FC-major.  In one launch (bf16, 8 rows or more, of 8193 .. 32768 tokens):
//
//   calib_kernel        workgroups that score a slice of a row's full head each (all planes, fp32 chain in FC order) and list the largest; the last of a row, by
//                       ticket, finds the top-K set; beside them one per (b, h, FC): the scores of the one FC, their top-K set, and how many of it are in the full head's.
//
// or in two:
//
//   calib_full_kernel   the full head's scores and lists; every FC's cut, from a sample;
//   calib_fc_kernel     one workgroup per (b, h): the top-K set of the full head; one per (b, h, FC), as above.
//
// The single-FC scores never exist in memory: a workgroup streams its plane once and writes one number.
// One Llama-3-8B layer at 32768 tokens, K = 2048: 2.3 us for a launch that clears and 29.  The 67 MB of keys are asked for twice, and 123 MB come from memory: 18 us
// at the rate of a large read; then the full head's set and the FCs that come last.  In two launches 36.85: the first's end and the second's, where all
// workgroups select at once, with nothing to stream.
#include <type_traits>

#include "fasa_device.h"
#include "fasa_internal.h"
#include "row_list.h"
#include "score_common.h"
#include "select_common.h"

namespace fasa {

constexpr int kCalibMaxCtx = 262144;   // a row's set of an FC lives in LDS (33 KB)
constexpr int kCalibPerThread = 16;    // scores in flight per thread
constexpr int kCalibShort = 8192;      // tokens of a row that the registers of 256 threads hold twice over
constexpr int kCalibWords0 = (kCalibShort + 30) / 31, kCalibWords1 = (32768 + 30) / 31;   // of a set (CalibSets)

// The top-K sets.  A word has 31 tokens, and its top bit says that it is there: the full head's set is read with no other sign.
struct CalibSets {
  uint32_t* full;      // [row][words]: of the full head
  uint32_t* fc;        // [row][FC][words]: of an FC whose workgroup did not find the full head's
  uint32_t* state;     // [row][FC]: 0; 1: the FC's set is in fc; 2: the full head's is in full
  uint32_t* tickets;   // [row]: workgroups that have scored their slices of the full head
  int words;           // ceil(N / 31)
  float4* cuts;        // [row][FC]: the cut of the FC's list, the largest of the scores it is from, the sums of the queries' two components
  // The full head's largest scores by segments (row_list.h); pitch 0: none (launch_calib)
  uint32_t* lists;
  uint2* lims;
  int pitch, nsegs;
  __host__ __device__ __forceinline__ size_t list_words() const { return ((size_t)nsegs * (pitch + pitch / 4) + 3) & ~(size_t)3; }
  __device__ __forceinline__ ListRow list(int row) const {
    uint32_t* keys = lists + row * list_words();
    return {keys, keys + nsegs * pitch, lims + (size_t)row * nsegs, pitch};
  }
  template <int NT>
  __device__ __forceinline__ void clear(int row) const {
    for (int i = threadIdx.x; i < words; i += NT) full[(size_t)row * words + i] = 0;
    if (threadIdx.x < kHeadDim / 2) state[row * (kHeadDim / 2) + threadIdx.x] = 0;
    if (threadIdx.x == 0) tickets[row] = 0;
  }
};
constexpr uint32_t kCalibThere = 0x80000000u;
constexpr int kCalibLooks = 64;        // for the full head's set, some 50 us
__device__ __forceinline__ void set_bit(uint32_t* bits, uint32_t tok) { atomicOr(&bits[tok / 31u], 1u << (tok % 31u)); }

// The cut of an FC's list, by a wave: of 1024 scores (float32: 512; a fourth of that for rows that one workgroup of 256 holds), four (two) neighbours at each of
// kSpots places, the one that the K best reach and a good many more.  Made where the planes go by anyway, beside the full head's scores: an FC's workgroup that began with it
// had its first 64 KB in flight, and nothing behind them, until its sample had come, was counted and the cut known (8 rows of 32768: 8.8 us).
template <typename ET, int SPOTS>
struct CalibSample {
  static constexpr int TPT = ScoreTraits<ET>::TPT, L = SPOTS / kWave, SMP = SPOTS * TPT;
  uint4 w[L];
  int n[L];
  __device__ __forceinline__ void request(const ET* p, int N) {
    const int lane = lane_id();
#pragma unroll
    for (int i = 0; i < L; ++i) {
      n[i] = (int)((long long)(i * kWave + lane) * N / SPOTS) & ~(TPT - 1);
      w[i] = *reinterpret_cast<const uint4*>(p + (size_t)n[i] * 2);
    }
  }
  __device__ __forceinline__ void make_cut(float qlo, float qhi, int N, int kk, uint32_t* bins, float& cut, float& top) const;
};
template <typename ET, int SPOTS>
__device__ __forceinline__ void CalibSample<ET, SPOTS>::make_cut(float qlo, float qhi, int N, int kk, uint32_t* bins, float& cut, float& top) const {
  float x[L * TPT];
#pragma unroll
  for (int i = 0; i < L; ++i) {
    float s[TPT];
#pragma unroll
    for (int k = 0; k < TPT; ++k) s[k] = 0.f;
    fma_pairs<ET>(w[i], qlo, qhi, s);
#pragma unroll
    for (int k = 0; k < TPT; ++k) x[i * TPT + k] = n[i] + k < N ? s[k] : s[0];
  }
  // neighbours may be alike: a wider margin than independent ones would need
  const float ps = (float)kk * ((float)SMP / (float)N);
  const int r = (int)(ps + 5.0f * sqrtf(ps) + 3.0f);
  cut = -INFINITY;
  top = 0.f;
  if (r <= SMP) cut = list_cut(x, r, bins, top);
}

template <typename ET, int SPOTS>
__device__ __forceinline__ void calib_cut(const ET* p, float qlo, float qhi, int N, int kk, uint32_t* bins, float& cut, float& top) {
  CalibSample<ET, SPOTS> sample;
  sample.request(p, N);
  sample.make_cut(qlo, qhi, N, kk, bins, cut, top);
}

// Full-head scores of a slice of 256 * TPT tokens: 1-D grid of rows * 16 workgroups whose waves find an FC's cut each, and rows * nslices.
template <typename ET, int PAIR_SHIFT, int PAIR_ADD>
__global__ __launch_bounds__(256, 4) void calib_full_kernel(const ET* __restrict__ q, const ET* __restrict__ Kp,
                                                         float* __restrict__ S, CalibSets sets, int rows, int nslices,
                                                         uint32_t m_slices, int G, int N, int n_cap, int kk) {
  constexpr int D = kHeadDim, F = D / 2, NW = 16;
  constexpr int TPT = ScoreTraits<ET>::TPT;
  __shared__ SegLds seg[4];
  __shared__ float ql[kMaxGroup][D];
  __shared__ float2 qs[F];
  const int t = threadIdx.x, n_cuts = rows * (F / 4);
  if ((int)blockIdx.x < n_cuts) {
    int r, part;                                              // (on the die of the row's full head, which reads the same lines)
    constexpr uint32_t m_cuts = div_magic(F / 4, 65535);
    row_slice_of_block(rows, F / 4, m_cuts, r, part);
    const int f = part * 4 + __builtin_amdgcn_readfirstlane(t >> 6), id = r * F + f;
    const ET* qh = q + (size_t)r * G * D + (f << PAIR_SHIFT);
    ET a[kMaxGroup], b[kMaxGroup];
#pragma unroll
    for (int g = 0; g < kMaxGroup; ++g) {
      a[g] = qh[(size_t)min(g, G - 1) * D];
      b[g] = qh[(size_t)min(g, G - 1) * D + PAIR_ADD];
    }
    float qlo = 0.f, qhi = 0.f;
#pragma unroll
    for (int g = 0; g < kMaxGroup; ++g) {   // g ascending, as everywhere
      float x, y;
      if constexpr (sizeof(ET) == 2) { x = __uint_as_float((uint32_t)a[g] << 16); y = __uint_as_float((uint32_t)b[g] << 16); }
      else { x = a[g]; y = b[g]; }
      qlo += g < G ? x : 0.f;
      qhi += g < G ? y : 0.f;
    }
    const ET* p = Kp + (size_t)id * n_cap * 2;
    float cut, top;
    if (N <= kCalibShort) calib_cut<ET, 64>(p, qlo, qhi, N, kk, seg[t >> 6].bins, cut, top);
    else calib_cut<ET, 256>(p, qlo, qhi, N, kk, seg[t >> 6].bins, cut, top);
    if ((t & 63) == 0) sets.cuts[id] = make_float4(cut, top, qlo, qhi);
    return;
  }
  int row, slice;
  row_slice_of_block(rows, nslices, m_slices, row, slice, blockIdx.x - (unsigned)n_cuts);
  if (slice == 0) sets.clear<256>(row);                       // for the launch behind this one
  const ET* qh = q + (size_t)row * G * D + (t & (D - 1));
  ET qcol[kMaxGroup / 2];                                   // head dim t mod 128 of query heads t / 128, + 2, ...
#pragma unroll
  for (int j = 0; j < kMaxGroup / 2; ++j) qcol[j] = qh[(size_t)min((t >> 7) + 2 * j, G - 1) * D];
  const int n0 = (slice * 256 + t) * TPT;
  const bool active = n0 < N;
  const ET* p = Kp + ((size_t)row * F * n_cap + (active ? n0 : 0)) * 2;
  const size_t plane = (size_t)n_cap * 2;
  uint4 w[NW];
#pragma unroll
  for (int u = 0; u < NW; ++u) w[u] = *reinterpret_cast<const uint4*>(p + (size_t)u * plane);
#pragma unroll
  for (int j = 0; j < kMaxGroup / 2; ++j) {
    if constexpr (sizeof(ET) == 2) ql[(t >> 7) + 2 * j][t & (D - 1)] = __uint_as_float((uint32_t)qcol[j] << 16);
    else ql[(t >> 7) + 2 * j][t & (D - 1)] = qcol[j];
  }
  __syncthreads();
  if (t < F) {   // g ascending, as everywhere
    float lo = 0.f, hi = 0.f;
    for (int g = 0; g < G; ++g) {
      lo += ql[g][t << PAIR_SHIFT];
      hi += ql[g][(t << PAIR_SHIFT) + PAIR_ADD];
    }
    qs[t] = make_float2(lo, hi);
  }
  __syncthreads();
  float acc[TPT];
#pragma unroll
  for (int k = 0; k < TPT; ++k) acc[k] = 0.f;
  // 16 planes in flight: a plane's register takes the plane 16 further on as soon as it is used.  (Not
  // unrolled: the compiler would put all 64 loads first, and spill.)
#pragma unroll 1
  for (int f0 = 0; f0 < F; f0 += NW) {
#pragma unroll
    for (int u = 0; u < NW; ++u) {
      const float2 qf = qs[f0 + u];
      fma_pairs<ET>(w[u], qf.x, qf.y, acc);
      w[u] = *reinterpret_cast<const uint4*>(p + (size_t)min(f0 + NW + u, F - 1) * plane);
    }
  }
  if (active) {
    float* out = S + (size_t)row * n_cap + n0;
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      if (n0 + k < N) out[k] = acc[k];
  }
  if constexpr (TPT * kWave == kListSeg) {
    const int ls = __builtin_amdgcn_readfirstlane(slice * (256 * TPT / kListSeg) + (t >> 6));
    if (sets.pitch && ls * kListSeg < N)
      seg_list<false>(acc, min(N - ls * kListSeg, kListSeg), ls, sets.list(row), seg[t >> 6]);
  }
}

// What calib_kernel counts in, and the words that say that a set is there: a workgroup per row.
__global__ __launch_bounds__(256) void calib_clear_kernel(CalibSets sets) { sets.clear<256>(blockIdx.x); }

// Full-head scores of a slice of 1024 tokens (bf16), two a thread: a workgroup reads twice as much as an FC's, and a compute unit with one of them and two FCs' as much as
// any other.
constexpr int kSliceNT = 512, kSliceTokens = 2 * kSliceNT;
struct CalibSlice {
  SegLds seg[4];
  float ql[kMaxGroup][kHeadDim];
  float2 qs[kHeadDim / 2];
  __align__(16) float score[kSliceTokens];
};
template <int PAIR_SHIFT, int PAIR_ADD>
__device__ __forceinline__ void calib_slice(CalibSlice& sm, const uint16_t* __restrict__ q, const uint16_t* __restrict__ Kp, float* __restrict__ S,
                                            const CalibSets& sets, int row, int slice, int G, int N, int n_cap) {
  constexpr int D = kHeadDim, F = D / 2, NW = 16, QH = kSliceNT / D, QL = kMaxGroup / QH;
  const int t = threadIdx.x;
  const uint16_t* qh = q + (size_t)row * G * D + (t & (D - 1));
  uint16_t qcol[QL];                                          // head dim t mod 128 of query heads t / 128, + QH, ...
#pragma unroll
  for (int j = 0; j < QL; ++j) qcol[j] = qh[(size_t)min((t >> 7) + QH * j, G - 1) * D];
  const int n0 = slice * kSliceTokens + 2 * t;
  const uint16_t* p = Kp + ((size_t)row * F * n_cap + (n0 < N ? n0 : 0)) * 2;
  const size_t plane = (size_t)n_cap * 2;
  uint2 w[NW];
#pragma unroll
  for (int u = 0; u < NW; ++u) w[u] = *reinterpret_cast<const uint2*>(p + (size_t)u * plane);
#pragma unroll
  for (int j = 0; j < QL; ++j) sm.ql[(t >> 7) + QH * j][t & (D - 1)] = __uint_as_float((uint32_t)qcol[j] << 16);
  __syncthreads();
  if (t < F) {   // g ascending, as everywhere
    float lo = 0.f, hi = 0.f;
    for (int g = 0; g < G; ++g) {
      lo += sm.ql[g][t << PAIR_SHIFT];
      hi += sm.ql[g][(t << PAIR_SHIFT) + PAIR_ADD];
    }
    sm.qs[t] = make_float2(lo, hi);
  }
  __syncthreads();
  float acc[2] = {0.f, 0.f};
  // 16 planes in flight: a plane's register takes the plane 16 further on as soon as it is used.  (Not
  // unrolled: the compiler would put all 64 loads first, and spill.)
#pragma unroll 1
  for (int f0 = 0; f0 < F; f0 += NW) {
#pragma unroll
    for (int u = 0; u < NW; ++u) {
      const float2 qf = sm.qs[f0 + u];                        // (as fma_pairs)
      acc[0] = fmaf(qf.y, bf16_hi(w[u].x), fmaf(qf.x, bf16_lo(w[u].x), acc[0]));
      acc[1] = fmaf(qf.y, bf16_hi(w[u].y), fmaf(qf.x, bf16_lo(w[u].y), acc[1]));
      w[u] = *reinterpret_cast<const uint2*>(p + (size_t)min(f0 + NW + u, F - 1) * plane);
    }
  }
  float* out = S + (size_t)row * n_cap + n0;
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (n0 + k < N) st_agent(out + k, acc[k]);
  if (sets.pitch) {
    *reinterpret_cast<float2*>(sm.score + 2 * t) = make_float2(acc[0], acc[1]);
    __syncthreads();
    static_assert(kSliceTokens == 4 * kListSeg, "a segment for each of four waves");
    const int ls = __builtin_amdgcn_readfirstlane(slice * 4 + (t >> 6));
    if (t < kListSeg && ls * kListSeg < N) {
      const float4 x = *reinterpret_cast<const float4*>(sm.score + 4 * t);
      const float xs[4] = {x.x, x.y, x.z, x.w};
      seg_list<true>(xs, min(N - ls * kListSeg, kListSeg), ls, sets.list(row), sm.seg[t >> 6]);
    }
  }
}

// LIST: entries of a row's list.
template <int NT, int WORDS, int LIST>
struct CalibLds {
  static constexpr int kThreads = NT, kWords = WORDS, kList = LIST;
  static constexpr int kSpots = NT == 256 ? 64 : 256;         // of calib_top's sample
  using Tok = typename std::conditional<WORDS <= kCalibWords1, uint16_t, uint32_t>::type;
  union {
    struct { uint32_t score[kList + kWave]; Tok tok[kList + kWave]; };   // what reaches the cut; a place per lane for what does not
    struct { __align__(16) float sample[4 * kSpots]; __align__(16) uint32_t bins[256]; };
  };
  union {                                                     // (the set is made when there is nothing left to count)
    uint32_t hist[kSelBins];
    uint32_t bits[WORDS];
  };
  uint2 cand[kSelCand];
  float2 cut_top;
  uint32_t wtot[NT / kWave], wtot2[NT / kWave];
  uint32_t thr[4];
  uint32_t n_list, n_cnd, count, missing;
  uint32_t early[kHeadDim / 2];
};

// The K best of entries that the threads hold in registers, by one histogram of 512 bins of 2^shift keys from klo on (0: no entry; klo > 0).  win: a thread's entries above
// the K-th's bin; those in it go to sm.cand, and `taken` tells that this thread's candidate `taken_tok` is one of the K.  The histogram is zero at the call, a barrier
// ago, and all have used it when this returns true.  False: fewer than K entries, or too many candidates (it is zero then, a barrier ago).
// (In a loop over a list in LDS, a test around each count and each bit, threshold and set took 4 us: three workgroups on a compute unit are bound by
// instructions there.)
constexpr int kCalibHeld = 8;          // entries per thread of an FC's list
template <int EPT, typename Lds, typename Token>
__device__ __forceinline__ bool calib_held(Lds& sm, const uint32_t (&key)[EPT], Token&& token, uint32_t klo, int shift, int kk, uint32_t& win, bool& taken,
                                           uint32_t& taken_tok) {
  constexpr int NT = Lds::kThreads;
  const int t = threadIdx.x, lane = t & 63;
  uint32_t bin[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {                             // (what is not counted: a word of the lane's own)
    bin[k] = key[k] >= klo ? min((key[k] - klo) >> shift, (uint32_t)kListBins - 1u) : (uint32_t)(kListBins + lane);
    atomicAdd(&sm.hist[bin[k]], 1u);
  }
  __syncthreads();
  const BinAt b = wave_find_bin(sm.hist, (uint32_t)kk);
  if (b.n == 0 || b.n > kSelCand) {
    __syncthreads();
    for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;
    __syncthreads();
    return false;
  }
  const int need = kk - b.above;
  uint32_t act = 0;
  win = 0;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    win |= bin[k] > (uint32_t)b.bin && bin[k] < (uint32_t)kListBins ? 1u << k : 0u;
    act |= bin[k] == (uint32_t)b.bin ? 1u << k : 0u;
  }
#pragma unroll
  for (int k = 0; k < EPT; ++k) {                             // (few lanes have one)
    if (act >> k & 1u) {
      const uint32_t c = __builtin_amdgcn_atomic_inc32(&sm.n_cnd, 0xffffffffu, __ATOMIC_RELAXED, "workgroup");
      sm.cand[c & (kSelCand - 1)] = make_uint2(key[k], token(k));
    }
  }
  __syncthreads();
  taken = false;
  taken_tok = 0;
  static_assert(NT >= kSelCand, "a thread per candidate");
  if ((t & ~(kWave - 1)) < b.n) {                             // (the waves that have any)
    const int rank = rank_in_list<1>(sm.cand, b.n, t);
    taken = t < b.n && rank < need;
    taken_tok = sm.cand[min(t, b.n - 1)].y;
  }
  return true;
}

// Top-K of a row by one workgroup of NT threads, which hold a stretch of it as loaded: load1(i, c0) requests piece i of what the
// scores of tokens c0 .. c0 + NT * kCalibPerThread - 1 are made of (kCalibPerThread / TPT pieces a thread),
// get(c0, i, t, x, full) makes those of tokens c0 + (i * NT + t) * TPT + k, a NaN beyond the row unless it is said to
// be full (cheap: made again in every pass, which keeps 16 registers free and two workgroups of 1024 on a
// compute unit); opaque() hides the pieces from the compiler, which would otherwise keep the scores.
// pick(klo, ktop): the list has been made already, from elsewhere, out of all scores from klo on.  cut(top) is the cut, and a score at the upper end.  score_at(n): one token's score.  The set goes to sm.bits; or, HELD and where the
// threads hold the list (short ones, which a loop goes through in a round or two, gain nothing: 2 rows of 20011 19.8 -> 21.0), to held(win, tok, taken, taken_tok) (calib_held).
// What reaches the cut is gathered into a list in LDS first (some 7 instructions a score per wave, where counting
// and classifying all scores under a test takes 30); a list that comes out short of K or beyond its
// room is not used.  Infinite scores rank like any others; where NaNs rank is unspecified, but the set has K tokens.
template <int TPT, bool HELD, typename Lds, typename Load1, typename Get, typename Opaque, typename Pick, typename Cut, typename ScoreAt, typename Held>
__device__ __forceinline__ void calib_select(Lds& sm, int N, int kk, Load1&& load1, Get&& get, Opaque&& opaque, Pick&& pick, Cut&& cut,
                                             ScoreAt&& score_at, Held&& held) {
  const int t = threadIdx.x;
  constexpr int NT = Lds::kThreads, R = NT * kCalibPerThread, NP = kCalibPerThread / TPT;
  auto load = [&](int c0) {
#pragma unroll
    for (int i = 0; i < NP; ++i) load1(i, c0);
  };
  const bool resident = N <= R;
  if (t == 0) { sm.n_list = 0; sm.n_cnd = 0; sm.thr[2] = 0; }
  for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;
  uint32_t klo = 0, khi = 0xffffffffu, ktop = 0;
  int shift = 22, need = kk, n_cand;
  if (pick(klo, ktop)) {
    shift = first_shift(klo, ktop);
  } else {
    load(0);
    float top;
    const float flo = cut(top);
    __syncthreads();
    klo = 0;
    if (flo > -INFINITY) {
      klo = score_key(flo);
      shift = first_shift(klo, score_key(top));
    }
    const int lane = lane_id();
    // One addition to the list's length per wave and piece: its latency hides behind the other waves, where
    // counting first would make every score twice.
    auto append = [&](int c0, auto full, auto more) {
      int tt = t;
      asm volatile("" : "+v"(tt));                            // (token numbers made anew, not kept)
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        float x[TPT];
        get(c0, i, tt, x, full);
        if constexpr (more) load1(i, c0 + R);                 // a piece of the next stretch where this one's has been used
        unsigned long long m[TPT];
        uint32_t cnt = 0;                                     // of the wave
#pragma unroll
        for (int k = 0; k < TPT; ++k) {
          m[k] = __ballot(x[k] >= flo);
          cnt += (uint32_t)__popcll(m[k]);
        }
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&sm.n_list, cnt);
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
        for (int k = 0; k < TPT; ++k) {
          const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], base));
          // (HELD, whose workgroups share a compute unit with others that need its instruction slots: no branch, and what is not listed to a place of the lane's
          // own: 8 rows of 32768 32.15 -> 32.0)
          const bool in = x[k] >= flo && pos < (uint32_t)Lds::kList;
          const uint32_t at = !HELD || in ? pos : (uint32_t)(Lds::kList + lane);
          if (HELD || in) {
            sm.score[at] = __float_as_uint(x[k]);
            sm.tok[at] = (typename Lds::Tok)(c0 + (i * NT + tt) * TPT + k);
          }
          base += (uint32_t)__popcll(m[k]);
        }
        __builtin_amdgcn_sched_barrier(0);                    // (piece by piece: registers)
      }
    };
    int c0 = 0;
    for (; c0 + R < N; c0 += R) append(c0, std::true_type{}, std::true_type{});
    if (c0 + R == N) append(c0, std::true_type{}, std::false_type{});
    else append(c0, std::false_type{}, std::false_type{});
    __syncthreads();
  }
  const int M = (int)sm.n_list;
  const bool listed = M >= kk && M <= Lds::kList;
  if (HELD && listed && M <= kCalibHeld * NT && klo > 0u) {
    uint32_t key[kCalibHeld], tok[kCalibHeld], win, taken_tok;
    bool taken;
#pragma unroll
    for (int k = 0; k < kCalibHeld; ++k) {
      const int i = k * NT + t, at = min(i, Lds::kList - 1);  // (beyond M: whatever it holds)
      const uint32_t x = sm.score[at];
      tok[k] = sm.tok[at];
      key[k] = i < M ? score_key(__uint_as_float(x)) : 0u;
    }
    if (calib_held<kCalibHeld>(sm, key, [&](int k) { return tok[k]; }, klo, shift + 1, kk, win, taken, taken_tok)) {
      held(win, tok, taken, taken_tok);
      return;
    }
  }
  // Without a list: all scores of the row, told from what lies beyond it by index.  As keys throughout: a NaN score has
  // a place in the order of keys like any other.
  auto for_scores = [&](int c0, auto&& f) {
    int tt = t;
    asm volatile("" : "+v"(tt));
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      float x[TPT];
      get(c0, i, tt, x, std::true_type{});
#pragma unroll
      for (int k = 0; k < TPT; ++k) {
        const int n = c0 + (i * NT + tt) * TPT + k;
        if (n < N) f(score_key(x[k]), n);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  bool none = false;
  for (;;) {
    const bool whole = klo == 0 && khi == 0xffffffffu;
    auto count = [&](uint32_t key) {
      if (key >= klo && key <= khi) atomicAdd(&sm.hist[min((key - klo) >> shift, (uint32_t)kSelBins - 1u)], 1u);
    };
    if (listed) {
      for (int i = t; i < M; i += NT) count(score_key(__uint_as_float(sm.score[i])));
    } else for (int c0 = 0; c0 < N; c0 += R) {
      if (!resident) load(c0);
      opaque();
      for_scores(c0, [&](uint32_t key, int) { count(key); });
    }
    if (find_threshold(sm, klo, khi, shift, need, n_cand)) break;
    if (t == 0) sm.thr[2] = 0;                                     // (all have read it)
    if (n_cand == 0) {
      none = whole;                                                // (fewer than K scores: the callers pass K < N)
      if (none) break;
      klo = 0; khi = 0xffffffffu; shift = 22;                      // the sample misled: the whole range
    }
  }
  for (int i = t; i < Lds::kWords; i += NT) sm.bits[i] = 0;
  __syncthreads();
  if (none) return;
  auto take_one = [&](int n) { set_bit(sm.bits, (uint32_t)n); };
  const bool ranked = n_cand <= kSelCand;
  auto place = [&](uint32_t key, int n) {
    if (key > khi) take_one(n);
    else if (ranked && key >= klo) {
      const uint32_t p = atomicAdd(&sm.n_cnd, 1u);
      if (p < (uint32_t)kSelCand) sm.cand[p] = make_uint2(key, (uint32_t)n);
    }
  };
  if (listed) {
    for (int i = t; i < M; i += NT) {
      place(score_key(__uint_as_float(sm.score[i])), (int)sm.tok[i]);
    }
  } else for (int c0 = 0; c0 < N; c0 += R) {
    if (!resident) load(c0);
    opaque();
    for_scores(c0, place);
  }
  __syncthreads();
  if (ranked) {
    static_assert(NT >= kSelCand, "a thread per candidate");
    if ((t & ~(kWave - 1)) < n_cand) {                        // (the waves that have any)
      const int rank = rank_in_list<1>(sm.cand, n_cand, t);
      if (t < n_cand && rank < need) take_one((int)sm.cand[t].y);
    }
  } else {                                                    // one key, more tokens than the list holds: in index order
    // (Four tokens a thread and pass, of two barriers each.  us, one / four: 8 rows of 32768 whose FCs have thousands of ties 76.6 / 69.1, of 12000 39.4 / 36.9; 8 float32 rows
    // of 12000 with 7 scores 55.0 / 49.2.)
    int tied = 0;
    for (int i0 = 0; i0 < N && tied < need; i0 += 4 * NT) {
      uint32_t mine = 0, tot;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int n = i0 + 4 * t + k;
        mine |= n < N && score_key(score_at(min(n, N - 1))) == klo ? 1u << k : 0u;
      }
      int p = tied + (int)block_prefix_sum<NT>((uint32_t)__popc(mine), sm.wtot, tot);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if ((mine >> k & 1u) && p++ < need) take_one(i0 + 4 * t + k);
      }
      tied += (int)tot;
    }
  }
}

template <int EPT, typename Lds>
__device__ __forceinline__ void calib_bits(Lds& sm, uint32_t win, const uint32_t (&tok)[EPT], bool taken, uint32_t taken_tok) {
  __syncthreads();                                            // (the histogram has been read, and its storage is the set's)
  for (int i = threadIdx.x; i < Lds::kWords; i += Lds::kThreads) sm.bits[i] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < EPT; ++k)
    if (win >> k & 1u) set_bit(sm.bits, tok[k]);
  if (taken) set_bit(sm.bits, taken_tok);
}

// The full head's set out of the row's lists, if the threads hold them (tried): false, where they are longer, or K of their entries don't reach the highest of their
// completeness keys.
template <typename Lds>
__device__ __forceinline__ bool calib_top_listed(Lds& sm, const CalibSets& sets, int row, int N, int kk, bool& tried) {
  constexpr int NT = Lds::kThreads, NWV = NT / kWave, Q = 4;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, per = sets.pitch / 4, nq = sets.nsegs * per;
  if (nq == 0 || nq > Q * NT) return false;
  tried = true;
  const ListRow l = sets.list(row);
  const __amdgpu_buffer_rsrc_t rk = agent_buffer(l.keys);
  uint2 lim = make_uint2(0u, 0u);
  for (int i = t; i < sets.nsegs; i += NT) {
    const uint2 x = ld_agent(l.lims + i);
    lim = make_uint2(max(lim.x, x.x), max(lim.y, x.y));
  }
  uint4 k4[Q];
  uint32_t t4[Q];
#pragma unroll
  for (int u = 0; u < Q; ++u) {
    const int g = min(u * NT + t, nq - 1);
    k4[u] = agent_load_u128(rk, (uint32_t)g * 16u);
    t4[u] = ld_agent(l.toks + g);
  }
  for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;
  if (t == 0) sm.n_cnd = 0;
  const uint32_t a = wave_max_key(lim.x), b = wave_max_key(lim.y);
  if (lane == kWave - 1) { sm.wtot[wave] = a; sm.wtot2[wave] = b; }
  __syncthreads();
  uint32_t klo = 1, ktop = 0;
#pragma unroll
  for (int w = 0; w < NWV; ++w) { klo = max(klo, sm.wtot[w]); ktop = max(ktop, sm.wtot2[w]); }
  uint32_t key[4 * Q];
#pragma unroll
  for (int u = 0; u < Q; ++u) {
    const bool in = u * NT + t < nq;
    key[4 * u] = in ? k4[u].x : 0u; key[4 * u + 1] = in ? k4[u].y : 0u;
    key[4 * u + 2] = in ? k4[u].z : 0u; key[4 * u + 3] = in ? k4[u].w : 0u;
  }
  const float inv_per = __builtin_amdgcn_rcpf((float)per);
  const auto token_of = [&](int quad, uint32_t byte) {        // (quotients of at most 4096 by at most 32: exact)
    return min((uint32_t)(((float)quad + 0.5f) * inv_per) * (uint32_t)kListSeg + (byte & 255u), (uint32_t)N - 1u);
  };
  const auto token = [&](int e) { return token_of((e >> 2) * NT + t, t4[e >> 2] >> (8 * (e & 3))); };
  uint32_t win, taken_tok;
  bool taken;
  if (!calib_held<4 * Q>(sm, key, token, klo, list_shift(klo, ktop), kk, win, taken, taken_tok)) return false;
  uint32_t tok[4 * Q];
#pragma unroll
  for (int e = 0; e < 4 * Q; ++e) tok[e] = token(e);
  calib_bits(sm, win, tok, taken, taken_tok);
  return true;
}

// The full head's top-K set, by the workgroup that scored the last slice of its row, which then counts for the FCs that came first (a
// wave each).  Out of the row's lists, whose entries from the highest of their completeness keys on are all there are; if fewer than K of them are (a row's best lie
// together), or there are none, out of all scores by the cut of a sample.
template <bool SHARED, typename Lds>
__device__ __forceinline__ void calib_top(Lds& sm, const float* __restrict__ S, const CalibSets& sets, float* CA_sum, int row, int N, int n_cap,
                                          int kk) {
  constexpr int NT = Lds::kThreads, F = kHeadDim / 2, NWV = NT / kWave;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, words = sets.words;
  const float* s = S + (size_t)row * n_cap;
  __builtin_amdgcn_s_setprio(3);                              // (64 workgroups may end up waiting to be counted)
  constexpr int SP = Lds::kSpots, SMP = SP * 4;
  const int n_spot = (int)(((long long)(t & (SP - 1)) * N) / SP) & ~3;
  const __amdgpu_buffer_rsrc_t rs = agent_buffer(s);          // (SHARED: scored and listed in this launch)
  const auto scores = [&](int n) {
    if constexpr (SHARED) return agent_load_u128(rs, (uint32_t)n * 4u);
    else return *reinterpret_cast<const uint4*>(s + n);
  };
  const uint4 spot = scores(n_spot);      // (ahead of all that a wait for it would be one for, too)
  bool tried = false;
  const auto pick = [&](uint32_t& klo, uint32_t& ktop) {
    if constexpr (!SHARED && Lds::kWords <= kCalibWords1) return false;   // (no lists: launch_calib)
    if (!sets.pitch || (SHARED && tried)) return false;
    const ListRow l = sets.list(row);
    const __amdgpu_buffer_rsrc_t rk = agent_buffer(l.keys);
    const int per = sets.pitch / 4, nq = sets.nsegs * per;
    uint2 x = make_uint2(0u, 0u);                             // of this thread's segment
    static_assert(NT * kListSeg >= (Lds::kWords - 1) * 31, "one at most");
    uint32_t a = 0, b = 0;
    for (int i = t; i < sets.nsegs; i += NT) {
      x = SHARED ? ld_agent(l.lims + i) : l.lims[i];
      a = max(a, x.x);
      b = max(b, x.y);
    }
    constexpr int U = 2048 / NT;                              // quads in flight
    uint4 k4[U];
    uint32_t t4[U];
    const auto request = [&](int g0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int g = min(g0 + u * NT + t, nq - 1);
        if constexpr (SHARED) k4[u] = agent_load_u128(rk, (uint32_t)g * 16u);
        else k4[u] = reinterpret_cast<const uint4*>(l.keys)[g];
        t4[u] = SHARED ? ld_agent(l.toks + g) : l.toks[g];
      }
    };
    request(0);
    a = wave_max_key(a);
    b = wave_max_key(b);
    if (lane == kWave - 1) { sm.wtot[wave] = a; sm.wtot2[wave] = b; }
    __syncthreads();
    klo = 1;
    ktop = 0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) { klo = max(klo, sm.wtot[w]); ktop = max(ktop, sm.wtot2[w]); }
    if constexpr (!SHARED) {
      // Where a row's best lie together hardly a segment's list reaches the highest of the keys.  How many entries do is told by what is here already, as if
      // a segment had fewer scores by the same factor for every step up from its cut, where it has `pitch`, to its largest.  us, lists read all the same / like this: 4 rows of 70000,
      // K = 3000, rising 56.3 / 54.1, neighbours alike 57.0 / 55.0, independent 47.2 / 47.3 (no lists: 51.5, 52.4, 52.0); 8 of 131072, 4096: 137.4 / 135.8, 184.1 / 182.3, 124.4 /
      // 124.3 (133.8, 179.6, 133.1); 1 of 33000, 1000: 25.1 / 24.2, 25.2 / 24.4, 22.1 / 22.1 (21.65, 21.9, 21.65).
      const float xk = key_score(klo), xc = key_score(x.x), xt = key_score(x.y);
      const float n = t < sets.nsegs && xt > xk ? exp2f(__log2f((float)sets.pitch) * (xt - xk) * __builtin_amdgcn_rcpf(xt - xc)) : 0.f;
      const uint32_t e = wave_prefix_sum((uint32_t)(16.f * n));
      __syncthreads();                                        // (all have read the keys)
      if (lane == kWave - 1) sm.wtot[wave] = e;
      __syncthreads();
      uint32_t reach = 0;
#pragma unroll
      for (int w = 0; w < NWV; ++w) reach += sm.wtot[w];
      if (reach < 16u * (uint32_t)kk) return false;
    }
    for (int g0 = 0; g0 < nq; g0 += U * NT) {
      if (g0) request(g0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int g = g0 + u * NT + t;
        const uint32_t keys[4] = {k4[u].x, k4[u].y, k4[u].z, k4[u].w};
        unsigned long long m[4];
        uint32_t cnt = 0, base = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          m[k] = __ballot(g < nq && keys[k] >= klo);
          cnt += (uint32_t)__popcll(m[k]);
        }
        if (lane == 0 && cnt) base = atomicAdd(&sm.n_list, cnt);
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        const int n0 = g / per * kListSeg;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], base));
          if (((m[k] >> lane) & 1ull) && pos < (uint32_t)Lds::kList) {
            sm.score[pos] = __float_as_uint(key_score(keys[k]));
            sm.tok[pos] = (typename Lds::Tok)min((uint32_t)n0 + (t4[u] >> (8 * k) & 255u), (uint32_t)N - 1u);
          }
          base += (uint32_t)__popcll(m[k]);
        }
      }
    }
    __syncthreads();
    const uint32_t M = sm.n_list;
    if (M >= (uint32_t)kk && M <= (uint32_t)Lds::kList) return true;
    __syncthreads();                                          // (all have read it)
    if (t == 0) sm.n_list = 0;
    return false;
  };
  uint4 w[kCalibPerThread / 4];
  if (!SHARED || !calib_top_listed(sm, sets, row, N, kk, tried)) calib_select<4, SHARED>(
      sm, N, kk,
      [&](int i, int c0) {
        const int n = c0 + (i * NT + t) * 4;
        w[i] = scores(n < N ? n : 0);
      },
      [&](int c0, int i, int tt, float (&x)[4], auto full) {
        const int n = c0 + (i * NT + tt) * 4;
        x[0] = full || n < N ? __uint_as_float(w[i].x) : NAN; x[1] = full || n + 1 < N ? __uint_as_float(w[i].y) : NAN;
        x[2] = full || n + 2 < N ? __uint_as_float(w[i].z) : NAN; x[3] = full || n + 3 < N ? __uint_as_float(w[i].w) : NAN;
      },
      []() {}, pick,
      [&](float& top) {
        if (t < SP) {
          const float x[4] = {__uint_as_float(spot.x), __uint_as_float(spot.y), __uint_as_float(spot.z), __uint_as_float(spot.w)};
#pragma unroll
          for (int k = 0; k < 4; ++k) sm.sample[k * SP + t] = n_spot + k < N ? x[k] : x[0];
        }
        __syncthreads();
        if (t < kWave) {
          float x[SMP / kWave], best = 0.f, cut = -INFINITY;
#pragma unroll
          for (int k = 0; k < SMP / kWave; ++k) x[k] = sm.sample[k * kWave + t];
          const float ps = (float)kk * ((float)SMP / (float)N);
          const int r = (int)(ps + 5.0f * sqrtf(ps) + 3.0f);  // (as calib_cut)
          if (r <= SMP) cut = list_cut(x, r, sm.bins, best);
          if (t == 0) sm.cut_top = make_float2(cut, best);
        }
        __syncthreads();
        top = sm.cut_top.y;
        return sm.cut_top.x;
      },
      [&](int n) { return SHARED ? ld_agent(s + n) : s[n]; },
      [&](uint32_t win, const auto& tok, bool taken, uint32_t taken_tok) { calib_bits(sm, win, tok, taken, taken_tok); });
  __syncthreads();
  for (int i = t; i < words; i += NT) st_agent(sets.full + (size_t)row * words + i, sm.bits[i] | kCalibThere);
  publish_barrier();
  if (t < F) sm.early[t] = atomicExch(&sets.state[row * F + t], 2u);
  __syncthreads();
  // four FCs at a time, those that have left their sets
  const unsigned long long left = __ballot(lane < F && sm.early[lane & (F - 1)] == 1u);
  static_assert(F == kWave, "a lane per FC");
  for (int n0 = 4 * wave, n = __popcll(left); n0 < n; n0 += 4 * NWV) {
    int f[4];
    unsigned long long m = left;
    for (int i = 0; i < n0; ++i) m &= m - 1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f[j] = m ? __ffsll((long long)m) - 1 : -1;
      m &= m - 1;
    }
    uint32_t sum[4] = {};
    for (int i = lane; i < words; i += kWave) {
      const uint32_t x = sm.bits[i];
#pragma unroll
      for (int j = 0; j < 4; ++j) sum[j] += (uint32_t)__popc(ld_agent(sets.fc + ((size_t)row * F + max(f[j], 0)) * words + i) & x);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t all = wave_prefix_sum(sum[j]);
      if (lane == kWave - 1 && f[j] >= 0) CA_sum[row * F + f[j]] += (float)all / (float)kk;
    }
  }
}

// A (row, FC), by a workgroup: CA_sum[row][i] += |top-K of FC i's scores & the full head's| / K.  Another workgroup finds the full head's set meanwhile, which an FC needs at
// its end only.  It looks for it for a bounded while; if it is not there even then the FC leaves its own set in memory, says so in its state word, and whoever of the
// two comes second to that word counts.
// us, in two launches, cuts made here and the FCs tested against the full head's set where it was there / cuts made in the launch before, with a look for a while: 8 rows of 32768,
// K = 2048: 39.9 / 34.9; of 16384, 1500: 29.2 / 24.8; of 12000, 7 heads: 28.6 / 23.9; 4 rows of 32000, 3500: 30.6 / 28.2; 2 of 20011, 700: 21.4 / 20.0; 8 of 8192, 512: 20.6 /
// 18.9; of 1015: 15.5 / 14.4.  In one launch there is none before that could make cuts at no cost: 8 rows of 32768 with a launch for them 32.0, made here 31.25.
// OWN_CUT: made here, from a sample that the first wave asks for ahead of all else; else it and the queries' sums come from the launch before.
template <bool OWN_CUT, int PAIR_SHIFT, int PAIR_ADD, typename ET, typename Lds>
__device__ __forceinline__ void calib_fc(Lds& sm, const ET* __restrict__ q, const ET* __restrict__ Kp, const CalibSets& sets, float* __restrict__ CA_sum,
                                         int row, int part, int G, int N, int n_cap, int kk) {
  constexpr int NT = Lds::kThreads, F = kHeadDim / 2, TPT = ScoreTraits<ET>::TPT;
  const int t = threadIdx.x, words = sets.words;
  const int id = row * F + part;
  if (t == 0) { sm.count = 0; sm.missing = 0; }
  const ET* p = Kp + (size_t)id * n_cap * 2;
  ET qa[kMaxGroup], qb[kMaxGroup];
  CalibSample<ET, Lds::kSpots> sample;
  float4 cq = make_float4(0.f, 0.f, 0.f, 0.f);
  if constexpr (OWN_CUT) {
    const ET* qh = q + (size_t)row * G * kHeadDim + (part << PAIR_SHIFT);
#pragma unroll
    for (int g = 0; g < kMaxGroup; ++g) {
      qa[g] = qh[(size_t)min(g, G - 1) * kHeadDim];
      qb[g] = qh[(size_t)min(g, G - 1) * kHeadDim + PAIR_ADD];
    }
    if (t < kWave) sample.request(p, N);
  } else {
    cq = sets.cuts[id];
  }
  float qlo = cq.z, qhi = cq.w;
  uint4 w[kCalibPerThread / TPT];
  auto load1 = [&](int i, int c0) {
    const int n = c0 + (i * NT + t) * TPT;
    w[i] = *reinterpret_cast<const uint4*>(p + (size_t)(n < N ? n : 0) * 2);
  };
  auto get = [&](int c0, int i, int tt, float (&x)[TPT], auto full) {
    const int n = c0 + (i * NT + tt) * TPT;
#pragma unroll
    for (int k = 0; k < TPT; ++k) x[k] = 0.f;
    fma_pairs<ET>(w[i], qlo, qhi, x);
#pragma unroll
    for (int k = 0; k < TPT; ++k) x[k] = full || n + k < N ? x[k] : NAN;
  };
  auto opaque = [&]() {
#pragma unroll
    for (int i = 0; i < kCalibPerThread / TPT; ++i) asm volatile("" : "+v"(w[i].x), "+v"(w[i].y), "+v"(w[i].z), "+v"(w[i].w));
  };
  auto score_at = [&](int n) {
    float lo, hi;
    if constexpr (sizeof(ET) == 2) {
      const uint32_t x = reinterpret_cast<const uint32_t*>(p)[n];
      lo = bf16_lo(x); hi = bf16_hi(x);
    } else {
      const float2 x = reinterpret_cast<const float2*>(p)[n];
      lo = x.x; hi = x.y;
    }
    return fmaf(qhi, hi, fmaf(qlo, lo, 0.f));
  };
  const uint32_t* full = sets.full + (size_t)row * words;
  // The other is as long in the making, and longer where a row's best lie together, so a wave looks for it for a while: what is left here for the workgroup that makes
  // it is counted by that alone.  us, 32 looks / 64: 8 rows of 32768 whose best lie together (rising; neighbours alike) 37.3 / 34.35, 36.3 / 34.75, of 12000 25.95 / 23.85, 25.5 /
  // 23.6; 128 looks as 64 (an autoregression of 0.98, six looks: 50).
  const auto look = [&]() {
    if (t < kWave) {
      int looks = kCalibLooks;
      while (ld_agent(full + words - 1) == 0u && looks-- > 0) __builtin_amdgcn_s_sleep(8);
    }
  };
  // What the threads hold of the FC's set, if they do (calib_held)
  uint32_t win = 0, tok[kCalibHeld], taken_tok = 0;
  bool holds = false, taken = false;
  calib_select<TPT, OWN_CUT>(sm, N, kk, load1, get, opaque, [](uint32_t&, uint32_t&) { return false; }, 
                   [&](float& top) {                          // (behind the requests for the first stretch)
                     if constexpr (!OWN_CUT) {
                       top = cq.y;
                       return cq.x;
                     }
#pragma unroll
                     for (int g = 0; g < kMaxGroup; ++g) {    // g ascending, as everywhere
                       float x, y;
                       if constexpr (sizeof(ET) == 2) { x = __uint_as_float((uint32_t)qa[g] << 16); y = __uint_as_float((uint32_t)qb[g] << 16); }
                       else { x = qa[g]; y = qb[g]; }
                       qlo += g < G ? x : 0.f;
                       qhi += g < G ? y : 0.f;
                     }
                     if (t < kWave) {
                       float cut, best;
                       sample.make_cut(qlo, qhi, N, kk, sm.bins, cut, best);
                       if (t == 0) sm.cut_top = make_float2(cut, best);
                     }
                     __syncthreads();
                     top = sm.cut_top.y;
                     return sm.cut_top.x;
                   }, score_at,
                   [&](uint32_t w, const auto& toks, bool cand, uint32_t cand_tok) {
                     holds = true;
                     win = w;
                     taken = cand;
                     taken_tok = cand_tok;
#pragma unroll
                     for (int k = 0; k < kCalibHeld; ++k) tok[k] = toks[k];
                   });
  look();                                                     // (the only time: what is not there by then is met through the state word)
  __syncthreads();                                            // (all have made their part of the set, or read the histogram, whose storage the sets have)
  uint32_t mine = 0, there = kCalibThere;
  const auto meet = [&]() {
    there = kCalibThere;
    mine = 0;
    for (int i = t; i < words; i += NT) {
      const uint32_t x = ld_agent(full + i);
      there &= x;
      mine += (uint32_t)__popc(x & sm.bits[i]);
    }
  };
  if (holds) {
    for (int i = t; i < words; i += NT) {
      const uint32_t x = ld_agent(full + i);
      there &= x;
      sm.bits[i] = x;
    }
  } else {
    meet();
  }
  if (there == 0) sm.missing = 1;
  __syncthreads();
  if (sm.missing) {
    if (holds) {
      calib_bits(sm, win, tok, taken, taken_tok);
      __syncthreads();
    }
    for (int i = t; i < words; i += NT) st_agent(sets.fc + (size_t)id * words + i, sm.bits[i]);
    publish_barrier();
    if (t == 0) sm.missing = atomicExch(&sets.state[id], 1u);
    __syncthreads();
    if (sm.missing != 2u) return;                             // (counted by whoever publishes the full head's)
    meet();
  } else if (holds) {
    const auto in = [&](uint32_t n) { return sm.bits[n / 31u] >> (n % 31u) & 1u; };
    mine = taken ? in(taken_tok) : 0u;
#pragma unroll
    for (int k = 0; k < kCalibHeld; ++k) mine += (win >> k & 1u) & in(win >> k & 1u ? tok[k] : 0u);
  }
  mine = wave_prefix_sum(mine);
  if (lane_id() == kWave - 1) atomicAdd(&sm.count, mine);
  __syncthreads();
  if (t == 0) CA_sum[id] += (float)sm.count / (float)kk;
}

template <typename ET, typename Lds, int WAVES>
__global__ __launch_bounds__(Lds::kThreads, WAVES) void calib_fc_kernel(const ET* __restrict__ Kp, const float* __restrict__ S, CalibSets sets,
                                                                       float* __restrict__ CA_sum, int rows, int N, int n_cap, int kk) {
  constexpr int F = kHeadDim / 2;
  __shared__ Lds sm;
  if ((int)blockIdx.x < rows) {
    calib_top<false>(sm, S, sets, CA_sum, (int)blockIdx.x, N, n_cap, kk);
    return;
  }
  const int id = (int)blockIdx.x - rows;
  calib_fc<false, 0, 0, ET>(sm, (const ET*)nullptr, Kp, sets, CA_sum, id / F, id % F, 1, N, n_cap, kk);
}

// All in one launch: the first rows * nslices workgroups score the full head, and the last of a row finds its set; one per (row, FC).  The keys are asked for twice at
// about the same time, by workgroups that share a compute unit, and a row's set is found under the FCs' streams.
using CalibRowLds = CalibLds<kSliceNT, kCalibWords1, 7680>;
template <int PAIR_SHIFT, int PAIR_ADD>
__global__ __launch_bounds__(kSliceNT, 6) void calib_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ Kp, float* __restrict__ S,
                                                            CalibSets sets, float* __restrict__ CA_sum, int rows, int nslices, uint32_t m_slices, int G,
                                                            int N, int n_cap, int kk) {
  constexpr int F = kHeadDim / 2;
  __shared__ union Lds {
    __device__ Lds() {}
    CalibRowLds row;
    CalibSlice slice;
  } sm;
  __shared__ uint32_t ticket;
  const int n_full = rows * nslices;
  int row, part;
  if ((int)blockIdx.x < n_full) {
    row_slice_of_block(rows, nslices, m_slices, row, part);
    calib_slice<PAIR_SHIFT, PAIR_ADD>(sm.slice, q, Kp, S, sets, row, part, G, N, n_cap);
    publish_barrier();
    if (threadIdx.x == 0) ticket = atomicAdd(&sets.tickets[row], 1u);
    __syncthreads();
    if (ticket == (uint32_t)nslices - 1u) calib_top<true>(sm.row, S, sets, CA_sum, row, N, n_cap, kk);
    return;
  }
  constexpr uint32_t m_fcs = div_magic(F, 65535 * F);
  row_slice_of_block(rows, F, m_fcs, row, part, blockIdx.x - (unsigned)n_full);
  calib_fc<true, PAIR_SHIFT, PAIR_ADD, uint16_t>(sm.row, q, Kp, sets, CA_sum, row, part, G, N, n_cap, kk);
}

// K >= N: both sets are all tokens
__global__ __launch_bounds__(256) void calib_all_kernel(float* __restrict__ CA_sum, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) CA_sum[i] += 1.0f;
}

// One launch for all (behind one that clears) where that is the faster: bf16, 8 rows or more, of 8193 .. 32768 tokens.  us, two launches / so, independent scores; rising; neighbours alike;
// thousands of ties: 8 rows of 32768, K = 2048: 36.85 / 31.45; 37.0 / 34.5; 36.9 / 34.7; 72.4 / 69.1; of 16384, 1500: 24.35 / 21.75; 24.4 / 24.6; 24.4 / 24.35; 42.3 / 43.3; of 12000, 1000: 23.2 /
// 21.4; 23.2 / 24.2; 23.25 / 23.7; 34.25 / 36.8; 32 of 16384, 1024: 67.7 / 65.2; 67.4 / 67.2; 67.8 / 67.1; 109.6 / 122.8.  On the other side fewer rows, which have workgroups of 1024: 4 of
// 32000, 3500: 29.2 / 26.1; 29.5 / 31.85; 30.3 / 32.3; 68.4 / 73.6; 4 of 20000, 1500: 24.95 / 19.6; 24.85 / 26.0; 25.25 / 25.9; 36.1 / 34.4; 2 of 20011, 700: 20.2 / 18.1; 20.0 / 23.9; 20.1 / 23.95;
// 27.2 / 25.45; 7 of 32768, 2048: 33.55 / 34.2; 33.75 / 36.9; 34.05 / 37.3; 61.8 / 71.9; and shorter ones: 8 of 8192, 512: 18.95 / 18.3; 18.9 / 21.3; 19.1 / 21.25; 37.85 / 27.8; of 5000: 18.05 / 17.15;
// 18.0 / 20.45; of 1015: 14.5 / 17.25; 14.5 / 19.7; 4 of 3000: 15.5 / 17.2; 15.4 / 19.7.  Measured before FCs waited as long: 8 of 131072: 124 / 131; float32, 8 of 20000: 41.1 / 43.7, of 6000: 19.6 / 17.4.
static bool calib_one_launch(const fasa_shape& s) {
  return s.dtype == FASA_BF16 && s.n_ctx > kCalibShort && s.n_ctx <= 32768 && s.batch * s.n_kv_heads >= 8;
}

template <typename ET, int PS, int PA>
static hipError_t launch_calib_p(const fasa_shape& s, const void* q, const void* Kp_all, int kk, float* S, const CalibSets& sets,
                                 float* CA_sum, hipStream_t st) {
  const int rows = s.batch * s.n_kv_heads, half = s.head_dim / 2;
  if constexpr (sizeof(ET) == 2) {
    if (calib_one_launch(s)) {
      const hipError_t e = launch("fasa_calib_clear", calib_clear_kernel, dim3(rows), dim3(256), st, sets);
      if (e != hipSuccess) return e;
      const int nslices = (s.n_ctx + kSliceTokens - 1) / kSliceTokens;
      // (the profiler has one name for the launch that counts the FCs, and the full head's work in it is the FCs' there)
      return launch("fasa_calib_fc", calib_kernel<PS, PA>, dim3(rows * (nslices + half)), dim3(kSliceNT), st, (const ET*)q, (const ET*)Kp_all, S, sets, CA_sum, rows, nslices, div_magic(nslices, (long long)rows * nslices), s.n_q_heads / s.n_kv_heads, s.n_ctx,
                    s.n_cap, kk);
    }
  }
  const int per = 256 * ScoreTraits<ET>::TPT, nslices = (s.n_ctx + per - 1) / per;
  hipError_t e = launch("fasa_calib_full", calib_full_kernel<ET, PS, PA>, dim3(rows * (half / 4 + nslices)), dim3(256), st, (const ET*)q,
                        (const ET*)Kp_all, S, sets, rows, nslices, div_magic(nslices, (long long)rows * nslices),
                        s.n_q_heads / s.n_kv_heads, s.n_ctx, s.n_cap, kk);
  if (e != hipSuccess) return e;
  const auto stage = [&](auto kernel, int nt) {
    return launch("fasa_calib_fc", kernel, dim3(rows * (1 + half)), dim3(nt), st, (const ET*)Kp_all, S, sets, CA_sum, rows, s.n_ctx, s.n_cap, kk);
  };
  // Rows that fit in the registers of 256 threads twice over: several workgroups per compute unit.  Longer ones: two of 1024 share a compute unit, and three of
  // 512 do where two don't hold the FCs' and the full head's workgroups at once, which fewer than 8 rows' are.  float32, us,
  // 1024 / 512: 8 rows of 9000 31.9 / 26.4, of 20000 51.0 / 41.1, of 32768, K = 2048, 63.6 / 59.8; 16 of 12000 60.7 / 48.9.
  if (s.n_ctx <= kCalibShort) return stage(calib_fc_kernel<ET, CalibLds<256, kCalibWords0, 4096>, 4>, 256);
  if (s.n_ctx > 32768) return stage(calib_fc_kernel<ET, CalibLds<1024, (kCalibMaxCtx + 30) / 31, 13312>, 4>, 1024);
  if constexpr (sizeof(ET) == 2) return stage(calib_fc_kernel<ET, CalibLds<1024, kCalibWords1, 8192>, 8>, 1024);
  else if (rows * (1 + half) <= 2 * kAssumedCUs) return stage(calib_fc_kernel<ET, CalibLds<1024, kCalibWords1, 8192>, 4>, 1024);
  else return stage(calib_fc_kernel<ET, CalibLds<512, kCalibWords1, 7680>, 4>, 512);
}

// Cuts, lists (5 bytes a place), what describes their segments, states, tickets, sets.
static size_t calib_list_segs(int n) { return ((size_t)n + kListSeg - 1) / kListSeg; }
size_t calib_scratch_bytes(int rows, int n_cap) {
  const size_t half = kHeadDim / 2, lists = calib_list_segs(n_cap) * (kListSeg * 5 + sizeof(uint2)) + 16;
  return rows * (half * (sizeof(float4) + sizeof(uint32_t)) + sizeof(uint32_t) + lists + (1 + half) * (((size_t)n_cap + 30) / 31) * sizeof(uint32_t));
}

hipError_t launch_calib(const fasa_shape& s, const void* q, const void* Kp_all, int kk, float* S, void* scratch, float* CA_sum,
                        hipStream_t st) {
  const size_t rows = (size_t)s.batch * s.n_kv_heads;
  CalibSets sets;
  sets.words = (s.n_ctx + 30) / 31;
  sets.nsegs = (int)calib_list_segs(s.n_ctx);
  sets.pitch = s.dtype == FASA_BF16 ? list_room(kk, s.n_ctx) : 0;
  // None for half of a row, nor in two launches up to 32768 tokens: so few rows all have their places at once, the full head's set is found while the FCs stream, and
  // lists that turn out to be of no use hold it up.  us, lists / none, independent scores; rising; neighbours alike: 1 row of 9000, K = 300: 16.6 / 16.6; 20.2 / 16.5; 20.2 / 16.6; 2 of 20011,
  // 700: 19.95 / 20.05; 23.3 / 20.0; 23.3 / 20.05; 4 of 12000, 1000: 20.9 / 19.9; 22.4 / 20.0; 22.6 / 20.0; of 32000, 3500: 28.9 / 28.95; 31.3 / 29.25; 32.25 / 30.3; 7 of 32768, 2048:
  // 34.2 / 33.3; 35.0 / 33.2; 35.2 / 33.55.  Longer rows, whose FCs wait for a place: beside calib_top's use of them.
  if (sets.pitch > kListSeg / 2 || !(calib_one_launch(s) || s.n_ctx > 32768)) sets.pitch = 0;
  sets.cuts = (float4*)scratch;
  sets.lists = (uint32_t*)(sets.cuts + rows * (kHeadDim / 2));
  sets.lims = (uint2*)(sets.lists + rows * sets.list_words());
  sets.state = (uint32_t*)(sets.lims + rows * sets.nsegs);
  sets.tickets = sets.state + rows * (kHeadDim / 2);
  sets.full = sets.tickets + rows;
  sets.fc = sets.full + rows * sets.words;
  constexpr int D = kHeadDim;
  if (kk >= s.n_ctx) {
    const int n = s.batch * s.n_kv_heads * (D / 2);
    return launch("fasa_calib_all", calib_all_kernel, dim3((n + 255) / 256), dim3(256), st, CA_sum, n);
  }
  const bool inter = s.pairing == FASA_PAIR_INTERLEAVED;   // FC i: dims (2i, 2i + 1), else (i, i + d/2)
  if (s.dtype == FASA_BF16)
    return inter ? launch_calib_p<uint16_t, 1, 1>(s, q, Kp_all, kk, S, sets, CA_sum, st)
                 : launch_calib_p<uint16_t, 0, D / 2>(s, q, Kp_all, kk, S, sets, CA_sum, st);
  return inter ? launch_calib_p<float, 1, 1>(s, q, Kp_all, kk, S, sets, CA_sum, st)
               : launch_calib_p<float, 0, D / 2>(s, q, Kp_all, kk, S, sets, CA_sum, st);
}

int calib_max_ctx() { return kCalibMaxCtx; }

}  // namespace fasa
