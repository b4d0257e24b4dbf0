// Offline calibration (paper Sec. 3.3 eq. ca_k and Alg. 1): contextual agreement of every single
// frequency chunk with the full head, for one query.  Kp_all holds all d/2 FCs, FC-major.  Two launches:
//
//   calib_full_kernel   full-head scores alpha (all planes, fp32 chain in FC order);
//   calib_fc_kernel     one workgroup per (b, h): the top-K set of alpha; one per (b, h, FC): the scores of the one FC, their top-K
//                       set, and how many of it are in that of alpha.
//
// The single-FC scores never exist in memory: a workgroup streams its plane once and writes one number.
// One Llama-3-8B layer at 32768 tokens, K = 2048 (67 MB of keys): 13.6 + 26.1 us.  (The full head's set by a launch in between, one
// workgroup a row: 13.6 + 11.3 + 21.7, several: 13.6 + 8.9 + 21.7.  Scoring all FCs to memory, 67 MB of scores, selecting them
// with the decode step's kernels and intersecting index lists: 135.)
#include <type_traits>

#include "fasa_device.h"
#include "fasa_internal.h"
#include "row_list.h"
#include "score_common.h"
#include "select_common.h"

namespace fasa {

constexpr int kCalibMaxCtx = 262144;   // a row's set of an FC lives in LDS (33 KB)
constexpr int kCalibPerThread = 16;    // scores in flight per thread
constexpr int kCalibWords0 = (8192 + 30) / 31, kCalibWords1 = (32768 + 30) / 31;   // of a set (CalibSets)

// The top-K sets.  A word has 31 tokens, and its top bit says that it is there: the full head's set is read with no other sign.
struct CalibSets {
  uint32_t* full;      // [row][words]: of the full head
  uint32_t* fc;        // [row][FC][words]: of an FC whose workgroup did not find the full head's
  uint32_t* state;     // [row][FC]: 0; 1: the FC's set is in fc; 2: the full head's is in full
  int words;           // ceil(N / 31)
  template <int NT>
  __device__ __forceinline__ void clear(int row) const {
    for (int i = threadIdx.x; i < words; i += NT) full[(size_t)row * words + i] = 0;
    if (threadIdx.x < kHeadDim / 2) state[row * (kHeadDim / 2) + threadIdx.x] = 0;
  }
};
constexpr uint32_t kCalibThere = 0x80000000u;
__device__ __forceinline__ void set_bit(uint32_t* bits, uint32_t tok) { atomicOr(&bits[tok / 31u], 1u << (tok % 31u)); }

// Full-head scores of a slice of 256 * TPT tokens: 1-D grid of rows * nslices workgroups.
template <typename ET, int PAIR_SHIFT, int PAIR_ADD>
__global__ __launch_bounds__(256, 4) void calib_full_kernel(const ET* __restrict__ q, const ET* __restrict__ Kp,
                                                         float* __restrict__ S, CalibSets sets, int rows, int nslices,
                                                         uint32_t m_slices, int G, int N, int n_cap) {
  constexpr int D = kHeadDim, F = D / 2, NW = 16;
  constexpr int TPT = ScoreTraits<ET>::TPT;
  __shared__ float ql[kMaxGroup][D];
  __shared__ float2 qs[F];
  int row, slice;
  row_slice_of_block(rows, nslices, m_slices, row, slice);
  const int t = threadIdx.x;
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
}

template <int NT, int WORDS>
struct CalibLds {
  static constexpr int kThreads = NT;
  // (two workgroups of 1024 share a compute unit's LDS, or one has it)
  static constexpr int kList = NT != 1024 ? 4096 : WORDS <= kCalibWords1 ? 8192 : 13312;   // (8 rows of 131072, K = 4096: 212 -> 137 us)
  uint2 list[kList];                                          // scores at or above the cut: (score bits, token)
  uint32_t hist[kSelBins];
  // Places of the row that are sampled, the TPT consecutive tokens of one load each.  With 256 single tokens, ranked by counting,
  // the list of K = 4096 of 32768 was 7000 entries long and one FC in twenty overflowed: 54.6 us, like this 45.6 (K = 2048: 42.9 / 42.7;
  // 8 rows of 8192, 512, 128 single tokens: 22.2 / 20.8).
  static constexpr int kSpots = NT == 1024 ? 256 : 64;
  union {                                                     // (the sample is spent before there are candidates)
    uint2 cand[kSelCand];
    struct { __align__(16) float sample[4 * kSpots]; __align__(16) uint32_t bins[256]; };
  };
  float2 cut_top;
  uint32_t wtot[NT / kWave];
  uint32_t thr[4];
  uint32_t n_list, n_cnd, count, missing;
  uint32_t early[kHeadDim / 2];
};

// Top-K of a row by one workgroup of NT threads, which hold a stretch of it as loaded: load1(i, c0) requests piece i of what the
// scores of tokens c0 .. c0 + NT * kCalibPerThread - 1 are made of (kCalibPerThread / TPT pieces a thread),
// get(c0, i, t, x, full) makes those of tokens c0 + (i * NT + t) * TPT + k, a NaN beyond the row unless it is said to
// be full (cheap: made again in every pass, which keeps 16 registers free and two workgroups of 1024 on a
// compute unit); opaque() hides the pieces from the compiler, which would otherwise keep the scores.
// sample(n) requests the TPT tokens from n on, scores_of() makes their scores.  score_at(n): one token's score.  take_one(n): token n is in the set; early() and ready() run before it, with a barrier of the
// workgroup between them.
// What reaches the cut is gathered into a list in LDS first (some 7 instructions a score per wave, where counting
// and classifying all scores under a test takes 30); a list that comes out short of K or beyond its
// room is not used.  Infinite scores rank like any others; where NaNs rank is unspecified, but the set has K tokens.
template <int NT, int WORDS, int TPT, typename Load1, typename Get, typename Opaque, typename Sample, typename ScoresOf, typename ScoreAt,
          typename Early, typename Ready, typename TakeOne>
__device__ __forceinline__ void calib_select(CalibLds<NT, WORDS>& sm, int N, int kk, Load1&& load1, Get&& get,
                                             Opaque&& opaque, Sample&& sample, ScoresOf&& scores_of, ScoreAt&& score_at,
                                             Early&& early, Ready&& ready, TakeOne&& take_one) {
  const int t = threadIdx.x;
  constexpr int R = NT * kCalibPerThread, NP = kCalibPerThread / TPT;
  auto load = [&](int c0) {
#pragma unroll
    for (int i = 0; i < NP; ++i) load1(i, c0);
  };
  const bool resident = N <= R;
  constexpr int SP = CalibLds<NT, WORDS>::kSpots, SMP = SP * TPT;
  float sx[TPT];
  const int n_spot = (int)(((long long)(t & (SP - 1)) * N) / SP) & ~(TPT - 1);
  auto spot = sample(n_spot);                                 // (requested ahead of the stretch)
  load(0);
  if (t == 0) { sm.n_list = 0; sm.n_cnd = 0; sm.thr[2] = 0; }
  for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;
  scores_of(spot, sx);
  if (t < SP) {
#pragma unroll
    for (int k = 0; k < TPT; ++k) sm.sample[k * SP + t] = n_spot + k < N ? sx[k] : sx[0];
  }
  __syncthreads();
  if (t < kWave) {
    float x[SMP / kWave], top = 0.f, cut = -INFINITY;
#pragma unroll
    for (int k = 0; k < SMP / kWave; ++k) x[k] = sm.sample[k * kWave + t];
    // neighbours may be alike: a wider margin than independent ones would need
    const float ps = (float)kk * ((float)SMP / (float)N);
    const int r = (int)(ps + 5.0f * sqrtf(ps) + 3.0f);
    if (r <= SMP) cut = list_cut(x, r, sm.bins, top);
    if (t == 0) sm.cut_top = make_float2(cut, top);
  }
  __syncthreads();
  const float flo = sm.cut_top.x;
  early();
  uint32_t klo = 0, khi = 0xffffffffu;
  int shift = 22, need = kk, n_cand;
  if (flo > -INFINITY) {
    klo = score_key(flo);
    shift = first_shift(klo, score_key(sm.cut_top.y));
  }
  {
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
          if (x[k] >= flo && pos < (uint32_t)CalibLds<NT, WORDS>::kList)
            sm.list[pos] = make_uint2(__float_as_uint(x[k]), (uint32_t)(c0 + (i * NT + tt) * TPT + k));
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
  const bool listed = M >= kk && M <= CalibLds<NT, WORDS>::kList;
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
  for (;;) {
    const bool whole = klo == 0 && khi == 0xffffffffu;
    auto count = [&](uint32_t key) {
      if (key >= klo && key <= khi) atomicAdd(&sm.hist[min((key - klo) >> shift, (uint32_t)kSelBins - 1u)], 1u);
    };
    if (listed) {
      for (int i = t; i < M; i += NT) count(score_key(__uint_as_float(sm.list[i].x)));
    } else for (int c0 = 0; c0 < N; c0 += R) {
      if (!resident) load(c0);
      opaque();
      for_scores(c0, [&](uint32_t key, int) { count(key); });
    }
    if (find_threshold(sm, klo, khi, shift, need, n_cand)) break;
    if (t == 0) sm.thr[2] = 0;                                     // (all have read it)
    if (n_cand == 0) {
      if (whole) return;                                           // (fewer than K scores: the callers pass K < N)
      klo = 0; khi = 0xffffffffu; shift = 22;                      // the sample misled: the whole range
    }
  }
  ready();
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
      const uint2 e = sm.list[i];
      place(score_key(__uint_as_float(e.x)), (int)e.y);
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
    int tied = 0;
    for (int i0 = 0; i0 < N && tied < need; i0 += NT) {
      const int n = i0 + t;
      const bool tie = n < N && score_key(score_at(min(n, N - 1))) == klo;
      uint32_t tot;
      const uint32_t before = block_prefix_sum<NT>(tie ? 1u : 0u, sm.wtot, tot);
      if (tie && tied + (int)before < need) take_one(n);
      tied += (int)tot;
    }
  }
}

// The full head's top-K set, by one workgroup of calib_fc_kernel's launch per row, which then counts for the FCs that came first (a
// wave each).
template <int NT, int WORDS>
__device__ __forceinline__ void calib_top(CalibLds<NT, WORDS>& sm, uint32_t* bits, const float* __restrict__ S, const CalibSets& sets,
                                          float* CA_sum, int row, int N, int n_cap, int kk) {
  constexpr int F = kHeadDim / 2;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, words = sets.words;
  const float* s = S + (size_t)row * n_cap;
  __builtin_amdgcn_s_setprio(3);                              // (64 workgroups may end up waiting to be counted)
  for (int i = t; i < words; i += NT) bits[i] = 0;
  float4 w[kCalibPerThread / 4];
  calib_select<NT, WORDS, 4>(
      sm, N, kk,
      [&](int i, int c0) {
        const int n = c0 + (i * NT + t) * 4;
        w[i] = *reinterpret_cast<const float4*>(s + (n < N ? n : 0));
      },
      [&](int c0, int i, int tt, float (&x)[4], auto full) {
        const int n = c0 + (i * NT + tt) * 4;
        x[0] = full || n < N ? w[i].x : NAN; x[1] = full || n + 1 < N ? w[i].y : NAN;
        x[2] = full || n + 2 < N ? w[i].z : NAN; x[3] = full || n + 3 < N ? w[i].w : NAN;
      },
      []() {}, [&](int n) { return *reinterpret_cast<const float4*>(s + n); },
      [](const float4& v, float (&x)[4]) { x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w; }, [&](int n) { return s[n]; }, []() {},
      []() {}, [&](int n) { set_bit(bits, (uint32_t)n); });
  __syncthreads();
  for (int i = t; i < words; i += NT) st_agent(sets.full + (size_t)row * words + i, bits[i] | kCalibThere);
  publish_barrier();
  if (t < F) sm.early[t] = atomicExch(&sets.state[row * F + t], 2u);
  __syncthreads();
  for (int f = wave; f < F; f += NT / kWave) {
    if (sm.early[f] != 1u) continue;
    const uint32_t* p = sets.fc + ((size_t)row * F + f) * words;
    uint32_t sum = 0;
#pragma unroll 8
    for (int i = lane; i < words; i += kWave) sum += (uint32_t)__popc(ld_agent(p + i) & bits[i]);
    sum = wave_prefix_sum(sum);
    if (lane == kWave - 1) CA_sum[row * F + f] += (float)sum / (float)kk;
  }
}

// One workgroup per (row, FC): CA_sum[row][i] += |top-K of FC i's scores & the full head's| / K.  The first `rows` workgroups find
// the full head's set meanwhile, which an FC needs at its end only.  Nobody waits: an FC that finds the set there when it starts
// (a later round of workgroups) tests its tokens against it; one that does not makes its own set and compares the two at
// its end; if the other is not there even then it leaves its own in memory, says so in its state word, and whoever of the
// two comes second to that word counts.
// us, with launches for the full head's set (the better of one or several workgroups a row) / like this: 8 rows of 32768, K = 2048:
// 46.8 / 42.8, of 8192, 512: 26.9 / 21.6; 64 rows of 4096: 54.0 / 50.7; 1 row of 20000: 28.5 / 21.8; 2 of 100000: 108 / 77.  With
// several workgroups a row here: 8 rows of 32768: 46.3, of 8192: 21.0 - they take the places of FCs where the chip is full.
template <typename ET, int NT, int WORDS, int PAIR_SHIFT, int PAIR_ADD>
__global__ __launch_bounds__(NT, sizeof(ET) == 2 && NT == 1024 && WORDS == kCalibWords1 ? 8 : 4) void calib_fc_kernel(
    const ET* __restrict__ q, const ET* __restrict__ Kp, const float* __restrict__ S, CalibSets sets, float* __restrict__ CA_sum,
    int rows, int G, int N, int n_cap, int kk) {
  constexpr int D = kHeadDim, F = D / 2, WPT = (WORDS + NT - 1) / NT;
  constexpr int TPT = ScoreTraits<ET>::TPT;
  __shared__ CalibLds<NT, WORDS> sm;
  __shared__ uint32_t bits[WORDS];
  if ((int)blockIdx.x < rows) {
    calib_top<NT, WORDS>(sm, bits, S, sets, CA_sum, (int)blockIdx.x, N, n_cap, kk);
    return;
  }
  const int id = (int)blockIdx.x - rows, words = sets.words;
  const int row = id / F, f = id % F, t = threadIdx.x;
  if (t == 0) { sm.count = 0; sm.missing = 0; }
  const ET* qh = q + (size_t)row * G * D + (f << PAIR_SHIFT);
  float qlo = 0.f, qhi = 0.f;
  {
    ET a[kMaxGroup], b[kMaxGroup];
#pragma unroll
    for (int g = 0; g < kMaxGroup; ++g) {
      a[g] = qh[(size_t)min(g, G - 1) * D];
      b[g] = qh[(size_t)min(g, G - 1) * D + PAIR_ADD];
    }
#pragma unroll
    for (int g = 0; g < kMaxGroup; ++g) {
      float x, y;
      if constexpr (sizeof(ET) == 2) { x = __uint_as_float((uint32_t)a[g] << 16); y = __uint_as_float((uint32_t)b[g] << 16); }
      else { x = a[g]; y = b[g]; }
      qlo += g < G ? x : 0.f;
      qhi += g < G ? y : 0.f;
    }
  }
  const ET* p = Kp + (size_t)id * n_cap * 2;
  const uint32_t* full = sets.full + (size_t)row * words;
  uint32_t there = kCalibThere;
#pragma unroll
  for (int j = 0; j < WPT; ++j) {
    const int i = min(j * NT + t, words - 1);
    const uint32_t x = ld_agent(full + i);
    bits[i] = x;
    there &= x;
  }
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
  uint32_t mine = 0;
  bool have = true;
  calib_select<NT, WORDS, TPT>(
      sm, N, kk, load1, get, opaque, [&](int n) { return *reinterpret_cast<const uint4*>(p + (size_t)n * 2); },
      [&](const uint4& v, float (&x)[TPT]) {
#pragma unroll
        for (int k = 0; k < TPT; ++k) x[k] = 0.f;
        fma_pairs<ET>(v, qlo, qhi, x);
      },
      score_at, [&]() { if (there == 0) sm.missing = 1; },
      [&]() {
        have = sm.missing == 0;
        if (have) return;
        for (int i = t; i < words; i += NT) bits[i] = 0;
        __syncthreads();
      },
      [&](int n) {
        if (have) mine += (bits[(uint32_t)n / 31u] >> ((uint32_t)n % 31u)) & 1u;
        else set_bit(bits, (uint32_t)n);
      });
  if (!have) {
    auto meet = [&]() {
      there = kCalibThere;
      mine = 0;
      for (int i = t; i < words; i += NT) {
        const uint32_t x = ld_agent(full + i);
        there &= x;
        mine += (uint32_t)__popc(x & bits[i]);
      }
    };
    if (t == 0) sm.missing = 0;
    __syncthreads();
    meet();
    if (there == 0) sm.missing = 1;
    __syncthreads();
    if (sm.missing) {
      for (int i = t; i < words; i += NT) st_agent(sets.fc + (size_t)id * words + i, bits[i]);
      publish_barrier();
      if (t == 0) sm.missing = atomicExch(&sets.state[id], 1u);
      __syncthreads();
      if (sm.missing != 2u) return;                           // (counted by whoever publishes the full head's)
      meet();
    }
  }
  mine = wave_prefix_sum(mine);
  if (lane_id() == kWave - 1) atomicAdd(&sm.count, mine);
  __syncthreads();
  if (t == 0) CA_sum[id] += (float)sm.count / (float)kk;
}

// K >= N: both sets are all tokens
__global__ __launch_bounds__(256) void calib_all_kernel(float* __restrict__ CA_sum, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) CA_sum[i] += 1.0f;
}

template <typename ET, int PS, int PA>
static hipError_t launch_calib_p(const fasa_shape& s, const void* q, const void* Kp_all, int kk, float* S, const CalibSets& sets,
                                 float* CA_sum, hipStream_t st) {
  const int rows = s.batch * s.n_kv_heads, half = s.head_dim / 2;
  const int per = 256 * ScoreTraits<ET>::TPT, nslices = (s.n_ctx + per - 1) / per;
  hipError_t e = launch("fasa_calib_full", calib_full_kernel<ET, PS, PA>, dim3(rows * nslices), dim3(256), st, (const ET*)q,
                        (const ET*)Kp_all, S, sets, rows, nslices, div_magic(nslices, (long long)rows * nslices),
                        s.n_q_heads / s.n_kv_heads, s.n_ctx, s.n_cap);
  if (e != hipSuccess) return e;
  const auto stage = [&](auto nt_c, auto words_c) {
    constexpr int NT = decltype(nt_c)::value, WORDS = decltype(words_c)::value;
    return launch("fasa_calib_fc", calib_fc_kernel<ET, NT, WORDS, PS, PA>, dim3(rows * (1 + half)), dim3(NT), st, (const ET*)q,
                  (const ET*)Kp_all, S, sets, CA_sum, rows, s.n_q_heads / s.n_kv_heads, s.n_ctx, s.n_cap, kk);
  };
  // rows that fit in the registers of 256 threads: several workgroups per compute unit instead of one of
  // 1024 each; rows that fit in those of 1024: a set small enough for two
  if (s.n_ctx <= 8192) return stage(std::integral_constant<int, 256>{}, std::integral_constant<int, kCalibWords0>{});
  if (s.n_ctx <= 32768) return stage(std::integral_constant<int, 1024>{}, std::integral_constant<int, kCalibWords1>{});
  return stage(std::integral_constant<int, 1024>{}, std::integral_constant<int, (kCalibMaxCtx + 30) / 31>{});
}

size_t calib_scratch_bytes(int rows, int n_cap) {
  return (size_t)rows * (kHeadDim / 2 + (1 + kHeadDim / 2) * (((size_t)n_cap + 30) / 31)) * sizeof(uint32_t);
}

hipError_t launch_calib(const fasa_shape& s, const void* q, const void* Kp_all, int kk, float* S, void* scratch, float* CA_sum,
                        hipStream_t st) {
  const size_t rows = (size_t)s.batch * s.n_kv_heads;
  CalibSets sets;
  sets.words = (s.n_ctx + 30) / 31;
  sets.state = (uint32_t*)scratch;
  sets.full = sets.state + rows * (kHeadDim / 2);
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
