// Lists of the scores of a row that can be among its B best (paper Sec. 4.1, TopK-I), made by the workgroups that
// score it: what TopK-I has to look at shrinks from N scores to a few times B (list_rank) before the row is selected.
//
//   cut      every workgroup of a row scores the same sample of the row's tokens and takes a score of it that a few
//            more than B of the row's scores should reach (list_cut).  All arrive at the same bits.
//   list     a workgroup writes the scores of its segment of the row that reach the cut, as (key, token), to the
//            segment's own stretch of the row's list, and their number (list_count, list_write): no position is shared, so there is no
//            atomic, and a stretch has room for the whole segment.
//   select   list_load, select_listed: whoever selects holds the entries in registers, as many of each segment as are likely;
//            what a segment has beyond, where a row's best lie together, goes through LDS.  A list shorter than B,
//            because the sample misled, or far too long is not used: row_select.
// What the scores look like costs time, never exactness.
#pragma once

#include "attend_common.h"
#include "score_common.h"
#include "select_common.h"

namespace fasa {

constexpr int kListMaxSegs = 512;       // segments of a row
constexpr int kListScoreNT = 256;       // scoring threads of a workgroup that makes lists
constexpr int kListMinCtx = 1024;       // shorter rows are listed whole: the sample's clusters would meet
constexpr int kListCntPitch = (int)(kFuseRecBytesPerRow / sizeof(uint32_t));
static_assert(kListCntPitch >= kListMaxSegs, "a row's counts lie where the split form has its records");

// The sample: kWave * TPT tokens, in clusters of consecutive ones (64 bytes of a plane) that are evenly spaced over the row.
// First token of lane i's TPT; n: tokens of the row that lie in the planes.  In range of the row's capacity for any n, and of
// the row itself for n >= kListMinCtx - 1.
template <typename ET>
__device__ __forceinline__ int list_sample_token(int i, int n) {
  constexpr int TPT = ScoreTraits<ET>::TPT, CL = 32 / (int)sizeof(ET), NC = kWave * TPT / CL;
  const int c = i * TPT / CL;
  return ((n * (2 * c + 1) / (2 * NC)) & ~(CL - 1)) + (i * TPT & (CL - 1));
}

// Which of m sample scores the cut is: four standard deviations (and three) above the B m / N of them that are expected
// among the B best, half a deviation more than sample_rank(): a list that comes out short costs three passes over all
// scores of the row, in every one of its workgroups.  alike: by how much a cluster's scores being alike widens the variance
// (ListCut).  A list is N r / m long: of 256 scores, independent ones, 1.7 B for 6219 of 32905 tokens, 2.2 B for 2048 of 32768, 3.8 B
// for 256 of 16384, 5 B for 1024 of 131072, 8.5 B for 64 of 20011.
__host__ __device__ __forceinline__ int list_rank(int bsel, int n, int m, float alike = 1.0f) {
  const float ps = (float)bsel * ((float)m / (float)n);
  return (int)(ps + 4.0f * sqrtf(ps * alike) + 3.0f);
}

// The cut: a score that at least r (1 .. 64 KPL) of the sample's scores reach and hardly more, in steps of a 256th of
// the spread of the finite ones, by one wave whose lanes hold KPL of them each: a histogram in `bins` (256 words of LDS)
// and one suffix sum (what it takes is its latency: four rounds of ballots, two bits each, take twice as long).  No
// more than r finite scores, or hardly: no cut (-inf).
struct SampleBins {
  float lo, hi, spread;    // of the sample's finite scores
};
__device__ __forceinline__ float cut_of_bins(const SampleBins& sb, int r, const uint32_t* bins) {
  const int lane = lane_id();
  const uint4 c = *reinterpret_cast<const uint4*>(bins + 4 * lane);
  const uint32_t s2 = c.w + c.z, s1 = s2 + c.y, s0 = s1 + c.x;
  const uint32_t above = wave_suffix_sum(s0) - s0;             // in higher lanes' bins
  const uint32_t need = (uint32_t)r;
  const int j = above + c.w >= need ? 3 : above + s2 >= need ? 2 : above + s1 >= need ? 1 : 0;
  const unsigned long long m = __ballot(above + s0 >= need);   // a run of low lanes
  const int last = m ? 63 - __clzll((long long)m) : 0;
  const int bin = 4 * last + __builtin_amdgcn_readlane(j, last);
  return bin > 0 && sb.spread < INFINITY ? fmaf((float)bin, sb.spread * (1.0f / 256.0f), sb.lo) : -INFINITY;
}
template <int KPL>
__device__ __forceinline__ SampleBins sample_bins(const float (&x)[KPL], uint32_t* bins) {
  const int lane = lane_id();
  *reinterpret_cast<uint4*>(bins + 4 * lane) = make_uint4(0, 0, 0, 0);
  float hi = -INFINITY, lo = INFINITY;
#pragma unroll
  for (int k = 0; k < KPL; ++k) {
    const bool finite = fabsf(x[k]) < INFINITY;
    hi = finite ? fmaxf(hi, x[k]) : hi;
    lo = finite ? fminf(lo, x[k]) : lo;
  }
  hi = wave_max(hi);
  lo = -wave_max(-lo);
  const float spread = hi - lo, inv = 256.0f * __builtin_amdgcn_rcpf(spread);
  // same wave writes and reads: its LDS operations complete in order; the fences only keep the compiler from moving them
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int k = 0; k < KPL; ++k)    // (infinite scores: the bins at the ends; NaNs: the lowest)
    atomicAdd(&bins[(uint32_t)fminf(fmaxf((x[k] - lo) * inv, 0.0f), 255.0f)], 1u);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  return {lo, hi, spread};
}
// `top`: the sample's largest finite score.
template <int KPL>
__device__ __forceinline__ float list_cut(const float (&x)[KPL], int r, uint32_t* bins, float& top) {
  const SampleBins sb = sample_bins(x, bins);
  top = sb.hi;
  return cut_of_bins(sb, r, bins);
}

// The cut of a sample of clusters, TPT scores of one in each of four adjacent lanes.  Scores of neighbouring tokens may be
// alike, and the sample is then worth little more than its clusters: few of them hold all that reaches the cut.  Of
// independent scores 16 (1 - (1 - r / 256)^16) of the 16 clusters are expected to have one; where less than 0.85 of these do, and
// two fewer, the cut is taken again, for a variance up to 16 times as wide.  Short lists, simulated, 400 - 4000 rows each of
// 16384 tokens, B = 256, of 32768, 2048, of 32905, 6219, and 250 of 131072, 1024: independent scores none, and the cut is taken again
// in 2 % of the rows; an autoregression of 0.9, 0.98 and 0.998: at most 0.05 %, 0.2 %, 0.4 % and 0.4 % (one row) - with one cut, 3 - 15 %.
// (A sample of 64 places of 4 tokens needs no second cut and has as few short lists, but it reads four times as many lines: 128
// rows of 16384: 41.1 -> 49.8 us.)
struct ListCut {
  int r, bsel, n;
  float few;               // clusters
  template <int TPT>
  __device__ __forceinline__ static ListCut plan(int bsel, int n) {
    constexpr int M = kWave * TPT;
    const int r = list_rank(bsel, n, M);
    float none = 1.0f - fminf((float)r, (float)M) * (1.0f / M), p = none * none;    // ^ (4 TPT), the size of a cluster
    p *= p;
#pragma unroll
    for (int k = 1; k < TPT; k *= 2) p *= p;
    const float expected = (kWave / 4) * (1.0f - p);
    return {__builtin_amdgcn_readfirstlane(r), bsel, n, fminf(0.85f * expected, expected - 2.0f)};
  }
  template <int TPT>
  __device__ __forceinline__ float take(const float (&x)[TPT], uint32_t* bins, float& top) const {
    const SampleBins sb = sample_bins(x, bins);
    top = sb.hi;
    float cut = cut_of_bins(sb, r, bins);
    bool mine = false;
#pragma unroll
    for (int k = 0; k < TPT; ++k) mine |= x[k] >= cut;
    unsigned long long m = __ballot(mine);
    m |= m >> 1;
    m |= m >> 2;
    const float hit = (float)__popcll(m & 0x1111111111111111ull);
    if (__builtin_expect(hit < few, false)) {
      const int wider = list_rank(bsel, n, kWave * TPT, fminf(25.0f - 24.0f * hit / few, 4.0f * TPT));
      cut = wider <= kWave * TPT ? cut_of_bins(sb, wider, bins) : -INFINITY;
    }
    return cut;
  }
};

// A segment's list, all its waves together: acc[k] is the score of token n0 + k, which counts if it is below N.  wcnt: LDS,
// one word a wave.  list_count, a block barrier, list_write.  SHARED: read in the same launch.
template <int TPT>
__device__ __forceinline__ void list_count(const float (&acc)[TPT], int n0, int N, float cut, uint32_t* wcnt,
                                           unsigned long long (&m)[TPT]) {
  uint32_t mine = 0;
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    m[k] = __ballot(n0 + k < N && acc[k] >= cut);
    mine += (uint32_t)__popcll(m[k]);
  }
  if (lane_id() == 0) wcnt[threadIdx.x >> 6] = mine;
}
template <bool SHARED, int NT, int TPT>
__device__ __forceinline__ void list_write(const float (&acc)[TPT], int n0, const unsigned long long (&m)[TPT], const uint32_t* wcnt,
                                           uint2* seg, uint32_t* count) {
  const int wave = (int)(threadIdx.x >> 6);
  uint32_t base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) {
    const uint32_t c = wcnt[w];
    base += w < wave ? c : 0u;
    total += c;
  }
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], base));
    if ((m[k] >> lane_id()) & 1ull) {
      const uint2 e = make_uint2(score_key(acc[k]), (uint32_t)(n0 + k));
      if constexpr (SHARED) st_agent(&seg[pos], e);
      else seg[pos] = e;
    }
    base += (uint32_t)__popcll(m[k]);
  }
  if (threadIdx.x == 0) {
    if constexpr (SHARED) st_agent(count, total);
    else *count = total;
  }
}

// A row's lists as the selection sees them
struct ListView {
  const uint2* list;     // of the row
  int nsegs;             // segments of it
  int seg_tokens;        // tokens (and entries of room) of a segment
  int lanes;             // of those that load a segment's first 2 * lanes entries
  uint32_t magic;        // 2^32 / lanes + 1
  int n_cap;
  int n;                 // tokens of the row
};

// Entries 2j, 2j + 1 of the thread: two adjacent ones of a segment, whatever the memory holds there (list_mask)
template <bool SHARED, int NT, int EPT>
__device__ __forceinline__ void list_load(const ListView& v, uint32_t (&key)[EPT], uint32_t (&tok)[EPT]) {
  const __amdgpu_buffer_rsrc_t rs = agent_buffer(v.list);
#pragma unroll
  for (int j = 0; j < EPT / 2; ++j) {
    const uint32_t g = (uint32_t)(j * NT) + threadIdx.x, seg = __umulhi(g, v.magic);
    const int pos = (int)seg * v.seg_tokens + (int)(g - seg * (uint32_t)v.lanes) * 2;
    const int at = (int)seg < v.nsegs && pos < v.n_cap ? pos : 0;
    uint4 x;
    if constexpr (SHARED) x = agent_load_u128(rs, (uint32_t)at * 8u);
    else x = *reinterpret_cast<const uint4*>(v.list + at);
    key[2 * j] = x.x;
    tok[2 * j] = x.y;
    key[2 * j + 1] = x.z;
    tok[2 * j + 1] = x.w;
  }
}
// ... and key 0 where there is no entry.  seg_cnt: entries of the segments.
template <int NT, int EPT>
__device__ __forceinline__ void list_mask(const ListView& v, const uint32_t* seg_cnt, uint32_t (&key)[EPT], uint32_t (&tok)[EPT]) {
#pragma unroll
  for (int j = 0; j < EPT / 2; ++j) {
    const uint32_t g = (uint32_t)(j * NT) + threadIdx.x, seg = __umulhi(g, v.magic);
    const uint32_t off = (g - seg * (uint32_t)v.lanes) * 2;
    const uint32_t c = (int)seg < v.nsegs ? seg_cnt[min((int)seg, kListMaxSegs - 1)] : 0u;
    key[2 * j] = off < c ? key[2 * j] : 0u;
    key[2 * j + 1] = off + 1 < c ? key[2 * j + 1] : 0u;
    tok[2 * j] = min(tok[2 * j], (uint32_t)v.n - 1u);        // (a stray entry can never become a stray address)
    tok[2 * j + 1] = min(tok[2 * j + 1], (uint32_t)v.n - 1u);
  }
}

// ---------------------------------------------------------------------------------------------
// Selection of a row's set: B tokens to sm.put (find_threshold in select_common.h does the narrowing)
// ---------------------------------------------------------------------------------------------
// Places of the set that a workgroup keeps: p0 .. p1 - 1 of 0 .. B - 1 (all of them where it works alone)
template <typename Lds>
__device__ __forceinline__ void keep_place(Lds& sm, int p, int p0, int p1, uint32_t tok) {
  if (p >= p0 && p < p1) sm.put(p - p0, tok);
}

// The threshold range's share of the set, after its candidates have been listed in sm.cand (if they fit)
template <typename Lds>
__device__ __forceinline__ void resolve_threshold(Lds& sm, uint32_t klo, int bsel, int need, int n_cand,
                                                  const float* srow, int N, int p0, int p1) {
  constexpr int NT = Lds::kThreads;
  const int t = threadIdx.x;
  const int n_above = bsel - need;
  auto place = [&](int p, uint32_t tok) { keep_place(sm, p, p0, p1, tok); };
  if (n_cand <= kSelCand) {   // taken iff fewer than `need` candidates sort before it
    constexpr int P = NT / kSelCand;
    if ((t & ~(kWave - 1)) / P < n_cand) {                    // (the waves that have any)
      const int ci = t / P;
      const int rank = rank_in_list<P>(sm.cand, n_cand, ci);
      if (t % P == 0 && ci < n_cand && rank < need) place(n_above + rank, sm.cand[ci].y);
    }
  } else {                     // a tie of more than kSelCand tokens: the first `need` of them
    int tied = 0;              // met so far
    for (int i0 = 0; i0 < N && tied < need; i0 += NT) {
      const int n = i0 + t;
      const bool tie = n < N && score_key(ld_agent(srow + min(n, N - 1))) == klo;
      uint32_t tot;
      const uint32_t before = block_prefix_sum<NT>(tie ? 1u : 0u, sm.wtot, tot);
      if (tie && tied + (int)before < need) place(n_above + tied + (int)before, (uint32_t)n);
      tied += (int)tot;
    }
  }
  __syncthreads();
}

// All of a row's scores, out of memory: where there is no usable list.  klo, ktop: a key that B scores are likely to reach, and
// one at the upper end (0, 0: nothing is known).  SHARED: other workgroups of this launch wrote the scores.  Places go by
// wave.  The histogram is zero at the call (a barrier ago); ends with a block barrier.  The row is read in 16-byte
// pieces, four in flight (S is n_cap long, a multiple of 64).
template <bool SHARED, typename Lds>
__device__ __forceinline__ void row_select(Lds& sm, int bsel, const float* srow, int N, int p0, int p1, uint32_t klo = 0,
                                           uint32_t ktop = 0) {
  constexpr int NT = Lds::kThreads, NWV = Lds::kWaves;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const __amdgpu_buffer_rsrc_t rs = agent_buffer(srow);
  auto for_scores = [&](auto&& f) {                           // f(key, token, token < N), all threads together
    for (int i0 = 0; i0 < N; i0 += 16 * NT) {
      uint4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int n = i0 + (u * NT + t) * 4;
        if constexpr (SHARED) x[u] = agent_load_u128(rs, (uint32_t)(n < N ? n : 0) * 4u);
        else x[u] = *reinterpret_cast<const uint4*>(srow + (n < N ? n : 0));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int n = i0 + (u * NT + t) * 4;
        f(score_key(__uint_as_float(x[u].x)), n, n < N);
        f(score_key(__uint_as_float(x[u].y)), n + 1, n + 1 < N);
        f(score_key(__uint_as_float(x[u].z)), n + 2, n + 2 < N);
        f(score_key(__uint_as_float(x[u].w)), n + 3, n + 3 < N);
      }
    }
  };
  uint32_t khi = 0xffffffffu;
  int shift = klo ? first_shift(klo, ktop) : 22, need = bsel, n_cand;
  for (;;) {
    for_scores([&](uint32_t key, int, bool in) {
      if (in && key >= klo && key <= khi) atomicAdd(&sm.hist[min((key - klo) >> shift, (uint32_t)kSelBins - 1u)], 1u);
    });
    if (find_threshold(sm, klo, khi, shift, need, n_cand)) break;
    if (n_cand == 0) { klo = 0; shift = 22; }                 // fewer reach it: the whole range
  }
  uint32_t pw = 0, pc = 0;
  for (int pass = 0; pass < 2; ++pass) {                      // count per wave, then place
    for_scores([&](uint32_t key, int n, bool in) {
      const bool win = in && key > khi, cnd = in && key >= klo && key <= khi;
      const unsigned long long mw = __ballot(win), mc = __ballot(cnd);
      if (pass) {
        const uint32_t p = __builtin_amdgcn_mbcnt_hi((uint32_t)(mw >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mw, pw));
        const uint32_t c = __builtin_amdgcn_mbcnt_hi((uint32_t)(mc >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mc, pc));
        if (win) keep_place(sm, (int)p, p0, p1, (uint32_t)n);
        if (cnd && c < (uint32_t)kSelCand) sm.cand[c] = make_uint2(key, (uint32_t)n);
      }
      pw += (uint32_t)__popcll(mw);
      pc += (uint32_t)__popcll(mc);
    });
    __syncthreads();
    if (!pass) {
      if (lane == 0) { sm.wtot[wave] = pw; sm.wtot2[wave] = pc; }
      __syncthreads();
      pw = pc = 0;
      for (int w = 0; w < NWV - 1; ++w) {
        pw += w < wave ? sm.wtot[w] : 0u;
        pc += w < wave ? sm.wtot2[w] : 0u;
      }
    }
  }
  resolve_threshold(sm, klo, bsel, need, n_cand, srow, N, p0, p1);
}

// The same among listed scores that the threads hold (key 0: none; klo > 0).
// more(f): calls f(valid, key, token) for listed scores that no thread holds, whole waves at a time, in the same order
// each time; `over` (the same in all threads) says that there are any.  Places go by thread, then by wave of the rest.
// False: fewer than B scores are listed (the histogram is zero then).
template <int EPT, typename Lds, typename More>
__device__ __forceinline__ bool select_entries(Lds& sm, const uint32_t (&key)[EPT], const uint32_t (&tok)[EPT], bool over,
                                               More&& more, uint32_t klo, int shift, int bsel, const float* srow, int N,
                                               int p0, int p1) {
  constexpr int NWV = Lds::kWaves;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  uint32_t khi = 0xffffffffu;
  int need = bsel, n_cand;
  FASA_T_DECL(6);
  FASA_T(0);
  auto count = [&](uint32_t d) { atomicAdd(&sm.hist[min(d >> shift, (uint32_t)kSelBins - 1u)], 1u); };   // d: key - klo
  for (;;) {
    const uint32_t span = khi - klo;                          // (an empty entry's 0 - klo is larger)
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const uint32_t d = key[k] - klo;
      if (d <= span) count(d);
    }
    if (over) more([&](bool valid, uint32_t k, uint32_t) { if (valid && k - klo <= span) count(k - klo); });
    FASA_T(1);
    if (find_threshold(sm, klo, khi, shift, need, n_cand)) break;
    if (n_cand == 0) return false;
  }
  FASA_T(2);
  const uint32_t span = khi - klo;
  uint32_t n_win = 0, cnd = 0;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    n_win += key[k] > khi ? 1u : 0u;
    cnd |= key[k] - klo <= span ? 1u << k : 0u;
  }
  // both counts of a thread fit 16 bits, and so do their sums (at most EPT * NT entries)
  static_assert(EPT <= 32 && EPT * Lds::kThreads < 65536, "packed flags and counts");
  const uint32_t mine = n_win | ((uint32_t)__popc(cnd) << 16);
  const uint32_t incl = wave_prefix_sum(mine);
  if (lane == kWave - 1) sm.wtot[wave] = incl;
  __syncthreads();
  uint32_t before = incl - mine, all = 0;
#pragma unroll
  for (int w = 0; w < NWV; ++w) {
    const uint32_t x = sm.wtot[w];
    before += w < wave ? x : 0u;
    all += x;
  }
  // Winners: a wave whose winners are other workgroups' share skips the writing (of 32 workgroups a row, all but one or two
  // waves).  Candidates: few threads have one, so each takes its own one by one.
  {
    uint32_t p = (before & 0xffffu) - (uint32_t)p0;           // place in this workgroup's share
    const uint32_t len = (uint32_t)(p1 - p0);
    if (__ballot((int)p < (int)len && (int)(p + n_win) > 0) != 0ull) {
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const bool w = key[k] > khi;
        if (w && p < len) sm.put((int)p, tok[k]);
        p += w ? 1u : 0u;
      }
    }
    uint32_t pc = before >> 16;
    while (__ballot(cnd != 0u) != 0ull) {
      const int j = __ffs((int)cnd) - 1;                      // (-1: none)
      uint2 e = make_uint2(0u, 0u);
#pragma unroll
      for (int k = 0; k < EPT; ++k) e = j == k ? make_uint2(key[k], tok[k]) : e;
      if (j >= 0 && pc < (uint32_t)kSelCand) sm.cand[pc] = e;
      ++pc;
      cnd &= cnd - 1u;
    }
  }
  if (over) {
    uint32_t w0 = 0, c0 = 0;                                  // of this wave
    more([&](bool valid, uint32_t k, uint32_t) {
      w0 += (uint32_t)__popcll(__ballot(valid && k > khi));
      c0 += (uint32_t)__popcll(__ballot(valid && k >= klo && k <= khi));
    });
    __syncthreads();                                          // all have read wtot
    if (lane == 0) { sm.wtot[wave] = w0; sm.wtot2[wave] = c0; }
    __syncthreads();
    w0 = all & 0xffffu; c0 = all >> 16;
    for (int w = 0; w < wave; ++w) { w0 += sm.wtot[w]; c0 += sm.wtot2[w]; }
    more([&](bool valid, uint32_t k, uint32_t n) {
      const bool win1 = valid && k > khi, cnd1 = valid && k >= klo && k <= khi;
      const unsigned long long mw = __ballot(win1), mc = __ballot(cnd1);
      const uint32_t p = __builtin_amdgcn_mbcnt_hi((uint32_t)(mw >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mw, w0));
      const uint32_t c = __builtin_amdgcn_mbcnt_hi((uint32_t)(mc >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mc, c0));
      if (win1) keep_place(sm, (int)p, p0, p1, n);
      if (cnd1 && c < (uint32_t)kSelCand) sm.cand[c] = make_uint2(k, n);
      w0 += (uint32_t)__popcll(mw);
      c0 += (uint32_t)__popcll(mc);
    });
  }
  __syncthreads();
  FASA_T(3);
  resolve_threshold(sm, klo, bsel, need, n_cand, srow, N, p0, p1);
  FASA_T(4);
  FASA_T_PRINT(t == 0 && blockIdx.x == 0, "entries: count %llu threshold %llu place %llu resolve (%d of %d) %llu (x10ns)\n",
               FASA_T_D(1, 0), FASA_T_D(2, 1), FASA_T_D(3, 2), need, n_cand, FASA_T_D(4, 3));
  return true;
}

// What the threads do not hold.  Autoregressive scores of 0.98 have lists of 3 - 15 B, a segment's between none and all of it; us per
// step, with one cut for all kinds of rows and lists read on from memory in every pass of the selection / like this: 8 rows of
// 32768, 4 heads, B = 2048: 35.1 / 25.9, 128 rows of 16384, B = 256: 54.4 / 48.7, 32 rows of 32905, 7 heads, B = 6219: 75.2 / 59.9,
// 8 rows of 131072, B = 1024: 121 / 57.2 (independent scores: 17.8, 41.4, 50.0, 40.6, either way).

// What the lists of the wave's segments (lane l: segment l * waves + wave, c entries) hold beyond the threads' entries, to the
// wave's own part of sm.extra, where it fits: 64 entries at a time, four times in flight.  Returns their number.
template <bool SHARED, typename Lds>
__device__ __forceinline__ uint32_t gather_own(Lds& sm, const ListView& v, uint32_t c) {
  const int lane = lane_id(), wave = threadIdx.x >> 6, first = 2 * v.lanes;
  uint2* out = sm.extra + wave * Lds::kExtraPerWave;
  uint32_t have = 0;
  unsigned long long m = __ballot((int)c > first);
  const uint2* list = v.list;
  int i0 = 0, n = 0;                                          // of the segment at hand
  while (m != 0ull || i0 < n) {
    uint2 x[4];
    int left[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (i0 >= n && m != 0ull) {
        const int l = __ffsll((long long)m) - 1;
        m &= m - 1ull;
        n = min(__builtin_amdgcn_readlane((int)c, l), v.seg_tokens);
        list = v.list + (size_t)(l * Lds::kWaves + wave) * v.seg_tokens;
        i0 = first;
      }
      left[j] = max(n - i0, 0);
      const uint2* e = list + min(i0 + lane, max(n, 1) - 1);
      x[j] = SHARED ? ld_agent(e) : *e;
      i0 += kWave;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (lane < left[j]) out[have + (uint32_t)lane] = make_uint2(x[j].x, min(x[j].y, (uint32_t)v.n - 1u));
      have += (uint32_t)min(left[j], kWave);
    }
  }
  return have;
}

// A key that the B-th best of the listed scores reaches, found among those that the threads hold, if there are B of them from klo
// on (else klo).  The histogram is zero at the call and, with a block barrier, at the end.
template <int EPT, typename Lds>
__device__ __forceinline__ uint32_t held_threshold(Lds& sm, const uint32_t (&key)[EPT], uint32_t klo, int shift, int bsel) {
  uint32_t khi = 0xffffffffu;
  int need = bsel, n_cand;
  for (;;) {
    const uint32_t span = khi - klo;                          // (an empty entry's 0 - klo is larger)
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const uint32_t d = key[k] - klo;
      if (d <= span) atomicAdd(&sm.hist[min(d >> shift, (uint32_t)kSelBins - 1u)], 1u);
    }
    if (find_threshold(sm, klo, khi, shift, need, n_cand)) break;
    if (n_cand == 0) return klo;
  }
  __syncthreads();                                            // all have read thr
  for (int i = threadIdx.x; i < kSelBins; i += Lds::kThreads) sm.hist[i] = 0;
  if (threadIdx.x == 0) sm.thr[2] = 0;
  __syncthreads();
  return klo;
}

// What the lists hold beyond the threads' entries, from the key klo on, to LDS: pieces of 64 entries, numbered through all
// segments; wave w takes pieces w, w + waves, ..., four in flight, to its own part of sm.extra.  Returns the wave's number of
// entries; sm.thr[3] becomes 1 if there was no room.  The pieces' list lies in the histogram, which is zero at the call and, with a
// block barrier, at the end.
template <bool SHARED, typename Lds>
__device__ __forceinline__ uint32_t gather_beyond(Lds& sm, const ListView& v, uint32_t klo) {
  constexpr int NT = Lds::kThreads, NWV = Lds::kWaves;
  static_assert(NT >= kListMaxSegs, "a thread a segment");
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t first = 2u * (uint32_t)v.lanes, c = t < v.nsegs ? min(sm.seg_cnt[t], (uint32_t)v.seg_tokens) : 0u;
  const uint32_t mine = c > first ? (c - first + kWave - 1u) / kWave : 0u;
  uint32_t pieces;
  const uint32_t before = block_prefix_sum<NT>(mine, sm.wtot, pieces);
  for (uint32_t i = 0; i < mine; ++i)
    if (before + i < (uint32_t)kSelBins) sm.hist[before + i] = (uint32_t)t << 16 | i;
  __syncthreads();
  uint2* out = sm.extra + wave * Lds::kExtraPerWave;
  uint32_t have = 0;
  const int np = (int)min(pieces, (uint32_t)kSelBins);
  for (int p0 = wave; p0 < np; p0 += 4 * NWV) {
    uint2 x[4];
    int left[4];                                              // entries of the piece
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = p0 + j * NWV;
      const uint32_t d = sm.hist[min(p, np - 1)];
      const int s = (int)(d >> 16), i0 = (int)(first + (d & 0xffffu) * kWave), n = (int)min(sm.seg_cnt[s], (uint32_t)v.seg_tokens);
      left[j] = p < np ? n - i0 : 0;
      const uint2* e = v.list + (size_t)s * v.seg_tokens + min(i0 + lane, n - 1);
      x[j] = SHARED ? ld_agent(e) : *e;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = lane < left[j] && x[j].x >= klo;
      const unsigned long long m = __ballot(in);
      const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, have));
      if (in && at < (uint32_t)Lds::kExtraPerWave) out[at] = make_uint2(x[j].x, min(x[j].y, (uint32_t)v.n - 1u));
      have += (uint32_t)__popcll(m);
    }
  }
  if (lane == 0 && (have > (uint32_t)Lds::kExtraPerWave || pieces > (uint32_t)kSelBins)) sm.thr[3] = 1;
  __syncthreads();
  for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;
  __syncthreads();
  return have;
}

// Selection of a row out of its segments' lists in memory (row_list.h).  kcut: what they were made with; ktop: the sample's
// largest key.  SHARED: the lists were made in this launch.
template <bool SHARED, int EPT, typename Lds>
__device__ __forceinline__ void select_listed(Lds& sm, const ListView& v, const uint32_t* cnt, uint32_t kcut, uint32_t ktop,
                                              int bsel, const float* srow, int N, int p0, int p1) {
  constexpr int NT = Lds::kThreads, NWV = Lds::kWaves;
  static_assert(NT == kListMaxSegs, "a thread a segment");
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  uint32_t key[EPT], tok[EPT];
  const int mine = lane * NWV + wave;                         // segment
  uint32_t c = SHARED ? ld_agent(cnt + min(mine, v.nsegs - 1)) : cnt[min(mine, v.nsegs - 1)];
  list_load<SHARED, NT, EPT>(v, key, tok);
  for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;
  if (t == 0) sm.thr[2] = sm.thr[3] = 0;
  c = mine < v.nsegs ? c : 0u;
  sm.seg_cnt[mine] = c;
  FASA_T_DECL(5);
  FASA_T(0);
  const uint32_t sum = wave_prefix_sum(c), held = 2u * (uint32_t)v.lanes;
  uint32_t beyond = 0;                                        // entries that the threads do not hold
  if (__ballot(c > held) != 0ull) beyond = wave_prefix_sum(c > held ? min(c, (uint32_t)v.seg_tokens) - held : 0u);
  if (lane == kWave - 1) { sm.wtot[wave] = sum; sm.wtot2[wave] = beyond; }
  __syncthreads();
  uint32_t M = 0, over = 0;
#pragma unroll
  for (int w = 0; w < NWV; ++w) { M += sm.wtot[w]; over = max(over, sm.wtot2[w]); }
  list_mask<NT, EPT>(v, sm.seg_cnt, key, tok);
  FASA_T(1);
  FASA_T_PRINT(t == 0 && blockIdx.x == 0, "list counts arrive + barrier %llu M %d over %d of %d\n", FASA_T_D(1, 0), (int)M, (int)over, EPT * NT);
  uint32_t have = 0;                                          // entries of this wave in sm.extra
  const uint2* extra = sm.extra + wave * Lds::kExtraPerWave;
  auto more = [&](auto&& f) {                                 // (a wave reads what it wrote itself)
    for (uint32_t i0 = 0; i0 < have; i0 += kWave) {
      const uint2 x = extra[min(i0 + (uint32_t)lane, (uint32_t)Lds::kExtraPerWave - 1u)];
      f(i0 + (uint32_t)lane < have, x.x, x.y);
    }
  };
  uint32_t klo = max(kcut, 1u);
  bool usable = (int)M >= bsel;
  if (over != 0 && usable) {
    if (over <= (uint32_t)Lds::kExtraPerWave) {
      have = gather_own<SHARED>(sm, v, c);
    } else {
      klo = held_threshold<EPT>(sm, key, klo, kcut ? first_shift(kcut, ktop) : 22, bsel);
      have = gather_beyond<SHARED>(sm, v, klo);
      usable = sm.thr[3] == 0;                                // (not: ties, a cut that could not be made)
    }
  }
  if (usable && select_entries<EPT>(sm, key, tok, over != 0, more, klo, kcut ? first_shift(klo, max(ktop, klo)) : 22, bsel, srow, N, p0,
                                    p1))
    return;
  // Or the sample misled, and the threshold lies below the cut, as a first guess by no more than its best lies above.
  __syncthreads();                                            // (all have read the counts)
  const float cut = key_score(kcut), down = (int)M >= bsel ? cut : cut - (key_score(ktop) - cut);
  row_select<false>(sm, bsel, srow, N, p0, p1, down > -INFINITY ? score_key(down) : 0u, ktop);
}

}  // namespace fasa
