// Lists of the scores of a row that can be among its B best (paper Sec. 4.1, TopK-I), made by the workgroups that
// score it: what TopK-I has to look at shrinks from N scores to one or two times B before the row is selected.
//
//   cut      every workgroup of a row scores the same sample of the row's tokens and takes a score of it that a few
//            more than B of the row's scores should reach (list_cut).  All arrive at the same bits.
//   list     a workgroup writes the scores of its segment of the row that reach the cut, as (key, token), to the
//            segment's own stretch of the row's list, and their number (list_count, list_write): no position is shared, so there is no
//            atomic, and a stretch has room for the whole segment.
//   select   list_load, select_entries: whoever selects holds the entries in registers.  A segment that has more than
//            `load` is read on from memory in every pass; a list shorter than B, because the sample misled, is not used.
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
// among the B best, half a deviation more than sample_rank(): a list that comes out short (two to five in 100000) costs
// three passes over all scores of the row, in every one of its workgroups.
__host__ __device__ __forceinline__ int list_rank(int bsel, int n, int m) {
  const float ps = (float)bsel * ((float)m / (float)n);
  return (int)(ps + 4.0f * sqrtf(ps) + 3.0f);
}

// The cut: a score that at least r (1 .. 64 KPL) of the sample's scores reach and hardly more, in steps of a 256th of
// their spread, by one wave whose lanes hold KPL of them each: a histogram in `bins` (256 words of LDS) and one suffix sum
// (what it takes is its latency: four rounds of ballots, two bits each, take twice as long).  Infinite scores in the
// sample, or all equal: no cut (-inf).  `top`: the sample's largest score.
template <int KPL>
__device__ __forceinline__ float list_cut(const float (&x)[KPL], int r, uint32_t* bins, float& top) {
  const int lane = lane_id();
  *reinterpret_cast<uint4*>(bins + 4 * lane) = make_uint4(0, 0, 0, 0);
  float hi = -INFINITY, lo = INFINITY;
#pragma unroll
  for (int k = 0; k < KPL; ++k) {
    hi = fmaxf(hi, x[k]);
    lo = fminf(lo, x[k]);
  }
  hi = wave_max(hi);
  lo = -wave_max(-lo);
  top = hi;
  const float spread = hi - lo, inv = 256.0f * __builtin_amdgcn_rcpf(spread);
  // same wave writes and reads: its LDS operations complete in order; the fences only keep the compiler from moving them
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int k = 0; k < KPL; ++k) atomicAdd(&bins[min((uint32_t)(int)((x[k] - lo) * inv), 255u)], 1u);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const uint4 c = *reinterpret_cast<const uint4*>(bins + 4 * lane);
  const uint32_t s2 = c.w + c.z, s1 = s2 + c.y, s0 = s1 + c.x;
  const uint32_t above = wave_suffix_sum(s0) - s0;             // in higher lanes' bins
  const uint32_t need = (uint32_t)r;
  const int j = above + c.w >= need ? 3 : above + s2 >= need ? 2 : above + s1 >= need ? 1 : 0;
  const unsigned long long m = __ballot(above + s0 >= need);   // a run of low lanes
  const int last = m ? 63 - __clzll((long long)m) : 0;
  const int bin = 4 * last + __builtin_amdgcn_readlane(j, last);
  return spread > 0.0f && spread < INFINITY ? fmaf((float)bin, spread * (1.0f / 256.0f), lo) : -INFINITY;
}

// A segment's list, all its waves together: acc[k] is the score of token n0 + k, which counts if it is below N.  wcnt: LDS,
// one word a wave.  list_count, a block barrier, list_write.
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
template <int NT, int TPT>
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
    if ((m[k] >> lane_id()) & 1ull) seg[pos] = make_uint2(score_key(acc[k]), (uint32_t)(n0 + k));
    base += (uint32_t)__popcll(m[k]);
  }
  if (threadIdx.x == 0) *count = total;
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
template <int NT, int EPT>
__device__ __forceinline__ void list_load(const ListView& v, uint32_t (&key)[EPT], uint32_t (&tok)[EPT]) {
#pragma unroll
  for (int j = 0; j < EPT / 2; ++j) {
    const uint32_t g = (uint32_t)(j * NT) + threadIdx.x, seg = __umulhi(g, v.magic);
    const int pos = (int)seg * v.seg_tokens + (int)(g - seg * (uint32_t)v.lanes) * 2;
    const uint4 x = *reinterpret_cast<const uint4*>(v.list + ((int)seg < v.nsegs && pos < v.n_cap ? pos : 0));
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

}  // namespace fasa
