// Lists of the scores of a row that can be among its B best (paper Sec. 4.1, TopK-I), made by the waves that
// score it: what TopK-I has to look at shrinks from N scores to a few times B (list_room) before the row is selected.
//
//   list     a wave that holds the scores of a segment of 256 tokens writes the largest of them, `room` at most, as keys and
//            tokens to the segment's own places of the row's list (seg_list), the places left over as keys 0, and the key from
//            which on the segment is listed completely.  Nothing is shared between waves: no sample, no barrier, no atomic, and all
//            segments' lists are equally long.
//   select   select_listed: whoever selects holds the row's list in registers.  From the highest of the segments' completeness
//            keys on the list holds all of the row's scores; if B of its entries reach that key, the B best of the row are among
//            them.  If not, a row's best lie together, in segments with more of them than there was room for: those
//            segments' scores are read again, from a key on that B scores reach, and counted with the listed ones.  row_select, which
//            reads all of a row's scores, is left for rows of which fewer than B are listed or whose best don't fit in LDS (ties in their
//            thousands, NaNs).
// What the scores look like costs time, never exactness.
#pragma once

#include "attend_common.h"
#include "score_common.h"
#include "select_common.h"

namespace fasa {

constexpr int kListSeg = 256;           // tokens of a segment: four per lane of a wave
constexpr int kListMaxSegs = 2048;      // segments of a row
constexpr int kListBins = 512;          // of the selection's histogram
constexpr uint32_t kListAll = 0x007fffffu;   // the key of -inf: a segment is listed whole
constexpr int kListLimPitch = (int)(kFuseRecBytesPerRow / sizeof(uint2));
static_assert(kListLimPitch >= kListMaxSegs, "a row's segments are described where the split form has its records");

// How many scores of a segment are worth listing (a multiple of 4): four standard deviations and five above the 256 B / N of them that
// are expected among the B best.  Of independent scores hardly one segment in 10^6 has more of them than that, and a row's list is 1.7 B long
// for 6219 of 32905 tokens, 2.5 B for 2048 of 32768, 5 B for 256 of 16384, 6 B for 1024 of 131072.
__host__ __device__ __forceinline__ int list_room(int bsel, int n) {
  const float p = (float)bsel * ((float)kListSeg / (float)n);
  const int room = ((int)fmaf(4.0f, sqrtf(p), p) + 5 + 3) & ~3;
  return room < kListSeg ? room : kListSeg;
}
// Places of a segment in a row of n tokens that has `places` of them (a multiple of 4; at least 4 a segment).  A row with fewer
// tokens than another and no larger budget has need of fewer places in all, so this is list_room but for its rounding up to whole quads.
// (The quotient is exact below 256, and no place is beyond the row's.  Both sides of the lists come to the same number by the same instructions; a
// division and a root as the language has them, behind the sequence's length and ahead of its selection: paged, 16 sequences, 29.45 -> 29.35 us.)
__device__ __forceinline__ int list_pitch(int places, int bsel, int n) {
  const float q = ((float)places + 0.5f) * __builtin_amdgcn_rcpf((float)((n + kListSeg - 1) / kListSeg));
  const float p = (float)bsel * ((float)kListSeg * __builtin_amdgcn_rcpf((float)n));
  const int room = ((int)fmaf(4.0f, __builtin_amdgcn_sqrtf(p), p) + 5 + 3) & ~3;       // list_room
  return min(min(room, kListSeg), (int)fminf(q, (float)kListSeg) & ~3);
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

// ---------------------------------------------------------------------------------------------
// A segment's list, by one wave
// ---------------------------------------------------------------------------------------------
struct SegLds {
  union {
    __align__(16) uint32_t bins[256];
    __align__(16) uint32_t keys[kListSeg];
  };
  union {
    __align__(16) uint8_t toks[kListSeg];
    uint32_t toks4[kListSeg / 4];
  };
};

// Where a row's lists lie: [segment][pitch] keys, then, behind the keys' `places`, as many token numbers inside the segment, a byte each,
// and per segment the key from which on it is listed completely and its largest finite score's.  The places of a row follow from the longest row
// and the largest budget, so that whoever selects can ask for all of them, in order, before it knows how long its row is; what
// of them is a segment's (pitch, a multiple of 4, at most 256) is the row's own: a short one among longer ones with the same budget has more of
// its best in every segment.
struct ListRow {
  uint32_t* keys;
  uint32_t* toks;          // four a word
  uint2* lims;
  int pitch;
  // 5 bytes a place, and no more places than whole segments: no more than the row's 8 bytes per token of capacity (a multiple of 64) from 257
  // tokens on
  __host__ __device__ __forceinline__ static ListRow at(uint2* list, uint2* lims, int row, int n_cap, int places, int pitch) {
    uint32_t* keys = (uint32_t*)(list + (size_t)row * n_cap);
    return {keys, keys + places, lims + (size_t)row * kListLimPitch, pitch};
  }
};

// The lowest of the 256 bins from which on there are at most `room` scores (1 .. 256).  Bin 0 and those above hold more.
__device__ __forceinline__ int seg_bin(const uint32_t* bins, uint32_t room) {
  const int lane = lane_id();
  const uint4 c = *reinterpret_cast<const uint4*>(bins + 4 * lane);
  const uint32_t s2 = c.w + c.z, s1 = s2 + c.y, s0 = s1 + c.x;
  const uint32_t above = wave_suffix_sum(s0) - s0;             // in higher lanes' bins
  const int j = above + s1 <= room ? 1 : above + s2 <= room ? 2 : above + c.w <= room ? 3 : 4;
  const unsigned long long m = __ballot(above + s0 > room);    // a run of low lanes, lane 0 among them
  const int last = 63 - __clzll((long long)(m | 1ull));
  return 4 * last + __builtin_amdgcn_readlane(j, last);
}

// Lists the segment of `tokens` tokens whose score 4 lane + k is x[k]: at most as many of them as it has places, 8 or more.  The cut is the lowest edge of a bin (256 over the
// spread of the scores) that no more scores reach; where the bins are so coarse that a quarter of the places is
// left, because one score lies far from all others, the scores of the bin below the cut are cut into 256 again, from their least to their largest.  SHARED: read in this launch.
template <bool SHARED>
__device__ __forceinline__ void seg_list(const float (&x)[4], int tokens, int seg, const ListRow& l, SegLds& sm) {
  const int lane = lane_id(), room = l.pitch;
  bool in[4];
  float hi = -INFINITY, lo = INFINITY;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    in[k] = 4 * lane + k < tokens;
    const bool finite = in[k] && fabsf(x[k]) < INFINITY;
    hi = finite ? fmaxf(hi, x[k]) : hi;
    lo = finite ? fminf(lo, x[k]) : lo;
  }
  // Up to half a segment's room: the lowest of the lanes' highest, which at least 64 scores reach and one far below the rest does not move
  if (room <= kListSeg / 2) lo = hi > -INFINITY ? hi : INFINITY;
  hi = wave_max(hi);
  lo = -wave_max(-lo);
  const uint32_t top = hi > -INFINITY ? score_key(hi) : 0u;
  unsigned long long m[4];
  int n = 0;
  auto reach = [&](float c) {
    n = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      m[k] = __ballot(in[k] && x[k] >= c);
      n += __popcll(m[k]);
    }
  };
  float cut = -INFINITY, higher = -INFINITY;
  bool fits = true;
  if (tokens > room) {
    for (int zoom = 0;; ++zoom) {
      *reinterpret_cast<uint4*>(sm.bins + 4 * lane) = make_uint4(0, 0, 0, 0);
      const float spread = hi - lo, inv = 256.0f * __builtin_amdgcn_rcpf(spread);
      // the wave's LDS operations complete in order; the fences only keep the compiler from moving them
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int k = 0; k < 4; ++k)  // (infinite scores: the bins at the ends; NaNs: the lowest)
        if (in[k]) atomicAdd(&sm.bins[(uint32_t)fminf(fmaxf((x[k] - lo) * inv, 0.0f), 255.0f)], 1u);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const int bin = seg_bin(sm.bins, (uint32_t)room);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const float step = spread * (1.0f / 256.0f);
      cut = fmaf((float)bin, step, lo);
      reach(cut);
      if (n > room) {              // (the edge as a score and the edge between bins differ by a rounding; or all scores are equal)
        cut = fmaf((float)(bin + 1), step, lo);
        reach(cut);
      }
      fits = n <= room && cut == cut;      // (no cut: no score is finite)
      if (!fits && zoom > 0) {     // (ties: the cut that they lie below)
        cut = higher;
        reach(cut);
        fits = true;
        break;
      }
      if (__builtin_expect(!fits || 4 * n >= 3 * room || zoom == 2 || !(spread < INFINITY), true)) break;
      higher = cut;
      hi = -INFINITY;
      lo = INFINITY;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool below = in[k] && x[k] < cut && x[k] >= cut - step;
        hi = below ? fmaxf(hi, x[k]) : hi;
        lo = below ? fminf(lo, x[k]) : lo;
      }
      hi = wave_max(hi);
      lo = -wave_max(-lo);
      if (!(hi > lo)) break;       // (ties)
    }
  } else {
    reach(cut);
  }
  *reinterpret_cast<uint4*>(sm.keys + 4 * lane) = make_uint4(0, 0, 0, 0);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  uint32_t base = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], base));
    if (fits && ((m[k] >> lane) & 1ull)) {
      sm.keys[pos] = score_key(x[k]);
      sm.toks[pos] = (uint8_t)(4 * lane + k);
    }
    base += (uint32_t)__popcll(m[k]);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const uint2 lim = make_uint2(fits ? score_key(cut) : 0xffffffffu, top);
  if (4 * lane < l.pitch) {
    const uint4 k4 = *reinterpret_cast<const uint4*>(sm.keys + 4 * lane);
    const uint32_t t4 = sm.toks4[lane];
    const size_t at = (size_t)seg * (l.pitch / 4) + lane;
    if constexpr (SHARED) {
      st_agent(reinterpret_cast<uint2*>(l.keys) + 2 * at, make_uint2(k4.x, k4.y));
      st_agent(reinterpret_cast<uint2*>(l.keys) + 2 * at + 1, make_uint2(k4.z, k4.w));
      st_agent(l.toks + at, t4);
    } else {
      reinterpret_cast<uint4*>(l.keys)[at] = k4;
      l.toks[at] = t4;
    }
  }
  if (lane == 0) {
    if constexpr (SHARED) st_agent(l.lims + seg, lim);
    else l.lims[seg] = lim;
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
    // (One score a thread and pass in the one-launch step, whose kernels have no registers left)
    if constexpr (!Lds::kWideTies) {
      for (int i0 = 0; i0 < N && tied < need; i0 += NT) {
        const int n = i0 + t;
        const bool tie = n < N && score_key(ld_agent(srow + min(n, N - 1))) == klo;
        uint32_t tot;
        const uint32_t before = block_prefix_sum<NT>(tie ? 1u : 0u, sm.wtot, tot);
        if (tie && tied + (int)before < need) place(n_above + tied + (int)before, (uint32_t)n);
        tied += (int)tot;
      }
    } else for (int i0 = 0; i0 < N && tied < need; i0 += 4 * NT) {
      const __amdgpu_buffer_rsrc_t rs = agent_buffer(srow);
      const int n = i0 + 4 * t;                               // (S is n_cap long, a multiple of 64)
      const uint4 x = agent_load_u128(rs, (uint32_t)(n < N ? n : 0) * 4u);
      const uint32_t xs[4] = {x.x, x.y, x.z, x.w};
      uint32_t mine = 0, tot;
#pragma unroll
      for (int k = 0; k < 4; ++k) mine |= n + k < N && score_key(__uint_as_float(xs[k])) == klo ? 1u << k : 0u;
      int p = tied + (int)block_prefix_sum<NT>((uint32_t)__popc(mine), sm.wtot, tot);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool tie = (mine >> k) & 1u;
        if (tie && p < need) place(n_above + p, (uint32_t)(n + k));
        p += tie ? 1 : 0;
      }
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

// The bin of kListBins with (entries in bins above it) < need <= (entries from it on), found by every wave for itself: a round trip
// to LDS and a scan, where the search that shares it among all threads has four barriers.  n = 0: fewer than `need` in all.
struct BinAt {
  int bin, above, n;
};
__device__ __forceinline__ BinAt wave_find_bin(const uint32_t* hist, uint32_t need) {
  const int lane = lane_id();
  const uint4 a = reinterpret_cast<const uint4*>(hist)[lane], b = reinterpret_cast<const uint4*>(hist)[kWave + lane];
  const uint32_t sa = a.x + a.y + a.z + a.w, sb = b.x + b.y + b.z + b.w;
  const uint32_t ib = wave_suffix_sum(sb), tb = (uint32_t)__builtin_amdgcn_readlane((int)ib, 0), ia = wave_suffix_sum(sa) + tb;
  const bool up = tb >= need;
  const uint4 c = up ? b : a;
  const uint32_t incl = up ? ib : ia, s4 = incl - (up ? sb : sa);         // s4: in bins above this lane's four
  const uint32_t s3 = s4 + c.w, s2 = s3 + c.z, s1 = s2 + c.y;
  const unsigned long long m = __ballot(s4 < need && need <= incl);
  if (m == 0ull) return {0, 0, 0};
  const int l = __ffsll((long long)m) - 1;
  const int j = s3 >= need ? 3 : s2 >= need ? 2 : s1 >= need ? 1 : 0;
  const uint32_t above = j == 3 ? s4 : j == 2 ? s3 : j == 1 ? s2 : s1, n = j == 3 ? c.w : j == 2 ? c.z : j == 1 ? c.y : c.x;
  return {(up ? kListBins / 2 : 0) + 4 * l + __builtin_amdgcn_readlane(j, l), __builtin_amdgcn_readlane((int)above, l),
          __builtin_amdgcn_readlane((int)n, l)};
}
// log2 of the bins' width for keys from klo to ktop
__device__ __forceinline__ int list_shift(uint32_t klo, uint32_t ktop) {
  return max(0, 23 - __clz((int)(ktop > klo ? ktop - klo : 0u)));
}

// The same among listed scores that the threads hold (key 0: none; klo > 0).  Places go by thread.
// False: fewer than B scores are listed (the histogram is zero then).
template <int EPT, typename Lds>
__device__ __forceinline__ bool select_entries(Lds& sm, const uint32_t (&key)[EPT], const uint32_t (&tok)[EPT], uint32_t klo, int shift,
                                               int bsel, const float* srow, int N) {
  constexpr int NWV = Lds::kWaves;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
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
    if (n_cand == 0) return false;
  }
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
  uint32_t before = incl - mine;
#pragma unroll
  for (int w = 0; w < NWV; ++w) before += w < wave ? sm.wtot[w] : 0u;
  uint32_t p = before & 0xffffu, pc = before >> 16;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const bool w = key[k] > khi;
    if (w) keep_place(sm, (int)p, 0, bsel, tok[k]);
    p += w ? 1u : 0u;
  }
  while (__ballot(cnd != 0u) != 0ull) {                       // few threads have a candidate: each takes its own one by one
    const int j = __ffs((int)cnd) - 1;                        // (-1: none)
    uint2 e = make_uint2(0u, 0u);
#pragma unroll
    for (int k = 0; k < EPT; ++k) e = j == k ? make_uint2(key[k], tok[k]) : e;
    if (j >= 0 && pc < (uint32_t)kSelCand) sm.cand[pc] = e;
    ++pc;
    cnd &= cnd - 1u;
  }
  __syncthreads();
  resolve_threshold(sm, klo, bsel, need, n_cand, srow, N, 0, bsel);
  return true;
}

// ---------------------------------------------------------------------------------------------
// Selection of a row whose scores all lie in the workgroup's registers
// ---------------------------------------------------------------------------------------------
constexpr int kHeldMany = 128;          // candidates that take longer to rank than another pass (244 by the pass: a step of 8 float32 rows of 1000 12.4 -> 10.2 us)
constexpr int kHeldPairs = 512;         // tokens from which on the first two waves are full, and of two waves one says what is usual (HeldEnds)

// The first pass' bins: equally wide, from `lo` up to `hi`, or no further beyond `mid` than that is from `lo`.  What is above shares the last bin, what is below the first.
// Monotone whatever rounds or overflows: the ends decide how many scores share a bin, never which bin is above which.
struct LinBins {
  float lo, inv;
};
__host__ __device__ __forceinline__ LinBins lin_bins(float lo, float mid, float hi) {
  constexpr float most = 3.4028235e38f;
  lo = fmaxf(lo, -most);
  const float top = fminf(mid > lo ? fminf(hi, mid + (mid - lo)) : hi, most), bin = (top - lo) * (1.0f / kListBins);
#ifdef __HIP_DEVICE_COMPILE__
  return {lo, __builtin_amdgcn_rcpf(bin)};
#else
  return {lo, 1.0f / bin};
#endif
}
__host__ __device__ __forceinline__ uint32_t held_bin(const LinBins& b, float x) {
  return (uint32_t)fminf(fmaxf((x - b.lo) * b.inv, 0.0f), (float)(kListBins - 1));
}

// Bins for what those don't tell apart: from `lo` to `mid` 64 to 256 of them next to each other, as many for twice that distance, and so on: the upper bits of a float.  A
// score far above all others costs bins no more than it is binary orders of magnitude away, eight of them at most, and what lies beyond shares the last bin.
struct LogBins {
  float lo, c;
  uint32_t base;
  int shift;
};
__host__ __device__ __forceinline__ LogBins log_bins(float lo, float mid, float hi) {
  constexpr float most = 3.4028235e38f;
  LogBins b;
  b.lo = fminf(fmaxf(lo, -most), most);
  const float spread = hi - b.lo, c = mid - b.lo;
  b.c = fminf(c > 0.f ? c : spread, most);
  b.base = __builtin_bit_cast(uint32_t, b.c);
  const uint32_t span = __builtin_bit_cast(uint32_t, spread + b.c) - b.base;
  const int shift = span ? 23 - __builtin_clz(span) : 0;
  b.shift = shift < 0 ? 0 : shift > 17 ? 17 : shift;          // 512 bins are eight binary orders of magnitude then
  return b;
}
__host__ __device__ __forceinline__ uint32_t held_bin(const LogBins& b, float x) {
  const uint32_t bin = (__builtin_bit_cast(uint32_t, fmaxf(x - b.lo, 0.f) + b.c) - b.base) >> b.shift;
  return bin < (uint32_t)kListBins - 1u ? bin : (uint32_t)kListBins - 1u;
}

// Between what scores lie: the largest and the least of the threads' own `hi` and `lo`; and what few exceed, and few fall below: of two waves the one whose best
// (least) is less far out, so that a few scores far away don't show.  A block barrier.
struct HeldEnds {
  float lo, low, mid, hi;
};
template <typename Lds>
__device__ __forceinline__ HeldEnds held_ends(Lds& sm, float lo, float hi) {
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  hi = fmaxf(wave_max(hi), -INFINITY);                        // (a wave without a score)
  lo = fminf(-wave_max(-lo), INFINITY);
  if (lane == 0) { sm.wtot[wave] = __float_as_uint(hi); sm.wtot2[wave] = __float_as_uint(lo); }
  __syncthreads();
  HeldEnds e{lo, INFINITY, -INFINITY, hi};
#pragma unroll
  for (int w = 0; w < Lds::kWaves; w += 2) {
    const float h0 = __uint_as_float(sm.wtot[w]), h1 = __uint_as_float(sm.wtot[w + 1]), l0 = __uint_as_float(sm.wtot2[w]), l1 = __uint_as_float(sm.wtot2[w + 1]);
    e.hi = fmaxf(e.hi, fmaxf(h0, h1));
    e.lo = fminf(e.lo, fminf(l0, l1));
    e.mid = fmaxf(e.mid, fminf(h0, h1));
    e.low = fminf(e.low, fmaxf(l0, l1));
  }
  if (e.low == INFINITY) e.low = e.lo;                        // (one wave has them all)
  return e;
}

// Of the thread's scores those in bins above the `need`-th best's, which are in the set, and those in it.
struct Held {
  uint32_t win, act;
  int need, n;
  uint32_t at;             // that bin
};
// How the first pass went, of the scores from `from` on.
struct HeldFound {
  LinBins bins;
  float from;
  uint32_t at;
  int need, n;
};
// Counts bin_of(k), the bin of the k-th; bins from kListBins on: not counted.  A block barrier.  n = 0: fewer than `need` are.
template <int NV, typename Lds, typename BinOf>
__device__ __forceinline__ Held held_count(Lds& sm, Held h, BinOf&& bin_of) {
  uint32_t bin[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    bin[k] = bin_of(k);
    atomicAdd(&sm.hist[bin[k]], 1u);
  }
  __syncthreads();
  const BinAt b = wave_find_bin(sm.hist, (uint32_t)h.need);
  const uint32_t at = b.n ? (uint32_t)b.bin : (uint32_t)kListBins;
  h.act = 0;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    h.win |= bin[k] > at && bin[k] < (uint32_t)kListBins ? 1u << k : 0u;
    h.act |= bin[k] == at ? 1u << k : 0u;
  }
  h.need -= b.above;
  h.n = b.n;
  h.at = at;
  return h;
}
// The set's places: the winners' by thread, then, if there are no more than can be ranked, the candidates'.  Ends with a block barrier.
template <int NV, typename Lds, typename Token>
__device__ __forceinline__ void held_place(Lds& sm, const float (&x)[NV], Token&& token, Held h, int bsel, const float* srow, int N) {
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const uint32_t n_win = (uint32_t)__popc(h.win), incl = wave_prefix_sum(n_win);
  if (lane == kWave - 1) sm.wtot[wave] = incl;                // (all have read them: a barrier lies between)
  float v[NV];                                                // (or a choice of places to load from is made of the choice below, and x is kept in memory for it)
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = x[k];
  while (h.act != 0u) {                                       // (few lanes have a candidate)
    const int j = __ffs((int)h.act) - 1;
    float xj = v[0];
    int tj = token(0);
#pragma unroll
    for (int k = 1; k < NV; ++k) { xj = j == k ? v[k] : xj; tj = j == k ? token(k) : tj; }
    const uint32_t c = __builtin_amdgcn_atomic_inc32(&sm.n_cnd, 0xffffffffu, __ATOMIC_RELAXED, "workgroup");
    sm.cand[c & (kSelCand - 1)] = make_uint2(score_key(xj), (uint32_t)tj);
    h.act &= h.act - 1u;
  }
  __syncthreads();
  uint32_t p = incl - n_win;
#pragma unroll
  for (int w = 0; w < Lds::kWaves; ++w) p += w < wave ? sm.wtot[w] : 0u;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const bool w = h.win >> k & 1u;
    sm.put_if(w, (int)p, (uint32_t)token(k));
    p += w ? 1u : 0u;
  }
  if (h.n <= kSelCand) resolve_threshold(sm, 0u, bsel, h.need, h.n, srow, N, 0, bsel);
  else __syncthreads();
}

// The B best of such a row: x[k] of token token(k), a NaN where the row has ended.  A histogram of 512 bins gives the bin that the B-th lies in; the few in it are candidates,
// ranked by counting, and every score above is in the set.  False where that bin has more than are ranked in the time of another pass, or fewer than B scores are numbers:
// select_held_again goes on.  What the scores look like costs time, never exactness.
// Bound by the latency of a few instructions of each kind behind each other.  Four barriers, where a sample's cut, a list of what reaches it and the selection out of that had
// eleven; and what a lane has no use for goes to a word of its own in LDS, since sixteen branches around one LDS instruction each took 1.3 us.  us per step: 8 rows of
// 1531, B = 192, 10.6 -> 9.25; 1 float32 row of 4096, 256, 11.25 -> 9.95 (16 scores a thread, half of them beyond the row, and with branches 11.8).
// With bins from the least to the largest, whatever they are, one score far above all others left the rest in one bin: 8 rows of 6000, B = 256, 16.85, like this 11.95; 1 float32 row of
// 4096 12.5 / 9.95; fasa_topk of 16 rows of 2048 with one far above and one far below 5.8 / 3.45.
template <int NV, typename Lds, typename Token>
__device__ __forceinline__ bool select_held(Lds& sm, const float (&x)[NV], Token&& token, int bsel, const float* srow, int N) {
  constexpr int NT = Lds::kThreads;
  static_assert(NV <= 16 && kListBins + kWave <= kSelBins, "flags in a word; words for what is not counted");
  const int t = threadIdx.x;
  if (t == 0) sm.n_cnd = 0;
  for (int i = t; i < kListBins; i += NT) sm.hist[i] = 0;
  float hi = x[0], lo = x[0];
#pragma unroll
  for (int k = 1; k < NV; ++k) hi = fmaxf(hi, x[k]);
  // From the lowest of the threads' highest on: a score of each thread that has any, and so B of them (the row's tokens lie in fours, at most)
  const bool few = bsel <= min(NT, N / 4);
  if (few) lo = hi;
  else {
#pragma unroll
    for (int k = 1; k < NV; ++k) lo = fminf(lo, x[k]);
  }
  const HeldEnds e = held_ends(sm, lo, hi);
  const bool pairs = N >= kHeldPairs;
  const LinBins bins = lin_bins(few || !pairs ? e.lo : e.low, pairs ? e.mid : e.hi, e.hi);
  const float from = few ? e.lo : -INFINITY;
  const Held h = held_count<NV>(sm, Held{0u, 0u, bsel, 0, 0u}, [&](int k) { return x[k] >= from ? held_bin(bins, x[k]) : (uint32_t)(kListBins + lane_id()); });
  // For select_held_again, which makes its flags anew: kept in registers for what hardly ever comes they cost the one-launch step 0.1 - 0.8 us, and left in LDS in the
  // unlikely branch alone 0.2 - 0.5.
  if (t == 0) sm.found = {bins, from, h.at, h.need, h.n};
  if (__builtin_expect((uint32_t)(h.n - 1) >= (uint32_t)kHeldMany, false)) return false;
  held_place<NV>(sm, x, token, h, bsel, srow, N);
  return true;
}

// Up to two more passes, over what is left in the bin, and ties by the hundred by index, out of pieces of four tokens (or as many as a thread has), a piece's thread after
// thread.  False: they were too few, or fewer than B scores are numbers (the histogram is zero then, a barrier before the call's end is the caller's).  us, two passes of equally wide
// bins and row_select / this: fasa_topk of 16 rows of 2048, B = 256, ties by the hundred 19.0 / 5.25, a half at the type's lowest value 17.7 / 6.5; 8 of 1000, 500, every second score
// so 13.4 / 5.65.
template <int NV, typename Lds, typename Token>
__device__ __forceinline__ bool select_held_again(Lds& sm, const float (&x)[NV], Token&& token, int bsel, const float* srow, int N) {
  constexpr int NT = Lds::kThreads, P = NV < 4 ? NV : 4;
  const int t = threadIdx.x;
  __syncthreads();
  const HeldFound f = sm.found;
  Held h{0u, 0u, f.need, f.n, f.at};
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const uint32_t bin = held_bin(f.bins, x[k]);
    h.win |= x[k] >= f.from && bin > f.at ? 1u << k : 0u;
    h.act |= x[k] >= f.from && bin == f.at ? 1u << k : 0u;
  }
  bool tied = false;
#pragma unroll 1
  for (int pass = 0; pass < 2 && h.n > kHeldMany; ++pass) {
    float hi = -INFINITY, lo = INFINITY;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const bool in = h.act >> k & 1u;
      hi = in ? fmaxf(hi, x[k]) : hi;
      lo = in ? fminf(lo, x[k]) : lo;
    }
    __syncthreads();                                          // (all have read the histogram, and the last ends)
    for (int i = t; i < kListBins; i += NT) sm.hist[i] = 0;
    const HeldEnds e = held_ends(sm, lo, hi);
    tied = e.hi == e.lo;
    if (tied) break;
    const LogBins bins = log_bins(e.low, e.mid, e.hi);
    const uint32_t act = h.act;
    h = held_count<NV>(sm, h, [&](int k) { return act >> k & 1u ? held_bin(bins, x[k]) : (uint32_t)(kListBins + lane_id()); });
  }
  if (h.n == 0 || (h.n > kSelCand && !tied)) {
    __syncthreads();
    for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;
    if (t == 0) sm.thr[2] = 0;
    return false;
  }
  if (tied) {                                                 // the first `need` of them
    int p = bsel - h.need;
#pragma unroll
    for (int k0 = 0; k0 < NV; k0 += P) {
      const uint32_t m = h.act >> k0 & ((1u << P) - 1u);
      uint32_t all;
      int at = p + (int)block_prefix_sum<NT>((uint32_t)__popc(m), sm.wtot, all);
#pragma unroll
      for (int k = 0; k < P; ++k) {
        const bool in = m >> k & 1u;
        if (in && at < bsel) sm.put(at, (uint32_t)token(k0 + k));
        at += in ? 1 : 0;
      }
      p += (int)all;
    }
    h.act = 0;
    h.n = kSelCand + 1;                                       // (nothing to rank)
  }
  __syncthreads();                                            // (all have read the waves' counts, and how the first pass went)
  held_place<NV>(sm, x, token, h, bsel, srow, N);
  return true;
}

// ---------------------------------------------------------------------------------------------
// Selection of a row out of its segments' lists
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t wave_max_key(uint32_t v) {            // (in lane 63)
  v = max(v, dpp_u32<0x111, 0xF>(v));
  v = max(v, dpp_u32<0x112, 0xF>(v));
  v = max(v, dpp_u32<0x114, 0xF>(v));
  v = max(v, dpp_u32<0x118, 0xF>(v));
  v = max(v, dpp_u32<0x142, 0xA>(v));
  v = max(v, dpp_u32<0x143, 0xC>(v));
  return v;
}

// What select_listed has found: places 0 .. n_above - 1 of the set are filled, the others belong to the `need` best of the n_cand
// candidates in sm.cand (as many as fit there), whose keys are klo and above.
struct ListSet {
  bool usable;
  uint32_t klo;
  int n_above, need, n_cand;
  uint32_t from;           // the key from which on the row's scores were looked at
  uint32_t how;            // kList..., counts of the list << 8, waits for scores read again << 16
  uint32_t ktop;           // the key of the row's largest finite score
};
constexpr uint32_t kListAlone = 1, kListReread = 2, kListRow = 3;   // out of the list; with scores read again; out of all of the row's scores

// Scores of the segments that are not listed completely from a key on.  A wave takes 256 / waves tokens of every such segment, so that waves share what
// lies together, with kLoads 16-byte loads in flight (four: 32 segments; eight cost registers that two workgroups don't have).  All threads call.
template <typename Lds>
struct Beyond {
  static constexpr int NT = Lds::kThreads, LPS = kWave / Lds::kWaves, SPL = kWave / LPS;   // lanes per segment, segments per load
  static constexpr int LOADS = Lds::kLoads, MOST = LOADS * SPL;
  float4 x[LOADS];
  uint32_t end[LOADS];     // where the list of their segment begins
  int at[LOADS];           // the first one's token
  int n = 0;               // segments

  // Those among c0 .. c0 + NT - 1, in order, to sm.lim.  lim: where the list of segment c0 + t begins (0: none).
  __device__ __forceinline__ void find(Lds& sm, uint32_t lim, int c0, uint32_t klo) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const unsigned long long m = __ballot(lim > klo);
    if (lane == 0) sm.wtot[wave] = (uint32_t)__popcll(m);
    __syncthreads();                                          // (all have read the last ones, too)
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < Lds::kWaves; ++w) {
      const uint32_t c = sm.wtot[w];
      before += w < wave ? c : 0u;
      all += c;
    }
    if (lim > klo)
      sm.lim[__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, before))] =
          make_uint2(lim, (uint32_t)(c0 + t));
    n = __builtin_amdgcn_readfirstlane((int)all);
    __syncthreads();
  }
  __device__ __forceinline__ void load(const Lds& sm, const float* srow, int N, int m0) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    uint2 e[LOADS];
#pragma unroll
    for (int j = 0; j < LOADS; ++j) e[j] = sm.lim[min(m0 + j * SPL + lane / LPS, n - 1)];
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      const bool in = m0 + j * SPL + lane / LPS < n;
      // (another part of every segment: a row that rises has its best at the end of each)
      const int a = (int)e[j].y * kListSeg + ((wave + (int)e[j].y) & (Lds::kWaves - 1)) * (4 * LPS) + 4 * (lane & (LPS - 1));
      x[j] = *reinterpret_cast<const float4*>(srow + (a < N ? a : 0));     // (S is n_cap long, a multiple of 64)
      at[j] = a;
      end[j] = in ? e[j].x : 0u;
    }
  }
  // f(in, key, token) for all lanes, four times a load, from klo (> 0) on
  template <typename F>
  __device__ __forceinline__ void each(int N, int m0, uint32_t klo, F&& f) const {
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      if (m0 + j * SPL >= n) break;
      const float xs[4] = {x[j].x, x[j].y, x[j].z, x[j].w};
      const uint32_t span = end[j] > klo ? end[j] - klo : 0u;
      const int tokens = N - at[j];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t key = score_key(xs[k]);
        f(k < tokens && key - klo < span, key, (uint32_t)(at[j] + k));
      }
    }
  }
};

// What a thread holds of a row's list, requested before anything about the row but its place is known: quads t, t + NT, ... of its
// places, whatever segments they belong to.  n_max: tokens of the longest row.
// SHARED: listed in this launch.
template <bool SHARED, int NT, int Q>
struct ListHeld {
  uint2 lim;               // of segment t
  uint32_t key[4 * Q], tok4[Q];
  __device__ __forceinline__ void request(const ListRow& l, int n_max, int places) {
    const int t = threadIdx.x, most = (n_max + kListSeg - 1) / kListSeg, nq = places / 4;
    const __amdgpu_buffer_rsrc_t rk = agent_buffer(l.keys);
    lim = SHARED ? ld_agent(l.lims + min(t, most - 1)) : l.lims[min(t, most - 1)];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int g = j * NT + t, at = g < nq ? g : 0;
      uint4 x;
      if constexpr (SHARED) x = agent_load_u128(rk, (uint32_t)at * 16u);
      else x = reinterpret_cast<const uint4*>(l.keys)[at];
      key[4 * j] = x.x; key[4 * j + 1] = x.y; key[4 * j + 2] = x.z; key[4 * j + 3] = x.w;
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int g = j * NT + t, at = g < nq ? g : 0;
      if constexpr (SHARED) tok4[j] = ld_agent(l.toks + at);
      else tok4[j] = l.toks[at];
    }
  }
};

// Selection of a row out of its list by all threads: places p0 .. p1 - 1 of its set to sm.put, as far as they
// are known without ranking the candidates.  Ends with a block barrier.
template <bool SHARED, int Q, typename Lds>
__device__ __forceinline__ ListSet select_listed(Lds& sm, const ListRow& l, ListHeld<SHARED, Lds::kThreads, Q>& held, int bsel, const float* srow,
                                                 int N, int p0, int p1) {
  constexpr int NT = Lds::kThreads, NWV = Lds::kWaves, EPT = 4 * Q;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, per = l.pitch / 4;
  uint2& lt = held.lim;
  uint32_t (&key)[EPT] = held.key;
  uint32_t (&tok4)[Q] = held.tok4;
  for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;
  if (t == 0) { sm.thr[2] = sm.thr[3] = 0; sm.n_cnd = 0; }
  const int nsegs = (N + kListSeg - 1) / kListSeg, nq = nsegs * per;
  if (t >= nsegs) lt = make_uint2(0u, 0u);
  for (int i = NT + t; i < nsegs; i += NT) {
    const uint2 x = SHARED ? ld_agent(l.lims + i) : l.lims[i];
    lt = make_uint2(max(lt.x, x.x), max(lt.y, x.y));
  }
  {
    const uint32_t a = wave_max_key(lt.x), b = wave_max_key(lt.y);
    if (lane == kWave - 1) { sm.wtot[wave] = a; sm.wtot2[wave] = b; }
  }
  // The tokens are needed much later, and only by the waves whose winners are in the share, so the compiler would move their loads
  // there: 8 rows of 32768, B = 2048, 18.1 us, like this 17.0.
#pragma unroll
  for (int j = 0; j < Q; ++j) asm volatile("" : "+v"(tok4[j]));
  __syncthreads();
  FASA_T_DECL(10);
  FASA_T(0);
  uint32_t klo = 1, ktop = 0;
#pragma unroll
  for (int w = 0; w < NWV; ++w) { klo = max(klo, sm.wtot[w]); ktop = max(ktop, sm.wtot2[w]); }
  uint32_t from = klo, how = kListAlone;
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const bool in = j * NT + t < nq;
#pragma unroll
    for (int k = 0; k < 4; ++k) key[4 * j + k] = in ? key[4 * j + k] : 0u;
  }
  bool over = false;                                          // there are entries that no thread holds:
  uint32_t have = 0;                                          // so many of this wave's in sm.extra
  const uint2* extra = sm.extra + wave * Lds::kExtraPerWave;
  auto more = [&](auto&& f) {                                 // (a wave reads what it wrote itself)
    for (uint32_t i0 = 0; i0 < have; i0 += kWave) {
      const uint2 x = extra[min(i0 + (uint32_t)lane, (uint32_t)Lds::kExtraPerWave - 1u)];
      f(i0 + (uint32_t)lane < have, x.x, x.y);
    }
  };
  uint32_t khi = 0;
  int shift = 0, need = 0, n_cand = 0;
  auto clear = [&]() {
    __syncthreads();                                          // all have read it
    for (int i = t; i < kListBins; i += NT) sm.hist[i] = 0;
    __syncthreads();
  };
  auto whole_range = [&](uint32_t lo) { klo = lo; khi = 0xffffffffu; shift = list_shift(lo, ktop); need = bsel; };
  // one range: true if it holds `need` entries
  auto search = [&]() {
    how += 1u << 8;
    const uint32_t span = khi - klo;                          // (an empty entry's 0 - klo is larger)
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const uint32_t d = key[k] - klo;
      if (d <= span) atomicAdd(&sm.hist[min(d >> shift, (uint32_t)kListBins - 1u)], 1u);
    }
    if (over) more([&](bool valid, uint32_t k, uint32_t) {
      if (valid && k - klo <= span) atomicAdd(&sm.hist[min((k - klo) >> shift, (uint32_t)kListBins - 1u)], 1u);
    });
    __syncthreads();
    const BinAt b = wave_find_bin(sm.hist, (uint32_t)need);
    n_cand = b.n;
    if (b.n == 0) return false;
    need -= b.above;
    narrow_range<kListBins>(klo, khi, (uint32_t)b.bin, shift);
    return true;
  };
  // the range of the keys that there are in it, and the histogram cleared
  auto tighten = [&]() {
    const uint32_t lo = klo, span = khi - klo;
    uint32_t above = 0, below = 0;                            // of the lowest, of the highest; 0: none
    auto look = [&](uint32_t k) {
      const bool in = k - lo <= span;
      above = max(above, in ? k : 0u);
      below = max(below, in ? ~k : 0u);
    };
#pragma unroll
    for (int k = 0; k < EPT; ++k) look(key[k]);
    if (over) more([&](bool valid, uint32_t k, uint32_t) { look(valid ? k : 0u); });
    above = wave_max_key(above);
    below = wave_max_key(below);
    if (lane == kWave - 1) { sm.wtot[wave] = above; sm.wtot2[wave] = below; }
    __syncthreads();                                          // (all have read the histogram, too)
    for (int i = t; i < kListBins; i += NT) sm.hist[i] = 0;
    above = below = 0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) { above = max(above, sm.wtot[w]); below = max(below, sm.wtot2[w]); }
    klo = ~below;
    khi = above;
    shift = max(0, 23 - __clz((int)(khi - klo)));             // (khi - klo) >> shift < kListBins
    __syncthreads();
  };
  // until it has at most kSelCand entries, or one key (ties); always true: the same entries are searched
  auto narrow = [&]() {
    while (n_cand > kSelCand && klo != khi) {
      tighten();
      if (klo == khi || !search()) break;
    }
  };
  whole_range(klo);
  if (__builtin_expect(!search(), false)) {
    // Segments with more of the best than they had places for.  Lanes count in eight histograms here, one bin's side by side: neighbours that
    // are alike would all wait for one word.  us per step, a key by two to four counts of the list and two or three passes over the segments / like
    // this, 8 rows of 32768, B = 2048: independent scores 14.0 / 13.9, an autoregression of 0.98 22.5 / 20.1, of 0.998 33.4 / 20.6, rising
    // 34.3 / 19.3; 32 of 32905, 6219: 33.1 / 32.2, 45.5 / 41.1, 62.3 / 42.2, 76.0 / 41.7; 8 of 131072, 1024: 17.7 / 17.7, 34.4 / 25.8, 54.8 /
    // 26.5, 46.2 / 23.6.  Of what rising rows take longer, the failed count is 1.5, the key 1.5, the scores 1.9, counting 1.9, keeping 1.4.
    uint32_t* const wide = reinterpret_cast<uint32_t*>(sm.extra);
    static_assert(sizeof(sm.extra) >= kListBins * 32 && NT >= kListBins, "eight histograms, a bin of each by a thread");
    auto none = [&](uint32_t reached) { clear(); return ListSet{false, reached, 0, 0, 0, from, how | kListRow, ktop}; };
    auto clear_wide = [&]() {                                 // (all have read it: a barrier ago)
      if (t < kListBins) {
        reinterpret_cast<uint4*>(wide)[2 * t] = make_uint4(0, 0, 0, 0);
        reinterpret_cast<uint4*>(wide)[2 * t + 1] = make_uint4(0, 0, 0, 0);
      }
      __syncthreads();
    };
    auto add = [&](uint32_t k, uint32_t n) { atomicAdd(&wide[min((k - klo) >> shift, (uint32_t)kListBins - 1u) * 8u + (uint32_t)(lane & 7)], n); };
    auto search_wide = [&]() {
      how += 1u << 8;
      const uint32_t lo = klo;
#pragma unroll
      for (int k = 0; k < EPT; ++k)
        if (key[k] >= lo) add(key[k], 1u);
      __syncthreads();
      if (t < kListBins) {
        const uint4 a = reinterpret_cast<const uint4*>(wide)[2 * t], b = reinterpret_cast<const uint4*>(wide)[2 * t + 1];
        sm.hist[t] = a.x + a.y + a.z + a.w + b.x + b.y + b.z + b.w;
      }
      __syncthreads();
      const BinAt b = wave_find_bin(sm.hist, (uint32_t)need);
      n_cand = b.n;
      if (b.n == 0) return false;
      need -= b.above;
      narrow_range<kListBins>(klo, khi, (uint32_t)b.bin, shift);
      return true;
    };
    // no listed entry lies below the lowest of the completeness keys, but for those of a short last segment that is listed whole
    uint32_t lowest = wave_max_key(t >= nsegs || lt.x <= kListAll || nsegs > NT ? 0u : ~lt.x);
    if (lane == kWave - 1) sm.wtot[wave] = lowest;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NWV; ++w) lowest = max(lowest, sm.wtot[w]);
    lowest = lowest != 0u ? ~lowest : 1u;
    FASA_T(5);
    Beyond<Lds> beyond;
    auto for_beyond = [&](bool held, auto&& f) {
      for (int c0 = 0; c0 < nsegs; c0 += NT) {
        if (!held) {
          uint32_t lim = lt.x;
          if (nsegs > NT) {
            const uint2* p = l.lims + min(c0 + t, nsegs - 1);
            lim = c0 + t < nsegs ? (SHARED ? ld_agent(p) : *p).x : 0u;
          }
          beyond.find(sm, lim, c0, klo);
        }
        for (int m0 = 0; m0 < beyond.n; m0 += Beyond<Lds>::MOST) {
          if (!held) {
            beyond.load(sm, srow, N, m0);
            how += 1u << 16;
          }
          beyond.each(N, m0, klo, f);
        }
      }
    };
    // A key that B scores reach, and not many more: first as if a segment's scores went on below its list as they do in it, half as dense, and
    // in the best scores' four binades, where bins are fine; should fewer than B reach that, by the listed ones alone.  The scores of the segments that are
    // not listed completely from there on are read and counted with the listed ones.
    const float top = key_score(ktop);
    for (int attempt = nsegs <= NT && top > 0.f ? 0 : 1;; ++attempt) {
      const bool guess = attempt == 0;
      whole_range(guess ? max(lowest, score_key(top * 0.0625f)) : attempt < 2 ? lowest : 1u);
      if (guess) need += bsel / 16;
      clear_wide();
      if (guess && lt.x > klo && lt.y > lt.x) {
        const float lim = key_score(lt.x), w = 0.25f * (float)(kListSeg - l.pitch);
        const float step = (key_score(lt.y) - lim) * w * __builtin_amdgcn_rcpf((float)l.pitch);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t k = score_key(fmaf(-step, (float)j + 0.5f, lim));
          if (k > klo && k < lt.x) add(k, (uint32_t)(0.5f * w));
        }
      }
      if (!search_wide()) {
        if (attempt == 2) return none(0u);                    // fewer than B are listed
        continue;
      }
      FASA_T(6);
      from = klo;
      whole_range(klo);
      clear_wide();
      for_beyond(false, [&](bool in, uint32_t key, uint32_t) { if (in) add(key, 1u); });
      FASA_T(7);
      if (search_wide()) break;
      if (attempt == 2) return none(0u);
    }
    FASA_T(8);
    // What reaches the threshold's bin is kept (all would not fit: where scores rise through the row, 16 B)
    uint2* out = sm.extra + wave * Lds::kExtraPerWave;
    for_beyond(Lds::kLoads > 1 /* one load is not worth its registers */ && nsegs <= NT && beyond.n <= Beyond<Lds>::MOST, [&](bool in, uint32_t key, uint32_t tok) {
      const unsigned long long b = __ballot(in);
      const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, have));
      if (in && pos < (uint32_t)Lds::kExtraPerWave) out[pos] = make_uint2(key, tok);
      have += (uint32_t)__popcll(b);
    });
    if (lane == 0 && have > (uint32_t)Lds::kExtraPerWave) sm.thr[3] = 1;
    __syncthreads();
    if (sm.thr[3] != 0) return none(klo);                      // (ties)
    over = true;
    how += kListReread - kListAlone;
    FASA_T(9);
    FASA_T_PRINT(t == 0 && blockIdx.x == 0, "beyond: first %llu listed key %llu read(%d) %llu search %llu keep(%d) %llu (x10ns)\n", FASA_T_D(5, 0), FASA_T_D(6, 5),
                 beyond.n, FASA_T_D(7, 6), FASA_T_D(8, 7), (int)have, FASA_T_D(9, 8));
  }
  narrow();
  FASA_T(1);
  const int n_above = bsel - need;
  const uint32_t span = khi - klo;
  uint32_t n_win = 0;
#pragma unroll
  for (int k = 0; k < EPT; ++k) n_win += key[k] > khi ? 1u : 0u;
  const uint32_t incl = wave_prefix_sum(n_win);
  uint32_t w0 = 0;                                            // winners of this wave in sm.extra
  if (over) more([&](bool valid, uint32_t k, uint32_t) { w0 += (uint32_t)__popcll(__ballot(valid && k > khi)); });
  if (lane == kWave - 1) { sm.wtot[wave] = incl; sm.wtot2[wave] = w0; }   // (all have read them: a barrier lies between)
  const float inv_per = __builtin_amdgcn_rcpf((float)per);
  auto token = [&](int j, int k) {                            // (quotients of at most 4096 by at most 64: exact)
    const uint32_t seg = (uint32_t)(((float)(j * NT + t) + 0.5f) * inv_per);
    return min(seg * (uint32_t)kListSeg + (tok4[j] >> (8 * k) & 255u), (uint32_t)N - 1u);
  };
  auto candidate = [&](uint32_t k, uint32_t tok) {
    const uint32_t p = __builtin_amdgcn_atomic_inc32(&sm.n_cnd, 0xffffffffu, __ATOMIC_RELAXED, "workgroup");
    if (p < (uint32_t)kSelCand) sm.cand[p] = make_uint2(k, tok);
  };
  if (p1 > n_above) {                                         // (of 32 workgroups a row, one or two)
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (key[4 * j + k] - klo <= span) candidate(key[4 * j + k], token(j, k));
    if (over) more([&](bool valid, uint32_t k, uint32_t n) { if (valid && k - klo <= span) candidate(k, n); });
  }
  __syncthreads();
  uint32_t before = incl - n_win, all = 0;
#pragma unroll
  for (int w = 0; w < NWV; ++w) {
    const uint32_t x = sm.wtot[w];
    before += w < wave ? x : 0u;
    all += x;
  }
  {
    uint32_t p = before - (uint32_t)p0;                       // place in this workgroup's share
    const uint32_t len = (uint32_t)(p1 - p0);
    if (__ballot((int)p < (int)len && (int)(p + n_win) > 0) != 0ull) {   // (of 32 workgroups a row, one or two waves)
#pragma unroll
      for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const bool w = key[4 * j + k] > khi;
          if (w && p < len) sm.put((int)p, token(j, k));
          p += w ? 1u : 0u;
        }
    }
  }
  if (over) {
    uint32_t p = all;
    for (int w = 0; w < wave; ++w) p += sm.wtot2[w];
    more([&](bool valid, uint32_t k, uint32_t n) {
      const unsigned long long b = __ballot(valid && k > khi);
      const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, p));
      if (valid && k > khi) keep_place(sm, (int)at, p0, p1, n);
      p += (uint32_t)__popcll(b);
    });
  }
  __syncthreads();
  FASA_T(2);
  FASA_T_PRINT(t == 0 && blockIdx.x == 0, "listed: threshold %llu places %llu (x10ns), %d entries, %d of %d candidates\n", FASA_T_D(1, 0),
               FASA_T_D(2, 1), 4 * nq, need, n_cand);
  return {true, klo, n_above, need, n_cand, from, how, ktop};
}

}  // namespace fasa
