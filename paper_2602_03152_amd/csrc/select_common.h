// Pieces of TopK-I (paper Sec. 4.1) shared by the stand-alone selection kernel and the fused
// selection + attention kernel: the block-wide search of the threshold bin in a histogram and the
// exact resolve of the threshold bin's candidates (ties towards the lower token index).
#pragma once

#include "fasa_device.h"
#include "fasa_internal.h"
#include "fasa_trace.h"

namespace fasa {

// A candidate is (order-preserving score key, token index).  Its composite sorts candidates the way
// the selection ranks tokens: larger key first, equal keys by lower index (the index is inverted).
// CB = significant bits of the composite:
//   52  all candidates share the top 12 key bits (bins of the exponent-based histogram): the low 20
//       key bits and the index decide;
//   64  candidates of an arbitrary score interval (bins of the adaptive histogram): the whole key.
template <int CB>
__device__ __forceinline__ unsigned long long cand_composite(uint2 c) {
  if constexpr (CB == 52)
    return ((unsigned long long)(c.x & ((1u << kKeyLowBits) - 1u)) << 32) | (unsigned long long)(~c.y);
  else
    return ((unsigned long long)c.x << 32) | (unsigned long long)(~c.y);
}

// Block-wide search in a histogram of 256 * PER bins of which thread t holds bins PER t .. PER t + PER - 1
// in hb[]: the bin b with  (entries in bins above b) < need <= (entries in bins >= b).  All 256 threads
// call; out[0..2] = b, entries above it, entries inside it (LDS; left as they are if need exceeds the
// total, the caller presets them).  Ends with a block barrier.
template <int PER>
__device__ __forceinline__ void find_bin_256(const uint32_t* hb, uint32_t need, uint32_t* wtot, uint32_t* out) {
  const int t = threadIdx.x;
  uint32_t mine = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) mine += hb[j];
  const uint32_t incl = block256_suffix_sum(mine, wtot);
  uint32_t cum = incl - mine;
  const bool owner = cum < need && need <= incl;   // true for exactly one thread of the block
  // branch-free scan of the thread's bins from the top; the one hit is kept in registers
  uint32_t bj = 0, ba = 0, bn = 0;
#pragma unroll
  for (int j = PER - 1; j >= 0; --j) {
    const bool hit = cum < need && cum + hb[j] >= need;
    bj = hit ? (uint32_t)j : bj;
    ba = hit ? cum : ba;
    bn = hit ? hb[j] : bn;
    cum += hb[j];
  }
  if (owner) {
    out[0] = (uint32_t)(t * PER) + bj;
    out[1] = ba;
    out[2] = bn;
  }
  __syncthreads();
}

// Rank of candidate i among the n candidates of an LDS list: how many of them sort before it (larger
// key, or equal key and lower index).  Composites are distinct, so ranks are a permutation of 0..n-1
// and "rank < need" takes exactly the `need` best.  32-bit compares only; the list is read eight
// entries at a time (one LDS round trip per eight).  Thread t serves candidate t / PARTS and counts
// the entries j = t % PARTS (mod PARTS); the PARTS partial counts of a candidate sit in adjacent lanes
// and are added with DPP moves.  Returns the rank in every one of the candidate's threads.
template <int PARTS>
__device__ __forceinline__ int rank_in_list(const uint2* lc, int n, int i) {
  const int t = threadIdx.x;
  const uint2 me = lc[min(i, n - 1)];
  int rank = 0;
  for (int j0 = t % PARTS; j0 < n; j0 += 8 * PARTS) {
    uint2 c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) c[u] = lc[min(j0 + u * PARTS, n - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool before = c[u].x > me.x || (c[u].x == me.x && c[u].y < me.y);
      rank += (j0 + u * PARTS < n && before) ? 1 : 0;
    }
  }
  if constexpr (PARTS >= 2) rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
  if constexpr (PARTS >= 4) rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
  return rank;
}

constexpr int kSelBins = 1024;
constexpr int kSelCand = 256;    // candidates of the threshold bin ranked by counting

// The keys of SMP of a row's scores (thread i < SMP brings sval) in ssort, largest first, by all NT threads of a block.
// They are made distinct in their low bits: ranks are a permutation, and a cut may be any value.  (The low bits are
// cleared again in ssort: such a key need not be one that a score can have.)  Two block barriers, the last at the end;
// init() runs ahead of the first (ahead of this call it costs one instance of the step a spilled register).
template <int NT, int SMP, typename Init>
__device__ __forceinline__ void rank_sample(float sval, uint32_t* sample, uint32_t* ssort, Init&& init) {
  const int t = threadIdx.x;
  if (t < SMP) sample[t] = (score_key(sval) & ~(uint32_t)(SMP - 1)) | (uint32_t)t;
  init();
  __syncthreads();
  constexpr int P = NT / SMP;                                 // threads per sample value: adjacent lanes
  static_assert(P == 4 || P == 8, "a quad or half a row of lanes per value");
  const uint32_t me = sample[t / P];
  int rank = 0;
#pragma unroll
  for (int u = 0; u < SMP / 4 / P; ++u) {
    const uint4 o = reinterpret_cast<const uint4*>(sample)[P * u + t % P];
    rank += (o.x > me ? 1 : 0) + (o.y > me ? 1 : 0) + (o.z > me ? 1 : 0) + (o.w > me ? 1 : 0);
  }
  rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xF, 0xF, true);                           // quad_perm [1,0,3,2]
  rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xF, 0xF, true);                           // quad_perm [2,3,0,1]
  if constexpr (P == 8) rank += __builtin_amdgcn_update_dpp(0, rank, 0x141, 0xF, 0xF, true);    // row_half_mirror
  if (t % P == 0) ssort[rank & (SMP - 1)] = me & ~(uint32_t)(SMP - 1);
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------
// Selection by one workgroup of all its row's scores: the B best.  A first range of keys klo .. 2^32 - 1 (no
// score below it may be among the B best) is cut into kSelBins bins of 2^shift keys:
//   histogram  a suffix sum gives the threshold bin: bins above it hold fewer than B scores, bins from it
//              upwards at least B.
//   narrow     while the threshold bin holds more than kSelCand scores it becomes the next range, 1024
//              times finer.  What the scores look like costs passes, never exactness.
//   resolve    the bin's candidates are ranked by counting (key, then lower index).  A bin that is one key
//              wide and still too full is a tie of that many tokens: they are taken in index order, out of
//              the row's scores in memory.
// ---------------------------------------------------------------------------------------------
// The threshold bin, which holds a key of klo .. khi, as the next range.  The last bin reaches up to khi; no other beyond it: a
// bin that a NaN's key lies in may end past the largest key there is.
template <int BINS = kSelBins>
__host__ __device__ __forceinline__ void narrow_range(uint32_t& klo, uint32_t& khi, uint32_t bin, int shift) {
  klo += bin << shift;
  const uint32_t left = khi - klo, width = (1u << shift) - 1u;
  if (bin + 1 < (uint32_t)BINS) khi = klo + (width < left ? width : left);
}
// After the counting: true once klo .. khi is the final range (need of its n_cand scores are taken, and all
// above it); else the range to count next, the histogram zeroed - the same range, with n_cand 0, if fewer than
// need scores were counted in it.  sm.thr[2] has to be 0 at the call then; where every score of the range is counted
// (need is met in all passes) only at the first.  A range of one key with more than kSelCand scores ends the search too.
template <typename Lds>
__device__ __forceinline__ bool find_threshold(Lds& sm, uint32_t& klo, uint32_t& khi, int& shift, int& need, int& n_cand) {
  const int t = threadIdx.x;
  __syncthreads();
  constexpr int NT = Lds::kThreads, BPT = kSelBins / NT;     // bins per thread: 4, 2 or 1
  uint32_t hb[BPT], mine = 0;
#pragma unroll
  for (int j = 0; j < BPT; ++j) { hb[j] = sm.hist[BPT * t + j]; mine += hb[j]; }
  const uint32_t incl = block_suffix_sum<NT>(mine, sm.wtot);
  uint32_t above = incl - mine;                               // scores in bins above this thread's
  if (above < (uint32_t)need && (uint32_t)need <= incl) {
#pragma unroll
    for (int j = BPT - 1; j >= 0; --j) {
      if (above < (uint32_t)need && above + hb[j] >= (uint32_t)need) {
        sm.thr[0] = (uint32_t)(BPT * t + j);
        sm.thr[1] = above;
        sm.thr[2] = hb[j];
      }
      above += hb[j];
    }
  }
  __syncthreads();
  n_cand = (int)sm.thr[2];
  if (n_cand > 0) {
    const uint32_t bin = sm.thr[0];
    need -= (int)sm.thr[1];
    narrow_range(klo, khi, bin, shift);
    if (n_cand <= kSelCand || klo == khi) return true;
    shift = max(0, 22 - __clz((int)(khi - klo)));             // (khi - klo) >> shift < 1024
  }
#pragma unroll
  for (int j = 0; j < BPT; ++j) sm.hist[BPT * t + j] = 0;
  __syncthreads();
  return false;
}
// log2 of the bins' width for keys from kcut to twice the distance to ktop: span >> shift < 1024
__device__ __forceinline__ int first_shift(uint32_t kcut, uint32_t ktop) {
  const unsigned long long span = 2ull * (ktop - kcut) + kSelBins;
  return max(0, 54 - __clzll((long long)span));
}

// Exact selection of the `need` largest composites among cand[0..n).  Whole block participates.
// SHARED_SRC: the list lives in global memory and was written by other workgroups.
// dhw: LDS scratch of 4096 counters, or null.  With it the first pass takes the top 12 bits of the
// composite at once, which for a few hundred candidates of one exponent-based bin almost always isolates
// the boundary candidate, so that no second pass is needed; without it every pass takes 8 bits.
// out receives the token numbers of the taken candidates (at most `need`), in no particular order.
// out_slot (paged caches, else null): receives the pool slot of every token written to out.
// out_lds (or null): LDS copy of what the attention gathers by (the slot if out_slot is given, else the
// token number), same positions as out.
template <bool SHARED_SRC, int NT, int CB>
__device__ void resolve_candidates(const uint2* cand, int n, int need, int32_t* out,
                                   uint32_t* dh /*256*/, uint32_t* wtot /*NT/64*/,
                                   uint32_t* bc /*4: digit, need, count, out counter*/,
                                   uint32_t* dhw, int32_t* out_slot, const PageMap& pm, int b,
                                   int32_t* out_lds = nullptr) {
  const int t = threadIdx.x;
  const uint32_t out_cap = (uint32_t)need;  // never write past the row's share of T
  unsigned long long prefix = 0;
  int shift = CB;            // bits of the composite not yet decided
  // The list is walked four entries per thread at a time, the four reads issued together (one LDS
  // or memory round trip per chunk instead of one per entry); entry u of chunk i0 is i0 + u*NT + t.
  constexpr int CH = 4;
  auto load_chunk = [&](int i0, uint2 (&c)[CH]) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int i = min(i0 + u * NT + t, n - 1);
      c[u] = SHARED_SRC ? ld_agent(&cand[i]) : cand[i];
    }
  };
  FASA_T_DECL(5);
  FASA_T(0);
  if (need < n) {
    bool done = false;
    if (NT == 256 && dhw != nullptr) {
      shift = CB - 12;       // 12-bit digit first, then 8-bit digits
      for (int i = t; i < kHistBins; i += NT) dhw[i] = 0;
      if (t == 0) { bc[0] = 0; bc[1] = 0; bc[2] = 0; }
      __syncthreads();
      for (int i0 = 0; i0 < n; i0 += CH * NT) {
        uint2 c[CH];
        load_chunk(i0, c);
#pragma unroll
        for (int u = 0; u < CH; ++u)
          if (i0 + u * NT + t < n) atomicAdd(&dhw[(uint32_t)(cand_composite<CB>(c[u]) >> (CB - 12))], 1u);
      }
      __syncthreads();
      FASA_T(1);
      uint32_t hb[16];
      const uint4* hp = reinterpret_cast<const uint4*>(dhw + t * 16);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint4 v = hp[j];
        hb[4 * j] = v.x; hb[4 * j + 1] = v.y; hb[4 * j + 2] = v.z; hb[4 * j + 3] = v.w;
      }
      find_bin_256<16>(hb, (uint32_t)need, wtot, bc);
      prefix = bc[0];
      const uint32_t in_digit = bc[2];
      need -= (int)bc[1];
      done = (uint32_t)need == in_digit;     // everything under this prefix is a winner
      __syncthreads();                       // bc is rewritten by the passes below
      FASA_T(2);
    }
    while (!done && shift > 0) {
      const int width = shift >= 8 ? 8 : shift;   // the last digit is whatever is left over
      const bool first = shift == 64;             // nothing decided yet: every candidate is in play
      shift -= width;
      if (t < 256) dh[t] = 0;
      __syncthreads();
      for (int i0 = 0; i0 < n; i0 += CH * NT) {
        uint2 c[CH];
        load_chunk(i0, c);
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          const unsigned long long cc = cand_composite<CB>(c[u]);
          const bool in_play = first || (cc >> ((shift + width) & 63)) == prefix;
          if (i0 + u * NT + t < n && in_play)
            atomicAdd(&dh[(uint32_t)(cc >> shift) & ((1u << width) - 1u)], 1u);
        }
      }
      __syncthreads();
      const uint32_t cnt = t < 256 ? dh[t] : 0u;
      const uint32_t incl = block_suffix_sum<NT>(cnt, wtot);
      const uint32_t excl = incl - cnt;
      if (t < 256 && excl < (uint32_t)need && (uint32_t)need <= incl) {
        bc[0] = (uint32_t)t;
        bc[1] = (uint32_t)need - excl;
        bc[2] = cnt;
      }
      __syncthreads();
      prefix = (prefix << width) | bc[0];
      need = (int)bc[1];
      const uint32_t in_digit = bc[2];
      // no barrier needed here: bc is next written three barriers into the following pass
      if ((uint32_t)need == in_digit) break;  // everything under this prefix is a winner
    }
  } else {
    shift = 63;   // take all: (c >> 63) >= 0
  }
  FASA_T(3);
  // output: one position atomic per wave and chunk (ballots give every taken entry its offset)
  for (int i0 = 0; i0 < n; i0 += CH * NT) {
    uint2 c[CH];
    load_chunk(i0, c);
    unsigned long long m[CH];
    uint32_t taken = 0;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      m[u] = __ballot(i0 + u * NT + t < n && (cand_composite<CB>(c[u]) >> shift) >= prefix);
      taken += (uint32_t)__popcll(m[u]);
    }
    int sl[CH];
    if (out_slot) {   // paged cache: where the rows live; looked up before the stores below
#pragma unroll
      for (int u = 0; u < CH; ++u) sl[u] = kv_slot(pm, b, (int)(c[u].y & 0x7fffffffu));
    }
    uint32_t pos = 0;
    if (lane_id() == 0 && taken) pos = atomicAdd(&bc[3], taken);
    pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos);
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const uint32_t mine = pos + __builtin_amdgcn_mbcnt_hi((uint32_t)(m[u] >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)m[u], 0u));
      if (((m[u] >> lane_id()) & 1ull) && mine < out_cap) {
        out[mine] = (int32_t)c[u].y;
        if (out_slot) out_slot[mine] = sl[u];
        if (out_lds) out_lds[mine] = out_slot ? sl[u] : (int32_t)c[u].y;
      }
      pos += (uint32_t)__popcll(m[u]);
    }
  }
  FASA_T(4);
  FASA_T_PRINT(t == 0 && blockIdx.x < 64, "resolve: widehist %llu findbin %llu passes %llu output %llu (x10ns)\n",
               FASA_T_D(1, 0), FASA_T_D(2, 1), FASA_T_D(3, 2), FASA_T_D(4, 3));
}

}  // namespace fasa
