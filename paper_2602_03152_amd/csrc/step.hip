// The decode step by workgroups that know a row's whole set (paper Sec. 4.1 - 4.2, Alg. 2 order): they select the row's B best
// tokens out of a list of the few scores that can be among them, and attend over them.  Three forms:
//
//   step_kernel    the whole step in ONE launch.  A row of at most 512 * TPT tokens is scored, selected
//                  and attended by one workgroup.  A longer row is scored by several; each publishes its
//                  scores with write-through stores and takes the row's ticket, and the one that
//                  finishes last selects and attends.  For small problems, where launches and
//                  dependent round trips are the time.
//   list_kernel    selection and attention after a scoring launch that leaves such lists in memory (row_list.h; bf16).  One
//                  workgroup per row, or several, each of which finds the same set and attends over an equal share
//                  of it.
//   row_kernel     selection and attention of a row whose scores lie in S (after score_kernel without a
//                  histogram), one workgroup per row: float32 problems that fill the machine.
//
// See plan_step and plan_list for where the lines lie; beyond them fused.hip splits a row over many workgroups.
#include <type_traits>

#include "mfma_tile.h"
#include "row_list.h"
#include "score_common.h"
#include "select_common.h"

namespace fasa {

constexpr int kStepNT = 512;                 // threads per workgroup of step_kernel
constexpr int kRowNT = 1024;                 // threads per workgroup of row_kernel
constexpr int kListNT = 512;                 // threads per workgroup of list_kernel
constexpr int kListMaxWgs = 64;              // workgroups per row of it
constexpr int kListMaxShare = 2048;          // most tokens that one of them attends over
constexpr int kListPerThread = 8;            // places of a row's list, per thread
constexpr int kStepMaxCtx = 16 * kStepNT;    // longest row of step_kernel: what its last workgroup's registers hold

struct StepArgs {
  const void* q;
  void* K;
  void* V;
  void* Kp;
  const int32_t* fc_idx;
  const void* k_new;       // readable even when nothing is appended (then q)
  const void* v_new;
  float* S;
  int32_t* T;
  float* O;
  RowCtl* ctl;
  const int32_t* n_ctx_seq;
  const int32_t* budget_seq;
  long long sb, sh, sn;    // K/V element strides
  PageMap pm;
  int rows, nslices, G, Hkv, F, N_max, n_cap, budget_max, t_pitch, append, pairing;
  uint32_t m_slices, m_hkv;  // div_magic of nslices (list_kernel: of nwgs) and Hkv
  float scale_log2e;
  // list_kernel: the workgroups' partials [row][nwgs]
  float* part_acc;
  float* part_ml;
};

// LDS of selection and attention; phases that never overlap share storage.
// LIST: places of a list in LDS; MOST: most selected tokens of the workgroup.
template <int NT, int GM, int LIST = kListPerThread * NT, int MOST = kStepMaxBudget>
struct RowLds {
  static constexpr int kThreads = NT;
  static constexpr int kWaves = NT / kWave;
  static constexpr int kList = LIST, kMost = MOST;
  static constexpr int kLoads = 4;                           // of segments that are read again
  static constexpr bool kWideTies = LIST == 1;
  static constexpr int kExtraPerWave = LIST == 1 ? 896 : 1;  // (two workgroups still share a compute unit's LDS)
  union {
    float o[kWaves][kMaxGroup][kHeadDim];                    // weighted V per wave
    uint4 k[kWaves][kTurnWords];                             // a tile's K rows, by the wave whose o lies there later
    uint2 list[kList];                                       // scores at or above the cut: (score bits, token)
    uint2 extra[kWaves * kExtraPerWave];                     // entries of lists that no thread holds
    unsigned char merge[8192 + GM * kListMaxWgs * 4];        // combine_row: partitions, then weights
  };
  union {
    uint32_t hist[kSelBins];
    uint32_t sample[kSample];
  };
  uint2 cand[kSelCand];
  uint32_t cand_at[kSelCand];                                // where their rows lie
  uint32_t ssort[kSample];                                   // keys of the sample, largest first
  __align__(16) uint32_t wl[MOST + 16 + kWave];   // selected tokens, then what the gather reads for them; a word per lane
  float m[kWaves][GM], l[kWaves][GM];
  float scs[kWaves][16];
  uint32_t wtot[kWaves], wtot2[kWaves];
  uint32_t thr[4];
  uint2 lim[LIST == 1 ? NT : 1];                             // where lists of segments begin, and which (list_kernel)
  uint32_t n_list, n_cnd;
  int p_new;                                                 // place of the appended row in wl, or -1
  HeldFound found;
  __device__ __forceinline__ void put(int place, uint32_t tok) { wl[place] = tok; }
  // (no branch: a lane that has nothing to put writes a word of its own)
  __device__ __forceinline__ void put_if(bool yes, int place, uint32_t tok) { wl[yes ? place : kMost + 16 + lane_id()] = tok; }
};

// 16-byte store that goes through to the coherence point (see st_agent), counted by the compiler.  The
// buffer is the same in all lanes (else every lane would become a store of its own).
__device__ __forceinline__ void st_agent_f4(__amdgpu_buffer_rsrc_t rs, uint32_t byte_offset, float4 v) {
  const u32x4_t w = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
  __builtin_amdgcn_raw_buffer_store_b128(w, rs, (int)byte_offset, 0, kCachePolicySc1);
}

// Selection of a row inside its list of M <= EPT * NT scores in LDS (score bits, token) that reach the cut kcut (0: everything does)
template <int EPT, typename Lds>
__device__ __forceinline__ bool select_list(Lds& sm, int M, uint32_t kcut, uint32_t ktop, int bsel, const float* srow, int N) {
  uint32_t key[EPT], tok[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int i = k * Lds::kThreads + threadIdx.x;
    const uint2 e = sm.list[i];                               // (beyond M: whatever it holds)
    key[k] = i < M ? score_key(__uint_as_float(e.x)) : 0u;
    tok[k] = e.y;
  }
  return select_entries<EPT>(sm, key, tok, max(kcut, 1u), kcut ? first_shift(kcut, ktop) : 22, bsel, srow, N);
}

// Selection of a row inside its list, or - should it be shorter than B or longer than its room, because the sample misled or
// thousands of scores are equal - among all of the row's scores in memory.
template <typename Lds>
__device__ __forceinline__ void select_row(Lds& sm, int M, uint32_t kcut, uint32_t ktop, int bsel, const float* srow, int N) {
  if (M >= bsel && M <= Lds::kList) {
    // (Instances for short lists, which nearly all are: 128 float32 rows of 16384, 4 heads, B = 256: 70.6 -> 69.7 us)
    const bool ok = M <= 2 * Lds::kThreads ? select_list<2>(sm, M, kcut, ktop, bsel, srow, N)
                    : M <= 4 * Lds::kThreads ? select_list<4>(sm, M, kcut, ktop, bsel, srow, N)
                                             : select_list<kListPerThread>(sm, M, kcut, ktop, bsel, srow, N);
    if (ok) return;
  }
  publish_barrier();                                          // this workgroup's own scores are in memory
  row_select<true>(sm, bsel, srow, N, 0, bsel);
}

// Attention over the tokens in sm.wl[0 .. cnt): T is written, and every wave leaves its (max, sum, weighted V)
// in LDS (a block barrier ago when this returns).  p0: place of the first of them in T; with_q: a tile that has the queries.  Wave w takes 16-row tiles w, w + waves, ... (bf16:
// mfma_tile.h; float32: vector ALUs).
// ready: how many of the tokens are known already; late(put), called by all threads if that is fewer than cnt, calls put(i, c) for the others, each
// of which is one of the n_cand tokens sm.cand[c].y.  Tiles of known tokens alone are requested before that.
struct NothingLate { template <typename Put> __device__ void operator()(Put&&) const {} };
// STREAM: V's rows are read non-temporal (not K's: a wave's load of those is half a line of each of 16 rows).
template <typename ET, int GM, bool STREAM = false, typename Lds, typename Late = NothingLate>
__device__ __forceinline__ void row_attend(const StepArgs& a, Lds& sm, int row, int b, int h, int G, int cnt, int n_app,
                                           int p0 = 0, const MfmaTile<GM>* with_q = nullptr, int ready = 1 << 30, int n_cand = 0,
                                           Late&& late = Late()) {
  constexpr bool kLate = !std::is_same<typename std::decay<Late>::type, NothingLate>::value;
  static_assert(!kLate || sizeof(ET) == 2, "float32 steps know all tokens");
  constexpr int D = kHeadDim;
  constexpr int NT = Lds::kThreads, NWV = Lds::kWaves;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const ET* q = (const ET*)a.q + (size_t)row * G * D;
  // T, and what the gather reads: the row's element offset / 8, padded to whole tiles with the last row
  const bool paged = a.pm.table != nullptr;
  int32_t* trow = a.T + (size_t)row * a.t_pitch + p0;
  auto place_of = [&](int n) {
    return (uint32_t)((unsigned long long)kv_row_offset(a.pm, paged ? b : 0, n, a.sb, a.sn) >> 3);
  };
  const int n_known = kLate ? min(ready, cnt) : cnt;
  int t_at = n_known, t_tok = 0;
  if constexpr (kLate) {
    // Where their rows lie, by the wave that attends over them: no barrier.  T can wait for the first tile's requests.  A last tile is filled up
    // with the last row, whose values are in use: another's may be anything, and NaNs stay NaNs at weight 0.  The candidates of a paged cache
    // as well: a look-up behind the rows' loads would wait for them.
    const int end = ready >= cnt ? (cnt + 15) & ~15 : n_known;
    for (int i0 = wave * 16; i0 < end; i0 += 64 * NWV) {
      if (t_at < n_known) trow[t_at] = t_tok;
      t_at = i0 + (lane >> 4) * (16 * NWV) + (lane & 15);
      if (t_at < end) {
        t_tok = (int)sm.wl[min(t_at, n_known - 1)];           // (of the same tile: not a place yet)
        sm.wl[t_at] = place_of(t_tok);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (paged && ready < cnt)
      for (int i = t; i < n_cand; i += NT) sm.cand_at[i] = place_of((int)sm.cand[i].y);
  } else {
    for (int i = t; i < cnt; i += NT) {
      const int n = (int)sm.wl[i];
      trow[i] = n;
      if (n == n_app) sm.p_new = i;
      const uint32_t e = place_of(n);
      sm.wl[i] = e;
      if (i == cnt - 1)
        for (int j = cnt; j & 15; ++j) sm.wl[j] = e;
    }
    __syncthreads();
  }
  const ET* Kb = (const ET*)a.K + (paged ? 0 : b * a.sb) + h * a.sh;
  const ET* Vb = (const ET*)a.V + (paged ? 0 : b * a.sb) + h * a.sh;
  const ET* kn = (const ET*)a.k_new + (size_t)row * D;
  const ET* vn = (const ET*)a.v_new + (size_t)row * D;
  // the appended row is read from k_new / v_new: its place in the caches is being written in this launch
  const int p_new = sm.p_new;
  if constexpr (sizeof(ET) == 2) {
    const int lo = lane & 15, hi = lane >> 4;
    MfmaTile<GM> tile;
    if (with_q) tile = *with_q;
    // (The appended row by its distance: with a choice of pointers the compiler no longer knew them for global ones, and a flat load makes every wait
    // one for all loads and all of LDS.  8 rows of 32768, B = 2048: 16.9 -> 16.6 us; 32 of 32905, 7 heads: 45.3 -> 44.9; 8 of 1531, B = 192: 10.70 -> 10.60.)
    const long long k_app = ((const char*)kn - (const char*)Kb) / 2, v_app = ((const char*)vn - (const char*)Vb) / 2;
    // (K's rows whole, as V's: turn_k.  us per step: 8 rows of 1531, B = 192: 9.43 -> 9.19; 128 of 16384, 256: 34.87 -> 34.70; 32 of 32905, 7 heads,
    // 6219: 39.60 -> 39.46, with K read non-temporal as well 40.4.)
    auto rows_of = [&](int j0, long long app, long long (&o)[4]) {
      const uint4 e4 = *reinterpret_cast<const uint4*>(&sm.wl[j0 + 4 * hi]);
      const uint32_t e[4] = {e4.x, e4.y, e4.z, e4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = (long long)((size_t)e[i] << 3);
      if constexpr (!kLate) {
        if (p_new >= j0 && p_new < j0 + 16) {                 // (wave-uniform test)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = p_new == j0 + 4 * hi + i ? app : o[i];
        }
      }
    };
    auto load_k = [&](TileKV<uint16_t>& kv, int j0) {
      long long o[4];
      rows_of(j0, k_app, o);
#pragma unroll
      for (int i = 0; i < 4; ++i) kv.kc[i] = *reinterpret_cast<const uint4*>(Kb + o[i] + 8 * lo);
    };
    auto load_v = [&](TileKV<uint16_t>& kv, int j0) {
      long long o[4];
      rows_of(j0, v_app, o);
#pragma unroll
      for (int i = 0; i < 4; ++i) kv.template load_v<STREAM>(i, Vb + o[i] + 8 * lo);
    };
    const int jw = wave * 16;
    TileKV<uint16_t> kv;
    if constexpr (kLate) {
      const bool early = ready >= cnt || jw + 16 <= ready;
      if (early && jw < cnt) {
        load_k(kv, jw);
        load_v(kv, jw);
      }
      if (t_at < n_known) trow[t_at] = t_tok;
      if (ready < cnt) {
        if (paged) __syncthreads();                           // (cand_at)
        late([&](int i, int c) {
          const int n = (int)sm.cand[c].y;
          const uint32_t e = paged ? sm.cand_at[c] : place_of(n);
          trow[i] = n;
          sm.wl[i] = e;
          if (i == cnt - 1)
            for (int j = cnt; j & 15; ++j) sm.wl[j] = e;
        });
        __syncthreads();
        if (!early && jw < cnt) {
          load_k(kv, jw);
          load_v(kv, jw);
        }
      }
    }
    tile.reset();
    if (jw < cnt) {
      const int n_tiles = (cnt - jw + 16 * NWV - 1) / (16 * NWV);
      float sv[4];
      if (!with_q) tile.load_q(q, lo, hi, G);
      if constexpr (!kLate) {
        load_k(kv, jw);
        load_v(kv, jw);
      }
      for (int i = 0; i + 1 < n_tiles; ++i) {
        const int j0 = jw + 16 * NWV * i;
        turn_k(kv.kc, sm.k[wave], lo, hi);
        tile.logits(kv, a.scale_log2e, sv);
        // the next tile's K runs under this tile's P.V and its V under the next logits; the scheduler is
        // kept from moving any of it (it would need 60 registers more than a wave has here, and spill)
        __builtin_amdgcn_sched_barrier(0);
        load_k(kv, j0 + 16 * NWV);
        __builtin_amdgcn_sched_barrier(0);
        tile.accumulate_full(kv, sv, &sm.scs[wave][0], lo, hi);
        __builtin_amdgcn_sched_barrier(0);
        load_v(kv, j0 + 16 * NWV);
        __builtin_amdgcn_sched_barrier(0);
      }
      const int j0 = jw + 16 * NWV * (n_tiles - 1);
      turn_k(kv.kc, sm.k[wave], lo, hi);
      tile.logits(kv, a.scale_log2e, sv);
      bool valid[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) valid[e] = j0 + 4 * hi + e < cnt;
      tile.accumulate(kv, sv, valid, &sm.scs[wave][0], lo, hi);
    }
    tile.finish(&sm.m[wave][0], &sm.l[wave][0], &sm.o[wave][0][0], lo, hi, G);
  } else {
    // float32: a 16-lane group per row, lane c owning head dims 8c .. 8c+7
    const int c = lane & 15, gr = lane >> 4;
    constexpr int U = 2;                                      // rows in flight per group and batch
    constexpr int GH = GM < 4 ? GM : 4;                       // query heads per pass over the rows (registers)
    for (int g0 = 0; g0 < G; g0 += GH) {
      float qr[GH][8], oc[GH][8], mr[GH], lr[GH];
#pragma unroll
      for (int g = 0; g < GH; ++g) {
        const ET* qp = q + (size_t)min(g0 + g, G - 1) * D + 8 * c;
#pragma unroll
        for (int k = 0; k < 8; ++k) { qr[g][k] = qp[k] * a.scale_log2e; oc[g][k] = 0.f; }
        mr[g] = kNegBig;
        lr[g] = 0.f;
      }
      for (int j0 = wave * 4 * U; j0 < cnt; j0 += 4 * U * NWV) {
        float4 kr[U][2], vr[U][2];
        bool valid[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int j = j0 + 4 * u + gr;
          valid[u] = j < cnt;
          const uint32_t e = sm.wl[min(j, cnt - 1)];
          const float4* kp4 = reinterpret_cast<const float4*>((j == p_new ? kn : Kb + ((size_t)e << 3)) + 8 * c);
          const float4* vp4 = reinterpret_cast<const float4*>((j == p_new ? vn : Vb + ((size_t)e << 3)) + 8 * c);
          kr[u][0] = kp4[0]; kr[u][1] = kp4[1];
          vr[u][0] = vp4[0]; vr[u][1] = vp4[1];
        }
#pragma unroll
        for (int g = 0; g < GH; ++g) {
          float s[U], mx = mr[g];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float kf[8] = {kr[u][0].x, kr[u][0].y, kr[u][0].z, kr[u][0].w, kr[u][1].x, kr[u][1].y, kr[u][1].z, kr[u][1].w};
            float d = 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) d = fmaf(qr[g][k], kf[k], d);
            s[u] = row16_sum(d);
            mx = valid[u] ? fmaxf(mx, s[u]) : mx;
          }
          const float sc = exp2f(mr[g] - mx);
          mr[g] = mx;
          lr[g] *= sc;
#pragma unroll
          for (int k = 0; k < 8; ++k) oc[g][k] *= sc;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float pv = valid[u] ? exp2f(s[u] - mx) : 0.f;
            const float vf[8] = {vr[u][0].x, vr[u][0].y, vr[u][0].z, vr[u][0].w, vr[u][1].x, vr[u][1].y, vr[u][1].z, vr[u][1].w};
            lr[g] += pv;
#pragma unroll
            for (int k = 0; k < 8; ++k) oc[g][k] = fmaf(pv, vf[k], oc[g][k]);
          }
        }
      }
      // the four groups of the wave hold the same head dims
#pragma unroll
      for (int g = 0; g < GH; ++g) {
        const float mn = xor32_max(xor16_max(mr[g])), sc = exp2f(mr[g] - mn);
        lr[g] = xor32_sum(xor16_sum(lr[g] * sc));
#pragma unroll
        for (int k = 0; k < 8; ++k) oc[g][k] = xor32_sum(xor16_sum(oc[g][k] * sc));
        if (gr == 0 && g0 + g < G) {
          if (c == 0) { sm.m[wave][g0 + g] = mn; sm.l[wave][g0 + g] = lr[g]; }
          float4* o4 = reinterpret_cast<float4*>(&sm.o[wave][g0 + g][8 * c]);
          o4[0] = make_float4(oc[g][0], oc[g][1], oc[g][2], oc[g][3]);
          o4[1] = make_float4(oc[g][4], oc[g][5], oc[g][6], oc[g][7]);
        }
      }
    }
  }
  __syncthreads();
}

// Sum over the waves: thread (query head g, 4 head dims d4) gets max, sum of weights, weighted V.
template <typename Lds>
__device__ __forceinline__ void wave_totals(const Lds& sm, int g, int d4, float& mn, float& ls, float4& o) {
  mn = sm.m[0][g];
#pragma unroll
  for (int i = 1; i < Lds::kWaves; ++i) mn = fmaxf(mn, sm.m[i][g]);
  ls = 0.f;
  o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < Lds::kWaves; ++i) {
    const float sc = exp2f(sm.m[i][g] - mn);
    ls = fmaf(sm.l[i][g], sc, ls);
    const float4 x = *reinterpret_cast<const float4*>(&sm.o[i][g][4 * d4]);
    o.x = fmaf(x.x, sc, o.x); o.y = fmaf(x.y, sc, o.y); o.z = fmaf(x.z, sc, o.z); o.w = fmaf(x.w, sc, o.w);
  }
}
template <typename Lds>
__device__ __forceinline__ void write_output(const StepArgs& a, const Lds& sm, int row, int G) {
  constexpr int D = kHeadDim;
  const int t = threadIdx.x;
  if (t < G * (D / 4)) {
    const int g = t / (D / 4), d4 = t % (D / 4);
    float mn, ls;
    float4 o;
    wave_totals(sm, g, d4, mn, ls, o);
    const float inv = 1.0f / ls;
    *reinterpret_cast<float4*>(a.O + ((size_t)row * G + g) * D + 4 * d4) =
        make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
  }
}

// The list of a row whose scores the caller's threads hold in registers: score(k), k < NV, of token
// token(k, c0) (a NaN where the row has ended).  With more than `resident` tokens in the row they hold one stretch of it at a time, c0 its
// first token, and reload(c0) brings it in.
// 128 scores of the row, evenly spaced (`sval` of thread i < 128), are ranked; the sample_rank-th best is the cut.
// Returns the list's length; kcut, ktop: keys of the cut (0: none) and of the sample's best.
template <int NV, typename Lds, typename Score, typename Token, typename Reload>
__device__ __forceinline__ int make_list(Lds& sm, int N, int bsel, float sval, int resident, Score&& score, Token&& token,
                                         Reload&& reload, uint32_t& kcut, uint32_t& ktop) {
  constexpr int NT = Lds::kThreads;
  const int t = threadIdx.x, lane = t & 63;
  rank_sample<NT, kSample>(sval, sm.sample, sm.ssort, [&]() {
    if (t == 0) { sm.n_list = 0; sm.p_new = -1; sm.thr[2] = 0; }
  });
  for (int i = t; i < kSelBins; i += NT) sm.hist[i] = 0;     // (shares storage with the sample)
  const int r = sample_rank(bsel, N);
  kcut = r > kSample ? 0u : sm.ssort[r - 1];
  ktop = sm.ssort[0];
  const float cut = r > kSample ? -INFINITY : key_score(kcut);
  auto stretch = [&](int c0) {
    unsigned long long m[NV];                                 // per wave: which lanes' k-th score reaches the cut
    uint32_t cnt = 0;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      m[k] = __ballot(score(k) >= cut);
      cnt += (uint32_t)__popcll(m[k]);
    }
    uint32_t base = 0;
    if (lane == 0 && cnt) base = atomicAdd(&sm.n_list, cnt);
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], base));
      if (score(k) >= cut && pos < (uint32_t)Lds::kList) sm.list[pos] = make_uint2(__float_as_uint(score(k)), (uint32_t)token(k, c0));
      base += (uint32_t)__popcll(m[k]);
    }
  };
  for (int c0 = 0; c0 < N; c0 += resident) {
    if (N > resident) reload(c0);
    stretch(c0);
  }
  __syncthreads();
  return (int)sm.n_list;
}

constexpr uint32_t kStepGroup = 15, kStepPairing = 16, kStepAppend = 64, kStepRagged = 128;
struct StepGrid {
  int rows, nslices;
  uint32_t m_slices;
};
// MULTI: rows of several slices (scores handed over through S and a ticket); else one slice per row.  flags: query heads per KV
// head | kStepPairing * pairing | kStepAppend | kStepRagged.
template <typename ET, int NB, int GM, bool MULTI>
__device__ __forceinline__ void step_row(const void* q0, void* Kp0, const int32_t* fc_idx, const void* k_new, const void* v_new,
                                         uint32_t flags, int Hkv, uint32_t m_hkv, int N_max, int n_cap, int F0, const StepGrid& grid,
                                         const StepArgs& a) {
  constexpr int D = kHeadDim;
  constexpr int TPT = ScoreTraits<ET>::TPT;
  constexpr int SL = kStepNT * TPT;
  constexpr int NW = NB == 1 ? 8 : 16;       // planes in flight per thread
  __shared__ union {
    struct {
      float ql[kMaxGroup][kHeadDim];                           // the group's queries
      float2 qs[kHeadDim / 2];
      float2 kpair[kHeadDim / 2];                              // the appended key's listed dims
      uint32_t knew[kHeadDim];                                 // the appended key, as stored
    };
    RowLds<kStepNT, GM> row;
  } sm;
  __shared__ uint32_t ticket;

  int row = blockIdx.x, slice = 0, b, h;
  if constexpr (MULTI) row_slice_of_block(grid.rows, grid.nslices, grid.m_slices, row, slice);
  head_of_row(row, Hkv, m_hkv, b, h);
  const int G = min((int)(flags & kStepGroup), GM), pairing = (int)(flags / kStepPairing % 4);
  const int t = threadIdx.x;
  const int N = flags & kStepRagged ? seq_n_ctx(a.n_ctx_seq, b, N_max) : N_max;
  if (slice * SL >= N) return;                                // beyond this sequence (ragged batches only)
  const int nvalid = (N + SL - 1) / SL;
  const ET* q = (const ET*)q0 + (size_t)row * G * D;

  // ---- scores.  Order of issue as in score_kernel: what the planes do not depend on first, then all
  // plane loads unconditionally, then a wait for the former only ----
  ET qcol[2];                                                 // head dim t mod 128 of query heads t / 128 and + 4
#pragma unroll
  for (int j = 0; j < 2; ++j) qcol[j] = q[(size_t)min((t >> 7) + 4 * j, G - 1) * D + (t & (D - 1))];
  const int F = NB ? NB * 8 : F0, fe = min(t, F - 1);
  const int32_t fci = fc_idx[list_word(pairing, F, h, fe, 0)];
  const int32_t fcj = fc_idx[list_word(pairing, F, h, fe, 1)];
  const ET newkv = ((const ET*)((t & 255) < D ? k_new : v_new))[(size_t)row * D + (t & (D - 1))];
  const int n0 = (slice * kStepNT + t) * TPT;
  const bool active = n0 < N;
  ET* Kp = (ET*)Kp0 + (size_t)row * F * n_cap * 2;
  const ET* p = Kp + (size_t)(active ? n0 : 0) * 2;
  const size_t plane = (size_t)n_cap * 2;
  uint4 w[NW];
#pragma unroll
  for (int u = 0; u < NW; ++u)
    w[u] = *reinterpret_cast<const uint4*>(p + (size_t)(NB ? u : min(u, F - 1)) * plane);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float x;
    if constexpr (sizeof(ET) == 2) x = __uint_as_float((uint32_t)qcol[j] << 16);
    else x = qcol[j];
    sm.ql[(t >> 7) + 4 * j][t & (D - 1)] = x;                 // heads beyond the group: copies, not added
  }
  const int n_app = N - 1;
  const bool append = (flags & kStepAppend) != 0, own_wg = append && n_app / SL == slice;
  if (t < D) {
    if constexpr (sizeof(ET) == 2) sm.knew[t] = (uint32_t)newkv;
    else sm.knew[t] = __float_as_uint(newkv);
  }
  __syncthreads();
  uint32_t pair_x = 0, pair_y = 0;
  if (t < F) {   // sum_g (q_g . k) = (sum_g q_g) . k, g ascending
    const int pr = pair_dims(pairing, fci, fcj);
    float lo = 0.f, hi = 0.f;
#pragma unroll
    for (int g = 0; g < kMaxGroup; ++g) {
      const float x = sm.ql[g][pr & 255], y = sm.ql[g][pr >> 8];
      lo += g < G ? x : 0.f;
      hi += g < G ? y : 0.f;
    }
    sm.qs[t] = make_float2(lo, hi);
    pair_x = sm.knew[pr & 255];
    pair_y = sm.knew[pr >> 8];
    if constexpr (sizeof(ET) == 2) sm.kpair[t] = make_float2(__uint_as_float(pair_x << 16), __uint_as_float(pair_y << 16));
    else sm.kpair[t] = make_float2(__uint_as_float(pair_x), __uint_as_float(pair_y));
  }
  __syncthreads();
  float acc[TPT];
#pragma unroll
  for (int k = 0; k < TPT; ++k) acc[k] = 0.f;
  if constexpr (NB > 0) {
#pragma unroll
    for (int u = 0; u < NB * 8; ++u) {
      const float2 qf = sm.qs[u];
      fma_pairs<ET>(w[u % NW], qf.x, qf.y, acc);
      if (u + NW < NB * 8) w[u % NW] = *reinterpret_cast<const uint4*>(p + (size_t)(u + NW) * plane);
    }
  } else {
    for (int f0 = 0; f0 < F; f0 += NW) {
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        if (f0 + u < F) {
          const float2 qf = sm.qs[f0 + u];
          fma_pairs<ET>(w[u], qf.x, qf.y, acc);
          w[u] = *reinterpret_cast<const uint4*>(p + (size_t)min(f0 + NW + u, F - 1) * plane);
        }
      }
    }
  }
  // the appended token's score comes from the new row itself: the planes did not hold it
  if (own_wg && (n_app - slice * SL) / TPT == t) {
    float s = 0.f;
#pragma unroll 8
    for (int f = 0; f < F; ++f) {
      const float2 qf = sm.qs[f], kf = sm.kpair[f];
      s = fmaf(qf.y, kf.y, fmaf(qf.x, kf.x, s));
    }
#pragma unroll
    for (int k = 0; k < TPT; ++k) acc[k] = n_app % TPT == k ? s : acc[k];
  }
  float* srow = a.S + (size_t)row * n_cap;
  const int bsel = min(seq_bsel(a.budget_seq, b, N, a.budget_max), kStepMaxBudget);
  const __amdgpu_buffer_rsrc_t rs = agent_buffer(srow);
  if (active) {
    float* out = srow + n0;
    if (n0 + TPT <= N) {
      if constexpr (TPT == 4) st_agent_f4(rs, (uint32_t)n0 * 4u, make_float4(acc[0], acc[1], acc[2], acc[3]));
      else st_agent(reinterpret_cast<float2*>(out), make_float2(acc[0], acc[1]));
    } else {
#pragma unroll
      for (int k = 0; k < TPT; ++k)
        if (n0 + k < N) st_agent(out + k, acc[k]);
    }
  }
  if constexpr (MULTI) {
    publish_barrier();
    if (t == 0) ticket = atomicAdd(&a.ctl[row].done_sel, 1u);
  }
  // Alg. 2, UpdateCache: the new row joins K, V and the planes.  Nothing in this launch reads it there
  // (the gather takes it from k_new / v_new), so nothing waits for these stores.
  if (own_wg) {
    if (t < F) {
      if constexpr (sizeof(ET) == 2)
        *reinterpret_cast<uint32_t*>(Kp + ((size_t)t * n_cap + n_app) * 2) = pair_x | (pair_y << 16);
      else
        *reinterpret_cast<uint2*>(Kp + ((size_t)t * n_cap + n_app) * 2) = make_uint2(pair_x, pair_y);
    }
    if (t < 2 * D) {
      ET* dst = (ET*)(t < D ? a.K : a.V) + kv_row_offset(a.pm, b, n_app, a.sb, a.sn) + h * a.sh + (t & (D - 1));
      *dst = newkv;
    }
  }
  bool done;
  if constexpr (MULTI) {
    __syncthreads();
    if (ticket != (uint32_t)nvalid - 1u) return;
    if (t == 0) a.ctl[row].done_sel = 0;                      // clean for the next call
    if (t == 0) sm.row.p_new = -1;
  } else {
    __syncthreads();                                          // (all have read the queries' sums: shared storage)
    if (t == 0) sm.row.p_new = -1;
  }
  if constexpr (MULTI) {
    // (the row is readable in 16-byte pieces: S is n_cap long, a multiple of 64)
    auto held = [&](auto pieces) {
      constexpr int CH = decltype(pieces)::value;
      float v[4 * CH];
#pragma unroll
      for (int it = 0; it < CH; ++it) {
        const int n = (it * kStepNT + t) * 4;
        const uint4 x = agent_load_u128(rs, (uint32_t)(n < N ? n : 0) * 4u);
        v[4 * it] = n < N ? __uint_as_float(x.x) : NAN; v[4 * it + 1] = n + 1 < N ? __uint_as_float(x.y) : NAN;
        v[4 * it + 2] = n + 2 < N ? __uint_as_float(x.z) : NAN; v[4 * it + 3] = n + 3 < N ? __uint_as_float(x.w) : NAN;
      }
      const auto token = [&](int k) { return ((k >> 2) * kStepNT + t) * 4 + (k & 3); };
      if (select_held(sm.row, v, token, bsel, srow, N)) return true;
      return select_held_again(sm.row, v, token, bsel, srow, N);
    };
    constexpr int CH = kStepMaxCtx / (4 * kStepNT);
    done = N <= kStepMaxCtx / 2 ? held(std::integral_constant<int, CH / 2>{}) : held(std::integral_constant<int, CH>{});
  } else {
#pragma unroll
    for (int k = 0; k < TPT; ++k) acc[k] = n0 + k < N ? acc[k] : NAN;
    const auto token = [&](int k) { return n0 + k; };
    done = select_held(sm.row, acc, token, bsel, srow, N);
    if (!done) done = select_held_again(sm.row, acc, token, bsel, srow, N);
  }
  if (!done) {
    publish_barrier();                                        // this workgroup's own scores are in memory
    row_select<true>(sm.row, bsel, srow, N, 0, bsel);
  }
  row_attend<ET, GM>(a, sm.row, row, b, h, G, bsel, append ? n_app : -1);
  write_output(a, sm.row, row, G);
}

// What the first loads depend on comes first and one by one: sixteen words of such arguments are in registers when a kernel starts.
template <typename ET, int NB, int GM>
__global__ __launch_bounds__(kStepNT, 4) void step_kernel(const void* q, void* Kp, const int32_t* fc_idx, const void* k_new, const void* v_new,
                                                          uint32_t flags, int Hkv, uint32_t m_hkv, int N_max, int n_cap, int F,
                                                          const StepArgs a) {
  step_row<ET, NB, GM, false>(q, Kp, fc_idx, k_new, v_new, flags, Hkv, m_hkv, N_max, n_cap, F, StepGrid{}, a);
}
// (1 float32 row of 4096 with k_new and v_new ahead of the rest, as above: 11.65 us, like this 11.24)
template <typename ET, int NB, int GM>
__global__ __launch_bounds__(kStepNT, 4) void step_multi_kernel(const void* q, void* Kp, const int32_t* fc_idx, uint32_t flags, int Hkv,
                                                                uint32_t m_hkv, int N_max, int n_cap, int rows, int nslices,
                                                                uint32_t m_slices, int F, const void* k_new, const void* v_new,
                                                                const StepArgs a) {
  step_row<ET, NB, GM, true>(q, Kp, fc_idx, k_new, v_new, flags, Hkv, m_hkv, N_max, n_cap, F, StepGrid{rows, nslices, m_slices}, a);
}

// One workgroup per row; the scores lie in S (an earlier launch).
template <int GM>
__global__ __launch_bounds__(kRowNT) void row_kernel(const StepArgs a) {
  using ET = float;
  __shared__ RowLds<kRowNT, GM> sm;
  const int row = blockIdx.x;
  int b, h;
  head_of_row(row, a.Hkv, a.m_hkv, b, h);
  const int G = min(a.G, GM);
  const int t = threadIdx.x;
  const int N = seq_n_ctx(a.n_ctx_seq, b, a.N_max);
  const int bsel = min(seq_bsel(a.budget_seq, b, N, a.budget_max), kStepMaxBudget);
  const float* srow = a.S + (size_t)row * a.n_cap;
  const float sval = srow[(int)(((long long)(t & (kSample - 1)) * N) >> 7)];
  constexpr int CH = 4;
  float v[4 * CH];
  auto load_scores = [&](int c0) {
#pragma unroll
    for (int it = 0; it < CH; ++it) {
      const int n = c0 + (it * kRowNT + t) * 4;
      const float4 x = *reinterpret_cast<const float4*>(srow + (n < N ? n : 0));
      v[4 * it] = n < N ? x.x : NAN; v[4 * it + 1] = n + 1 < N ? x.y : NAN;
      v[4 * it + 2] = n + 2 < N ? x.z : NAN; v[4 * it + 3] = n + 3 < N ? x.w : NAN;
    }
  };
  constexpr int R = CH * kRowNT * 4;
  if (N <= R) load_scores(0);
  uint32_t kcut, ktop;
  const int M = make_list<4 * CH>(sm, N, bsel, sval, R, [&](int k) { return v[k]; },
                                         [&](int k, int c0) { return c0 + ((k >> 2) * kRowNT + t) * 4 + (k & 3); }, load_scores, kcut, ktop);
  select_row(sm, M, kcut, ktop, bsel, srow, N);
  row_attend<ET, GM>(a, sm, row, b, h, G, bsel, -1);
  write_output(a, sm, row, G);
}

// nwgs workgroups per row; the scores lie in S, the lists of the largest in `list` (score_list_kernel).  Every workgroup of a
// row finds the row's set, out of the same lists and so in the same order, and attends over its share of it: nothing about
// the selection is left open for the workgroup that merges, and all gather the same number of rows (fused.hip's slices
// differ by 14 %, and leave a threshold bin to resolve at the end).  A chain of round trips and of the instructions between them.
// The candidates of the threshold bin are ranked by the one or two workgroups whose shares end in it, while the rows of the
// tokens already known are under way.  us per step, lists of 1024 tokens by a cut of a sample of the row, and candidates ranked by all
// workgroups ahead of the gather / like this: 8 rows of 32768, 4 heads, B = 2048: 17.8 / 16.5; 32 rows, 7 heads, B = 6219: 49.9 / 44.9;
// 8 rows of 131072, F = 32, B = 1024: 40.6 / 36.9; 128 rows of 16384, B = 256: 41.3 / 37.7; 64 rows of 126490, 7 heads, B = 6250 (which had
// the split form): 57.3 / 43.9; 3 rows of 96425, 4 heads, B = 3490: 26.4 / 19.4; 2 rows of 6987, F = 32, B = 911: 15.9 / 15.7; paged, 32
// sequences' rows of 1600 - 6423, B = 66: 13.9 / 14.2.
// (What the lists' loads depend on comes first and one by one: such arguments are in registers when a kernel starts.  places: of a row's list;
// negative where sequences have lengths and budgets of their own, which N_max and budget bound; share_max: tokens of a workgroup, whole tiles.)
// STREAM: rows of kStreamBytes and more.  32 rows of 32905, 7 heads, 6219 (102 MB of them), three sets of buffers: 41.2 -> 40.1 us per step, ten: 45.0 -> 43.7, K's
// rows as well: 42.5; half as much of 32 rows of 32768, 3000: 30.5 / 30.7.
template <int G, int Q, bool STREAM>
__global__ __launch_bounds__(kListNT, 2) void list_kernel(uint2* lists, uint2* lims, int rows, int nwgs, uint32_t m_wgs, int N_max, int n_cap,
                                                          int places, int budget, int share_max, int Hkv, uint32_t m_hkv, int pitch,
                                                          const StepArgs a) {
  using ET = uint16_t;
  constexpr int D = kHeadDim;
  __shared__ RowLds<kListNT, G, 1, kListMaxShare> sm;
  __shared__ float red[G];
  __shared__ uint32_t ticket;
  int row, wg, b, h;
  row_slice_of_block(rows, nwgs, m_wgs, row, wg);
  head_of_row(row, Hkv, m_hkv, b, h);
  const int t = threadIdx.x, lane = t & 63;
  ListRow list = ListRow::at(lists, lims, row, n_cap, abs(places), pitch);
  ListHeld<false, kListNT, Q> held;
  held.request(list, N_max, abs(places));
  int N = N_max, bsel = budget, share = share_max;
  if (places < 0) {
    N = seq_n_ctx(a.n_ctx_seq, b, N_max);
    bsel = seq_bsel(a.budget_seq, b, N, budget);
    list.pitch = list_pitch(-places, bsel, N);
    share = ((int)fast_div((uint32_t)(bsel + nwgs - 1), (uint32_t)nwgs, m_wgs) + 15) & ~15;
  }
  const int p0 = wg * share, p1 = min(bsel, p0 + share);
  if (p0 >= bsel) return;
  FASA_T_DECL(8);
  FASA_T(0);
  const float* srow = a.S + (size_t)row * n_cap;
  MfmaTile<G> tile;
  if (t == 0) sm.p_new = -1;
  const ListSet set = select_listed<false, Q>(sm, list, held, bsel, srow, N, p0, p1);
  tile.load_q((const ET*)a.q + (size_t)row * G * D, lane & 15, lane >> 4);
  int ready = set.n_above - p0;
  if (!set.usable) {
    row_select<false>(sm, bsel, srow, N, p0, p1, set.klo, set.ktop);
    ready = p1 - p0;
  } else if (set.n_cand > kSelCand && ready < p1 - p0) {       // ties that no list of candidates holds
    resolve_threshold(sm, set.klo, bsel, set.need, set.n_cand, srow, N, p0, p1);
    ready = p1 - p0;
  }
  FASA_T(1);
  // the candidates are ranked while the rows of the others are under way
  row_attend<ET, G, STREAM>(a, sm, row, b, h, G, p1 - p0, -1, p0, &tile, ready, set.n_cand, [&](auto&& put) {
    constexpr int P = kListNT / kSelCand;
    if ((t & ~(kWave - 1)) / P < set.n_cand) {                // (the waves that have any)
      const int ci = t / P;
      const int rank = rank_in_list<P>(sm.cand, set.n_cand, ci), p = set.n_above + rank;
      if (t % P == 0 && ci < set.n_cand && rank < set.need && p >= p0 && p < p1) put(p - p0, ci);
    }
  });
  FASA_T(2);
  if (wg == 0 && t == 0) *reinterpret_cast<uint2*>(&a.ctl[row].list_cut) = make_uint2(set.from, set.how);   // (here: what waits for a load would wait for a store ahead of it too)
  if (share >= bsel) {
    write_output(a, sm, row, G);
    return;
  }
  const size_t pbase = ((size_t)row * nwgs + wg) * G;
  if (t < G * (D / 4)) {
    const int g = t / (D / 4), d4 = t % (D / 4);
    float mn, ls;
    float4 o;
    wave_totals(sm, g, d4, mn, ls, o);
    float2* pa = reinterpret_cast<float2*>(a.part_acc + (pbase + g) * D + 4 * d4);
    st_agent(pa, make_float2(o.x, o.y));
    st_agent(pa + 1, make_float2(o.z, o.w));
    if (d4 == 0) st_agent(reinterpret_cast<float2*>(a.part_ml + (pbase + g) * 2), make_float2(mn, ls));
  }
  FASA_T(3);
  publish_barrier();
  if (t == 0) ticket = atomicAdd(&a.ctl[row].done_att, 1u);
  const int nvalid = (bsel + share - 1) / share;              // (under the ticket's round trip)
  __syncthreads();
  FASA_T(4);
  FASA_T_PRINT(t == 0 && row == 0 && (wg == 0 || ticket == (uint32_t)nvalid - 1u),
               "list wg %d: select %llu attend %llu partial %llu publish+ticket %llu (x10ns)\n", wg, FASA_T_D(1, 0),
               FASA_T_D(2, 1), FASA_T_D(3, 2), FASA_T_D(4, 3));
  if (ticket != (uint32_t)nvalid - 1u) return;
  if (t == 0) a.ctl[row].done_att = 0;                        // clean for the next call
  combine_row<G, NothingUnderLoads, 16, kListNT, kListMaxWgs>(a.part_acc, a.part_ml, a.O, row, nvalid, nwgs,
                                                              reinterpret_cast<float*>(sm.merge + 8192), red,
                                                              reinterpret_cast<float*>(sm.merge));
}

// ---------------------------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------------------------
// Where the row form is the faster one after the scores of a float32 cache (a bf16 cache's rows have lists).  It pays where the workgroups of the split form (fused.hip; two
// per compute unit, at most 4096 tokens each) no longer fit at once, and while reading the scores, not
// gathering on one compute unit, is what a row takes: the line in B falls with rows * N.
static bool row_form(const fasa_shape& s, long long rows, int bsel) {
  const long long n = s.n_ctx, cells = rows * n;
  if (rows <= 64 && rows * ((n + 4095) / 4096) <= 2 * kAssumedCUs) return false;
  // A row whose list overflows is read again from memory several times over, and holds up the launch: its expected length
  // plus four standard deviations has to fit.  64 rows of 65536, us (fused.hip / row form): B = 64: 76.6 / 68.1, B = 512:
  // 79.4 / 99.0; 40 rows of 100000, B = 512: 79 / 153
  const float r = (float)sample_rank(bsel, s.n_ctx);
  if ((r + 4.f * sqrtf(r)) * (float)n > (float)(kSample * kListPerThread * kRowNT)) return false;
  const bool few = bsel * 2048ll <= cells;
  // 1 head.  N = 4096, B = 64: 64 rows 20.5 / 20.8, 80: 23.5 / 22.6; B = 512: 128 rows 40.3 / 41.7; 1024 rows, B = 200:
  // 164 / 170.  N = 8192, B = 256: 80 rows 34.3 / 33.8, 96: 38.3 / 37.3; B = 512: 96 rows 43.5 / 44.9.  N = 16384, B = 256:
  // 128 rows 72.8 / 67.5; 64 rows of 33000, B = 512: 81.6 / 76.6
  const int group = s.n_q_heads / s.n_kv_heads;
  if (group == 1) return (n >= 5120 || rows <= kAssumedCUs) && few;
  // up to 4 heads (the vector ALUs attend there).  2 heads, B = 256: 128 rows of 8192 46.7 / 47.0, of 16384 72.5 / 70.4; 4 heads,
  // B = 256: 128 rows of 8192 46.4 / 47.5, 256: 77.8 / 74.6; 96 rows of 16384 58.8 / 59.1, 128: 72.4 / 70.9; 64 rows of 33000,
  // B = 512: 80.6 / 79.4, 48 of 50000: 85.4 / 88.1.  8 heads, 128 rows of 16384: 75.7 / 84.3
  return rows >= 64 && n >= 8192 && cells > 3 << 19 && bsel <= 512 && group <= 4;
}

StepForm plan_step(const fasa_shape& s, const PageMap& pm) {
  const int bsel = s.budget < s.n_ctx ? s.budget : s.n_ctx;
  if (bsel > kStepMaxBudget) return kStepNone;
  // what the gather reads is a 32-bit offset in units of 8 elements
  const long long most = pm.table ? (long long)pm.n_pool * s.kv_stride_b + (1ll << pm.shift) * s.kv_stride_n
                                  : (long long)s.n_ctx * s.kv_stride_n;
  if ((most >> 3) >= 0xfffffff0ll) return kStepNone;
  // Lines of the one-launch form, measured over 1 .. 512 rows, 1k .. 64k tokens, 64 .. 1024 selected, us per step.
  // One compute unit gathers about 50 KB per us, which is what ends its reach
  // in B; reading a row's scores back is what ends it in N.
  const long long rows = (long long)s.batch * s.n_kv_heads;
  const int per = kStepNT * (s.dtype == FASA_BF16 ? 4 : 2);
  const long long ns = (s.n_ctx + per - 1) / per;
  if (s.dtype == FASA_BF16) {
    // one slice, against lists (list_kernel), one launch / lists: 8 rows of 2048, B = 64: 8.1 / 11.05, 512: 11.35 / 13.45, 1000: 14.75 / 14.45; 128 rows, 256: 12.05 / 14.75;
    // 512 rows, 64: 19.0 / 26.0, 512: 45.2 / 49.9
    if (ns == 1) return kStepOne;
    // Several slices, where the lists of a scoring launch do not do better: B = 256, 40 rows of 8192: 14.15 / 15.0, 128 of 4000: 15.3 / 16.65; 8 rows of 6000, B = 40: 10.45 / 11.2, 256:
    // 11.9 / 12.3, 320: 12.3 / 13.4, 256 with F = 32: 13.05 / 13.25; of 4000, 320: 11.5 / 13.4; of 3000, 40: 9.65 / 11.25.  The line was drawn when the one launch selected out of a list
    // of its own.  On its other side today: 8 rows of 8192, 256: 11.85 / 12.4, 32 rows: 13.6 / 14.15; 8 rows of 4000, 400: 12.2 / 13.25, 512: 12.9 / 13.4; of 6000, 512: 13.65 / 13.5.
    return ns <= 4 && rows * ns <= kAssumedCUs && bsel <= 320 && (rows > 32 || ns < 4) ? kStepOne : kStepNone;
  } else {
    // float32, fused.hip / one launch / row_kernel: the vector ALUs attend, in proportion to the query heads, where fused.hip has the matrix cores.  1 head:
    // 1 row of 4096, B = 256: 17.3 / 12.7 / 15.5, 32 rows of 8192, B = 600: 22.2 / 22.1 / 26.3.  4 heads, 8 rows, B = 64:
    // of 1024: 17.1 / 12.9 / 17.2, of 4096: 15.4 / 15.2 / 17.3, 32 rows of 4096: 17.0 / 18.1 / 19.1; 8 heads, 8 rows of
    // 1024, B = 64: 18.1 / 16.5 / 21.5
    const int group = s.n_q_heads / s.n_kv_heads;
    if (ns <= (group == 1 ? 8 : 1) && rows * ns <= kAssumedCUs && bsel * group <= 512) return kStepOne;
  }
  return row_form(s, rows, bsel) ? kStepRow : kStepNone;
}

template <typename ET, int NB, int GM>
static hipError_t launch_step_v(const StepArgs& a, hipStream_t st) {
  const uint32_t flags = (uint32_t)a.G | kStepPairing * (uint32_t)a.pairing | (a.append ? kStepAppend : 0u) |
                         (a.n_ctx_seq || a.budget_seq ? kStepRagged : 0u);
  const dim3 grid(a.rows * a.nslices), block(kStepNT);
  if (a.nslices == 1)
    return launch("fasa_step", step_kernel<ET, NB, GM>, grid, block, st, a.q, a.Kp, a.fc_idx, a.k_new, a.v_new, flags, a.Hkv, a.m_hkv,
                  a.N_max, a.n_cap, a.F, a);
  // float32 rows of several slices: with one query head only (plan_step)
  if constexpr (sizeof(ET) == 2 || GM == 1)
    return launch("fasa_step", step_multi_kernel<ET, NB, GM>, grid, block, st, a.q, a.Kp, a.fc_idx, flags, a.Hkv, a.m_hkv, a.N_max, a.n_cap,
                  a.rows, a.nslices, a.m_slices, a.F, a.k_new, a.v_new, a);
  return hipErrorInvalidValue;
}
// The list lengths in use have an instance each, where no load of the planes stands under a test.  float32, us, with the
// instance for any length -> with its own: 1 row of 1000 tokens, B = 256: F = 8 11.9 -> 10.2, F = 16 12.5 -> 11.0, F = 24 13.4 ->
// 11.7, F = 32 14.3 -> 12.5; of 4096, F = 16: 14.7 -> 13.2; 4 heads, 8 rows of 1000, B = 64, F = 16: 13.9 -> 12.4; 8 heads: 17.4 -> 16.0
template <typename ET, int GM>
static hipError_t launch_step_f(const StepArgs& a, hipStream_t st) {
  switch (a.F) {
    case 8: return launch_step_v<ET, 1, GM>(a, st);
    case 16: return launch_step_v<ET, 2, GM>(a, st);
    case 24: return launch_step_v<ET, 3, GM>(a, st);
    case 32: return launch_step_v<ET, 4, GM>(a, st);
    default: return launch_step_v<ET, 0, GM>(a, st);
  }
}
int list_quads(int n, int bsel, int nt, int most) {
  const int nsegs = (n + kListSeg - 1) / kListSeg;
  if (nsegs > kListMaxSegs) return 0;
  const int q = (nsegs * (list_room(bsel, n) / 4) + nt - 1) / nt;
  if (q > most) return 0;
  return q <= 4 ? q : q <= 6 ? 6 : 8;                          // (the instances there are)
}

// Places of a row's list: its segments', or, where sequences have lengths and budgets of their own, all that the threads hold.
int list_places(int n, int bsel, int quads, bool by_sequence) {
  const int nsegs = (n + kListSeg - 1) / kListSeg, held = quads * kListNT * 4;
  if (!by_sequence) return nsegs * list_room(bsel, n);
  return held < nsegs * kListSeg ? held : nsegs * kListSeg;
}

ListPlan plan_list(const fasa_shape& s, const PageMap& pm, int max_splits) {
  ListPlan p{0, 0};
  if (s.dtype != FASA_BF16) return p;                          // (float32 rows are attended on the vector ALUs here)
  const long long most = pm.table ? (long long)pm.n_pool * s.kv_stride_b + (1ll << pm.shift) * s.kv_stride_n
                                  : (long long)s.n_ctx * s.kv_stride_n;
  if ((most >> 3) >= 0xfffffff0ll) return p;
  const int bsel = s.budget < s.n_ctx ? s.budget : s.n_ctx, rows = s.batch * s.n_kv_heads;
  // 32 entries a thread, which is what its registers hold beside the tiles: rows of up to 49000 tokens with 18.9 % of them selected,
  // 67000 with 12.5 %.  us, split form / lists: 32 rows of 20000, 7 heads, B = 8000: 52.5 / 46.8; 8 rows of 22000, 8 heads, 7500: 27.6 / 21.1; of 45000,
  // 4 heads, 9000: 33.4 / 26.1.  With more than a third selected 24: 17400 tokens with half.  That is no line of speed: with 32 on its other
  // side, too, 1 row of 20000, B = 9000: 23.2 / 21.4, 8 rows, 4 heads: 26.5 / 25.1, 2 of 20001, 8 heads: 25.1 / 22.6.  It is where short bf16 rows still take
  // the split form (longer lists, and shares of more than 2048 tokens, take it anyway), whose instances are tested there.
  const int quads = list_quads(s.n_ctx, bsel, kListNT, bsel > s.n_ctx / 3 ? 6 : 8);
  if (!quads) return p;
  // One workgroup up to B = 256: what it gathers (50 KB per us) takes less than a hand-over and a merge, also where that leaves half of the
  // compute units idle.  us with 1 / 2 / 4, 4 heads, of 16384 tokens in caches that the last-level cache holds: 8 rows, B = 128: 11.4 / 13.3 / 13.3, 256:
  // 12.7 / 13.8 / 13.5, 320: 13.0 / 14.2 / 13.7, 512: 14.9 / 15.0 / 13.9; 32 rows, 256: 16.2 / 17.2 / 16.8, 320: 16.9 / 17.9 / 17.3; 64 rows, 256: 21.6 /
  // 22.6 / 22.4; 128 rows, 128: 30.1 / 32.0, 256: 31.5 / 33.3, 320: 32.2 / 34.0.  (One is the best up to 400 or so.)
  // Beyond, as many as fit at once, one per compute unit, with at least 64 tokens each: 80 rows, B = 700: 28.8 / 28.0 / 27.6 (3) /
  // 29.5 (4); 8 rows of 32768, B = 2048, 4 / 8 / 16 / 32: 18.9 / 16.6 / 15.2 / 15.1; 32 rows, 7 heads, B = 6219, 4 / 8 / 16: 40.9 / 38.2 / 44.7
  int w = bsel <= 256 ? 1 : kAssumedCUs / rows;
  if (w > (bsel + 63) / 64) w = (bsel + 63) / 64;
  if (w > kListMaxWgs) w = kListMaxWgs;
  // ... and no more than the row's last workgroup merges in one go (combine_row: eight partials in flight for each of 512 / 32 G threads, four
  // times over at most), for up to 400 tokens each.  us, as many as fit / so: 4 rows, 8 heads, B = 3205 (50 / 16): 22.4 / 20.2; 1 row, 8 heads, 4748
  // (64 / 16): 19.1 / 17.9, 8000 (64 / 16 / 32): 23.5 / 23.0 / 21.8; 8 rows, 7 heads, 1821 (28 / 16): 18.6 / 17.8; 8 rows, 8 heads, 1500 (24 /
  // 16): 15.9 / 15.3; 3 rows, 4 heads, 3490 (55 / 32): 19.8 / 19.3; 4 rows, 1 head, 8000 (64 / 32): 21.7 / 21.4; 2 rows, 2 heads, 4000
  // (63 / 32): 17.5 / 16.7
  const int chunk = s.n_q_heads / s.n_kv_heads <= 4 ? 32 : 16, merged = chunk * ((bsel + 400 * chunk - 1) / (400 * chunk));
  if (w > merged) w = merged;
  if (w > max_splits) w = max_splits;
  if (w < 1) w = 1;
  const int share = ((bsel + w - 1) / w + 15) / 16 * 16;
  if (share > kListMaxShare) return p;
  p.nwgs = (bsel + share - 1) / share;
  p.quads = quads;
  return p;
}

struct ListLaunch {
  uint2 *list, *lims;
  int nwgs, quads, places, pitch;
};
template <int G, int Q>
static hipError_t launch_list_q(const fasa_shape& s, const ListLaunch& l, const StepArgs& a, hipStream_t st) {
  const int bsel = s.budget < s.n_ctx ? s.budget : s.n_ctx;
  const long long wgs = (long long)a.rows * l.nwgs;
  auto kernel = list_kernel<G, Q, false>;
  if constexpr (Q >= 3) {                                      // (as much with shorter lists takes a hundred rows and more)
    if (gather_bytes(s) >= kStreamBytes) kernel = list_kernel<G, Q, true>;
  }
  return launch("fasa_list", kernel, dim3((unsigned)wgs), dim3(kListNT), st, l.list, l.lims, a.rows, l.nwgs,
                div_magic(l.nwgs, wgs > bsel + l.nwgs ? wgs : bsel + l.nwgs), a.N_max, a.n_cap,
                a.n_ctx_seq || a.budget_seq ? -l.places : l.places, bsel, ((bsel + l.nwgs - 1) / l.nwgs + 15) & ~15, a.Hkv, a.m_hkv, l.pitch, a);
}
template <int G>
static hipError_t launch_list_g(const fasa_shape& s, const ListLaunch& l, const StepArgs& a, hipStream_t st) {
  switch (l.quads) {
    case 1: return launch_list_q<G, 1>(s, l, a, st);
    case 2: return launch_list_q<G, 2>(s, l, a, st);
    case 3: return launch_list_q<G, 3>(s, l, a, st);
    case 4: return launch_list_q<G, 4>(s, l, a, st);
    case 6: return launch_list_q<G, 6>(s, l, a, st);
    case 8: return launch_list_q<G, 8>(s, l, a, st);
    default: return hipErrorInvalidValue;
  }
}

static StepArgs step_args(const fasa_shape& s, const void* q, void* K, void* V, void* Kp, const int32_t* fc_idx, const void* k_new,
                          const void* v_new, float* S, int32_t* T, float* O, RowCtl* ctl, RaggedLens rl, PageMap pm);

hipError_t launch_list_step(const fasa_shape& s, const ListPlan& p, const void* q, void* K, void* V, void* Kp,
                            const int32_t* fc_idx, const void* k_new, const void* v_new, float* S, int32_t* T, float* O,
                            RowCtl* ctl, uint2* list, uint2* lims, float* part_acc, float* part_ml, hipStream_t st,
                            RaggedLens rl, PageMap pm) {
  const int bsel = s.budget < s.n_ctx ? s.budget : s.n_ctx;
  const int pitch = list_room(bsel, s.n_ctx), places = list_places(s.n_ctx, bsel, p.quads, rl.n_ctx || rl.budget);
  const hipError_t e = launch_score_list(s, q, Kp, fc_idx, S, ListOut{list, lims, places, pitch}, st, rl,
                                         AppendArgs{k_new, v_new, K, V, pm, false});
  if (e != hipSuccess) return e;
  StepArgs a = step_args(s, q, K, V, Kp, fc_idx, k_new, v_new, S, T, O, ctl, rl, pm);
  a.part_acc = part_acc; a.part_ml = part_ml;
  const ListLaunch l{list, lims, p.nwgs, p.quads, places, pitch};
  switch (s.n_q_heads / s.n_kv_heads) {
    case 1: return launch_list_g<1>(s, l, a, st);
    case 2: return launch_list_g<2>(s, l, a, st);
    case 3: return launch_list_g<3>(s, l, a, st);
    case 4: return launch_list_g<4>(s, l, a, st);
    case 5: return launch_list_g<5>(s, l, a, st);
    case 6: return launch_list_g<6>(s, l, a, st);
    case 7: return launch_list_g<7>(s, l, a, st);
    case 8: return launch_list_g<8>(s, l, a, st);
    default: return hipErrorInvalidValue;
  }
}

static StepArgs step_args(const fasa_shape& s, const void* q, void* K, void* V, void* Kp, const int32_t* fc_idx, const void* k_new,
                          const void* v_new, float* S, int32_t* T, float* O, RowCtl* ctl, RaggedLens rl, PageMap pm) {
  StepArgs a{};
  a.q = q; a.K = K; a.V = V; a.Kp = Kp; a.fc_idx = fc_idx;
  a.append = k_new != nullptr;
  a.k_new = k_new ? k_new : q;      // rows * head_dim elements are there: the queries are no fewer
  a.v_new = v_new ? v_new : q;
  a.S = S; a.T = T; a.O = O; a.ctl = ctl;
  a.n_ctx_seq = rl.n_ctx; a.budget_seq = rl.budget;
  a.sb = s.kv_stride_b; a.sh = s.kv_stride_h; a.sn = s.kv_stride_n;
  a.pm = pm;
  a.rows = s.batch * s.n_kv_heads;
  const int per = kStepNT * (s.dtype == FASA_BF16 ? 4 : 2);
  a.nslices = (s.n_ctx + per - 1) / per;
  a.m_slices = div_magic(a.nslices, (long long)a.rows * a.nslices);
  a.G = s.n_q_heads / s.n_kv_heads; a.Hkv = s.n_kv_heads; a.m_hkv = div_magic(s.n_kv_heads, a.rows); a.F = s.n_fc; a.N_max = s.n_ctx; a.n_cap = s.n_cap;
  a.budget_max = s.budget;
  a.t_pitch = s.budget < s.n_ctx ? s.budget : s.n_ctx;
  a.pairing = s.pairing;
  a.scale_log2e = 1.4426950408889634f / sqrtf((float)s.head_dim);
  return a;
}

hipError_t launch_step(const fasa_shape& s, StepForm form, const void* q, void* K, void* V, void* Kp,
                       const int32_t* fc_idx, const void* k_new, const void* v_new, float* S, int32_t* T, float* O,
                       RowCtl* ctl, hipStream_t st, RaggedLens rl, PageMap pm) {
  const StepArgs a = step_args(s, q, K, V, Kp, fc_idx, k_new, v_new, S, T, O, ctl, rl, pm);
  const int G = s.n_q_heads / s.n_kv_heads;
  if (form == kStepRow) {                                      // (float32: a bf16 cache's lists come from the scoring launch)
    const hipError_t e = launch_score(s, q, Kp, fc_idx, S, nullptr, st, rl, AppendArgs{k_new, v_new, K, V, pm, false});
    if (e != hipSuccess) return e;
    if (G == 1) return launch("fasa_row", row_kernel<1>, dim3(a.rows), dim3(kRowNT), st, a);
    if (G <= 4) return launch("fasa_row", row_kernel<4>, dim3(a.rows), dim3(kRowNT), st, a);
    return hipErrorInvalidValue;                               // (row_form)
  }
  if (s.n_ctx > kStepMaxCtx) return hipErrorInvalidValue;      // (plan_step)
  if (s.dtype == FASA_BF16) return launch_step_f<uint16_t, 8>(a, st);
  if (G == 1) return launch_step_f<float, 1>(a, st);
  if (G <= 4) return launch_step_f<float, 4>(a, st);
  return launch_step_f<float, 8>(a, st);
}

}  // namespace fasa
