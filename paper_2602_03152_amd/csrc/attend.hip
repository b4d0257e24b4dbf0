// FAC (paper Sec. 4.2, eq. fac_output): exact softmax attention over the selected rows of K and V,
// as split-K flash decoding: every workgroup owns a chunk of the row's index list, gathers the
// K/V rows it names, keeps a running (max, sum, weighted V) per query head of the GQA group, and
// the workgroup that finishes a row last merges the row's chunks.  The same kernel with the index list replaced by the
// identity is the full-KV baseline (paper Sec. 4.4).
#include "mfma_tile.h"

namespace fasa {

constexpr int kAttU = 4;                  // rows in flight per 16-lane group and batch
constexpr int kAttBatch = 4 * kAttU;      // rows per wave and batch

// 8 consecutive head dims of one cached row
struct Row8 {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const float4*>(p);
    b = *reinterpret_cast<const float4*>(p + 4);
  }
  __device__ __forceinline__ void unpack(float* f) const {
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
};

// float32 caches with one or two query heads per KV head, on the vector ALUs: there the matrix cores, which always
// compute 16 heads, take longer over a tile than its loads (full KV, 4 rows of 20000, one head: 18.0 us like this,
// 20.2 on the matrix cores; two heads 14.9 / 15.8; from four heads on the matrix cores: 31.3 / 30.5, eight 24.5 / 19.1).
// 1-D grid of rows * n_splits workgroups, 256 threads.  A wave is 4 groups of 16 lanes; a group
// reads one cached row of 512 bytes with two load instructions, lane c owning head dims [8c, 8c+8) of K (for
// the logit) and of V (for the output).  The workgroup that finishes a row last merges the row's partials into O.
template <int G, bool DENSE>
__global__ __launch_bounds__(256) void attend_valu_kernel(const float* __restrict__ q,
                                                     const float* __restrict__ K,
                                                     const float* __restrict__ V,
                                                     const int32_t* __restrict__ T,
                                                     float* __restrict__ O,
                                                     RowCtl* __restrict__ ctl,
                                                     float* __restrict__ part_acc,
                                                     float* __restrict__ part_ml, int rows,
                                                     int n_splits, uint32_t m_splits, int Hkv, uint32_t m_hkv, int count_max,
                                                     int n_ctx_max, int tok_per_split, long long sb,
                                                     long long sh, long long sn,
                                                     float scale_log2e,
                                                     const int32_t* __restrict__ n_ctx_seq,
                                                     const int32_t* __restrict__ budget_seq,
                                                     PageMap pm) {
  constexpr int D = kHeadDim;
  __shared__ float sm_m[4][G], sm_l[4][G];
  __shared__ float sm_acc[4][G][D];
  __shared__ float wsm[G * kMaxSplitsLds];
  __shared__ float red[G];
  __shared__ uint32_t ticket;

  int row, split;
  row_slice_of_block(rows, n_splits, m_splits, row, split);
  int b, h;
  head_of_row(row, Hkv, m_hkv, b, h);
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int r = lane >> 4, c = lane & 15;

  // entries of this row: the shape's values, or this sequence's own (never more than the shape's)
  const int n_ctx = seq_n_ctx(n_ctx_seq, b, n_ctx_max);
  const int count = DENSE ? n_ctx : seq_bsel(budget_seq, b, n_ctx, count_max);
  const int s0 = split * tok_per_split;
  const int s1 = min(count, s0 + tok_per_split);

  float qr[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float* qp = q + ((size_t)row * G + g) * D + 8 * c;
#pragma unroll
    for (int k = 0; k < 8; ++k) qr[g][k] = qp[k] * scale_log2e;
  }
  float acc[G][8], m[G], l[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = kNegBig;
    l[g] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[g][k] = 0.f;
  }

  // list entries are token numbers, or pool slots of a paged cache (block << shift | offset)
  const bool paged = pm.table != nullptr;
  const int pshift = paged ? pm.shift : 31, pmask = paged ? (1 << pm.shift) - 1 : 0x7fffffff;
  const long long blk_stride = paged ? sb : 0;
  const int slot_max = paged ? (pm.n_pool << pm.shift) - 1 : n_ctx - 1;
  const float* Kb = K + (paged ? 0 : b * sb) + h * sh + 8 * c;
  const float* Vb = V + (paged ? 0 : b * sb) + h * sh + 8 * c;
  const int32_t* Trow = DENSE ? nullptr : T + (size_t)row * count_max;

  for (int j0 = s0 + wave * kAttBatch; j0 < s1; j0 += 4 * kAttBatch) {
    bool valid[kAttU];
    Row8 kv[kAttU], vv[kAttU];
    long long off[kAttU];
#pragma unroll
    for (int u = 0; u < kAttU; ++u) {
      const int j = j0 + u * 4 + r;
      valid[u] = j < s1;
      const int jj = valid[u] ? j : s0;              // any in-range entry; its weight is zeroed
      // a stray index can never become a stray address: entries are clamped to the cache
      const int tok = DENSE ? jj : min(max(Trow[jj], 0), slot_max);
      off[u] = (long long)(tok >> pshift) * blk_stride + (long long)(tok & pmask) * sn;
    }
#pragma unroll
    for (int u = 0; u < kAttU; ++u) kv[u].load(Kb + off[u]);
#pragma unroll
    for (int u = 0; u < kAttU; ++u) vv[u].load(Vb + off[u]);

    float s[kAttU][G];
#pragma unroll
    for (int u = 0; u < kAttU; ++u) {
      float kf[8];
      kv[u].unpack(kf);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float d = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) d = fmaf(qr[g][k], kf[k], d);
        s[u][g] = row16_sum(d);   // all 16 lanes of the group end up with the logit
      }
    }
    float p[kAttU][G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float mx = m[g];
#pragma unroll
      for (int u = 0; u < kAttU; ++u) mx = valid[u] ? fmaxf(mx, s[u][g]) : mx;
      const float sc = exp2f(m[g] - mx);
      m[g] = mx;
      float ls = l[g] * sc;
#pragma unroll
      for (int u = 0; u < kAttU; ++u) {
        p[u][g] = valid[u] ? exp2f(s[u][g] - mx) : 0.f;
        ls += p[u][g];
      }
      l[g] = ls;
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[g][k] *= sc;
    }
#pragma unroll
    for (int u = 0; u < kAttU; ++u) {
      float vf[8];
      vv[u].unpack(vf);
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[g][k] = fmaf(p[u][g], vf[k], acc[g][k]);
    }
  }

  // merge the 4 groups of the wave (lanes c, c+16, c+32, c+48 hold the same head dims)
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float mn = xor32_max(xor16_max(m[g]));
    const float sc = exp2f(m[g] - mn);
    m[g] = mn;
    l[g] = xor32_sum(xor16_sum(l[g] * sc));
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[g][k] = xor32_sum(xor16_sum(acc[g][k] * sc));
  }
  if (r == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (c == 0) { sm_m[wave][g] = m[g]; sm_l[wave][g] = l[g]; }
#pragma unroll
      for (int k = 0; k < 8; ++k) sm_acc[wave][g][8 * c + k] = acc[g][k];
    }
  }
  __syncthreads();

  // merge the 4 waves; one (query head, head dim) per thread and pass
  const size_t pbase = ((size_t)row * n_splits + split) * G;
  for (int i = t; i < G * D; i += 256) {
    const int g = i / D, dim = i % D;
    float mn = sm_m[0][g];
#pragma unroll
    for (int w = 1; w < 4; ++w) mn = fmaxf(mn, sm_m[w][g]);
    float ls = 0.f, a = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float sc = exp2f(sm_m[w][g] - mn);
      ls = fmaf(sm_l[w][g], sc, ls);
      a = fmaf(sm_acc[w][g][dim], sc, a);
    }
    if (n_splits == 1) {
      O[((size_t)row * G + g) * D + dim] = a / ls;   // nothing to merge
    } else {
      // read by the row's last workgroup: published with agent-scope stores
      st_agent(&part_acc[(pbase + g) * D + dim], a);
      if (dim == 0) {
        st_agent(&part_ml[(pbase + g) * 2], mn);
        st_agent(&part_ml[(pbase + g) * 2 + 1], ls);
      }
    }
  }
  if (n_splits == 1) return;

  // ---- the row's last workgroup merges the splits ----
  publish_barrier();
  if (t == 0) ticket = atomicAdd(&ctl[row].done_att, 1u);
  __syncthreads();
  if (ticket != (uint32_t)n_splits - 1u) return;
  if (t == 0) ctl[row].done_att = 0;   // clean for the next call
  combine_row<G>(part_acc, part_ml, O, row, n_splits, n_splits, wsm, red, &sm_acc[0][0][0]);
}

// ---------------------------------------------------------------------------------------------
// Both products of a 16-row tile run on the matrix cores (mfma_tile.h): the logits
// K_tile . Q^T of the GQA group and the weighted sum P . V_tile.  The tile loop is software-pipelined:
// while a tile is computed, the next tile's K/V rows and, of a list, the entries of the tile after it are in
// flight.  Loads inside the loop are unconditional (straight-line code keeps the compiler's wait
// counts exact: a test around a load would turn every later wait into a wait for everything);
// entries beyond the range are clamped into it and only fetched, the K/V prefetch is issued for real
// tiles only (the last tile is peeled).
// ---------------------------------------------------------------------------------------------
template <typename ET, int G, bool DENSE>
__global__ __launch_bounds__(256, sizeof(ET) == 4 ? 2 : 1) void attend_kernel(const ET* __restrict__ q,
                                                          const ET* __restrict__ K,
                                                          const ET* __restrict__ V,
                                                          const int32_t* __restrict__ T,
                                                          float* __restrict__ O,
                                                          RowCtl* __restrict__ ctl,
                                                          float* __restrict__ part_acc,
                                                          float* __restrict__ part_ml, int rows,
                                                          int n_splits, uint32_t m_splits, int Hkv, uint32_t m_hkv, int count_max,
                                                          int n_ctx_max, int tok_per_split, long long sb,
                                                          long long sh, long long sn,
                                                          float scale_log2e,
                                                          const int32_t* __restrict__ n_ctx_seq,
                                                          const int32_t* __restrict__ budget_seq,
                                                          PageMap pm) {
  constexpr int D = kHeadDim;
  // the waves' totals, later the merge's partition scratch (< 8 KB) and, behind it, its split weights
  constexpr int ACC_BYTES = 4 * G * D * 4;
  constexpr int MERGE_BYTES = 8192 + G * kMaxSplitsLds * 4;
  __shared__ __align__(16) unsigned char big[ACC_BYTES > MERGE_BYTES ? ACC_BYTES : MERGE_BYTES];
  __shared__ float sm_m[4][G], sm_l[4][G];
  __shared__ float red[G];
  __shared__ uint32_t ticket;
  __shared__ __align__(16) float scs[4][16];      // per wave: rescale factor of each head's running sums
  float (*sm_o)[G][D] = reinterpret_cast<float (*)[G][D]>(big);
  float* wsm = reinterpret_cast<float*>(big + 8192);

  int row, split;
  row_slice_of_block(rows, n_splits, m_splits, row, split);
  int b, h;
  head_of_row(row, Hkv, m_hkv, b, h);
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int lo = lane & 15, hi = lane >> 4;

  // entries of this row: the shape's values, or this sequence's own (never more than the shape's)
  const int n_ctx = seq_n_ctx(n_ctx_seq, b, n_ctx_max);
  const int count = DENSE ? n_ctx : seq_bsel(budget_seq, b, n_ctx, count_max);
  const int s0 = split * tok_per_split;
  const int s1 = min(count, s0 + tok_per_split);
  FASA_T_DECL(5);
  FASA_T(0);

  MfmaTile<G, ET> tile;
  tile.load_q(q + ((size_t)row * G) * D, lo, hi);
  tile.reset();

  // list entries are token numbers, or pool slots of a paged cache (block << shift | offset)
  const bool paged = pm.table != nullptr;
  const int pshift = paged ? pm.shift : 31, pmask = paged ? (1 << pm.shift) - 1 : 0x7fffffff;
  const long long blk_stride = paged ? sb : 0;
  const int slot_max = paged ? (pm.n_pool << pm.shift) - 1 : n_ctx - 1;
  const ET* Kb = K + (paged ? 0 : b * sb) + h * sh + kChunk<ET> * hi;
  const ET* Vb = V + (paged ? 0 : b * sb) + h * sh + 8 * lo;
  const int32_t* Trow = DENSE ? nullptr : T + (size_t)row * count_max;

  struct TileIdx { int k; int v[4]; };        // list entries of one tile: K row lo, V rows 4hi .. 4hi+3
  auto load_idx = [&](int j0) {
    TileIdx r;
    if constexpr (DENSE) {
      r.k = min(j0 + lo, s1 - 1);
#pragma unroll
      for (int i = 0; i < 4; ++i) r.v[i] = min(j0 + 4 * hi + i, s1 - 1);
    } else {
      // a stray index can never become a stray address: entries are clamped to the cache below
      r.k = Trow[min(j0 + lo, s1 - 1)];
#pragma unroll
      for (int i = 0; i < 4; ++i) r.v[i] = Trow[min(j0 + 4 * hi + i, s1 - 1)];
    }
    return r;
  };
  auto row_off = [&](int e) {
    const int sl = min(max(e, 0), slot_max);
    return (long long)(sl >> pshift) * blk_stride + (long long)(sl & pmask) * sn;
  };
  auto load_kv = [&](const TileIdx& ix) {
    TileKV<ET> r;
    r.load_k(Kb + row_off(ix.k));
#pragma unroll
    for (int i = 0; i < 4; ++i) r.load_v(i, Vb + row_off(ix.v[i]));
    return r;
  };
  auto compute_tile = [&](const TileKV<ET>& kv, int j0) {
    float sv[4];
    tile.logits(kv, scale_log2e, sv);
    bool valid[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) valid[e] = j0 + 4 * hi + e < s1;
    tile.accumulate(kv, sv, valid, &scs[wave][0], lo, hi);
  };

  const int jw = s0 + wave * 16;               // this wave's tiles start at jw, jw + 64, ...
  if (jw < s1) {
    const int n_tiles = (s1 - jw + 63) / 64;
    TileIdx ix_next = load_idx(jw + 64);
    TileKV<ET> cur = load_kv(load_idx(jw));
    for (int i = 0; i + 1 < n_tiles; ++i) {     // (a tile with another behind it is full)
      const int j0 = jw + 64 * i;
      if constexpr (DENSE) {
        // one set of registers, as in attend_wide_kernel
        float sv[4];
        tile.logits(cur, scale_log2e, sv);
        __builtin_amdgcn_sched_barrier(0);
        cur.load_k(Kb + row_off(ix_next.k));
        __builtin_amdgcn_sched_barrier(0);
        tile.accumulate_full(cur, sv, &scs[wave][0], lo, hi);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 4; ++k) cur.load_v(k, Vb + row_off(ix_next.v[k]));
        ix_next = load_idx(j0 + 128);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        // (one set of registers measured the same: 16 rows, 1250 of 20011: 8.00 / 7.98, 32 rows, 6219 of 32905: 22.5 / 22.7)
        const TileKV<ET> nxt = load_kv(ix_next);
        ix_next = load_idx(j0 + 128);
        compute_tile(cur, j0);
        cur = nxt;
      }
    }
    compute_tile(cur, jw + 64 * (n_tiles - 1));
  }
  FASA_T(1);
  tile.finish(&sm_m[wave][0], &sm_l[wave][0], &sm_o[wave][0][0], lo, hi);
  __syncthreads();

  // workgroup totals: thread (query head g, 4 head dims)
  const size_t pbase = ((size_t)row * n_splits + split) * G;
  if (t < G * (D / 4)) {
    const int g = t / (D / 4), d4 = t % (D / 4);
    float mn, ls;
    float4 a;
    tile_wg_totals<G>(&sm_m[0][0], &sm_l[0][0], &sm_o[0][0][0], g, d4, mn, ls, a);
    if (n_splits == 1) {
      *reinterpret_cast<float4*>(O + ((size_t)row * G + g) * D + 4 * d4) =
          make_float4(a.x / ls, a.y / ls, a.z / ls, a.w / ls);
    } else {
      float2* pa = reinterpret_cast<float2*>(part_acc + (pbase + g) * D + 4 * d4);
      st_agent(pa, make_float2(a.x, a.y));
      st_agent(pa + 1, make_float2(a.z, a.w));
      if (d4 == 0) st_agent(reinterpret_cast<float2*>(part_ml + (pbase + g) * 2), make_float2(mn, ls));
    }
  }
  if (n_splits == 1) return;
  FASA_T(2);
  publish_barrier();
  if (t == 0) ticket = atomicAdd(&ctl[row].done_att, 1u);
  __syncthreads();
  FASA_T(3);
  FASA_T_PRINT(t == 0 && row == 0 && split == 0, "attend blk0: tiles %llu merge %llu publish+ticket %llu (x10ns)\n",
               FASA_T_D(1, 0), FASA_T_D(2, 1), FASA_T_D(3, 2));
  if (ticket != (uint32_t)n_splits - 1u) return;
  if (t == 0) ctl[row].done_att = 0;
  combine_row<G>(part_acc, part_ml, O, row, n_splits, n_splits, wsm, red, reinterpret_cast<float*>(big));
  FASA_T(4);
  FASA_T_PRINT(t == 0 && row == 0, "attend last(row0, split %d): tiles %llu merge %llu publish+ticket %llu combine %llu (x10ns)\n",
               split, FASA_T_D(1, 0), FASA_T_D(2, 1), FASA_T_D(3, 2), FASA_T_D(4, 3));
}

// Attention of a bf16 cache where much of it is read.  One workgroup of eight waves per compute unit: half the partial
// results that two of four waves publish, and as many waves again to merge them, which is what a row's end costs (64 splits
// of 4 heads are 128 KB for one compute unit to read back).  In 104 registers (108 with a list), so that a grid a little
// larger than the chip shares it.  Full KV,
// us, two workgroups of four waves (attend_kernel's tiles) / like this: 8 rows of 32768, 4 heads: 30.9 / 26.4 (5.1 TB/s; 5.6 of
// it without launch and merge); of 8192: 11.7 / 10.4; of 131072: 95.3 / 91.7; 4 rows of 20000, 7 heads: 22.8 / 14.4; two
// workgroups of eight waves: 29.5 / 11.4 / 94.8 / 22.0; one of sixteen: 28.2 / 11.5 / 94.6 / 14.9.
//
// L = NoList: all rows; SparseList: those that T names (token numbers, or pool slots of a paged cache: block << shift | offset).
// (An empty argument: with the list's arguments unused, full KV of 8 rows of 8192 takes 0.3 us longer.)
// NoList<NT>: which of V (1) and K (2) are read non-temporal (kStreamBytes): V where K and V have that many bytes, K as well where it alone does.  A wave's load of K is
// half a line of each of 16 rows, and the other half, a load later, may come from memory again if lines are not kept; V's are whole rows.  us over three sets of
// buffers, kept / V / both: 8 rows of 24000, 4 heads (98 MB): 19.5 / 18.8 / 20.0; of 16384: 14.1 / 14.45 / 14.8; of 32768 (134 MB): 26.6 / 23.4 / 24.3; of 65536:
// 48.5 / 44.0 / 43.0; 32 rows of 32768: 92.1 / 84.1 / 83.3; 12 sets, 8 rows of 32768: 26.7 / 25.0 / 24.7.
constexpr int kWideNT = 512;
template <int NT> struct NoList {
  static constexpr bool used = false;
  static constexpr bool nt_v = NT & 1, nt_k = (NT & 2) != 0;
};
struct SparseList {
  static constexpr bool used = true, nt_v = false, nt_k = false;
  const int32_t* T;
  const int32_t *n_ctx_seq, *budget_seq;
  int count_max;
  PageMap pm;
};
template <int G, class L>
__global__ __launch_bounds__(kWideNT, 4) void attend_wide_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V, float* __restrict__ O,
    RowCtl* __restrict__ ctl, float* __restrict__ part_acc, float* __restrict__ part_ml, int rows, int n_splits, uint32_t m_splits,
    int Hkv, uint32_t m_hkv, int N_max, int tok_per_split, long long sb, long long sh, long long sn, float scale_log2e, L list) {
  constexpr bool LIST = L::used;
  constexpr int D = kHeadDim, NWV = kWideNT / kWave, STEP = 16 * NWV;   // rows of a round of tiles
  constexpr int ACC_BYTES = NWV * G * D * 4, MERGE_BYTES = 8192 + G * kMaxSplitsLds * 4;
  __shared__ __align__(16) unsigned char big[ACC_BYTES > MERGE_BYTES ? ACC_BYTES : MERGE_BYTES];
  __shared__ float sm_m[NWV][G], sm_l[NWV][G];
  __shared__ float red[G];
  __shared__ uint32_t ticket;
  __shared__ __align__(16) float scs[NWV][16];
  float (*sm_o)[G][D] = reinterpret_cast<float (*)[G][D]>(big);

  int row, split;
  row_slice_of_block(rows, n_splits, m_splits, row, split);
  int b, h;
  head_of_row(row, Hkv, m_hkv, b, h);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lo = lane & 15, hi = lane >> 4;
  int N = N_max, count = N_max;
  PageMap pm = kNoPaging;
  const int32_t* Trow = nullptr;
  if constexpr (LIST) {
    N = seq_n_ctx(list.n_ctx_seq, b, N_max);
    count = seq_bsel(list.budget_seq, b, N, list.count_max);
    pm = list.pm;
    Trow = list.T + (size_t)row * list.count_max;
  }
  const int s0 = split * tok_per_split, s1 = min(count, s0 + tok_per_split);

  MfmaTile<G> tile;
  tile.load_q(q + ((size_t)row * G) * D, lo, hi);
  tile.reset();
  const bool paged = pm.table != nullptr;
  const int pshift = paged ? pm.shift : 31, pmask = paged ? (1 << pm.shift) - 1 : 0x7fffffff;
  const int slot_max = paged ? (pm.n_pool << pm.shift) - 1 : N - 1;
  const uint16_t* Kr = K + (paged ? 0 : b * sb) + h * sh + 8 * hi;
  const uint16_t* Vr = V + (paged ? 0 : b * sb) + h * sh + 8 * lo;
  TileKV<uint16_t> kv;
  // Rows j0 .. j0 + 15, clamped to the split's last: K row lo, V rows 4hi .. 4hi + 3.  A list's entries (ek, ev) are requested a
  // tile ahead of their rows.
  int ek = 0, ev[4] = {0, 0, 0, 0};
  auto load_idx = [&](int j0) {
    if constexpr (LIST) {
      ek = Trow[min(j0 + lo, s1 - 1)];
#pragma unroll
      for (int i = 0; i < 4; ++i) ev[i] = Trow[min(j0 + 4 * hi + i, s1 - 1)];
    }
  };
  auto row_off = [&](int e) {
    const int sl = min(max(e, 0), slot_max);                   // a stray index can never become a stray address
    return (long long)(sl >> pshift) * (paged ? sb : 0) + (long long)(sl & pmask) * sn;
  };
  auto load_k = [&](int j0) {
    if constexpr (LIST) kv.load_k(Kr + row_off(ek));
    else kv.template load_k<L::nt_k>(Kr + (long long)min(j0 + lo, s1 - 1) * sn);
  };
  auto load_v = [&](int j0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (LIST) kv.load_v(i, Vr + row_off(ev[i]));
      else kv.template load_v<L::nt_v>(i, Vr + (long long)min(j0 + 4 * hi + i, s1 - 1) * sn);
    }
  };
  const int jw = s0 + wave * 16;
  if (jw < s1) {
    const int n_tiles = (s1 - jw + STEP - 1) / STEP;
    float sv[4];
    load_idx(jw);
    load_k(jw);
    load_v(jw);
    load_idx(jw + STEP);
    int j0 = jw;
    for (int i = 0; i + 1 < n_tiles; ++i, j0 += STEP) {        // (a tile with another behind it is full)
      // One set of registers: the next tile's K goes where this one's has been used, and runs under this tile's P . V, its V
      // under the next logits.  (With a second set the compiler waits for all of the next tile before this one's last
      // products, to move it over; two sets used in turn are slower where much is read.)
      tile.logits(kv, scale_log2e, sv);
      __builtin_amdgcn_sched_barrier(0);
      load_k(j0 + STEP);
      __builtin_amdgcn_sched_barrier(0);
      tile.accumulate_full(kv, sv, &scs[wave][0], lo, hi);
      __builtin_amdgcn_sched_barrier(0);
      load_v(j0 + STEP);
      load_idx(j0 + 2 * STEP);
      __builtin_amdgcn_sched_barrier(0);
    }
    tile.logits(kv, scale_log2e, sv);
    bool valid[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) valid[e] = j0 + 4 * hi + e < s1;
    tile.accumulate(kv, sv, valid, &scs[wave][0], lo, hi);
  }
  tile.finish(&sm_m[wave][0], &sm_l[wave][0], &sm_o[wave][0][0], lo, hi);
  __syncthreads();

  const size_t pbase = ((size_t)row * n_splits + split) * G;
  if (t < G * (D / 4)) {
    const int g = t / (D / 4), d4 = t % (D / 4);
    float mn, ls;
    float4 a;
    tile_wg_totals<G, NWV>(&sm_m[0][0], &sm_l[0][0], &sm_o[0][0][0], g, d4, mn, ls, a);
    if (n_splits == 1) {
      *reinterpret_cast<float4*>(O + ((size_t)row * G + g) * D + 4 * d4) =
          make_float4(a.x / ls, a.y / ls, a.z / ls, a.w / ls);
    } else {
      float2* pa = reinterpret_cast<float2*>(part_acc + (pbase + g) * D + 4 * d4);
      st_agent(pa, make_float2(a.x, a.y));
      st_agent(pa + 1, make_float2(a.z, a.w));
      if (d4 == 0) st_agent(reinterpret_cast<float2*>(part_ml + (pbase + g) * 2), make_float2(mn, ls));
    }
  }
  if (n_splits == 1) return;
  publish_barrier();
  if (t == 0) ticket = atomicAdd(&ctl[row].done_att, 1u);
  __syncthreads();
  if (ticket != (uint32_t)n_splits - 1u) return;
  if (t == 0) ctl[row].done_att = 0;
  combine_row<G, NothingUnderLoads, 16, kWideNT>(part_acc, part_ml, O, row, n_splits, n_splits,
                                                  reinterpret_cast<float*>(big + 8192), red, reinterpret_cast<float*>(big));
}

template <int G>
static hipError_t launch_wide_g(const fasa_shape& s, bool dense, const AttendPlan& p, const void* q, const void* K, const void* V,
                                const int32_t* T, float* O, RowCtl* ctl, float* part_acc, float* part_ml, hipStream_t st,
                                RaggedLens rl, PageMap pm) {
  const int rows = s.batch * s.n_kv_heads;
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)s.head_dim);
  const dim3 grid(rows * p.n_splits), block(kWideNT);
  const uint32_t m_splits = div_magic(p.n_splits, (long long)rows * p.n_splits), m_hkv = div_magic(s.n_kv_heads, rows);
  const uint16_t *q16 = (const uint16_t*)q, *k16 = (const uint16_t*)K, *v16 = (const uint16_t*)V;
  const long long sb = s.kv_stride_b, sh = s.kv_stride_h, sn = s.kv_stride_n;
  if (dense) {
    const auto all = [&](auto list) {
      return launch("fasa_dense_attend", attend_wide_kernel<G, decltype(list)>, grid, block, st, q16, k16, v16, O, ctl, part_acc, part_ml,
                    rows, p.n_splits, m_splits, s.n_kv_heads, m_hkv, s.n_ctx, p.tok_per_split, sb, sh, sn, scale_log2e, list);
    };
    const long long of_k = (long long)rows * s.n_ctx * s.head_dim * 2;
    return of_k >= kStreamBytes ? all(NoList<3>{}) : 2 * of_k >= kStreamBytes ? all(NoList<1>{}) : all(NoList<0>{});
  }
  return launch("fasa_sparse_attend", attend_wide_kernel<G, SparseList>, grid, block, st, q16, k16, v16, O, ctl, part_acc, part_ml,
                rows, p.n_splits, m_splits, s.n_kv_heads, m_hkv, s.n_ctx, p.tok_per_split, sb, sh, sn, scale_log2e,
                SparseList{T, rl.n_ctx, rl.budget, p.count, pm});
}
static hipError_t launch_wide(const fasa_shape& s, bool dense, const AttendPlan& p, const void* q, const void* K, const void* V,
                              const int32_t* T, float* O, RowCtl* ctl, float* part_acc, float* part_ml, hipStream_t st,
                              RaggedLens rl, PageMap pm) {
  switch (s.n_q_heads / s.n_kv_heads) {
    case 1: return launch_wide_g<1>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 2: return launch_wide_g<2>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 3: return launch_wide_g<3>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 4: return launch_wide_g<4>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 5: return launch_wide_g<5>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 6: return launch_wide_g<6>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 7: return launch_wide_g<7>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 8: return launch_wide_g<8>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    default: return hipErrorInvalidValue;
  }
}

template <typename ET, int G>
static hipError_t launch_attend_g(const fasa_shape& s, bool dense, const AttendPlan& p,
                                  const void* q, const void* K, const void* V, const int32_t* T,
                                  float* O, RowCtl* ctl, float* part_acc, float* part_ml,
                                  hipStream_t st, RaggedLens rl, PageMap pm) {
  const int rows = s.batch * s.n_kv_heads;
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)s.head_dim);
  auto kernel = [&]() {
    if constexpr (sizeof(ET) == 4 && G <= 2) return dense ? attend_valu_kernel<G, true> : attend_valu_kernel<G, false>;
    else return dense ? attend_kernel<ET, G, true> : attend_kernel<ET, G, false>;
  }();
  return launch(dense ? "fasa_dense_attend" : "fasa_sparse_attend", kernel, dim3(rows * p.n_splits), dim3(256), st,
                (const ET*)q, (const ET*)K, (const ET*)V, T, O, ctl, part_acc, part_ml, rows, p.n_splits,
                div_magic(p.n_splits, (long long)rows * p.n_splits), s.n_kv_heads, div_magic(s.n_kv_heads, rows), p.count, s.n_ctx, p.tok_per_split, (long long)s.kv_stride_b,
                (long long)s.kv_stride_h, (long long)s.kv_stride_n, scale_log2e, rl.n_ctx, rl.budget, pm);
}

template <typename ET>
static hipError_t launch_attend_t(const fasa_shape& s, bool dense, const AttendPlan& p,
                                  const void* q, const void* K, const void* V, const int32_t* T,
                                  float* O, RowCtl* ctl, float* part_acc, float* part_ml,
                                  hipStream_t st, RaggedLens rl, PageMap pm) {
  switch (s.n_q_heads / s.n_kv_heads) {
    case 1: return launch_attend_g<ET, 1>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 2: return launch_attend_g<ET, 2>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 3: return launch_attend_g<ET, 3>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 4: return launch_attend_g<ET, 4>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 5: return launch_attend_g<ET, 5>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 6: return launch_attend_g<ET, 6>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 7: return launch_attend_g<ET, 7>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    case 8: return launch_attend_g<ET, 8>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_attend(const fasa_shape& s, bool dense, const void* q, const void* K,
                         const void* V, const int32_t* T, float* O, RowCtl* ctl, float* part_acc,
                         float* part_ml, hipStream_t st, RaggedLens rl, PageMap pm) {
  const int rows = s.batch * s.n_kv_heads;
  if (dense && pm.table != nullptr) return hipErrorInvalidValue;   // identity lists are token numbers
  const int count = dense ? s.n_ctx : (s.budget < s.n_ctx ? s.budget : s.n_ctx);
  const AttendPlan p = plan_attend(rows, count, s.n_q_heads / s.n_kv_heads);
  if (s.dtype == FASA_BF16 && dense && (rl.n_ctx || rl.budget)) return hipErrorInvalidValue;   // (no caller has full KV of those)
  // A list is attended like full KV where that halves many partials, attend_kernel / so: 4 rows, B = 6219, 7 heads (97 splits):
  // 15.1 / 11.0 us; 1 row, 20000 (256): 17.3 / 14.7; 2 rows, 9000 (141): 17.4 / 13.5; 1 row, 3000 (47): 9.1 / 8.75; but 8 rows,
  // 2048 (32): 7.3 / 7.4; 24 rows, 1000 (16): 8.1 / 8.4; 2 rows, 333 (6): 5.9 / 6.7
  // Short full KV has few partials to halve and no workgroups to share a compute unit with: up to 16 splits, while a
  // workgroup has one for itself, attend_kernel is the faster one, attend_kernel / wide: 8 rows of 500 (8 splits):
  // 5.75 / 6.28 us; of 1000 (16): 5.85 / 6.30; 16 rows of 700 (11): 5.86 / 6.37; 1 row of 700 (11): 5.76 / 5.93.  From 17 to 36 the two are
  // as good as each other: over 16 shapes of 1 - 8 rows and 1 - 8 heads, called one after another, 1.027 times as fast with this
  // one (0.95 - 1.08: 8 rows, 4 heads, of 1100: 6.73 / 6.31, of 1500: 6.35 / 6.39, 7 heads: 7.23 / 7.31, 2 heads, of 1200: 5.69 / 5.99), while in
  // graphs attend_kernel leads by 3 - 10 % where there are up to 4 heads (of 1200: 6.01 / 6.27) and up to 200 workgroups.  Beyond: 8 rows
  // of 2000 (32): 6.88 / 6.60; of 2300, 7 heads: 9.43 / 7.93; 32 rows of 1000 (16, 512 workgroups): 7.33 / 7.14; 32 rows of 600 (9, 288
  // workgroups), 8 heads: 8.33 / 6.70
  const bool wide = dense ? p.n_splits > 16 || rows * p.n_splits > kAssumedCUs : p.n_splits > 40;
  if (s.dtype == FASA_BF16 && wide)
    return launch_wide(s, dense, plan_attend_wide(rows, count), q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
  return s.dtype == FASA_BF16
             ? launch_attend_t<uint16_t>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm)
             : launch_attend_t<float>(s, dense, p, q, K, V, T, O, ctl, part_acc, part_ml, st, rl, pm);
}

}  // namespace fasa
