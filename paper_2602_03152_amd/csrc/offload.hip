// Memory-optimised variant (paper Sec. 4.3 and Alg. 2, "FASA-M"): only the dominant key dims (the
// FC-major copy Kp) stay in HBM; the non-dominant key dims and all values live in pinned host
// memory that the GPU can address.  Per step the B selected rows are fetched over PCIe by the GPU
// itself (zero-copy reads, no host-side gather), the full key rows are rebuilt from the two parts
// (Alg. 2: SelectTokens + TransferToGPU + Combine) into a compact staging buffer and attended in the same
// kernel (bf16) or by the usual attention kernel over that buffer (float32).
#include "mfma_tile.h"

namespace fasa {

constexpr int kOffTile = 64;   // tokens per workgroup of the split kernel

// Where output dim j of a rebuilt key row comes from: bit 15 set -> dominant pair entry
// (f * 2 + which), else index into the row's non-dominant part.
__device__ __forceinline__ void build_dim_map(const int32_t* __restrict__ fc_idx_h, int F, int pairing,
                                              uint16_t* src /*[D]*/, uint8_t* is_dom /*[D]*/) {
  constexpr int D = kHeadDim;
  const int t = threadIdx.x;
  if (t < D) is_dom[t] = 0;
  __syncthreads();
  if (t < F) {
    const int pr = pair_dims(pairing, fc_idx_h[t], 0);   // FC numbers only (rotate-half or interleaved)
    const int lo = pr & 255, hi = pr >> 8;
    is_dom[lo] = 1;
    is_dom[hi] = 1;
    src[lo] = (uint16_t)(0x8000u | (uint32_t)(2 * t));
    src[hi] = (uint16_t)(0x8000u | (uint32_t)(2 * t + 1));
  }
  __syncthreads();
  if (t < D && !is_dom[t]) {
    int pos = 0;
    for (int j = 0; j < t; ++j) pos += is_dom[j] ? 0 : 1;
    src[t] = (uint16_t)pos;
  }
  __syncthreads();
}

// grid = (ceil(tokens / kOffTile), rows): dominant dims -> Kp planes (HBM), the rest -> host rows
template <typename ET>
__global__ __launch_bounds__(256) void offload_split_kernel(const ET* __restrict__ K,
                                                            const int32_t* __restrict__ fc_idx,
                                                            ET* __restrict__ Kp,
                                                            ET* __restrict__ Knd, int Hkv, int F,
                                                            int n_cap, int n_begin, int n_end,
                                                            long long sb, long long sh, long long sn,
                                                            int pairing) {
  constexpr int D = kHeadDim;
  constexpr int PITCH = D + 16 / sizeof(ET);
  __shared__ __align__(16) ET tile[kOffTile][PITCH];
  __shared__ uint16_t src[D];
  __shared__ uint8_t is_dom[D];
  const int row = blockIdx.y;
  const int b = row / Hkv, h = row % Hkv;
  const int n0 = n_begin + blockIdx.x * kOffTile;
  const int nt = min(kOffTile, n_end - n0);
  const int t = threadIdx.x;
  build_dim_map(fc_idx + h * F, F, pairing, src, is_dom);

  constexpr int VEC = 16 / sizeof(ET);
  constexpr int LPR = D / VEC;
  const ET* ksrc = K + b * sb + h * sh;
  for (int i = t; i < nt * LPR; i += 256) {
    const int r = i / LPR, c = i % LPR;
    *reinterpret_cast<uint4*>(&tile[r][c * VEC]) =
        *reinterpret_cast<const uint4*>(ksrc + (long long)(n0 + r) * sn + c * VEC);
  }
  __syncthreads();
  const int nd = D - 2 * F;
  ET* kp = Kp + ((long long)row * F) * n_cap * 2;
  ET* knd = Knd + (long long)row * n_cap * nd;
  // every dim of every token goes to exactly one of the two destinations
  for (int i = t; i < nt * D; i += 256) {
    const int r = i / D, dim = i % D;
    const uint32_t s = src[dim];
    const ET v = tile[r][dim];
    if (s & 0x8000u) {
      const int f = (int)(s & 0x7FFFu) >> 1, which = (int)(s & 1u);
      kp[((long long)f * n_cap + (n0 + r)) * 2 + which] = v;
    } else {
      knd[(long long)(n0 + r) * nd + s] = v;
    }
  }
}

// The host link moves lines of 128 bytes, 2.4 ns each (53 GB/s; a copy engine reaches 56), wherever they lie: a
// 192-byte row that touches two lines costs what a 256-byte row does, and the reads of one step of the Llama-3-8B
// layer shape (8 x 2048 rows of 256 and of 192 bytes) cannot take less than 154 - 158 us.  From 0.5 to 2 MB of
// outstanding reads the rate is the same; with 4 MB and more it falls to 44 GB/s.  So the kernels that read host
// memory run on few workgroups which go through the list, about kOffInFlight bytes at a time.
constexpr int kOffInFlight = 1 << 20;

// float32 caches.  grid = (workgroups, rows), TOK = 256 / (D / VEC) tokens per workgroup at a time.
// Reads the selected tokens' non-dominant key part and value row from host memory, their dominant
// pairs from Kp, and writes full rows KT[row][j][:], VT[row][j][:] (j = position in the index list).
__global__ __launch_bounds__(256) void offload_gather_kernel(const float* __restrict__ Kp,
                                                             const float* __restrict__ Knd,
                                                             const float* __restrict__ Vh,
                                                             const int32_t* __restrict__ fc_idx,
                                                             const int32_t* __restrict__ T,
                                                             float* __restrict__ KT, float* __restrict__ VT,
                                                             int Hkv, int F, int n_cap, int n_ctx,
                                                             int count, long long sb, long long sh,
                                                             long long sn, int pairing) {
  constexpr int D = kHeadDim;
  constexpr int VEC = 16 / (int)sizeof(float);
  constexpr int LPR = D / VEC;
  constexpr int TOK = 256 / LPR;
  __shared__ uint16_t src[D];
  __shared__ uint8_t is_dom[D];
  __shared__ int toks[TOK];
  __shared__ float l_nd[TOK][D];
  __shared__ float l_dom[TOK][D];
  const int row = blockIdx.y;
  const int b = row / Hkv, h = row % Hkv;
  const int t = threadIdx.x;
  build_dim_map(fc_idx + h * F, F, pairing, src, is_dom);
  const int nd = D - 2 * F;
  const float* knd = Knd + (long long)row * n_cap * nd;
  const float* kp = Kp + ((long long)row * F) * n_cap * 2;
  const int s = t / LPR, c = t % LPR;
  for (int j0 = blockIdx.x * TOK; j0 < count; j0 += gridDim.x * TOK) {
    const int nt = min(TOK, count - j0);
    if (t < nt) toks[t] = min(max(T[(size_t)row * count + j0 + t], 0), n_ctx - 1);
    __syncthreads();
    for (int i = t; i < nt * nd; i += 256) {
      const int r = i / nd, j = i % nd;
      l_nd[r][j] = knd[(long long)toks[r] * nd + j];                       // host memory, coalesced per row
    }
    for (int i = t; i < nt * 2 * F; i += 256) {
      const int r = i / (2 * F), e = i % (2 * F);
      l_dom[r][e] = kp[((long long)(e >> 1) * n_cap + toks[r]) * 2 + (e & 1)];
    }
    uint4 vrow = make_uint4(0, 0, 0, 0);
    if (s < nt) vrow = *reinterpret_cast<const uint4*>(Vh + b * sb + h * sh + (long long)toks[s] * sn + c * VEC);
    __syncthreads();
    if (s < nt) {
      float out[VEC];
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        const uint32_t m = src[c * VEC + k];
        out[k] = (m & 0x8000u) ? l_dom[s][m & 0x7FFFu] : l_nd[s][m];
      }
      const size_t o = ((size_t)row * count + j0 + s) * D + c * VEC;
      *reinterpret_cast<uint4*>(KT + o) = *reinterpret_cast<const uint4*>(out);
      *reinterpret_cast<uint4*>(VT + o) = vrow;
    }
    // the next round writes toks before its first barrier and l_nd, l_dom behind it: toks is not read past the
    // barrier above, and every thread is past its reads of l_nd and l_dom when it reaches the next one
  }
}

// bf16 caches: gather, Combine and attention in one kernel, on the link's time: while some waves wait for their
// rows, others rebuild keys and attend.  1-D grid of rows * n_splits workgroups, 4 waves each; a wave takes every
// fourth tile of 16 list entries of its workgroup's part of the list and has one tile's rows outstanding (a
// tile is 16 x (512 - 4F) bytes, 7 KB at F = 16; under load its reads take about 15 us, rebuilding and
// attending 2: no second tile in flight is needed).
//   loads     V rows as the tiles want them (lane (lo, hi): 16 bytes of rows 4hi .. 4hi+3); the non-dominant
//             parts, which lie back to back in units of 16 bytes (WIDE: F a multiple of 4) or 4 bytes, lane after
//             lane; the dominant pairs from the Kp planes in HBM (lane: entry lo, planes hi, hi + 4, ..);
//   Combine   the parts side by side in LDS, from where each lane picks the 32 head dims of its four K chunks
//             by a map that stays in registers; K and V rows also go to the stage;
//   attend    mfma_tile.h; partials and the merge by the row's last workgroup as in attend.hip.
// Measured (8 rows, N = 32768, 2048 selected, F = 16): the step 189.4 us with the append, the gather (162 us) and
// the attention as kernels of their own, 182.5 us like this; the same from 16 to 64 workgroups.
constexpr int kOffPitch = 65;   // words of one entry in LDS: odd, so 16 entries at one offset are 16 banks
template <int G, bool WIDE>
__global__ __launch_bounds__(256) void offload_attend_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ Kp, const uint16_t* __restrict__ Knd,
    const uint16_t* __restrict__ Vh, const int32_t* __restrict__ fc_idx, const int32_t* __restrict__ T,
    uint16_t* __restrict__ KT, uint16_t* __restrict__ VT, float* __restrict__ O, RowCtl* __restrict__ ctl,
    float* __restrict__ part_acc, float* __restrict__ part_ml, int rows, int n_splits, uint32_t m_splits,
    int tiles_per_split, int Hkv, uint32_t m_hkv, int F, int n_cap, int n_ctx, int count, long long sb, long long sh, long long sn, int pairing,
    float scale_log2e) {
  constexpr int D = kHeadDim;
  constexpr int ACC_BYTES = 4 * G * D * 4;
  constexpr int MERGE_BYTES = 8192 + G * kMaxSplitsLds * 4;
  __shared__ __align__(16) unsigned char big[ACC_BYTES > MERGE_BYTES ? ACC_BYTES : MERGE_BYTES];
  __shared__ uint32_t raw[4][16][kOffPitch];      // per wave: 64 - F words of non-dominant dims, F dominant pairs
  __shared__ uint16_t src[D];
  __shared__ uint8_t is_dom[D];
  __shared__ float sm_m[4][G], sm_l[4][G];
  __shared__ float red[G];
  __shared__ uint32_t ticket;
  __shared__ __align__(16) float scs[4][16];
  float (*sm_o)[G][D] = reinterpret_cast<float (*)[G][D]>(big);
  float* wsm = reinterpret_cast<float*>(big + 8192);

  int row, split;
  row_slice_of_block(rows, n_splits, m_splits, row, split);
  int b, h;
  head_of_row(row, Hkv, m_hkv, b, h);
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int lo = lane & 15, hi = lane >> 4;
  const int n_tiles = (count + 15) >> 4;
  const int t1 = min(n_tiles, (split + 1) * tiles_per_split);
  const int W = D / 2 - F;                        // words of an entry's non-dominant part

  const int32_t* Trow = T + (size_t)row * count;
  // a stray index can never become a stray address: entries are clamped to the cache
  auto token_of = [&](int tile) { return min(max(Trow[min(16 * tile + lo, count - 1)], 0), n_ctx - 1); };
  int tile_no = split * tiles_per_split + wave;
  int tok = token_of(min(tile_no, n_tiles - 1));
  MfmaTile<G> tile;
  tile.load_q(q + ((size_t)row * G) * D, lo, hi);
  tile.reset();
  build_dim_map(fc_idx + h * F, F, pairing, src, is_dom);
  uint32_t pick[4][2];                            // where dims 8 (hi + 4i) + k of an entry lie: element numbers, a byte each
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t m = src[8 * (hi + 4 * i) + k];
      const uint32_t e = (m & 0x8000u) ? (m & 0x7fffu) + 2 * W : m;
      pick[i][k >> 2] = k & 3 ? pick[i][k >> 2] | (e << (8 * (k & 3))) : e;
    }

  const uint16_t* Vb = Vh + b * sb + h * sh + 8 * lo;
  const uint32_t* ndp = reinterpret_cast<const uint32_t*>(Knd) + (size_t)row * n_cap * W;
  const uint32_t* kpp = reinterpret_cast<const uint32_t*>(Kp) + ((size_t)row * F) * n_cap;
  constexpr int UW = WIDE ? 4 : 1;                // words per unit
  constexpr int NR = 16 / UW;                     // most units per lane
  const int per = W / UW, units = 16 * per;
  const uint32_t inv = per ? (65536u + (uint32_t)per - 1) / (uint32_t)per : 0u;   // i / per = i * inv >> 16 for i < 1024

  for (; tile_no < t1; tile_no += 4) {
    TileKV<uint16_t> kv;
    uint32_t nd[NR][UW], dom[16];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      kv.vr[e] = *reinterpret_cast<const uint4*>(Vb + (long long)__shfl(tok, 4 * hi + e) * sn);
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (64 * i < units) {
        const int u = min(64 * i + lane, units - 1);
        const int r = (int)((uint32_t)u * inv >> 16);
        const uint32_t* p = ndp + (size_t)__shfl(tok, r) * W + (u - r * per) * UW;
        if constexpr (WIDE) {
          const uint4 x = *reinterpret_cast<const uint4*>(p);
          nd[i][0] = x.x; nd[i][1] = x.y; nd[i][2] = x.z; nd[i][3] = x.w;
        } else {
          nd[i][0] = *p;
        }
      }
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (4 * u < F) dom[u] = kpp[(size_t)min(4 * u + hi, F - 1) * n_cap + tok];
    const int tok_next = token_of(min(tile_no + 4, n_tiles - 1));

#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (4 * u < F && 4 * u + hi < F) raw[wave][lo][W + 4 * u + hi] = dom[u];
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (64 * i < units) {
        const int u = min(64 * i + lane, units - 1);      // (lanes beyond the last unit rewrite it)
        const int r = (int)((uint32_t)u * inv >> 16);
#pragma unroll
        for (int k = 0; k < UW; ++k) raw[wave][r][(u - r * per) * UW + k] = nd[i][k];
      }
    // same wave writes and reads: LDS operations of a wave complete in order; the fences only keep the
    // compiler from moving the accesses across
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint16_t* mine = reinterpret_cast<const uint16_t*>(&raw[wave][lo][0]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = mine[(pick[i][k >> 2] >> (8 * (k & 3))) & 127u];
      kv.kc[i] = make_uint4(x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16), x[6] | (x[7] << 16));
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();   // read before the next tile overwrites it
    const int j0 = 16 * tile_no;
    const size_t o = ((size_t)row * count + j0) * D;
    if (j0 + lo < count) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<uint4*>(KT + o + (size_t)lo * D + 8 * (hi + 4 * i)) = kv.kc[i];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (j0 + 4 * hi + e < count) *reinterpret_cast<uint4*>(VT + o + (size_t)(4 * hi + e) * D + 8 * lo) = kv.vr[e];
    float sv[4];
    tile.logits(kv, scale_log2e, sv);
    bool valid[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) valid[e] = j0 + 4 * hi + e < count;
    tile.accumulate(kv, sv, valid, &scs[wave][0], lo, hi);
    tok = tok_next;
  }
  tile.finish(&sm_m[wave][0], &sm_l[wave][0], &sm_o[wave][0][0], lo, hi);
  __syncthreads();

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
  publish_barrier();
  if (t == 0) ticket = atomicAdd(&ctl[row].done_att, 1u);
  __syncthreads();
  if (ticket != (uint32_t)n_splits - 1u) return;
  if (t == 0) ctl[row].done_att = 0;
  combine_row<G>(part_acc, part_ml, O, row, n_splits, n_splits, wsm, red, reinterpret_cast<float*>(big));
}

hipError_t launch_offload_split(const fasa_shape& s, const void* K, const int32_t* fc_idx, void* Kp,
                                void* Knd, int n_begin, int n_end, hipStream_t st) {
  const int rows = s.batch * s.n_kv_heads;
  dim3 grid((n_end - n_begin + kOffTile - 1) / kOffTile, rows), block(256);
  if (s.dtype == FASA_BF16)
    return launch("fasa_offload_split", offload_split_kernel<uint16_t>, grid, block, st,
                  (const uint16_t*)K, fc_idx, (uint16_t*)Kp, (uint16_t*)Knd, s.n_kv_heads, s.n_fc,
                  s.n_cap, n_begin, n_end, (long long)s.kv_stride_b, (long long)s.kv_stride_h,
                  (long long)s.kv_stride_n, s.pairing);
  return launch("fasa_offload_split", offload_split_kernel<float>, grid, block, st, (const float*)K,
                fc_idx, (float*)Kp, (float*)Knd, s.n_kv_heads, s.n_fc, s.n_cap, n_begin, n_end,
                (long long)s.kv_stride_b, (long long)s.kv_stride_h, (long long)s.kv_stride_n, s.pairing);
}

hipError_t launch_offload_gather(const fasa_shape& s, const void* Kp, const void* Knd, const void* Vh,
                                 const int32_t* fc_idx, const int32_t* T, void* KT, void* VT,
                                 hipStream_t st) {
  const int rows = s.batch * s.n_kv_heads;
  const int count = s.budget < s.n_ctx ? s.budget : s.n_ctx;
  const int wgs = kOffInFlight / (8 * 1024);              // 8 tokens of at most 1 KB each per workgroup
  const int want = wgs / rows > 1 ? wgs / rows : 1, most = (count + 7) / 8;
  return launch("fasa_offload_gather", offload_gather_kernel, dim3(want < most ? want : most, rows), dim3(256), st,
                (const float*)Kp, (const float*)Knd, (const float*)Vh, fc_idx, T, (float*)KT, (float*)VT, s.n_kv_heads,
                s.n_fc, s.n_cap, s.n_ctx, count, (long long)s.kv_stride_b, (long long)s.kv_stride_h,
                (long long)s.kv_stride_n, s.pairing);
}

template <int G>
static hipError_t launch_offload_attend_g(const fasa_shape& s, int n_splits, int tiles_per_split, const void* q,
                                          const void* Kp, const void* Knd, const void* Vh, const int32_t* fc_idx,
                                          const int32_t* T, void* KT, void* VT, float* O, RowCtl* ctl, float* part_acc,
                                          float* part_ml, hipStream_t st) {
  const int rows = s.batch * s.n_kv_heads;
  const int count = s.budget < s.n_ctx ? s.budget : s.n_ctx;
  return launch("fasa_offload_attend", s.n_fc % 4 == 0 ? offload_attend_kernel<G, true> : offload_attend_kernel<G, false>,
                dim3(rows * n_splits), dim3(256), st, (const uint16_t*)q, (const uint16_t*)Kp, (const uint16_t*)Knd,
                (const uint16_t*)Vh, fc_idx, T, (uint16_t*)KT, (uint16_t*)VT, O, ctl, part_acc, part_ml, rows, n_splits,
                div_magic(n_splits, (long long)rows * n_splits), tiles_per_split, s.n_kv_heads, div_magic(s.n_kv_heads, rows), s.n_fc, s.n_cap, s.n_ctx, count, (long long)s.kv_stride_b,
                (long long)s.kv_stride_h, (long long)s.kv_stride_n, s.pairing, 1.4426950408889634f / sqrtf((float)s.head_dim));
}

hipError_t launch_offload_attend(const fasa_shape& s, int max_splits, const void* q, const void* Kp, const void* Knd,
                                 const void* Vh, const int32_t* fc_idx, const int32_t* T, void* KT, void* VT, float* O,
                                 RowCtl* ctl, float* part_acc, float* part_ml, hipStream_t st) {
  const int rows = s.batch * s.n_kv_heads;
  const int count = s.budget < s.n_ctx ? s.budget : s.n_ctx;
  const int tiles = (count + 15) / 16;
  const int wave_bytes = 16 * (4 * kHeadDim - 4 * s.n_fc);                   // one tile's rows of both kinds
  int n_splits = (kOffInFlight / wave_bytes / 4 + rows - 1) / rows;          // 4 waves per workgroup
  if (n_splits > (tiles + 3) / 4) n_splits = (tiles + 3) / 4;
  if (n_splits > max_splits) n_splits = max_splits;
  if (n_splits > kMaxSplitsLds) n_splits = kMaxSplitsLds;
  if (n_splits < 1) n_splits = 1;
  const int per = (tiles + n_splits - 1) / n_splits;
  n_splits = (tiles + per - 1) / per;
  switch (s.n_q_heads / s.n_kv_heads) {
#define FASA_G(G) case G: return launch_offload_attend_g<G>(s, n_splits, per, q, Kp, Knd, Vh, fc_idx, T, KT, VT, O, ctl, part_acc, part_ml, st)
    FASA_G(1); FASA_G(2); FASA_G(3); FASA_G(4); FASA_G(5); FASA_G(6); FASA_G(7); FASA_G(8);
#undef FASA_G
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fasa
