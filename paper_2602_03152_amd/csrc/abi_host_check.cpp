// Host-side exerciser of the C ABI for sanitizer builds (paper_2602_03152_amd/build.py --sanitize):
// walks every entry point's argument validation and the pure host functions - workspace sizes and
// launch plans over a sweep of shapes, the dominant-list checker, the dominant-FC choice - without a
// GPU.  Compiled together with the library's sources with AddressSanitizer and
// UndefinedBehaviorSanitizer on the host side (device code is untouched); any report fails the run.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "fasa.h"
#include "fasa_internal.h"
#include "row_list.h"
#include "select_common.h"

#define EXPECT(cond) do { if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); return 1; } } while (0)

static fasa_shape shape(int batch, int hq, int hkv, int f, int n, int cap, int budget, int dtype = FASA_BF16) {
  fasa_shape s{};
  s.batch = batch; s.n_q_heads = hq; s.n_kv_heads = hkv; s.head_dim = 128; s.n_fc = f; s.n_ctx = n; s.n_cap = cap;
  s.budget = budget; s.dtype = dtype; s.pairing = FASA_PAIR_ROTATE_HALF;
  s.kv_stride_n = 128; s.kv_stride_h = (int64_t)cap * 128; s.kv_stride_b = (int64_t)hkv * cap * 128;
  return s;
}

int main() {
  void* A = reinterpret_cast<void*>(0x10000);   // a fake aligned "device pointer": validation must fail before it is touched
  // ---- workspace sizes and launch plans over a sweep of shapes (pure host arithmetic) ----
  size_t checked = 0;
  for (int batch : {1, 2, 3, 8, 16, 64})
    for (int hkv : {1, 2, 3, 4, 8})
      for (int g : {1, 2, 4, 7, 8})
        for (int n : {1, 2, 63, 64, 1000, 4096, 32768, 33279, 131072, (1 << 20) + 77})
          for (int budget : {1, 2, 255, 2048, 6193, 1 << 21}) {
            const int cap = (n + 63) / 64 * 64;
            fasa_shape s = shape(batch, hkv * g, hkv, 16, n, cap, budget);
            const size_t b = fasa_workspace_bytes(&s);
            EXPECT(b > 0 && b % 256 == 0);
            EXPECT(fasa_offload_stage_bytes(&s) % 256 == 0);
            // argument validation of the step with too small a workspace, then with a null pointer
            EXPECT(fasa_decode_step(&s, A, A, A, A, (const int32_t*)A, nullptr, nullptr, (float*)A, (int32_t*)A, (float*)A, A,
                                    b / 2, nullptr) == FASA_EWORKSPACE);
            EXPECT(fasa_workspace_init(&s, A, b - 1, nullptr) == FASA_EWORKSPACE);
            EXPECT(fasa_decode_step(&s, nullptr, A, A, A, (const int32_t*)A, nullptr, nullptr, (float*)A, (int32_t*)A,
                                    (float*)A, A, b, nullptr) == FASA_EINVAL);
            ++checked;
          }
  // ---- the step's forms: every plan is one the kernels are built for ----
  int forms[3] = {0, 0, 0}, lists = 0, topks = 0, asked = 0;
  for (int dtype : {FASA_BF16, FASA_F32})
    for (int rows : {1, 3, 8, 64, 65, 72, 128, 256, 257, 512, 4096})
      for (int g : {1, 2, 3, 4, 5, 8})
        for (int n : {1, 257, 1024, 1025, 2048, 2049, 4097, 5119, 5120, 8192, 8193, 16385, 32768, 32769, 65536, 140000, 1 << 20, (1 << 20) + 64})
          for (int budget : {1, 63, 64, 320, 321, 512, 513, 1024, 1025, 6000}) {
            const int cap = (n + 63) / 64 * 64, bsel = budget < n ? budget : n, per = dtype == FASA_BF16 ? 2048 : 1024;
            const fasa_shape s = shape(rows, g, 1, 16, n, cap, budget, dtype);
            const fasa::StepForm form = fasa::plan_step(s, fasa::kNoPaging);
            ++forms[form];
            if (form == fasa::kStepOne)     // the row fits the last workgroup's registers; several float32 slices: one head only
              EXPECT(bsel <= fasa::kStepMaxBudget && n <= 8192 && (dtype == FASA_BF16 || n <= per || g == 1));
            if (form == fasa::kStepRow) EXPECT(bsel <= fasa::kStepMaxBudget && dtype == FASA_F32 && g <= 4);
            // the lists' loads fit the threads that make them, and the shares cover the budget
            const fasa::ListPlan l = fasa::plan_list(s, fasa::kNoPaging, 256);
            if (l.quads) {
              const int nsegs = (n + 255) / 256, share = ((bsel + l.nwgs - 1) / l.nwgs + 15) / 16 * 16, q = l.quads;
              EXPECT(dtype == FASA_BF16 && nsegs <= 2048);
              EXPECT((q == 1 || q == 2 || q == 3 || q == 4 || q == 6 || q == 8) && l.nwgs >= 1 &&
                     l.nwgs <= 64 && share <= 2048 && (long long)share * l.nwgs >= bsel && share * (l.nwgs - 1) < bsel);
              // 512 threads hold four places a quad; keys and token bytes lie in 8 bytes per token of capacity
              const int room = fasa::list_room(bsel, n), one = fasa::list_places(n, bsel, q, false), own = fasa::list_places(n, bsel, q, true);
              EXPECT(room >= 8 && room <= 256 && room % 4 == 0 && one == nsegs * room);
              for (int places : {one, own})
                EXPECT(places % 4 == 0 && places >= one && places <= q * 512 * 4 && places <= nsegs * 256);
              if (form == fasa::kStepNone && bsel < n) {          // (where it is asked: no row of fewer than 257 tokens)
                EXPECT(5ll * one <= 8ll * cap && 5ll * own <= 8ll * cap);
                ++asked;
              }
              ++lists;
            }
            const fasa::TopkPlan k = fasa::plan_topk(n, bsel);
            if (k.quads) {
              const int nsegs = (n + 255) / 256, places = nsegs * fasa::list_room(bsel, n);
              EXPECT(bsel < n && nsegs <= 2048 && k.quads <= 4 && places <= k.quads * 512 * 4);
              if (n > 2048) EXPECT(5ll * places <= 8ll * cap);
              ++topks;
            }
            const fasa::FusePlan p = fasa::plan_fused(s, true);
            if (p.tpb) EXPECT(p.slice_len <= p.tpb && p.nslices <= 256 && (long long)p.nslices * p.slice_len >= n &&
                              (long long)(p.nslices - 1) * p.slice_len < n);
          }
  EXPECT(lists > 0 && topks > 0 && asked > 0 && forms[fasa::kStepNone] > 0 && forms[fasa::kStepOne] > 0 && forms[fasa::kStepRow] > 0);
  // ---- eight waves per compute unit: the splits cover the tokens, the workspace holds them, and they fill their rounds ----
  for (int rows = 1; rows <= 600; ++rows)
    for (int count : {1, 17, 700, 1500, 3000, 4096, 8192, 30001, 131072}) {
      const fasa::AttendPlan p = fasa::plan_attend_wide(rows, count), most = fasa::plan_attend(rows, count, 4);
      EXPECT(p.n_splits >= 1 && p.n_splits <= most.n_splits && (long long)p.n_splits * p.tok_per_split >= count &&
             (long long)(p.n_splits - 1) * p.tok_per_split < count);
      const long long wgs = (long long)rows * p.n_splits, rounds = (wgs + 255) / 256;
      if (rows > 128 && count >= 3000 && most.n_splits >= 4) EXPECT(wgs * 10 >= rounds * 256 * 6);
    }
  // ---- the threshold's range only narrows, whatever key the threshold bin holds (a NaN's is the largest there is) ----
  for (uint32_t key : {0u, 1u, 0x007fffffu, 0x3d3dffffu, 0x7fffffffu, 0x80000000u, 0xbf800000u, 0xff7fffffu, 0xff800000u, 0xffc00000u, 0xffffffffu})
    for (uint32_t from : {1u, 0x007fffffu, 0x3d3dffffu, 0x3fbfffffu, 0x7fffffffu, 0x80000001u, 0xbe4ccccdu, 0xc0000000u, 0xff800000u})
      for (int first : {22, 23, 16, 1}) {
        if (from > key) continue;
        uint32_t klo = from, khi = 0xffffffffu;
        int shift = first;
        for (int pass = 0; pass < 6 && klo != khi; ++pass) {
          const uint32_t d = (key - klo) >> shift, bin = d < 1023u ? d : 1023u, lo = klo, hi = khi;
          fasa::narrow_range(klo, khi, bin, shift);
          EXPECT(lo <= klo && klo <= key && key <= khi && khi <= hi);
          shift = 22 - __builtin_clz((khi - klo) | 1u);
          if (shift < 0) shift = 0;
        }
      }
  // the same among 512 bins, the first of them up to the largest finite score's key (selection out of lists); after a bin the search
  // may go on with the range of the keys in it
  for (uint32_t key : {1u, 0x007fffffu, 0x3d3dffffu, 0x7fffffffu, 0x80000000u, 0xbf800000u, 0xc0400001u, 0xff7fffffu, 0xff800000u, 0xffffffffu})
    for (uint32_t from : {1u, 0x007fffffu, 0x3d3dffffu, 0x7fffffffu, 0x80000001u, 0xbe4ccccdu, 0xc0000000u, 0xff800000u})
      for (uint32_t top : {0u, 0x3fbfffffu, 0x80000001u, 0xbf800000u, 0xc0400000u, 0xff7fffffu}) {
        if (from > key) continue;
        uint32_t klo = from, khi = 0xffffffffu;
        const uint32_t span = top > from ? top - from : 0u;
        int shift = span ? 23 - __builtin_clz(span) : 0, passes = 0;
        if (shift < 0) shift = 0;
        EXPECT((span >> shift) < (uint32_t)fasa::kListBins);
        while (klo != khi) {
          const uint32_t d = (key - klo) >> shift, last = fasa::kListBins - 1, bin = d < last ? d : last, lo = klo, hi = khi;
          fasa::narrow_range<fasa::kListBins>(klo, khi, bin, shift);
          EXPECT(lo <= klo && klo <= key && key <= khi && khi <= hi && ++passes < 8);
          shift = klo == khi ? 0 : 23 - __builtin_clz(khi - klo);
          if (shift < 0) shift = 0;
        }
      }
  // ---- places of a segment: the kernels' quotient, whose reciprocal is off by an ulp at most, is the whole one below 256 ----
  for (int segs = 1; segs <= 2048; ++segs)
    for (int places = 4; places <= 16384 && places < 256 * segs; places += places < 64 || places > 16320 ? 4 : 92)
      for (float off : {-1.2e-7f, 0.f, 1.2e-7f}) {
        const float r = 1.0f / (float)segs, q = ((float)places + 0.5f) * (r + r * off);
        EXPECT((int)q == places / segs);
      }
  // ---- quotients by multiplication: exact up to the bound that the factor was made for, and no factor where they would not be ----
  for (long long d : {1ll, 2ll, 3ll, 5ll, 7ll, 8ll, 31ll, 64ll, 129ll, 256ll, 1000ll, 1023ll, 2048ll, 4097ll, 8191ll, 8192ll, 46340ll, 65535ll})
    for (long long most : {d, 2 * d + 1, 1000 * d, (1ll << 31) / d - 1, (1ll << 31) / d, (1ll << 31) / d + 1, (1ll << 31) - 1}) {
      const uint32_t m = fasa::div_magic((int)d, most);
      EXPECT((m != 0) == (most * d < (1ll << 31)));
      if (!m) continue;                                        // (fast_div divides)
      for (long long k : {0ll, 1ll, 2ll, 3ll, most / d / 3, most / d / 2, most / d - 1, most / d})
        for (long long n : {k * d - 1, k * d, k * d + 1, k * d + d - 1, most - 1, most}) {
          if (n < 0 || n > most) continue;
          EXPECT((long long)(((unsigned long long)((uint32_t)n << 1) * m) >> 32) == n / d);
        }
    }
  // ---- bins of scores held in registers: monotone, whatever the ends are; and where one score lies far from all others few share the B-th's bin, as if it did not ----
  {
    const float inf = __builtin_inff(), most = 3.4028235e38f;
    const std::vector<float> xs = {-inf, -most, -1e30f, -100.f, -20.5f, -20.f, -1e-3f, -1e-44f, 0.f, 1e-44f, 1e-38f, 1e-3f, 19.f, 20.f, 20.000002f, 64.f, 1e4f, 1e30f, 1.7e38f, most, inf};
    for (float lo : xs)
      for (float mid : xs)
        for (float hi : xs) {
          if (!(lo <= mid && mid <= hi)) continue;
          const fasa::LinBins lin = fasa::lin_bins(lo, mid, hi);
          const fasa::LogBins log = fasa::log_bins(lo, mid, hi);
          uint32_t last_lin = 0, last_log = 0;
          for (float x : xs) {
            const uint32_t a = fasa::held_bin(lin, x), b = fasa::held_bin(log, x);
            EXPECT(last_lin <= a && a < (uint32_t)fasa::kListBins && last_log <= b && b < (uint32_t)fasa::kListBins);
            last_lin = a;
            last_log = b;
          }
        }
    constexpr int NT = 512;
    uint32_t seed = 12345u;
    auto normal = [&]() {
      float z = -6.f;
      for (int i = 0; i < 12; ++i) { seed = seed * 1664525u + 1013904223u; z += (float)(seed >> 8) * 0x1p-24f; }
      return z;
    };
    for (int n : {257, 600, 1531, 2048, 4096, 6000, 8192})
      for (int b : {16, n / 8, n / 2})
        for (float far : {0.f, 1e4f, 1e12f, 3e38f, inf, -1e4f, -1e12f, -3e38f, -inf}) {
          if (far != 0.f && n < fasa::kHeldPairs) continue;
          std::vector<float> x(n);
          for (float& v : x) v = 20.f * normal();
          if (far != 0.f) x[n / 3] = far;
          const bool few = b <= (NT < n / 4 ? NT : n / 4);
          float hi_t[NT], lo_t[NT], h[8], l[8];
          for (int t = 0; t < NT; ++t) { hi_t[t] = -inf; lo_t[t] = inf; }
          for (int i = 0; i < n; ++i) {
            const int t = i / 4 % NT;
            if (x[i] > hi_t[t]) hi_t[t] = x[i];
            if (x[i] < lo_t[t]) lo_t[t] = x[i];
          }
          for (int w = 0; w < 8; ++w) {
            h[w] = -inf; l[w] = inf;
            for (int t = 64 * w; t < 64 * w + 64; ++t) {
              if (hi_t[t] > h[w]) h[w] = hi_t[t];
              const float v = few ? (4 * t < n ? hi_t[t] : inf) : lo_t[t];
              if (v < l[w]) l[w] = v;
            }
          }
          float lo = inf, low = inf, mid = -inf, hi = -inf;
          for (int w = 0; w < 8; w += 2) {
            hi = std::max({hi, h[w], h[w + 1]});
            lo = std::min({lo, l[w], l[w + 1]});
            mid = std::max(mid, std::min(h[w], h[w + 1]));
            low = std::min(low, std::max(l[w], l[w + 1]));
          }
          if (low == inf) low = lo;
          const bool pairs = n >= fasa::kHeldPairs;
          const fasa::LinBins bins = fasa::lin_bins(few || !pairs ? lo : low, pairs ? mid : hi, hi);
          std::vector<int> count(fasa::kListBins);
          for (float v : x)
            if (v >= (few ? lo : -inf)) ++count[fasa::held_bin(bins, v)];
          int bin = fasa::kListBins - 1, above = 0;
          while (bin > 0 && above + count[bin] < b) above += count[bin--];
          EXPECT(above + count[bin] >= b && count[bin] <= fasa::kHeldMany);
        }
  }
  // ---- bad shapes ----
  {
    fasa_shape s = shape(1, 32, 8, 16, 1000, 1024, 100);
    fasa_shape t = s; t.n_cap = 1000;          EXPECT(fasa_workspace_bytes(&t) == 0);
    t = s; t.n_ctx = 2000;                     EXPECT(fasa_workspace_bytes(&t) == 0);
    t = s; t.budget = 0;                       EXPECT(fasa_workspace_bytes(&t) == 0);
    t = s; t.head_dim = 64;                    EXPECT(fasa_topk(&t, (const float*)A, (int32_t*)A, A, 1 << 30, nullptr) == FASA_EUNSUPPORTED);
    t = s; t.n_q_heads = 30;                   EXPECT(fasa_score(&t, A, A, (const int32_t*)A, (float*)A, nullptr) == FASA_EINVAL);
    t = s; t.pairing = 7;                      EXPECT(fasa_score(&t, A, A, (const int32_t*)A, (float*)A, nullptr) == FASA_EINVAL);
    EXPECT(fasa_workspace_bytes(nullptr) == 0);
    EXPECT(fasa_pack_kcache(&s, A, (const int32_t*)A, A, 5, 4, nullptr) == FASA_EINVAL);
    EXPECT(fasa_pack_kcache(&s, A, (const int32_t*)A, A, 7, 7, nullptr) == FASA_OK);     // empty range: nothing launched
    EXPECT(fasa_decode_step_static(&s, nullptr, A, A, A, (const int32_t*)A, nullptr, nullptr, (float*)A, (int32_t*)A,
                                   (float*)A, nullptr) == FASA_EINVAL);
    fasa_shape big = shape(64, 32, 8, 16, 65536, 65536, 4096);
    EXPECT(fasa_decode_step_static(&big, A, A, A, A, (const int32_t*)A, nullptr, nullptr, (float*)A, (int32_t*)A, (float*)A,
                                   nullptr) == FASA_EWORKSPACE);
    fasa_paging pg{(const int32_t*)A, 4, 16, 100, 0};
    EXPECT(fasa_pack_kcache_paged(&s, &pg, A, (const int32_t*)A, A, 0, 65, nullptr) == FASA_EINVAL);   // table ends at 64
    pg.page_size = 12;
    EXPECT(fasa_pack_kcache_paged(&s, &pg, A, (const int32_t*)A, A, 0, 16, nullptr) == FASA_EINVAL);   // not a power of two
    EXPECT(fasa_calibration_workspace_bytes(&s, 0) == 0);
    EXPECT(fasa_calibration_workspace_bytes(&s, 64) > 0);
  }
  // ---- dominant-list checker and dominant-FC choice (host arrays) ----
  {
    fasa_shape s = shape(1, 8, 2, 4, 100, 128, 10);
    std::vector<int32_t> fc = {0, 5, 63, 7, 1, 2, 3, 4};
    EXPECT(fasa_validate_fc_idx(&s, fc.data()) == FASA_OK);
    fc[3] = 64;  EXPECT(fasa_validate_fc_idx(&s, fc.data()) == FASA_EINVAL);
    fc[3] = 5;   EXPECT(fasa_validate_fc_idx(&s, fc.data()) == FASA_EINVAL);   // twice in one head
    fc[3] = -1;  EXPECT(fasa_validate_fc_idx(&s, fc.data()) == FASA_EINVAL);
    s.pairing = FASA_PAIR_LIST;
    std::vector<int32_t> pairs = {0, 64, 1, 127, 2, 3, 9, 10,  5, 6, 7, 8, 100, 101, 11, 12};
    EXPECT(fasa_validate_fc_idx(&s, pairs.data()) == FASA_OK);
    pairs[15] = 128; EXPECT(fasa_validate_fc_idx(&s, pairs.data()) == FASA_EINVAL);
    s.pairing = FASA_PAIR_ROTATE_HALF;
    std::vector<float> ca(2 * 64);
    for (int i = 0; i < 128; ++i) ca[i] = (float)((i * 37) % 64) / 64.f;
    std::vector<int32_t> out(8, -1);
    EXPECT(fasa_select_dominant_fcs(&s, ca.data(), out.data()) == FASA_OK);
    EXPECT(fasa_validate_fc_idx(&s, out.data()) == FASA_OK);
    EXPECT(fasa_select_dominant_fcs(&s, nullptr, out.data()) == FASA_EINVAL);
  }
  for (int c : {0, -1, -2, -3, -4, -99}) EXPECT(fasa_strerror(c) != nullptr);
  char name[8];
  EXPECT(fasa_profile_entry(0, name, sizeof name, nullptr, nullptr) == FASA_EINVAL);
  std::printf("abi_host_check: %zu shapes, all checks passed\n", checked);
  return 0;
}
