// Host check of the span planner (kf_api.cpp built against the HIP test
// double): over random launches on devices of 8 to 1024 compute units, a span
// plan's workspace fits both a workspace sized by the query for any table at
// least as large and the library's scratch array, its regions do not meet,
// and the record places of the cut routes are distinct and inside the plan.
#include <stdio.h>

#include <algorithm>
#include <random>
#include <vector>

#include "kf.h"
#include "kf_internal.h"

static int g_cus = 256;
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = g_cus; return hipSuccess; }
namespace kf {
hipError_t launch_append(const AppendArgs&, bool, hipStream_t) { return hipSuccess; }
static PartialArgs g_launch;  // the last launch
hipError_t launch_partial(const PartialArgs& a, bool, hipStream_t) { g_launch = a; return hipSuccess; }
hipError_t launch_merge(const MergeArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_gather(const PartialArgs&, bool, int, int, void*, void*, hipStream_t) { return hipSuccess; }
hipError_t scratch_address(void** out) { *out = nullptr; return hipSuccess; }
}  // namespace kf

static std::mt19937 rng(7);
static int64_t rnd(int64_t lo, int64_t hi) { return std::uniform_int_distribution<int64_t>(lo, hi)(rng); }

#define CHECK(c)                                                   \
  do {                                                             \
    if (!(c)) {                                                    \
      printf("line %d: %s (R=%d H=%d G=%d P=%d fp8=%d wg=%d)\n", __LINE__, #c, R, H, G, maxp, fp8, p.wg_cols); \
      return 1;                                                    \
    }                                                              \
  } while (0)

// A merge that combines records has one workgroup per (sequence, head): a
// sequence beside others of at least one route each holds no more rows than the
// workgroup keeps in LDS, and there is a wave for every 64 rows.
static int merges() {
  for (int n = 1; n <= 65535; n += n < 300 ? 1 : 97)
    for (int r = n; r <= 4 * n + 64 && r <= 65535; ++r)
      if (kf::merge_combines(r, n, 1) && (r - (n - 1) > kf::kLdsRows || (r + 63) / 64 > n)) {
        printf("%d routes of %d sequences combined in the merge\n", r, n);
        return 1;
      }
  return 0;
}

// Tables on either side of the launch rule's lines (256 compute units).
static int rules() {
  struct {
    int R, H, G, pages, ids;
    bool fp8, span;
  } t[] = {
      {192, 32, 1, 81, 8400, false, true},   // whole units, long reserves beside short ones
      {64, 8, 4, 64, 3072, false, false},    // whole units, near their longest: 16 pages a slot
      {64, 8, 4, 94, 6016 - 1920, false, true},      // 30 pages a slot
      {64, 8, 4, 94, 6016 - 1919, false, false},
      {64, 8, 16, 125, 8000 - 3200, false, true},    // 50 with 16 query heads per KV head
      {64, 8, 16, 125, 8000 - 3199, false, false},
      {101, 8, 5, 65, 5584, false, true},    // 808 units: a compute unit holds four
      {101, 8, 16, 65, 5584, false, false},
      {65, 8, 4, 76, 4200, false, false},    // 520: all but eight hold two
      {237, 16, 1, 27, 5700, true, true},    // fp8: wherever ragged
      {237, 16, 1, 27, 5700, false, false},
      {64, 8, 4, 600, 20000, false, true},   // ragged and split
      {40, 8, 4, 500, 20000, false, true},   // 320 equal units in 3 ranges: 960 on 256 CUs
      {40, 8, 4, 500, 20000, true, false},
      {44, 8, 4, 500, 22000, true, false},   // 352 in 2: 704
      {50, 8, 4, 500, 25000, true, true},    // 400 in 5: 2000, more than four each
      {48, 8, 4, 500, 24000, false, false},  // 384 in 2: 768, three each
      {65, 8, 4, 500, 32500, true, true},    // 520 units: more than slots
      {827, 2, 16, 500, 200000, true, true},  // 16 query heads: the table fits LDS
      {828, 2, 16, 500, 200000, true, false},
      {1024, 2, 15, 500, 200000, true, true},
      {1025, 2, 4, 500, 200000, true, false},
  };
  for (const auto& c : t) {
    const kf::ChunkPlan plan =
        kf::plan_chunks(c.R, c.H, c.pages, kf::ragged_table(c.ids, c.R, c.pages), c.fp8, false);
    const bool got = kf::plan_span(c.R, c.H, c.G, c.pages, c.ids, c.fp8, false, plan, 512).wg_cols > 0;
    if (got != c.span) {
      printf("R=%d H=%d G=%d pages=%d ids=%d fp8=%d (plan %d ranges): span %d\n", c.R, c.H, c.G, c.pages,
             c.ids, c.fp8, plan.max_chunks, got);
      return 1;
    }
  }
  return 0;
}

int main(int argc, char** argv) {
  if (merges()) return 1;
  if (argc == 1 && rules()) return 1;
  g_cus = argc > 1 ? atoi(argv[1]) : 256;  // one device per process: the count is cached
  int spans = 0;
  for (int it = 0; it < 4000; ++it) {
    const int hs[] = {1, 2, 4, 8, 16, 32, 40, 600};
    const int R = (int)(rnd(0, 3) ? rnd(1, 300) : rnd(1, 1200)), H = hs[rnd(0, 7)], G = (int)rnd(1, 16);
    const int maxp = (int)(rnd(0, 3) ? rnd(1, 600) : rnd(1, 9000));
    const bool fp8 = rnd(0, 1), list = !rnd(0, 9);
    kf_shape s{1, G * H, H, KF_HEAD_DIM, KF_PAGE_SIZE, fp8 ? KF_KV_FP8_E4M3 : KF_KV_BF16, 10,
               (int)rnd(1, (int64_t)R * maxp), 0.1f, 0};
    const int64_t slots = 2 * (int64_t)g_cus;
    const kf::ChunkPlan c = kf::plan_chunks(R, H, maxp, kf::ragged_table(s.num_page_ids, R, maxp), fp8, list);
    const kf::SpanPlan p = kf::plan_span(R, H, G, maxp, s.num_page_ids, fp8, list, c, slots);
    // what the query says is what the launch does, with a workspace of the queried size
    int32_t wgs = -1;
    CHECK(kf_partial_attn_spans(&s, R, maxp, list, &wgs) == KF_OK && wgs == p.wg_cols);
    char* const at = reinterpret_cast<char*>((uintptr_t)1 << 30);
    int32_t* const i32 = reinterpret_cast<int32_t*>(at);
    float* const f32 = reinterpret_cast<float*>(at);
    const size_t ws = kf_partial_attn_workspace_bytes(&s, R, maxp);
    const int st =
        list ? kf_partial_attn_subset(&s, at, at, at, f32, f32, (kf_route*)at, R, i32, R, maxp, i32,
                                      f32, f32, at, ws, i32, nullptr)
             : kf_partial_attn(&s, at, at, at, f32, f32, (kf_route*)at, R, maxp, i32, f32, f32, at,
                               ws, i32, nullptr);
    CHECK(st == KF_OK && kf::g_launch.span_cols == wgs * kf::kWaves);
    if (!p.wg_cols) continue;
    ++spans;
    // two workgroups fit the 160 KiB of a compute unit
    CHECK(!list && R <= kf::kSpanRoutes &&
          2 * (kf::span_lds_bytes(G, R) + kf::kSpanStaticLds) <= 160 << 10);
    CHECK((int64_t)p.wg_cols * H <= std::max<int64_t>(slots, H));
    CHECK(p.total <= KF_SCRATCH_BYTES);
    CHECK(p.total <= kf_partial_attn_workspace_bytes(&s, R, maxp));
    CHECK(p.total <= kf_partial_attn_workspace_bytes(&s, R + (int)rnd(0, 50), maxp));
    const int64_t places = p.wg_cols + std::min(p.wg_cols, R), recs = places * H * G;
    CHECK((int64_t)p.ml_off >= R * 8 && (int64_t)(p.o_off - p.ml_off) >= recs * 8 &&
          (int64_t)(p.total - p.o_off) >= recs * kf::kDim * 4);
    // the kernel's columns over random route lengths
    std::vector<int> tiles(R);
    int64_t T = 0;
    for (int& t : tiles) T += t = rnd(0, 4) ? (int)rnd(0, maxp) : 0;
    const int64_t cols = std::max<int64_t>(1, std::min<int64_t>(p.wg_cols * kf::kWaves, T));
    if (!T) continue;
    const int64_t q = T / cols, rem = T % cols, edge = rem * (q + 1);
    auto of = [&](int64_t t) { return t < edge ? t / (q + 1) : rem + (t - edge) / q; };
    std::vector<char> used(places, 0);
    int64_t pre = 0;
    for (int u = 0; u < R; pre += tiles[u], ++u) {
      if (!tiles[u]) continue;
      const int64_t c0 = of(pre) / kf::kWaves, c1 = of(pre + tiles[u] - 1) / kf::kWaves;
      for (int64_t w = c0; c1 > c0 && w <= c1; ++w) {
        const int64_t at = w + std::min<int64_t>(u, c0);
        CHECK(at < places && !used[at]);
        used[at] = 1;
      }
    }
  }
  printf("span_plan ok: %d span launches\n", spans);
  return spans > 100 ? 0 : 1;
}
