// gfx950 kernels of the weightless attention node's decode step
// (KernelFlume, arXiv 2606.29207, Section 3.2 steps 3-4, Section 5.1):
//   append_kernel   -- tail append of the step's K/V token
//   partial_kernel  -- local attention over token-range routes -> (o, lse)
//   span_kernel     -- the same for ragged batches, cut into equal wave columns
//   order_kernel    -- dispatch order of a split launch of several rounds
//   combine_kernel  -- reduction of the records of split units and spans
//   merge_kernel    -- log-sum-exp merge of the partials of each sequence
//
// partial_kernel is HBM-bound (4 flop per KV byte at 4 query heads per KV
// head).  Four waves own a (route, KV head) unit -- or, when the host plans
// chunks, one of its ceil(pages / chunk_pages) page ranges: a 256-thread
// workgroup, two per CU, or one half of a 512-thread workgroup that holds
// two short unsplit bf16 units, one per CU.  Wave w takes tiles w, w+4, ... of
// the range, its full tiles taken from a per-route starting offset, so the
// summation order is fixed and results are bitwise reproducible (and the
// same for any placement of the pages).  Each wave streams tiles of 2 (bf16)
// or 4 (fp8) pages:
//   * lane (grp = lane/16, i = lane%16).  For q.K^T the MFMA A operand row i
//     is token (page i/4 of the tile, slot 4c + i%4) for c = 0..3, so the
//     16x16 result lands with lane (grp, head i) holding all 16 scores of
//     page grp of the tile.  Those are exactly the P^T values the same lane
//     feeds as the B operand of p.V, whose A operand is read straight from
//     the dimension-major V page (V^T rows are contiguous in slots): no LDS
//     or cross-lane traffic between the two products.
//   * both products use v_mfma_f32_16x16x32_bf16; query heads of the group
//     fill the N = 16 columns (G <= 16, the rest zero).
//   * p (fp32) enters p.V as bf16 hi + bf16 lo, two MFMAs, so the products
//     carry ~2^-17 relative error instead of bf16's 2^-9.
//   * all 32 loads of a tile are issued before any of its arithmetic, and
//     the page ids of the wave's next tile are fetched a tile ahead.
//   * softmax state per head is shared by the four lane groups (max reduced
//     across groups per tile), the running sum is kept per lane and reduced
//     once at the end; the four waves are combined through LDS.
// Workgroups never exchange data with each other inside a kernel: when a
// unit is chunked, the chunk partials go to the workspace and combine_kernel
// or a fused step's merge_kernel (the next launch on the stream) sums them in
// a fixed order, so results are deterministic.
#include <atomic>
#include <mutex>
#include <type_traits>

#include "kf_internal.h"


namespace kf {
namespace {

// Slice index of (page, KV head) in a pool: page-major pools are
// [num_pages][Hkv][...], head-major ones [Hkv][num_pages][...].
__device__ __forceinline__ size_t pool_slice(int page, int g, int H, int P, int32_t head_major) {
  return head_major ? (size_t)g * P + page : (size_t)page * H + g;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLn2 = 0.69314718055994530942f;
constexpr int kThreads = kWaves * 64;


__device__ __forceinline__ float neg_inf() { return -__builtin_inff(); }
__device__ __forceinline__ float qnan() { return __builtin_nanf(""); }

__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Lane i's value of x, i uniform over the wave.
__device__ __forceinline__ float read_lane(float x, int i) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), i));
}

__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// 16 E4M3FN codes (one dword = 4 codes, lowest byte first) -> 16 bf16 in two
// 8-element operands, exactly (every E4M3 value is a bf16 value).
__device__ __forceinline__ void fp8x16_to_bf16(u32x4 codes, u32x4& lo8, u32x4& hi8) {
  uint32_t o[8];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    o[2 * w] = __builtin_bit_cast(uint32_t,
                                  __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes[w], 1.0f, false));
    o[2 * w + 1] = __builtin_bit_cast(uint32_t,
                                      __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes[w], 1.0f, true));
  }
  lo8 = u32x4{o[0], o[1], o[2], o[3]};
  hi8 = u32x4{o[4], o[5], o[6], o[7]};
}

template <class T>
__device__ __forceinline__ u32x4 ld16(const T* p) {
  return *reinterpret_cast<const u32x4*>(p);
}

// K/V pages are read exactly once per step: stream them with the
// non-temporal hint so they do not displace reusable lines in the caches.
template <class T>
__device__ __forceinline__ u32x4 ld16_stream(const T* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}

// ------------------------------------------------------------------- append
// float32 -> E4M3FN code, round to nearest even, clamped to +-448 (finite
// input); the sign bit is the input's.  Normal range: the 3 leading mantissa
// bits rounded at bit 20 (a carry moves into the exponent); below 2^-6 the
// grid is uniform with step 2^-9.
__device__ __forceinline__ uint32_t e4m3_rne(float v) {
  const uint32_t sign = (__builtin_bit_cast(uint32_t, v) >> 24) & 0x80u;
  const float a = fminf(fabsf(v), 448.0f);
  uint32_t code;
  if (a < 0.015625f) {
    code = (uint32_t)__builtin_rintf(a * 512.0f);
  } else {
    const uint32_t ab = __builtin_bit_cast(uint32_t, a);
    const uint32_t man = ab & 0x7FFFFFu;
    const uint32_t rounded = man + 0x7FFFFu + ((man >> 20) & 1u);
    code = ((((ab >> 23) & 0xFFu) - 120u) << 3) + (rounded >> 20);
  }
  return sign | code;
}

// E4M3FN code -> float32 (exact; the code widens to bf16, then to fp32).
__device__ __forceinline__ float e4m3_value(uint32_t code) {
  const uint32_t b2 = __builtin_bit_cast(uint32_t,
                                         __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(code, 1.0f, false));
  return __builtin_bit_cast(float, b2 << 16);
}

// The 16 slots of a lane's two dims (2*lane, 2*lane + 1) of one fp8 (page, KV
// head): dword i holds slots 4q .. 4q + 3 (q = i / 2) of dim 2*lane + i % 2.
struct E4m3Slots {
  uint32_t x[8];
};

__device__ __forceinline__ E4m3Slots load_e4m3_slots(const uint8_t* page, bool is_v, int lane) {
  E4m3Slots s;
  if (is_v) {  // two rows of 16 slots
    typedef u32x4 u32x4_a4 __attribute__((aligned(4)));  // an append's pools are 4-byte aligned
    const u32x4_a4* rows = reinterpret_cast<const u32x4_a4*>(page) + 2 * lane;
    const u32x4 r0 = rows[0], r1 = rows[1];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s.x[2 * q] = r0[q];
      s.x[2 * q + 1] = r1[q];
    }
  } else {  // a dim pair per slot
    const uint16_t* toks = reinterpret_cast<const uint16_t*>(page) + lane;
    uint32_t t[kPage];
#pragma unroll
    for (int k = 0; k < kPage; ++k) t[k] = toks[k * (kDim / 2)];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      s.x[i] = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) s.x[i] |= ((t[4 * (i >> 1) + b] >> (8 * (i & 1))) & 0xFFu) << (8 * b);
    }
  }
  return s;
}

// The E4M3 append rule for one token of one (page, KV head) of K (is_v
// false, page [slot][d]) or V (page [d][slot]), by one wave whose lane holds
// dims 2 lane, 2 lane + 1 (their bf16 bits in x2); all arithmetic in float32.
// The first token of a page sets scale = amax/28 (16x headroom below 448); a
// later token with amax > 448*scale first re-encodes the page's earlier slots
// to amax/28; the token is stored as RNE(x/scale).  Returns the page's scale
// afterwards (old_scale is ignored for slot 0); the caller stores it.  The
// page's slots are loaded when they are re-encoded, all at once, or come with
// the call (slots, not NULL); V rows are then stored whole.
__device__ __forceinline__ float append_e4m3_head(uint8_t* page, float old_scale, int slot,
                                                  bool is_v, uint32_t x2, int lane,
                                                  const E4m3Slots* slots) {
  const int d0 = 2 * lane;
  const float x0 = __builtin_bit_cast(float, x2 << 16);
  const float x1 = __builtin_bit_cast(float, x2 & 0xFFFF0000u);
  float amax = fmaxf(fabsf(x0), fabsf(x1));
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) amax = fmaxf(amax, __shfl_xor(amax, m));
  E4m3Slots old;
  if (slots) old = *slots;
  float scale;
  if (slot == 0) {
    scale = amax > 0.0f ? amax / 28.0f : 1.0f;
  } else {
    scale = old_scale;
    if (amax > 448.0f * scale) {
      const float fresh = amax / 28.0f;
      auto redo = [&](uint32_t code) -> uint32_t {
        return e4m3_rne(e4m3_value(code) * scale / fresh);
      };
      if (!slots) old = load_e4m3_slots(page, is_v, lane);
      uint32_t* rows = reinterpret_cast<uint32_t*>(page) + 4 * d0;
      uint16_t* toks = reinterpret_cast<uint16_t*>(page) + lane;
#pragma unroll 1
      for (int q = 0; q < 4; ++q) {  // x is turned around by a quad of slots each time
        uint32_t c[2] = {0, 0};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const uint32_t code = (old.x[i] >> (8 * b)) & 0xFFu;
            c[i] |= (4 * q + b < slot ? redo(code) : code) << (8 * b);
          }
        if (is_v) {
          rows[q] = c[0];
          rows[4 + q] = c[1];
        } else {
#pragma unroll
          for (int b = 0; b < 4; ++b)
            if (4 * q + b < slot)
              toks[(4 * q + b) * (kDim / 2)] =
                  (uint16_t)(((c[0] >> (8 * b)) & 0xFFu) | ((c[1] >> (8 * b)) & 0xFFu) << 8);
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) old.x[i] = old.x[i + 2];
        old.x[6] = c[0];
        old.x[7] = c[1];
      }
      scale = fresh;
    }
  }
  const uint32_t c0 = e4m3_rne(x0 / scale), c1 = e4m3_rne(x1 / scale);
  if (is_v && slots) {
    u32x4* rows = reinterpret_cast<u32x4*>(page) + d0;
    u32x4 r[2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t keep = slot >> 2 == q ? ~(0xFFu << (8 * (slot & 3))) : ~0u;
      r[0][q] = (old.x[2 * q] & keep) | (c0 << (8 * (slot & 3)) & ~keep);
      r[1][q] = (old.x[2 * q + 1] & keep) | (c1 << (8 * (slot & 3)) & ~keep);
    }
    rows[0] = r[0];
    rows[1] = r[1];
  } else if (is_v) {
    page[d0 * kPage + slot] = (uint8_t)c0;
    page[(d0 + 1) * kPage + slot] = (uint8_t)c1;
  } else {
    reinterpret_cast<uint16_t*>(page)[slot * (kDim / 2) + lane] = (uint16_t)(c0 | c1 << 8);
  }
  return scale;
}

// The token's V elements written into slot `slot` of a bf16 page's 128 rows
// of 16 slots, by one wave, as whole rows.  A step's appends are bound by what
// their writes cost the memory afterwards, not by their bytes: 2-byte stores,
// one per row, leave a partial line in every row, and the attention that
// follows pays for it (192 sequences of 32 KV heads: partial kernel 235 us
// after them, 226 us after whole rows; the step 250.3 -> 246.8 us).
__device__ __forceinline__ void append_v_rows(uint16_t* page, int slot, const uint16_t* v_new,
                                              int lane) {
  typedef u32x4 u32x4_a4 __attribute__((aligned(4)));  // an append's pools are 4-byte aligned
  u32x4_a4* rows = reinterpret_cast<u32x4_a4*>(page);  // two per row
  u32x4 x[4];
  uint32_t v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[i] = rows[64 * i + lane];
    v[i] = v_new[32 * i + (lane >> 1)];
  }
  const int wd = (slot & 7) >> 1, sh = 16 * (slot & 1);
  const bool mine = (lane & 1) == slot >> 3;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (mine && k == wd) x[i][k] = (x[i][k] & ~(0xFFFFu << sh)) | v[i] << sh;
    rows[64 * i + lane] = x[i];
  }
}

template <bool FP8>
__global__ __launch_bounds__(1024) void append_kernel(AppendArgs a) {
  const int b = blockIdx.x;
  const int r = a.tail_route[b];
  if (r < 0) return;
  int flag = 0;
  int32_t seq = 0, tb = 0, te = 0, base = 0, cap = 0, pid = 0;
  if (r >= a.num_routes) {
    flag = KF_EFLAG_BAD_ROUTE;
  } else {
    const int32_t* rp = reinterpret_cast<const int32_t*>(a.routes + r);
    seq = rp[0]; tb = rp[2]; te = rp[3]; base = rp[4]; cap = rp[5];
    const int j = te - tb;
    if (seq != b || j < 0) {
      flag = KF_EFLAG_BAD_ROUTE;
    } else if (j / kPage >= cap) {
      flag = KF_EFLAG_TAIL_FULL;
    } else if (base < 0 || (int64_t)base + j / kPage >= a.num_page_ids) {
      flag = KF_EFLAG_BAD_ROUTE;
    } else {
      pid = a.page_ids[base + j / kPage];
      if (pid < 0 || pid >= a.num_pages) flag = KF_EFLAG_BAD_PAGE;
    }
  }
  if (flag) {
    if (threadIdx.x == 0) atomicOr(a.err_flags, flag);
    return;
  }
  const int slot = (te - tb) % kPage;
  const int H = a.num_kv_heads;
  if constexpr (!FP8) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int g = w; g < H; g += nw) {
      const size_t head = pool_slice(pid, g, H, a.num_pages, a.head_major);
      const size_t tok = ((size_t)b * H + g) * kDim;
      uint32_t* krow = reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.k_pool) +
                                                   (head * kPage + slot) * kDim);
      append_v_rows(static_cast<uint16_t*>(a.v_pool) + head * kDim * kPage, slot, a.v_new + tok,
                    lane);
      krow[lane] = reinterpret_cast<const uint32_t*>(a.k_new + tok)[lane];
    }
  } else {
    // One wave per (KV head, K|V)
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int pr = w; pr < 2 * H; pr += nw) {
      const int g = pr >> 1;
      const bool is_v = pr & 1;
      float* scale = (is_v ? a.v_scale : a.k_scale) + (size_t)pid * H + g;
      uint8_t* page = static_cast<uint8_t*>(is_v ? a.v_pool : a.k_pool) +
                      pool_slice(pid, g, H, a.num_pages, a.head_major) * (kPage * kDim);
      const uint32_t x2 = reinterpret_cast<const uint32_t*>(
          (is_v ? a.v_new : a.k_new) + ((size_t)b * H + g) * kDim)[lane];
      const float s_new = append_e4m3_head(page, *scale, slot, is_v, x2, lane, nullptr);
      if (lane == 0) *scale = s_new;
    }
  }
  __syncthreads();  // every thread has read tok_end before it moves
  if (threadIdx.x == 0) a.routes[r].tok_end = te + 1;
}

// ------------------------------------------------------------------ partial
// The murmur3 32-bit finaliser: a route's tile walk starts at
// route_hash(route) / 2^32 of its full tiles.
__device__ __forceinline__ uint32_t route_hash(uint32_t x) {
  x ^= x >> 16;
  x *= 0x85EBCA6Bu;
  x ^= x >> 13;
  x *= 0xC2B2AE35u;
  x ^= x >> 16;
  return x;
}

struct RouteView {
  int seq, n, npages, base;
  bool bad;
  bool app;       // fused step: this route takes the step's token (local index n - 1)
  int app_pid;    // page id and slot that receive it
  int app_slot;
};

// The append rule of append_kernel, seen from the route: route r takes the
// step's token iff it is its sequence's tail and the token's page is
// reserved, listed and inside the pool.  The merge kernel takes the same
// decision from the sequence side (tail_append_status).
__device__ __forceinline__ bool fused_append(const PartialArgs& a, int r, int seq, int j, int base,
                                             int cap, int& pid) {
  if (!a.tail_route || seq < 0 || seq >= a.num_seqs || a.tail_route[seq] != r) return false;
  if (j < 0 || j / kPage >= cap || base < 0 || (int64_t)base + j / kPage >= a.num_page_ids)
    return false;
  pid = a.page_ids[base + j / kPage];
  return pid >= 0 && pid < a.num_pages;
}

// Route row r as the kernels see it, with the device-side consistency checks
// (in a fused step, after the step's append).
__device__ __forceinline__ RouteView read_route(const PartialArgs& a, int r) {
  const int32_t* rp = reinterpret_cast<const int32_t*>(a.routes + r);
  RouteView v;
  v.seq = rp[0];
  const int tb = rp[2], te = rp[3], cap = rp[5];
  v.base = rp[4];
  v.n = te - tb;
  v.app_pid = 0;
  v.app = fused_append(a, r, v.seq, v.n, v.base, cap, v.app_pid);
  v.app_slot = v.n & (kPage - 1);
  if (v.app) v.n += 1;
  v.npages = v.n > 0 ? (v.n + kPage - 1) / kPage : 0;
  v.bad = v.seq < 0 || v.seq >= a.num_seqs || v.n < 0 || v.base < 0 || v.npages > cap ||
          v.npages > a.max_pages_per_route || (int64_t)v.base + v.npages > a.num_page_ids;
  return v;
}

// Fused step: write the step's token of KV head g into the route's page
// (publish_to_workgroup then makes it visible to every wave of the
// workgroup before any of them loads the page).  fp8 pools follow the E4M3
// append rule (waves 0 and 1 take K and V) and hand the page's new scales to
// the workgroup in s_app[0..1]: the scalar cache is not coherent with vector
// stores, so the tail page's scales must not be read back through scalar
// loads in this launch.  tid: thread index within the unit's 256 threads.
template <bool FP8>
__device__ __forceinline__ void store_new_token(const PartialArgs& a, const RouteView& rv, int g,
                                                int tid, float* s_app) {
  const int H = a.num_kv_heads;
  const uint16_t* kn = a.k_new + ((size_t)rv.seq * H + g) * kDim;
  const uint16_t* vn = a.v_new + ((size_t)rv.seq * H + g) * kDim;
  const size_t head = pool_slice(rv.app_pid, g, H, a.num_pages, a.head_major);
  if constexpr (!FP8) {
    if (tid < kDim) {
      static_cast<uint16_t*>(a.k_pool_w)[(head * kPage + rv.app_slot) * kDim + tid] = kn[tid];
      static_cast<uint16_t*>(a.v_pool_w)[(head * kDim + tid) * kPage + rv.app_slot] = vn[tid];
    }
  } else {
    const int wv = tid >> 6, lane = tid & 63;
    if (wv < 2) {
      const bool is_v = wv == 1;
      // scales are [num_pages][Hkv] in either pool layout
      float* scale = (is_v ? a.v_scale_w : a.k_scale_w) + (size_t)rv.app_pid * H + g;
      uint8_t* page = static_cast<uint8_t*>(is_v ? a.v_pool_w : a.k_pool_w) + head * (kPage * kDim);
      const float s_new = append_e4m3_head(page, *scale, rv.app_slot, is_v,
                                           reinterpret_cast<const uint32_t*>(is_v ? vn : kn)[lane],
                                           lane, nullptr);
      if (lane == 0) {
        *scale = s_new;
        s_app[wv] = s_new;
      }
    }
  }
}

// Orders the workgroup's earlier global stores before every later load of
// its waves (the waves of a workgroup share the compute unit's L1).
__device__ __forceinline__ void publish_to_workgroup() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Tile geometry.  A wave tile is TP pages: 2 for bf16 (16 KiB of K+V), 4 for
// fp8 (also 16 KiB).  Lane (grp = lane/16, li = lane%16):
//   q.K^T MFMA c (c < TP) takes K row li = token (kpage(li), kslot(c, li));
//   the 16x16 result gives lane (grp, head li) the TP*4 slots
//   vslot0 + 4c + r4 of tile page vpage(grp), which are exactly the k-slots
//   the lane feeds to p.V (NH = TP/2 MFMAs of 8 slots per 16-dim block).
template <bool FP8>
struct Geo {
  static constexpr int TP = FP8 ? 4 : 2;  // pages per tile
  static constexpr int NC = TP;           // q.K^T MFMAs of 16 rows per tile
  static constexpr int NH = TP / 2;       // p.V MFMAs (8 slots each) per 16-dim block
  static __device__ __forceinline__ int kpage(int li) { return FP8 ? li >> 2 : li >> 3; }
  static __device__ __forceinline__ int kslot0(int li) {
    return FP8 ? (li & 3) : 8 * ((li >> 2) & 1) + (li & 3);
  }
  static __device__ __forceinline__ int vpage(int grp) { return FP8 ? grp : grp >> 1; }
  static __device__ __forceinline__ int vslot0(int grp) { return FP8 ? 0 : 8 * (grp & 1); }
};

// Raw bytes of one tile as one lane loads them.
template <bool FP8>
struct TileRaw;
template <>
struct TileRaw<false> {
  u32x4 k[2][4];  // [c][kk]: 8 bf16 of K row kslot(c), dims 32*kk + 8*grp ..
  u32x4 v[8];     // [b8]: 8 bf16 of V^T row d = 16*b8 + li, slots vslot0 ..
};
template <>
struct TileRaw<true> {
  u32x4 k[4][2];  // [c][pp]: 16 E4M3 of K row kslot(c), dims 64*pp + 16*grp ..
  u32x4 v[8];     // [b8]: the 16 E4M3 slots of V^T row d = 16*b8 + li
  float ks, vs;   // K and V scales of the lane's page (vpage)
};

// Softmax state of one query head per lane column: lane (grp, li) holds dims
// 16*b8 + 4*grp + r4 of head li; m is shared by the four lane groups, l is
// the lane's own part of the sum.
struct Attn {
  f32x4 o[8];
  float m, l;
};

__device__ __forceinline__ void reset(Attn& s) {
#pragma unroll
  for (int b8 = 0; b8 < 8; ++b8) s.o[b8] = f32x4{0.f, 0.f, 0.f, 0.f};
  s.m = neg_inf();
  s.l = 0.0f;
}

// One tile: scores, softmax update, O^T += V^T P^T.  ks: score scale (with
// the page's K scale), vs: V scale, of the lane's page; tok0: the lane's
// first route-local token, lim: the token bound.  MASK: the tile can hold
// slots past the bound; their V bits are zeroed and they add nothing.
// SPAN: a span wave's chains are several times as long as a chunk wave's, so
// its terms are rounded less.  The tile's sum of p, and for bf16 its p.V, start
// from zero and are then added, one rounding of the running sum per tile
// instead of one per pair of slots or matrix product, and the bf16 p (at most
// 1, so it cannot round up to infinity) is split into its nearest bf16 and the
// rest, half the error of the truncated split.  The adds take the place of the
// rescaling product, so none of it costs time (237.96 -> 238.0 us, 61.2 ->
// 61.3, 1165.8 -> 1164.8); fp8 tiles have no registers to spare for p.V.
// Error of the partials against 64 bits with the chunk plan, and as spans
// without and with it: 192 multi-head sequences 2.88e-7, 3.29e-7, 2.28e-7, 24
// of 16 heads per KV head 5.2e-7, 5.5e-7, 3.4e-7, the agentic batch 8.3e-7,
// 9.3e-7, 5.8e-7; fp8 batches 5.2 to 5.5e-6 in all three, the split's.
template <bool FP8, bool MASK, bool SPAN = false>
__device__ __forceinline__ void attend(const TileRaw<FP8>& t, const u32x4 (&qb)[4], float ks,
                                       float vs, int tok0, int lim, Attn& st) {
  constexpr bool TILE_SUM = SPAN && !FP8;
  constexpr int NC = Geo<FP8>::NC, NH = Geo<FP8>::NH;
  // ---- S^T = K Q^T (fp8 codes widen to bf16 right before their MFMA)
  f32x4 s[NC];
#pragma unroll
  for (int cc = 0; cc < NC; ++cc) {
    s[cc] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (!FP8) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) s[cc] = mfma16(t.k[cc][kk], qb[kk], s[cc]);
    } else {
#pragma unroll
      for (int pp = 0; pp < 2; ++pp) {
        u32x4 k0, k1;
        fp8x16_to_bf16(t.k[cc][pp], k0, k1);
        s[cc] = mfma16(k0, qb[2 * pp], s[cc]);
        s[cc] = mfma16(k1, qb[2 * pp + 1], s[cc]);
      }
    }
  }
  float mt = neg_inf();
#pragma unroll
  for (int cc = 0; cc < NC; ++cc)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float v = (tok0 + 4 * cc + r4 < lim) ? s[cc][r4] * ks : neg_inf();
      s[cc][r4] = v;
      mt = fmaxf(mt, v);
    }
  mt = fmaxf(mt, __shfl_xor(mt, 16));
  mt = fmaxf(mt, __shfl_xor(mt, 32));
  const float m_new = fmaxf(st.m, mt);
  const float alpha = exp2_fast(st.m - m_new);
  st.m = m_new;
  if constexpr (!SPAN) st.l *= alpha;
  if constexpr (!TILE_SUM) {
#pragma unroll
    for (int b8 = 0; b8 < 8; ++b8) st.o[b8] *= alpha;
  }

  // ---- P^T operands: half h2 holds slots 8*h2 + j (j < 8) of the lane's
  // range, i.e. MFMA c = 2*h2 + j/4, row r4 = j%4; bf16 hi + lo
  u32x4 phi[NH], plo[NH];
  float sum_l = 0.0f;  // SPAN: of the tile
#pragma unroll
  for (int h2 = 0; h2 < NH; ++h2)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int cc = 2 * h2 + (jj >> 1), r4 = 2 * (jj & 1);
      const float e0 = exp2_fast(s[cc][r4] - m_new);
      const float e1 = exp2_fast(s[cc][r4 + 1] - m_new);
      (SPAN ? sum_l : st.l) += e0 + e1;
      float x0 = e0 * vs, x1 = e1 * vs;
      if constexpr (MASK && FP8) {  // a masked slot adds nothing, whatever its page's scales
        const int t0 = tok0 + 8 * h2 + 2 * jj;
        x0 = t0 < lim ? x0 : 0.0f;
        x1 = t0 + 1 < lim ? x1 : 0.0f;
      }
      uint32_t b0, b1;
      if constexpr (TILE_SUM) {
        phi[h2][jj] = pack_bf16_rne(x0, x1);
        b0 = phi[h2][jj] << 16;
        b1 = phi[h2][jj] & 0xFFFF0000u;
      } else {
        b0 = __builtin_bit_cast(uint32_t, x0) & 0xFFFF0000u;
        b1 = __builtin_bit_cast(uint32_t, x1) & 0xFFFF0000u;
        phi[h2][jj] = (b0 >> 16) | b1;
      }
      plo[h2][jj] = pack_bf16_rne(x0 - __builtin_bit_cast(float, b0),
                                  x1 - __builtin_bit_cast(float, b1));
    }

  if constexpr (SPAN) st.l = __builtin_fmaf(st.l, alpha, sum_l);

  // ---- O^T += V^T P^T; V of slots past the range is zeroed (unused slots
  // may hold anything)
  uint32_t msk[NH][4];
#pragma unroll
  for (int h2 = 0; h2 < NH; ++h2)
#pragma unroll
    for (int wd = 0; wd < 4; ++wd) {
      const int t0 = tok0 + 8 * h2 + 2 * wd;
      msk[h2][wd] = (t0 < lim ? 0x0000FFFFu : 0u) | (t0 + 1 < lim ? 0xFFFF0000u : 0u);
    }
#pragma unroll
  for (int b8 = 0; b8 < 8; ++b8) {
    u32x4 vr[NH];
    if constexpr (!FP8) vr[0] = t.v[b8];
    else fp8x16_to_bf16(t.v[b8], vr[0], vr[1]);
    if constexpr (MASK) {
#pragma unroll
      for (int h2 = 0; h2 < NH; ++h2)
#pragma unroll
        for (int wd = 0; wd < 4; ++wd) vr[h2][wd] &= msk[h2][wd];
    }
    if constexpr (TILE_SUM) {
      f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h2 = 0; h2 < NH; ++h2) sum = mfma16(vr[h2], plo[h2], sum);
#pragma unroll
      for (int h2 = 0; h2 < NH; ++h2) sum = mfma16(vr[h2], phi[h2], sum);
#pragma unroll
      for (int k = 0; k < 4; ++k) st.o[b8][k] = __builtin_fmaf(st.o[b8][k], alpha, sum[k]);
    } else {
#pragma unroll
      for (int h2 = 0; h2 < NH; ++h2) {
        st.o[b8] = mfma16(vr[h2], phi[h2], st.o[b8]);
        st.o[b8] = mfma16(vr[h2], plo[h2], st.o[b8]);
      }
    }
  }
}

// Wave-uniform description of one tile: its first route-local page and the
// page ids of its (up to four) pages.
struct TileInfo {
  int tp0;
  int pid0, pid1, pid2, pid3;
};

template <class T>
__device__ __forceinline__ T pick4(T v0, T v1, T v2, T v3, int i) {
  return (i & 2) ? ((i & 1) ? v3 : v2) : ((i & 1) ? v1 : v0);
}

// Record marks of a split launch, so that the combine needs no route row: a
// unit whose outputs are already in o_part/lse_part carries the sum -1 in its
// first record (a real sum is >= 0 or NaN), an unused record place the
// maximum -inf and the sum 0.
__device__ __forceinline__ void mark_whole(const PartialArgs& a, int u, int g, int tid) {
  const size_t rec = ((size_t)u * a.num_kv_heads + g) * a.max_chunks;
  if (tid < a.group) {
    a.ws_ml[(rec * a.group + tid) * 2] = 0.0f;
    a.ws_ml[(rec * a.group + tid) * 2 + 1] = -1.0f;
  }
}

// UPW = units per workgroup.  1: a 256-thread workgroup owns one (route, KV
// head) unit or one chunk of it, two workgroups per CU.  2 (unsplit bf16
// launches of units of at most kMaxPagesTwoUnit pages): a 512-thread
// workgroup owns units u and u + gridDim.z, waves 0-3 the first and 4-7 the
// second, one workgroup per CU, so both units of a CU start at once.  In
// that mode all 512 threads reach every barrier: a half without work (no
// unit, a bad or empty one) skips its work, never the barriers.
template <bool FP8, int UPW, bool HM>
__global__ __launch_bounds__(kThreads * UPW, 2 / UPW) void partial_kernel(PartialArgs a) {
  using GeoT = Geo<FP8>;
  constexpr int TP = GeoT::TP, NC = GeoT::NC;
  __shared__ float s_o_u[UPW][kWaves][KF_MAX_GROUP][kLdsStride];
  __shared__ float s_m_u[UPW][kWaves][KF_MAX_GROUP];
  __shared__ float s_l_u[UPW][kWaves][KF_MAX_GROUP];
  __shared__ float s_fm_u[UPW][KF_MAX_GROUP];
  __shared__ float s_fl_u[UPW][KF_MAX_GROUP];
  __shared__ float s_app_u[UPW][2];  // fused fp8 append: the tail page's new K and V scales
  // Each wave's half is uniform, but taking it into a scalar register
  // (readfirstlane) made the compiler keep the main loop's next tile in
  // flight for less of each iteration: 2% slower on the Llama layer.
  const int half = UPW == 2 ? (int)(threadIdx.x / kThreads) : 0;
  auto& s_o = s_o_u[half];
  auto& s_m = s_m_u[half];
  auto& s_l = s_l_u[half];
  auto& s_fm = s_fm_u[half];
  auto& s_fl = s_fl_u[half];
  float* s_app = s_app_u[half];

  int c = blockIdx.x;
  int g = blockIdx.y, u = blockIdx.z + half * gridDim.z;  // u: position in the launch
  if (UPW == 1 && a.order) {
    // a split launch of several rounds: take the work item of this
    // workgroup's place in the dispatch order; places past the last item
    // have no work
    const uint32_t i = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    if (i >= a.order[0]) return;
    const uint32_t e0 = a.order[2 + 2 * (size_t)i], e1 = a.order[3 + 2 * (size_t)i];
    u = (int)e0;
    g = (int)(e1 >> 16);
    c = (int)(e1 & 0xFFFFu);
  }
  if constexpr (FP8) {
    // Unsplit fp8 units: workgroups are dealt round-robin over the 8 XCDs.
    // Give XCD k the k-th eighth of the (head, route) space instead, so the
    // heads of a route, whose per-page scales share cache lines, meet in one
    // L2 (the fp8 layer reads ~1% faster; bf16 pools gain nothing from it).
    const unsigned NT = gridDim.y * gridDim.z;
    if (gridDim.x == 1 && (NT & 7u) == 0) {
      const unsigned L = blockIdx.y + gridDim.y * blockIdx.z;
      const unsigned Lp = (L & 7u) * (NT >> 3) + (L >> 3);
      g = Lp % gridDim.y;
      u = Lp / gridDim.y;
    }
  }
  const int G = a.group, Hq = a.num_q_heads, H = a.num_kv_heads;
  const int tid = threadIdx.x & (kThreads - 1), lane = tid & 63, grp = lane >> 4, li = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hq0 = g * G;

  // ---- this unit's page range [p0, p1), or no work for this half: outputs
  // of a bad or empty route are written here
  bool work = false, writer = false;
  int r = -1, nchunks = 1, p0 = 0, p1 = 0;
  RouteView rv{};
  if (u < a.num_units_routes) {
    r = a.route_list ? a.route_list[u] : u;
    if (r < 0 || r >= a.num_routes) {  // a list entry naming no route: nothing to write
      if (c == 0 && g == 0 && tid == 0) atomicOr(a.err_flags, KF_EFLAG_BAD_ROUTE);
    } else {
      rv = read_route(a, r);
      if (rv.bad || rv.npages == 0) {
        if (c == 0) {
          if (rv.app) store_new_token<FP8>(a, rv, g, tid, s_app);  // the pool takes the token all the same
          const float ov = rv.bad ? qnan() : 0.0f, lv = rv.bad ? qnan() : neg_inf();
          for (int e = tid; e < G * kDim; e += kThreads)
            a.o_part[((size_t)r * Hq + hq0 + e / kDim) * kDim + e % kDim] = ov;
          if (tid < G) a.lse_part[(size_t)r * Hq + hq0 + tid] = lv;
          if (rv.bad && tid == 0) atomicOr(a.err_flags, KF_EFLAG_BAD_ROUTE);
          if (UPW == 1 && a.max_chunks > 1) mark_whole(a, u, g, tid);
        }
      } else {
        nchunks = (rv.npages + a.chunk_pages - 1) / a.chunk_pages;
        if (c < nchunks) {
          work = true;
          writer = rv.app && c == nchunks - 1;  // the chunk with the last page
          p0 = (int)((int64_t)c * rv.npages / nchunks);
          p1 = (int)((int64_t)(c + 1) * rv.npages / nchunks);
        }
      }
    }
  }
  if (writer) store_new_token<FP8>(a, rv, g, tid, s_app);
  if constexpr (UPW == 1) {
    if (!work) return;
    if (writer) publish_to_workgroup();
  } else {
    publish_to_workgroup();
  }
  const int seq = rv.seq, n = rv.n;
  const int app_page = (rv.n - 1) >> 4;             // route-local page of the new token
  const int ntiles = (p1 - p0 + TP - 1) / TP;
  const int lim = min(n, p1 * kPage);  // route-local token bound of this range
  const int32_t* __restrict__ pids = a.page_ids + rv.base;
  // All workgroups start together and stream at about the same pace, so
  // without care every route reads the same offset of its range at the same
  // moment, and in a contiguous pool (routes of a sequence equal sizes apart)
  // the DRAM channels hit at each moment then depend on the pool's layout:
  // the same work ran up to ~9% slower on some page reservations.  Each route
  // therefore walks its full tiles starting from its own offset, rot, taken
  // from a hash of the route index (the murmur3 finaliser), the same for
  // every KV head and chunk of the route, so the heads keep reading the same
  // pages together.  A hash and not a low-discrepancy sequence: offsets
  // spread evenly by the golden ratio made layers with 2 and 16 KV heads
  // stream 8-10% slower (the evenly spaced offsets of equally sized routes
  // meet the same DRAM channels), and per-head offsets lost 1-2% on 4 and 8
  // heads.  A partial last tile keeps its place at the end and is computed
  // masked.  The order depends on the route index only, never on page ids.
  const int nfull = (lim == p1 * kPage && (p1 - p0) % TP == 0) ? ntiles : ntiles - 1;
  const int rot =
      nfull > 1 ? (int)(((uint64_t)route_hash((uint32_t)r) * (uint32_t)nfull) >> 32) : 0;

  auto next_tile = [&](int cur) -> int { return cur + kWaves; };  // wave w: w, w+4, ...

  // Page ids are uniform, so they arrive through scalar loads; a page past
  // the range or outside the pool reads page 0 and is masked (its p set to 0
  // whatever its scales hold) or flagged.  fp8 page scales arrive with the
  // tile's vector loads instead, each lane loading those of its own page: a
  // scalar load of a scale would wait on the scalar load of its page id, and
  // every wait on a scalar load waits on all of them (fp8 layer 1.9% faster).
  bool pid_bad = false;
  auto page_at = [&](int pg) -> int {  // page id of route-local page pg of the range
    const bool in = pg < p1;
    int v = pids[in ? pg : p0];
    v = in ? v : 0;
    if (v < 0 || v >= a.num_pages) {
      pid_bad = true;
      v = 0;
    }
    return v;
  };
  auto tile_info = [&](int tile) -> TileInfo {  // tile: index within the range
    TileInfo t;
    const int tr = tile < nfull ? (tile + rot < nfull ? tile + rot : tile + rot - nfull) : tile;
    t.tp0 = p0 + tr * TP;
    t.pid0 = page_at(t.tp0);
    t.pid1 = page_at(t.tp0 + 1);
    t.pid2 = TP > 2 ? page_at(t.tp0 + 2) : 0;
    t.pid3 = TP > 2 ? page_at(t.tp0 + 3) : 0;
    return t;
  };

  const int kpage = GeoT::kpage(li), vpage = GeoT::vpage(grp);
  const size_t head_elems = (size_t)kPage * kDim;  // elements of one (page, kv head)
  const int koff = GeoT::kslot0(li) * kDim + (FP8 ? 16 : 8) * grp;
  const int voff = li * kPage + GeoT::vslot0(grp);

  auto issue = [&](TileRaw<FP8>& t, const TileInfo& ti) {
    const int pk = pick4(ti.pid0, ti.pid1, ti.pid2, ti.pid3, kpage);
    const int pv = pick4(ti.pid0, ti.pid1, ti.pid2, ti.pid3, vpage);
    const size_t hk = (HM ? (size_t)g * a.num_pages + pk : (size_t)pk * H + g) * head_elems;
    const size_t hv = (HM ? (size_t)g * a.num_pages + pv : (size_t)pv * H + g) * head_elems;
    if constexpr (!FP8) {
      const uint16_t* kb = static_cast<const uint16_t*>(a.k_pool) + hk + koff;
      const uint16_t* vb = static_cast<const uint16_t*>(a.v_pool) + hv + voff;
#pragma unroll
      for (int cc = 0; cc < NC; ++cc)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) t.k[cc][kk] = ld16_stream(kb + cc * 4 * kDim + 32 * kk);
#pragma unroll
      for (int b8 = 0; b8 < 8; ++b8) t.v[b8] = ld16_stream(vb + b8 * 16 * kPage);
    } else {
      const uint8_t* kb = static_cast<const uint8_t*>(a.k_pool) + hk + koff;
      const uint8_t* vb = static_cast<const uint8_t*>(a.v_pool) + hv + voff;
#pragma unroll
      for (int cc = 0; cc < NC; ++cc)
#pragma unroll
        for (int pp = 0; pp < 2; ++pp) t.k[cc][pp] = ld16_stream(kb + cc * 4 * kDim + 64 * pp);
#pragma unroll
      for (int b8 = 0; b8 < 8; ++b8) t.v[b8] = ld16_stream(vb + b8 * 16 * kPage);
      t.ks = a.k_scale[(size_t)pv * H + g];
      t.vs = a.v_scale[(size_t)pv * H + g];
    }
  };

  // B operand of q.K^T: query head hq0 + li (zero columns past the group).
  u32x4 qb[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int d0 = FP8 ? 64 * (kk >> 1) + 16 * grp + 8 * (kk & 1) : 32 * kk + 8 * grp;
    qb[kk] = work && li < G ? ld16(a.q + ((size_t)seq * Hq + hq0 + li) * kDim + d0)
                           : u32x4{0, 0, 0, 0};
  }

  Attn acc;
  reset(acc);

  // MASK: only a wave's final tile can hold slots past the range, so masking
  // is a compile-time property and the steady-state loop has no branch.
  auto compute = [&](const TileRaw<FP8>& t, const TileInfo& ti, auto mask_tag) {
    constexpr bool MASK = decltype(mask_tag)::value;
    float ks = a.scale_log2, vs = 1.0f;
    if constexpr (FP8) {
      float kss = t.ks;
      vs = t.vs;
      if (writer && ti.tp0 + vpage == app_page) {  // the tail page's scales were just written
        kss = s_app[0];
        vs = s_app[1];
      }
      ks *= kss;
    }
    const int tok0 = (ti.tp0 + vpage) * kPage + GeoT::vslot0(grp);  // route-local token, c = r4 = 0
    attend<FP8, MASK>(t, qb, ks, vs, tok0, lim, acc);
  };

  // ---- two register buffers: while one tile is computed, the loads of the
  // wave's next tile are in flight.  Between issuing a tile and computing
  // the previous one there is no branch, so the compiler waits only for the
  // tile it computes; tile ids and their page ids are fetched a tile ahead.
  // A wave's tile ids increase, so a tile computed inside the loop always
  // precedes one already issued and is full; only the tile computed after
  // the loop can be the range's last and is computed masked.
  TileRaw<FP8> ra, rb;
  const std::integral_constant<bool, false> full{};
  const std::integral_constant<bool, true> masked{};
  if (w < ntiles) {
    const int last = ntiles - 1;
    TileInfo ia = tile_info(w);
    issue(ra, ia);
    int tb = next_tile(w);
    TileInfo ib = tile_info(min(tb, last));
    bool final_in_b = false;
    while (true) {
      if (tb > last) break;
      issue(rb, ib);
      const int tn = next_tile(tb);
      const TileInfo in = tile_info(min(tn, last));
      __builtin_amdgcn_sched_barrier(0);
      compute(ra, ia, full);
      if (tn > last) {
        final_in_b = true;
        break;
      }
      ia = in;
      issue(ra, ia);
      tb = next_tile(tn);
      const TileInfo in2 = tile_info(min(tb, last));
      __builtin_amdgcn_sched_barrier(0);
      compute(rb, ib, full);
      ib = in2;
    }
    if (final_in_b) compute(rb, ib, masked);
    else compute(ra, ia, masked);
  }

  float m_run = acc.m, l_run = acc.l;
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  const bool wave_bad = __ballot(pid_bad) != 0;
  if (wave_bad) m_run = qnan();  // a bad page poisons the unit: NaN weights below

  // ---- combine the waves: lane (grp, li) holds d = 16*b8 + 4*grp + r4
  if (li < G) {
#pragma unroll
    for (int b8 = 0; b8 < 8; ++b8)
      *reinterpret_cast<f32x4*>(&s_o[w][li][16 * b8 + 4 * grp]) = acc.o[b8];
    if (grp == 0) {
      s_m[w][li] = m_run;
      s_l[w][li] = l_run;
    }
  }
  __syncthreads();
  if (tid < G) {
    // a NaN wave max (a bad page) makes the unit's max NaN: fmaxf would skip
    // it, and a range whose waves are all bad would then read as empty (-inf)
    // and be dropped by the combine instead of poisoning the unit
    float M = neg_inf();
    bool nan_m = false;
    for (int ww = 0; ww < kWaves; ++ww) {
      const float mw = s_m[ww][tid];
      nan_m |= mw != mw;
      M = fmaxf(M, mw);
    }
    if (nan_m) M = qnan();
    float L = 0.0f;
    for (int ww = 0; ww < kWaves; ++ww) {
      const float mw = s_m[ww][tid];
      const float wt = mw == neg_inf() ? 0.0f : exp2_fast(mw - M);
      s_m[ww][tid] = wt;  // becomes the wave's weight
      L += wt * s_l[ww][tid];
    }
    s_fm[tid] = M;
    s_fl[tid] = L;
  }
  if (lane == 0 && wave_bad) atomicOr(a.err_flags, KF_EFLAG_BAD_PAGE);  // whichever wave saw it
  __syncthreads();
  if (!work) return;  // after the workgroup's last barrier

  if (nchunks == 1) {
    for (int e = tid; e < G * kDim; e += kThreads) {
      const int h = e / kDim, d = e % kDim;
      float O = 0.0f;
#pragma unroll
      for (int ww = 0; ww < kWaves; ++ww) O += s_m[ww][h] * s_o[ww][h][d];
      a.o_part[((size_t)r * Hq + hq0 + h) * kDim + d] = O / s_fl[h];
    }
    if (tid < G)
      a.lse_part[(size_t)r * Hq + hq0 + tid] = (s_fm[tid] + __log2f(s_fl[tid])) * kLn2;
    if (UPW == 1 && a.max_chunks > 1) mark_whole(a, u, g, tid);
    return;
  }
  // chunked unit: unnormalised output and (max, sum) of this page range; the
  // unit's last range marks the record places that the unit leaves unused
  const size_t rec = ((size_t)u * H + g) * a.max_chunks + c;
  if (c == nchunks - 1)
    for (int e = tid; e < (a.max_chunks - nchunks) * G; e += kThreads) {
      a.ws_ml[((rec + 1) * G + e) * 2] = neg_inf();
      a.ws_ml[((rec + 1) * G + e) * 2 + 1] = 0.0f;
    }
  for (int e = tid; e < G * kDim; e += kThreads) {
    const int h = e / kDim, d = e % kDim;
    float O = 0.0f;
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) O += s_m[ww][h] * s_o[ww][h][d];
    __builtin_nontemporal_store(O, &a.ws_o[(rec * G + h) * kDim + d]);
  }
  if (tid < G) {
    a.ws_ml[(rec * G + tid) * 2] = s_fm[tid];
    a.ws_ml[(rec * G + tid) * 2 + 1] = s_fl[tid];
  }
}

// ------------------------------------------------------------------- spans
// A span launch cuts the whole launch's tiles, and not each unit's pages,
// into equal parts: the tiles of all routes, route after route, are split
// into `cols` columns of equal length, and wave (column, KV head) streams its
// column's tiles of that head, whatever routes they belong to.  One resident
// round of workgroups (two per compute unit) then carries a ragged batch
// without empty, short or late workgroups, and a wave starts once and keeps
// its two tiles in flight across routes.  The four waves of a workgroup hold
// four columns in a row of one KV head.  A wave writes a route that lies
// inside its column straight to o_part; the parts of routes that its column
// cuts go to LDS, where the workgroup joins parts of one route, and only
// routes cut by a workgroup's bounds leave records (place: workgroup column +
// launch position) for the combine.
//
// A cut route's parts are kept in workgroup-column order: with c0 the column
// of its first part, the part of workgroup column c of launch position u has
// record place c + min(u, c0).  The places of two routes never meet: the next
// cut route begins in the column where this one ends, or later, and both u
// and c0 grow by at least one.  Table in the workspace, for the combine: two
// words per launch position, the place of its first record and its number of
// records (0: the outputs are in place).
struct SpanCols {
  int q, rem, cols;  // the first rem columns hold q + 1 tiles, the others q
  __device__ __forceinline__ int begin(int c) const { return c * q + min(c, rem); }
  __device__ __forceinline__ int of(int t) const {
    const int edge = rem * (q + 1);
    return t < edge ? t / (q + 1) : rem + (t - edge) / q;
  }
};

__device__ __forceinline__ SpanCols span_cols(int tiles, int cols) {
  return {tiles / cols, tiles % cols, cols};
}

// One tile of a wave's walk (wave-uniform): the route's tokens from the tile's
// first one on, its launch position and marks, its page ids.
struct SpanTile {
  int left;
  uint32_t uf;  // launch position and marks: kSpanLast ends its part, kSpanToken takes the step's
                // token, kSpanBad has a page id outside the pool
  int pid0, pid1, pid2, pid3;
};
constexpr uint32_t kSpanToken = 1u << 29, kSpanLast = 1u << 30, kSpanBad = 1u << 31;

// A tile with slots past the route: their V bits zeroed (such slots may hold
// anything), and for fp8 the V scale of a page wholly past it.  tok: the
// lane's first token within the tile.
template <bool FP8>
__device__ __forceinline__ void mask_tile(TileRaw<FP8>& t, int tok, int left) {
  u32x4 msk;
#pragma unroll
  for (int wd = 0; wd < 4; ++wd) {
    uint32_t m = 0;
    constexpr int N = FP8 ? 4 : 2;  // slots per dword
#pragma unroll
    for (int k = 0; k < N; ++k)
      m |= tok + N * wd + k < left ? (FP8 ? 0xFFu << (8 * k) : 0xFFFFu << (16 * k)) : 0u;
    msk[wd] = m;
  }
#pragma unroll
  for (int b8 = 0; b8 < 8; ++b8) t.v[b8] &= msk;
  if constexpr (FP8) t.vs = tok < left ? t.vs : 0.0f;
}

// The step's token of (route, KV head g) written by one wave (the fused
// append of store_new_token): loaded first, stored later.  Lane: dims 2*lane
// and 2*lane + 1.
struct WaveToken {
  uint32_t k2, v2;
  float ks, vs;         // fp8: the page's scales
  E4m3Slots k_at, v_at; // fp8: the page's slots, in case the token re-encodes them
  int pid, slot;
};

template <bool FP8>
__device__ __forceinline__ WaveToken load_wave_token(const PartialArgs& a, int seq, int pid,
                                                     int slot, int g, int lane) {
  const size_t tok = ((size_t)seq * a.num_kv_heads + g) * kDim;
  WaveToken t;
  t.k2 = reinterpret_cast<const uint32_t*>(a.k_new + tok)[lane];
  t.v2 = reinterpret_cast<const uint32_t*>(a.v_new + tok)[lane];
  t.ks = t.vs = 1.0f;
  if constexpr (FP8) {
    t.ks = a.k_scale[(size_t)pid * a.num_kv_heads + g];
    t.vs = a.v_scale[(size_t)pid * a.num_kv_heads + g];
    const size_t at = pool_slice(pid, g, a.num_kv_heads, a.num_pages, a.head_major) * (kPage * kDim);
    t.k_at = load_e4m3_slots(static_cast<const uint8_t*>(a.k_pool) + at, false, lane);
    t.v_at = load_e4m3_slots(static_cast<const uint8_t*>(a.v_pool) + at, true, lane);
  }
  t.pid = pid;
  t.slot = slot;
  return t;
}

template <bool FP8>
__device__ __forceinline__ void store_wave_token(const PartialArgs& a, const WaveToken& t, int g,
                                                 int lane) {
  const int H = a.num_kv_heads;
  const size_t head = pool_slice(t.pid, g, H, a.num_pages, a.head_major);
  if constexpr (!FP8) {
    reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.k_pool_w) +
                                (head * kPage + t.slot) * kDim)[lane] = t.k2;
    uint16_t* vp = static_cast<uint16_t*>(a.v_pool_w) + (head * kDim + 2 * lane) * kPage + t.slot;
    vp[0] = (uint16_t)t.v2;
    vp[kPage] = (uint16_t)(t.v2 >> 16);
  } else {
    const float k_s = append_e4m3_head(static_cast<uint8_t*>(a.k_pool_w) + head * (kPage * kDim),
                                       t.ks, t.slot, false, t.k2, lane, &t.k_at);
    const float v_s = append_e4m3_head(static_cast<uint8_t*>(a.v_pool_w) + head * (kPage * kDim),
                                       t.vs, t.slot, true, t.v2, lane, &t.v_at);
    if (lane == 0) {
      a.k_scale_w[(size_t)t.pid * H + g] = k_s;
      a.v_scale_w[(size_t)t.pid * H + g] = v_s;
    }
  }
}

// Constant-address-space view of a table that the kernel does not write:
// uniform reads stay scalar loads beside the kernel's stores.
typedef const int32_t __attribute__((address_space(4)))* const_i32;
__device__ __forceinline__ const_i32 as_const(const int32_t* p) { return (const_i32)(uintptr_t)p; }

template <bool FP8, bool HM>
__global__ __launch_bounds__(kThreads, 2) void span_kernel(PartialArgs a) {
  using GeoT = Geo<FP8>;
  constexpr int TP = GeoT::TP, NC = GeoT::NC;
  extern __shared__ f32x4 s_lds[];
  float* s_dyn = reinterpret_cast<float*>(s_lds);  // parts: [2 * kWaves][G][kLdsStride], (max, sum)
  __shared__ int s_sum[kWaves], s_start[kWaves], s_part[2 * kWaves];
  static_assert(sizeof(s_sum) + sizeof(s_start) + sizeof(s_part) == kSpanStaticLds, "");
  const int U = a.num_units_routes, H = a.num_kv_heads, G = a.group, Hq = a.num_q_heads;
  const int tid = threadIdx.x, lane = tid & 63, grp = lane >> 4, li = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = blockIdx.x % H, blk = blockIdx.x / H;  // KV head, workgroup column
  const int hq0 = g * G;

  // ---- the route table: first tiles (U + 1), page lists, lengths, sequences
  int* s_pre = reinterpret_cast<int*>(s_dyn + 2 * kWaves * G * (kLdsStride + 2));
  int *s_base = s_pre + U + 1, *s_n = s_base + U, *s_seq = s_n + U;
  constexpr int PER = kSpanRoutes / kThreads;
  const int per = (U + kThreads - 1) / kThreads;
  int cnt[PER], sum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = tid * per + i;
    cnt[i] = 0;
    if (i < per && u < U) {
      const RouteView rv = read_route(a, u);
      if (!rv.bad) cnt[i] = (rv.npages + TP - 1) / TP;
      s_base[u] = rv.base;
      s_n[u] = rv.bad && rv.n == 0 ? -1 : rv.n;  // 0: empty
      s_seq[u] = rv.app ? ~rv.seq : cnt[i] ? rv.seq : 0;
      if (blockIdx.x == 0 && rv.bad) atomicOr(a.err_flags, KF_EFLAG_BAD_ROUTE);
      sum += cnt[i];
    }
  }
  int incl = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(incl, d);
    if (lane >= d) incl += v;
  }
  if (lane == 63) s_sum[w] = incl;
  if (tid < kWaves) s_start[tid] = -1;
  if (tid < 2 * kWaves) s_part[tid] = -1;
  __syncthreads();
  int pre = incl - sum, T = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    if (i < w) pre += s_sum[i];
    T += s_sum[i];
  }
  const SpanCols sc = span_cols(T, max(1, min(a.span_cols, T)));
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = tid * per + i;
    if (i < per && u < U) {
      s_pre[u] = pre;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {  // the route at the start of each wave's column
        const int c = blk * kWaves + v, t = sc.begin(c);
        if (c < sc.cols && pre <= t && t < pre + cnt[i]) s_start[v] = u;
      }
      if (blockIdx.x == 0) {
        const int c0 = cnt[i] ? sc.of(pre) / kWaves : 0;
        const int c1 = cnt[i] ? sc.of(pre + cnt[i] - 1) / kWaves : 0;
        a.span_table[2 * u] = c0 + min(u, c0);
        a.span_table[2 * u + 1] = c1 > c0 ? c1 - c0 + 1 : 0;
      }
      pre += cnt[i];
    }
  }
  if (tid == 0) s_pre[U] = T;
  __syncthreads();

  // ---- outputs of routes without tiles (empty or bad), spread over the workgroups
  for (int u = blockIdx.x; u < U; u += gridDim.x) {
    if (s_pre[u + 1] != s_pre[u]) continue;
    const bool bad = s_n[u] != 0;
    const float ov = bad ? qnan() : 0.0f, lv = bad ? qnan() : neg_inf();
    for (int e = tid; e < Hq * kDim; e += kThreads) a.o_part[(size_t)u * Hq * kDim + e] = ov;
    for (int h = tid; h < Hq; h += kThreads) a.lse_part[(size_t)u * Hq + h] = lv;
  }

  // ---- this wave's column
  const int col = blk * kWaves + w;
  const int t0 = sc.begin(col), t1 = col < sc.cols ? sc.begin(col + 1) : t0;
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  const const_i32 page_ids = as_const(a.page_ids);
  // The fused step's tokens, for the routes that end inside this column (and
  // bad routes there, whose pools take theirs all the same; column 0 has
  // those before the first tile).  Each is loaded while the one before it is
  // stored, and stored before the loads of the tile that holds its page,
  // which see the wave's own stores: bf16 tokens right before that tile, fp8
  // ones, which may re-encode their page, before the column's first tile.
  WaveToken tok;
  int tok_u = a.tail_route && (t1 > t0 || col == 0) ? (col == 0 ? 0 : uni(s_start[w])) : U;
  auto next_token = [&](bool tiles) -> bool {  // tiles: of routes with tiles, or of bad ones
    // 64 routes at a time: a table may hold many empty ones (64 chats and 192
    // empty rows, their outputs combined by combine_kernel: step 114.9 us one
    // route after another, 91.9 so)
    for (; tok_u < U; tok_u += 64) {
      const int v = tok_u + lane;
      const bool here = v < U && s_pre[min(v, U - 1) + 1] <= t1;
      const uint64_t hit = __ballot(here && s_seq[min(v, U - 1)] < 0 &&
                                    (FP8 || (s_pre[min(v, U - 1) + 1] > s_pre[min(v, U - 1)]) == tiles));
      if (hit) {
        const int u = tok_u + __builtin_ctzll(hit), at = uni(s_n[u]) - 1;
        tok = load_wave_token<FP8>(a, ~uni(s_seq[u]), page_ids[uni(s_base[u]) + at / kPage],
                                   at % kPage, g, lane);
        tok_u = u + 1;
        return true;
      }
      if (__ballot(here) != ~0ull) break;
    }
    tok_u = U;
    return false;
  };
  {
    const int from = tok_u;
    for (bool any = next_token(false); any;) {
      const WaveToken x = tok;
      any = next_token(false);
      store_wave_token<FP8>(a, x, g, lane);
    }
    if constexpr (FP8) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
      tok_u = from;
      next_token(true);
    }
  }
  if (t1 > t0) {
    int u = uni(s_start[w]);
    int tbeg = uni(s_pre[u]), tend = uni(s_pre[u + 1]), base = uni(s_base[u]), n = uni(s_n[u]);
    bool app = uni(s_seq[u]) < 0;

    int t = t0;
    auto tile_info = [&]() -> SpanTile {  // the cursor's tile
      SpanTile x;
      const int p0 = (t - tbeg) * TP, np = (n + kPage - 1) / kPage;
      x.left = n - p0 * kPage;
      x.uf = (uint32_t)u | (t + 1 == tend || t + 1 == t1 ? kSpanLast : 0u) |
             (app && t + 1 == tend ? kSpanToken : 0u);
      auto page_at = [&](int pg) -> int {  // pages past the route read page 0 and are masked
        const bool in = pg < np;
        int v = page_ids[base + (in ? pg : 0)];
        v = in ? v : 0;
        if ((uint32_t)v >= (uint32_t)a.num_pages) {
          x.uf |= kSpanBad;
          v = 0;
        }
        return v;
      };
      x.pid0 = page_at(p0);
      x.pid1 = page_at(p0 + 1);
      x.pid2 = TP > 2 ? page_at(p0 + 2) : 0;
      x.pid3 = TP > 2 ? page_at(p0 + 3) : 0;
      return x;
    };
    auto advance = [&]() {  // to the next tile, if the column has one
      if (t + 1 >= t1) return;
      ++t;
      if (t == tend) {
        // the next route with tiles, 64 at a time (there is one: t < t1)
        for (++u;; u += 64) {
          const uint64_t m = __ballot(s_pre[min(u + lane, U - 1) + 1] > t);
          if (m) {
            u += __builtin_ctzll(m);
            break;
          }
        }
        tbeg = t;
        tend = uni(s_pre[u + 1]);
        base = uni(s_base[u]);
        n = uni(s_n[u]);
        app = uni(s_seq[u]) < 0;
      }
    };

    const int kpage = GeoT::kpage(li), vpage = GeoT::vpage(grp);
    const size_t head_elems = (size_t)kPage * kDim;
    const int koff = GeoT::kslot0(li) * kDim + (FP8 ? 16 : 8) * grp;
    const int voff = li * kPage + GeoT::vslot0(grp);
    auto issue = [&](TileRaw<FP8>& x, const SpanTile& ti) {
      if (!FP8 && (ti.uf & kSpanToken)) {
        store_wave_token<FP8>(a, tok, g, lane);
        next_token(true);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      }
      const int pk = pick4(ti.pid0, ti.pid1, ti.pid2, ti.pid3, kpage);
      const int pv = pick4(ti.pid0, ti.pid1, ti.pid2, ti.pid3, vpage);
      const size_t hk = (HM ? (size_t)g * a.num_pages + pk : (size_t)pk * H + g) * head_elems;
      const size_t hv = (HM ? (size_t)g * a.num_pages + pv : (size_t)pv * H + g) * head_elems;
      if constexpr (!FP8) {
        const uint16_t* kb = static_cast<const uint16_t*>(a.k_pool) + hk + koff;
        const uint16_t* vb = static_cast<const uint16_t*>(a.v_pool) + hv + voff;
#pragma unroll
        for (int cc = 0; cc < NC; ++cc)
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) x.k[cc][kk] = ld16_stream(kb + cc * 4 * kDim + 32 * kk);
#pragma unroll
        for (int b8 = 0; b8 < 8; ++b8) x.v[b8] = ld16_stream(vb + b8 * 16 * kPage);
      } else {
        const uint8_t* kb = static_cast<const uint8_t*>(a.k_pool) + hk + koff;
        const uint8_t* vb = static_cast<const uint8_t*>(a.v_pool) + hv + voff;
#pragma unroll
        for (int cc = 0; cc < NC; ++cc)
#pragma unroll
          for (int pp = 0; pp < 2; ++pp) x.k[cc][pp] = ld16_stream(kb + cc * 4 * kDim + 64 * pp);
#pragma unroll
        for (int b8 = 0; b8 < 8; ++b8) x.v[b8] = ld16_stream(vb + b8 * 16 * kPage);
        x.ks = a.k_scale[(size_t)pv * H + g];
        x.vs = a.v_scale[(size_t)pv * H + g];
      }
    };
    u32x4 qb[4];
    auto load_q = [&](const SpanTile& ti) {
      const int s0 = uni(s_seq[ti.uf & 0xFFFFu]), sq = s0 < 0 ? ~s0 : s0;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const int d0 = FP8 ? 64 * (kk >> 1) + 16 * grp + 8 * (kk & 1) : 32 * kk + 8 * grp;
        qb[kk] = li < G ? ld16(a.q + ((size_t)sq * Hq + hq0 + li) * kDim + d0) : u32x4{0, 0, 0, 0};
      }
    };

    Attn acc;
    reset(acc);
    uint32_t marks = 0;  // of the part's tiles
    const int tok0 = vpage * kPage + GeoT::vslot0(grp);  // the lane's first token within a tile
    auto compute = [&](TileRaw<FP8>& x, const SpanTile& ti) {
      if (ti.left < TP * kPage) mask_tile<FP8>(x, tok0, ti.left);
      float ks = a.scale_log2, vs = 1.0f;
      if constexpr (FP8) {
        ks *= x.ks;
        vs = x.vs;
      }
      marks |= ti.uf;
      attend<FP8, false, true>(x, qb, ks, vs, tok0, ti.left, acc);
    };
    // end of a part: write the route, or hand the part to the workgroup
    auto finish = [&](const SpanTile& ti) {
      float l = acc.l;
      l += __shfl_xor(l, 16);
      l += __shfl_xor(l, 32);
      float m = acc.m;
      const int pu = ti.uf & 0xFFFFu, pb = uni(s_pre[pu]), pe = uni(s_pre[pu + 1]);
      if (marks & kSpanBad) {  // a bad page poisons the route
        m = qnan();
        if (lane == 0) atomicOr(a.err_flags, KF_EFLAG_BAD_PAGE);
      }
      // The lane's place, opaque to the compiler: addresses formed from the
      // loop's own would be hoisted out of it and spilled, and their reload
      // here waits for the tiles in flight.
      int lo = lane;
      asm volatile("" : "+v"(lo));
      const int li = lo & 15, grp = lo >> 4;
      if (pb >= t0 && pe <= t1) {
        const size_t row = (size_t)pu * Hq + hq0 + li;
        if (li < G) {
          const float lw = m != m ? qnan() : l;
#pragma unroll
          for (int b8 = 0; b8 < 8; ++b8) {
            f32x4 o = acc.o[b8];
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] /= lw;
            *reinterpret_cast<f32x4*>(a.o_part + row * kDim + 16 * b8 + 4 * grp) = o;
          }
          if (grp == 0) a.lse_part[row] = (m + __log2f(l)) * kLn2;
        }
      } else {
        const int slot = 2 * w + (pe > t1 ? 1 : 0);
        if (li < G) {
          float* o = s_dyn + (slot * G + li) * kLdsStride;
#pragma unroll
          for (int b8 = 0; b8 < 8; ++b8)
            *reinterpret_cast<f32x4*>(o + 16 * b8 + 4 * grp) = acc.o[b8];
          if (grp == 0) {
            float* ml = s_dyn + 2 * kWaves * G * kLdsStride + (slot * G + li) * 2;
            ml[0] = m;
            ml[1] = l;
          }
        }
        if (lane == 0) s_part[slot] = pu;
      }
      reset(acc);
      marks = 0;
    };

    // ---- two register buffers, as in partial_kernel; the tile in flight may
    // belong to the next route
    TileRaw<FP8> ra, rb;
    SpanTile ia = tile_info();
    load_q(ia);
    issue(ra, ia);
    int left = t1 - t0 - 1;  // tiles after the one in hand
    advance();
    SpanTile ib = tile_info();
    bool final_in_b = false;
    auto one = [&](TileRaw<FP8>& x, const SpanTile& ti, const SpanTile& next) {
      compute(x, ti);
      if (ti.uf & kSpanLast) {
        load_q(next);  // on its way while the part ends
        finish(ti);
      }
    };
    while (true) {
      if (left == 0) break;
      issue(rb, ib);
      --left;
      advance();
      const SpanTile in = tile_info();
      __builtin_amdgcn_sched_barrier(0);
      one(ra, ia, ib);
      if (left == 0) {
        final_in_b = true;
        break;
      }
      ia = in;
      issue(ra, ia);
      --left;
      advance();
      const SpanTile in2 = tile_info();
      __builtin_amdgcn_sched_barrier(0);
      one(rb, ib, ia);
      ib = in2;
    }
    if (final_in_b) {
      compute(rb, ib);
      ia = ib;
    } else {
      compute(ra, ia);
    }
    finish(ia);
  }
  __syncthreads();

  // ---- join the parts of each cut route over the workgroup's columns: every
  // thread forms the weights of its head itself, all loads of a route's parts
  // independent of each other
  constexpr int NP = 2 * kWaves;
  const float* s_ml = s_dyn + NP * G * kLdsStride;
  const int wt0 = sc.begin(min(blk * kWaves, sc.cols));
  const int wt1 = sc.begin(min(blk * kWaves + kWaves, sc.cols));
  int part[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) part[k] = uni(s_part[k]);
  int done = -1;  // a route's parts are in consecutive slots, so each is met once
#pragma unroll 1
  for (int i = 0; i < NP; ++i) {
    const int u = uni(s_part[i]);
    if (u < 0 || u == done) continue;
    done = u;
    const bool whole = s_pre[u] >= wt0 && s_pre[u + 1] <= wt1;
    const size_t rec = ((size_t)(blk + min(u, sc.of(s_pre[u]) / kWaves)) * H + g) * G;
#pragma unroll 1
    for (int e = tid; e < G * (kDim / 4); e += kThreads) {  // four dims of one head
      const int h = e / (kDim / 4), d = e % (kDim / 4) * 4;
      float m[NP], M = neg_inf();
      bool nan = false;
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        m[k] = part[k] == u ? s_ml[(k * G + h) * 2] : neg_inf();
        nan |= m[k] != m[k];
        M = fmaxf(M, m[k]);
      }
      if (nan) M = qnan();
      float L = 0.0f;
      f32x4 O = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < NP; ++k)
        if (part[k] == u) {
          const float wt = m[k] == neg_inf() ? 0.0f : exp2_fast(m[k] - M);
          L += wt * s_ml[(k * G + h) * 2 + 1];
          O += wt * *reinterpret_cast<const f32x4*>(s_dyn + (k * G + h) * kLdsStride + d);
        }
      if (whole) {
        const size_t row = (size_t)u * Hq + hq0 + h;
        *reinterpret_cast<f32x4*>(a.o_part + row * kDim + d) = O / L;
        if (d == 0) a.lse_part[row] = (M + __log2f(L)) * kLn2;
      } else {
        __builtin_nontemporal_store(O, reinterpret_cast<f32x4*>(a.span_o + (rec + h) * kDim + d));
        if (d == 0) {
          a.span_ml[(rec + h) * 2] = M;
          a.span_ml[(rec + h) * 2 + 1] = L;
        }
      }
    }
  }
}

// The dispatch order of a split launch of several rounds.  The hardware
// deals the workgroups of a launch in order over the XCDs and, within an
// XCD, round-robin over its shader engines, and an XCD stops dealing at a
// workgroup whose engine has no free slot: a run of long ranges on one
// engine then idles the others.  Work items (launch position u, KV head,
// range) are therefore listed largest range first (64 size classes), so
// neighbouring workgroups hold ranges of about the same length, and units
// that need no range (empty or bad routes) keep one item for their outputs.
// Which workgroup computes an item does not change any result.  One
// workgroup; the order within a size class follows LDS atomics.  Up to
// kOrderLdsUnits units keep their range count and class in LDS between the
// two passes (more read their routes again).
constexpr int kOrderLdsUnits = 16384;
__global__ __launch_bounds__(1024) void order_kernel(PartialArgs a) {
  __shared__ uint32_t s_count[kOrderBuckets];
  __shared__ uint32_t s_next[kOrderBuckets];
  __shared__ uint16_t s_k[kOrderLdsUnits];
  __shared__ uint8_t s_cls[kOrderLdsUnits];
  const int tid = threadIdx.x, H = a.num_kv_heads, U = a.num_units_routes;
  const bool keep = U <= kOrderLdsUnits;
  if (tid < kOrderBuckets) s_count[tid] = 0;
  __syncthreads();
  // ranges of unit u and the size class of its ranges (0: the largest)
  auto unit = [&](int u, int& k, int& cls) {
    const int r = a.route_list ? a.route_list[u] : u;
    k = 1;
    int size = 0;
    if (r >= 0 && r < a.num_routes) {
      const RouteView rv = read_route(a, r);
      if (!rv.bad && rv.npages > 0) {
        k = (rv.npages + a.chunk_pages - 1) / a.chunk_pages;
        size = (rv.npages + k - 1) / k;
      }
    }
    const int64_t q = (int64_t)size * kOrderBuckets / ((int64_t)a.chunk_pages + 1);
    cls = kOrderBuckets - 1 - (int)(q < kOrderBuckets - 1 ? q : kOrderBuckets - 1);
  };
  for (int u = tid; u < U; u += blockDim.x) {
    int k, cls;
    unit(u, k, cls);
    atomicAdd(&s_count[cls], (uint32_t)(k * H));
    if (keep) {
      s_k[u] = (uint16_t)k;   // k <= max_chunks <= 65535
      s_cls[u] = (uint8_t)cls;
    }
  }
  __syncthreads();
  if (tid == 0) {
    uint32_t run = 0;
    for (int b = 0; b < kOrderBuckets; ++b) {
      s_next[b] = run;
      run += s_count[b];
    }
    a.order[0] = run;
    a.order[1] = 0;
  }
  __syncthreads();
  for (int u = tid; u < U; u += blockDim.x) {
    int k, cls;
    if (keep) {
      k = s_k[u];
      cls = s_cls[u];
    } else {
      unit(u, k, cls);
    }
    const uint32_t pos = atomicAdd(&s_next[cls], (uint32_t)(k * H));
    for (int g = 0; g < H; ++g)
      for (int c = 0; c < k; ++c) {
        const size_t i = pos + (size_t)g * k + c;
        a.order[2 + 2 * i] = (uint32_t)u;
        a.order[3 + 2 * i] = ((uint32_t)g << 16) | (uint32_t)c;
      }
  }
}

// The records of one (launch position, query head): k places, `stride`
// records apart; those in use come first.  k = 0: the outputs are in place.
struct Pieces {
  size_t rec0;
  int stride, k;
};

__device__ __forceinline__ Pieces pieces_of(const RecordArgs& a, int u, int h) {
  const int g = h / a.group, hl = h - g * a.group;
  if (a.span_table) {
    const int first = a.span_table[2 * u], k = a.span_table[2 * u + 1];
    return {((size_t)first * a.num_kv_heads + g) * a.group + hl, a.num_kv_heads * a.group, k};
  }
  return {(((size_t)u * a.num_kv_heads + g) * a.max_chunks) * a.group + hl, a.group, a.max_chunks};
}

// The outputs (dims 2*lane and 2*lane + 1) of eight records of a block from
// `base` on, record j first: WAVES = 1 the next eight, WAVES = 4 every fourth,
// v[q][s] that of record j + 4 * q + s.  Places from cnt on repeat the last
// (branches round the few loads saved made chat batches 1.5% slower).
template <int WAVES>
__device__ __forceinline__ void load_pieces(const RecordArgs& a, const Pieces& p, int base, int j,
                                            int cnt, int lane, float2 (&v)[2 * WAVES][4 / WAVES]) {
  const float2* o = reinterpret_cast<const float2*>(a.o) + lane;
#pragma unroll
  for (int q = 0; q < 2 * WAVES; ++q)
#pragma unroll
    for (int s = 0; s < 4 / WAVES; ++s)
      v[q][s] = o[(p.rec0 + (size_t)(base + min(j + 4 * q + s, cnt - 1)) * p.stride) * (kDim / 2)];
}

// Weighted output sums of up to 64 records (record base + i: weight in lane i
// of wi, bit i of `used` set if it holds anything) added to four subsets of
// records (subset s: s, s + 4, ...), each in record order.  WAVES = 4: this
// wave's subset only; WAVES = 1: all four.  Eight records' loads in flight;
// LOADED: v holds the first eight already.
template <int WAVES, bool LOADED>
__device__ __forceinline__ void piece_sums(const RecordArgs& a, const Pieces& p, int base,
                                           uint64_t used, float wi, int lane, int wave,
                                           float2 (&v)[2 * WAVES][4 / WAVES],
                                           float2 (&acc)[4 / WAVES]) {
  constexpr int NS = 4 / WAVES, UN = 2 * WAVES;
  // places not in use (and ranges whose every score is -inf) add nothing
  const int cnt = used ? 64 - __builtin_clzll(used) : 0, j0 = WAVES == 1 ? 0 : wave;
  for (int j = j0; j < cnt; j += 4 * UN) {
    if (!LOADED || j != j0) load_pieces<WAVES>(a, p, base, j, cnt, lane, v);
#pragma unroll
    for (int q = 0; q < UN; ++q)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int jj = min(j + 4 * q + s, cnt - 1);
        const bool in = j + 4 * q + s < cnt && ((used >> jj) & 1);
        const float wj = read_lane(wi, jj), w = in ? wj : 0.0f;
        // explicit FMAs: the same bits from every instantiation
        acc[s].x = __builtin_fmaf(w, in ? v[q][s].x : 0.0f, acc[s].x);
        acc[s].y = __builtin_fmaf(w, in ? v[q][s].y : 0.0f, acc[s].y);
      }
  }
}

// Reduce the records of one (launch position, query head) to the normalised
// output (the lane's dims) and lse; false: the outputs are already in place.
// WAVES = 4: called by the 256 threads of a workgroup, and the result is wave
// 0's; WAVES = 1: by one wave.  EARLY: the first outputs' loads go out beside
// the (max, sum) loads and not after the weights.  The same bits either way: every wave forms
// the maximum and the sum alike, the outputs add up as ((S0 + S1) + S2) + S3.
template <int WAVES, bool EARLY = false>
__device__ __forceinline__ bool combine_unit(const RecordArgs& a, const Pieces& p, int lane,
                                             int wave, float2 (*s_sum)[64], float2& o, float& lse) {
  if (p.k == 0) return false;
  const float2* ml = reinterpret_cast<const float2*>(a.ml) + p.rec0;
  auto record = [&](int i) -> float2 {
    return i < p.k ? ml[(size_t)i * p.stride] : make_float2(neg_inf(), 0.0f);
  };
  const float2 first = record(lane);  // all of them, with up to 64 places
  float2 v[2 * WAVES][4 / WAVES];
  if constexpr (EARLY)
    load_pieces<WAVES>(a, p, 0, WAVES == 1 ? 0 : wave, min(p.k, 64), lane, v);
  if (__shfl(first.y, 0) == -1.0f) return false;
  float M = first.x;
  for (int i = lane + 64; i < p.k; i += 64) M = fmaxf(M, record(i).x);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) M = fmaxf(M, __shfl_xor(M, m));
  auto weight = [&](float m) { return m == neg_inf() ? 0.0f : exp2_fast(m - M); };
  float w = weight(first.x), L = first.x == neg_inf() ? 0.0f : w * first.y;
  float2 acc[4 / WAVES];
#pragma unroll
  for (int s = 0; s < 4 / WAVES; ++s) acc[s] = make_float2(0.0f, 0.0f);
  piece_sums<WAVES, EARLY>(a, p, 0, __ballot(first.x != neg_inf()), w, lane, wave, v, acc);
  for (int base = 64; base < p.k; base += 64) {
    const float2 r = record(base + lane);
    w = weight(r.x);
    L = r.x == neg_inf() ? L : __builtin_fmaf(w, r.y, L);
    piece_sums<WAVES, false>(a, p, base, __ballot(r.x != neg_inf()), w, lane, wave, v, acc);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) L += __shfl_xor(L, m);
  float2 t;
  if constexpr (WAVES == 4) {
    s_sum[wave][lane] = acc[0];
    __syncthreads();
    t = s_sum[0][lane];
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      t.x += s_sum[s][lane].x;
      t.y += s_sum[s][lane].y;
    }
    __syncthreads();  // s_sum may be used again
  } else {
    t = acc[0];
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      t.x += acc[s].x;
      t.y += acc[s].y;
    }
  }
  o = make_float2(t.x / L, t.y / L);
  lse = (M + __log2f(L)) * kLn2;
  return true;
}

__device__ __forceinline__ void store_row(const RecordArgs& a, int r, int h, int lane, float2 o,
                                          float lse) {
  const size_t row = (size_t)r * a.num_q_heads + h;
  reinterpret_cast<float2*>(a.o_part)[row * (kDim / 2) + lane] = o;
  if (lane == 0) a.lse_part[row] = lse;
}

// Combine up to 64 rows of one query head by one wave: lane i holds launch
// position u (-1: none).  sink(i, o, lse) takes each row that has records;
// returns their lanes (the outputs of the others are in place).  Bound by the
// chain table, (max, sum) and outputs of a row, so four rows of up to four
// records walk it together, 16 lanes holding the (max, sum) pairs of each; a
// row of more records has loads enough of its own and goes alone.
// combine_unit's sums in combine_unit's order: the same bits.  MARKS: marks of
// rows in place are read ahead, one load more in the chain, for tables where
// most rows may be.
template <bool MARKS, class Sink>
__device__ __forceinline__ uint64_t combine_rows(const RecordArgs& a, int u, int h, int lane,
                                                 Sink&& sink) {
  constexpr int R = 4, K = 4, LANES = 64 / R;
  Pieces p{0, 0, 0};
  if (u >= 0) {
    p = pieces_of(a, u, h);
    if (MARKS && p.k > 0 && a.ml[p.rec0 * 2 + 1] == -1.0f) p.k = 0;  // mark_whole
  }
  uint64_t done = 0;
  const int stride = a.span_table ? a.num_kv_heads * a.group : a.group;
  const int rec0 = (int)p.rec0;  // a workspace of 2^31 records would be 1 TB
  const uint64_t many = __ballot(p.k > K);
  const float2* ml = reinterpret_cast<const float2*>(a.ml);
  const float2* out = reinterpret_cast<const float2*>(a.o) + lane;
  for (uint64_t left = __ballot(p.k > 0) & ~many; left;) {
    int row[R], rec[R], k[R], cnt = 0;
#pragma unroll
    for (int s = 0; s < R; ++s) {  // places past the last row repeat the first
      row[s] = left ? __builtin_ctzll(left) : row[0];
      cnt += left != 0;
      left &= left - 1;
      rec[s] = __builtin_amdgcn_readlane(rec0, row[s]);
      k[s] = __builtin_amdgcn_readlane(p.k, row[s]);
    }
    const int ms = lane / LANES, mi = lane % LANES;
    const bool in = mi < pick4(k[0], k[1], k[2], k[3], ms);
    const float2 r = in ? ml[pick4(rec[0], rec[1], rec[2], rec[3], ms) + (size_t)mi * stride]
                        : make_float2(neg_inf(), 0.0f);
    float2 v[R][K];
#pragma unroll
    for (int s = 0; s < R; ++s)
#pragma unroll
      for (int q = 0; q < K; ++q)
        v[s][q] = out[(rec[s] + (size_t)min(q, k[s] - 1) * stride) * (kDim / 2)];
    float M = r.x;
#pragma unroll
    for (int m = K / 2; m >= 1; m >>= 1) M = fmaxf(M, __shfl_xor(M, m));
    const float w = r.x == neg_inf() ? 0.0f : exp2_fast(r.x - M);
    float L = r.x == neg_inf() ? 0.0f : w * r.y;
#pragma unroll
    for (int m = K / 2; m >= 1; m >>= 1) L += __shfl_xor(L, m);
    const uint64_t used = __ballot(r.x != neg_inf());
#pragma unroll
    for (int s = 0; s < R; ++s) {
      if (s >= cnt) break;
      if (read_lane(r.y, LANES * s) == -1.0f) continue;  // in place
      done |= 1ull << row[s];
      float2 t = make_float2(0.0f, 0.0f);
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const int i = LANES * s + q;
        const bool has = (used >> i) & 1;
        const float wj = has ? read_lane(w, i) : 0.0f;
        // a subset's only record, rounded before it is added
        t.x += __builtin_fmaf(wj, has ? v[s][q].x : 0.0f, 0.0f);
        t.y += __builtin_fmaf(wj, has ? v[s][q].y : 0.0f, 0.0f);
      }
      const float Ls = read_lane(L, LANES * s), Ms = read_lane(M, LANES * s);
      sink(row[s], make_float2(t.x / Ls, t.y / Ls), (Ms + __log2f(Ls)) * kLn2);
    }
  }
  for (uint64_t left = many; left; left &= left - 1) {
    const int i = __builtin_ctzll(left);
    float2 o;
    float lse;
    if (!combine_unit<1>(a, {(size_t)__builtin_amdgcn_readlane(rec0, i), stride,
                             __builtin_amdgcn_readlane(p.k, i)},
                         lane, 0, nullptr, o, lse))
      continue;
    done |= 1ull << i;
    sink(i, o, lse);
  }
  return done;
}

// Small and bound by its chain of dependent loads, so the chain is short:
// every (max, sum) of a head arrives in one load and its weights are read
// across lanes, no route row is read (mark_whole), eight records' outputs are
// in flight, and the records themselves are written past the L2
// (non-temporal), where the next kernel finds them on every XCD.  Of 164 units
// with 16 heads and 13 ranges: 18.3 -> 10 us.
//
// Combine the records of each (launch position, query head) whose outputs are
// not in place yet: one wave each (four heads per workgroup), or, with many
// records, the four waves of a workgroup.
template <int WAVES, bool EARLY>
__global__ __launch_bounds__(kThreads) void combine_kernel(RecordArgs a) {
  __shared__ float2 s_sum[4][64];
  const int u = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = WAVES == 4 ? blockIdx.x : blockIdx.x * 4 + wave;
  if (h >= a.num_q_heads) return;
  const int r = a.route_list ? a.route_list[u] : u;
  if (r < 0 || r >= a.num_routes) return;  // flagged by partial_kernel
  float2 o;
  float lse;
  if (combine_unit<WAVES, EARLY>(a, pieces_of(a, u, h), lane, wave, s_sum, o, lse) &&
      (WAVES == 1 || wave == 0))
    store_row(a, r, h, lane, o, lse);
}

// ------------------------------------------------------------------- gather
// Test export: the resident tokens of one route copied out through the same
// route checks (read_route) and page lookup as the attention kernels.  Block
// p copies route-local page p: out[j][g][:] for j = 16 p + slot.
template <class T>
__global__ __launch_bounds__(256) void gather_kernel(PartialArgs a, int route, int max_tokens,
                                                     T* out_k, T* out_v) {
  const int p = blockIdx.x, tid = threadIdx.x, H = a.num_kv_heads;
  const RouteView rv = read_route(a, route);
  if (rv.bad) {
    if (p == 0 && tid == 0) atomicOr(a.err_flags, KF_EFLAG_BAD_ROUTE);
    return;
  }
  const int n = min(rv.n, max_tokens);
  if (p * kPage >= n) return;
  const int pid = a.page_ids[rv.base + p];
  if (pid < 0 || pid >= a.num_pages) {
    if (tid == 0) atomicOr(a.err_flags, KF_EFLAG_BAD_PAGE);
    return;
  }
  const T* kp = static_cast<const T*>(a.k_pool);
  const T* vp = static_cast<const T*>(a.v_pool);
  for (int e = tid; e < H * kPage * kDim; e += blockDim.x) {
    const int g = e / (kPage * kDim), slot = (e / kDim) % kPage, d = e % kDim;
    const int j = p * kPage + slot;
    if (j >= n) continue;
    const size_t head = pool_slice(pid, g, H, a.num_pages, a.head_major);
    out_k[((size_t)j * H + g) * kDim + d] = kp[(head * kPage + slot) * kDim + d];
    out_v[((size_t)j * H + g) * kDim + d] = vp[(head * kDim + d) * kPage + slot];
  }
}

// -------------------------------------------------------------------- merge
// The append decision of sequence b in a fused step, with append_kernel's
// checks and flags: 0 = no append, 1 = appended, else an error flag.
__device__ __forceinline__ int tail_append_status(const MergeArgs& a, int b, int& r) {
  r = a.tail_route[b];
  if (r < 0) return 0;
  if (r >= a.num_routes) return KF_EFLAG_BAD_ROUTE << 8;
  const int32_t* rp = reinterpret_cast<const int32_t*>(a.routes + r);
  const int seq = rp[0], tb = rp[2], te = rp[3], base = rp[4], cap = rp[5];
  const int j = te - tb;
  if (seq != b || j < 0) return KF_EFLAG_BAD_ROUTE << 8;
  if (j / kPage >= cap) return KF_EFLAG_TAIL_FULL << 8;
  if (base < 0 || (int64_t)base + j / kPage >= a.num_page_ids) return KF_EFLAG_BAD_ROUTE << 8;
  const int pid = a.page_ids[base + j / kPage];
  if (pid < 0 || pid >= a.num_pages) return KF_EFLAG_BAD_PAGE << 8;
  return 1;
}

// Bound by reading the rows once more rows arrive than one wave's loads in
// flight cover: 128 rows per sequence (32 sequences, 32 heads, 68 MB) took
// 16.1 us with one wave of four loads, 12.5 us with four waves of eight (16
// each: 13.2); below eight rows a sequence one wave is enough.  A wave's first
// eight rows are loaded beside their lse, not after the weights, and only rows
// that there are: 128 rows 12.5 -> 12.3 us, 32 to 100
// sequences of 3 or 4 rows 4.2 -> 3.75.
//
// Sequence b's rows r0 .. r0 + n - 1 of query head h merged by WAVES waves;
// lane holds dims 2*lane, 2*lane+1.  Rows are summed in four subsets (subset
// s: rows s, s + 4, ...), each in row order, then ((S0 + S1) + S2) + S3: the
// same bits for one wave and for four.
template <int WAVES>
__device__ __forceinline__ void merge_rows(const MergeArgs& a, int b, int h, int r0, int n, int lane,
                                           int wave, float3 (*s_sum)[64], float* s_max) {
  constexpr float kLog2e = 1.44269504088896340736f;
  constexpr int NS = 4 / WAVES, UN = 8 / NS;  // eight rows' loads in flight
  const int Hq = a.num_q_heads;
  const float* lse = a.lse_part + (size_t)r0 * Hq + h;
  float2* out = reinterpret_cast<float2*>(a.out + ((size_t)b * Hq + h) * kDim) + lane;
  float* lse_out = a.lse_out + (size_t)b * Hq + h;
  constexpr int BLOCK = 64 * WAVES;  // rows whose weights one block of lanes holds
  const size_t rs = (size_t)Hq * kDim / 2;  // float2 elements from one row to the next
  const float2* o = reinterpret_cast<const float2*>(a.o_part + ((size_t)r0 * Hq + h) * kDim) + lane;
  // the lane's row of a block (one wave: base + lane), and the wave's first row
  const int mine = WAVES == 1 ? lane : 4 * lane + wave, j0 = WAVES == 1 ? 0 : wave;
  const float first = mine < n ? lse[(size_t)mine * Hq] : neg_inf();
  float2 v[UN][NS];
  auto load = [&](int base, int j) {  // rows that there are: n and j are uniform
#pragma unroll
    for (int q = 0; q < UN; ++q)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        v[q][s] = make_float2(0.0f, 0.0f);
        if (base + j + 4 * q + s < n) v[q][s] = o[(size_t)(base + j + 4 * q + s) * rs];
      }
  };
  load(0, j0);
  float M = first;
  bool nan_seen = first != first;
  for (int i = mine + BLOCK; i < n; i += BLOCK) {
    const float l = lse[(size_t)i * Hq];
    nan_seen |= l != l;
    M = fmaxf(M, l);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) M = fmaxf(M, __shfl_xor(M, m));
  if (__ballot(nan_seen) != 0) M = qnan();
  if constexpr (WAVES == 4) {
    if (lane == 0) s_max[wave] = M;
    __syncthreads();
    M = neg_inf();
    bool any = false;
    for (int w = 0; w < 4; ++w) {
      any |= s_max[w] != s_max[w];
      M = fmaxf(M, s_max[w]);
    }
    if (any) M = qnan();
  }
  if (M != M || M == neg_inf()) {  // a NaN row; no rows or only empty ones
    if (WAVES == 1 || wave == 0) {
      const float v = M != M ? qnan() : 0.0f;
      *out = make_float2(v, v);
      if (lane == 0) *lse_out = M;
    }
    return;
  }
  float3 acc[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) acc[s] = make_float3(0.0f, 0.0f, 0.0f);
  for (int base = 0; base < n; base += BLOCK) {
    const int i = base + mine;
    const float l = base == 0 ? first : i < n ? lse[(size_t)i * Hq] : neg_inf();
    const float wl = i < n ? exp2_fast((l - M) * kLog2e) : 0.0f;
    const int cnt = min(BLOCK, n - base);
    for (int j = j0; j < cnt; j += 4 * UN) {
      if (base + j > j0) load(base, j);
#pragma unroll
      for (int q = 0; q < UN; ++q)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const int jj = j + 4 * q + s, jc = min(jj, cnt - 1);
          const float wj = read_lane(wl, WAVES == 1 ? jc : jc >> 2);
          const float wr = jj < cnt ? wj : 0.0f;
          acc[s].x = __builtin_fmaf(wr, v[q][s].x, acc[s].x);
          acc[s].y = __builtin_fmaf(wr, v[q][s].y, acc[s].y);
          acc[s].z += wr;
        }
    }
  }
  float3 t;
  if constexpr (WAVES == 4) {
    s_sum[wave][lane] = acc[0];
    __syncthreads();
    if (wave != 0) return;
    t = s_sum[0][lane];
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      t.x += s_sum[s][lane].x;
      t.y += s_sum[s][lane].y;
      t.z += s_sum[s][lane].z;
    }
  } else {
    t = acc[0];
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      t.x += acc[s].x;
      t.y += acc[s].y;
      t.z += acc[s].z;
    }
  }
  *out = make_float2(t.x / t.z, t.y / t.z);
  if (lane == 0) *lse_out = M + __logf(t.z);
}

// merge_rows<1> over rows held in LDS (n <= kLdsRows), by one wave; the same
// order of sums, so the same bits.
__device__ __forceinline__ void merge_lds_rows(const MergeArgs& a, int b, int h, int n, int lane,
                                               const float2 (*s_row)[64], const float* s_lse) {
  constexpr float kLog2e = 1.44269504088896340736f;
  const size_t at = (size_t)b * a.num_q_heads + h;
  float2* out = reinterpret_cast<float2*>(a.out + at * kDim) + lane;
  const float l = lane < n ? s_lse[lane] : neg_inf();
  float M = l;
#pragma unroll
  for (int m = kLdsRows / 2; m >= 1; m >>= 1) M = fmaxf(M, __shfl_xor(M, m));
  M = read_lane(M, 0);
  const bool nan = __ballot(l != l) != 0;
  if (nan || M == neg_inf()) {
    const float v = nan ? qnan() : 0.0f;
    *out = make_float2(v, v);
    if (lane == 0) a.lse_out[at] = nan ? qnan() : neg_inf();
    return;
  }
  const float wl = lane < n ? exp2_fast((l - M) * kLog2e) : 0.0f;
  float3 acc[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[s] = make_float3(0.0f, 0.0f, 0.0f);
  for (int j = 0; j < n; j += 4)
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (j + s < n) {
        const float w = read_lane(wl, j + s);
        const float2 v = s_row[j + s][lane];
        acc[s].x = __builtin_fmaf(w, v.x, acc[s].x);
        acc[s].y = __builtin_fmaf(w, v.y, acc[s].y);
        acc[s].z += w;
      }
  float3 t = acc[0];
#pragma unroll
  for (int s = 1; s < 4; ++s) {
    t.x += acc[s].x;
    t.y += acc[s].y;
    t.z += acc[s].z;
  }
  *out = make_float2(t.x / t.z, t.y / t.z);
  if (lane == 0) a.lse_out[at] = M + __logf(t.z);
}

// A fused step's bookkeeping for workgroup b of num_seqs: sequence b's tail
// moves past its new token (or raises the append's flag); with RECORDS, the
// routes that no valid CSR row lists under their own sequence, which no merge
// workgroup is sure to visit, have their records combined here.
template <int WAVES, bool RECORDS>
__device__ __forceinline__ void step_bookkeeping(const MergeArgs& a, int b, int lane, int wave) {
  if (threadIdx.x == 0) {
    int r = 0;
    const int st = tail_append_status(a, b, r);
    if (st == 1)
      a.routes[r].tok_end += 1;  // no other wave of this launch reads it
    else if (st)
      atomicOr(a.err_flags, st >> 8);
  }
  if constexpr (RECORDS) {
    // every wave takes 64 rows and a share of the heads; there are at least
    // as many waves as blocks of rows (merge_combines)
    const int blocks = (a.num_routes + 63) / 64, id = b * WAVES + wave;
    const int share = a.num_seqs * WAVES / blocks;
    if (id >= share * blocks) return;
    const int u = id % blocks * 64 + lane;
    bool orphan = false;
    if (u < a.num_routes) {
      const int seq = a.routes[u].seq;
      orphan = seq < 0 || seq >= a.num_seqs;
      if (!orphan) {
        const int r0 = a.seq_route_begin[seq], r1 = a.seq_route_begin[seq + 1];
        orphan = r0 < 0 || r1 > a.num_routes || u < r0 || u >= r1;
      }
    }
    if (__ballot(orphan) == 0) return;
    for (int h = id / blocks; h < a.num_q_heads; h += share)
      combine_rows<true>(a.rec, orphan ? u : -1, h, lane, [&](int i, float2 o, float lse) {
        store_row(a.rec, id % blocks * 64 + i, h, lane, o, lse);
      });
  }
}

// Merge of sequence blockIdx.y's query head blockIdx.x by WAVES waves.  A
// fused step has one more workgroup per sequence, for its bookkeeping.  With
// RECORDS (a fused step of a split launch) the workgroup first combines its
// rows' records; up to kLdsRows rows stay in LDS for the merge.
template <int WAVES, bool RECORDS>
__global__ __launch_bounds__(64 * WAVES) void merge_kernel(MergeArgs a) {
  __shared__ float3 s_sum[WAVES][64];
  __shared__ float s_max[WAVES];
  const int h = blockIdx.x, b = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int Hq = a.num_q_heads;
  if (h == Hq) {
    step_bookkeeping<WAVES, RECORDS>(a, b, lane, wave);
    return;
  }
  const int r0 = a.seq_route_begin[b], r1 = a.seq_route_begin[b + 1];
  if (r0 < 0 || r1 < r0 || r1 > a.num_routes) {
    if (threadIdx.x < 64)
      reinterpret_cast<float2*>(a.out + ((size_t)b * Hq + h) * kDim)[lane] =
          make_float2(qnan(), qnan());
    if (threadIdx.x == 0) {
      a.lse_out[(size_t)b * Hq + h] = qnan();
      if (h == 0) atomicOr(a.err_flags, KF_EFLAG_BAD_ROUTE);
    }
    return;
  }
  if constexpr (RECORDS) {
    __shared__ float2 s_row[kLdsRows][64];
    __shared__ float2 s_rec[WAVES][64];
    __shared__ float s_lse[kLdsRows];
    const int n = r1 - r0;
    if (n == 1) {
      const size_t row = (size_t)r0 * Hq + h;
      // a whole unit's row is in place; its loads go out with the records'
      float2 o = reinterpret_cast<const float2*>(a.o_part)[row * (kDim / 2) + lane];
      float lse = a.lse_part[row];
      const Pieces p = pieces_of(a.rec, r0, h);
      const bool share = WAVES == 4 && p.k > kRecordsOneWave;
      if (wave != 0 && !share) return;
      const bool got = WAVES == 4 && share
                           ? combine_unit<WAVES>(a.rec, p, lane, wave, s_rec, o, lse)
                           : combine_unit<1>(a.rec, p, lane, wave, s_rec, o, lse);
      if (wave != 0) return;
      if (got) store_row(a.rec, r0, h, lane, o, lse);
      s_row[0][lane] = o;
      if (lane == 0) s_lse[0] = lse;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      merge_lds_rows(a, b, h, 1, lane, s_row, s_lse);
      return;
    }
    if (n <= kLdsRows) {  // lane i of a wave: row i * WAVES + wave
      constexpr int PER = kLdsRows / WAVES;
      float2 o[PER];
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (i * WAVES + wave < n)
          o[i] = reinterpret_cast<const float2*>(
              a.o_part)[((size_t)(r0 + i * WAVES + wave) * Hq + h) * (kDim / 2) + lane];
      const int mine = lane * WAVES + wave;
      const float lse = mine < n ? a.lse_part[(size_t)(r0 + mine) * Hq + h] : 0.0f;
      const uint64_t got = combine_rows<false>(
          a.rec, mine < n ? r0 + mine : -1, h, lane, [&](int i, float2 oi, float li) {
            const int row = i * WAVES + wave;
            store_row(a.rec, r0 + row, h, lane, oi, li);
            s_row[row][lane] = oi;
            if (lane == 0) s_lse[row] = li;
          });
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (i * WAVES + wave < n && !((got >> i) & 1)) s_row[i * WAVES + wave][lane] = o[i];
      if (mine < n && !((got >> lane) & 1)) s_lse[mine] = lse;
      __syncthreads();
      if (wave == 0) merge_lds_rows(a, b, h, n, lane, s_row, s_lse);
      return;
    }
    for (int base = 0; base < n; base += 64 * WAVES) {
      const int first = r0 + base + wave, mine = base + lane * WAVES + wave;
      combine_rows<true>(a.rec, mine < n ? r0 + mine : -1, h, lane, [&](int i, float2 o, float lse) {
        store_row(a.rec, first + i * WAVES, h, lane, o, lse);
      });
    }
    publish_to_workgroup();  // the rows written above, before the merge reads them
  }
  merge_rows<WAVES>(a, b, h, r0, r1 - r0, lane, wave, s_sum, s_max);
}

template <bool FP8, int UPW>
hipError_t launch_partial_kernel(const PartialArgs& a, dim3 grid, hipStream_t stream) {
  if (a.head_major)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(partial_kernel<FP8, UPW, true>), grid, dim3(kThreads * UPW), 0,
                       stream, a);
  else
    hipLaunchKernelGGL(HIP_KERNEL_NAME(partial_kernel<FP8, UPW, false>), grid, dim3(kThreads * UPW), 0,
                       stream, a);
  return hipGetLastError();
}

template <bool FP8>
hipError_t launch_span_kernel(const PartialArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)(a.span_cols / kWaves * a.num_kv_heads));
  const size_t lds = span_lds_bytes(a.group, a.num_units_routes);
  if (a.head_major)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(span_kernel<FP8, true>), grid, dim3(kThreads), lds, stream, a);
  else
    hipLaunchKernelGGL(HIP_KERNEL_NAME(span_kernel<FP8, false>), grid, dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

template <bool EARLY>
hipError_t launch_combine(const RecordArgs& rec, int num_launch, hipStream_t stream) {
  if (rec.places > kChunksOneWave)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(combine_kernel<4, EARLY>),
                       dim3(rec.num_q_heads, num_launch), dim3(kThreads), 0, stream, rec);
  else
    hipLaunchKernelGGL(HIP_KERNEL_NAME(combine_kernel<1, EARLY>),
                       dim3((rec.num_q_heads + 3) / 4, num_launch), dim3(kThreads), 0, stream, rec);
  return hipGetLastError();
}

}  // namespace

// ------------------------------------------------------------------ scratch
// Chunk partials of kf_decode_step_no_alloc: a fixed array in device memory
// that the runtime sets up with the code object on each device, so that the
// call allocates nothing.  Host code never uses the array's name as an
// address: the per-device address comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[KF_SCRATCH_BYTES];

namespace {
constexpr int kScratchDevices = 64;
std::atomic<void*> g_scratch_ptr[kScratchDevices];
std::mutex g_scratch_mu;
}  // namespace

hipError_t scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (!p) {
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return e;
      if (!p) return hipErrorInvalidSymbol;
      g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
  }
  *out = p;
  return hipSuccess;
}

hipError_t launch_append(const AppendArgs& a, bool fp8, hipStream_t stream) {
  if (a.num_seqs == 0) return hipSuccess;
  // a wave per KV head (fp8: and one for K, one for V), at most 16
  const int waves = fp8 ? 2 * a.num_kv_heads : a.num_kv_heads;
  const dim3 block(64 * (waves < 16 ? waves : 16));
  if (fp8)
    hipLaunchKernelGGL(append_kernel<true>, dim3(a.num_seqs), block, 0, stream, a);
  else
    hipLaunchKernelGGL(append_kernel<false>, dim3(a.num_seqs), block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_partial(const PartialArgs& a, bool fp8, hipStream_t stream) {
  if (a.num_units_routes == 0) return hipSuccess;
  const RecordArgs rec = records_of(a);
  if (a.span_cols > 0) {
    const hipError_t es = fp8 ? launch_span_kernel<true>(a, stream) : launch_span_kernel<false>(a, stream);
    if (es != hipSuccess || a.merge_combines) return es;
    return launch_combine<false>(rec, a.num_units_routes, stream);
  }
  if (!fp8 && a.units_per_wg == 2)
    return launch_partial_kernel<false, 2>(a, dim3(1, a.num_kv_heads, (a.num_units_routes + 1) / 2),
                                           stream);
  const dim3 grid(a.max_chunks, a.num_kv_heads, a.num_units_routes);
  if (a.order) {
    hipLaunchKernelGGL(order_kernel, dim3(1), dim3(1024), 0, stream, a);
    const hipError_t eo = hipGetLastError();
    if (eo != hipSuccess) return eo;
  }
  hipError_t e = fp8 ? launch_partial_kernel<true, 1>(a, grid, stream)
                     : launch_partial_kernel<false, 1>(a, grid, stream);
  if (e != hipSuccess || a.max_chunks == 1 || a.merge_combines) return e;
  // Early output loads pay where almost all record places are in use, as in
  // equal tables, and the launch is small enough for its latency to count
  // (4096 tokens, 2 KV heads: step 13.9 -> 13.2 us); in a ragged one
  // the loads of unused places cost more (8 chats: 20.5 -> 20.8 us).
  if (!a.route_list && (int64_t)a.num_units_routes * a.num_q_heads <= kEarlyRecordHeads &&
      !ragged_table(a.num_page_ids, a.num_units_routes, a.max_pages_per_route))
    return launch_combine<true>(rec, a.num_units_routes, stream);
  return launch_combine<false>(rec, a.num_units_routes, stream);
}

hipError_t launch_gather(const PartialArgs& a, bool fp8, int route, int max_tokens, void* out_k,
                         void* out_v, hipStream_t stream) {
  const int blocks = (max_tokens + kPage - 1) / kPage;
  if (blocks == 0) return hipSuccess;
  if (fp8)
    hipLaunchKernelGGL(gather_kernel<uint8_t>, dim3(blocks), dim3(256), 0, stream, a, route,
                       max_tokens, static_cast<uint8_t*>(out_k), static_cast<uint8_t*>(out_v));
  else
    hipLaunchKernelGGL(gather_kernel<uint16_t>, dim3(blocks), dim3(256), 0, stream, a, route,
                       max_tokens, static_cast<uint16_t*>(out_k), static_cast<uint16_t*>(out_v));
  return hipGetLastError();
}

hipError_t launch_merge(const MergeArgs& a, hipStream_t stream) {
  if (a.num_seqs == 0 || a.num_q_heads == 0) return hipSuccess;
  const dim3 grid(a.num_q_heads + (a.tail_route ? 1 : 0), a.num_seqs);
  const int rows = a.num_routes / a.num_seqs;  // mean rows per sequence
  // One wave per head leaves no idle waves where grids are large (64 sequences
  // of 64 heads: step 68.3 us, with four 73.6; 217 of 8: 28.0 and 29.2; 119 of
  // 8: 13.4 and 14.1); in small ones four waves cost nothing (8 of 32 heads: 23.9
  // and 24.0) and take a sequence of many rows faster (16 rows beside 15
  // sequences of 64 heads, one wave 40.9, four 33.6).
  if (a.rec.ml && wide_merge(a.num_seqs, a.num_q_heads) && (rows > 0 ? rows : 1) * a.rec.places <= kRecordsOneWave)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(merge_kernel<1, true>), grid, dim3(64), 0, stream, a);
  else if (a.rec.ml)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(merge_kernel<4, true>), grid, dim3(256), 0, stream, a);
  else if (rows >= kMergeRowsFourWaves)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(merge_kernel<4, false>), grid, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(HIP_KERNEL_NAME(merge_kernel<1, false>), grid, dim3(64), 0, stream, a);
  return hipGetLastError();
}

}  // namespace kf
