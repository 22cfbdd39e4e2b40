// Bulk query of a PHOBIC MPHF on the device (Sec. 4, "Hash Function": the position of key x with
// pilot p in a partition of m slots is (h(x, floor(p / m)) + p) mod m, plus the partition offset).
//
// One thread per key.  Per key: hash -> partition j -> two offset residues (adjacent, compact) ->
// bucket i by the tabulated bucket function -> encoder i entry j (Compact: one fixed-width field;
// Rice: low bits plus the unary high part located through the select samples) -> position.
// The image (tens of MB at 10^8 keys) stays resident; the accesses per key are a handful of
// dependent cache-line reads that mostly hit the L2 / Infinity Cache.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <cstring>
#include <string>
#include <vector>

#include "phobic_internal.h"

namespace phobic {
namespace {

constexpr int kQBlock = 256;

// From the select entry e of the block holding one ta: the position of a one at or before one ta
// (the block's sample, or its sub-sample when ta lies past one and the distance was stored), and in
// r how many ones separate the two.
__device__ __forceinline__ uint64_t sel_start(uint64_t e, uint64_t ta, uint32_t& r) {
  const uint32_t left = (uint32_t)(ta % kSelBlock), k = left / kSelSub;
  const uint32_t rel = k ? (uint32_t)(e >> (32 + 10 * (k - 1))) & 1023u : kSelRelNone;
  const bool sub = rel != kSelRelNone;
  r = sub ? left % kSelSub : left;
  return (e & 0xFFFFFFFFULL) + (sub ? rel : 0u);
}

// The lookups are bound by their cache requests, so every field is read with one load: sections are
// read at 4-byte steps, where 8 bytes hold any field of up to 33 bits and 12 any pair of up to 65.
// Each section ends in a zero word, so the bytes past the last field are inside the image.  With aligned
// 8-byte reads and a second one where a field straddles, and the unary stream read a word at a time,
// the same lookups took longer: 1M keys of a 10^8-key table 38.9 -> 35.2 us, 1000 keys of a 10^6-key
// table 9.2 -> 8.0 us (a launch in a queue of them), all 10^8 keys of a build 3.07 -> 2.62 ms.
typedef uint64_t u64_at4 __attribute__((aligned(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_at4 __attribute__((aligned(4)));

// The field of w <= 32 bits at bit pos.
__device__ __forceinline__ uint32_t field32(const uint64_t* __restrict__ sec, uint64_t pos, uint32_t w) {
  const uint64_t v = *(const u64_at4*)((const uint32_t*)sec + (pos >> 5)) >> (pos & 31);
  return (uint32_t)(v & ((1ULL << w) - 1));
}

// The residues of offsets j and j + 1, adjacent fields of woff bits (the same for all lookups).
__device__ __forceinline__ void offset_pair(const uint64_t* __restrict__ offs, uint64_t j, uint32_t woff,
                                            uint64_t& r0, uint64_t& r1) {
  const uint64_t pos = j * woff;
  const uint64_t mask = (1ULL << woff) - 1;
  if (woff == 0) {
    r0 = r1 = 0;
  } else if (woff <= 16) {
    const uint64_t v = *(const u64_at4*)((const uint32_t*)offs + (pos >> 5)) >> (pos & 31);
    r0 = v & mask;
    r1 = (v >> woff) & mask;
  } else if (woff <= 32) {
    const uint32_t* p = (const uint32_t*)offs + (pos >> 5);
    const uint32_t sh = (uint32_t)(pos & 31);
    const uint64_t lo = *(const u64_at4*)p;
    const uint64_t v = sh ? (lo >> sh) | ((uint64_t)p[2] << (64 - sh)) : lo;
    r0 = v & mask;
    r1 = (v >> woff) & mask;
  } else {
    r0 = get_bits(offs, pos, woff);
    r1 = get_bits(offs, pos + woff, woff);
  }
}

// 128 bits of the unary stream from bit `base` (a multiple of 32) on, and how far the search for a value
// has come: `need` ones of the window precede the value's own one, `last` is the position of the one
// before the window (of value t - 1, if need is 0).
struct UnaryWindow {
  uint64_t lo, hi, last;
  uint64_t base;
  uint32_t need;
};
__device__ __forceinline__ void unary_load(const uint64_t* __restrict__ un, UnaryWindow& w) {
  const u32x4 v = *(const u32x4_at4*)((const uint32_t*)un + (w.base >> 5));
  w.lo = ((uint64_t)v.y << 32) | v.x;
  w.hi = ((uint64_t)v.w << 32) | v.z;
}
// Whether the value's one lies past the window; the search then moves on by a window (not loaded yet).
__device__ __forceinline__ bool unary_past(UnaryWindow& w) {
  const uint32_t c = __popcll(w.lo) + __popcll(w.hi);
  if (w.need < c) return false;
  if (c) w.last = w.base + (w.hi ? 127 - __clzll((long long)w.hi) : 63 - __clzll((long long)w.lo));
  w.need -= c;
  w.base += 128;
  return true;
}
// q = distance of the value's one from the one before it, less one.
__device__ __forceinline__ uint32_t unary_value(const UnaryWindow& w) {
  uint64_t lo = w.lo, hi = w.hi, prev = w.last;
  if (w.need) {  // the one before lies in the window: number need - 1 of it
    const uint32_t c0 = __popcll(lo), k = w.need - 1;
    const bool up = k >= c0;
    const uint32_t b = select_in_word(up ? hi : lo, up ? k - c0 : k);
    const uint64_t above = b == 63 ? 0 : ~0ULL << (b + 1);
    prev = w.base + b + (up ? 64 : 0);
    lo = up ? 0 : lo & above;
    hi = up ? hi & above : hi;
  }
  const uint64_t cur = w.base + (lo ? (uint32_t)__ffsll((long long)lo) - 1 : 63 + (uint32_t)__ffsll((long long)hi));
  return (uint32_t)(cur - prev - 1);
}

// bucket_of over a table held in 64-bit words, or in 32-bit words where the last point, 2^32, reads
// as 0: the difference of two points is then still right modulo 2^32, and it is below 2^32.  Every
// other point is below 2^32 (the bucket functions stay below 1 short of x = 1 by far more than 2^-32).
__device__ __forceinline__ uint32_t bucket_of_tab(uint64_t lo, const uint64_t* __restrict__ T, uint32_t B) {
  return bucket_of(lo, T, B);
}
__device__ __forceinline__ uint32_t bucket_of_tab(uint64_t lo, const uint32_t* __restrict__ T, uint32_t B) {
  const uint32_t k = (uint32_t)(lo >> 53);
  const uint64_t f = (lo >> 21) & 0xFFFFFFFFULL;
  const uint32_t t0 = T[k], t1 = T[k + 1];
  const uint64_t y = (uint64_t)t0 + (((uint64_t)(uint32_t)(t1 - t0) * f) >> 32);
  const uint32_t b = (uint32_t)((y * B) >> 32);
  return b < B - 1 ? b : B - 1;
}

// kN lookups per thread in lockstep: every stage issues the reads of all kN lookups before any of
// them is consumed, so one wavefront keeps kN times as many independent cache-line reads in flight
// (the query is bound by the latency of its chain of dependent reads, not by bandwidth).
template <int kN, typename TabT>
__device__ __forceinline__ void query_codes(const QueryArgs& a, const TabT* __restrict__ T,
                                            const uint64_t* __restrict__ E, const uint64_t (&hi)[kN],
                                            const uint64_t (&lo)[kN], uint64_t (&res)[kN]) {
  const uint64_t* __restrict__ offs = a.img + a.sec_off;
  const uint64_t* __restrict__ un = a.img + a.sec_unary;
  const uint64_t* __restrict__ sel = a.img + a.sec_sel;
  const bool rice = a.coding == PHOBIC_IC_RICE;
  uint64_t j[kN], e[kN], r0[kN], r1[kN];
  uint32_t i[kN], p[kN];  // pilots are at most 2^32 - 1
#pragma unroll
  for (int q = 0; q < kN; q++) {
    j[q] = __umul64hi(hi[q], a.K);
    i[q] = bucket_of_tab(lo[q], T, a.B);
  }
#pragma unroll
  for (int q = 0; q < kN; q++) e[q] = E[i[q]];
  // offsets, low bits and select samples: independent of each other.  A lookup whose encoder is
  // Rice (u) reads the unary stream at its value t = (i - ncompact) K + j; one of a Compact encoder
  // (all of a Compact image, the first ncompact of a mixed one) is done with its field.
  uint64_t t[kN], sample[kN];
  bool u[kN];
#pragma unroll
  for (int q = 0; q < kN; q++) {
    offset_pair(offs, j[q], a.woff, r0[q], r1[q]);
    const uint32_t w = (uint32_t)(e[q] & 0xFF);
    p[q] = field32(a.img + a.sec_data, (e[q] >> 8) + j[q] * w, w);
    u[q] = rice && i[q] >= a.ncompact;
    t[q] = u[q] ? (uint64_t)(i[q] - a.ncompact) * a.K + j[q] : 0;
    sample[q] = u[q] ? sel[(t[q] ? t[q] - 1 : 0) / kSelBlock] : 0;
  }
  if (rice) {
    UnaryWindow w[kN];
    bool more[kN];
#pragma unroll
    for (int q = 0; q < kN; q++) {
      uint32_t r = 0;
      const uint64_t start = t[q] ? sel_start(sample[q], t[q] - 1, r) : 0;
      w[q].base = start & ~31ULL;
      w[q].need = t[q] ? r + 1 : 0;  // ones from `start` on before the value's own
      w[q].last = ~0ULL;             // value 0: the one before is at -1
      w[q].lo = w[q].hi = 1;         // a Compact lookup is done
      if (u[q]) {
        unary_load(un, w[q]);
        w[q].lo &= ~0ULL << (start & 31);
      }
    }
    // most windows hold the value's one; the others go on
    bool any = false;
#pragma unroll
    for (int q = 0; q < kN; q++) {
      more[q] = u[q] && unary_past(w[q]);
      any |= more[q];
    }
    while (any) {
      any = false;
#pragma unroll
      for (int q = 0; q < kN; q++)
        if (more[q]) unary_load(un, w[q]);
#pragma unroll
      for (int q = 0; q < kN; q++) {
        more[q] = more[q] && unary_past(w[q]);
        any |= more[q];
      }
    }
#pragma unroll
    for (int q = 0; q < kN; q++)
      if (u[q]) {
        const uint32_t b = (uint32_t)(e[q] & 0xFF);  // 32 bits wide: the high part is 0
        p[q] |= b < 32 ? unary_value(w[q]) << b : 0u;
      }
  }
#pragma unroll
  for (int q = 0; q < kN; q++) {
    const uint64_t o0 = expected_offset(j[q], a.R) + (uint64_t)a.dmin + r0[q];
    const uint64_t o1 = expected_offset(j[q] + 1, a.R) + (uint64_t)a.dmin + r1[q];
    const uint32_t m = (uint32_t)(o1 - o0);
    if (m == 0) {  // only a non-member reaches an empty partition
      res[q] = o0 < a.n ? o0 : a.n - 1;
      continue;
    }
    const uint32_t s = p[q] / m;
    const uint32_t d = p[q] - s * m;
    uint32_t pos = pos_hash(fingerprint(hi[q], lo[q]), (uint64_t)(s + 1) * kPhi64, m) + d;
    if (pos >= m) pos -= m;
    const uint64_t g = o0 + pos;
    res[q] = g < a.n ? g : get_bits(a.img + a.sec_remap, (g - a.n) * a.wremap, a.wremap);
  }
}

// One lookup per thread, everything read through the caches: a launch of up to kQFew lookups has all of
// them in flight at once, so it ends after one chain of dependent reads, and neither the workgroup's copy
// to LDS nor four lookups in lockstep pay (k_query_u64, below).  A launch in a queue of them, us, before and
// now, at lambda 7, before k_query_mid (a call of the host costs 7.1 of them):
//   10^6-key table:  1000 lookups 8.5 -> 7.1, 65 536 8.5 -> 7.1, 262 144 8.9 -> 7.0, 400 000 10.6 -> 8.1
//   10^8-key table:  1000 8.7 -> 7.1, 65 536 10.0 -> 7.2, 262 144 16.4 -> 12.1, 400 000 21.2 -> 16.2, 600 000
//                    27.4 -> 22.3, 10^6 35.2 -> 32.2, 10^7 273 -> 276, 10^8 2618 -> 2896
// The line lies where the device's 2^19 threads are full: 10^6 lookups on each of two streams, which fill
// it together, take 26.9 us a batch with k_query_u64 and 28.3 with this kernel.
constexpr uint64_t kQFew = 1ull << 19;
__global__ __launch_bounds__(kQBlock) void k_query_few(QueryArgs a, const uint64_t* __restrict__ keys, uint64_t n,
                                                        uint64_t* __restrict__ out) {
  const uint64_t x = blockIdx.x * (uint64_t)kQBlock + threadIdx.x;
  if (x >= n) return;
  if (a.n == 0) {
    out[x] = 0;
    return;
  }
  uint64_t hi[1], lo[1], res[1];
  hash_key_u64(keys[x], a.seed, hi[0], lo[0]);
  query_codes<1>(a, a.table, a.img + a.sec_enc, hi, lo, res);
  out[x] = res[0];
}

// Two lookups per thread, the bucket table in LDS and the encoder words through the caches: calls that fill
// the device a few times over.  The copy to LDS is 8 KB for 512 lookups instead of 11 for 1024, so less of a
// call passes before its first image reads, and two lookups in lockstep leave room for more wavefronts.
// us, k_query_u64 / this kernel, 10^8-key table at lambda 7, Rice: 10^6 lookups 36.4 / 34.1, 3*10^6 92.1 /
// 87.9, 10^7 271.4 / 266.0, a batch of 10^6 on each of two streams 26.8 / 26.6; Compact: 21.8 / 20.9, 55.2 /
// 52.7, 161.8 / 157.2, 21.8 / 21.1; 10^7-key table at lambda 5: 24.0 / 21.2, 57.1 / 52.2, 158.8 / 154.5, 15.2 /
// 15.4.  10^8 lookups in one call take 2623 / 2665, hence the line at kQMid; as 100 calls that alternate between
// two streams, each reading new keys, 2711 / 2759, the one loss for what single calls gain.
constexpr uint64_t kQMid = 1ull << 24;
constexpr int kQMidN = 2;
__global__ __launch_bounds__(kQBlock) void k_query_mid(QueryArgs a, const uint64_t* __restrict__ keys, uint64_t n,
                                                        uint64_t* __restrict__ out) {
  __shared__ uint32_t sT[kTableIntervals + 1];
  const uint64_t x0 = blockIdx.x * (uint64_t)(kQBlock * kQMidN) + threadIdx.x;
  if (a.n == 0) {
    for (uint64_t x = x0; x < n && x < x0 + kQBlock * kQMidN; x += kQBlock) out[x] = 0;
    return;
  }
  for (uint32_t x = threadIdx.x; x <= kTableIntervals; x += kQBlock) sT[x] = (uint32_t)a.table[x];
  __syncthreads();
  if (x0 >= n) return;
  uint64_t hi[kQMidN], lo[kQMidN], res[kQMidN];
#pragma unroll
  for (int q = 0; q < kQMidN; q++) {
    const uint64_t x = x0 + q * kQBlock;
    hash_key_u64(keys[x < n ? x : x0], a.seed, hi[q], lo[q]);
  }
  query_codes<kQMidN>(a, (const uint32_t*)sT, a.img + a.sec_enc, hi, lo, res);
#pragma unroll
  for (int q = 0; q < kQMidN; q++) {
    const uint64_t x = x0 + q * kQBlock;
    if (x < n) out[x] = res[q];
  }
}

constexpr int kQN = 4;
constexpr uint32_t kQEncLds = 1024;  // encoders the LDS-staged query holds

// Thread x handles keys x, x + stride, ..., kQN of them per round.  The bucket-function table (as 32-bit
// words) and, if kEnc (B <= kQEncLds), the encoder words are read from LDS, where the workgroup copies
// them first: a wavefront's read of either touches dozens of cache lines, and the lookup is bound by
// its cache requests (10.9 KB per workgroup at B = 358, 7% off the query time at 10^8 keys).
template <bool kEnc>
__global__ __launch_bounds__(kQBlock) void k_query_u64(QueryArgs a, const uint64_t* __restrict__ keys, uint64_t n,
                                                        uint64_t* __restrict__ out) {
  if (a.n == 0) {
    for (uint64_t x = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; x < n; x += (uint64_t)gridDim.x * blockDim.x)
      out[x] = 0;
    return;
  }
  __shared__ uint32_t sT[kTableIntervals + 1];
  __shared__ uint64_t sE[kEnc ? kQEncLds : 1];
  const uint64_t* E = a.img + a.sec_enc;
  for (uint32_t x = threadIdx.x; x <= kTableIntervals; x += kQBlock) sT[x] = (uint32_t)a.table[x];
  if (kEnc)
    for (uint32_t x = threadIdx.x; x < a.B; x += kQBlock) sE[x] = E[x];
  __syncthreads();
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t x0 = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; x0 < n; x0 += stride * kQN) {
    uint64_t hi[kQN], lo[kQN], res[kQN];
#pragma unroll
    for (int q = 0; q < kQN; q++) {
      const uint64_t x = x0 + q * stride;
      hash_key_u64(keys[x < n ? x : x0], a.seed, hi[q], lo[q]);
    }
    if (kEnc)
      query_codes<kQN>(a, (const uint32_t*)sT, (const uint64_t*)sE, hi, lo, res);
    else
      query_codes<kQN>(a, (const uint32_t*)sT, E, hi, lo, res);
#pragma unroll
    for (int q = 0; q < kQN; q++) {
      const uint64_t x = x0 + q * stride;
      if (x < n) out[x] = res[q];
    }
  }
}

__global__ __launch_bounds__(kQBlock) void k_query_str(QueryArgs a, const uint8_t* __restrict__ bytes,
                                                       const uint64_t* __restrict__ offs, uint64_t n,
                                                       uint64_t* __restrict__ out) {
  for (uint64_t x = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; x < n; x += (uint64_t)gridDim.x * blockDim.x) {
    if (a.n == 0) {
      out[x] = 0;
      continue;
    }
    const uint64_t s0 = offs[x], s1 = offs[x + 1];
    uint64_t hi[1], lo[1], res[1];
    hash_key_str(bytes + s0, s1 - s0, a.seed, hi[0], lo[0]);
    query_codes<1>(a, a.table, a.img + a.sec_enc, hi, lo, res);
    out[x] = res[0];
  }
}

// Several requests in one launch: blocks [bstart[r], bstart[r+1]) serve request r.
struct QueryJob {
  QueryArgs qa;
  const uint64_t* keys;
  uint64_t* out;
  uint64_t n;
};
constexpr uint32_t kMultiItems = 4;

// Lookups first + t kQBlock + threadIdx.x (t < kMultiItems) of request jb, in lockstep (query_codes).
// The block exists for the request, so its first lookup is in range and stands in for those past the
// end.
__device__ __forceinline__ void multi_items(const QueryJob& jb, const uint32_t* T, const uint64_t* E, uint64_t first) {
  uint64_t hi[kMultiItems], lo[kMultiItems], res[kMultiItems];
#pragma unroll
  for (uint32_t t = 0; t < kMultiItems; t++) {
    const uint64_t x = first + t * kQBlock + threadIdx.x;
    hash_key_u64(jb.keys[x < jb.n ? x : first], jb.qa.seed, hi[t], lo[t]);
  }
  query_codes<(int)kMultiItems>(jb.qa, T, E, hi, lo, res);
#pragma unroll
  for (uint32_t t = 0; t < kMultiItems; t++) {
    const uint64_t x = first + t * kQBlock + threadIdx.x;
    if (x < jb.n) jb.out[x] = res[t];
  }
}

// As k_query_u64 (the bucket table and encoder words staged in LDS when B <= kQEncLds), one request
// per block.
__global__ __launch_bounds__(kQBlock) void k_query_multi(const QueryJob* __restrict__ jobs,
                                                         const uint64_t* __restrict__ bstart, uint32_t count) {
  __shared__ uint32_t sj;
  __shared__ uint32_t sT[kTableIntervals + 1];
  __shared__ uint64_t sE[kQEncLds];
  if (threadIdx.x == 0) {
    uint32_t lo = 0, hi = count;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (bstart[mid] <= blockIdx.x) lo = mid; else hi = mid;
    }
    sj = lo;
  }
  __syncthreads();
  const QueryJob& jb = jobs[sj];
  const uint64_t first = (uint64_t)(blockIdx.x - bstart[sj]) * kQBlock * kMultiItems;
  if (jb.qa.n == 0) {  // an empty MPHF: every key maps to 0
    for (uint32_t t = 0; t < kMultiItems; t++) {
      const uint64_t x = first + t * kQBlock + threadIdx.x;
      if (x < jb.n) jb.out[x] = 0;
    }
    return;
  }
  const uint64_t* E = jb.qa.img + jb.qa.sec_enc;
  for (uint32_t x = threadIdx.x; x <= kTableIntervals; x += kQBlock) sT[x] = (uint32_t)jb.qa.table[x];
  if (jb.qa.B <= kQEncLds) {
    for (uint32_t x = threadIdx.x; x < jb.qa.B; x += kQBlock) sE[x] = E[x];
    __syncthreads();
    multi_items(jb, sT, sE, first);
  } else {
    __syncthreads();
    multi_items(jb, sT, E, first);
  }
}

// ---------------------------------------------------------------------------------------------
// Allocation-free multi-request query: the job table lives in `scratch`, a fixed device array of
// this library (one per GPU, kept until the process ends), instead of a pool allocation.  Its
// layout: kNoAllocRequests jobs, then kNoAllocRequests block starts.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kNoAllocRequests = 4096;
constexpr size_t kNoAllocJobBytes = (size_t)kNoAllocRequests * sizeof(QueryJob);
constexpr size_t kNoAllocBytes = kNoAllocJobBytes + (size_t)kNoAllocRequests * sizeof(uint64_t);
static __device__ __align__(256) uint8_t scratch[kNoAllocBytes];

constexpr int kNoAllocDevices = 64;
std::mutex g_noalloc_mu;                   // guards the table below and the host staging
void* g_noalloc_dev[kNoAllocDevices] = {};  // device address of `scratch` per device
// Host staging of one call's table (pageable; a copy from it is staged before the copy call returns).
alignas(64) uint8_t g_noalloc_host[kNoAllocBytes];

uint32_t query_grid(uint64_t n, uint32_t per_thread = 1) {
  uint64_t g = (n + (uint64_t)kQBlock * per_thread - 1) / ((uint64_t)kQBlock * per_thread);
  return (uint32_t)(g < 1 ? 1 : (g > 1048576 ? 1048576 : g));
}

}  // namespace
}  // namespace phobic

using namespace phobic;

extern "C" phobic_status phobic_query_u64(const phobic_mphf* h, const uint64_t* d_keys, uint64_t n, uint64_t* d_pos,
                                          void* hip_stream) {
  if (!h) return fail(PHOBIC_E_INVALID, "null handle");
  if (n == 0) return PHOBIC_OK;
  if (!d_keys || !d_pos) return fail(PHOBIC_E_INVALID, "null key or output pointer");
  if (n <= kQFew)
    hipLaunchKernelGGL(k_query_few, dim3(query_grid(n)), dim3(kQBlock), 0, (hipStream_t)hip_stream, h->qa, d_keys, n,
                       d_pos);
  else if (n <= kQMid)
    hipLaunchKernelGGL(k_query_mid, dim3(query_grid(n, kQMidN)), dim3(kQBlock), 0, (hipStream_t)hip_stream, h->qa,
                       d_keys, n, d_pos);
  else if (h->qa.B <= kQEncLds)
    hipLaunchKernelGGL((k_query_u64<true>), dim3(query_grid(n, kQN)), dim3(kQBlock), 0, (hipStream_t)hip_stream,
                       h->qa, d_keys, n, d_pos);
  else
    hipLaunchKernelGGL((k_query_u64<false>), dim3(query_grid(n, kQN)), dim3(kQBlock), 0, (hipStream_t)hip_stream,
                       h->qa, d_keys, n, d_pos);
  PHOBIC_HIP(hipGetLastError());
  return PHOBIC_OK;
}

extern "C" phobic_status phobic_query_str(const phobic_mphf* h, const uint8_t* d_bytes, const uint64_t* d_offsets,
                                          uint64_t n, uint64_t* d_pos, void* hip_stream) {
  if (!h) return fail(PHOBIC_E_INVALID, "null handle");
  if (n == 0) return PHOBIC_OK;
  if (!d_bytes || !d_offsets || !d_pos) return fail(PHOBIC_E_INVALID, "null key or output pointer");
  hipLaunchKernelGGL(k_query_str, dim3(query_grid(n)), dim3(kQBlock), 0, (hipStream_t)hip_stream, h->qa, d_bytes,
                     d_offsets, n, d_pos);
  PHOBIC_HIP(hipGetLastError());
  return PHOBIC_OK;
}

extern "C" phobic_status phobic_query_multi_u64(const phobic_mphf* const* h_handles, const uint64_t* const* h_keys,
                                                const uint64_t* h_counts, uint64_t* const* h_outs, uint32_t count,
                                                void* hip_stream) {
  if (count == 0) return PHOBIC_OK;
  if (!h_handles || !h_keys || !h_counts || !h_outs) return fail(PHOBIC_E_INVALID, "null argument");
  std::vector<QueryJob> jobs;
  std::vector<uint64_t> bstart;
  uint64_t blocks = 0;
  for (uint32_t r = 0; r < count; r++) {
    if (!h_handles[r]) return fail(PHOBIC_E_INVALID, "null handle in request " + std::to_string(r));
    const uint64_t n = h_counts[r];
    if (n == 0) continue;
    if (!h_keys[r] || !h_outs[r]) return fail(PHOBIC_E_INVALID, "null pointer in request " + std::to_string(r));
    jobs.push_back(QueryJob{h_handles[r]->qa, h_keys[r], h_outs[r], n});
    bstart.push_back(blocks);
    blocks += (n + (uint64_t)kQBlock * kMultiItems - 1) / ((uint64_t)kQBlock * kMultiItems);
  }
  if (jobs.empty()) return PHOBIC_OK;
  if (blocks > 0x7FFFFFFFULL) return fail(PHOBIC_E_INVALID, "too many keys in one call");
  hipStream_t st = (hipStream_t)hip_stream;
  const size_t jbytes = jobs.size() * sizeof(QueryJob), bbytes = bstart.size() * sizeof(uint64_t);
  // per-thread pinned staging; the event of its last copy guards reuse
  struct Staging {
    void* p = nullptr;
    size_t cap = 0;
    hipEvent_t ev = nullptr;
  };
  thread_local Staging stg;
  if (!stg.ev) PHOBIC_HIP(hipEventCreateWithFlags(&stg.ev, hipEventDisableTiming));
  PHOBIC_HIP(hipEventSynchronize(stg.ev));
  if (stg.cap < jbytes + bbytes) {
    if (stg.p) (void)hipHostFree(stg.p);
    stg.p = nullptr;
    stg.cap = 0;
    const size_t cap = std::max<size_t>(jbytes + bbytes, 1 << 16);
    PHOBIC_HIP(hipHostMalloc(&stg.p, cap, hipHostMallocDefault));
    stg.cap = cap;
  }
  std::memcpy(stg.p, jobs.data(), jbytes);
  std::memcpy((char*)stg.p + jbytes, bstart.data(), bbytes);
  void* dbuf = nullptr;
  PHOBIC_HIP(pool_alloc(&dbuf, jbytes + bbytes, st));
  hipError_t e = hipMemcpyAsync(dbuf, stg.p, jbytes + bbytes, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipEventRecord(stg.ev, st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_query_multi, dim3((uint32_t)blocks), dim3(kQBlock), 0, st, (const QueryJob*)dbuf,
                       (const uint64_t*)((char*)dbuf + jbytes), (uint32_t)jobs.size());
    e = hipGetLastError();
  }
  (void)hipFreeAsync(dbuf, st);
  if (e != hipSuccess) return fail(PHOBIC_E_DEVICE, std::string("query_multi: ") + hipGetErrorString(e));
  return PHOBIC_OK;
}

extern "C" phobic_status phobic_query_multi_u64_noalloc(const phobic_mphf* const* h_handles,
                                                        const uint64_t* const* h_keys, const uint64_t* h_counts,
                                                        uint64_t* const* h_outs, uint32_t count, void* hip_stream) {
  if (count == 0) return PHOBIC_OK;
  if (!h_handles || !h_keys || !h_counts || !h_outs) return fail(PHOBIC_E_INVALID, "null argument");
  if (count > kNoAllocRequests)
    return fail(PHOBIC_E_INVALID, "at most " + std::to_string(kNoAllocRequests) + " requests per call");
  int dev = 0;
  PHOBIC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kNoAllocDevices) return fail(PHOBIC_E_INVALID, "device index out of range");
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (!g_noalloc_dev[dev]) {  // once per device, with that device current: the array's own address
    void* ptr = nullptr;
    PHOBIC_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(PHOBIC_E_DEVICE, "no device address for the query scratch array");
    g_noalloc_dev[dev] = ptr;
  }
  uint8_t* dscr = (uint8_t*)g_noalloc_dev[dev];
  QueryJob* jobs = (QueryJob*)g_noalloc_host;
  uint64_t* bstart = (uint64_t*)(g_noalloc_host + kNoAllocJobBytes);
  uint32_t nj = 0;
  uint64_t blocks = 0;
  for (uint32_t r = 0; r < count; r++) {
    if (!h_handles[r]) return fail(PHOBIC_E_INVALID, "null handle in request " + std::to_string(r));
    const uint64_t n = h_counts[r];
    if (n == 0) continue;
    if (!h_keys[r] || !h_outs[r]) return fail(PHOBIC_E_INVALID, "null pointer in request " + std::to_string(r));
    jobs[nj] = QueryJob{h_handles[r]->qa, h_keys[r], h_outs[r], n};
    bstart[nj] = blocks;
    nj++;
    blocks += (n + (uint64_t)kQBlock * kMultiItems - 1) / ((uint64_t)kQBlock * kMultiItems);
  }
  if (nj == 0) return PHOBIC_OK;
  if (blocks > 0x7FFFFFFFULL) return fail(PHOBIC_E_INVALID, "too many keys in one call");
  hipStream_t st = (hipStream_t)hip_stream;
  PHOBIC_HIP(hipMemcpyAsync(dscr, jobs, nj * sizeof(QueryJob), hipMemcpyHostToDevice, st));
  PHOBIC_HIP(hipMemcpyAsync(dscr + kNoAllocJobBytes, bstart, nj * sizeof(uint64_t), hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(k_query_multi, dim3((uint32_t)blocks), dim3(kQBlock), 0, st, (const QueryJob*)dscr,
                     (const uint64_t*)(dscr + kNoAllocJobBytes), nj);
  PHOBIC_HIP(hipGetLastError());
  return PHOBIC_OK;
}
