// Device code of the look-ahead fetch: workgroups beside the matching ones
// read host rows into HBM staging while Stage One runs, and the gather that
// follows takes those rows from there.
//
// Why: the host link is what bounds a step, and it used to idle from the
// step's start to the end of Stage One (14-27 us).  An index that no slot of
// its request holds when the step begins must miss (Eq. 10 needs c[o] == x),
// so its row crosses the link whatever Stage One decides.  A fetching
// workgroup needs only the request's selections and cached indices: it sets a
// bit per cached index in LDS (32 bits per slot, so about 3% of the new
// indices are taken for cached ones and left to the gather), and each
// selected index whose bit is clear claims an entry of a small table, up to a
// quota of rows.  Nothing waits for another workgroup: the launch boundary
// orders the staged rows before the gather's reads.
//
// A staged row is a copy of a host row made in this step, so using it is right
// whatever chose it; the matching workgroup may write the table back while it
// is read here, which can only change which rows are fetched.  The table is
// rewritten by every launch, and the gather looks every host entry up in it.
//
// Size: one CU reads about 2.5 GB/s from the host, so some 20-30 of them keep
// the link busy; 32 workgroups (32 / B of them share a request of a small
// batch by hash) were as good as 48 and better than 64 (three tokens, 32
// requests: 351 against 362 us).  The quota of 256 KiB + 256 KiB per token is
// what the link carries between the bitmap's end, about 4 us into the launch,
// and the end of Stage One; half of it left the link idle (batch 16: 84.6
// against 80.4 us) and twice gave nothing (80.8): the launch only got longer.
// Step before and after (us): 16 requests 89.8 -> 80.9, 64 requests with two
// tokens 524 -> 508, 4 requests with two tokens 59.6 -> 47.0, one request
// 21.4 -> 17.9 (S = 8192, K = 2048, 1152-byte rows).
#pragma once

#include "avsg_internal.h"

namespace avsg {
namespace {

// Where index x of request r is looked up among the rows fetched ahead: the
// workgroup whose share of the request it belongs to and its entry in that
// workgroup's table, from different bits of one multiplicative hash.
struct AheadSpot {
  int wg, entry;
};
__device__ __forceinline__ AheadSpot ahead_spot(const AheadView& a, int r, int32_t x) {
  const uint32_t h = static_cast<uint32_t>(x) * 0x9E3779B1u;
  const int part = static_cast<int>(((h >> 16) * static_cast<uint32_t>(a.parts)) >> 16);
  return {r * a.parts + part, static_cast<int>((h >> 8) & static_cast<uint32_t>(a.entries - 1))};
}

typedef int fetch_i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int fetch_u32x4 __attribute__((ext_vector_type(4)));

// Values of V-sized chunks [0, total) of the listed rows, chunk q0 + u * NT of
// a thread in v[u].
template <typename V, int NT, int U>
__device__ __forceinline__ void fetch_load(V (&v)[U], const int32_t* list, int total, int chunks, uint64_t src,
                                           int64_t row_bytes, int q0) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = q0 + u * NT;
    if (q < total) {
      const int i = q / chunks, ch = q - i * chunks;
      v[u] = load_global<V>(src + static_cast<uint64_t>(list[i]) * static_cast<uint64_t>(row_bytes) +
                            static_cast<uint64_t>(ch) * sizeof(V));
    }
  }
}
// Staged rows are contiguous in list order, so chunk q goes to dst + q * sizeof(V).
template <typename V, int NT, int U>
__device__ __forceinline__ void fetch_store(const V (&v)[U], int total, uint64_t dst, int q0) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = q0 + u * NT;
    if (q < total) store_global<V>(dst + static_cast<uint64_t>(q) * sizeof(V), v[u]);
  }
}
template <typename V, int NT, int U>
__device__ __forceinline__ void fetch_copy(const int32_t* list, int n, uint64_t src, uint64_t dst, int64_t row_bytes) {
  const int chunks = static_cast<int>(row_bytes / static_cast<int64_t>(sizeof(V))), total = n * chunks;
  for (int q0 = threadIdx.x; q0 < total; q0 += U * NT) {
    V v[U];
    fetch_load<V, NT, U>(v, list, total, chunks, src, row_bytes, q0);
    fetch_store<V, NT, U>(v, total, dst, q0);
  }
}

// Look-ahead fetch of workgroup w (request w / parts, its share w % parts).
template <int NT>
__device__ __forceinline__ void fetch_ahead(const MatchParams& p, const AheadParams& a, int w, unsigned char* lds) {
  constexpr int kPre = 8;   // selections of a thread requested before the table is in
  const int S = p.S, tid = threadIdx.x;
  const int r = w / a.view.parts;
  uint32_t* seen = reinterpret_cast<uint32_t*>(lds);              // [S] one bit per index mod 32 S
  int32_t* ex = reinterpret_cast<int32_t*>(seen + S);             // [entries] index of an entry, -1 = free
  int32_t* ek = ex + a.view.entries;                              // [entries] its place in the list
  int32_t* list = ek + a.view.entries;                            // [quota] indices fetched
  int32_t* count = list + a.view.quota;
  const int32_t* xg = p.topk + static_cast<size_t>(r) * p.n_q * p.K;
  const int n = p.n_q * p.K;
  const fetch_i32x4* gc = reinterpret_cast<const fetch_i32x4*>(p.table_c + static_cast<size_t>(r) * S);

  fetch_i32x4 c[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    c[k] = -1;
    if (tid + k * NT < S / 4) c[k] = gc[tid + k * NT];
  }
  int32_t x[kPre];
#pragma unroll
  for (int u = 0; u < kPre; ++u) x[u] = tid + u * NT < n ? xg[tid + u * NT] : -1;
  const int64_t rows_r = p.rows[r];
  const uint64_t src0 = a.host_ptrs[r], src1 = a.n_streams > 1 ? a.host_ptrs[p.B + r] : 0;
  for (int j = tid; j < S / 4; j += NT) reinterpret_cast<fetch_u32x4*>(seen)[j] = 0u;
  for (int j = tid; j < a.view.entries; j += NT) {
    ex[j] = -1;
    ek[j] = -1;
  }
  if (tid == 0) *count = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c[k][e] >= 0)
        atomicOr(&seen[(static_cast<uint32_t>(c[k][e]) >> 5) & static_cast<uint32_t>(S - 1)], 1u << (c[k][e] & 31));
  __syncthreads();
  auto take = [&](int32_t v) __attribute__((always_inline)) {
    if (v < 0 || static_cast<int64_t>(v) >= rows_r) return;
    if ((seen[(static_cast<uint32_t>(v) >> 5) & static_cast<uint32_t>(S - 1)] >> (v & 31)) & 1u) return;
    const AheadSpot at = ahead_spot(a.view, r, v);
    if (at.wg != w || *static_cast<volatile int32_t*>(count) >= a.view.quota) return;
    if (atomicCAS(&ex[at.entry], -1, v) != -1) return;
    const int k = atomicAdd(count, 1);
    if (k < a.view.quota) {
      list[k] = v;
      ek[at.entry] = k;
    }
  };
#pragma unroll
  for (int u = 0; u < kPre; ++u) take(x[u]);
  for (int j = tid + kPre * NT; j < n; j += NT) take(xg[j]);
  __syncthreads();
  const int m = *count < a.view.quota ? *count : a.view.quota;
  if (tid == 0 && m > 0)
    atomicAdd(p.stats + static_cast<size_t>(r) * kNumStats + kStatEarlyStaged, static_cast<unsigned long long>(m));
  const size_t first = static_cast<size_t>(w) * a.view.quota;
  const uint64_t dst0 = a.view.stage0 + first * static_cast<uint64_t>(a.row_bytes0);
  if (a.n_streams > 1) {
    const uint64_t dst1 = a.view.stage1 + first * static_cast<uint64_t>(a.row_bytes1);
    if ((a.row_bytes1 & 15) == 0) fetch_copy<fetch_u32x4, NT, 2>(list, m, src1, dst1, a.row_bytes1);
    else fetch_copy<uint32_t, NT, 4>(list, m, src1, dst1, a.row_bytes1);
  }
  if ((a.row_bytes0 & 15) == 0) fetch_copy<fetch_u32x4, NT, 2>(list, m, src0, dst0, a.row_bytes0);
  else fetch_copy<uint32_t, NT, 4>(list, m, src0, dst0, a.row_bytes0);
  for (int j = tid; j < a.view.entries; j += NT)
    a.view.table[static_cast<size_t>(w) * a.view.entries + j] = ek[j] >= 0 ? make_int2(ex[j], ek[j]) : make_int2(-1, 0);
}

}  // namespace
}  // namespace avsg
