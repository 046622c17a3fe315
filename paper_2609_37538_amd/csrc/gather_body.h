// Device code of Stage Two shared by the gather kernels and the pipelined
// step kernel (see gather.hip for the work assignments).
#pragma once

#include "avsg_internal.h"
#include "fetch_body.h"

namespace avsg {
namespace {


constexpr int GT = kGatherThreads;
constexpr int TILE = kGatherTile;
constexpr int kMaxBatch = 1024;
constexpr int kUnroll = 4;
// Loads a thread keeps in flight for 16-byte chunks of host rows in the balanced
// and resident gathers (device copies and 4-byte chunks: kUnroll).  The link is
// full with 0.5 MB in flight, and 256 workgroups have 1 MB with one load per
// thread; what is beyond that queues before every other access of the kernel
// (claims, list entries, slot copies): four per thread cost 16 requests 79.7
// against 77.8 us and 192 requests with high reuse 70.9 against 69.0.  With few
// workers one load is no loss against four through flat accesses, which wait
// for one another (16 requests, 4, 16 and 64 workers: 270, 89.8 and 65.6 us
// per step against 290, 89.0 and 70.8).
constexpr int kHostUnroll = 1;
// The request and position gathers keep kUnroll in flight with at most this many
// workgroups, and the position gather also where at most a quarter of a tile
// misses (the lanes of a hit read nothing).  All misses, us per step with four
// loads per thread and with one: request gather, 16 requests 182 / 233, 64
// requests 679 / 707, 128 requests 1347 / 1347, 200 requests 2167 / 2092, 400
// requests 2188 / 2098 (24 to 40 requests are 1-4% slower with four, and 7-9%
// faster where a tenth misses); position gather, 16 workers 481 / 647, 128
// workers 366 / 384, 256 workers with one request 71.0 / 61.2, with 48 requests
// 540 / 514; a tenth of misses, 256 workers with 16 requests 26.3 / 27.9.
constexpr int kDeepWorkgroups = 128;

__device__ __forceinline__ int lane_index() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Miss totals fit an int: at most 1024 requests of 16384 reservations.

// Exclusive prefix of the per-request miss totals into pre[0..B] (pre[B] = N).
__device__ inline void request_prefix(const GatherParams& p, int* pre, int* wtot) {
  const int tid = threadIdx.x, lane = lane_index(), wave = tid >> 6;
  const int per = (p.B + GT - 1) / GT;
  const int r0 = tid * per;
  int local = 0;
  for (int k = 0; k < per; ++k) {
    const int r = r0 + k;
    if (r < p.B) {
      // four counts at a time, their loads in flight together
      const int32_t* c = p.miss_counts + static_cast<size_t>(r) * p.count_stride;
      int t = 0;
      for (int g = 0; g < p.counts_per_req; g += 4) {
        int32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = c[g + u < p.counts_per_req ? g + u : g];
#pragma unroll
        for (int u = 0; u < 4; ++u) t += g + u < p.counts_per_req ? v[u] : 0;
      }
      pre[r + 1] = t;
      local += t;
    }
  }
  const int incl = wave_inclusive_scan(local);
  if (lane == 63) wtot[wave] = incl;
  __syncthreads();
  int base = incl - local;
  for (int w = 0; w < wave; ++w) base += wtot[w];
  for (int k = 0; k < per; ++k) {
    const int r = r0 + k;
    if (r < p.B) {
      base += pre[r + 1];
      pre[r + 1] = base;
    }
  }
  if (tid == 0) pre[0] = 0;
  __syncthreads();
}

// First tiles of the resident-reuse gather: workgroup w < ch copies tile
// w div B of request w mod B's host list before any prefix is known.  Request
// r has nfirst(r) such workgroups; its n host entries go to them in tiles of
// ceil(n / nfirst) rows, at least one and at most T0, so few entries still
// spread over many CUs (one workgroup reads ~2.5 GB/s from the host).  No
// request gets first tiles when one would get more than eight (ch > 8 B): on 256
// CUs that is below 16 requests, 192 of whose workgroups start with host rows
// (128 from 16 on, eight each).  Step with them and without, us, one token, two
// tokens: 12 requests 33.4 / 32.8, 88.9 / 89.7; 14 requests 36.5 / 36.2, 101.5 /
// 103.0; 16 requests 39.2 / 40.0, 114.1 / 115.1; 24 requests 52.3 / 53.1, 164.3 /
// 165.8; 48 requests 91.4 / 92.7, 316.6 / 318.4.
__device__ __forceinline__ bool first_tiles_on(int B, int ch) { return ch <= 8 * B; }
__device__ __forceinline__ int first_tiles(int r, int B, int ch) {
  return first_tiles_on(B, ch) && r < ch ? (ch - 1 - r) / B + 1 : 0;
}
__device__ __forceinline__ int first_tile_rows(int n, int nfirst, int T0) {
  const int t = nfirst > 0 ? (n + nfirst - 1) / nfirst : 1;
  return t < 1 ? 1 : (t > T0 ? T0 : t);
}

// Prefixes for the resident-reuse gather: of the host entries that remain
// after each request's first tiles (pre_a; cov[r] = the entries of request r
// the first tiles copy) and of the resident entries (pre_b), B + 1 entries
// each.  With at most GT requests thread r's two counts are ha and hb, which
// the caller requested before its first tile so the loads overlap it.
// wtot: 2 * GT / 64 entries.
__device__ inline void request_prefix_resid(const GatherParams& pa, int* pre_a, int* cov, const GatherParams& pb,
                                            int* pre_b, int* wtot, int ch, int T0, int32_t ha, int32_t hb) {
  const int tid = threadIdx.x, lane = lane_index(), wave = tid >> 6;
  constexpr int NW = GT / 64;
  const int per = (pa.B + GT - 1) / GT;
  const int r0 = tid * per;
  int la = 0, lb = 0;
  for (int k = 0; k < per; ++k) {
    const int r = r0 + k;
    if (r < pa.B) {
      int ta = per == 1 ? ha : pa.miss_counts[static_cast<size_t>(r) * pa.count_stride];
      const int tb = per == 1 ? hb : pb.miss_counts[static_cast<size_t>(r) * pb.count_stride];
      const int nfirst = first_tiles(r, pa.B, ch);
      const int span = nfirst * first_tile_rows(ta, nfirst, T0);
      const int c = ta < span ? ta : span;
      cov[r] = c;
      ta -= c;
      pre_a[r + 1] = ta;
      pre_b[r + 1] = tb;
      la += ta;
      lb += tb;
    }
  }
  const int ia = wave_inclusive_scan(la), ib = wave_inclusive_scan(lb);
  if (lane == 63) {
    wtot[wave] = ia;
    wtot[NW + wave] = ib;
  }
  __syncthreads();
  int ba = ia - la, bb = ib - lb;
  for (int w = 0; w < wave; ++w) {
    ba += wtot[w];
    bb += wtot[NW + w];
  }
  for (int k = 0; k < per; ++k) {
    const int r = r0 + k;
    if (r < pa.B) {
      ba += pre_a[r + 1];
      bb += pre_b[r + 1];
      pre_a[r + 1] = ba;
      pre_b[r + 1] = bb;
    }
  }
  if (tid == 0) {
    pre_a[0] = 0;
    pre_b[0] = 0;
  }
  __syncthreads();
}

template <typename T>
__device__ __forceinline__ int find_request(const T* pre, int B, T j) {
  int lo = 0, hi = B;  // pre[lo] <= j < pre[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= j) lo = mid;
    else hi = mid;
  }
  return lo;
}

// A 16-byte vector as a clang vector type: arrays of it stay in registers
// (HIP's uint4 is a union-based struct that is kept in scratch memory here).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Rows i < tn: copy chunks * sizeof(V) bytes from src[i] to dst[i] (src[i] == 0
// skips the row), and also to dstx[i], dsty[i] and dstz[i] where those are
// given and nonzero, with NT threads each keeping U loads in flight.  kOffGrid:
// the chunks are row16 and a row's last one is at offset `last`, which may lie
// before its place.
template <typename V, int U = kUnroll, int NT = GT, bool kOffGrid = false>
__device__ __forceinline__ void copy_rows(const uint64_t* src, const uint64_t* dst, int tn,
                                          int chunks, const uint64_t* dstx = nullptr,
                                          const uint64_t* dsty = nullptr, const uint64_t* dstz = nullptr,
                                          uint64_t last = 0u) {
  const int total = tn * chunks;
  for (int q0 = threadIdx.x; q0 < total; q0 += NT * U) {
    V v[U];
    uint64_t sa[U], da[U], xa[U], ya[U], za[U];
    // addresses first, then every load, then the stores: nothing stands
    // between the loads, so a thread's U loads are in flight together
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u * NT;
      const int i = q < total ? q / chunks : 0;
      uint64_t off = static_cast<uint64_t>(static_cast<uint32_t>(q - i * chunks)) * sizeof(V);
      if (kOffGrid) off = off < last ? off : last;
      const uint64_t s = src[i];
      const bool live = (q < total) & (s != 0);
      sa[u] = live ? s + off : 0;
      da[u] = dst[i] + off;
      xa[u] = dstx && dstx[i] ? dstx[i] + off : 0;
      ya[u] = dsty && dsty[i] ? dsty[i] + off : 0;
      za[u] = dstz && dstz[i] ? dstz[i] + off : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (sa[u]) v[u] = load_chunk<V, kOffGrid>(sa[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (sa[u]) {
        store_chunk<V, kOffGrid>(da[u], v[u]);
        if (xa[u]) store_chunk<V, kOffGrid>(xa[u], v[u]);
        if (ya[u]) store_chunk<V, kOffGrid>(ya[u], v[u]);
        if (za[u]) store_chunk<V, kOffGrid>(za[u], v[u]);
      }
  }
}

// The same for rows of row_bytes bytes: aligned 16-byte chunks where
// the rows are whole ones, row16 for other rows of at least 16 bytes (as 4-byte
// chunks, 300-byte rows of 40 requests took 29.0 us per step against 28.1 and
// 580-byte rows of 11 requests 41.7 against 41.0), 4-byte ones below.  U chunks in
// flight per thread.  kRow16 = false leaves the row16 path out: beside the third
// further slot of four tokens it costs whole rows more (one request 34.9
// against 34.6 us) than it gives the others.
template <int U, bool kRow16 = true>
__device__ __forceinline__ void copy_rows_of(int64_t row_bytes, const uint64_t* src, const uint64_t* dst, int tn,
                                             const uint64_t* dstx = nullptr, const uint64_t* dsty = nullptr,
                                             const uint64_t* dstz = nullptr) {
  if ((row_bytes & 15) == 0)
    copy_rows<u32x4, U>(src, dst, tn, static_cast<int>(row_bytes / 16), dstx, dsty, dstz);
  else if (kRow16 && row_bytes >= 16)
    copy_rows<u32x4, U, GT, true>(src, dst, tn, static_cast<int>((row_bytes + 15) / 16), dstx, dsty, dstz,
                        static_cast<uint64_t>(row_bytes - 16));
  else
    copy_rows<uint32_t, kUnroll>(src, dst, tn, static_cast<int>(row_bytes / 4), dstx, dsty, dstz);
}

// Rows of a staged tile; deep: kUnroll reads in flight per thread.
__device__ inline void copy_tile_rows(const GatherParams& p, int tn, uint64_t* src0, uint64_t* dst0,
                               uint64_t* src1, uint64_t* dst1, bool deep) {
  auto stream = [&](int64_t row_bytes, const uint64_t* src, const uint64_t* dst) {
    if (deep) copy_rows_of<kUnroll>(row_bytes, src, dst, tn);
    else copy_rows_of<kHostUnroll>(row_bytes, src, dst, tn);
  };
  stream(p.row_bytes0, src0, dst0);
  if (p.n_streams > 1) stream(p.row_bytes1, src1, dst1);
  __syncthreads();
}

// Copy entries [a, b) of the batch-wide list.  kDevice: an entry is (source
// slot, slot) of the request's own buffers; otherwise (host row, slot), and
// with p.fan and staging for it (dstx0/1, dsty0/1), the row also goes to the
// entry's fan slots, and with p.third (dstz0/1) to a third one.  Entry j of the batch-wide list is entry cov[r] + j -
// pre[r] of request r's list (cov: rows of each request left out of the
// batch-wide list, or none); with fixed_r >= 0, [a, b) are entries of request
// fixed_r's own list and pre is not read.
template <bool kDevice, int U = kDevice ? kUnroll : kHostUnroll, bool kRow16 = true>
__device__ __forceinline__ void copy_range(const GatherParams& p, const int* pre, int a, int b,
                           uint64_t* src0, uint64_t* dst0, uint64_t* src1, uint64_t* dst1,
                           uint64_t* dstx0 = nullptr, uint64_t* dstx1 = nullptr,
                           uint64_t* dsty0 = nullptr, uint64_t* dsty1 = nullptr,
                           const int* cov = nullptr, int fixed_r = -1, uint64_t* dstz0 = nullptr,
                           uint64_t* dstz1 = nullptr) {
  const size_t per_req = static_cast<size_t>(p.n_q) * p.K;
  for (int t0 = a; t0 < b; t0 += TILE) {
    const int tn = (b - t0) < TILE ? (b - t0) : TILE;
    for (int i = threadIdx.x; i < tn; i += GT) {
      const int j = t0 + i;
      const int r = fixed_r >= 0 ? fixed_r : find_request(pre, p.B, j);
      const int k = fixed_r >= 0 ? j : (cov ? cov[r] : 0) + j - pre[r];   // entry of request r
      const size_t at = static_cast<size_t>(r) * per_req + static_cast<size_t>(k);
      // the entry and everything that depends on the request alone are
      // requested together (a condition between them would put one memory
      // latency behind the other); then comes the look-up among the rows
      // fetched ahead, which needs the entry's index
      const int2 e = p.miss_list[at];
      int2 fan = make_int2(-1, -1);
      if (dstx0) fan = p.fan[at];
      int third = -1;
      if (dstz0) third = p.third[at];
      const bool two = p.n_streams > 1;
      const int64_t rows_r = p.rows[r];
      const uint64_t buf0 = p.buf_ptrs[r], buf1 = two ? p.buf_ptrs[p.B + r] : 0;
      uint64_t from0 = buf0, from1 = buf1;
      if (!kDevice) {
        from0 = p.host_ptrs[r];
        from1 = two ? p.host_ptrs[p.B + r] : 0;
      }
      const bool ok = (e.x >= 0) & (e.y >= 0) & (e.y < p.S) &
                      (kDevice ? e.x < p.S : static_cast<int64_t>(e.x) < rows_r);
      uint64_t row = static_cast<uint64_t>(e.x);
      if (!kDevice && r < p.ahead.served) {
        const AheadSpot spot = ahead_spot(p.ahead, r, e.x);
        const int64_t f = load_global<int64_t>(reinterpret_cast<uint64_t>(
            p.ahead.table + static_cast<size_t>(spot.wg) * p.ahead.entries + spot.entry));
        const bool staged = static_cast<int32_t>(f) == e.x;   // the row is in HBM already
        from0 = staged ? p.ahead.stage0 : from0;
        from1 = staged ? p.ahead.stage1 : from1;
        row = staged ? static_cast<uint64_t>(spot.wg) * p.ahead.quota + static_cast<uint64_t>(f >> 32) : row;
      }
      src0[i] = ok ? from0 + row * p.row_bytes0 : 0;
      dst0[i] = buf0 + static_cast<uint64_t>(e.y) * p.row_bytes0;
      if (fan.x >= p.S) fan.x = -1;
      if (fan.y >= p.S) fan.y = -1;
      if (third >= p.S) third = -1;
      if (dstx0) {
        dstx0[i] = fan.x >= 0 ? buf0 + static_cast<uint64_t>(fan.x) * p.row_bytes0 : 0;
        dsty0[i] = fan.y >= 0 ? buf0 + static_cast<uint64_t>(fan.y) * p.row_bytes0 : 0;
      }
      if (dstz0) dstz0[i] = third >= 0 ? buf0 + static_cast<uint64_t>(third) * p.row_bytes0 : 0;
      if (two) {
        src1[i] = ok ? from1 + row * p.row_bytes1 : 0;
        dst1[i] = buf1 + static_cast<uint64_t>(e.y) * p.row_bytes1;
        if (dstx1) {
          dstx1[i] = fan.x >= 0 ? buf1 + static_cast<uint64_t>(fan.x) * p.row_bytes1 : 0;
          dsty1[i] = fan.y >= 0 ? buf1 + static_cast<uint64_t>(fan.y) * p.row_bytes1 : 0;
        }
        if (dstz1) dstz1[i] = third >= 0 ? buf1 + static_cast<uint64_t>(third) * p.row_bytes1 : 0;
      }
    }
    __syncthreads();
    copy_rows_of<U, kRow16>(p.row_bytes0, src0, dst0, tn, dstx0, dsty0, dstz0);
    if (p.n_streams > 1) copy_rows_of<U, kRow16>(p.row_bytes1, src1, dst1, tn, dstx1, dsty1, dstz1);
    __syncthreads();
  }
}

}  // namespace
}  // namespace avsg
