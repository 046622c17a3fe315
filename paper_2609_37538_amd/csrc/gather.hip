// Stage Two of AVSG on gfx950: miss-only copy of host rows into reserved slots.
//
// The miss list is ordered by (request, token, miss rank) (Section 3.4).  The
// balanced kernel (S3, Eq. 6) runs C workers; worker w takes the consecutive
// misses [floor(w N / C), floor((w+1) N / C)) of the batch-wide list of N
// misses, so any two workers differ by at most one row, and consecutive
// workers run on one XCD (xcd_worker).  The request
// kernel (S1, Eq. 13) runs one workgroup per request.  Inside a workgroup a
// tile of misses is staged in LDS as (source, destination) address pairs, and
// the lanes copy the rows with 16-byte loads from pinned, device-mapped host
// memory (row16, at 4-byte boundaries for rows such as the 132-byte indexer-key
// ones).  The
// position kernel (S2, Eq. 14) splits the flattened N_g*K selected positions
// into C near-equal contiguous ranges; hit positions issue no copy but still
// occupy their worker's share.  With the resident-reuse plan of the matching
// kernel, the resident kernel copies the host list (each row also to its two
// fan slots) and the rows already in the device buffer; with more than four
// tokens per step the device-copy kernel then fills the repeats left over.
#include "gather_body.h"

namespace avsg {
namespace {

// Worker index of workgroup b among C workers.  The dispatcher deals
// workgroups to the eight XCDs of the chip round-robin (workgroup b to XCD
// b mod 8), and each XCD has its own L2; consecutive workers get consecutive
// stretches of the miss list, which hold the same request's tokens, so they
// go to one XCD: a row that several tokens of a step miss (a lost install) is
// then read over the host link once and served from that XCD's L2 after.
// A bijection of [0, C) for any C; the split of Eq. 6 and Eq. 14 is unchanged.
__device__ __forceinline__ long long xcd_worker(long long b, long long C) {
  constexpr long long X = kXcds;
  const long long x = b % X, q = C / X, rem = C % X;
  return x * q + (x < rem ? x : rem) + b / X;
}

__global__ __launch_bounds__(GT) void gather_balanced_kernel(GatherParams p) {
  __shared__ int pre[kMaxBatch + 1], wtot[GT / 64];
  __shared__ uint64_t src0[TILE], dst0[TILE], src1[TILE], dst1[TILE];
  request_prefix(p, pre, wtot);
  const long long N = pre[p.B];
  const long long C = gridDim.x, w = xcd_worker(blockIdx.x, C);
  const int a = static_cast<int>((w * N) / C);          // Eq. 6: consecutive, floor/ceil(N/C) each
  const int b = static_cast<int>(((w + 1) * N) / C);
  copy_range<false>(p, pre, a, b, src0, dst0, src1, dst1);
}

// Resident-reuse Stage Two over two lists: host rows (each also written to
// its fan slots, the two largest repeats of its index in the step), and rows
// already in a slot of the same request (not written this step).  Part of the
// workgroups starts with the resident list and the others with the host list,
// so the HBM copies run while the host link is busy (the link saturates with
// far fewer workgroups); each group then moves to the other list.  From 16
// requests on half of them start with the resident list, below a quarter: few
// rows need the many workgroups (11 requests, three tokens: 41.7 against 43.7
// us with half; one request, four tokens: 37.8 against 39.2), while with many
// rows fewer host readers leave the other accesses shorter queues (192
// requests with high reuse 66.3 against 68.7 us, 16 requests 77.3 against
// 77.7, 32 requests 347.1 against 348.2; 5/8 is no better than half).
// A host-first workgroup's first tile is a stretch of one request's own host
// list (first_tiles; none when a request would get more than eight of them),
// which needs no batch-wide prefix, so host reads start one list read after
// the launch; without first tiles, tile w of the batch-wide list goes to
// workgroup w.  Tile i of the resident list first goes to the i-th
// resident-first workgroup.  Later tiles are claimed (an atomic counter), so
// the workgroups that finish first take more (a CU's host-read rate varies up
// to 2x across the chip; they end the kernel more evenly than a static Eq. 6
// split); a list that the first tiles cover is not claimed from at all (two
// claims, about 1 us each, at the end of a step with few rows).  A list
// shorter than one full tile per workgroup of its group is cut into tiles of
// ceil(n / group) rows.  claim[0] and claim[1] count the claimed resident and
// host rows; the matching kernel resets both.
//
// What bounds it: the host link, which it keeps busy from its first read to
// its end (16 requests: 61 us for 3.4 MB).  What it can shorten is the chain
// before that read: launch, counts, list entry with the request's addresses,
// look-up among the staged rows.  Step before and after batching those reads,
// 32-bit prefixes by DPP, the unclaimed first tiles and a single row read in
// flight per thread (see kHostUnroll), us: 16 requests 80.7 -> 77.3; 4
// requests, two tokens 47.5 -> 45.0; 11 requests, three tokens 45.6 -> 41.7;
// one request, four tokens 42.8 -> 37.8; 192 requests with high reuse 70.1 ->
// 66.3; 64 requests, two tokens 509.1 -> 507.4.
constexpr int kHostTile = 6;

// Rows per tile of a list of n entries shared by `group` workgroups.
__device__ __forceinline__ int tile_rows(int n, int group, int max_rows) {
  const int t = (n + group - 1) / group;
  return t < 1 ? 1 : (t > max_rows ? max_rows : t);
}

// Copy tiles of T entries of a list of n entries: `first` (or none, -1) then
// claimed tiles, which start at row `base` (none are left to claim, and no
// claim is made, when that is the list's end).
template <bool kDevice, bool kRow16>
__device__ void copy_tiles(const GatherParams& p, const int* pre, int n, int T, int first, int base, int* counter,
                           int* next, uint64_t* src0, uint64_t* dst0, uint64_t* src1, uint64_t* dst1,
                           uint64_t* dstx0 = nullptr, uint64_t* dstx1 = nullptr, uint64_t* dsty0 = nullptr,
                           uint64_t* dsty1 = nullptr, const int* cov = nullptr, uint64_t* dstz0 = nullptr,
                           uint64_t* dstz1 = nullptr) {
  int t0 = first;
  for (;;) {
    if (t0 < 0) {
      if (base >= n) break;
      if (threadIdx.x == 0) *next = base + atomicAdd(counter, T);
      __syncthreads();
      t0 = *next;
      __syncthreads();
    }
    if (t0 >= n) break;
    copy_range<kDevice, kDevice ? kUnroll : kHostUnroll, kRow16>(p, pre, t0, t0 + T < n ? t0 + T : n, src0, dst0, src1, dst1, dstx0, dstx1, dsty0,
                        dsty1, cov, -1, dstz0, dstz1);
    t0 = -1;
  }
}

// THIRD: host entries have a third further slot (four tokens per step).
template <bool THIRD>
__global__ __launch_bounds__(GT) void gather_resident_kernel(GatherParams hp, GatherParams rp,
                                                              int* claim) {
  __shared__ int pre_h[kMaxBatch + 1], pre_r[kMaxBatch + 1], cov[kMaxBatch];
  __shared__ int wtot[2 * (GT / 64)];
  __shared__ uint64_t src0[TILE], dst0[TILE], src1[TILE], dst1[TILE], dstx0[TILE], dstx1[TILE], dsty0[TILE],
      dsty1[TILE];
  __shared__ uint64_t dstz[THIRD ? 2 * TILE : 1];
  uint64_t* const dstz0 = THIRD ? dstz : nullptr;
  uint64_t* const dstz1 = THIRD ? dstz + TILE : nullptr;
  __shared__ int next;
  const int C = static_cast<int>(gridDim.x), w = static_cast<int>(blockIdx.x);
  const int B = hp.B;
  const int cr = B >= 16 ? C / 2 : C / 4;   // workgroups that start with the resident list (may be 0)
  const int ch = C - cr;                 // >= 1
  // the counts of the prefixes below are requested before the first tile, so
  // their latency overlaps it
  const size_t rq = static_cast<int>(threadIdx.x) < B ? threadIdx.x : 0;
  const int32_t ha = hp.miss_counts[rq * hp.count_stride], hb = rp.miss_counts[rq * rp.count_stride];
  const bool first_on = first_tiles_on(B, ch);
  if (w < ch && first_on) {
    // first tile, before any prefix: entries [k T, (k+1) T) of request
    // w mod B's host list, k = w div B (the host link starts one list read
    // after the launch)
    const int r = w % B, k = w / B;
    const int cnt = hp.miss_counts[static_cast<size_t>(r) * hp.count_stride];
    const int T = first_tile_rows(cnt, first_tiles(r, B, ch), kHostTile);
    const int lo = k * T;
    const int hi = lo + T < cnt ? lo + T : cnt;
    if (lo < hi)
      copy_range<false, kHostUnroll, !THIRD>(hp, nullptr, lo, hi, src0, dst0, src1, dst1, dstx0, dstx1, dsty0, dsty1, nullptr, r,
                        dstz0, dstz1);
  }
  // the rest of the host list, batch-wide (every group; without first tiles
  // tile w goes first to host-first workgroup w), then claimed tiles, and the
  // resident list (tile i of it first to the i-th resident-first workgroup,
  // the rest claimed)
  request_prefix_resid(hp, pre_h, cov, rp, pre_r, wtot, ch, kHostTile, ha, hb);
  const int N = pre_h[B], R = pre_r[rp.B];
  const int tr = tile_rows(R, cr > 0 ? cr : ch, TILE);
  const int res_base = cr * tr;
  const int th = first_on ? kHostTile : tile_rows(N, ch, kHostTile);
  const int host_base = first_on ? 0 : ch * th;
  if (w >= ch) {
    const int i = C - 1 - w;       // 0 .. cr-1
    copy_tiles<true, !THIRD>(rp, pre_r, R, tr, i * tr, res_base, claim, &next, src0, dst0, src1, dst1);
    copy_tiles<false, !THIRD>(hp, pre_h, N, kHostTile, -1, host_base, claim + 1, &next, src0, dst0, src1, dst1,
                      dstx0, dstx1, dsty0, dsty1, cov, dstz0, dstz1);
  } else {
    copy_tiles<false, !THIRD>(hp, pre_h, N, th, first_on ? -1 : w * th, host_base, claim + 1, &next, src0, dst0, src1, dst1,
                      dstx0, dstx1, dsty0, dsty1, cov, dstz0, dstz1);
    copy_tiles<true, !THIRD>(rp, pre_r, R, tr, -1, res_base, claim, &next, src0, dst0, src1, dst1);
  }
}

// Device-to-device row copies (source slot -> slot) over the same balanced
// split; runs after the host copies of the step, so every source holds its row.
__global__ __launch_bounds__(GT) void copy_device_kernel(GatherParams p) {
  __shared__ int pre[kMaxBatch + 1], wtot[GT / 64];
  __shared__ uint64_t src0[TILE], dst0[TILE], src1[TILE], dst1[TILE];
  request_prefix(p, pre, wtot);
  const long long N = pre[p.B];
  const long long C = gridDim.x, w = blockIdx.x;
  const int a = static_cast<int>((w * N) / C);
  const int b = static_cast<int>(((w + 1) * N) / C);
  copy_range<true>(p, pre, a, b, src0, dst0, src1, dst1);
}

static_assert(TILE <= 64, "the first wave stages a tile");
__global__ __launch_bounds__(GT) void gather_position_kernel(GatherParams p) {
  __shared__ int live;
  __shared__ uint64_t src0[TILE], dst0[TILE], src1[TILE], dst1[TILE];
  const long long per_req = static_cast<long long>(p.n_q) * p.K;
  const long long P = per_req * p.B;
  const long long C = gridDim.x, w = xcd_worker(blockIdx.x, C);
  const long long a = (w * P) / C;          // Eq. 14: near-equal ranges of positions
  const long long b = ((w + 1) * P) / C;
  for (long long t0 = a; t0 < b; t0 += TILE) {
    const int tn = static_cast<int>((b - t0) < TILE ? (b - t0) : TILE);
    for (int i = threadIdx.x; i < tn; i += GT) {
      const long long pos = t0 + i;
      const int r = static_cast<int>(pos / per_req);
      const int32_t x = p.topk[pos];
      const int32_t o = p.slots[pos];
      const bool miss = p.hit_mask[pos] == 0;
      const bool ok = miss && x >= 0 && static_cast<int64_t>(x) < p.rows[r] && o >= 0 && o < p.S;
      const int alive = __popcll(__ballot(ok));   // a tile is staged by one wave
      if (i == 0) live = alive;
      src0[i] = ok ? p.host_ptrs[r] + static_cast<uint64_t>(x) * p.row_bytes0 : 0;
      dst0[i] = p.buf_ptrs[r] + static_cast<uint64_t>(o) * p.row_bytes0;
      if (p.n_streams > 1) {
        src1[i] = ok ? p.host_ptrs[p.B + r] + static_cast<uint64_t>(x) * p.row_bytes1 : 0;
        dst1[i] = p.buf_ptrs[p.B + r] + static_cast<uint64_t>(o) * p.row_bytes1;
      }
    }
    __syncthreads();
    copy_tile_rows(p, tn, src0, dst0, src1, dst1, C <= kDeepWorkgroups || live * 4 <= tn);
  }
}

template <int U>
__global__ __launch_bounds__(GT) void gather_request_kernel(GatherParams p) {
  __shared__ int pre[kMaxBatch + 1], wtot[GT / 64];
  __shared__ uint64_t src0[TILE], dst0[TILE], src1[TILE], dst1[TILE];
  request_prefix(p, pre, wtot);
  const int r = blockIdx.x;                 // Eq. 13: one worker per request
  copy_range<false, U>(p, pre, pre[r], pre[r + 1], src0, dst0, src1, dst1);
}

}  // namespace

hipError_t launch_gather_balanced(const GatherParams& p, int workers, hipStream_t s) {
  if (p.B > kMaxBatch || workers < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gather_balanced_kernel, dim3(workers), dim3(GT), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_copy_device(const GatherParams& p, int workers, hipStream_t s) {
  if (workers < 1 || p.B > kMaxBatch) return hipErrorInvalidValue;
  hipLaunchKernelGGL(copy_device_kernel, dim3(workers), dim3(GT), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_gather_resident(const GatherParams& host, const GatherParams& dev, int* claim,
                                  int workers, hipStream_t s) {
  if (workers < 1 || host.B > kMaxBatch || !claim || !host.fan) return hipErrorInvalidValue;
  if (host.third)
    hipLaunchKernelGGL(gather_resident_kernel<true>, dim3(workers), dim3(GT), 0, s, host, dev, claim);
  else
    hipLaunchKernelGGL(gather_resident_kernel<false>, dim3(workers), dim3(GT), 0, s, host, dev, claim);
  return hipGetLastError();
}

hipError_t launch_gather_position(const GatherParams& p, int workers, hipStream_t s) {
  if (workers < 1 || !p.hit_mask || !p.topk || !p.slots) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gather_position_kernel, dim3(workers), dim3(GT), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_gather_request(const GatherParams& p, hipStream_t s) {
  if (p.B > kMaxBatch) return hipErrorInvalidValue;
  if (p.B <= kDeepWorkgroups)
    hipLaunchKernelGGL(gather_request_kernel<kUnroll>, dim3(p.B), dim3(GT), 0, s, p);
  else
    hipLaunchKernelGGL(gather_request_kernel<kHostUnroll>, dim3(p.B), dim3(GT), 0, s, p);
  return hipGetLastError();
}

}  // namespace avsg
