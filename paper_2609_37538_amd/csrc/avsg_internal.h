// Internal declarations shared by the translation units of libavsg (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace avsg {

// Threads of one matching workgroup (one request per workgroup).
constexpr int kMatchThreads = 1024;
// Threads of one gather workgroup.
constexpr int kGatherThreads = 256;
// Misses staged per gather tile.
constexpr int kGatherTile = 64;
// XCDs of an MI355X (gfx950): 8 accelerator dies of 32 CUs, each with its own L2.
constexpr int kXcds = 8;

// Sixteen bytes of a row at any 4-byte boundary (global memory takes a 16-byte
// access of a lane there): a row of at least 16 bytes is ceil(bytes / 16) of
// them, the last one over the row's last 16 bytes, so rows off the 16-byte grid
// need no 4-byte accesses (132-byte rows 9 in place of 33, 580-byte rows 37 in
// place of 145).
// (The attribute belongs to the type's name and is lost in a template argument,
// so functions name the type themselves.)
typedef unsigned int chunk16 __attribute__((ext_vector_type(4)));
typedef unsigned int row16 __attribute__((ext_vector_type(4), aligned(4)));

// Loads and stores at a device-visible address held as a number, as global
// memory accesses: through a plain pointer they become flat ones, which also
// count as LDS accesses, so that a wave waits for its row loads in flight
// before each LDS read that follows them.
template <typename V>
__device__ __forceinline__ V load_global(uint64_t a) {
  return *reinterpret_cast<const __attribute__((address_space(1))) V*>(a);
}
template <typename V>
__device__ __forceinline__ void store_global(uint64_t a, V v) {
  *reinterpret_cast<__attribute__((address_space(1))) V*>(a) = v;
}
__device__ __forceinline__ chunk16 load_row16(uint64_t a) {
  return *reinterpret_cast<const __attribute__((address_space(1))) row16*>(a);
}
__device__ __forceinline__ void store_row16(uint64_t a, chunk16 v) {
  *reinterpret_cast<__attribute__((address_space(1))) row16*>(a) = v;
}
// A chunk V of a row; kOffGrid: row16.
template <typename V, bool kOffGrid>
__device__ __forceinline__ V load_chunk(uint64_t a) {
  if constexpr (kOffGrid) return load_row16(a);
  else return load_global<V>(a);
}
template <typename V, bool kOffGrid>
__device__ __forceinline__ void store_chunk(uint64_t a, V v) {
  if constexpr (kOffGrid) store_row16(a, v);
  else store_global<V>(a, v);
}

// Inclusive prefix sum over the 64 lanes of a wave, register to register
// with DPP: shifts by 1, 2, 4 and 8 lanes inside each 16-lane row (a lane
// whose source lies outside its row adds 0), then the last lane of row 0 is
// broadcast into row 1 and of row 2 into row 3, and the last lane of row 1
// (by then the total of rows 0-1) into rows 2 and 3.  Every lane of the wave
// must be active.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
  return v;
}


// Per-request device counters (uint64 each, cumulative).
enum StatIndex : int {
  kStatHits = 0,
  kStatMisses,
  kStatLostExhausted,
  kStatLostCollision,
  kStatAllocDecays,
  kStatRevivals,
  kStatInvalidations,
  kStatBadIndices,
  kStatMaxStepDecays,
  kStatResident,
  kStatDuplicate,
  kStatEarly,          // rows fetched before Stage One (early-fetch transfer)
  kStatEarlyStaged,    // rows parked in HBM staging until their slots were known (early-fetch transfer: of
                       // those; look-ahead fetch: all of its rows)
  kStatEarlyDeferred,  // of those, rows read from the host only after Stage One (staging full)
  kNumStats
};

// Word written to every bucket/slot by a reset: lifetime -1, invalid, fp 0, slot 0.
constexpr uint32_t kEmptyWord = 0xFF800000u;

struct MatchParams {
  int32_t B, K, n_q, S, m, R, L;
  uint32_t a1, a2;
  uint32_t f_mask;              // F - 1, F = 2^(23-m)
  const int32_t* topk;          // [B][n_q][K]
  const int64_t* verified;      // [B] or nullptr
  const int64_t* rows;          // [B]
  int32_t* table_c;             // [B][S]
  uint32_t* table_q;            // [B][S]
  int32_t* slots_out;           // [B][n_q][K]
  int32_t* miss_counts;         // [B][n_q]
  int2* miss_list;              // [B][n_q*K]  (index, slot)
  unsigned long long* stats;    // [B][kNumStats]
  uint8_t* hit_mask;            // [B][n_q][K] 1 = hit, or nullptr (not written)
  // Stage Two plan of the resident-reuse gather (written when plan_words > 0)
  int32_t plan_words;           // words of the end-of-step index map in LDS
  int32_t plan_list_off;        // LDS byte offset of the step's transfer list kept as 16-bit slots
  int32_t plan_scan_off;        // LDS byte offset of the scan's per-wave candidate lists (0: none)
  int2* host_list;              // [B][n_q*K] (index, slot) copied from the host
  int2* host_fan;               // [B][n_q*K] the two further slots a host entry is also copied to (-1: none)
  int32_t* host_third;          // [B][n_q*K] a third further slot (-1: none), with plan_third
  int32_t* plan_third;          // [B][plan_words] that slot by map position (four tokens per step), or nullptr
  int2* res_list;               // [B][n_q*K] (source slot, slot): row already resident
  int2* rep_list;               // [B][n_q*K] (source slot, slot): repeat of a host entry
  int32_t* plan_counts;         // [B][3] host, resident, repeat entries
  int32_t* plan_claim;          // [2] resident and host rows claimed by the gather (reset here)
  // early-fetch transfer (nullptr otherwise): the keys fetched before Stage
  // One leave the plan, and each request flags when its O is final
  const int32_t* early_x;       // [B][n_q*K] early keys of each request
  const int32_t* early_n;       // [B] number of early keys
  uint32_t* early_done;         // [B] 1 once the request's slots are written
};

// Host rows that the matching launch reads into HBM staging ahead of the
// gather (fetch_body.h): one small table per fetching workgroup.
struct AheadView {
  int32_t served;               // requests [0, served) are fetched for (0: no row is fetched ahead)
  int32_t parts;                // fetching workgroups per request
  int32_t quota;                // rows a workgroup fetches at most
  int32_t entries;              // entries of a workgroup's table, a power of two, at most 256
  int2* table;                  // [served * parts][entries] (index, its place among the workgroup's rows; -1 = none)
  uint64_t stage0, stage1;      // [served * parts][quota] staged rows of each stream
};

struct AheadParams {
  AheadView view;
  int32_t n_streams;
  const uint64_t* host_ptrs;    // [n_streams][B]
  int64_t row_bytes0, row_bytes1;
};

struct GatherParams {
  int32_t B, n_q, K, S;
  // entry counts of request r: miss_counts[r * count_stride + g], g < counts_per_req
  const int32_t* miss_counts;
  int32_t counts_per_req, count_stride;
  const int2* miss_list;        // [B][n_q*K] (index or source slot, slot)
  const int2* fan;              // [B][n_q*K] two further destination slots per entry (-1: none), or nullptr
  const int32_t* third;         // [B][n_q*K] a third further slot per entry (-1: none), or nullptr
  const int64_t* rows;          // [B]
  int32_t n_streams;
  const uint64_t* host_ptrs;    // [n_streams][B] device-visible addresses of host row 0
  const uint64_t* buf_ptrs;     // [n_streams][B] device buffer base addresses
  int64_t row_bytes0, row_bytes1;
  // position-level assignment only
  const int32_t* topk;          // [B][n_q][K]
  const int32_t* slots;         // [B][n_q][K]
  const uint8_t* hit_mask;      // [B][n_q][K]
  AheadView ahead;              // rows already in HBM staging (served = 0: none)
};

// Device-wide chunk queue of the pipelined step (workspace resident).
struct PipeParams {
  int* head;          // next queue entry to claim
  int* tail;          // queue entries reserved by producers
  int* done;          // requests whose Stage One has finished
  int* exit_count;    // workgroups that have left
  int* error;         // set when a consumer gave up waiting
  int* last_epoch;    // stamp of the last finished step (advanced on the device)
  int4* chunks;       // [max_chunks] (request, first miss, count, epoch)
  int max_chunks;
  int epoch;          // this step's stamp, never 0 (set by the kernel from last_epoch)
};

// Early-fetch transfer: the rows of indices that no slot held when the step
// began are read from the host while Stage One runs (workspace resident).
struct EarlyParams {
  int32_t B, K, n_q, S;
  uint32_t map_words;           // LDS map of the list kernel
  const int32_t* topk;          // [B][n_q][K]
  const int64_t* rows;          // [B]
  const int32_t* table_c;       // [B][S] cached indices as the step begins
  const int32_t* slots;         // [B][n_q][K] O of this step
  int32_t* early_x;             // [B][n_q*K] early keys
  int4* early_pos;              // [B][n_q*K] flat positions g*K+i of each key, -1 padded
  int32_t* early_n;             // [B]
  uint32_t* done;               // [B] O final (set by the matching workgroups)
  int* ctl;                     // [0] rows claimed, [1] staging rows claimed, [2] finish entries
  int4* fin;                    // [B*n_q*K] (request, key, staging row or -1, 0) left to finish
  int32_t stage_rows;           // staging capacity in rows (0: none)
  int32_t direct;               // write rows straight into known slots
  uint64_t stage0, stage1;      // staging bases per stream
  unsigned long long* stats;    // [B][kNumStats]
  int32_t n_streams;
  const uint64_t* host_ptrs;    // [n_streams][B]
  const uint64_t* buf_ptrs;     // [n_streams][B]
  int64_t row_bytes0, row_bytes1;
  // the matching workgroup's own lists (resident-reuse plan of the rest)
  const int2* host_list;
  const int2* host_fan;
  const int2* res_list;
  const int2* rep_list;
};

struct DualPtrParams {
  int32_t B, K;
  const int32_t* topk;          // [B][K]
  const int64_t* rows;          // [B]
  int2* state;                  // [B][K] (cached id, slot) sorted by id
  int32_t* slots_out;           // [B][K]
  int32_t* miss_counts;         // [B]
  int2* miss_list;              // [B][K]
  unsigned long long* stats;    // [B][kNumStats]
};

// Arguments of avsg_step_static's set-up kernel.  4 KB of kernel arguments hold
// at most 480 values, more of them go in further launches; a launch with few
// takes the short form, since the runtime's argument memory is what bounds the
// number of launches in flight (at 4 KB each, 400 calls in a row waited for it).
constexpr int kSetupWords = 480, kSetupWordsShort = 48;
template <int WORDS>
struct StaticSetup {
  unsigned long long *host_ptrs, *buf_ptrs, *rows;
  int32_t ptrs;                 // entries of host_ptrs and of buf_ptrs
  int32_t first, n;             // values [first, first + n) of [host_ptrs | buf_ptrs | rows]
  int32_t pair_period;
  // cold start: hash tables or (index, slot) pairs to empty, counters to zero (0: none)
  int32_t* table_c;
  uint32_t* table_q;
  size_t table_words;
  int2* pair;
  size_t pairs;
  unsigned long long* stats;
  size_t n_stats;
  unsigned long long v[WORDS];
};
static_assert(sizeof(StaticSetup<kSetupWords>) <= 4096, "one launch's arguments");

// LDS bytes of the matching kernel for (S, K); 0 if K exceeds the supported
// indices per thread.
size_t match_lds_bytes(int S, int K);
// threads of the matching workgroup for (S, K)
int match_threads(int S, int K);
size_t dualptr_lds_bytes(int K);

// `ahead`: served * parts further workgroups fetch rows beside the matching ones
hipError_t launch_match_hash(const MatchParams& p, const AheadParams& ahead, size_t lds, hipStream_t s);
// the one-launch step of small single-token steps (K <= 1024):
// `shares` workgroups per request; tickets[B] are 0 between steps
hipError_t launch_match_copy(const MatchParams& p, const GatherParams& g, uint32_t* tickets, int shares, size_t lds,
                             hipStream_t s);
// dynamic LDS of a fetching workgroup
size_t ahead_lds_bytes(int S, int entries, int quota);
hipError_t prepare_match_hash(size_t lds);
hipError_t launch_reset_tables(int32_t* c, uint32_t* q, size_t n, hipStream_t s);
hipError_t launch_zero_u64(unsigned long long* p, size_t n, hipStream_t s);
// validate mode: verdict[B * n_q] per token row (1 index out of range, 2 index
// repeated, 3 both, 0 valid); K <= 8192
hipError_t launch_validate_topk(const int32_t* topk, const int64_t* rows, int B, int n_q, int K,
                                int32_t* verdict, hipStream_t s);
hipError_t launch_static_setup(const StaticSetup<kSetupWords>& a, hipStream_t s);
hipError_t launch_gather_balanced(const GatherParams& p, int workers, hipStream_t s);
hipError_t launch_gather_request(const GatherParams& p, hipStream_t s);
hipError_t launch_gather_position(const GatherParams& p, int workers, hipStream_t s);
// device-to-device row copies: miss_list entries are (source slot, slot)
hipError_t launch_copy_device(const GatherParams& p, int workers, hipStream_t s);
// resident-reuse Stage Two: host entries, then resident copies, both claimed
// tile by tile; `dev` describes the resident list, `claim` the two counters
hipError_t launch_gather_resident(const GatherParams& host, const GatherParams& dev, int* claim,
                                  int workers, hipStream_t s);
// words of the end-of-step index map the matching kernel can hold for (S, K, n_q);
// 0 when the plan does not fit in the kernel's LDS
int plan_map_words(int S, int K, int n_q);
// LDS byte offset of the transfer list the matching kernel keeps for the plan
size_t plan_list_offset(int S, int K, int n_q);
size_t plan_scan_offset(int S, int K, int n_q);
// dynamic LDS of the matching workgroup for (S, K, n_q), with room for the
// end-of-step plan when `plan`; 0 when it does not fit
size_t stage_one_lds_bytes(int S, int K, int n_q, bool plan);
int pipelined_chunk_misses();
size_t pipelined_lds_bytes(int S, int K);
hipError_t prepare_step_pipelined(size_t lds);
hipError_t launch_step_pipelined(const MatchParams& mp, const GatherParams& gp, const PipeParams& q,
                                 int workgroups, size_t lds, hipStream_t s);
// early-fetch step: list kernel (one workgroup per request), matching +
// early copies in one launch (B matching workgroups + `workers` copiers), then
// the finishing kernel for rows fetched before their slots were known
uint32_t early_map_words(int K, int n_q);
size_t early_list_lds_bytes(int K, int n_q);
size_t early_step_lds_bytes(int S, int K, int n_q);
hipError_t prepare_step_early(size_t list_lds, size_t step_lds);
hipError_t launch_early_list(const EarlyParams& e, size_t lds, hipStream_t s);
hipError_t launch_step_early(const MatchParams& mp, const EarlyParams& e, int workers, size_t lds,
                             hipStream_t s);
hipError_t launch_finish_early(const EarlyParams& e, int workers, hipStream_t s);
hipError_t launch_match_dualptr(const DualPtrParams& p, size_t lds, hipStream_t s);
hipError_t prepare_match_dualptr(size_t lds);
hipError_t launch_reset_dualptr(int2* state, int B, int K, hipStream_t s);

}  // namespace avsg
