// Internal declarations shared by the kernels (vtoken_kernels.hip, vtoken_copy.hip,
// vtoken_attention.hip, vtoken_planner.hip, vtoken_layout.hip) and the C ABI front end
// (vtoken_abi.hip). Not installed; the public interface is include/vtoken.h.
#pragma once

#include <stdint.h>
#include <hip/hip_runtime.h>

#include "vtoken.h"

namespace vtoken {

// Launch geometry of the metadata kernels (one workgroup per request each).
constexpr int kCountThreads = 512;
constexpr int kCountThreadsShort = 128;   // for requests averaging < kLongRequestTokens
constexpr int kPlanThreads = 1024;
constexpr int kPlanBallots = 8;                            // ballots per wave per tile
constexpr int kPlanTile = kPlanThreads * kPlanBallots;     // tokens per tile (8192)
constexpr int kPlanHead = 8192;   // free-list entries a plan workgroup holds in LDS (32 KiB)
// Batches of more than kFusedAdmitReqs requests (kFusedAdmitShortReqs when their requests
// average fewer than kLongRequestTokens tokens) run the admission once, in a launch of its
// own, instead of in every plan workgroup; it stages the first kAdmitStage live counts and
// table lengths in LDS, and their plan workgroups have kPlanThreadsSplit threads.
constexpr int kFusedAdmitReqs = 512;
constexpr int kFusedAdmitShortReqs = 256;
constexpr int kLongRequestTokens = 1024;
constexpr int kAdmitStage = 4096;
constexpr int kPlanThreadsSplit = 256;
// Batches this small are planned by one workgroup in one launch (they are bound by launch
// latency); larger ones by a count launch and a plan launch of one workgroup per request.
constexpr int kSmallReqs = 24;
constexpr int kSmallTokens = 8192;
constexpr int kFreeThreads = 256;

// Copy kernel geometry: 256 threads, each moving 16-byte units.
constexpr int kCopyThreads = 256;

// The plan's mode word (plan->counters[4]), written by the kernels that build a plan and
// checked by the copy and the freed list that consume it.
constexpr int32_t kPlanOutOfPlace = 1;   // vtoken_build_token_table
constexpr int32_t kPlanInPlace = 2;      // vtoken_build_token_table_inplace
constexpr int32_t kPlanPartial = 3;      // vtoken_plan_partial: the out-of-place copy; its
                                         // released blocks are the planner state's sources

struct MetaArgs {
  // batch
  const int32_t* seq_lens;
  const int32_t* tok_indptr;
  const int32_t* bt_indptr;
  const int32_t* block_ids;
  const uint8_t* live;
  const int32_t* free_list;
  int32_t num_reqs;
  int32_t num_tokens;
  int32_t num_bt_entries;
  int32_t free_len;
  // cache geometry
  int32_t block_size;
  int32_t num_blocks;
  // plan
  int32_t* token_slot;
  int32_t* live_count;
  int32_t* admitted;
  int32_t* dst_indptr;
  int32_t* new_bt_indptr;
  int32_t* new_block_ids;
  int32_t* src_plan;
  int32_t* freed_indptr;
  int32_t* counters;
  int64_t new_bt_capacity;
  int64_t src_plan_capacity;
  int32_t inplace;          // 1: destinations are each request's own leading blocks
};

struct CopyArgs {
  uint8_t* kv;
  int64_t plane_bytes;      // num_blocks * S * row_bytes
  int64_t row_bytes;        // H * D * elem_bytes, a multiple of 16
  int32_t num_planes;       // 2 * L
  int32_t block_size;       // S
  int32_t num_blocks;
  int32_t num_slots;        // num_blocks * S
  int32_t row_units;        // row_bytes / 16
  int32_t chunk_units;      // S * row_units
  int32_t max_used;         // upper bound on counters[0] the buffers can hold
  uint32_t row_magic;       // floor(2^32 / row_units) + 1 (0 if row_units == 1)
  int32_t order;            // 1 plane-major, otherwise block-major work order
  const int32_t* src_plan;
  const int32_t* free_list;
  int32_t* counters;        // read; the status word is set if the plan's mode does not match
  int32_t copy_grid;        // workgroups of the copy (set by the launch)
  // the freed list in the same launch (vtoken_repack_free): the num_reqs workgroups after the
  // copy's write request r's released blocks; num_reqs == 0: none (vtoken_repack). freed may be
  // null when the batch has no table entries (nothing to write)
  int32_t num_reqs;
  int64_t num_bt_entries;
  const int32_t* bt_indptr;
  const int32_t* block_ids;
  const int32_t* admitted;
  const int32_t* freed_indptr;
  int32_t* freed;
  int64_t freed_capacity;
};

// The released blocks of request r, written to freed[freed_indptr[r] ..): the last
// freed_indptr[r+1] - freed_indptr[r] entries of its old table (all of it out of place, the
// part past the new table in place), for an admitted request; nothing for the others. The
// threads of the calling workgroup share the copy; ranges are checked before any access.
__device__ inline void write_freed_blocks(int r, const int32_t* admitted,
                                          const int32_t* bt_indptr, const int32_t* freed_indptr,
                                          const int32_t* block_ids, int64_t num_bt_entries,
                                          int32_t* freed, int64_t capacity) {
  if (!admitted[r]) return;
  const int b0 = bt_indptr[r];
  const int m = bt_indptr[r + 1] - b0;
  const int64_t o = freed_indptr[r];
  const int n = freed_indptr[r + 1] - freed_indptr[r];
  if (b0 < 0 || m < 0 || (int64_t)b0 + m > num_bt_entries || o < 0 || n < 0 || n > m) return;
  const int first = b0 + m - n;
  for (int j = threadIdx.x; j < n; j += blockDim.x) {
    if (o + j < capacity) freed[o + j] = block_ids[first + j];
  }
}

// Arguments of the in-place copy.
struct InplaceArgs {
  uint8_t* kv;
  int64_t plane_bytes;
  int64_t row_bytes;
  int32_t num_planes;
  int32_t block_size;
  int32_t num_blocks;
  int32_t num_slots;
  int32_t row_units;
  int32_t chunk_units;
  uint32_t row_magic;
  int32_t num_reqs;
  int64_t src_plan_capacity;
  int64_t new_bt_capacity;
  const int32_t* src_plan;
  const int32_t* new_block_ids;
  const int32_t* dst_indptr;
  const int32_t* new_bt_indptr;
  const int32_t* admitted;
  int32_t* counters;        // read; the status word is set if the plan's mode does not match
  // the freed list in the same launch (vtoken_repack_inplace_free; variants 0 and 4), by the
  // free_reqs workgroups after the copy's; 0: none. freed may be null when the batch has no
  // table entries (nothing to write)
  int32_t free_reqs;
  int64_t num_bt_entries;
  const int32_t* bt_indptr;
  const int32_t* block_ids;
  const int32_t* freed_indptr;
  int32_t* freed;
  int64_t freed_capacity;
};

// Largest chunk (S * row_bytes) the in-place copy stages through LDS.
constexpr int64_t kMaxInplaceChunkBytes = 64 * 1024;

// Slot mapping (live tokens' slots per request, logical order).
struct SlotMapArgs {
  int32_t num_reqs;
  int32_t num_tokens;
  const int32_t* tok_indptr;
  const int32_t* token_slot;
  const int32_t* live_count;
  const int32_t* counters;
  int32_t* slot_indptr;
  int32_t* slots;
  int64_t slots_capacity;
  int32_t reserve;        // extra room per request (slot table); 0 for a packed mapping
  int32_t* slot_count;    // slot table counts, or null
};

struct AppendArgs {
  int32_t num_reqs;
  const int32_t* append_indptr;
  const int32_t* append_slots;
  const int32_t* slot_start;
  int32_t* slot_count;
  int32_t* slots;
  int32_t* status;
};

// How long the splits of a decode are (decode_split_rule()).
struct DecodeSplit {
  int32_t tokens;   // of a split in a batch whose requests are as long as the bound: a multiple of
                    // decode_round_tokens(), as are its halves below
  int32_t few;      // slots of a batch below which such splits leave the chip idle (0: none)
  int32_t room[3];  // slots of a request for which there is room at a half, a quarter, an eighth
};

// Paged decode attention of one layer through a slot mapping.
struct AttnArgs {
  const uint8_t* kv;
  int64_t plane_bytes;
  int64_t row_bytes;
  int32_t num_kv_heads;
  int32_t num_q_heads;
  int32_t head_dim;
  int32_t layer;
  int32_t kv_kind;   // 0 fp16, 1 bf16, 2 fp8 e4m3
  int32_t num_slots;
  int32_t num_reqs;
  int32_t splits;    // split records per (request, query head) in the workspace
  DecodeSplit split;
  int64_t max_count;     // slots a request may hold (more: NaN outputs)
  float scale;
  const float* q;
  float* out;
  float* workspace;
  const int32_t* slot_indptr;
  const int32_t* slots;
  const int32_t* slot_count;  // null: counts from slot_indptr
};

// Arguments of the partial reclamation pass (vtoken_plan_partial).
struct PlannerArgs {
  int32_t num_reqs;
  int32_t num_tokens;
  int32_t num_bt_entries;
  int32_t block_size;
  int32_t num_blocks;
  int32_t num_slots;
  int32_t free_len;
  int32_t theta_num, theta_den;
  int32_t max_live;
  int32_t min_eligible;
  int32_t free_watermark;
  int64_t max_sources;
  const int32_t* seq_lens;
  const int32_t* tok_indptr;
  const int32_t* bt_indptr;
  const int32_t* block_ids;
  const uint8_t* live;
  const int32_t* slot_in;
  const int32_t* free_list;
  const uint8_t* pinned;  // may be null
  uint64_t* live_bits;
  int32_t* refs;
  int32_t* n_b;
  int32_t* selected;
  int32_t* elig_cum;
  int32_t* src_count;
  int32_t* sources;
  int64_t* stats;
  int32_t* token_slot;
  int32_t* live_count;
  int32_t* admitted;
  int32_t* dst_indptr;
  int32_t* new_bt_indptr;
  int32_t* new_block_ids;
  int32_t* src_plan;
  int32_t* freed_indptr;
  int32_t* counters;
  int64_t new_bt_capacity;
  int64_t src_plan_capacity;
};

hipError_t launch_planner(const PlannerArgs& a, hipStream_t stream);

hipError_t launch_slot_mapping(const SlotMapArgs& a, hipStream_t stream);
// num_new: at least the slots the call appends, negative if unknown; it only picks the launch
hipError_t launch_append_slots(const AppendArgs& a, int64_t num_new, hipStream_t stream);
hipError_t launch_paged_decode(const AttnArgs& a, hipStream_t stream);
// The library-held decode workspace (vtoken_paged_decode_noalloc): its size, and its address
// on the device of `stream` (looked up on the first call per device; allocates nothing).
constexpr int64_t kDecodeScratchBytes = VTOKEN_DECODE_SCRATCH_BYTES;
hipError_t decode_scratch(hipStream_t stream, float** out);
// Decode split geometry. In a round each of a split workgroup's four waves takes 4 KiB of K (and
// of V) of one KV head, 64 bytes per lane and operand, but at least a tile of 16 tokens.
constexpr int kDecodeSplitWaves = 4;
constexpr int decode_wave_tokens(int head_dim, int elem_bytes) {
  return head_dim * elem_bytes > 256 ? 16 : 4096 / (head_dim * elem_bytes);
}
constexpr int decode_round_tokens(int head_dim, int elem_bytes) {
  return kDecodeSplitWaves * decode_wave_tokens(head_dim, elem_bytes);
}
// A split is 1, 2, 4 or 8 units of 32 KiB of K (whole rounds; head_dim 32, 64, 128, 256 -> 512,
// 256, 128, 64 tokens a unit for 16-bit caches, twice as many at 1 byte per element).
constexpr int decode_unit_tokens(int head_dim, int elem_bytes) {
  return 32768 / (head_dim * elem_bytes);
}
// Units per split for `pairs` (request, KV head) pairs of max_tokens slots each. Short splits
// pay the start of a workgroup (3 dependent reads, the query operands) and its record often, long
// ones leave the chip part idle at the end: the time is estimated as the workgroups' rounds
// through the chip plus half a workgroup's time, with a start of 3 us and a unit's 64 KiB of K
// and V at the workgroup's share of 7 TB/s (resident workgroups: 3 per CU, 2 with 512-byte head
// rows). Measured per layer for 1, 2, 4, 8 units (estimate's choice in brackets): bf16, 64
// requests of 678-2,521 slots, 8 heads x 128 86, 79.5, [78], 83 us; fp8, 29 of 5-20K 164, 149,
// [143], 144; fp8, 45 of 1.4-2.6K [37.4], 37.4, 39, 53; bf16, 18 of 6K, 4 x 256 107, 89, [83],
// 80; bf16, 5 of 1.0-1.6K, 8 x 256 23.4, [19.1], 20.7, 19.4.
constexpr int decode_split_units(int head_dim, int elem_bytes, int64_t pairs,
                                 int64_t max_tokens) {
  const int resident = 256 * (head_dim * elem_bytes > 256 ? 2 : 3);
  const double start = 3.0, unit = 65536.0 * resident / 7e6;   // us
  const int64_t tokens = decode_unit_tokens(head_dim, elem_bytes);
  int best = 1;
  double best_time = 0;
  for (int u = 1; u <= 8; u *= 2) {
    const double one = start + u * unit;
    const double groups = static_cast<double>(pairs) *
                          static_cast<double>((max_tokens + u * tokens - 1) / (u * tokens));
    const double time = groups * one / resident + one / 2;
    if (u == 1 || time < best_time) {
      best = u;
      best_time = time;
    }
  }
  return best;
}

// Workgroups of a split launch below which shorter splits are faster.
constexpr int kDecodeFewGroups = 384;   // 1.5 per CU

// The host knows the bound max_tokens, not the requests' slots, and takes units and room for splits
// as if every request were that long. Where the batch holds so much less that splits of this
// length would be fewer than kDecodeFewGroups workgroups, the kernels take shorter ones, as far as
// the room goes. That needs fewer (request, KV head) pairs than workgroups; other calls keep the
// kernels that don't look at the batch's slots (those are 0.2 us a kernel slower, 1% of 128 requests
// of 1,000 slots). Per layer with the host's and with halved splits: fp8, 8 requests of 2,000 slots,
// 8 heads x 128, bound 8,000 19.4 us (250 workgroups), 15.7 (500); bf16, 8 of 1,024, bound 4,096
// 15.4 (256), 13.0 (512); bf16, 16 of 1,500, 8 x 32, bound 12,000 19.1 (187), 15.1 (375); but
// bf16, 32 of 4,000, 1 x 128, bound 16,000 19.4 (500), 20.8 (1,000); bf16, 6 of 3,000, 4 x 256,
// bound 12,000 21.7 (562), 23.0 (1,125).
constexpr DecodeSplit decode_split_rule(int head_dim, int elem_bytes, int64_t num_reqs,
                                        int64_t heads, int64_t max_tokens) {
  const int64_t unit = decode_unit_tokens(head_dim, elem_bytes);
  const int units = decode_split_units(head_dim, elem_bytes, num_reqs * heads, max_tokens);
  const int64_t splits = max_tokens > 0 ? (max_tokens + units * unit - 1) / (units * unit) : 1;
  const bool shorten = units > 1 && num_reqs * heads < kDecodeFewGroups;
  DecodeSplit s{static_cast<int32_t>(units * unit),
                static_cast<int32_t>(shorten ? kDecodeFewGroups * units * unit / heads : 0),
                {-1, -1, -1}};
  for (int k = 0; k < 3 && (units >> (k + 1)) > 0; ++k) {
    const int64_t room = (units >> (k + 1)) * unit * splits;
    s.room[k] = static_cast<int32_t>(room < INT32_MAX ? room : INT32_MAX);
  }
  return s;
}

// Split slots of a request as long as the bound.
constexpr int32_t decode_splits(const DecodeSplit& s, int64_t max_tokens) {
  return max_tokens > 0 ? static_cast<int32_t>((max_tokens + s.tokens - 1) / s.tokens) : 1;
}

// Tokens per split of a request of `count` slots in a batch of `total`: its splits fit the room, or
// they are as long as the host's (the last one then takes what is left). A smaller total and a
// smaller room imply the larger ones, so the halvings add up (no branches: the kernels wait for
// this before their first load of K).
__host__ __device__ constexpr int decode_request_tokens(const DecodeSplit& s, int count,
                                                        int total) {
  const int halvings = ((total < s.few) & (count <= s.room[0])) +
                       ((total < s.few >> 1) & (count <= s.room[1])) +
                       ((total < s.few >> 2) & (count <= s.room[2]));
  return s.tokens >> halvings;
}

// The most slots a request may hold: max_tokens rounded up to whole units of the size below (at
// least one), which is what the C ABI has promised since splits had that size.
constexpr int64_t decode_max_count(int head_dim, int elem_bytes, int group, int64_t max_tokens) {
  const int64_t base = decode_unit_tokens(head_dim, elem_bytes);
  const bool twice = elem_bytes == 2 && (group == 8 || max_tokens >= 64 * base);
  const int64_t unit = twice ? 2 * base : base;
  return max_tokens > 0 ? (max_tokens + unit - 1) / unit * unit : unit;
}
// The smallest split over the element sizes: the workspace bound of the C ABI.
constexpr int decode_min_split_tokens(int head_dim) { return decode_unit_tokens(head_dim, 2); }
// Split slots per (request, KV head) in the split launch's grid (where the splits of a head are
// neighbours): an odd number. Workgroups are handed to the 8 XCDs in turn, so with an even one the
// requests' first splits, which hold the work, fall on the same XCDs: 20 slots left one XCD 12%
// above the mean (Llama-3-8B Random, 5% slower); 64 and 128, under bounds far above the requests,
// put all of it on one or two (fp8, 8 requests of 2,000 slots, bound 131,072: 110 us, 39 so).
__host__ __device__ constexpr int decode_grid_splits(int splits) { return splits | 1; }

// (request, split) pairs of the split launch's grid: whole octets, for the kernels that place the
// heads of a split on one XCD.
__host__ __device__ constexpr int64_t decode_grid_groups(int64_t n) { return (n + 7) / 8 * 8; }

hipError_t launch_build(const MetaArgs& a, hipStream_t stream);
// variant: 0 default (4), 1 LDS double buffer, 2 LDS single buffer, 3 registers, 4 row walk
// (num_tokens and held_bytes, the batch's tokens and the bytes of its blocks, only pick the kernel)
hipError_t launch_repack_inplace(const InplaceArgs& a, int variant, int64_t num_tokens,
                                 int64_t held_bytes, hipStream_t stream);
hipError_t launch_free(const MetaArgs& a, int32_t* freed, int64_t freed_capacity,
                       hipStream_t stream);
// The layout check (vtoken_layout.hip): words[0] is the flag word, words[1 ..] one bit per
// block; layout_words() words in all.
struct LayoutArgs {
  const int32_t* block_ids;
  const int32_t* free_list;
  int64_t num_bt_entries;
  int64_t free_len;
  int32_t num_blocks;
  int64_t num_words;
  uint32_t* words;
  int32_t* status;
};
int64_t layout_words(int32_t num_blocks);
hipError_t launch_check_layout(const LayoutArgs& a, hipStream_t stream);
// variant/grid/order as in vtoken_repack_options; returns hipErrorInvalidValue for an
// unknown variant or order.
hipError_t launch_repack(const CopyArgs& a, int variant, int grid, int order,
                         hipStream_t stream);
int num_repack_variants();

// Largest chunk (S * row_bytes / 16 units) and row (row_bytes / 16 units) the copy kernel's
// multiply-high division is exact for.
constexpr int64_t kMaxChunkUnits = (1 << 20) - 1;
constexpr int64_t kMaxRowUnits = 1 << 12;

// ---- device helpers shared by the metadata kernels (vtoken_kernels.hip, vtoken_planner.hip,
// which bring them in with `using namespace vtoken::meta`)
namespace meta {

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// Number of set bits of a wave-wide ballot in the lanes below this one.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// Lane i of each 16-lane row receives lane i - kN of its row, 0 for i < kN (DPP row shift).
template <int kN>
__device__ __forceinline__ int row_shr(int x) {
  static_assert(kN > 0 && kN < 16, "row shift");
  return __builtin_amdgcn_update_dpp(0, x, 0x110 + kN, 0xF, 0xF, true);
}

// Inclusive prefix sum over the 64 lanes (every lane active): within each 16-lane row by DPP
// row shifts (no LDS), then each row adds the totals of the rows below it, read from lanes
// 15, 31 and 47.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += row_shr<1>(v);
  v += row_shr<2>(v);
  v += row_shr<4>(v);
  v += row_shr<8>(v);
  const int t0 = __builtin_amdgcn_readlane(v, 15);
  const int t1 = __builtin_amdgcn_readlane(v, 31);
  const int t2 = __builtin_amdgcn_readlane(v, 47);
  const int row = lane_id() >> 4;
  return v + (row >= 1 ? t0 : 0) + (row >= 2 ? t1 : 0) + (row >= 3 ? t2 : 0);
}

// Inclusive prefix sum over lanes 0-15 (the first DPP row); the other rows scan their own.
__device__ __forceinline__ int row_inclusive_scan(int v) {
  v += row_shr<1>(v);
  v += row_shr<2>(v);
  v += row_shr<4>(v);
  return v + row_shr<8>(v);
}

// Exclusive scan of NV values per thread across the workgroup (at most 16 waves); total[k] is
// the sum. A wave whose values are all zero (requests past the batch's end) skips its own
// scan. The wave totals go through LDS once: lane w of every wave reads wave w's total and a
// 16-lane scan gives each wave its offset.
template <int NV>
__device__ __forceinline__ void block_exclusive_scan(int (&v)[NV], int (&total)[NV],
                                                     int (*lds)[NV]) {
  const int lane = lane_id();
  const int wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  int any = 0;
#pragma unroll
  for (int k = 0; k < NV; ++k) any |= v[k];
  int incl[NV];
  if (__ballot(any != 0) != 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) incl[k] = wave_inclusive_scan(v[k]);
  } else {
#pragma unroll
    for (int k = 0; k < NV; ++k) incl[k] = 0;
  }
  if (lane == 63) {
#pragma unroll
    for (int k = 0; k < NV; ++k) lds[wave][k] = incl[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int wt = row_inclusive_scan(lane < nwaves ? lds[lane][k] : 0);
    const int off = wave > 0 ? __builtin_amdgcn_readlane(wt, wave - 1) : 0;
    total[k] = __builtin_amdgcn_readlane(wt, nwaves - 1);
    v[k] = off + incl[k] - v[k];
  }
  __syncthreads();
}

// Nonzero bytes of a 32-bit word: each byte's bits are folded into its lowest bit (the bits
// shifted in from the next byte land at offsets >= 1 and are masked off).
__device__ __forceinline__ int nonzero_bytes(uint32_t w) {
  w |= w >> 4;
  w |= w >> 2;
  w |= w >> 1;
  return __popc(w & 0x01010101u);
}

// Division and remainder of non-negative positions and ranks by the block size S: shifts and
// masks when S is a power of two (the kernels that divide per token are instantiated for both).
template <bool kPow2>
struct BlockDiv {
  int s, sh;
  __device__ explicit BlockDiv(int S) : s(S), sh(__ffs(S) - 1) {}
  __device__ int div(int x) const { return kPow2 ? x >> sh : x / s; }
  __device__ int mod(int x) const { return kPow2 ? x & (s - 1) : x % s; }
};

}  // namespace meta

}  // namespace vtoken
