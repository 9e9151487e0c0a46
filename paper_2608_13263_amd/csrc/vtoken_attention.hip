// Consumer side of the repack on CDNA4 (gfx950): the attention slot mapping and a paged
// decode attention that reads the (repacked) KV cache through it.
//
//   slot_indptr_kernel   exclusive scan of the live counts (one workgroup; batches of more than
//                        2,048 requests)
//   slot_map_kernel      one workgroup per request: wave-ballot compaction of token_slot,
//                        the live tokens' slots in logical order (Sec. 3.4: the slot mapping
//                        is built through the token table, once per token)
//   decode_split_kernel  one workgroup per (request, KV head, split): scores and the weighted sum
//                        of V of the G query heads that share the KV head, both on the matrix
//                        cores, with a running softmax (flash-decoding partials)
//   decode_combine_kernel  one workgroup per (request, query head): merges the splits (no launch
//                        where one split covers every request)
//
// Decode attention is HBM-bound (2G flops per byte of K/V). Both products are small dense
// contractions (16 tokens x D x the G heads of a KV head, and their transposes) and run on
// MFMA, which leaves the vector ALUs to the softmax and the operand conversions.
#include <math.h>

#include <atomic>
#include <mutex>
#include <type_traits>

#include "vtoken_internal.h"

namespace vtoken {
namespace {


__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// ------------------------------------------------------------------------------------------
// Slot mapping.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void slot_indptr_kernel(SlotMapArgs a) {
  __shared__ int wave_tot[16];
  if (a.counters[3] != 0) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  int carry = 0;
  for (int base = 0; base < a.num_reqs; base += 1024) {
    const int r = base + tid;
    int live = r < a.num_reqs ? a.live_count[r] : 0;
    live = live < 0 ? 0 : live;
    if (r < a.num_reqs && a.slot_count != nullptr) a.slot_count[r] = live;
    int v = r < a.num_reqs ? live + a.reserve : 0;
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int t = __shfl_up(incl, d, 64);
      if (lane >= d) incl += t;
    }
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int off = carry, tot = 0;
    for (int w = 0; w < 16; ++w) {
      off += w < wave ? wave_tot[w] : 0;
      tot += wave_tot[w];
    }
    if (r < a.num_reqs) a.slot_indptr[r] = off + incl - v;
    carry += tot;
    __syncthreads();
  }
  if (tid == 0) a.slot_indptr[a.num_reqs] = carry;
}

// One workgroup per request compacts its live token slots in logical order: tiles of
// 16 waves x kSlotBallots x 64 tokens, every token_slot load of a tile in flight before its
// ballots, one pair of barriers per tile. kOffsets: each workgroup sums the counts of the
// requests before its own itself (at most kSlotOffsetReqs, two loads per thread, in flight with
// the first tile) and no launch of slot_indptr_kernel goes before: mapping of 8 requests of 300
// tokens 5.9 -> 4.0 us, 1,024 of 5,000 11.0 -> 9.3, 2,048 of 100 15.2 -> 13.9; at 4,096 requests the
// sums cost more than the launch (of 50 tokens 26.2 and 26.8 us, of 1,000 27.2 and 28.2).
constexpr int kSlotBallots = 8;
constexpr int kSlotOffsetReqs = 2048;

template <bool kOffsets>
__global__ __launch_bounds__(1024) void slot_map_kernel(SlotMapArgs a) {
  __shared__ int wave_tot[16];
  __shared__ int wave_before[16];
  const int r = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  int before = 0;
  if constexpr (kOffsets) {
#pragma unroll
    for (int q = 0; q < kSlotOffsetReqs / 1024; ++q) {
      const int i = q * 1024 + tid;
      const int live = a.live_count[i < r ? i : r];
      before += i < r ? (live < 0 ? 0 : live) + a.reserve : 0;
    }
  }
  if (a.counters[3] != 0) return;
  const int t0 = a.tok_indptr[r];
  const int n = a.tok_indptr[r + 1] - t0;
  int o;
  if constexpr (kOffsets) {
    int mine = a.live_count[r];
    mine = mine < 0 ? 0 : mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) before += __shfl_xor(before, d, 64);
    if (lane == 0) wave_before[wave] = before;
    __syncthreads();
    o = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) o += wave_before[w];
    if (tid == 0) {
      a.slot_indptr[r] = o;
      if (r == a.num_reqs - 1) a.slot_indptr[r + 1] = o + mine + a.reserve;
      if (a.slot_count != nullptr) a.slot_count[r] = mine;
    }
  } else {
    o = a.slot_indptr[r];
  }
  if (t0 < 0 || n < 0 || (int64_t)t0 + n > a.num_tokens || o < 0) return;
  const int32_t* ts = a.token_slot + t0;
  int carry = 0;
  for (int base = 0; base < n; base += 1024 * kSlotBallots) {
    // wave w holds positions base + w*64*kSlotBallots + k*64 + lane
    const int wbase = base + wave * (64 * kSlotBallots);
    int s[kSlotBallots];
#pragma unroll
    for (int k = 0; k < kSlotBallots; ++k) {
      const int p = wbase + k * 64 + lane;
      s[k] = p < n ? ts[p] : -1;
    }
    int rank[kSlotBallots];
    int local = 0;
#pragma unroll
    for (int k = 0; k < kSlotBallots; ++k) {
      const uint64_t m = __ballot(s[k] >= 0);
      rank[k] = local + lanes_below(m);
      local += __popcll(m);
    }
    if (lane == 0) wave_tot[wave] = local;
    __syncthreads();
    int off = carry, tot = 0;
    for (int w = 0; w < 16; ++w) {
      off += w < wave ? wave_tot[w] : 0;
      tot += wave_tot[w];
    }
#pragma unroll
    for (int k = 0; k < kSlotBallots; ++k) {
      const int64_t dst = (int64_t)o + off + rank[k];
      if (s[k] >= 0 && dst < a.slots_capacity) a.slots[dst] = s[k];
    }
    carry += tot;
    __syncthreads();
  }
}

// Append-only growth of a slot table: a request's new slots go after its current ones if its
// region has room. Where the caller says that few slots are new, one workgroup takes the whole
// batch in one launch, 8 to 1024 threads per request. Any others go to a workgroup per request,
// after a launch that clears the status word.
//
// Bound: latency, one after the other the ranges, the slots, the stores. One launch is 1.1-1.6 us
// less than two (8 requests of one new slot, with the clearing of the counts: 4.2 us for 5.8),
// but one compute unit moves few slots at a time (128 requests of 4,096 new slots took it 83 us, a
// workgroup per request 7.8) and the host does not know how the slots are spread: so there are at
// most kAppendSteps new slots per thread of a request, four rounds of loads where one request gets
// them all (8 requests, one of 2,000 new: 5.5 us for 6.3).
constexpr int kAppendSmallReqs = 128;
constexpr int kAppendSteps = 16;
constexpr int kAppendFlight = 4;   // loads of a thread in flight

// log2 of a request's threads in one workgroup: 10 (one request) .. 3 (65 to 128 of them).
constexpr int append_log2_most(int num_reqs) {
  int t = 10;
  while ((num_reqs << t) > 1024) --t;
  return t;
}
// The same, but down to 16 threads no more than hold num_new slots in one round of loads (8
// requests of one slot: 4.6 us with 128 threads each, 4.2 with 16).
constexpr int append_log2_threads(int num_reqs, int64_t num_new) {
  int t = append_log2_most(num_reqs);
  while (t > 4 && num_new <= (int64_t)kAppendFlight << (t - 1)) --t;
  return t;
}
constexpr bool append_in_one_launch(int num_reqs, int64_t num_new) {
  return num_reqs <= kAppendSmallReqs && num_new >= 0 &&
         num_new <= (int64_t)kAppendSteps << append_log2_most(num_reqs);
}

__global__ __launch_bounds__(1024) void append_small_kernel(AppendArgs a, int log2_threads) {
  const int threads = 1 << log2_threads;
  const int r = threadIdx.x >> log2_threads;
  const int sub = threadIdx.x & (threads - 1);
  int n = 0, cnt = 0;
  bool full = false;
  if (r < a.num_reqs) {
    const int a0 = a.append_indptr[r];
    n = a.append_indptr[r + 1] - a0;
    const int start = a.slot_start[r];
    const int cap = a.slot_start[r + 1] - start;
    cnt = a.slot_count[r];
    full = n > 0 && (a0 < 0 || cnt < 0 || (int64_t)cnt + n > cap);
    n = full ? 0 : n;
    int32_t* dst = a.slots + start + cnt;
    for (int base = sub; base < n; base += threads * kAppendFlight) {
      int s[kAppendFlight];
#pragma unroll
      for (int k = 0; k < kAppendFlight; ++k) {
        const int i = base + k * threads;
        s[k] = a.append_slots[a0 + (i < n ? i : base)];
      }
#pragma unroll
      for (int k = 0; k < kAppendFlight; ++k) {
        const int i = base + k * threads;
        if (i < n) dst[i] = s[k];
      }
    }
  }
  full = __syncthreads_or(full) != 0;   // also: every thread has read its request's count
  if (n > 0 && sub == 0) a.slot_count[r] = cnt + n;
  if (threadIdx.x == 0) a.status[0] = full ? VTOKEN_ERR_CAPACITY : 0;
}

__global__ __launch_bounds__(64) void append_status_kernel(AppendArgs a) {
  if (threadIdx.x == 0) a.status[0] = 0;
}

__global__ __launch_bounds__(256) void append_slots_kernel(AppendArgs a) {
  const int r = blockIdx.x;
  const int a0 = a.append_indptr[r];
  const int n = a.append_indptr[r + 1] - a0;
  if (n <= 0) return;
  const int start = a.slot_start[r];
  const int cap = a.slot_start[r + 1] - start;
  const int cnt = a.slot_count[r];
  if (a0 < 0 || cnt < 0 || (int64_t)cnt + n > cap) {
    if (threadIdx.x == 0) atomicCAS(a.status, 0, VTOKEN_ERR_CAPACITY);
    return;
  }
  for (int i = threadIdx.x; i < n; i += 256) a.slots[start + cnt + i] = a.append_slots[a0 + i];
  __syncthreads();
  if (threadIdx.x == 0) a.slot_count[r] = cnt + n;
}

// ------------------------------------------------------------------------------------------
// Paged decode attention.
// ------------------------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kPer = 8;  // elements of a head row per lane

// Eight consecutive elements of a K or V head row: 16 bytes of fp16 / bf16, 8 bytes of fp8.
template <int kKind>
struct Piece {
  typedef u32x4 type;
};
template <>
struct Piece<2> {
  typedef u32x2 type;
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
// the same in the caller's outputs and workspace, which are aligned to a float and no more
typedef f32x4 f32x4_out __attribute__((aligned(4)));
typedef f32x2 f32x2_in __attribute__((aligned(4)));

// The matrix-core operand type of the scores: fp16 caches multiply in fp16, bf16 and fp8
// caches in bf16 (every e4m3 value is exact in bf16).
template <int kKind>
struct ScoreOp {
  typedef bf16x8 type;
  typedef __bf16 elem;
};
template <>
struct ScoreOp<0> {
  typedef f16x8 type;
  typedef _Float16 elem;
};

template <int kKind>
__device__ __forceinline__ f32x4 score_mfma(typename ScoreOp<kKind>::type k,
                                            typename ScoreOp<kKind>::type q, f32x4 acc) {
  if constexpr (kKind == 0) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(k, q, acc, 0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(k, q, acc, 0, 0, 0);
  }
}

// Eight K elements as a matrix-core operand: the 16 loaded bytes as they are (fp16, bf16), or
// 8 fp8 bytes widened to bf16 by the gfx950 conversion instruction (scale 1).
template <int kKind>
__device__ __forceinline__ typename ScoreOp<kKind>::type k_operand(
    typename Piece<kKind>::type w) {
  if constexpr (kKind == 2) {
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const bf16x2 a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(static_cast<int>(w[i]), 1.f,
                                                                 false);
      const bf16x2 b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(static_cast<int>(w[i]), 1.f,
                                                                 true);
      o[4 * i] = a.x;
      o[4 * i + 1] = a.y;
      o[4 * i + 2] = b.x;
      o[4 * i + 3] = b.y;
    }
    return o;
  } else {
    return __builtin_bit_cast(typename ScoreOp<kKind>::type, w);
  }
}

typedef short i16x4 __attribute__((ext_vector_type(4)));

// Eight V elements as 16-bit values of the matrix-core type: fp16 / bf16 as loaded, fp8
// widened to bf16 (exact).
template <int kKind>
__device__ __forceinline__ u32x4 v_row16(typename Piece<kKind>::type w) {
  if constexpr (kKind == 2) {
    return __builtin_bit_cast(u32x4, k_operand<2>(w));
  } else {
    return w;
  }
}

// 16 (V elements) x 16 tokens x 16 (columns), for the rounds of one 16-token tile.
template <int kKind>
__device__ __forceinline__ f32x4 value_mfma4(i16x4 v, i16x4 p, f32x4 acc) {
  if constexpr (kKind == 0) {
    typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, v),
                                                 __builtin_bit_cast(f16x4, p), acc, 0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v, p, acc, 0, 0, 0);
  }
}

// LDS transpose read of gfx950 (ds_read_b64_tr_b16): in each group of 16 lanes, lane
// 4a + b receives element b of the four 16-bit values addressed by lanes a, a+4, a+8 and
// a+12 of its group (in that order).
__device__ __forceinline__ i16x4 lds_read_tr16(const uint8_t* lds_addr) {
  typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (lds_i16x4*)(reinterpret_cast<uintptr_t>(lds_addr)));
}

// Cross-lane steps of the decode without the LDS crossbar (ds_bpermute): DPP rotations inside
// 16-lane rows and the gfx950 row swaps (v_permlane16_swap, v_permlane32_swap). Every lane of
// the wave must be active.
//
// Lane i of each 16-lane row receives lane (i - kN) mod 16 of its row.
template <int kN>
__device__ __forceinline__ float row_ror(float x) {
  static_assert(kN > 0 && kN < 16, "row rotation");
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + kN, 0xF, 0xF, false));
}

// x combined with the value of lane i ^ 16 (kDist 16) or i ^ 32 (kDist 32): the swap leaves
// the even rows' values in one result and the odd rows' (the low half's and the high half's)
// in the other, in every lane.
template <int kDist, bool kMax>
__device__ __forceinline__ float xor_combine(float x) {
  const uint32_t u = __float_as_uint(x);
  float a, b;
  if constexpr (kDist == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  } else {
    static_assert(kDist == 32, "16 or 32");
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  }
  return kMax ? fmaxf(a, b) : a + b;
}

// Sum (or maximum) over the lanes i, i + kStride, i + 2 kStride, ... of the wave (kStride a
// power of two below 64); every lane receives its class's result.
template <int kStride, bool kMax>
__device__ __forceinline__ float lanes_reduce(float x) {
  if constexpr (kStride <= 1) x = kMax ? fmaxf(x, row_ror<1>(x)) : x + row_ror<1>(x);
  if constexpr (kStride <= 2) x = kMax ? fmaxf(x, row_ror<2>(x)) : x + row_ror<2>(x);
  if constexpr (kStride <= 4) x = kMax ? fmaxf(x, row_ror<4>(x)) : x + row_ror<4>(x);
  if constexpr (kStride <= 8) x = kMax ? fmaxf(x, row_ror<8>(x)) : x + row_ror<8>(x);
  if constexpr (kStride <= 16) x = xor_combine<16, kMax>(x);
  return xor_combine<32, kMax>(x);
}

// Requests whose outputs no split decides: without slots (zeros), and those whose slot range is
// malformed (the split kernel reads nothing for them) or holds more slots than max_tokens
// provides for (NaN).
__device__ __forceinline__ bool decode_fixed_output(const AttnArgs& a, int s0, int c) {
  return s0 < 0 || c <= 0 || c > a.max_count;
}

// Waves of a split workgroup.
constexpr int kSplitWaves = kDecodeSplitWaves;

// Split kernel of the paged decode, both products on the matrix cores.
//
// kKind: element type; kD: head_dim (32, 64, 128, 256); kShorten: the batch may hold so few slots
// that its splits are shorter than the host's (decode_split_rule()). One workgroup of four waves covers
// decode_request_tokens() tokens (a whole number of rounds) of one (request, KV head) and its 1,
// 2, 4 or 8 query heads; in round i wave w takes the kIT tokens from (i * 4 + w) * kIT on, 4 KiB
// of K and 4 KiB of V (8 KiB each with 512-byte head rows), and computes for them, on the matrix cores
// (MFMA 16x16x32, fp16 for fp16 caches, bf16 otherwise; fp8 widened to bf16):
//   scores  S[token][col] = K_tile (16 x kD) . Q2^T (kD x 16). The float32 query is split into
//           high and low 16-bit parts (q = hi + lo to ~2^-17; 2^-22 in fp16): column c < 8 of Q2
//           is the high part of head c, column c + 8 its low part (zero past the last head), so
//           one product carries both and the score of head c is S[.][c] + S[.][c + 8]. For bf16
//           operands a third part (to 2^-26) takes the scores' share out of the outputs' error
//           (3.1e-6 -> 1.9e-6 relative): with at most four heads it has columns c + 4, with eight
//           (kG8) a second product;
//   weights p = exp(score - m), m the wave's running maximum per head; where m grows, the sums so
//           far are scaled down;
//   values  O2[d][col] += V^T (16 elements x 32 tokens) . P2^T (32 tokens x 16) per 16-element
//           chunk, column c < 8 of P2^T the high part of head c's weights, column c + 8 their low
//           part, so O[.][c] = O2[.][c] + O2[.][c + 8], and a lane's column of O is that of its
//           scores: scaling it takes no exchange between lanes. The operand layout fixes which
//           tokens a lane holds: lane l has column l%16 and, of each 32-token step, tokens
//           4*(l/16)..+3 of its first 16-token tile and the same of its second; the V rows are
//           read in that order.
// The waves are merged with the usual max-rescaling into the split's record, or, where one split
// covers every request (a.splits == 1), into the outputs.
//
// Bound: HBM (with the arithmetic taken out, the loads alone run 3-5% faster). K and V are read
// the same way, 16 bytes per lane with consecutive lanes on one head row, so that every line is
// used by one non-temporal load (read in operand order, a line of K is split over two loads,
// which only plain loads serve at all well: 6.2 against 6.95 TB/s over a large cache); both go
// through this wave's LDS window into operand order (K rows padded by 16 bytes, V rows, read back
// by transpose reads, by 32, against bank conflicts). The next round's K loads are issued as soon
// as K is in the window, its V loads as soon as V is: the registers hold one round and a wave has
// 4 to 8 KiB in flight at any time, three waves per SIMD. Twice that per wave (8 KiB, two waves
// per SIMD) and four waves per SIMD measured the same within 2%; held to three waves, 8 KiB
// spills and is 10-20% slower. The query operands, the merge of the waves and the split record
// are paid once per split: in workgroups of one round they were over half of the 1,400
// instructions per wave, which bound fp8 batches.
// Measured per layer, merge included, against one round per workgroup and K in operand order:
// bf16, 64 requests of 678-2,521 slots, 8 heads x 128, G = 4 86.5 -> 78 us (421 MB); fp8, 29
// requests of 5,043-19,788, G = 8 169 -> 143 us (735 MB); bf16, 4 x 256, 18 requests of 6K
// 135 -> 83 us (437 MB).
// Non-finite K or V values are outside the contract (a zero weight times an infinite value
// gives NaN).
template <int kKind, int kD, bool kG8, bool kShorten>
__global__ __launch_bounds__(64 * kSplitWaves)
__attribute__((amdgpu_waves_per_eu(kD * (kKind == 2 ? 1 : 2) > 256 ? 2 : 3)))
void decode_split_kernel(AttnArgs a) {
  using OpT = typename ScoreOp<kKind>::type;
  using ElemT = typename ScoreOp<kKind>::elem;
  constexpr int kElem = kKind == 2 ? 1 : 2;
  constexpr int kWaves = kSplitWaves;
  constexpr int kThreads = 64 * kWaves;
  constexpr int kRow = kD * kElem;                   // bytes of a head row
  constexpr int kIT = decode_wave_tokens(kD, kElem);  // tokens of a wave per round: 16 .. 128
  constexpr int kStep = kWaves * kIT;                // tokens of a round
  constexpr int kTiles = kIT / 16;                   // 16-token score tiles
  constexpr int kChunks = kD / 32;                   // score k-steps
  constexpr int kKC = (kTiles + 1) / 2;              // 32-token value k-steps
  constexpr int kDC = kD / 16;                       // 16-element value chunks
  constexpr int kLanes = kRow / 16;                  // loads: lanes per token row
  constexpr int kTok = 64 / kLanes;                  // loads: tokens per instruction
  constexpr int kLd = kIT / kTok;                    // loads per operand and round
  constexpr int kSR = (kIT + 63) / 64;               // slot registers
  constexpr int kWin = kIT < 32 ? kIT : 32;          // V rows staged per k-step
  constexpr int kLdW = kWin / kTok;                  // V loads per k-step
  constexpr int kRowK = kRow + 16;                   // LDS bytes per K row
  constexpr int kRowV = kD * 2 + 32;                 // LDS bytes per V row (16-bit)
  static_assert(kLdW * kKC == kLd && kLdW * kTok == kWin, "round geometry");
  constexpr int kWinB = kIT * kRowK > kWin * kRowV ? kIT * kRowK : kWin * kRowV;
  constexpr int kRec = kD + 4;                       // merge: m, l, padding, kD values
  constexpr int kMergeB = kWaves * 8 * kRec * 4;
  constexpr int kLdsB = kWaves * kWinB > kMergeB ? kWaves * kWinB : kMergeB;
  __shared__ __attribute__((aligned(16))) uint8_t lds[kLdsB];
  constexpr bool kThird = kKind != 0;                // bf16 operands: a third query part
  constexpr int kHeads = kThird && !kG8 ? 4 : 8;     // heads side by side in the columns
  constexpr int kQ = kThird && kG8 ? 2 : 1;          // query operands per chunk
  __shared__ OpT q_s[kChunks * kQ][64];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.num_q_heads / a.num_kv_heads;   // query heads per KV head
  // the grid holds decode_grid_splits(a.splits) split slots per (request, KV head); one past
  // a.splits (a count rounded up to an odd one) returns at once
  const int gs = decode_grid_splits(a.splits);
  const int H = a.num_kv_heads;
  int split, h, r;
  if constexpr (kRow < 128) {
    // head rows shorter than a 128-byte line share it: the heads of a split run on one XCD, eight
    // workgroups apart (fp8, 4 and 8 heads x 32: 28.5 -> 19.7 us, 31.7 -> 21.7 us; with longer
    // rows the heads of a split at a time cost 2-5%)
    const int oct = blockIdx.x / (8 * H);
    const int x = blockIdx.x - oct * 8 * H;
    const int rs = oct * 8 + x % 8;
    h = x / 8;
    r = rs / gs;
    split = rs - r * gs;
  } else {
    split = blockIdx.x % gs;
    h = (blockIdx.x / gs) % H;
    r = blockIdx.x / (gs * H);
  }
  if (r >= a.num_reqs || split >= a.splits) return;
  const int total = kShorten ? a.slot_indptr[a.num_reqs] - a.slot_indptr[0] : 0;
  const int s0 = a.slot_indptr[r];
  const int c = a.slot_count != nullptr ? a.slot_count[r] : a.slot_indptr[r + 1] - s0;
  const int st = kShorten ? decode_request_tokens(a.split, c, total) : a.split.tokens;
  const int64_t qh0 = (int64_t)r * a.num_q_heads + h * G;   // first query head's row
  // (one branch for both, so that all the counts are read together)
  const bool fixed = decode_fixed_output(a, s0, c);
  const int t0 = split * st;
  if (fixed | (t0 >= c)) {
    if (!fixed || a.splits > 1) return;   // fixed outputs are written here if there is no merge
    const float fill = c == 0 && s0 >= 0 ? 0.f : __builtin_nanf("");
    for (int i = tid; i < G * kD; i += kThreads) a.out[qh0 * kD + i] = fill;
    return;
  }
  // the last split takes what is left (up to a.max_count)
  const int nt = split + 1 < a.splits && c - t0 > st ? st : c - t0;
  const int* slots = a.slots + s0 + t0;
  const uint8_t* kplane = a.kv + (int64_t)(2 * a.layer) * a.plane_bytes;
  const uint8_t* vplane = kplane + a.plane_bytes;
  const int grp = lane >> 4;    // operand k-group / result row group
  const int row = lane & 15;    // token of a tile (K operand) / column (Q, P, results)
  const int wt0 = wave * kIT;   // this wave's first token of round 0
  const int rounds = wt0 < nt ? (nt - wt0 + kStep - 1) / kStep : 0;
  const bool low = row >= 8;          // this lane's column holds low parts
  const int head = row & (kHeads - 1);
  const bool real = head < G;         // column of a query head (else zero padding)

  // Slot indices of round i: lane l holds token l (and l + 64, ..) of the wave's; tokens past the
  // split's end re-read its last one
  struct Slots {
    int s[kSR];
  };
  auto load_slots = [&](int i) {
    Slots x;
#pragma unroll
    for (int q = 0; q < kSR; ++q) {
      const int t = wt0 + i * kStep + q * 64 + lane;
      x.s[q] = slots[t < nt ? t : nt - 1];
    }
    return x;
  };
  bool bad = false;   // a slot outside the pool: never dereferenced, poisons the request
  int ls[kLd];        // slots of this lane's rows
  auto spread_slots = [&](Slots x) {
#pragma unroll
    for (int q = 0; q < kSR; ++q) {
      const bool ok = static_cast<unsigned>(x.s[q]) < static_cast<unsigned>(a.num_slots);
      bad |= !ok;
      x.s[q] = ok ? x.s[q] : 0;
    }
#pragma unroll
    for (int k = 0; k < kLd; ++k) {
      ls[k] = __shfl(x.s[k * kTok / 64], (k * kTok + lane / kLanes) & 63, 64);
    }
  };
  const int64_t lane0 = (int64_t)h * kRow + (lane % kLanes) * 16;
  auto load_rows = [&](const uint8_t* plane, u32x4 (&x)[kLd]) {
#pragma unroll
    for (int k = 0; k < kLd; ++k) {
      x[k] = __builtin_nontemporal_load(
          reinterpret_cast<const u32x4*>(plane + ((int64_t)ls[k] * a.row_bytes + lane0)));
    }
  };

  // ---- the query values and the first two rounds' slots, then the first round's K and V loads;
  // the query operands are built while those are in flight
  // The head dims of a k-chunk's lane group: any assignment gives the same dot products as
  // long as q and K use the same one. fp8 pairs the chunks (2c, 2c+1) so that a lane's two
  // 8-byte K pieces are 16 contiguous bytes, read by one LDS read.
  constexpr bool kPairK = kKind == 2 && kChunks % 2 == 0;
  auto head_dim_of = [&](int ch, int e) {
    return kPairK ? (ch >> 1) * 64 + grp * 16 + (ch & 1) * 8 + e : ch * 32 + grp * kPer + e;
  };
  Slots cur = load_slots(0);
  Slots nxt = load_slots(1);
  constexpr int kQC = (kChunks + kWaves - 1) / kWaves;   // query chunks a wave builds
  const float* qrow = a.q + (qh0 + (real ? head : 0)) * kD;
  float qraw[kQC][kPer];
#pragma unroll
  for (int x = 0; x < kQC; ++x) {
    // unconditional (a chunk past the last re-reads the last one, unused)
    const int ch = wave + x * kWaves < kChunks ? wave + x * kWaves : kChunks - 1;
#pragma unroll
    for (int e = 0; e < kPer; ++e) qraw[x][e] = qrow[head_dim_of(ch, e)];
  }
  __builtin_amdgcn_sched_barrier(0);
  u32x4 kr[kLd], vr[kLd];
  spread_slots(cur);
  load_rows(kplane, kr);
  load_rows(vplane, vr);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int x = 0; x < kQC; ++x) {
    const int ch = wave + x * kWaves;
    if (ch < kChunks) {
      OpT part, rest;
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const float q = real ? qraw[x][e] * a.scale : 0.f;
        const ElemT hi = static_cast<ElemT>(q);
        const float d = q - static_cast<float>(hi);
        const ElemT lo = static_cast<ElemT>(d);
        const ElemT third = static_cast<ElemT>(d - static_cast<float>(lo));
        part[e] = low ? lo : hi;
        if (kHeads == 4 && (row & 4) != 0) part[e] = low ? static_cast<ElemT>(0.f) : third;
        rest[e] = low ? static_cast<ElemT>(0.f) : third;
      }
      q_s[ch * kQ][lane] = part;
      if constexpr (kQ == 2) q_s[ch * kQ + 1][lane] = rest;
    }
  }
  __syncthreads();   // query operands in LDS; the K and V loads stay in flight
  // this wave's window; only this wave touches it, and a wave's LDS operations run in order, so
  // a compiler fence is all that its reads of other lanes' writes need
  uint8_t* win = lds + wave * kWinB;
  auto order_lds = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };

  float m = -INFINITY, l = 0.f;
  f32x4 o[kDC];
#pragma unroll
  for (int dc = 0; dc < kDC; ++dc) o[dc] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto round = [&](int i, auto more_t) {
    constexpr bool kMore = decltype(more_t)::value;
    // ---- K rows into the window; the next round's K loads
    order_lds();
    {
      uint8_t* dst = win + (lane / kLanes) * kRowK + (lane % kLanes) * 16;
#pragma unroll
      for (int k = 0; k < kLd; ++k) *reinterpret_cast<u32x4*>(dst + k * kTok * kRowK) = kr[k];
    }
    order_lds();
    if constexpr (kMore) {
      spread_slots(nxt);
      load_rows(kplane, kr);
      nxt = load_slots(i + 2);
    }
    __builtin_amdgcn_sched_barrier(0);

    OpT qop[kChunks * kQ];
#pragma unroll
    for (int ch = 0; ch < kChunks * kQ; ++ch) qop[ch] = q_s[ch][lane];
    // ---- scores: lane holds tokens 16 t + 4*grp + j of its column's head (the columns of a
    // head's parts summed: they then hold the same scores)
    f32x4 sc[kTiles];
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      const uint8_t* src = win + (t * 16 + row) * kRowK;
      // two chains of products
      f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
      auto score = [&](OpT k, int ch) {
        if constexpr (kQ == 2) {
          acc = score_mfma<kKind>(k, qop[ch * kQ], acc);
          acc2 = score_mfma<kKind>(k, qop[ch * kQ + kQ - 1], acc2);
        } else if (ch % 2 == 0) {
          acc = score_mfma<kKind>(k, qop[ch], acc);
        } else {
          acc2 = score_mfma<kKind>(k, qop[ch], acc2);
        }
      };
      if constexpr (kPairK) {
#pragma unroll
        for (int ch = 0; ch < kChunks; ch += 2) {
          const u32x4 w = *reinterpret_cast<const u32x4*>(src + ch * 32 + grp * 16);
          score(k_operand<kKind>(u32x2{w.x, w.y}), ch);
          score(k_operand<kKind>(u32x2{w.z, w.w}), ch + 1);
        }
      } else {
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) {
          const auto w = *reinterpret_cast<const typename Piece<kKind>::type*>(
              src + (ch * 32 + grp * kPer) * kElem);
          score(k_operand<kKind>(w), ch);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[j] += acc2[j];
        acc[j] += row_ror<8>(acc[j]);
        if (kHeads == 4) acc[j] += row_ror<4>(acc[j]);
      }
      sc[t] = acc;
    }
    const int left = nt - (wt0 + i * kStep);   // tokens of this round that exist
    if (left < kIT) {   // (uniform) the last round of the request's last split
#pragma unroll
      for (int t = 0; t < kTiles; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (16 * t + 4 * grp + j >= left) sc[t][j] = -INFINITY;
        }
    }

    // ---- softmax weights per head (the four lanes of a column share m)
    float mi = sc[0][0];
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) mi = fmaxf(mi, sc[t][j]);
    mi = fmaxf(m, lanes_reduce<16, true>(mi));
    if (__ballot(mi != m) != 0) {
      const float f = mi == m ? 1.f : __expf(m - mi);
      m = mi;
      l *= f;
#pragma unroll
      for (int dc = 0; dc < kDC; ++dc) o[dc] *= f;
    }
    const float msafe = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        sc[t][j] = __expf(sc[t][j] - msafe);
        l += sc[t][j];
      }

    // ---- O2 += V^T . P2^T, one 32-token step at a time through the window
#pragma unroll
    for (int kc = 0; kc < kKC; ++kc) {
      order_lds();
#pragma unroll
      for (int k = 0; k < kLdW; ++k) {
        const u32x4 w = vr[kc * kLdW + k];
        uint8_t* dst = win + (lane / kLanes + k * kTok) * kRowV + (lane % kLanes) * (32 / kElem);
        if constexpr (kKind == 2) {   // 16 fp8 values -> 16 bf16 values (32 bytes)
          *reinterpret_cast<u32x4*>(dst) = v_row16<kKind>(u32x2{w.x, w.y});
          *reinterpret_cast<u32x4*>(dst + 16) = v_row16<kKind>(u32x2{w.z, w.w});
        } else {
          *reinterpret_cast<u32x4*>(dst) = w;
        }
      }
      order_lds();
      if constexpr (kMore) {
        if (kc == kKC - 1) {   // V is in the window: the next round's loads
          load_rows(vplane, vr);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // P operand: column `row` (head row % 8, high or low part), tokens 4*grp..+3 of tile 2kc
      // then of tile 2kc+1
      ElemT pop[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int tile = 2 * kc + (j >> 2);
        if (tile >= kTiles) continue;
        const float p = sc[tile < kTiles ? tile : 0][j & 3];
        const ElemT hi = static_cast<ElemT>(p);
        pop[j] = low ? static_cast<ElemT>(p - static_cast<float>(hi)) : hi;
      }
      // V operand rows: lane 16*grp + rho supplies the row of token 4*grp + rho/4 of the first
      // tile (then of the second), elements 4*(rho%4)..+3 of the 16-element chunk
      const uint8_t* r1 = win + (4 * grp + row / 4) * kRowV + (row % 4) * 8;
#pragma unroll
      for (int dc = 0; dc < kDC; ++dc) {
        const i16x4 x1 = lds_read_tr16(r1 + dc * 32);
        if constexpr (kTiles > 1) {
          const i16x4 x2 = lds_read_tr16(r1 + 16 * kRowV + dc * 32);
          typedef short i16x8 __attribute__((ext_vector_type(8)));
          const i16x8 xv = {x1[0], x1[1], x1[2], x1[3], x2[0], x2[1], x2[2], x2[3]};
          const OpT pv = {pop[0], pop[1], pop[2], pop[3], pop[4], pop[5], pop[6], pop[7]};
          o[dc] = score_mfma<kKind>(__builtin_bit_cast(OpT, xv), pv, o[dc]);
        } else {
          typedef ElemT ElemT4 __attribute__((ext_vector_type(4)));
          const ElemT4 pv = {pop[0], pop[1], pop[2], pop[3]};
          o[dc] = value_mfma4<kKind>(x1, __builtin_bit_cast(i16x4, pv), o[dc]);
        }
      }
    }
  };
  for (int i = 0; i + 1 < rounds; ++i) round(i, std::true_type{});
  if (rounds > 0) round(rounds - 1, std::false_type{});

  // ---- merge the waves: [m, l] and O[head][d] per wave into LDS (element rows 4*grp + j of
  // chunk dc: four consecutive values per lane)
  l = lanes_reduce<16, false>(l);
  if (__ballot(bad) != 0 && rounds > 0) l = __builtin_nanf("");
#pragma unroll
  for (int dc = 0; dc < kDC; ++dc)
#pragma unroll
    for (int j = 0; j < 4; ++j) o[dc][j] += row_ror<8>(o[dc][j]);
  __syncthreads();  // the windows are reused for the merge
  float* mrg = reinterpret_cast<float*>(lds);        // [wave][head][kRec]
  if (row < G) {
    float* rec = mrg + (wave * 8 + row) * kRec;
    if (grp == 0) {
      rec[0] = m;
      rec[1] = l;
    }
#pragma unroll
    for (int dc = 0; dc < kDC; ++dc) {
      *reinterpret_cast<f32x4*>(rec + 4 + dc * 16 + 4 * grp) = o[dc];
    }
  }
  __syncthreads();
  for (int i = tid; i < G * (kD / 4); i += kThreads) {
    const int g = i / (kD / 4), d = i % (kD / 4) * 4;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, mrg[(w * 8 + g) * kRec]);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float* wr = mrg + (w * 8 + g) * kRec;
      const float f = wr[0] == -INFINITY ? 0.f : __expf(wr[0] - M);
      v += *reinterpret_cast<const f32x4*>(wr + 4 + d) * f;
      L += wr[1] * f;
    }
    if (a.splits == 1) {
      *reinterpret_cast<f32x4_out*>(a.out + (qh0 + g) * kD + d) = v * (1.f / L);
      continue;
    }
    float* rec = a.workspace + ((qh0 + g) * a.splits + split) * (kD + 2);
    rec[2 + d] = v.x;
    rec[3 + d] = v.y;
    rec[4 + d] = v.z;
    rec[5 + d] = v.w;
    if (d == 0) {
      rec[0] = M;
      rec[1] = L;
    }
  }
}

// Merge of the split partials of one (request, query head): M = max of the split maxima,
// weights w_s = exp(m_s - M), out = sum_s w_s acc_s / sum_s w_s l_s. Bound: latency (a merge
// reads ns records of kD + 2 floats). Every wave reads all the (m_s, l_s) pairs, 64 at a time, and
// so knows M, the weights and the divisor without a barrier; the records are shared out over the
// waves, a whole one per load, and the first kCombinePre of each wave are read before anything
// else is known. The waves' sums meet in LDS once. With all threads on every record, eight at a
// time, 282 records of 128 took 17 us, with 16 waves so 4.5.
constexpr int kCombinePre = 4;
constexpr int kCombineWaves = 4;
constexpr int kCombineWavesMany = 16;
constexpr int kCombineManySplits = 32;   // more splits: 16 waves

template <int kWaves, bool kShorten>
__global__ __launch_bounds__(64 * kWaves) void decode_combine_kernel(AttnArgs a) {
  constexpr int kMaxD = 256;
  __shared__ __attribute__((aligned(8))) float sum_s[kWaves][kMaxD];
  const int qh = blockIdx.x % a.num_q_heads;
  const int r = blockIdx.x / a.num_q_heads;
  if (r >= a.num_reqs) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int total = kShorten ? a.slot_indptr[a.num_reqs] - a.slot_indptr[0] : 0;
  const int s0 = a.slot_indptr[r];
  const int c = a.slot_count != nullptr ? a.slot_count[r] : a.slot_indptr[r + 1] - s0;
  const int st = kShorten ? decode_request_tokens(a.split, c, total) : a.split.tokens;
  const int D = a.head_dim;
  const int64_t rs = D + 2;  // record stride
  float* out = a.out + ((int64_t)r * a.num_q_heads + qh) * D;
  const int ns = min(static_cast<int>(((int64_t)c + st - 1) / st), a.splits);
  if (decode_fixed_output(a, s0, c) | (ns < 1)) {
    const float fill = c == 0 && s0 >= 0 ? 0.f : __builtin_nanf("");
    for (int d = tid; d < D; d += 64 * kWaves) out[d] = fill;
    return;
  }
  const float* rec0 = a.workspace + ((int64_t)r * a.num_q_heads + qh) * a.splits * rs;
  // A record's values in float pairs: pair lane and lane + 64
  const int p0 = lane * 2, p1 = 128 + lane * 2;
  auto pair = [&](int s, int p) {
    return s < ns && p < D ? *reinterpret_cast<const f32x2_in*>(rec0 + s * rs + 2 + p)
                           : f32x2{0.f, 0.f};
  };
  f32x2 x0[kCombinePre], x1[kCombinePre];
#pragma unroll
  for (int j = 0; j < kCombinePre; ++j) {
    x0[j] = pair(wave + j * kWaves, p0);
    x1[j] = pair(wave + j * kWaves, p1);
  }
  auto head_of = [&](int s) {   // (m_s, l_s)
    return s < ns ? *reinterpret_cast<const f32x2_in*>(rec0 + s * rs) : f32x2{-INFINITY, 0.f};
  };
  const f32x2 first = head_of(lane);
  float M = first.x;
  for (int s = lane + 64; s < ns; s += 64) M = fmaxf(M, rec0[s * rs]);
  M = lanes_reduce<1, true>(M);
  float L = 0.f;
  f32x2 v0 = {0.f, 0.f}, v1 = {0.f, 0.f};
  for (int base = 0; base < ns; base += 64) {
    const f32x2 ml = base == 0 ? first : head_of(base + lane);
    const float wt = base + lane < ns ? __expf(ml.x - M) : 0.f;
    L += ml.y * wt;
    auto weight = [&](int s) {   // of split base + s; zero past the last
      return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt), s));
    };
    int s = wave;
    if (base == 0) {
#pragma unroll
      for (int j = 0; j < kCombinePre; ++j) {
        const float w = weight(wave + j * kWaves);
        v0 += x0[j] * w;
        v1 += x1[j] * w;
      }
      s += kCombinePre * kWaves;
    }
    for (; s < 64 && base + s < ns; s += 4 * kWaves) {
      f32x2 y0[4], y1[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = s + j * kWaves < 64 ? base + s + j * kWaves : ns;
        y0[j] = pair(t, p0);
        y1[j] = pair(t, p1);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float w = s + j * kWaves < 64 ? weight(s + j * kWaves) : 0.f;
        v0 += y0[j] * w;
        v1 += y1[j] * w;
      }
    }
  }
  L = lanes_reduce<1, false>(L);
  static_assert(kCombinePre * kCombineWavesMany <= 64, "the first records have weights in a lane");
  if (p0 < D) *reinterpret_cast<f32x2*>(&sum_s[wave][p0]) = v0;
  if (p1 < D) *reinterpret_cast<f32x2*>(&sum_s[wave][p1]) = v1;
  __syncthreads();
  const float inv = 1.f / L;
  for (int d = tid; d < D; d += 64 * kWaves) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) v += sum_s[w][d];
    out[d] = v * inv;
  }
}

template <int kKind, int kD, bool kShorten>
auto split_kernel(bool g8) -> void (*)(AttnArgs) {
  if constexpr (kKind == 0) {
    return decode_split_kernel<kKind, kD, false, kShorten>;   // one kernel for all groups
  } else {
    return g8 ? decode_split_kernel<kKind, kD, true, kShorten>
              : decode_split_kernel<kKind, kD, false, kShorten>;
  }
}

template <int kKind, int kD>
auto pick_split(const AttnArgs& a) -> void (*)(AttnArgs) {
  const bool g8 = kKind != 0 && a.num_q_heads == 8 * a.num_kv_heads;
  return a.split.few > 0 ? split_kernel<kKind, kD, true>(g8) : split_kernel<kKind, kD, false>(g8);
}

template <int kKind>
hipError_t launch_split(const AttnArgs& a, hipStream_t stream) {
  const int64_t groups = decode_grid_groups((int64_t)a.num_reqs * decode_grid_splits(a.splits));
  const dim3 grid(static_cast<unsigned>(groups * a.num_kv_heads));
  void (*kernel)(AttnArgs) = nullptr;
  switch (a.head_dim) {
    case 32: kernel = pick_split<kKind, 32>(a); break;
    case 64: kernel = pick_split<kKind, 64>(a); break;
    case 128: kernel = pick_split<kKind, 128>(a); break;
    case 256: kernel = pick_split<kKind, 256>(a); break;
    default: return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(64 * kSplitWaves), 0, stream, a);
  return hipGetLastError();
}

template <bool kShorten>
hipError_t launch_combine(const AttnArgs& a, hipStream_t stream) {
  const bool many = a.splits > kCombineManySplits;
  const auto kernel = many ? decode_combine_kernel<kCombineWavesMany, kShorten>
                           : decode_combine_kernel<kCombineWaves, kShorten>;
  hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((int64_t)a.num_reqs * a.num_q_heads)),
                     dim3(64 * (many ? kCombineWavesMany : kCombineWaves)), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_append_slots(const AppendArgs& a, int64_t num_new, hipStream_t stream) {
  if (append_in_one_launch(a.num_reqs, num_new)) {
    hipLaunchKernelGGL(append_small_kernel, dim3(1), dim3(1024), 0, stream, a,
                       append_log2_threads(a.num_reqs, num_new));
    return hipGetLastError();
  }
  hipLaunchKernelGGL(append_status_kernel, dim3(1), dim3(64), 0, stream, a);
  if (a.num_reqs > 0) {
    hipLaunchKernelGGL(append_slots_kernel, dim3(a.num_reqs), dim3(256), 0, stream, a);
  }
  return hipGetLastError();
}

hipError_t launch_slot_mapping(const SlotMapArgs& a, hipStream_t stream) {
  if (a.num_reqs > 0 && a.num_reqs <= kSlotOffsetReqs) {
    hipLaunchKernelGGL(slot_map_kernel<true>, dim3(a.num_reqs), dim3(1024), 0, stream, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(slot_indptr_kernel, dim3(1), dim3(1024), 0, stream, a);
  if (a.num_reqs > 0) {
    hipLaunchKernelGGL(slot_map_kernel<false>, dim3(a.num_reqs), dim3(1024), 0, stream, a);
  }
  return hipGetLastError();
}

hipError_t launch_paged_decode(const AttnArgs& a, hipStream_t stream) {
  if (a.num_reqs <= 0) return hipSuccess;
  const int round = decode_round_tokens(a.head_dim, a.kv_kind == 2 ? 1 : 2);
  if (a.split.tokens <= 0 || a.split.tokens % round != 0) return hipErrorInvalidValue;
  hipError_t e;
  switch (a.kv_kind) {
    case 0: e = launch_split<0>(a, stream); break;
    case 1: e = launch_split<1>(a, stream); break;
    case 2: e = launch_split<2>(a, stream); break;
    default: return hipErrorInvalidValue;
  }
  // a single split has written the outputs
  if (a.splits == 1) return e;
  if (e != hipSuccess) return e;
  return a.split.few > 0 ? launch_combine<true>(a, stream) : launch_combine<false>(a, stream);
}

// Split partials of vtoken_paged_decode_noalloc: a library-held workspace for callers that
// cannot allocate. Each GPU that loads the library holds its own copy of the array until the
// process ends; its address on a device is looked up once, with that device current, and kept.
// The name below stands for the array only in device code: host code uses the address.
static __device__ __align__(256) float scratch[kDecodeScratchBytes / 4];

namespace {
constexpr int kMaxScratchDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxScratchDevices];
std::mutex g_scratch_mu;
}  // namespace

hipError_t decode_scratch(hipStream_t stream, float** out) {
  int cur = 0;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  int dev = cur;
  if (stream != nullptr) {
    e = hipStreamGetDevice(stream, &dev);
    if (e != hipSuccess) return e;
  }
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (p == nullptr) {
      // the lookup is per device and needs the stream's device current
      if (dev != cur && (e = hipSetDevice(dev)) != hipSuccess) return e;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (dev != cur) {
        const hipError_t back = hipSetDevice(cur);
        if (e == hipSuccess) e = back;
      }
      if (e != hipSuccess) return e;
      if (p == nullptr) return hipErrorInvalidSymbol;
      g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
  }
  *out = static_cast<float*>(p);
  return hipSuccess;
}

}  // namespace vtoken
