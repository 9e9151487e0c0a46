// The copies of the vToken repack for CDNA4 (gfx950, wave64): they consume a plan built by
// the metadata kernels (vtoken_kernels.hip) or the partial planner (vtoken_planner.hip).
//
//   repack_direct_kernel        the out-of-place gather-repack (Sec. 3.3, 3.3.4): every live
//                               K/V row of every admitted request into packed destination
//                               blocks, all layers, K and V, all KV heads in one launch
//   repack_inplace_rows_kernel  in-place compaction: one wave walks each (request, plane, column
//                               slice) chain in row order (the hazard rule below)
//   repack_inplace_kernel       its staging variants: one workgroup walks each (request, plane)
//                               chain in block order
//
// Both read the status word plan->counters[3] and do nothing when it is set, and check the
// plan's mode word plan->counters[4]. No MFMA, no arithmetic on the payload: byte movement.
#include <type_traits>

#include "vtoken_internal.h"

namespace vtoken {
namespace {

// A copy handed a plan built for the other mode copies nothing and reports it in the status
// word (first error wins), so the later calls of the pass do nothing either.
__device__ __forceinline__ void plan_mode_error(int32_t* counters) {
  if (blockIdx.x == 0 && threadIdx.x == 0) atomicCAS(&counters[3], 0, VTOKEN_ERR_PLAN_MODE);
}

// Number of set bits of a wave-wide ballot in the lanes below this one.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// ------------------------------------------------------------------------------------------
// Step 2: the gather-repack. Destination block g of a plane is one contiguous chunk of
// S*row_bytes bytes at block free_list[g], whose row j comes from the source slot
// src_plan[g*S + j]. A piece is (part of destination block g, plane), a part being one round of
// kU 16-byte units per thread (32 KiB at kU = 8): a chunk of several rounds (S = 32 or 48 at
// 2 KiB rows) is several pieces, and a chunk of at most 128 (64) units takes only two waves (one
// wave) of the workgroup, which then moves two (four) pieces side by side. Rows are
// head_dim-contiguous, so a wave's 64 lanes read and write 1 KiB of consecutive bytes per
// instruction (a whole 2 KiB row takes two).
//
// Bound: HBM, where a piece's loads are in flight early enough. A piece is a chain of dependent
// reads (counters, then destination block and plan entries, then rows) and then its stores, so
// a workgroup that takes one small piece and ends is bound by that chain: 404K pieces of 4 KiB
// (fp8, 80 layers, 2 heads x 64, S = 32) took 1.48 ms that way, 2.2 TB/s. Every workgroup
// therefore walks pieces with two of them in flight: the next piece's loads are issued before
// this one's stores, and the plan entries of the one after that before either (that call: 0.67
// ms, 4.9 TB/s; 1,600K pieces of 2 KiB, bf16, S = 8: 1.63 -> 1.31 ms; 205K of 8 KiB, fp8, S = 64:
// 766 -> 678 us; 32 KiB pieces are at the rate of a plain copy, up to 0.7% slower for the registers
// that the walk takes).
//
// Source slots of one destination block: with S <= 64, lane j of every wave holds
// src_plan[g*S + j] and rows are picked with a cross-lane shuffle; otherwise each unit reads
// its entry from memory. The copy is branch-free so the compiler can keep every load of a
// piece in flight (a conditional load or store would force a full wait on the vector
// memory counter): lanes of padding rows (src_plan -1, the tail of a request's last block)
// load the part's first row, which the workgroup reads anyway, and their stores go through a
// buffer resource spanning only the destination chunk with an out-of-range offset, which the
// hardware drops. Padding rows are a suffix of the block, so a part whose first row is
// padding is all padding: it reads slot 0's row and writes nothing.
// ------------------------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kBufferDword3 = 0x00020000u;  // raw buffer, 32-bit data format (gfx9)
constexpr uint32_t kDropOffset = 0x80000000u;    // beyond every chunk: store discarded

// Cache policies of the copy (CDNA4 cache-policy bits: sc0 = 1, nt = 2, sc1 = 16).
struct Policy {
  bool load_nt;
  int store_aux;
};
constexpr Policy kPolicies[] = {
    {true, 16},   // 0: default - non-temporal loads, sc1 stores (as 4)
    {false, 0},   // 1: plain loads, plain stores
    {true, 2},    // 2: non-temporal loads and stores
    {true, 0},    // 3: non-temporal loads, plain stores
    {true, 16},   // 4: non-temporal loads, sc1 stores (the default's kernels)
    {true, 17},   // 5: non-temporal loads, sc0 sc1 stores
    {true, 18},   // 6: non-temporal loads, sc1 nt stores
};
constexpr int kNumPolicies = sizeof(kPolicies) / sizeof(kPolicies[0]);

template <bool kNT>
__device__ __forceinline__ u32x4 load16(const u32x4* p) {
  if constexpr (kNT) {
    return __builtin_nontemporal_load(p);
  } else {
    return *p;
  }
}

// The destination pointer is the same for the whole workgroup; say so, so that the
// buffer resource lives in scalar registers.
__device__ __forceinline__ uint8_t* uniform_ptr(uint8_t* p) {
  const uint64_t x = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32));
  return reinterpret_cast<uint8_t*>((static_cast<uint64_t>(hi) << 32) | lo);
}

// Fewest workgroups the items are spread over (where there are as many items): 8 per CU.
constexpr int kMinCopyGrid = 2048;

// kU units per thread and piece; kW waves per piece (4: the whole workgroup); kWalk: a workgroup
// may take several items (else the grid has a workgroup for every item).
template <int kPolicy, bool kSmallS, int kU, int kW, bool kWalk>
__global__ __launch_bounds__(kCopyThreads) void repack_direct_kernel(CopyArgs a) {
  constexpr Policy pol = kPolicies[kPolicy];
  constexpr int kLanes = 64 * kW;                  // threads that share a piece
  constexpr int kSide = kCopyThreads / kLanes;     // pieces side by side in the workgroup
  constexpr int kRound = kLanes * kU;              // units of a piece
  static_assert(kU == 1 || kSide == 1, "several units per thread: the whole workgroup");
  if (a.counters[3] != 0) return;
  // plans of the full pass; plans of the partial pass too, but not with the freed list of
  // vtoken_repack_free (a partial pass releases its selected sources, not table tails)
  const int mode = a.counters[4];
  if (mode != kPlanOutOfPlace && (mode != kPlanPartial || a.num_reqs > 0)) {
    plan_mode_error(a.counters);
    return;
  }
  if (static_cast<int>(blockIdx.x) >= a.copy_grid) {   // the freed list (vtoken_repack_free)
    write_freed_blocks(static_cast<int>(blockIdx.x) - a.copy_grid, a.admitted, a.bt_indptr,
                       a.freed_indptr, a.block_ids, a.num_bt_entries, a.freed,
                       a.freed_capacity);
    return;
  }
  int used = a.counters[0];
  used = used < 0 ? 0 : (used > a.max_used ? a.max_used : used);
  if (used == 0) return;
  const int P = a.num_planes;
  const int chunk = a.chunk_units;
  const int parts = (chunk + kRound - 1) / kRound;
  // gp = g * parts + part: the parts of a destination block are consecutive in both orders
  const int used_parts = used * parts;
  const int64_t items = ((int64_t)used_parts * P + kSide - 1) / kSide;   // kSide pieces each
  // the workgroups that take items (the first ones; the others exit): with pieces below 16 KiB,
  // enough items each (where there are that many) that the chain of reads at a workgroup's start
  // is paid once per 32 KiB
  int grid = a.copy_grid;
  int64_t w = blockIdx.x;
  if (kWalk && kU < 4) {
    int64_t want = items * kU / 8;
    want = want > kMinCopyGrid ? want : kMinCopyGrid;
    if (want < grid) grid = static_cast<int>(want);
    if (w >= grid) return;
  }
  if (w >= items) return;
  const int S = a.block_size;
  const uint32_t chunk_bytes = static_cast<uint32_t>(chunk) * 16u;
  const int U = a.row_units;
  // j = u / U as a multiply-high with floor(2^32/U)+1: exact for u < 2^20 and
  // 2 <= U <= 2^12 (checked on the host)
  const uint32_t magic = a.row_magic;
  const bool unit_rows = U == 1;  // 16-byte rows: j = u (the constant would not fit)
  const int tid = static_cast<int>(threadIdx.x);
  const int lane = tid & 63;
  const int side = kSide == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / kLanes);
  const int sub = tid % kLanes;
  // lanes >= S read plan entry S-1 and never use it
  const int plan_lane = lane < S ? lane : S - 1;

  // Where a piece lies: (hi, lo) = (plane, gp) in the plane-major order, (gp, plane) in the
  // block-major one
  const bool plane_major = a.order == 1;
  const int inner = plane_major ? used_parts : P;
  struct Pos {
    int hi, lo;
  };
  const int64_t first = w * kSide + side;
  const int64_t stride = (int64_t)grid * kSide;
  Pos p;
  p.hi = static_cast<int>(first / inner);
  p.lo = static_cast<int>(first - (int64_t)p.hi * inner);
  const int step_hi = static_cast<int>(stride / inner);
  const int step_lo = static_cast<int>(stride - (int64_t)step_hi * inner);
  struct Piece {
    int g, part, plane;
    bool in;
  };
  // a position past the last piece (the end of the last item, the item after a workgroup's last)
  // reads the last piece and writes nothing
  auto locate = [&](const Pos& at) {
    Piece c;
    int gp = plane_major ? at.lo : at.hi;
    c.plane = plane_major ? at.hi : at.lo;
    c.in = static_cast<unsigned>(gp) < static_cast<unsigned>(used_parts) &&
           static_cast<unsigned>(c.plane) < static_cast<unsigned>(P);
    gp = c.in ? gp : used_parts - 1;
    c.plane = c.in ? c.plane : P - 1;
    c.g = parts == 1 ? gp : gp / parts;
    c.part = gp - c.g * parts;
    return c;
  };
  struct Meta {
    int dblk;   // destination block
    int pv;     // this lane's plan entry (S <= 64)
  };
  auto load_meta = [&](const Piece& c) {
    return Meta{a.free_list[c.g], kSmallS ? a.src_plan[(int64_t)c.g * S + plan_lane] : -1};
  };
  struct Flight {
    u32x4 buf[kU];
    uint32_t off[kU];
    uint8_t* dptr;
    uint32_t bytes;
  };
  auto load_piece = [&](const Piece& c, const Meta& m, Flight& f) {
    const int dblk = __builtin_amdgcn_readfirstlane(m.dblk);
    const bool dst_ok = c.in && static_cast<unsigned>(dblk) < static_cast<unsigned>(a.num_blocks);
    const uint8_t* pbase = a.kv + (int64_t)c.plane * a.plane_bytes;
    f.dptr = uniform_ptr(a.kv + (int64_t)c.plane * a.plane_bytes +
                         (dst_ok ? (int64_t)dblk * S * a.row_bytes : 0));
    f.bytes = dst_ok ? chunk_bytes : 0u;
    const int32_t* plan = a.src_plan + (int64_t)c.g * S;
    const int u0 = c.part * kRound;
    const int j0 = unit_rows ? u0 : static_cast<int>(__umulhi(static_cast<uint32_t>(u0), magic));
    int s0 = kSmallS ? __builtin_amdgcn_readlane(m.pv, j0)
                     : __builtin_amdgcn_readfirstlane(plan[j0]);
    // the part's first row is padding: so is the rest of the part
    if (static_cast<unsigned>(s0) >= static_cast<unsigned>(a.num_slots)) {
      if (!kWalk) return false;
      s0 = 0;
    }
    int src[kU];
    int col[kU];
#pragma unroll
    for (int v = 0; v < kU; ++v) {
      const int u = u0 + v * kLanes + sub;
      const int j = unit_rows ? u : static_cast<int>(__umulhi(static_cast<uint32_t>(u), magic));
      col[v] = u - j * U;
      int s;
      if (kSmallS) {
        s = __shfl(m.pv, j & 63, 64);
      } else {
        s = u < chunk ? plan[j] : -1;
      }
      const bool ok = (u < chunk) && static_cast<unsigned>(s) < static_cast<unsigned>(a.num_slots);
      src[v] = ok ? s : s0;
      f.off[v] = ok ? static_cast<uint32_t>(u) * 16u : kDropOffset;
    }
#pragma unroll
    for (int v = 0; v < kU; ++v) {
      f.buf[v] = load16<pol.load_nt>(
          reinterpret_cast<const u32x4*>(pbase + (int64_t)src[v] * a.row_bytes) + col[v]);
    }
    return true;
  };
  auto store_piece = [&](const Flight& f) {
    const __amdgpu_buffer_rsrc_t drsrc =
        __builtin_amdgcn_make_buffer_rsrc(f.dptr, 0, f.bytes, kBufferDword3);
#pragma unroll
    for (int v = 0; v < kU; ++v) {
      __builtin_amdgcn_raw_buffer_store_b128(f.buf[v], drsrc, f.off[v], 0, pol.store_aux);
    }
  };

  // Two pieces in flight. Vector-memory operations retire in order, so the plan entries of the
  // piece after next are read before the next one's loads: a wait for them then waits for no
  // row.
  Flight x, y;
  Piece c = locate(p);
  Meta m = load_meta(c);
  if (!kWalk || w + grid >= items) {
    if (load_piece(c, m, x)) store_piece(x);
    return;
  }
  auto issue = [&](Flight& f) {
    p.hi += step_hi;
    p.lo += step_lo;
    if (p.lo >= inner) {
      p.lo -= inner;
      ++p.hi;
    }
    const Piece cn = locate(p);
    const Meta mn = load_meta(cn);
    __builtin_amdgcn_sched_barrier(0);
    load_piece(c, m, f);
    __builtin_amdgcn_sched_barrier(0);
    c = cn;
    m = mn;
  };
  issue(x);
  for (;;) {
    issue(y);
    store_piece(x);
    if ((w += grid) + grid >= items) {
      store_piece(y);
      return;
    }
    issue(x);
    store_piece(y);
    if ((w += grid) + grid >= items) {
      store_piece(x);
      return;
    }
  }
}

// Default launch: the device-side count of items is not known on the host, only how many the
// buffers can hold, and every workgroup is dispatched even when the plan admits nothing, at
// about 4.5 per ns: an empty pass of 2^19 workgroups took 110 us, and a pass of 10K pieces with
// room for 230K (Llama-3-8B, 512 sources) 165 us for a copy of 110. So the grid has a workgroup
// for every item up to kFewItems, above that one for every eighth, up to a cap, and the kernel
// walks the rest. For 32 KiB pieces, caps of 2^17, 2^16, 2^15 and 2^14 cost a full Llama-3-8B
// copy (407K pieces, room for 1.3M) 0, 0.2%, 0.4% and 0.8% against one workgroup per piece; for
// 4 KiB ones (Llama-3-70B fp8 at TP 8, 1.7M pieces) 2^16 and 2^15 cost 0.3% and 0.7%. The copy of a full
// pass (vtoken_repack_free) takes the larger cap of its size, vtoken_repack, which also serves
// the partial passes that often move little or nothing, half of it (empty pass: 15 us at 2^16,
// 8 us at 2^15). Spreading the workgroups with items over the launch instead, so that the
// dispatch of the empty ones overlaps the copy, makes them slower: 49 destination blocks in a
// room for 28K took 37 us so, 5.5 us with the empty ones behind them.
constexpr int kFewItems = 1 << 13;
constexpr int kMaxCopyGrid = 1 << 17;        // pieces of 16 KiB and more
constexpr int kMaxCopyGridSmall = 1 << 16;   // smaller pieces

template <int kPolicy, int kU, int kW>
hipError_t launch_direct(const CopyArgs& a_in, int grid, hipStream_t stream) {
  // pieces: every (part of a destination block, plane) the buffers can hold; the kernel
  // indexes parts with 32-bit integers
  constexpr int kRound = 64 * kW * kU;
  constexpr int kSide = kCopyThreads / 64 / kW;
  CopyArgs a = a_in;
  const int64_t parts = (a.chunk_units + kRound - 1) / kRound;
  if ((int64_t)a.max_used * parts > 0x7fffffff) return hipErrorInvalidValue;
  const int64_t items = ((int64_t)a.max_used * parts * a.num_planes + kSide - 1) / kSide;
  // a launch with a workgroup for every item takes the kernel without the walk, whose second set
  // of rows costs registers (92 for 52 at kU = 8) and so workgroups in flight (3,712 pieces out
  // of the caches: 25 us, 28 with it); with small pieces only if all workgroups are resident at
  // once
  bool walk = kPolicy != 0;
  if (grid <= 0) {
    const int cap = (kU >= 4 ? kMaxCopyGrid : kMaxCopyGridSmall) / (a.num_reqs > 0 ? 1 : 2);
    const int64_t most = items / 8 > kFewItems ? items / 8 : kFewItems;
    grid = static_cast<int>(most < cap ? (items < most ? items : most) : cap);
    walk |= items > (kU >= 4 ? grid : kMinCopyGrid);
  } else {
    walk = true;
  }
  a.copy_grid = grid;
  // the freed list's workgroups follow the copy's
  const int64_t total = (int64_t)grid + a.num_reqs;
  if (total <= 0) return hipSuccess;
  const dim3 g(static_cast<unsigned>(total)), t(kCopyThreads);
  if constexpr (kPolicy == 0) {
    if (!walk) {
      const auto kernel = a.block_size <= 64 ? repack_direct_kernel<kPolicy, true, kU, kW, false>
                                             : repack_direct_kernel<kPolicy, false, kU, kW, false>;
      hipLaunchKernelGGL(kernel, g, t, 0, stream, a);
      return hipGetLastError();
    }
  }
  const auto kernel = a.block_size <= 64 ? repack_direct_kernel<kPolicy, true, kU, kW, true>
                                         : repack_direct_kernel<kPolicy, false, kU, kW, true>;
  hipLaunchKernelGGL(kernel, g, t, 0, stream, a);
  return hipGetLastError();
}

template <int kPolicy>
hipError_t launch_policy(const CopyArgs& a, int grid, hipStream_t stream) {
  // enough 16-byte units per thread to cover one chunk, at most 8; chunks below a workgroup's
  // 256 units go to the fewest waves that cover them
  const int per_thread = a.chunk_units / kCopyThreads;
  if (per_thread >= 8) return launch_direct<kPolicy, 8, 4>(a, grid, stream);
  if (per_thread >= 4) return launch_direct<kPolicy, 4, 4>(a, grid, stream);
  if (per_thread >= 2) return launch_direct<kPolicy, 2, 4>(a, grid, stream);
  if (a.chunk_units > 128) return launch_direct<kPolicy, 1, 4>(a, grid, stream);
  if (a.chunk_units > 64) return launch_direct<kPolicy, 1, 2>(a, grid, stream);
  return launch_direct<kPolicy, 1, 1>(a, grid, stream);
}

// ------------------------------------------------------------------------------------------
// In-place copy. Destination block b of request r is r's own b-th block, and the token of
// rank k sits at position p >= k, so the sources of destination block b lie in blocks >= b
// of the same request: block b may be written only after every read for blocks <= b.
// One workgroup walks one (request, plane) chain in block order: it stages the rows of
// block b that move (rows already in place are skipped) into LDS with direct 16-byte
// global->LDS loads, waits for them, synchronises, and writes them back from LDS. Reads for
// block b+1 touch blocks >= b+1 only, so they may start while block b is being written.
// With two LDS buffers one barrier per block suffices: a thread stages block b+1 into buffer
// (b+1)%2 only after passing barrier b, and every thread reaches barrier b only after its
// writes of block b-1, the last use of that buffer. With one buffer a second barrier after
// the writes protects it.
// ------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// kStage: 0 LDS double buffer, 1 LDS single buffer, 2 registers (no LDS; the barrier alone
// orders a block's reads before its writes, since every thread holds its own rows).
enum InplaceStage { kLdsDouble = 0, kLdsSingle = 1, kRegisters = 2 };

template <int kV, bool kSmallS, int kStage>
__global__ __launch_bounds__(kCopyThreads) void repack_inplace_kernel(InplaceArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t stage[];
  if (a.counters[3] != 0) return;
  if (a.counters[4] != kPlanInPlace) {
    plan_mode_error(a.counters);
    return;
  }
  const int P = a.num_planes;
  const int r = static_cast<int>(blockIdx.x / P);
  const int plane = static_cast<int>(blockIdx.x - (int64_t)r * P);
  if (r >= a.num_reqs || !a.admitted[r]) return;
  const int g0 = a.dst_indptr[r];
  const int need = a.dst_indptr[r + 1] - g0;
  const int nb0 = a.new_bt_indptr[r];
  const int S = a.block_size;
  if (g0 < 0 || need <= 0 || nb0 < 0 || (int64_t)(g0 + need) * S > a.src_plan_capacity ||
      (int64_t)nb0 + need > a.new_bt_capacity) {
    return;
  }
  const int U = a.row_units;
  const int chunk = a.chunk_units;
  const uint32_t magic = a.row_magic;
  const bool unit_rows = U == 1;
  const int tid = static_cast<int>(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint8_t* pbase = a.kv + (int64_t)plane * a.plane_bytes;
  const int chunk_bytes = chunk * 16;
  const int plan_lane = lane < S ? lane : S - 1;
  // the next block's table entry and plan entry are fetched one block ahead; the barrier
  // that ends each block has retired them by the time they are used
  int next_pv = kSmallS ? a.src_plan[(int64_t)g0 * S + plan_lane] : -1;
  int next_dblk = a.new_block_ids[nb0];
  int phase = 0;

  for (int b = 0; b < need; ++b) {
    const int dblk = __builtin_amdgcn_readfirstlane(next_dblk);
    const int pv = next_pv;
    const int bn = b + 1 < need ? b + 1 : b;
    next_dblk = a.new_block_ids[nb0 + bn];
    if (kSmallS) next_pv = a.src_plan[(int64_t)(g0 + bn) * S + plan_lane];
    if (static_cast<unsigned>(dblk) >= static_cast<unsigned>(a.num_blocks)) continue;
    const int dslot0 = dblk * S;
    if (kSmallS) {
      // every wave holds the same plan row, so this ballot is uniform over the workgroup:
      // a block whose rows are all in place needs no copy and no barrier
      const bool row_moves = lane < S && static_cast<unsigned>(pv) <
                             static_cast<unsigned>(a.num_slots) && pv != dslot0 + lane;
      if (__ballot(row_moves) == 0) continue;
    }
    const int32_t* plan = a.src_plan + (int64_t)(g0 + b) * S;
    // LDS buffer of this block (offsets into `stage`: the direct-load builtin needs an
    // address derived from the shared array itself)
    const int buf = kStage == kLdsDouble ? phase * chunk_bytes : 0;
    phase ^= 1;
    int src[kV];
    int col[kV];
    bool mv[kV];
#pragma unroll
    for (int v = 0; v < kV; ++v) {
      const int u = v * kCopyThreads + tid;
      const int j = unit_rows ? u : static_cast<int>(__umulhi(static_cast<uint32_t>(u), magic));
      col[v] = u - j * U;
      if (kSmallS) {
        src[v] = __shfl(pv, j & 63, 64);
      } else {
        src[v] = u < chunk ? plan[j] : -1;
      }
      // rows already in place (source slot == destination slot) are not copied
      mv[v] = (u < chunk) && static_cast<unsigned>(src[v]) < static_cast<unsigned>(a.num_slots) &&
              src[v] != dslot0 + j;
    }
    u32x4 regs[kStage == kRegisters ? kV : 1];
#pragma unroll
    for (int v = 0; v < kV; ++v) {
      if (mv[v]) {
        // addresses in locals of non-dependent type: a template-dependent argument makes
        // the host pass drop the kernel without a diagnostic
        const uint8_t* gsrc = pbase + (int64_t)src[v] * a.row_bytes + col[v] * 16;
        if (kStage == kRegisters) {
          regs[kStage == kRegisters ? v : 0] = load16<true>(reinterpret_cast<const u32x4*>(gsrc));
        } else {
          // lane i of a wave lands at the wave's base + 16 i
          const int loff = buf + (v * kCopyThreads + wave * 64) * 16;
          __builtin_amdgcn_global_load_lds(gsrc, (lds_ptr_t)(stage + loff), 16, 0, 0);
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kV; ++v) {
      if (mv[v]) {
        const int u = v * kCopyThreads + tid;
        const u32x4 val = kStage == kRegisters
                              ? regs[kStage == kRegisters ? v : 0]
                              : *reinterpret_cast<const u32x4*>(stage + buf + u * 16);
        *reinterpret_cast<u32x4*>(pbase + (int64_t)dslot0 * a.row_bytes + (int64_t)u * 16) = val;
      }
    }
    if (kStage == kLdsSingle) __syncthreads();
  }
}

// s_waitcnt immediate (gfx9 encoding): wait until at most n vector-memory operations are
// outstanding, without waiting on the other counters.
constexpr int vmcnt_imm(int n) {
  return (n & 0xF) | (((n >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8);
}

// Row walk of the in-place copy (the default): the chain of a (request, plane) is cut into
// column slices of at most 64 16-byte units, and every slice is a chain of its own, walked by
// one wave with no barrier inside. The workgroup stages the moves of some thousand destination
// rows in LDS at a time (source slot, destination slot; rows already in place, padding rows and
// rows of an invalid block are left out), and each of its waves walks them for its own slice in
// groups of kV instructions, the reads of the next group in flight while a group is written.
// Hazards: in logical order the positions q_k of the moves' destinations increase, and a row's
// source position p_k is larger than q_k. A move's destination can be the source of earlier
// moves only (p_j = q_k gives q_j < q_k), so a group is written once its own reads and those of
// the groups before have returned; and no later read lies at an earlier destination
// (p_j > q_j > q_k). Slices touch other bytes.
//
// Bound: HBM where there are thousands of chains, else what one compute unit gets out of rows
// far apart (16 KiB in flight per wave instead of 8 change nothing, the same waves on four times
// the compute units nearly double the rate). So a launch of few chains (launch_inplace_rows) has
// workgroups of one wave (kFew). Whole passes, before (one workgroup per (request,
// plane), a block at a time) and with workgroups of four waves and of one: fp8, 13 requests of
// 100K tokens, 1 layer x 8 heads x 128 (208 chains) 3,361, 1,631 and 951 us; bf16, 2 of 80K,
// 4 layers x 2 x 64 (32) 657, 355, 219; bf16, 6 of 72K, 32 x 2 x 64 (768) 4,627, 2,060, 1,935;
// Llama-3-8B, 4 of 2-8K (4,096) 368, 337, 394. Non-temporal stores gain where HBM bounds
// (Llama-3-70B at TP 8, 16 of 16-64K, H2O: 977 us with plain stores, 929 so) and lose with few
// chains (2 of 43K, 32 x 1 x 128, 256 chains: 158 us plain, 167 so) and in batches that the caches
// hold a good part of (kPlain).
constexpr int kLongestFirstMaxReqs = 256;
constexpr int kInplaceGroup = 8;                          // instructions of a group

template <int kV, int kWsh, int kMoveTile, bool kFew, bool kPlain>
__global__ __launch_bounds__(kFew ? 64 : kCopyThreads)
__attribute__((amdgpu_waves_per_eu(kFew ? 2 : 4)))
void repack_inplace_rows_kernel(InplaceArgs a, int slices, int64_t items) {
  constexpr int kThreads = kFew ? 64 : kCopyThreads;
  constexpr int kWaves = kThreads / 64;
  constexpr int kMoveRows = kThreads * kMoveTile;      // destination rows staged at a time,
                                                       // kMoveTile by a thread
  constexpr int kRows = 64 >> kWsh;                    // rows of an instruction
  constexpr int kGroup = kV * kRows;                   // rows of a group
  __shared__ int2 move_s[kMoveRows + 2 * kGroup];
  __shared__ int wave_tot[kWaves];
  __shared__ int need_s[kLongestFirstMaxReqs];
  __shared__ int r_s;
  if (a.counters[3] != 0) return;
  if (a.counters[4] != kPlanInPlace) {
    plan_mode_error(a.counters);
    return;
  }
  if (a.counters[1] == 0) return;   // nothing admitted
  const int S = a.block_size;
  const int tid = static_cast<int>(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t chains = (int64_t)a.num_planes * slices;
  const int64_t per_req = (chains + kWaves - 1) / kWaves;   // workgroups of a request
  const int64_t w = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (w >= items) {   // the freed list (vtoken_repack_inplace_free)
    if (w - items < a.free_reqs) {
      write_freed_blocks(static_cast<int>(w - items), a.admitted, a.bt_indptr, a.freed_indptr,
                         a.block_ids, a.num_bt_entries, a.freed, a.freed_capacity);
    }
    return;
  }
  // longest chains first: workgroups k * per_req .. take the request with the k-th longest
  // chain (ties by index), so the last workgroups to start are short ones and the tail of the
  // launch is short; for R <= 256 only (every workgroup ranks the requests)
  const int k = static_cast<int>(w / per_req);
  const int64_t chain = (w - (int64_t)k * per_req) * kWaves + wave;
  int r = k;
  if (a.num_reqs <= kLongestFirstMaxReqs) {
    for (int i = tid; i < a.num_reqs; i += kThreads) {
      need_s[i] = a.admitted[i] ? a.dst_indptr[i + 1] - a.dst_indptr[i] : 0;
    }
    __syncthreads();
    for (int i = tid; i < a.num_reqs; i += kThreads) {
      const int ni = need_s[i];
      int rank = 0;
      for (int j = 0; j < a.num_reqs; ++j) {
        const int nj = need_s[j];
        rank += (nj > ni) || (nj == ni && j < i);
      }
      if (rank == k) r_s = i;
    }
    __syncthreads();
    r = r_s;
  }
  if (!a.admitted[r]) return;
  const int g0 = a.dst_indptr[r];
  const int need = a.dst_indptr[r + 1] - g0;
  const int nb0 = a.new_bt_indptr[r];
  const int64_t rows = (int64_t)need * S;
  // (a table of 2^31 slots or more cannot be one of this pool)
  if (g0 < 0 || need <= 0 || nb0 < 0 || rows > INT32_MAX ||
      (int64_t)(g0 + (int64_t)need) * S > a.src_plan_capacity ||
      (int64_t)nb0 + need > a.new_bt_capacity) {
    return;
  }
  const int32_t* plan = a.src_plan + (int64_t)g0 * S;
  const int plane = static_cast<int>(chain / slices);
  const int unit = (static_cast<int>(chain - (int64_t)plane * slices) << kWsh) +
                   (lane & ((1 << kWsh) - 1));
  const bool mine = chain < chains && unit < a.row_units;   // this lane has bytes to move
  uint8_t* base = a.kv + (mine ? (int64_t)plane * a.plane_bytes + (int64_t)unit * 16 : 0);

  for (uint32_t c0 = 0; c0 < static_cast<uint32_t>(rows); c0 += kMoveRows) {
    // the moves of rows c0 .. c0 + kMoveRows, in order: wave w holds rows
    // w * 64 * kMoveTile + q * 64 + lane (positions clamped to the last row, all loads in
    // flight together)
    int src[kMoveTile], dst[kMoveTile], rank[kMoveTile];
    const uint32_t wrow = c0 + wave * (64 * kMoveTile) + lane;
#pragma unroll
    for (int q = 0; q < kMoveTile; ++q) {
      const int row = static_cast<int>(min(wrow + q * 64, static_cast<uint32_t>(rows) - 1));
      const int blk = row / S;
      src[q] = plan[row];
      dst[q] = a.new_block_ids[nb0 + blk];
      rank[q] = row - blk * S;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < kMoveTile; ++q) {
      const bool ok = wrow + q * 64 < static_cast<uint32_t>(rows) &&
                      static_cast<unsigned>(dst[q]) < static_cast<unsigned>(a.num_blocks) &&
                      static_cast<unsigned>(src[q]) < static_cast<unsigned>(a.num_slots);
      dst[q] = ok ? dst[q] * S + rank[q] : src[q];
    }
    int local = 0;
#pragma unroll
    for (int q = 0; q < kMoveTile; ++q) {
      const uint64_t m = __ballot(src[q] != dst[q]);
      rank[q] = local + lanes_below(m);
      local += __popcll(m);
    }
    if (lane == 0) wave_tot[wave] = local;
    __syncthreads();   // also: every wave has walked the previous moves
    int off = 0, total = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
      const int x = wave_tot[i];
      off += i < wave ? x : 0;
      total += x;
    }
#pragma unroll
    for (int q = 0; q < kMoveTile; ++q) {
      if (src[q] != dst[q]) move_s[off + rank[q]] = make_int2(src[q], dst[q]);
    }
    // the walk reads ahead of the last move: rows of slot 0, never written
    for (int i = total + tid; i < total + 2 * kGroup; i += kThreads) {
      move_s[i] = make_int2(0, 0);
    }
    __syncthreads();

    // a group: kV instructions of kRows rows
    typedef u32x4 Group[kV];
    const int2* mine_s = move_s + (lane >> kWsh);
    auto load = [&](int i, Group& g) {
      int from[kV];
#pragma unroll
      for (int v = 0; v < kV; ++v) from[v] = mine_s[i * kGroup + v * kRows].x;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < kV; ++v) {
        g[v] = load16<true>(
            reinterpret_cast<const u32x4*>(base + (int64_t)from[v] * a.row_bytes));
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto put = [&](int slot, u32x4 val) {
      u32x4* p = reinterpret_cast<u32x4*>(base + (int64_t)slot * a.row_bytes);
      if constexpr (kPlain) {
        *p = val;
      } else {
        __builtin_nontemporal_store(val, p);
      }
    };
    auto store = [&](int i, const Group& g) {
      int to[kV];
#pragma unroll
      for (int v = 0; v < kV; ++v) to[v] = mine_s[i * kGroup + v * kRows].y;
#pragma unroll
      for (int v = 0; v < kV; ++v) {
        put(to[v], g[v]);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    const int rows_left = total - (lane >> kWsh);
    auto store_last = [&](int i, const Group& g) {   // the moves that exist
#pragma unroll
      for (int v = 0; v < kV; ++v) {
        const int to = mine_s[i * kGroup + v * kRows].y;
        if (i * kGroup + v * kRows < rows_left) put(to, g[v]);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto wait = [](auto n) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(decltype(n)::value));
      __builtin_amdgcn_sched_barrier(0);
    };
    using None = std::integral_constant<int, 0>;
    using One = std::integral_constant<int, kV>;
    using Two = std::integral_constant<int, 2 * kV>;
    // Vector-memory operations retire in order, stores included: a group's reads have
    // returned when at most the operations issued after them are left, which are the kV
    // stores of the group before (from the second group on) and the kV reads of the next.
    if (total > 0 && mine) {
      const int last = (total - 1) / kGroup;
      Group x, y;
      load(0, x);
      load(1, y);
      wait(One{});
      if (last == 0) {
        store_last(0, x);
      } else {
        store(0, x);
        int i = 1;   // y holds group i
        for (; i + 2 <= last; i += 2) {
          load(i + 1, x);
          wait(Two{});
          store(i, y);
          load(i + 2, y);
          wait(Two{});
          store(i + 1, x);
        }
        load(i + 1, x);
        wait(Two{});
        store_last(i, y);
        wait(None{});
        store_last(i + 1, x);
      }
    }
  }
}

// Chains of the row walk: slices of 64 units (1 KiB), or the whole row where it is shorter, cut
// down to 128-byte slices until the launch has kInplaceChains chains (bf16, 9 requests of
// 5-23K, 32 layers x 8 x 128: 1,416 us with 4,608 chains, 1,398 with 18,432; bf16, 38 of 8K, 16
// layers: 1,590 and 1,561). Rows that are no whole number of 128-byte lines lose more to lines
// shared by slices: those are cut, down to 64 bytes, for kInplaceOddChains only, and a wave of
// theirs takes groups of 16 instructions instead (pairs of a request and a plane; us, cut for 512
// chains / for 160 / the copy before the row walk: 480-byte rows, 448 pairs of 5,000 tokens
// 215 / 147 / 155, 160 of 800 18.1 / 11.1 / 11.8; 960-byte rows, 448 of 5,000 411 / 323 / 311, 168
// of 5,000 124 / 132 / 143, 16 of 30,000 118 / 118 / 523, and 148 cut for 128 chains).
constexpr int64_t kInplaceChains = 16384;
constexpr int64_t kInplaceOddChains = 160;
// Launches of fewer chains have workgroups of one wave (above); with at most kInplaceNarrow slices
// to a row, where the waves of a workgroup share little, up to kInplaceFewNarrow: bf16, 32 layers
// x 2 x 64, 10 requests of 3,000 (1,280 chains) 73.9 us with workgroups of four, 55.4 so (55.6
// before the row walk); fp8, 80 x 1 x 128, 8 of 4,000 (1,280) 113 and 81 (104). With 4 slices of a
// row four waves are better (fp8, 32 x 4 x 128, 8 of 500, 2,048 chains: 26.3 and 29.2).
constexpr int64_t kInplaceFewChains = 1024;
constexpr int64_t kInplaceFewNarrow = 4096;
constexpr int kInplaceNarrow = 2;
// Plain stores, besides launches of fewer than kInplaceFewChains chains, where the caches hold a
// good part of the batch's blocks: bf16, 32 x 8 x 128, 8 of 500 (262 MB) 98 us with non-temporal
// ones, 80 so (78 before the row walk); 16 x 8 x 128, 4 of 4,000 (1.05 GB) 142 and 117 (169). Larger
// batches (Llama-3-8B, 4 of 2-8K, 2.7 GB: 327 and 337; 70B at TP 8: 909 and 939), those of more
// chains than kInplaceChains and the smallest (Llama-3-8B, 1 of 600: 17.0 and 17.4) keep
// non-temporal ones.
constexpr int64_t kInplacePlainMin = 96LL << 20;
constexpr int64_t kInplacePlainMax = 1LL << 30;
// One-wave workgroups stage 1,024 rows at a time, 512 where the requests average fewer tokens than
// kInplaceShort (8 of 300, 1 layer x 2 x 64: 7.6 and 6.6 us; 2 of 30,000, 4 x 5 x 96: 118 and 124).
constexpr int64_t kInplaceShort = 1024;
constexpr int64_t kMaxInplaceGrid = 1 << 22;

template <int kMoveTile, bool kFew, bool kPlain>
auto inplace_rows_kernel(int wsh) -> void (*)(InplaceArgs, int, int64_t) {
  constexpr int kOddGroup = kFew ? 2 * kInplaceGroup : kInplaceGroup;
  switch (wsh) {
    case 0: return repack_inplace_rows_kernel<kInplaceGroup, 0, kMoveTile, kFew, kPlain>;
    case 1: return repack_inplace_rows_kernel<kInplaceGroup, 1, kMoveTile, kFew, kPlain>;
    case 2: return repack_inplace_rows_kernel<kInplaceGroup, 2, kMoveTile, kFew, kPlain>;
    case 3: return repack_inplace_rows_kernel<kInplaceGroup, 3, kMoveTile, kFew, kPlain>;
    case 4: return repack_inplace_rows_kernel<kInplaceGroup, 4, kMoveTile, kFew, kPlain>;
    case 5: return repack_inplace_rows_kernel<kOddGroup, 5, kMoveTile, kFew, kPlain>;
    default: return repack_inplace_rows_kernel<kOddGroup, 6, kMoveTile, kFew, kPlain>;
  }
}

hipError_t launch_inplace_rows(const InplaceArgs& a, int64_t num_tokens, int64_t held_bytes,
                               hipStream_t stream) {
  int wsh = 0;   // log2 units of a slice
  while (wsh < 6 && (1 << wsh) < a.row_units) ++wsh;
  const int64_t pairs = (int64_t)a.num_reqs * a.num_planes;
  auto slices_of = [&](int sh) { return (a.row_units + (1 << sh) - 1) >> sh; };
  const bool lines = a.row_units % 8 == 0;
  const int64_t most = lines ? kInplaceChains : kInplaceOddChains;
  while (wsh > (lines ? 3 : 2) && pairs * slices_of(wsh) < most) --wsh;
  const int slices = slices_of(wsh);
  const int64_t chains = pairs * slices;
  const bool few = chains < (slices <= kInplaceNarrow ? kInplaceFewNarrow : kInplaceFewChains);
  const bool small = held_bytes < kInplacePlainMax;
  const int threads = few ? 64 : kCopyThreads;
  const int waves = threads / 64;
  const int64_t items = a.num_reqs * (((int64_t)a.num_planes * slices + waves - 1) / waves);
  // (a launch dimension holds 2^32 threads)
  const int64_t total = items + a.free_reqs;
  const int64_t gx = total < kMaxInplaceGrid ? total : kMaxInplaceGrid;
  const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>((total + gx - 1) / gx));
  void (*kernel)(InplaceArgs, int, int64_t) = nullptr;
  if (few) {
    const bool is_short = num_tokens < a.num_reqs * kInplaceShort;
    kernel = chains >= kInplaceFewChains && !small ? inplace_rows_kernel<16, true, false>(wsh)
             : is_short                            ? inplace_rows_kernel<8, true, true>(wsh)
                                                   : inplace_rows_kernel<16, true, true>(wsh);
  } else {
    const bool plain = small && held_bytes >= kInplacePlainMin && chains < kInplaceChains;
    kernel = plain ? inplace_rows_kernel<8, false, true>(wsh)
                   : inplace_rows_kernel<8, false, false>(wsh);
  }
  hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, stream, a, slices, items);
  return hipGetLastError();
}

template <int kV, bool kSmallS>
hipError_t launch_inplace_v(const InplaceArgs& a, int variant, hipStream_t stream) {
  const int64_t grid = (int64_t)a.num_reqs * a.num_planes;
  const int64_t chunk_bytes = (int64_t)a.chunk_units * 16;
  // LDS double buffer when asked and two fit
  int stage = variant == 1 ? kLdsDouble : variant == 2 ? kLdsSingle : kRegisters;
  if (stage == kLdsDouble && chunk_bytes * 2 > kMaxInplaceChunkBytes) stage = kLdsSingle;
  const dim3 g(static_cast<unsigned>(grid));
  const dim3 t(kCopyThreads);
  if (stage == kLdsDouble) {
    auto kernel = repack_inplace_kernel<kV, kSmallS, kLdsDouble>;
    hipLaunchKernelGGL(kernel, g, t, static_cast<size_t>(2 * chunk_bytes), stream, a);
  } else if (stage == kLdsSingle) {
    auto kernel = repack_inplace_kernel<kV, kSmallS, kLdsSingle>;
    hipLaunchKernelGGL(kernel, g, t, static_cast<size_t>(chunk_bytes), stream, a);
  } else {
    auto kernel = repack_inplace_kernel<kV, kSmallS, kRegisters>;
    hipLaunchKernelGGL(kernel, g, t, 0, stream, a);
  }
  return hipGetLastError();
}

template <bool kSmallS>
hipError_t launch_inplace_s(const InplaceArgs& a, int variant, hipStream_t stream) {
  // units per thread that cover one chunk (at most 16: chunks are at most 64 KiB)
  const int per_thread = (a.chunk_units + kCopyThreads - 1) / kCopyThreads;
  if (per_thread <= 1) return launch_inplace_v<1, kSmallS>(a, variant, stream);
  if (per_thread <= 2) return launch_inplace_v<2, kSmallS>(a, variant, stream);
  if (per_thread <= 4) return launch_inplace_v<4, kSmallS>(a, variant, stream);
  if (per_thread <= 8) return launch_inplace_v<8, kSmallS>(a, variant, stream);
  return launch_inplace_v<16, kSmallS>(a, variant, stream);
}

}  // namespace

hipError_t launch_repack_inplace(const InplaceArgs& a, int variant, int64_t num_tokens,
                                 int64_t held_bytes, hipStream_t stream) {
  if (variant < 0 || variant > 4) return hipErrorInvalidValue;
  if ((int64_t)a.num_reqs * a.num_planes <= 0) return hipSuccess;
  if ((int64_t)a.chunk_units * 16 > kMaxInplaceChunkBytes) return hipErrorInvalidValue;
  if (variant == 0 || variant == 4) {
    return launch_inplace_rows(a, num_tokens, held_bytes, stream);
  }
  return a.block_size <= 64 ? launch_inplace_s<true>(a, variant, stream)
                            : launch_inplace_s<false>(a, variant, stream);
}

hipError_t launch_repack(const CopyArgs& a_in, int variant, int grid, int order,
                         hipStream_t stream) {
  if (order < 0 || order > 2) return hipErrorInvalidValue;
  CopyArgs a = a_in;
  a.order = order;
  switch (variant) {
    case 0:
    case 4: return launch_policy<0>(a, grid, stream);
    case 1: return launch_policy<1>(a, grid, stream);
    case 2: return launch_policy<2>(a, grid, stream);
    case 3: return launch_policy<3>(a, grid, stream);
    case 5: return launch_policy<5>(a, grid, stream);
    case 6: return launch_policy<6>(a, grid, stream);
    default: return hipErrorInvalidValue;
  }
}

int num_repack_variants() { return kNumPolicies; }

}  // namespace vtoken
