#pragma once
// Receiver-conditioned importance of sender positions in two passes over K
// (gfx950 / CDNA4): device code and launch templates, included by
// the per-dtype translation units score_*.hip.
//
// For one unit (sender s, layer l, KV head g) the query rows are the m tokens
// of every query head in the group: R = G*m rows of D values, and the logits
// are S = scale * Q K^T (R x T).  Importance is the column sum of the row
// softmax, I[t] = sum_r exp(S[r,t] - lse_r).  Because every row carries its
// own normaliser, no column sum can start before the whole row is known, so
// K is traversed twice, chunk by chunk (an LDS tile to 8192 positions):
//
//   P1 (stats):   per row and chunk, the max and sum of exp2 in log2 units.
//   P2 (reduce):  fold the unit's chunk statistics in fixed chunk order into
//                 lse2 (log2 of the row normaliser), recompute the logits and
//                 add exp2(x - lse2) over the rows.
//
// A call runs P1 and P2 either as two plain launches of one item per workgroup
// (pass_kernel), or as one persistent kernel with a queue, whichever choose_form
// (score.hip) estimates to be shorter.  The latter:
//
// Scheduling.  Every P1 and P2 item of every unit sits in one ordered list
// (WorkList in kernels.h); resident workgroups take items from a device
// queue (one atomic counter) until the list is exhausted.  A P2 item waits
// until all P1 items of its unit (and row group) are counted in, on a
// per-unit counter.  The list places P2 of unit u lag steps after its P1, so
// by the time a P2 item is taken its statistics are normally complete;
// the whole stage is one
// launch with no idle boundaries between unit groups.  Dependencies always
// precede their dependants in the list and are taken only by running
// workgroups, so the waits always end whatever the number of resident
// workgroups; each wait is still bounded (PersistArgs::spin_limit) and a
// timeout raises an error flag, poisons the item's output (NaN importance)
// and stops every later wait.
//
// The chunk statistics that P1 workgroups hand to P2 workgroups inside the
// launch are written with device-scope atomic stores and read with
// device-scope atomic loads; each writer waits for its stores to complete
// before the workgroup counts itself in with a relaxed atomic add, so no
// cache-wide release/acquire maintenance is needed.
//
// Score items run the contraction on bf16 (fp32 for fp32 inputs) MFMA with
// fp32 accumulation.  Each wavefront holds 16*RB query rows in registers
// (RB = 1 to 8, so that a unit's rows fill one, two or four waves
// with few padding rows; make_score_plan);
// K tiles of 32 to 128 positions (tile_tokens) are staged through an LDS ring (XOR-swizzled 16-byte
// chunks so B-fragment reads are bank-conflict free) and shared by every
// wave of the workgroup.  The contraction index is permuted consistently for
// Q and K: each lane group (of 16 lanes, or of 32 for 32 x 32 blocks) holds a
// contiguous share of each row, so every fragment is one 16-byte load.  The scale is applied in
// fp32 to the accumulator (folded with log2 e), never to bf16 operands.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "kernels.h"

namespace cb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int ESZ, int D, int TT>
struct Geo {
  static constexpr int kRowBytes = D * ESZ;
  static constexpr int kChunks = kRowBytes / 16;          // 16-byte chunks per K row
  static constexpr int kTileBytes = TT * kRowBytes;
  static constexpr int kTileChunks = TT * kChunks;
};

// K-tile slot layout: thread `tid` of an NT-thread workgroup owns slots
// j*NT + tid, j < per, of a tile of rows of `chunks` 16-byte chunks stored
// swizzled.  When NT chunks span a multiple of the swizzle's period in whole
// rows, slot j of a thread is its slot 0 moved down j*NT/chunks rows: one
// per-lane offset serves every load of a tile.  Checked exhaustively at
// compile time where it is used.
struct SlotGeo {
  int row, off;
};
// Chunk c of row r is stored at c ^ swz_of(r): 16 consecutive rows then hold
// a chunk in 16 different 16-byte bank groups of the 256-byte bank row (two
// rows of 128 bytes share one).
__host__ __device__ constexpr int swz_of(int row, int chunks) {
  return chunks >= 16 ? row & 15 : (row >> 1) & 7;
}
constexpr SlotGeo slot_geo(int slot, int chunks, int row_bytes) {
  const int r = slot / chunks;
  const int c = (slot % chunks) ^ swz_of(r, chunks);
  return SlotGeo{r, r * row_bytes + c * 16};
}
constexpr bool slots_linear(int nt, int per, int chunks, int row_bytes) {
  if (nt % chunks != 0) return false;
  for (int tid = 0; tid < nt; ++tid)
    for (int j = 0; j < per; ++j) {
      const SlotGeo g0 = slot_geo(tid, chunks, row_bytes);
      const SlotGeo gj = slot_geo(j * nt + tid, chunks, row_bytes);
      if (gj.row != g0.row + j * (nt / chunks) || gj.off != g0.off + j * (nt / chunks) * row_bytes)
        return false;
    }
  return true;
}

__device__ __forceinline__ int swz_offset(int row, int c, int row_bytes) {
  return row * row_bytes + ((c ^ swz_of(row, row_bytes / 16)) << 4);
}

// MFMA output blocks of M x M.  The lanes form 64/M groups; lane (lg, lc) of
// an operand holds row lc's contiguous share lg of the contraction, and of the
// output column lc, rows row(i, lg) in its registers i.
template <int M> struct Mma;
template <> struct Mma<16> {
  typedef f32x4 Acc;
  static constexpr int kRegs = 4, kGroups = 4;
  __device__ static constexpr int row(int i, int lg) { return 4 * lg + i; }
};
template <> struct Mma<32> {
  typedef f32x16 Acc;
  static constexpr int kRegs = 16, kGroups = 2;
  __device__ static constexpr int row(int i, int lg) { return (i & 3) + 8 * (i >> 2) + 4 * lg; }
};

// One 16-byte segment of the contraction for an output block.
template <int ESZ, int M>
__device__ __forceinline__ void mfma_seg(const u32x4& a, const u32x4& b,
                                         typename Mma<M>::Acc& acc) {
  if constexpr (ESZ == 2 && M == 32) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                  __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  } else if constexpr (ESZ == 2) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                  __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  } else {
    static_assert(M == 16, "fp32 blocks are 16 x 16");
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]),
                                                 acc, 0, 0, 0);
  }
}

// Waves a SIMD should hold: two, so that one wave's MFMAs overlap another's
// exp/VALU epilogue; one for fp32 and for the queue's one-wave bf16 workgroups
// (four a compute unit; see tile_tokens).
constexpr int waves_per_simd(int esz, int waves, bool queue) {
  return esz == 2 && !(waves == 1 && queue) ? 2 : 1;
}

// LDS ring depth: as many K tiles as fit the workgroup's share of the
// 160 KiB LDS at two waves per SIMD (8/W workgroups per CU; at one for the
// queue's one-wave bf16 workgroups), between 2 and 4, after the other LDS arrays.
template <int ESZ, int D, int W, bool POS, int RB, bool QUEUE>
struct Stages {
  static constexpr int kTT = tile_tokens(ESZ, D, W, QUEUE);
  static constexpr int kTile = kTT * D * ESZ;
  static constexpr int kOther = W * ((POS ? 5 : 2) * kTT + 16 * RB) * 4;
  static constexpr int kShare = waves_per_simd(ESZ, W, QUEUE) == 1 && ESZ == 2 ? 4 : 8;
  static constexpr int kBudget = 160 * 1024 * W / kShare - kOther;
  static constexpr int kFit = kBudget / kTile;
  static constexpr int value = kFit < 2 ? 2 : (kFit > 4 ? 4 : kFit);
};

// s_waitcnt immediates (gfx9 encoding: vmcnt[3:0] and [15:14], expcnt[6:4],
// lgkmcnt[11:8]); counters not named are left at their maximum.
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
constexpr int kWaitVmcnt0 = vmcnt_imm(0);
constexpr int lgkmcnt_imm(int n) { return 15 | (3 << 14) | (7 << 4) | ((n & 15) << 8); }

// Wait until at most `later` tiles of kPer loads each are still in flight.
template <int kPer, int kStages>
__device__ __forceinline__ void wait_tiles(int later) {
  static_assert((kStages - 2) * kPer <= 63, "vmcnt holds at most 63");
  if (kStages >= 4 && later >= 2) {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kPer));
  } else if (kStages >= 3 && later >= 1) {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(kPer));
  } else {
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  }
}

// One 16-byte-per-lane load from global memory straight into LDS: lane i
// writes lds_base + 16*i.  Issued through asm so that the compiler's own
// wait-count insertion, which cannot tell the ring's buffers apart and would
// drain every in-flight tile before each LDS read, stays out of the ring;
// completion is tracked explicitly with wait_tiles() below.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is set on purpose
__device__ __forceinline__ void load_lds16(const void* gptr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(gptr), "s"(lds_base)
               : "memory", "m0");
}
// The same load with a uniform 64-bit base in scalar registers and a 32-bit
// per-lane byte offset.
__device__ __forceinline__ void load_lds16_s(const void* sbase, uint32_t voff, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(sbase), "s"(lds_base)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// A pointer every lane holds the same value of, moved to scalar registers.
__device__ __forceinline__ const unsigned char* uniform_ptr(const unsigned char* p) {
  const uint64_t v = reinterpret_cast<uintptr_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const unsigned char*>(((uint64_t)hi << 32) | lo);
}

// LDS offset of a shared-memory pointer (the low 32 bits of its flat address).
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)reinterpret_cast<uintptr_t>(p);
}

// Workgroup barrier that waits for this wave's LDS operations only; loads in
// flight to later ring stages stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(0));
  __builtin_amdgcn_s_barrier();
}

// Sum of v over the four lanes l, l^16, l^32, l^48 (the four lane groups
// that hold the same token column), returned in every one of them.  Two
// cross-row swaps instead of LDS-routed shuffles; the addition order is the
// same in every lane, so all four hold bitwise-equal sums.
__device__ __forceinline__ float sum_lane_groups(float v) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v),
                                                  false, false);
  const float s = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s),
                                                  false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// Sum / maximum over the two lane halves l, l^32, in both.
__device__ __forceinline__ float sum_lane_halves(float v) {
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v),
                                                  false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
__device__ __forceinline__ float max_lane_halves(float v) {
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v),
                                                  false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// Maximum over the four lane groups (see sum_lane_groups).
__device__ __forceinline__ float max_lane_groups(float v) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v),
                                                  false, false);
  const float s = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s),
                                                  false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// The sums of a and of b over the four lane groups: a's in lane groups 0 and
// 2, b's in 1 and 3.  Two swaps for both values, added in sum_lane_groups'
// order.
__device__ __forceinline__ float sum_two_lane_groups(float a, float b) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b),
                                                  false, false);
  const float s = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s),
                                                  false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// v plus its value in the paired lane group (lanes l and l^16), the same in
// both lanes.
__device__ __forceinline__ float sum_lane_pairs(float v) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v),
                                                  false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Position pooling inside a 16-lane DPP row (the 16 positions of a column
// block): row_shl:n gives lane c the value of lane c+n, row_shr:n that of
// lane c-n; lanes whose source falls outside the row read 0.  Values are
// the bit patterns of non-negative floats, whose unsigned order is their
// numeric order, so 0 is the identity of the maximum.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_z(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int N> __device__ __forceinline__ uint32_t row_shl(uint32_t v) { return dpp_z<0x100 + N>(v); }
template <int N> __device__ __forceinline__ uint32_t row_shr(uint32_t v) { return dpp_z<0x110 + N>(v); }
__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
// max over positions c-3..c (left part) and c..c+3 (right part) of a block
__device__ __forceinline__ uint32_t left4(uint32_t x) {
  const uint32_t l2 = umax(x, row_shr<1>(x));
  return umax(l2, row_shr<2>(l2));
}
__device__ __forceinline__ uint32_t right4(uint32_t x) {
  const uint32_t r2 = umax(x, row_shl<1>(x));
  return umax(r2, row_shl<2>(r2));
}

// Scheduler hint: interleave one MFMA with `valu` VALU instructions, n times.
template <int N, int VALU>
__device__ __forceinline__ void interleave_mfma_valu() {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // MFMA
    __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);   // VALU
  }
}

// Combine two (max, sum) pairs of exp2 partial sums.
__device__ __forceinline__ void lse_merge(float& m, float& z, float mo, float zo) {
  const float mn = fmaxf(m, mo);
  const float ms = (mn == -INFINITY) ? 0.f : mn;
  z = z * __builtin_amdgcn_exp2f(m - ms) + zo * __builtin_amdgcn_exp2f(mo - ms);
  m = mn;
}


// ---- device-scope hand-over between workgroups ---------------------------

__device__ __forceinline__ uint32_t poll_u32(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void count_in(uint32_t* p) {
  __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_f2(float2* p, float2 v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p),
                     __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 get_f2(const float2* p) {
  return __builtin_bit_cast(
      float2, __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p),
                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// Every wave waits for its own stores to complete, then the workgroup
// meets; after this one thread may publish the workgroup's results.
__device__ __forceinline__ void stores_done_barrier() {
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  __syncthreads();
}

// Thread 0 waits until *p >= target; all threads get the outcome.  Gives up
// after `limit` polls (raising the error flag; a limit of 0 gives up at
// once) or as soon as another wait has raised it.
__device__ __forceinline__ bool wait_for(const uint32_t* p, uint32_t target, uint32_t* err,
                                         uint32_t limit, int* s_ok) {
  if (threadIdx.x == 0) {
    int ok = 1;
    uint32_t n = 0;
    while (n < limit && poll_u32(p) < target) {
      ++n;
      if ((n & 63u) == 0 && poll_u32(err) != 0u) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
    if (ok && n >= limit) {
      __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ok = 0;
    }
    *s_ok = ok;
  }
  __syncthreads();
  return *s_ok != 0;
}

__device__ __forceinline__ int64_t take_item(uint32_t* sync) {
  return (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(sync), 1ull);
}

struct Item {
  int stage, unit, sub;
};

__device__ __forceinline__ Item decode(const WorkList& wl, int64_t item) {
  int i = 0;
  while (i + 1 < wl.nseg && item >= wl.seg_item[i + 1]) ++i;
  const int64_t rem = item - wl.seg_item[i];
  const int step = wl.seg_step[i] + (int)(rem / wl.seg_size[i]);
  int r = (int)(rem % wl.seg_size[i]);
  for (int s = 0; s < wl.nstages; ++s) {
    const int u = step - wl.lag[s];
    if (u >= 0 && u < wl.units) {
      if (r < wl.per_unit[s]) return Item{s, u, r};
      r -= wl.per_unit[s];
    }
  }
  return Item{-1, 0, 0};
}

// LDS of one workgroup, shared by every item type.
template <int ESZ, int D, int W, bool POS, int RB, bool QUEUE>
struct Shared {
  static constexpr int kTT = tile_tokens(ESZ, D, W, QUEUE);
  using Gm = Geo<ESZ, D, kTT>;
  static constexpr int kStages = Stages<ESZ, D, W, POS, RB, QUEUE>::value;
  unsigned char ktile[kStages][Gm::kTileBytes] __attribute__((aligned(16)));
  float imp[2][W][kTT];          // P2 per-wave column sums of a tile (by tile parity)
  // Position variant: per-wave correction numerators of a tile, by tile
  // index mod 3 (a tile's last block is finalised during the next tile).
  float num[POS ? 3 : 1][W][POS ? kTT : 1];
  float lse[W * 16 * RB];        // P2 row normalisers
  int64_t next;                  // next item, taken by thread 0 during this one
  int ok;                        // outcome of the last dependency wait
};

// ---- score items: P1 and P2 of one (unit, row group, chunk) ---------------
// Query row rho of a unit (0 <= rho < Rp): whether it is a real row, and its
// index h*m + r among the unit's G*m query rows.  The importance path uses
// rho = h*m + r; the position variant rho = r*Gp + h (padding heads h >= G).
template <bool POS>
__device__ __forceinline__ bool real_row(const PersistArgs& a, int rho, int* qrow) {
  if (!POS) {
    *qrow = rho;
    return rho < a.R;
  }
  const int r = rho >> a.gshift, h = rho & (a.Gp - 1);
  *qrow = h * a.m + r;
  return r < a.m && h < a.G;
}

// 32 x 32 blocks wherever a wave's bf16 rows allow, 16 x 16 for odd counts of
// 16 rows, fp32, and the pooling pass (whose windows run across the 16 lanes
// of a DPP row).  A 32 x 32 block takes half the MFMA issue slots and half the
// operand reads per logit.
template <int ESZ, int RB, bool POOL>
struct BlockDim {
  static constexpr int value = (ESZ == 2 && RB % 2 == 0 && !POOL) ? 32 : 16;
};

// Power mode and head grouping (log2 of the padded heads) of the pooling pass.
template <int MODE, int GSHIFT>
struct Power {
  static constexpr int kMode = MODE, kGshift = GSHIFT;
};

template <int ESZ, int D, int W, int RB, bool PASS2, bool POS, bool QUEUE>
__device__ __forceinline__ void score_item(const PersistArgs& a, int u, int sub,
                                           Shared<ESZ, D, W, POS, RB, QUEUE>& sh) {
  constexpr int M = BlockDim<ESZ, RB, PASS2 && POS>::value;
  using Mm = Mma<M>;
  using Acc = typename Mm::Acc;
  constexpr int kRegs = Mm::kRegs;
  constexpr int NB = 16 * RB / M;                // M-row blocks per wave
  constexpr int kRPW = 16 * RB;                  // query rows per wave
  constexpr int kGroupRows = kRowsPerGroup;
  constexpr int TT = tile_tokens(ESZ, D, W, QUEUE);   // positions per K tile
  using Gm = Geo<ESZ, D, TT>;
  constexpr int kBlocks = TT / M;                // M-position column blocks per tile
  constexpr int kSegs = Gm::kChunks / Mm::kGroups;   // 16-byte chunks per lane group
  constexpr int kPer = Gm::kTileChunks / (W * 64);   // 16-byte loads per thread per tile
  constexpr int kStages = Stages<ESZ, D, W, POS, RB, QUEUE>::value;  // K tiles resident/in flight in LDS
  static_assert(Gm::kTileChunks % (W * 64) == 0, "tile must split evenly");
  auto& ktile = sh.ktile;
  float* lse_lds = sh.lse;

  const int chunk = sub % a.chunks;
  const int rg = sub / a.chunks;
  const int layer = (u / a.Hkv) % a.L;
  const int kvh = u % a.Hkv;
  uint32_t* done1 = a.sync + kSyncHeader;

  // The thread index passes through an empty asm so that the per-lane
  // addresses derived from it are recomputed for each item instead of being
  // hoisted out of the persistent loop, where they would outlive the register
  // budget and be spilled to scratch memory.
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int lg = lane / M;          // lane group: which share of the contraction
  const int lc = lane & (M - 1);    // lane column: position within a block / query row

  const unsigned char* qb = static_cast<const unsigned char*>(a.q) +
                            (size_t)((layer * a.Hq + kvh * a.G) * a.m) * Gm::kRowBytes;
  const unsigned char* kb = static_cast<const unsigned char*>(a.k) +
                            (size_t)u * (size_t)a.T * Gm::kRowBytes;

  const int wrow0 = rg * kGroupRows + wave * kRPW;
  const bool wave_active = wrow0 < a.Rp;

  const int64_t t_begin = (int64_t)chunk * a.chunk_tokens;
  const int64_t t_end = (t_begin + a.chunk_tokens < a.T) ? t_begin + a.chunk_tokens : a.T;
  const int ntiles = (int)((t_end - t_begin + TT - 1) / TT);

  int64_t next = 0;

  // ---- K tiles: direct global -> LDS loads into a kStages-deep ring -----------
  // Lane `tid` owns LDS slot j*(W*64) + tid of a tile and fetches the K chunk
  // whose swizzled position that slot is: every load instruction of a wave
  // writes one contiguous KiB of LDS, and the swizzle stays the one the
  // B-fragment reads expect.  Rows past the chunk end are clamped to its last
  // row (always valid memory); their logits are masked or never stored.
  int koff[kPer];   // byte offset of this lane's chunk inside a tile's rows
  int krow[kPer];   // its row inside the tile
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int slot = j * (W * 64) + tid;
    krow[j] = slot / Gm::kChunks;
    const int c = (slot % Gm::kChunks) ^ swz_of(krow[j], Gm::kChunks);
    koff[j] = krow[j] * Gm::kRowBytes + c * 16;
  }
  const uint32_t lds_ring = lds_offset(&ktile[0][0]) + wave * 64 * 16;
  // Where every load of a tile shares the lane's offset, the full-tile loads
  // take a scalar base per load and one offset register (no per-load
  // 64-bit addresses to keep live across the tile loop).
  constexpr bool kLinear = slots_linear(W * 64, kPer, Gm::kChunks, Gm::kRowBytes);
  constexpr int kJBytes = (W * 64 / Gm::kChunks) * Gm::kRowBytes;
  auto issue_tile = [&](int tile, int buf) {
    const int64_t tbase = t_begin + (int64_t)tile * TT;
    const unsigned char* src = kb + (size_t)tbase * Gm::kRowBytes;
    const uint32_t dst = lds_ring + buf * Gm::kTileBytes;
    if (kLinear && tbase + TT <= t_end) {
      const unsigned char* ssrc = uniform_ptr(src);
#pragma unroll
      for (int j = 0; j < kPer; ++j)
        load_lds16_s(ssrc + (size_t)j * kJBytes, (uint32_t)koff[0],
                     __builtin_amdgcn_readfirstlane(dst + j * (W * 64) * 16));
    } else if (tbase + TT <= t_end) {
#pragma unroll
      for (int j = 0; j < kPer; ++j)
        load_lds16(src + koff[j], __builtin_amdgcn_readfirstlane(dst + j * (W * 64) * 16));
    } else {
      const int last = (int)(t_end - 1 - tbase);
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int over = krow[j] > last ? (krow[j] - last) * Gm::kRowBytes : 0;
        load_lds16(src + koff[j] - over, __builtin_amdgcn_readfirstlane(dst + j * (W * 64) * 16));
      }
    }
  };

  // The first K tiles are requested before anything else of the item, and the
  // query rows next, so that their latencies overlap each other's and the
  // wait for the statistics; not in the pooling pass, whose halo blocks would
  // wait for the tiles (864 units x 3001 positions: 502 against 515 us).
  constexpr bool kFirst = !(PASS2 && POS);
  if (kFirst)
    for (int j = 0; j < kStages - 1 && j < ntiles; ++j) issue_tile(j, j);

  // ---- query rows of this wave, resident in registers -----------------------
  u32x4 qf[NB][kSegs];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    int qrow;
    const bool real = real_row<POS>(a, wrow0 + nb * M + lc, &qrow);
    const u32x4* src = reinterpret_cast<const u32x4*>(qb + (size_t)(real ? qrow : 0) *
                                                              Gm::kRowBytes) + lg * kSegs;
#pragma unroll
    for (int sg = 0; sg < kSegs; ++sg) qf[nb][sg] = real ? src[sg] : u32x4{0, 0, 0, 0};
  }

  // ---- P2 prologue: wait for the row group's statistics, fold them --------
  // One thread per row (some take two with five row blocks per wave); chunks
  // are folded in ascending order, eight loads in flight, so every workgroup
  // of the unit derives bitwise-identical lse2.
  if (PASS2) {
    bool ok;
    if constexpr (!QUEUE) {
      // The statistics were written by an earlier launch: nothing to wait
      // for, and only a wait limit of 0 gives up.
      ok = a.spin_limit != 0u;
      if (tid == 0) {
        sh.ok = ok;
        if (!ok)
          __hip_atomic_fetch_or(a.sync + kSyncError, 1u, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
      }
    } else {
      ok = wait_for(done1 + (size_t)u * a.row_groups + rg, (uint32_t)a.chunks,
                    a.sync + kSyncError, a.spin_limit, &sh.ok);
    }
    const int row_base = rg * kGroupRows;
    for (int lr = tid; lr < W * kRPW; lr += W * 64) {
      const int row = row_base + lr;
      int qrow;
      if (!real_row<POS>(a, row, &qrow)) {   // padding: no weight
        lse_lds[lr] = INFINITY;
        continue;
      }
      if (!QUEUE && a.lse2) {
        const float l2 = ok ? a.lse2[(size_t)u * a.Rp + row] : __builtin_nanf("");
        lse_lds[lr] = l2;
        if (chunk == 0 && a.row_lse)
          a.row_lse[(size_t)u * a.R + qrow] = l2 * 0.69314718055994530942f;
        continue;
      }
      const float2* p = a.partial + (size_t)u * a.chunks * a.Rp + row;
      float m = -INFINITY, z = 0.f;
      int c = 0;
      for (; c + 8 <= a.chunks; c += 8) {
        float2 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = get_f2(p + (size_t)(c + j) * a.Rp);
#pragma unroll
        for (int j = 0; j < 8; ++j) lse_merge(m, z, v[j].x, v[j].y);
      }
      for (; c < a.chunks; ++c) {
        const float2 v = get_f2(p + (size_t)c * a.Rp);
        lse_merge(m, z, v.x, v.y);
      }
      const float l2 = ok ? m + __log2f(z) : __builtin_nanf("");
      lse_lds[lr] = l2;
      if (chunk == 0 && a.row_lse)
        a.row_lse[(size_t)u * a.R + qrow] = l2 * 0.69314718055994530942f;
    }
  }
  // ---- per-lane row state -----------------------------------------------------
  // P1 multiplies K by Q, so that a lane holds one query row a block (column
  // wrow0 + nb*M + lc) against kRegs positions and its (max, sum) are two
  // registers; P2 multiplies Q by K, so that a lane holds one position against
  // rows wrow0 + nb*M + row(i, lg) and adds them in registers.
  float st_m[NB], st_z[NB];       // pass 1: reference max / sum (log2 units)
  // pass 2: lse2 of the row (+inf for padding rows), in registers where they
  // fit beside the query rows, else read from LDS for each block
  constexpr bool kL2Regs = NB <= 2 || M == 16;
  float row_l2[kL2Regs ? NB : 1][kRegs];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    st_m[nb] = -INFINITY;
    st_z[nb] = 0.f;
  }

  // P2 output of one tile: the sum over waves (in wave order) of the
  // per-wave column sums; NaN if the statistics never arrived.
  float* imp_out = (a.row_groups > 1)
                       ? a.imp_partial + ((size_t)rg * a.units + u) * (size_t)a.T
                       : a.importance + (size_t)u * (size_t)a.T;
  auto flush_tile = [&](int tile, int t) {
    const int64_t pos = t_begin + (int64_t)tile * TT + t;
    if (pos >= t_end) return;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) s += sh.imp[tile & 1][w][t];
    imp_out[pos] = sh.ok ? s : __builtin_nanf("");
  };

  // Position variant: the correction numerator of a tile, combined over the
  // waves that hold rows of this row group, in wave order.
  float* num_out = nullptr;
  int num_waves = 0;
  if (POS) {
    num_out = (a.row_groups > 1)
                  ? a.numer_partial + ((size_t)rg * a.units + u) * (size_t)a.T
                  : a.numer + (size_t)u * (size_t)a.T;
    const int rows = a.Rp - rg * kGroupRows;
    num_waves = (rows + kRPW - 1) / kRPW;
    if (num_waves > W) num_waves = W;
  }
  auto flush_num = [&](int tile) {
    for (int t = tid; t < TT; t += W * 64) {
      const int64_t pos = t_begin + (int64_t)tile * TT + t;
      if (pos >= t_end) continue;
      float s = 0.f;
      for (int w = 0; w < num_waves; ++w) {
        const float v = sh.num[POS ? tile % 3 : 0][w][POS ? t : 0];
        s = a.pow_mode == kPowMax ? fmaxf(s, v) : s + v;
      }
      num_out[pos] = sh.ok ? s : __builtin_nanf("");
    }
  };

  // Logits of one column block (positions tb*M .. tb*M + M-1 of the tile)
  // against G row blocks from nb0 on.
  auto load_block = [&](const unsigned char* kt, int tb, u32x4 (&kf)[kSegs]) {
    const int row = tb * M + lc;
#pragma unroll
    for (int sg = 0; sg < kSegs; ++sg)
      kf[sg] = *reinterpret_cast<const u32x4*>(
          kt + swz_offset(row, lg * kSegs + sg, Gm::kRowBytes));
  };
  constexpr int G = M == 16 ? NB : 1;   // row blocks per pipeline step
  auto mfma_block = [&](const u32x4 (&kf)[kSegs], int nb0, Acc (&acc)[G]) {
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = Acc{};
#pragma unroll
    for (int sg = 0; sg < kSegs; ++sg)
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if constexpr (PASS2)
          mfma_seg<ESZ, M>(qf[nb0 + g][sg], kf[sg], acc[g]);
        else
          mfma_seg<ESZ, M>(kf[sg], qf[nb0 + g][sg], acc[g]);
      }
  };
  // Software pipeline over the (column block, row blocks) steps of a tile: the
  // MFMAs of a step are issued ahead of the exp epilogue of the one before, and
  // the scheduler is asked to interleave them, so the matrix unit and the
  // VALU work at the same time within one wave; a column block's LDS reads
  // are issued a step earlier still.  (No hints for fp32, which waits on
  // its 32-cycle MFMAs: they gain nothing and cost minutes of compile time.)
  constexpr int kSteps = kBlocks * (NB / G);
  constexpr int kKf = NB * M <= 64 ? 2 : 1;   // K fragment sets (registers)
  constexpr int kMfmaPerStep = G * kSegs * (ESZ == 4 ? 4 : 1);
  // `valu`: VALU instructions of the epilogue per accumulator register that the
  // hints spread over the MFMAs.
  auto pipelined_tile = [&](const unsigned char* kt, auto valu, auto&& epilogue) {
    constexpr int kValuPerMfma = decltype(valu)::value * G * kRegs / kMfmaPerStep;
    u32x4 kf[kKf][kSegs];
    Acc acc[2][G];
    load_block(kt, 0, kf[0]);
    mfma_block(kf[0], 0, acc[0]);
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
      const int tb = st / (NB / G), nb = st % (NB / G) * G;
      if (st + 1 < kSteps) {
        const int tn = (st + 1) / (NB / G), nn = (st + 1) % (NB / G) * G;
        if (kKf == 1 ? nn == 0 : (nb == 0 && tb + 1 < kBlocks))
          load_block(kt, kKf == 1 ? tn : tb + 1, kf[kKf == 1 ? 0 : (tb + 1) & 1]);
        mfma_block(kf[kKf == 1 ? 0 : tn & 1], nn, acc[(st + 1) & 1]);
      }
      epilogue(tb, nb, acc[st & 1]);
      if (ESZ == 2 && st + 1 < kSteps) interleave_mfma_valu<kMfmaPerStep, kValuPerMfma>();
    }
  };

  // ---- position variant: pooled per-token weights ---------------------------
  // The query rows are ordered rho = r*Gp + h, so lane (lg, lc) of row block
  // rb holds, summed over its four rows i, the weight of query token
  // (wrow0 + rb*16 + 4*lg) >> gshift over Gp = 4 heads, or over half of
  // Gp = 8 heads (the paired lane group holds the other half), at position
  // lc of the column block.  Pool_7 over positions runs across the 16 lanes
  // of a DPP row and into the neighbouring blocks: a block is finalised when
  // the next block is known, from its left4/right4 parts; the blocks beyond
  // the chunk's two ends are computed separately from K in global memory.
  uint32_t r4p[RB] = {};   // right4 of the previous block
  uint32_t pc[RB] = {};    // previous block pooled, except the next block's part
  // Numerator terms of a finalised block, summed over this lane's tokens (or
  // their maximum at p = inf).
  auto numer = [&](auto power, const uint32_t(&fin)[RB]) {
    constexpr int kMode = decltype(power)::kMode;
    float acc = 0.f;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      if constexpr (kMode == kPowSquare) {
        const float t = __uint_as_float(fin[rb]) * a.sq_scale;
        acc = __builtin_fmaf(t, t, acc);
      } else if constexpr (kMode == kPowGeneral) {
        acc += __builtin_amdgcn_exp2f(__builtin_fmaf(
            a.pow_p, __builtin_amdgcn_logf(__uint_as_float(fin[rb])), a.pow_kappa));
      } else {
        acc = fmaxf(acc, __uint_as_float(fin[rb]));
      }
    }
    // (with eight heads the paired lane group holds the same tokens)
    return decltype(power)::kGshift == 3 && kMode != kPowMax && (lg & 1) ? 0.f : acc;
  };
  // A wave's column sums of one block and numerators of the block before it
  // go to LDS in one store of all lanes, lane groups 0 and 2 the sum, 1 and 3
  // the numerator, with no branch in the tile: each lane's address for block 0
  // (whose predecessor is the last block of the tile before; before the first
  // tile that lands in a slot that is written again before it is read) and,
  // 16 positions a block further, for the others.
  auto numer_slot = [&](int tile, int tb) {
    return &sh.num[POS ? (tile + 3) % 3 : 0][wave][POS ? tb * 16 + lc : 0];
  };
  // Pool a new block x: finalise the previous one into fin, keep this one's
  // parts.
  auto pool_block = [&](const uint32_t (&x)[RB], uint32_t (&fin)[RB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const uint32_t l4 = left4(x[rb]), r4 = right4(x[rb]);
      fin[rb] = umax(pc[rb], row_shr<13>(l4));   // lanes 13..15 see this block's 0..2
      pc[rb] = umax(umax(l4, r4), row_shl<13>(r4p[rb]));   // lanes 0..2 see 13..15 before
      r4p[rb] = r4;
    }
  };
  // Column sums and pooled numerators of a tile.
  auto pos_tile = [&](auto power, const unsigned char* kt, int tile, auto&& pipeline) {
    constexpr int kMode = decltype(power)::kMode;
    float* const imp0 = &sh.imp[tile & 1][wave][lc];
    float* const first = (lg & 1) ? numer_slot(tile - 1, kBlocks - 1) : imp0;
    float* const rest = (lg & 1) ? numer_slot(tile, 0) : imp0 + 16;
    // Six instructions a register for the general power, whose epilogue is twice
    // the importance's, three otherwise.  Whole calls of the shapes below: p = 2
    // takes 0.962 of its time with branches at three and 0.974 at six; p = 3 420
    // us at three and 400 at six.
    constexpr int kValu = kMode == kPowGeneral ? 6 : 3;
    pipeline(kt, std::integral_constant<int, kValu>{}, [&](int tb, int, const Acc(&acc)[G]) {
      float part[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        float p;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[rb][i], a.c2, -row_l2[rb][i]));
          p = i == 0 ? e : p + e;
        }
        part[rb] = p;
      }
      float psum = part[0];
      if constexpr (RB >= 2) psum += part[1];
      if constexpr (RB >= 4)
        psum += part[2] + part[3];
      else if constexpr (RB == 3)
        psum += part[2];
      // (Columns past the sequence end repeat its last row, which every
      // window that reaches them holds already.)
      uint32_t x[RB], fin[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        x[rb] = __float_as_uint(decltype(power)::kGshift == 3 ? sum_lane_pairs(part[rb])
                                                              : part[rb]);
      pool_block(x, fin);
      const float nu = numer(power, fin);
      float v;
      if constexpr (kMode == kPowMax) {
        const float all = sum_lane_groups(psum), top = max_lane_groups(nu);
        v = (lg & 1) ? top : all;
      } else {
        v = sum_two_lane_groups(psum, nu);
      }
      (tb == 0 ? first : rest + (tb - 1) * 16)[0] = v;
    });
  };
  // Weights of the block of 16 positions from tstart, from K in global memory
  // (positions outside [0, T) weigh 0).
  auto halo_bits = [&](int64_t tstart, uint32_t(&x)[RB]) {
    const int64_t row = tstart + lc;
    const bool okr = row >= 0 && row < a.T;
    const u32x4* src = reinterpret_cast<const u32x4*>(kb + (size_t)(okr ? row : 0) *
                                                              Gm::kRowBytes) + lg * kSegs;
    u32x4 kf[kSegs];
#pragma unroll
    for (int sg = 0; sg < kSegs; ++sg) kf[sg] = src[sg];
    Acc acc[G];
    mfma_block(kf, 0, acc);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float p = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        p += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[rb][i], a.c2, -row_l2[rb][i]));
      if (a.gshift == 3) p = sum_lane_pairs(p);
      x[rb] = okr ? __float_as_uint(p) : 0u;
    }
  };
  // lse2 of the lane's rows of block nb: padding rows hold +inf in LDS
  auto load_row_l2 = [&](int nb, float (&l2)[kRegs]) {
#pragma unroll
    for (int i = 0; i < kRegs; ++i) l2[i] = lse_lds[wave * kRPW + nb * M + Mm::row(i, lg)];
  };
  if (PASS2 && POS) {
    __syncthreads();   // every row's lse2 is in LDS
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) load_row_l2(nb, row_l2[nb]);
    if (wave_active && t_begin > 0) {
      uint32_t hx[RB];
      halo_bits(t_begin - 16, hx);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) r4p[rb] = right4(hx[rb]);
    }
  }

  // Everything issued so far (first tiles, query rows, chunk statistics, the
  // left halo) must land before the ring's vmcnt bookkeeping starts.
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  if (!kFirst)
    for (int j = 0; j < kStages - 1 && j < ntiles; ++j) issue_tile(j, j);

  for (int tile = 0; tile < ntiles; ++tile) {
    const int buf = tile % kStages;
    // Wait for this tile's loads (later tiles may stay in flight), then make
    // every wave's loads visible; the barrier also retires the previous
    // tile's buffer, which the next issue overwrites.
    const int later = ((ntiles - 1 < tile + kStages - 2) ? ntiles - 1 : tile + kStages - 2) - tile;
    wait_tiles<kPer, kStages>(later);
    lds_barrier();
    if (tile + kStages - 1 < ntiles) issue_tile(tile + kStages - 1, (tile + kStages - 1) % kStages);
    // The next item is taken while the last tile is computed; no ring load
    // is in flight any more, so its latency hides behind the tile.
    if (QUEUE && tile == ntiles - 1 && tid == 0) next = take_item(a.sync);
    if (PASS2 && !POS && kL2Regs && tile == 0) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) load_row_l2(nb, row_l2[nb]);
    }
    // P2: the previous tile's per-wave column sums are complete; they are
    // added in wave order and the tile's importance is stored.  Numerators
    // trail by one more tile (a tile's last block is finalised in the next).
    if (PASS2 && tile > 0)
      for (int t = tid; t < TT; t += W * 64) flush_tile(tile - 1, t);
    if (PASS2 && POS && tile > 1) flush_num(tile - 2);
    if (!wave_active) {
      if (PASS2 && lg == 0)
#pragma unroll
        for (int tb = 0; tb < kBlocks; ++tb) sh.imp[tile & 1][wave][tb * M + lc] = 0.f;
      continue;
    }
    const unsigned char* kt = &ktile[buf][0];
    const int64_t tok0 = t_begin + (int64_t)tile * TT;
    const bool full = tok0 + TT <= t_end;

    if (PASS2) {
      // importance contribution: column sums of exp2(x - lse2) over the rows
      if constexpr (POS) {
        // The choice between the modes stands outside the tile, whose blocks
        // are then one straight line: a branch in each cut it into pieces
        // and left no MFMA to run beside the pooling, which bounds this pass by
        // its VALU instructions (whole calls, 36 x 8 units x 8192 with p = 2: 465
        // -> 443 us; 3 x 288 units x 3001 with p = 3 and eight heads: 466 -> 418).
        if (a.pow_mode == kPowMax) {
          a.gshift == 3 ? pos_tile(Power<kPowMax, 3>{}, kt, tile, pipelined_tile)
                        : pos_tile(Power<kPowMax, 2>{}, kt, tile, pipelined_tile);
        } else if (a.pow_mode == kPowSquare) {
          a.gshift == 3 ? pos_tile(Power<kPowSquare, 3>{}, kt, tile, pipelined_tile)
                        : pos_tile(Power<kPowSquare, 2>{}, kt, tile, pipelined_tile);
        } else {
          a.gshift == 3 ? pos_tile(Power<kPowGeneral, 3>{}, kt, tile, pipelined_tile)
                        : pos_tile(Power<kPowGeneral, 2>{}, kt, tile, pipelined_tile);
        }
      } else {
        float* dst = &sh.imp[tile & 1][wave][lc];
        float psum = 0.f;   // of the column block's row blocks so far
        pipelined_tile(kt, std::integral_constant<int, 3>{}, [&](int tb, int nb0, const Acc(&acc)[G]) {
          float part[G];
#pragma unroll
          for (int g = 0; g < G; ++g) {
            float l2[kRegs];
            if constexpr (!kL2Regs) load_row_l2(nb0 + g, l2);
            // four partial sums of every fourth register
            float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < kRegs; ++i) {
              const float r = kL2Regs ? row_l2[kL2Regs ? nb0 + g : 0][i] : l2[i];
              const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[g][i], a.c2, -r));
              if (kRegs == 4)
                p[0] = i == 0 ? e : p[0] + e;
              else
                p[i & 3] = i < 4 ? e : p[i & 3] + e;
            }
            part[g] = kRegs == 4 ? p[0] : (p[0] + p[1]) + (p[2] + p[3]);
          }
          float s = part[0];
#pragma unroll
          for (int g = 1; g < G; ++g) s += part[g];
          psum = nb0 == 0 ? s : psum + s;
          if (nb0 + G == NB) {
            const float sum = M == 16 ? sum_lane_groups(psum) : sum_lane_halves(psum);
            if (lg == 0) dst[tb * M] = sum;
          }
        });
      }
      continue;
    }

    // P1.  Each row's reference maximum m is the maximum over the first M
    // positions of the chunk, the same in the lanes that hold the row; the
    // fast path then adds exp2(x - m) with m fixed.  A row whose sum passes
    // 2^100 (a logit far above m) sends the whole tile to the slow path; below
    // that, fp32 keeps full relative
    // precision, so a fixed m costs nothing.
    const int left = (int)(t_end - tok0 < TT ? t_end - tok0 : TT) - Mm::row(0, lg);
    auto in_chunk = [&](int tb, int i) { return tb * M + Mm::row(i, 0) < left; };
    if (tile == 0) {
      u32x4 kf[kSegs];
      load_block(kt, 0, kf);
#pragma unroll
      for (int nb = 0; nb < NB; nb += G) {
        Acc acc[G];
        mfma_block(kf, nb, acc);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          float m = -INFINITY;
#pragma unroll
          for (int i = 0; i < kRegs; ++i)
            m = fmaxf(m, in_chunk(0, i) ? acc[g][i] * a.c2 : -INFINITY);
          st_m[nb + g] = M == 16 ? max_lane_groups(m) : max_lane_halves(m);
        }
      }
    }
    // (the ragged tail of a sequence takes the slow path too: it masks)
    bool redo = !full;
    if (full) {
      // The tile's sum, then one addition to the row's: the chain of additions
      // is as long as the item has tiles.  (Equal addends, whose rounding is the
      // same every time, were up to 2e-5 off in items of 131072 positions added
      // block by block.)
      float z[NB];
      pipelined_tile(kt, std::integral_constant<int, 3>{}, [&](int tb, int nb0, const Acc(&acc)[G]) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
          float p[4];
#pragma unroll
          for (int i = 0; i < kRegs; ++i) {
            const float e = __builtin_amdgcn_exp2f(
                __builtin_fmaf(acc[g][i], a.c2, -st_m[nb0 + g]));
            p[i & 3] = i < 4 ? e : p[i & 3] + e;
          }
          const float sum = (p[0] + p[1]) + (p[2] + p[3]);
          z[nb0 + g] = tb == 0 ? sum : z[nb0 + g] + sum;
        }
      });
      bool over = false;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        z[nb] += st_z[nb];
        over |= !(z[nb] <= 0x1p100f);
      }
      redo = __any(over);
      if (!redo)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) st_z[nb] = z[nb];
    }
    if (redo) {
      // Slow path: a new large maximum.  Online max / rescale per block and
      // lane, padding masked; from here on the lanes of a row may hold
      // different maxima.
#pragma unroll 1
      for (int tb = 0; tb < kBlocks; ++tb) {
        u32x4 kf[kSegs];
        load_block(kt, tb, kf);
#pragma unroll
        for (int nb = 0; nb < NB; nb += G) {
          Acc acc[G];
          mfma_block(kf, nb, acc);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            float x[kRegs], p[4], mn = st_m[nb + g];
#pragma unroll
            for (int i = 0; i < kRegs; ++i) {
              x[i] = in_chunk(tb, i) ? acc[g][i] * a.c2 : -INFINITY;
              mn = fmaxf(mn, x[i]);
            }
            const float ms = (mn == -INFINITY) ? 0.f : mn;
#pragma unroll
            for (int i = 0; i < kRegs; ++i) {
              const float e = __builtin_amdgcn_exp2f(x[i] - ms);
              p[i & 3] = i < 4 ? e : p[i & 3] + e;
            }
            st_z[nb + g] = st_z[nb + g] * __builtin_amdgcn_exp2f(st_m[nb + g] - ms) +
                           ((p[0] + p[1]) + (p[2] + p[3]));
            st_m[nb + g] = mn;
          }
        }
      }
    }
  }
  if (PASS2 && POS && wave_active) {
    // the chunk's last block: its right neighbour is the next chunk's first
    uint32_t hx[RB] = {};
    if (t_end < a.T) halo_bits(t_end, hx);
    uint32_t fin[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) fin[rb] = umax(pc[rb], row_shr<13>(left4(hx[rb])));
    float nu;
    if (a.pow_mode == kPowMax)
      nu = max_lane_groups(numer(Power<kPowMax, 2>{}, fin));
    else if (a.pow_mode == kPowSquare)
      nu = sum_lane_groups(a.gshift == 3 ? numer(Power<kPowSquare, 3>{}, fin)
                                         : numer(Power<kPowSquare, 2>{}, fin));
    else
      nu = sum_lane_groups(a.gshift == 3 ? numer(Power<kPowGeneral, 3>{}, fin)
                                         : numer(Power<kPowGeneral, 2>{}, fin));
    *numer_slot(ntiles - 1, kBlocks - 1) = nu;
  }
  __syncthreads();

  if (PASS2) {
    for (int t = tid; t < TT; t += W * 64) flush_tile(ntiles - 1, t);
    if (POS) {
      if (ntiles > 1) flush_num(ntiles - 2);
      flush_num(ntiles - 1);
    }
    if (QUEUE && tid == 0) sh.next = next;
    return;
  }

  // ---- P1: merge the lane groups of each row, publish its chunk statistics --
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float m = st_m[nb], z = st_z[nb];
#pragma unroll
    for (int off = M; off < 64; off <<= 1) {
      const float mo = __shfl_xor(m, off);
      const float zo = __shfl_xor(z, off);
      lse_merge(m, z, mo, zo);
    }
    const int row = wrow0 + nb * M + lc;
    if (lg == 0 && row < a.Rp)
      put_f2(a.partial + ((size_t)u * a.chunks + chunk) * a.Rp + row, make_float2(m, z));
  }
  if constexpr (QUEUE) {
    stores_done_barrier();
    if (tid == 0) {
      count_in(done1 + (size_t)u * a.row_groups + rg);
      sh.next = next;
    }
  }
}

template <int ESZ, int D, int W, bool POS, int RB>
__global__ __launch_bounds__(W * 64, waves_per_simd(ESZ, W, true)) void persistent_kernel(
    PersistArgs a) {
  __shared__ Shared<ESZ, D, W, POS, RB, true> sh;
  if (threadIdx.x == 0) sh.next = take_item(a.sync);
  __syncthreads();
  int64_t item = sh.next;
  while (item < a.wl.items) {
    const Item it = decode(a.wl, item);
    switch (it.stage) {
      case kStageP1: score_item<ESZ, D, W, RB, false, POS, true>(a, it.unit, it.sub, sh); break;
      case kStageP2: score_item<ESZ, D, W, RB, true, POS, true>(a, it.unit, it.sub, sh); break;
      default:   // not reached: every item index below wl.items decodes
        if (threadIdx.x == 0) sh.next = take_item(a.sync);
        break;
    }
    __syncthreads();
    item = sh.next;
  }
}

// One score pass of every item, one item per workgroup: blocks of one unit go
// to the same XCD (workgroups are dealt to the eight XCDs in turn), whose L2
// then serves its query rows.  The second pass takes the items last first:
// where they fill several rounds of workgroups it then starts on the keys the
// first pass read last (in one round all items run at once, and the order does
// nothing).
template <int ESZ, int D, int W, bool POS, int RB, bool PASS2>
__global__ __launch_bounds__(W * 64, waves_per_simd(ESZ, W, false)) void pass_kernel(
    PersistArgs a) {
  __shared__ Shared<ESZ, D, W, POS, RB, false> sh;
  if (!PASS2)   // the words later launches of the call count in
    for (int i = blockIdx.x * (W * 64) + threadIdx.x; i < a.sync_words; i += gridDim.x * (W * 64))
      a.sync[i] = 0u;
  const int per_unit = a.chunks * a.row_groups;
  const int n = a.units * per_unit;
  int item = (int)(blockIdx.x & 7u) * ((int)gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (item >= n) return;
  if (PASS2) item = n - 1 - item;
  const int u = item / per_unit;
  score_item<ESZ, D, W, RB, PASS2, POS, false>(a, u, item - u * per_unit, sh);
}

// lse2[row] of every query row from its chunks' (max, sum) pairs: eight
// threads a row, each folding every eighth chunk with eight loads in flight.
__global__ __launch_bounds__(256) void fold_stats(const float2* __restrict__ partial,
                                                  float* __restrict__ lse2, int chunks, int Rp,
                                                  int64_t rows) {
  __shared__ float2 part[8][32];
  const int r = threadIdx.x & 31, k = threadIdx.x >> 5;
  const int64_t row = (int64_t)blockIdx.x * 32 + r;
  float m = -INFINITY, z = 0.f;
  if (row < rows) {
    const int64_t u = row / Rp;
    const float2* p = partial + (size_t)u * chunks * Rp + (row - u * Rp);
    for (int c0 = k; c0 < chunks; c0 += 64) {
      float2 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int c = c0 + 8 * j;
        v[j] = c < chunks ? p[(size_t)c * Rp] : make_float2(-INFINITY, 0.f);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) lse_merge(m, z, v[j].x, v[j].y);
    }
  }
  part[k][r] = make_float2(m, z);
  __syncthreads();
  if (k != 0 || row >= rows) return;
#pragma unroll
  for (int j = 1; j < 8; ++j) lse_merge(m, z, part[j][r].x, part[j][r].y);
  lse2[row] = m + __log2f(z);
}

// out[u][t] = sum (or maximum) over row groups, in order.
__global__ void rowgroup_sum(const float* __restrict__ part, float* __restrict__ out,
                             int row_groups, int64_t per_group, int64_t n, int take_max) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s = 0.f;
  for (int r = 0; r < row_groups; ++r)
    s = take_max ? fmaxf(s, part[r * per_group + i]) : s + part[r * per_group + i];
  out[i] = s;
}

__global__ void zero_words(uint32_t* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// Resident workgroups per CU of one instantiation's kernels, cached per device.
struct Occupancy {
  int queue, passes;
};
std::mutex g_occ_mu;
Occupancy g_occ[64][2][2][4][2][9];
int g_cus[64];

// Row-group partial sums of a call into its outputs.
template <bool POS>
hipError_t finish_row_groups(const ScorePlan& p, const PersistArgs& a, hipStream_t s) {
  hipError_t e = hipSuccess;
  if (p.row_groups > 1) {
    const int64_t n = (int64_t)p.units * p.T;
    rowgroup_sum<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(a.imp_partial, a.importance,
                                                            p.row_groups, n, n, 0);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (POS) {
      rowgroup_sum<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(
          a.numer_partial, a.numer, p.row_groups, n, n, a.pow_mode == kPowMax);
      e = hipGetLastError();
    }
  }
  return e;
}

template <int ESZ, int D, int W, bool POS, int RB = 4>
hipError_t launch_w(const ScorePlan& p, PersistArgs& a, hipStream_t s, ScoreForm* only) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  const int wi = W == 1 ? 0 : W == 2 ? 1 : W == 4 ? 2 : 3;
  int queue_resident = 0, resident = 0;
  {
    std::lock_guard<std::mutex> lock(g_occ_mu);
    Occupancy& occ = g_occ[dev][ESZ == 2][D == 128][wi][POS][RB];
    if (occ.queue == 0) {
      const void* const f[3] = {
          reinterpret_cast<const void*>(&persistent_kernel<ESZ, D, W, POS, RB>),
          reinterpret_cast<const void*>(&pass_kernel<ESZ, D, W, POS, RB, false>),
          reinterpret_cast<const void*>(&pass_kernel<ESZ, D, W, POS, RB, true>)};
      int n[3];
      for (int i = 0; i < 3; ++i) {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n[i], f[i], W * 64, 0);
        if (e != hipSuccess) return e;
        if (n[i] < 1) n[i] = 1;
      }
      occ.passes = n[1] < n[2] ? n[1] : n[2];
      occ.queue = n[0];
    }
    if (g_cus[dev] == 0) {
      e = hipDeviceGetAttribute(&g_cus[dev], hipDeviceAttributeMultiprocessorCount, dev);
      if (e != hipSuccess) return e;
    }
    queue_resident = occ.queue * g_cus[dev];
    resident = occ.passes * g_cus[dev];
  }
  const ScoreForm form = choose_form(p, queue_resident, resident);
  if (only) {
    *only = form;
    return hipSuccess;
  }
  const int64_t groups = (int64_t)p.units * p.row_groups;
  a.chunk_tokens = form.chunk_tokens;
  a.chunks = (int)((p.T + a.chunk_tokens - 1) / a.chunk_tokens);
  if (!form.queue) {
    // Folding up to 16 chunks in every second-pass workgroup costs less than
    // a launch for it (8 chunks: 22.3 against 24.4 us for the whole call).
    if (a.chunks <= 16) a.lse2 = nullptr;
    a.sync_words = (int)p.sync_words;
    const unsigned g = (unsigned)((groups * a.chunks + 7) / 8 * 8);
    pass_kernel<ESZ, D, W, POS, RB, false><<<g, W * 64, 0, s>>>(a);
    if (a.lse2) {
      const int64_t rows = (int64_t)p.units * p.Rp;
      fold_stats<<<(unsigned)((rows + 31) / 32), 256, 0, s>>>(a.partial, a.lse2, a.chunks, a.Rp,
                                                              rows);
    }
    pass_kernel<ESZ, D, W, POS, RB, true><<<g, W * 64, 0, s>>>(a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return finish_row_groups<POS>(p, a, s);
  }
  int per_unit[kMaxStages];
  per_unit[kStageP1] = a.chunks * p.row_groups;
  per_unit[kStageP2] = a.chunks * p.row_groups;
  make_work_list(p.units, kMaxStages, per_unit, queue_resident, &a.wl);
  const int64_t grid = a.wl.items < queue_resident ? a.wl.items : queue_resident;
  zero_words<<<(unsigned)((p.sync_words + 255) / 256 < 1024 ? (p.sync_words + 255) / 256 : 1024),
               256, 0, s>>>(a.sync, (int64_t)p.sync_words);
  persistent_kernel<ESZ, D, W, POS, RB><<<(unsigned)grid, W * 64, 0, s>>>(a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return finish_row_groups<POS>(p, a, s);
}

template <int ESZ, int D, bool POS>
hipError_t launch_d(const ScorePlan& p, PersistArgs& a, hipStream_t s, ScoreForm* only) {
  switch (10 * p.waves + p.rb) {
    case 11: return launch_w<ESZ, D, 1, POS, 1>(p, a, s, only);
    case 12: return launch_w<ESZ, D, 1, POS, 2>(p, a, s, only);
    case 14: return launch_w<ESZ, D, 1, POS, 4>(p, a, s, only);
    case 24: return launch_w<ESZ, D, 2, POS, 4>(p, a, s, only);
    case 44: return launch_w<ESZ, D, 4, POS, 4>(p, a, s, only);
    case 84: return launch_w<ESZ, D, 8, POS, 4>(p, a, s, only);
  }
  if constexpr (ESZ == 2) {
    switch (10 * p.waves + p.rb) {
      case 13: return launch_w<ESZ, D, 1, POS, 3>(p, a, s, only);
      case 23: return launch_w<ESZ, D, 2, POS, 3>(p, a, s, only);
      case 43: return launch_w<ESZ, D, 4, POS, 3>(p, a, s, only);
    }
  }
  if constexpr (!POS) {
    if (p.waves == 4 && p.rb == 5) return launch_w<ESZ, D, 4, POS, 5>(p, a, s, only);
    if constexpr (ESZ == 2) {
      if (p.waves == 4 && p.rb == 6) return launch_w<ESZ, D, 4, POS, 6>(p, a, s, only);
      if (p.waves == 4 && p.rb == 8) return launch_w<ESZ, D, 4, POS, 8>(p, a, s, only);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Launch of the persistent score kernel for one element size and head
// dimension; each combination is instantiated in a translation unit of its
// own (score_<dtype>_d<D>.hip, and score_pos_<dtype>_d<D>.hip for the
// position variant) so that they compile in parallel.
template <int ESZ, int D>
hipError_t launch_score_d(const ScorePlan& p, PersistArgs& a, hipStream_t s, ScoreForm* only) {
  return launch_d<ESZ, D, false>(p, a, s, only);
}
template <int ESZ, int D>
hipError_t launch_position_d(const ScorePlan& p, PersistArgs& a, hipStream_t s, ScoreForm* only) {
  return launch_d<ESZ, D, true>(p, a, s, only);
}

}  // namespace cb
