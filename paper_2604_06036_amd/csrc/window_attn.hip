// (d) Joint prefill attention of refresh + suffix tokens over the mixed window cache, gfx950.
//
// Paper Sec. 3.5: refresh tokens and the normal suffix run one joint prefill pass; at each layer
// causal attention reads a cache that mixes reused (position-corrected) states with states
// written in the current pass.  Causality follows the window-sequence index of each query.
//
// bf16 kernels (matrix cores).  A "row" is one (query token, query head of one kv group) pair, so the K/V tiles a
// workgroup stages in LDS are shared by all query heads of the group.  Keys are swept in tiles of 64 through LDS:
//   S^T = K Q^T      v_mfma_f32_32x32x16_bf16, A = K fragment from LDS (ds_read_b128),
//                    B = Q^T fragment held in registers for the whole sweep;
//   online softmax   fp32, per-lane statistics: in the S^T layout a lane owns one query and 16
//                    of its 32 keys, the two half-waves exchange the running max;
//   O^T += V^T P^T   P^T is already in B-operand layout (no LDS round trip); the V^T fragment is
//                    fetched from the row-major V tile with the LDS transpose read
//                    (ds_read_b64_tr_b16), so V is never transposed in memory.
// Key ranges that lie wholly above a wave's causal frontier are skipped by that wave; only ranges that
// straddle a frontier pay for masking.  Cache rows past the workgroup's frontier are never read
// (they may be unallocated): the lanes that would fetch them fetch the frontier row instead.
//
// head_dim 128: a planning kernel lists the work items of the launch and persistent workgroups
// stream K/V tiles from HBM straight into LDS (global_load_lds), across item boundaries; long key
// sweeps of small batches are split over several items and merged by a second kernel.
// head_dim 64, and launches of few row tiles: one workgroup per row tile, no plan, key ranges shared inside it.
//
// fp32 kernel: the fp32 matrix instruction, 32 rows per workgroup, keys dealt to its waves.
#include <math.h>

#include <type_traits>

#include "common.h"


namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

struct AttnParams {
  const void* __restrict__ q;
  const void* __restrict__ k;
  const void* __restrict__ v;
  void* __restrict__ out;
  const int32_t* __restrict__ cu_q;
  const int32_t* __restrict__ q_pos;
  const int32_t* __restrict__ block_table;
  const int32_t* __restrict__ kv_len;
  int64_t stride_slot, stride_head;
  int32_t max_blocks, n_streams, n_q_heads, n_kv_heads, group;
  float scale, scale_log2e;
  int64_t n_q;
  // Split sweeps (AttnPlan::span): a row tile's keys may be shared by several work items; their un-normalised partial
  // results go to the workspace and a second kernel merges them.  (Merging in the last workgroup to finish was built
  // twice and is far slower here, also with write-through stores in place of an L2 write-back: single stream, 919 keys,
  // 42 against 23 us per call; 6,033 keys 133 against 117; 17,630 keys 310 against 290.)
  int32_t bm;
  int32_t pieces;          // workgroups that share a sweep without a plan (window_attn_bf16_tile_kernel<.., SPLIT>)
  const int32_t* ws_plan;   // plan header (list offsets per XCD, row-tile count, end item, first items)
  const int32_t* ws_items;  // item descriptors, 8 ints each, the 8 XCD lists back to back
  // refresh write fused into the launch (cs_refresh_prefill_attn): rows to write before attention
  const void* __restrict__ k_new;
  const void* __restrict__ v_new;
  const int32_t* __restrict__ new_slot;
  int64_t n_new;
  int32_t row_vecs, head_vecs;   // 16-byte vectors per new row / per head
  cs::u32x2* ws_own;     // CS_ATTN_OWN_ROWS: where the rows of each cache block are (OwnEntry), [streams][max_blocks]
  int32_t* ws_tiles;     // and the row tiles of a launch without a plan, [workgroups][8] (window_attn_own_rows_kernel)
  cs::u32x2* ws_warm;    // and of every stream its first query and how many cache entries its queries see
  int32_t n_warm;        // workgroups ahead of the row tiles that bring keys and values into L2 (warm_l2)
  int32_t* ws_sync;      // counters of the fused launch's launch-wide barrier (see launch_barrier)
  int32_t* ws_status;    // its status word
  int32_t clear_status;  // the launch without a plan zeroes it
  int32_t* ws_desc;      // [row tiles][8]: q0, rows_total, r_tile, kvh, n_split, list position of the first piece, see plan_spans
  float* ws_ml;          // [items][bm][2]: running max (raw score units), row sum
  float* ws_o;           // [items][bm][128]: un-normalised output rows
};

constexpr int kBM = 128;   // rows per row tile
constexpr int kBN = 64;    // keys per LDS tile
constexpr float kNegInf = -INFINITY;
constexpr int kMaxBlocks64 = 8192;      // head_dim 64: windows up to 131072 tokens (a limit of the interface; this kernel has none)

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// Two fp32 -> packed bf16 (round to nearest even) in one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Running-max slack of the online softmax, in log2 units: the reference maximum of a row is only
// raised (and the accumulators rescaled) when the tile maximum exceeds it by more than this, so
// probabilities stay below 2^kMaxSlack and almost every tile skips the rescale.
constexpr float kMaxSlack = 8.0f;

// ------------------------------------------------------------------------------------------
// Tile transport for head_dim 128 (the shape of every bf16 workload measured).
//
// K/V tiles are copied global -> LDS by the DMA form of the global load
// (global_load_lds_dwordx4: lane l of a wave deposits its 16 bytes at base + 16 l, the source
// address is free per lane), so nothing is staged through registers and there is one workgroup
// barrier per tile.  Because the DMA fixes the LDS position of each lane's chunk, bank conflicts
// are avoided by choosing WHICH 16-byte chunk of a row each lane fetches (an XOR swizzle on the
// source side) instead of padding rows:
//   K tile row r: chunk c is stored at position c ^ (r % 16)   (ds_read_b128 of 16 rows at one c)
//   V tile row r: chunk c is stored at position c ^ (4 (r % 4) + 2 ((r / 4) % 2))
//                 (a transpose read touches 8 rows x 2 chunks: this spreads them over all banks)
typedef __attribute__((address_space(3))) void lds_void_t;

// One 16-byte-per-lane DMA copy global -> LDS (lane l lands at lds_addr + 16 l).  Issued as inline
// assembly on purpose: the compiler then keeps no scoreboard entry for it and does not drain the
// whole prefetch queue before the next LDS read; completion is enforced by the explicit vmcnt
// waits and workgroup barriers of the pipeline below.  The "memory" clobber tells the compiler
// that LDS contents change here.
__device__ __forceinline__ void dma16(const void* gsrc, const void* lds_dst) {
  const uint32_t lds_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)lds_dst));
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(gsrc), "s"(lds_addr)
               : "memory", "m0");
}

// The same with a wave-uniform 64-bit base in SGPRs and a 32-bit byte offset per lane.
__device__ __forceinline__ void dma16_s(uint32_t off, const void* sbase, const void* lds_dst) {
  const uint32_t lds_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)lds_dst));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(sbase), "s"(lds_addr)
               : "memory", "m0");
}

// ... and with the LDS destination given as a byte address in an SGPR.
__device__ __forceinline__ uint32_t lds_address(const void* lds_ptr) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)lds_ptr));
}
__device__ __forceinline__ void dma16_sa(uint32_t off, const void* sbase, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(sbase), "s"(lds_addr)
               : "memory", "m0");
}

// 4 bytes per lane: lane l lands at lds_addr + 4 l
__device__ __forceinline__ void dma4_sa(uint32_t off, const void* sbase, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :
               : "v"(off), "s"(sbase), "s"(lds_addr)
               : "memory", "m0");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  // s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt in bits
  // 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8 left at their maxima)
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

typedef __attribute__((ext_vector_type(8))) int32_t i32x8;

// Scalar loads issued by hand: the results are uniform, travel outside the vector-memory queue
// (so waiting for them never drains tile requests) and are only read after the explicit wait.
__device__ __forceinline__ i32x8 sload8(const void* ptr) {
  i32x8 v;
  asm volatile("s_load_dwordx8 %0, %1, 0x0" : "=&s"(v) : "s"(ptr));
  return v;
}
__device__ __forceinline__ int32_t sload1(const void* ptr) {
  int32_t v;
  asm volatile("s_load_dword %0, %1, 0x0" : "=&s"(v) : "s"(ptr));
  return v;
}

typedef __attribute__((ext_vector_type(2))) int32_t i32x2;
typedef __attribute__((ext_vector_type(4))) int32_t i32x4;
__device__ __forceinline__ i32x2 sload2(const void* ptr) {
  i32x2 v;
  asm volatile("s_load_dwordx2 %0, %1, 0x0" : "=&s"(v) : "s"(ptr));
  return v;
}

// A pointer that is the same in all lanes, for an instruction that takes it in scalar registers.
template <typename T>
__device__ __forceinline__ T* uniform(T* ptr) {
  const uint64_t at = reinterpret_cast<uintptr_t>(ptr);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(at)), hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(at >> 32));
  return reinterpret_cast<T*>(static_cast<uintptr_t>(static_cast<uint64_t>(hi) << 32 | lo));
}

// Where a call that reads its queries' own rows (CS_ATTN_OWN_ROWS) finds those of a cache block, two words a block of every
// stream: the block's id (27 bits), the index, among the stream's queries, of the first of its rows that the call brings (21
// bits), and which of its 16 rows those are (16 bits: all of them stand for 16 rows that there are, also in a stream's last block).  They
// are consecutive among the call's rows, queries being in order.
constexpr int kOwnIdBits = 27, kOwnRowBits = 21;      // (slots are 32-bit: ids below 2^27; windows of up to 2^21 entries)
struct OwnEntry {
  uint32_t id, row, mask;
  __device__ __forceinline__ OwnEntry(const i32x2& e)      // the same in all lanes
      : OwnEntry(__builtin_amdgcn_readfirstlane(e.x), __builtin_amdgcn_readfirstlane(e.y)) {}
  __device__ __forceinline__ OwnEntry(uint32_t lo, uint32_t hi) {
    id = lo & ((1u << kOwnIdBits) - 1);
    row = lo >> kOwnIdBits | hi >> 16 << (32 - kOwnIdBits);
    mask = hi & 0xffffu;
  }
  static __device__ __forceinline__ cs::u32x2 packed(uint32_t id, uint32_t row, uint32_t mask) {
    return cs::u32x2{id | row << kOwnIdBits, row >> (32 - kOwnIdBits) << 16 | mask};
  }
  // of row r of the block: whether it is one of the call's own, and which of the stream's
  __device__ __forceinline__ bool own(int r) const { return mask >> r & 1; }
  __device__ __forceinline__ uint32_t row_of(int r) const { return row + __popc(mask & ((1u << r) - 1)); }
};

// ---- loads of data that does not change during the launch: through the constant address space they are scalar loads
typedef const __attribute__((address_space(4))) i32x8 const_i32x8;
__device__ __forceinline__ i32x8 const_load8(const int32_t* at) { return *(const_i32x8*)reinterpret_cast<uintptr_t>(at); }

// A scalar load that the compiler knows of turns every wait for an LDS read into a wait for all: it is waited for on the spot.
__device__ __forceinline__ void wait_scalar() { __builtin_amdgcn_s_waitcnt(0xc07f); }

// One row tile of a launch without a plan: stream, kv head, first row.
struct RowTile {
  int s, kvh, q0, rows_total, r_tile;
};

// Which (stream, kv head, tile of BM rows) is workgroup b?  False: none (n_q may be an upper bound).  Of more than 64
// streams each thread adds up the tiles of a few neighbours, and a scan over the workgroup finds whose streams hold the
// tile (s_tiles: an int a thread, free again on return); a scan over 64 streams, a lane each, then finds the stream.  All
// waves take the same values.  Longest sweeps of
// a stream come first, the kv heads of a tile are neighbours, so each XCD (workgroups go round robin) serves a share
// of every stream.  A list cut into one run per XCD, so that the tiles of a (stream, kv head) pair share its K and V
// in one L2, was level when all streams are alike and 5-13 % slower when they differ: the runs then carry unequal
// work (12 streams of 900 keys, head_dim 64: 33.4 against 30.5 us).
template <int BM, int WAVES>
__device__ __forceinline__ bool find_row_tile(const AttnParams& p, int b, int* s_tiles, RowTile& t) {
  const int lane = threadIdx.x & 63;
  const int x = b / p.n_kv_heads;
  // tiles of the lanes up to and with this one
  auto scan = [](int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8: inside each 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);      // row_bcast:15: lane 15 to the second 16, 47 to the fourth
    return v + __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);      // row_bcast:31: lane 31 to the upper half
  };
  int s0 = 0, end = p.n_streams, before = 0;
  while (end - s0 > 64) {                  // (a second time only beyond 4,096 streams a wave)
    const int share = (end - s0 - 1) / (64 * WAVES) + 1;
    const int first = static_cast<int>(min(threadIdx.x * static_cast<unsigned>(share), static_cast<unsigned>(end - s0))) + s0;
    const int mine_end = min(share, end - first);
    int mine = 0, from = p.cu_q[first];
    for (int k = 0; k < share; k += 4) {   // (past the thread's share: its end again, no rows)
      int to[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) to[i] = p.cu_q[first + min(k + i + 1, mine_end)];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mine += ((to[i] - from) * p.group + BM - 1) / BM;
        from = to[i];
      }
    }
    s_tiles[threadIdx.x] = scan(mine);
    __syncthreads();
    int w = 0;
    while (w < WAVES && x >= before + s_tiles[64 * w + 63]) before += s_tiles[64 * w++ + 63];
    if (w == WAVES) return false;
    const int incl = s_tiles[64 * w + lane];
    const int at = __ffsll(__ballot(x < before + incl)) - 1;
    if (at > 0) before += __builtin_amdgcn_readlane(incl, at - 1);
    s0 += (64 * w + at) * share;
    end = min(share, end - s0) + s0;
    __syncthreads();                       // (s_tiles may be written again)
  }
  const int s = s0 + lane;
  const int lo = s < end ? p.cu_q[s] : 0;
  const int rows = s < end ? (p.cu_q[s + 1] - lo) * p.group : 0;
  const int incl = scan((rows + BM - 1) / BM);
  const unsigned long long found = __ballot(x < before + incl);
  if (!found) return false;
  const int at = __ffsll(found) - 1;
  t.s = s0 + at;
  t.kvh = b % p.n_kv_heads;
  t.q0 = __builtin_amdgcn_readlane(lo, at);
  t.rows_total = __builtin_amdgcn_readlane(rows, at);
  t.r_tile = (before + __builtin_amdgcn_readlane(incl, at) - 1 - x) * BM;
  return true;
}

// The frontier of a row tile: the last cache entry that its last row sees, inside those that the stream's block-table row
// defines (-1: none).
template <int BM>
__device__ __forceinline__ int tile_frontier(const AttnParams& p, const RowTile& t) {
  const int cap = min(p.kv_len[t.s], p.max_blocks * CS_KV_BLOCK) - 1;
  return min(p.q_pos[t.q0 + (min(t.r_tile + BM, t.rows_total) - 1) / p.group], cap);
}

// bf16, one launch and no plan: a workgroup = one tile of 32 ROWW rows of one (stream, kv head), its waves
// arranged as KG key groups of ROWW row waves.  Group g sweeps key tiles g, g + KG, ...; the groups' partial
// results meet in LDS at the end, so a sweep is shared by KG times as many waves without a trip through memory
// and without a merge launch.  head_dim 64 always runs here, head_dim 128 where tile_route_128 says so.
// SPLIT: a sweep is cut into up to p.pieces runs of whole trips (KG key tiles each), a workgroup to a run; where there
// are several, their partial rows go to the workspace and window_attn_merge_kernel, told by `describe`, combines them.
// Tiles go to LDS by DMA with the persistent kernel's layout and swizzle idea.  STAGES 2: the next tile is requested
// at the top of a tile, one workgroup barrier per tile.  STAGES 1 (half the LDS: more workgroups per CU, or more key
// groups): K of the next tile is requested when S is done and lands behind P V, V when P V is done and lands behind
// S and the softmax; two barriers per tile.
// What bounds it: with few row tiles the serial chain of the longest sweep (per tile barrier, S, softmax, P V),
// hence the key groups; with many the vector pipe (head_dim 64 has the softmax of 128 over half the MFMAs).
// head_dim 64 against single-buffered tiles staged through registers, us a layer in a step: one stream of 900 keys,
// 16/4 heads 20.0 -> 15.2; 4 streams, 28/4 heads 29.0 -> 23.5; 12 streams, 16/4 35.0 -> 26.9; 32 streams 62.0 -> 58.7;
// 2 streams of 8,600 keys 231 -> 140.
template <int D>
__device__ __forceinline__ int k_swizzle(int r) { return D == 128 ? r & 15 : (r >> 1) & 7; }
template <int D>
__device__ __forceinline__ int v_swizzle(int r) {
  return D == 128 ? 4 * (r & 3) + 2 * ((r >> 2) & 1) : 4 * ((r >> 1) & 1) + 2 * ((r >> 2) & 1);
}

// A workgroup's share of the refresh write in a launch that reads its own rows where the caller has them
// (CS_ATTN_OWN_ROWS): 16 bytes of K and of V a thread, more than once where the launch has fewer threads.  Asked for behind
// everything that the sweep waits for (loads return in order) and stored behind the sweep.  A launch of its own took 3.9 us of a
// layer of one stream (900 keys, 28/4 heads) and its 28 layers 586 us; this share 0.7, reading the new rows in place of the
// cache 0.65 more, 516 us.  12 streams of head_dim 64, 24 layers 836 -> 784 us.  First workgroups of their own for the share:
// the same for one stream, 827 us for the 12.
template <int THREADS>
struct OwnMove {
  cs::u32x4 k, v;
  int slot = -1;
  uint32_t rem = 0;
  __device__ __forceinline__ void load(const AttnParams& p) {
    const uint32_t n_units = static_cast<uint32_t>(p.n_new) * p.row_vecs;      // (below 2^31: the host checks)
    const uint64_t apart = static_cast<uint64_t>(gridDim.x - p.n_warm) * THREADS;
    const uint32_t wg = blockIdx.x - p.n_warm;
    if (static_cast<uint64_t>(wg) * THREADS + threadIdx.x >= n_units) return;
    uint32_t unit = wg * THREADS + threadIdx.x;
    for (;;) {
      const uint32_t tok = unit / p.row_vecs;
      rem = unit - tok * p.row_vecs;
      slot = p.new_slot[tok];
      k = __builtin_nontemporal_load(static_cast<const cs::u32x4*>(p.k_new) + unit);
      v = __builtin_nontemporal_load(static_cast<const cs::u32x4*>(p.v_new) + unit);
      if (n_units - unit <= apart) break;
      unit += static_cast<uint32_t>(apart);
      store(p);
    }
  }
  __device__ __forceinline__ void store(const AttnParams& p) const {
    if (slot < 0) return;
    const int64_t to = static_cast<int64_t>(slot) * p.row_vecs + rem;
    __builtin_nontemporal_store(k, static_cast<cs::u32x4*>(const_cast<void*>(p.k)) + to);
    __builtin_nontemporal_store(v, static_cast<cs::u32x4*>(const_cast<void*>(p.v)) + to);
  }
  __device__ __forceinline__ void all(const AttnParams& p) {
    load(p);
    store(p);
  }
};

template <int D, int KG, int STAGES>
struct TileStages {
  __attribute__((aligned(1024))) uint16_t kv[KG][STAGES][2][kBN * D];
};

template <int D, int ROWW, int KG, int STAGES, bool SPLIT = false, bool OWN = false>
__device__ __forceinline__ void attend_row_tile(const AttnParams& p, int block, TileStages<D, KG, STAGES>& stages) {
  constexpr int BM = 32 * ROWW;
  constexpr int STEPS = D / 16, DB = D / 32;
  constexpr int TILE = kBN * D;        // elements of one K (or V) tile, unpadded
  constexpr int CPR = D / 8;           // 16-byte chunks per row
  constexpr int RPD = 64 / CPR;        // rows per 1-KiB DMA instruction
  constexpr int IPW = CPR / ROWW;      // DMA instructions per wave, per tile, per tensor
  constexpr int BPW = kBN / ROWW / CS_KV_BLOCK;      // cache blocks a wave requests per tile
  constexpr int IPB = IPW / BPW;       // its DMA instructions per block
  static_assert(BPW >= 1 && IPB * RPD == CS_KV_BLOCK, "a DMA instruction stays inside a cache block");

  auto& s_kv = stages.kv;
  constexpr bool SPREAD = KG > 2;      // the merge of the groups is shared by all waves (see there)
  __shared__ float s_ml[SPREAD ? KG : 1][ROWW][2][64];
  static_assert(KG == 1 || KG == 2 || KG == DB, "of four groups each finishes one block of columns");
  static_assert(sizeof(s_kv) >= sizeof(float) * (SPREAD ? KG : KG / 2) * ROWW * DB * 16 * 64, "the merge reuses the tile buffers");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rw = wave % ROWW, kg = wave / ROWW;
  const int n = lane & 31, h = lane >> 5;

  if (p.clear_status && block == 0 && threadIdx.x == 0) *p.ws_status = 0;
  int piece = 0;
  if constexpr (SPLIT) {                                // the pieces of a row tile are neighbours, like the kv heads of one
    const int x = block / p.n_kv_heads;
    piece = x % p.pieces;
    block = x / p.pieces * p.n_kv_heads + block % p.n_kv_heads;
  }
  auto describe = [&](const RowTile& t, int n_pieces) {  // to the merge kernel: once a row tile, also where there is none
    if (SPLIT && piece == 0 && threadIdx.x == 0) {
      int32_t* rd = p.ws_desc + static_cast<int64_t>(block) * 8;
      rd[0] = t.q0; rd[1] = t.rows_total; rd[2] = t.r_tile; rd[3] = t.kvh; rd[4] = n_pieces; rd[5] = block * p.pieces; rd[6] = 0;
    }
  };
  // The row tile: found from cu_q and q_pos, or, in a call that follows the one that plans, read from what that one left:
  // first query token and rows of the stream, first row, kv head, frontier, stream.
  OwnMove<64 * ROWW * KG> move;
  auto settle = [] { if (SPLIT || OWN) wait_scalar(); };      // (before the workgroup may end: no scalar load is left in flight)
  RowTile t = {};
  int wg_max, cap;
  if constexpr (OWN) {
    const i32x8 d = const_load8(p.ws_tiles + static_cast<int64_t>(block) * 8);
    t.q0 = d[0]; t.rows_total = d[1]; t.r_tile = d[2]; t.kvh = d[3]; t.s = d[5];
    cap = wg_max = d[4];
    if (t.rows_total <= 0) {
      describe(t, 0);
      move.all(p);
      settle();
      return;
    }
  } else {
    const bool found = find_row_tile<BM, ROWW * KG>(p, block, reinterpret_cast<int*>(&s_kv[0][0][0][0]), t);
    settle();
    if (!found) {
      describe(t, 0);
      settle();
      return;
    }
  }
  const int s = __builtin_amdgcn_readfirstlane(t.s), kvh = __builtin_amdgcn_readfirstlane(t.kvh);
  const int q0 = __builtin_amdgcn_readfirstlane(t.q0), rows_total = __builtin_amdgcn_readfirstlane(t.rows_total);
  const int r_tile = __builtin_amdgcn_readfirstlane(t.r_tile);

  // ---- this lane's row (query token, head) and causal frontier, kept inside the entries the stream's
  //      block-table row defines
  const int w_first = r_tile + rw * 32;
  const int row = w_first + n;
  const bool valid = row < rows_total;
  const int row_c = valid ? row : rows_total - 1;
  const int tok = q0 + row_c / p.group;
  const int head = kvh * p.group + row_c % p.group;
  if constexpr (!OWN) {
    cap = min(p.kv_len[s], p.max_blocks * CS_KV_BLOCK) - 1;
    wg_max = min(p.q_pos[q0 + (min(r_tile + BM, rows_total) - 1) / p.group], cap);
  }
  const int pos = p.q_pos[tok];
  int lim, wave_min, wave_max;
  auto frontiers = [&]() __attribute__((always_inline)) {
    lim = valid ? min(pos, cap) : -1;
    // positions do not decrease along the rows
    const int rows_here = min(32, rows_total - w_first);
    wave_min = rows_here > 0 ? __builtin_amdgcn_readlane(lim, 0) : -1;
    wave_max = rows_here > 0 ? __builtin_amdgcn_readlane(lim, max(rows_here, 1) - 1) : -1;
  };
  if (STAGES == 1) frontiers();
  if (!SPLIT && wg_max < 0) {                           // the stream defines no cache entry: rows left untouched
    if constexpr (OWN) move.all(p);
    settle();
    return;
  }
  const int n_key_tiles = wg_max / kBN + 1;
  const int last_blk = wg_max / CS_KV_BLOCK;
  // ---- this workgroup's key tiles [kt_begin, kt_end): pieces are whole trips of the groups
  int kt_begin = 0, kt_end = n_key_tiles, n_pieces = 1;
  if constexpr (SPLIT) {
    const int len = ((n_key_tiles + p.pieces - 1) / p.pieces + KG - 1) / KG * KG;
    n_pieces = wg_max < 0 ? 0 : (n_key_tiles + len - 1) / len;
    describe(t, n_pieces);
    settle();
    if (piece >= n_pieces) {
      if constexpr (OWN) move.all(p);
      settle();
      return;
    }
    kt_begin = piece * len;
    kt_end = min(kt_begin + len, n_key_tiles);
  }

  // ---- Q^T fragments: lane = (query n, half h) holds d-slice [16 step + 8 h, + 8).  With two stages they and the positions are
  //      asked for before the cache blocks' ids have come, and the positions looked at behind the first tile's requests: the
  //      compiler does not know of those, and where it waits for a load it waits for all of them.  us a step, 24 layers of
  //      head_dim 64: one stream, 16/4 heads 424 / 415, 12 streams, 8/1 heads 508 / 494, 32 streams, 16/4 heads 1,607 / 1,594; 8 streams, 8/1
  //      heads of 128 1,090 / 1,082.  With one stage the first K is what a sweep starts on, and Q in front of it 1 % slower.
  const int64_t q_at = (static_cast<int64_t>(tok) * p.n_q_heads + head) * D;
  const uint16_t* qrow = static_cast<const uint16_t*>(p.q) + q_at;
  bf16x8 qf[STEPS];
  auto load_queries = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < STEPS; ++st)
      qf[st] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const cs::u32x4*>(qrow + 16 * st + 8 * h));
  };
  if (STAGES == 2) load_queries();

  // ---- tile requests.  This wave fetches rows [16 BPW rw, + 16 BPW) of its group's tiles; inside a cache block
  //      a lane's source offset is constant.  The tile that holds the frontier takes per-lane addresses: rows past
  //      the frontier may be unallocated or hold anything, they fetch the frontier row instead (finite data,
  //      weight 0 after masking).  So does every tile when a block spans more than 32 bits of byte offset.
  const int32_t* bt = p.block_table + static_cast<int64_t>(s) * p.max_blocks;
  const uint16_t* kh = static_cast<const uint16_t*>(p.k) + static_cast<int64_t>(kvh) * p.stride_head;
  const uint16_t* vh = static_cast<const uint16_t*>(p.v) + static_cast<int64_t>(kvh) * p.stride_head;
  const int l_row = lane / CPR, l_pos = lane % CPR;
  const bool wide = p.stride_slot >= (1ll << 26);
  const int64_t blk_stride = static_cast<int64_t>(CS_KV_BLOCK) * p.stride_slot;
  auto chunk_of = [&](int i, bool v) { return l_pos ^ (v ? v_swizzle<D>(RPD * i + l_row) : k_swizzle<D>(RPD * i + l_row)); };
  uint32_t k_off[IPB], v_off[IPB];
#pragma unroll
  for (int i = 0; i < IPB; ++i) {
    const uint32_t at = static_cast<uint32_t>((RPD * i + l_row) * p.stride_slot);
    k_off[i] = (at + chunk_of(i, false) * 8) * 2;
    v_off[i] = (at + chunk_of(i, true) * 8) * 2;
  }
  // cache blocks of this wave's share of a tile: scalar loads, so that waiting for them does not drain the tile
  // requests; issued unconditionally (the last tile's blocks again when there is no next tile).  Every load is waited
  // for in the trip that issued it, also where nothing reads it: the compiler does not know that the register is
  // still to be written, and is free to reuse a dead one
  typedef typename std::conditional<OWN, i32x2, int>::type BlockAt;      // an entry of the table of own rows, or an id
  const i32x2* own_t = reinterpret_cast<const i32x2*>(p.ws_own) + static_cast<int64_t>(s) * p.max_blocks;
  auto load_block = [&](int blk) -> BlockAt {
    if constexpr (OWN) return sload2(own_t + blk);
    else return sload1(bt + blk);
  };
  BlockAt ids[BPW], ids_next[BPW];
  auto load_ids = [&](int kt) {
#pragma unroll
    for (int b = 0; b < BPW; ++b)
      ids_next[b] = load_block(min(min(kt, n_key_tiles - 1) * (kBN / CS_KV_BLOCK) + rw * BPW + b, last_blk));
  };
  auto wait_ids = [&]() {
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
      asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(ids_next[b]));
      ids[b] = ids_next[b];
    }
  };
  BlockAt last_id = load_block(last_blk);
  // (own rows: this call's, in the cache's layout; the same offsets inside 16 rows in a row)
  const int64_t own_at = static_cast<int64_t>(q0) * p.stride_slot + static_cast<int64_t>(kvh) * D;
  const uint16_t* kn = OWN ? static_cast<const uint16_t*>(p.k_new) + own_at : nullptr;
  const uint16_t* vn = OWN ? static_cast<const uint16_t*>(p.v_new) + own_at : nullptr;
  auto request = [&](int kt, int stage, int which) {
    const uint16_t* base = which ? vh : kh;
    uint16_t* dst = &s_kv[kg][stage][which][rw * IPW * 512];
    if constexpr (OWN) {
      const uint16_t* base_new = which ? vn : kn;
#pragma unroll
      for (int b = 0; b < BPW; ++b) {
        const OwnEntry e(ids[b]);
        if (kt != n_key_tiles - 1 && !wide && (e.mask == 0 || e.mask == 0xffffu)) {
          const uint16_t* src = uniform(e.mask ? base_new + e.row * p.stride_slot : base + e.id * blk_stride);
#pragma unroll
          for (int i = 0; i < IPB; ++i) dma16_s(which ? v_off[i] : k_off[i], src, dst + (b * IPB + i) * 512);
        } else {
          const OwnEntry last(last_id);
#pragma unroll
          for (int i = 0; i < IPB; ++i) {
            const int j_un = kt * kBN + (rw * BPW + b) * CS_KV_BLOCK + RPD * i + l_row;
            const bool over = j_un > wg_max;
            const OwnEntry at = over ? last : e;
            const int r = (over ? wg_max : j_un) % CS_KV_BLOCK;
            const uint16_t* src = at.own(r) ? base_new + at.row_of(r) * p.stride_slot
                                            : base + (static_cast<int64_t>(at.id) * CS_KV_BLOCK + r) * p.stride_slot;
            dma16(src + chunk_of(i, which == 1) * 8, dst + (b * IPB + i) * 512);
          }
        }
      }
      return;
    } else if (kt != n_key_tiles - 1 && !wide) {
#pragma unroll
      for (int b = 0; b < BPW; ++b) {
        const uint16_t* src = base + ids[b] * blk_stride;
#pragma unroll
        for (int i = 0; i < IPB; ++i) dma16_s(which ? v_off[i] : k_off[i], src, dst + (b * IPB + i) * 512);
      }
    } else {
#pragma unroll
      for (int b = 0; b < BPW; ++b)
#pragma unroll
        for (int i = 0; i < IPB; ++i) {
          const int j_un = kt * kBN + (rw * BPW + b) * CS_KV_BLOCK + RPD * i + l_row;
          const bool over = j_un > wg_max;
          const int j = over ? wg_max : j_un;
          const int64_t slot = static_cast<int64_t>(over ? last_id : ids[b]) * CS_KV_BLOCK + j % CS_KV_BLOCK;
          dma16(base + slot * p.stride_slot + chunk_of(i, which == 1) * 8, dst + (b * IPB + i) * 512);
        }
    }
  };

  int kt = kt_begin + kg;
  load_ids(kt);
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(last_id));
  wait_ids();
  if (kt < kt_end) {
    request(kt, 0, 0);
    if (STAGES == 2) request(kt, 0, 1);
  }
  if (STAGES == 2) load_ids(kt + KG);

  if (STAGES == 1) load_queries();
  if constexpr (OWN) move.load(p);

  // ---- LDS byte addresses of this lane's fragments
  uint32_t k_addr[STEPS], v_addr[DB];
#pragma unroll
  for (int st = 0; st < STEPS; ++st)
    k_addr[st] = lds_address(&s_kv[kg][0][0][0]) + 2 * (n * D + (((2 * st + h) ^ k_swizzle<D>(n)) << 3));
  const int i16 = lane & 15, gid = (lane >> 4) & 1;
  const int v_row = 4 * h + (i16 >> 2);
#pragma unroll
  for (int db = 0; db < DB; ++db)
    v_addr[db] = lds_address(&s_kv[kg][0][1][0]) +
                 2 * (v_row * D + (((4 * db + 2 * gid + ((i16 & 3) >> 1)) ^ v_swizzle<D>(v_row)) << 3) + 4 * (i16 & 1));

  f32x16 o[DB];
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = zero16;
  float m_run = kNegInf, l_run = 0.f;
  const float slack = kMaxSlack / p.scale_log2e;          // in raw score units

  if (STAGES == 2) wait_ids();

  if (STAGES == 2) {
    wait_vmcnt<0>();
    frontiers();
  }

  // Four groups: a SIMD holds a wave of group g and one of g + 2.  The upper groups run one barrier behind, so that one of
  // the two is at its matrix instructions while the other forms weights (a barrier more here for them, behind the sweep for
  // the others: all waves meet the same number).  us a step in step / behind: one stream of 900 keys 642 / 635, of 1,800
  // keys 883 / 865, 3 streams, 8/1 heads 617 / 608; one stream, 32/8 heads level.
  if (SPREAD && kg >= KG / 2) __syncthreads();
  const int n_trips = (kt_end - kt_begin + KG - 1) / KG;
  // The loop stands in a fixed place relative to the 64-byte lines that instructions are fetched by: the same instructions
  // 4 bytes off those of 8 bytes took 4-5 % longer (2 streams of 3,700 keys, 28/4 heads 90.8 us a layer instead of 86.6).
  asm volatile(".p2align 6");
  for (int trip = 0; trip < n_trips; ++trip, kt += KG) {
    wait_vmcnt<0>();
    __syncthreads();       // one stage: K has landed, every wave is done with the previous V; two: the tile, the other stage
    const bool here = kt < kt_end, computes = here && kt * kBN <= wave_max;
    const int stage = STAGES == 2 ? trip & 1 : 0;
    const uint32_t stage_off = stage * (2 * TILE * 2);
    if (STAGES == 2) {
      if (kt + KG < kt_end) {
        request(kt + KG, stage ^ 1, 0);
        request(kt + KG, stage ^ 1, 1);
      }
      load_ids(kt + 2 * KG);
    } else {
      if (here) request(kt, 0, 1);
      load_ids(kt + KG);                                 // (used after the S phase)
    }

    bf16x8 pb[2][2];
    if (computes) {
      const int j0 = kt * kBN;
      typedef __attribute__((address_space(3))) const cs::u32x4 lds_u32x4;
      auto k_frag = [&](int st, int kb) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, reinterpret_cast<lds_u32x4*>(static_cast<uintptr_t>(k_addr[st] + stage_off))[kb * 32 * D * 2 / 16]);
      };
      f32x16 sacc[2];
#pragma unroll
      for (int st = 0; st < STEPS; ++st)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag(st, kb), qf[st], st == 0 ? zero16 : sacc[kb], 0, 0, 0);
      if (D == 128) {
        // K fragments are read two steps ahead of their MFMAs (the scheduler would pull each read back to its use)
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int st = 0; st < STEPS - 2; ++st) {
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
      }
      // register r of block kb is key j0 + 32 kb + 8 (r / 4) + 4 h + r % 4 of query n
      if (j0 + kBN - 1 > wave_min) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = j0 + 32 * kb + 8 * (r / 4) + 4 * h + (r % 4);
            if (key > lim) sacc[kb][r] = kNegInf;
          }
      }
      float t_max = kNegInf;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) t_max = fmaxf(t_max, sacc[kb][r]);
      {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(t_max), __float_as_uint(t_max), false, false);
        t_max = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
      }
      if (__any(t_max > m_run + slack)) {
        const bool up = t_max > m_run + slack;
        const float m_new = up ? t_max : m_run;
        const float alpha = up ? __builtin_amdgcn_exp2f((m_run - m_new) * p.scale_log2e) : 1.f;
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      }
      const float m_scaled = (m_run == kNegInf ? 0.f : m_run) * p.scale_log2e;
      // Row sums of the rounded weights.  head_dim 64: the 4x4 matrix instruction with ones adds a lane's own four, since
      // v_dot2 waits for the matrix pipe.  us a step, two runs each (v_dot2 / this): 2 streams of 8,700 keys 1,773-1,780 /
      // 1,739-1,744, 4 streams of 1,000 keys 769-775 / 747-748, one 549-551 / 543-544, 12 of 1,100 level.  head_dim 128, with
      // twice the matrix work for each weight, keeps v_dot2: 4 streams 1,126 / 1,133, of 1,400 keys 1,402 / 1,417.
      f32x4 l_sum[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
      const s16x4 ones4 = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
          cs::u32x4 w;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float e0 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * mm + 2 * c], p.scale_log2e, -m_scaled));
            const float e1 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * mm + 2 * c + 1], p.scale_log2e, -m_scaled));
            const uint32_t pk = pack_bf16x2(e0, e1);
            if (D != 64)
              l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk),
                                                      __builtin_bit_cast(bf16x2, 0x3f803f80u), l_run, false);
            w[c] = pk;
          }
          pb[kb][mm] = __builtin_bit_cast(bf16x8, w);
          if (D == 64) {
            l_sum[0] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones4, __builtin_bit_cast(s16x4, cs::u32x2{w.x, w.y}), l_sum[0], 0, 0, 0);
            l_sum[1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones4, __builtin_bit_cast(s16x4, cs::u32x2{w.z, w.w}), l_sum[1], 0, 0, 0);
          }
        }
      if (D == 64) l_run += l_sum[0][0] + l_sum[1][0];
    }
    if (STAGES == 1) {
      wait_ids();
      wait_vmcnt<0>();
      __syncthreads();                     // V has landed; every wave is done with this K tile
      if (kt + KG < kt_end) request(kt + KG, 0, 0);
    }
    if (computes) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int mm = 0; mm < 2; ++mm)
#pragma unroll
          for (int db = 0; db < DB; ++db) {
            const int g0 = (32 * kb + 16 * mm) * D;
            const uint32_t a0 = v_addr[db] + stage_off;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(((lds_s16x4*)(static_cast<uintptr_t>(a0))) + g0 * 2 / 8);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(((lds_s16x4*)(static_cast<uintptr_t>(a0))) + (g0 + 8 * D) * 2 / 8);
            const s16x8 a = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pb[kb][mm], o[db], 0, 0, 0);
          }
    }
    if (STAGES == 2) wait_ids();
  }
  if (SPREAD && kg < KG / 2) __syncthreads();
  if constexpr (OWN) move.store(p);

  // ---- the groups' partial results (a group that met no visible key holds m = -inf, l = 0, O = 0).  Of two groups the
  //      second hands over to the first.  Of four, every wave leaves all of its columns in LDS and finishes one block of its
  //      rows' columns: two rounds of hand-over left six of the eight waves idle in the end.  us a step before / after (28
  //      layers): one stream of 900 keys, 28/4 heads 656 / 635, 3 streams, 8/1 heads 637 / 620, one stream of 1,800 keys
  //      902 / 885; one of 1,400 keys, and two groups merged this way, level.
  float l_tot = l_run + __shfl_xor(l_run, 32);
  if constexpr (SPREAD) {
    float4* s_o4 = reinterpret_cast<float4*>(&s_kv[0][0][0][0]);
    __syncthreads();                       // the tile buffers have been read
    float4* mine = s_o4 + (kg * ROWW + rw) * (DB * 4 * 64) + lane;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq)
        mine[(db * 4 + rq) * 64] = make_float4(o[db][4 * rq], o[db][4 * rq + 1], o[db][4 * rq + 2], o[db][4 * rq + 3]);
    s_ml[kg][rw][0][lane] = m_run;
    s_ml[kg][rw][1][lane] = l_tot;
    __syncthreads();
    float w[KG], m_all = kNegInf, l_all = 0.f;
#pragma unroll
    for (int g = 0; g < KG; ++g) m_all = fmaxf(m_all, s_ml[g][rw][0][lane]);
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      const float m = s_ml[g][rw][0][lane];
      w[g] = m == kNegInf ? 0.f : __builtin_amdgcn_exp2f((m - m_all) * p.scale_log2e);
      l_all = fmaf(w[g], s_ml[g][rw][1][lane], l_all);
    }
    const float inv = 1.f / l_all;
    uint16_t* orow = static_cast<uint16_t*>(p.out) + q_at + 32 * kg + 4 * h;
    const bool partial = SPLIT && n_pieces > 1;
    const int64_t prow = SPLIT ? (static_cast<int64_t>(block) * p.pieces + piece) * BM + rw * 32 + n : 0;
    if (partial && valid && kg == 0 && h == 0) *reinterpret_cast<float2*>(p.ws_ml + prow * 2) = make_float2(m_all, l_all);
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        const float4 x = s_o4[((g * ROWW + rw) * DB * 4 + kg * 4 + rq) * 64 + lane];
        t.x = fmaf(w[g], x.x, t.x); t.y = fmaf(w[g], x.y, t.y); t.z = fmaf(w[g], x.z, t.z); t.w = fmaf(w[g], x.w, t.w);
      }
      if (partial) {
        if (valid) *reinterpret_cast<float4*>(p.ws_o + prow * D + 32 * kg + 4 * h + 8 * rq) = t;
      } else if (valid) {                  // register r of a block is d = 32 db + 8 (r / 4) + 4 h + r % 4
        cs::u32x2 pk;
        pk.x = pack_bf16x2(t.x * inv, t.y * inv);
        pk.y = pack_bf16x2(t.z * inv, t.w * inv);
        *reinterpret_cast<cs::u32x2*>(orow + 8 * rq) = pk;
      }
    }
    return;
  }
  float* s_o = reinterpret_cast<float*>(&s_kv[0][0][0][0]);
#pragma unroll
  for (int half = KG / 2; half > 0; half >>= 1) {
    __syncthreads();                       // the tile buffers (or the previous hand-over) have been read
    if (kg >= half && kg < 2 * half) {
      float* at = s_o + ((kg - half) * ROWW + rw) * (DB * 16 * 64) + lane;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) at[(db * 16 + r) * 64] = o[db][r];
      s_ml[kg - half][rw][0][lane] = m_run;
      s_ml[kg - half][rw][1][lane] = l_tot;
    }
    __syncthreads();
    if (kg < half) {
      const float m_o = s_ml[kg][rw][0][lane], l_o = s_ml[kg][rw][1][lane];
      const float m_new = fmaxf(m_run, m_o);
      const float a = m_run == kNegInf ? 0.f : __builtin_amdgcn_exp2f((m_run - m_new) * p.scale_log2e);
      const float b = m_o == kNegInf ? 0.f : __builtin_amdgcn_exp2f((m_o - m_new) * p.scale_log2e);
      l_tot = fmaf(l_tot, a, l_o * b);
      m_run = m_new;
      const float* at = s_o + (kg * ROWW + rw) * (DB * 16 * 64) + lane;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = fmaf(o[db][r], a, at[(db * 16 + r) * 64] * b);
    }
  }

  // ---- normalise and store: register r of block db is d = 32 db + 8 (r / 4) + 4 h + r % 4
  if (kg == 0 && valid) {
    const float inv = 1.f / l_tot;
    uint16_t* orow = static_cast<uint16_t*>(p.out) + q_at;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        cs::u32x2 w;
        w.x = pack_bf16x2(o[db][4 * rq + 0] * inv, o[db][4 * rq + 1] * inv);
        w.y = pack_bf16x2(o[db][4 * rq + 2] * inv, o[db][4 * rq + 3] * inv);
        *reinterpret_cast<cs::u32x2*>(orow + 32 * db + 8 * rq + 4 * h) = w;
      }
  }
}

// Launches that leave CUs idle put some workgroups ahead of the row tiles, up to kWarmPerXcd an XCD, that read a word of each
// cache line of the keys and values past the first trip.  The row tiles of a (stream, kv head) sweep the same keys at the same
// pace, and every trip waited for a line's way from memory twice (K, then V): with the tiles in L2 already (the same tile asked
// for again and again) a step of one stream takes 506 us instead of 561, without any arithmetic 382 instead of 504.  What bounds it is its
// own chain: where the stream's entries are, the lines' places, the lines.  Which XCD a workgroup runs on (they go round robin)
// decides only whether this helps.  us a step of 28 layers, without / with: one
// stream of 900 keys, 28/4 heads 561 / 533, 32/8 665 / 612, 8/1 526 / 504, of 1,800 keys 782 / 704, of 450 424 / 417, two of 1,300 keys,
// 16/4 heads 848 / 792, of 900, 28/4 692 / 681; head_dim 64, one stream, 16/4 heads (24 layers) 414 / 412.
// Asked for by the row tiles' own threads, a line each behind the first trip's requests, the gain was half of that, and launches
// that fill the chip lost 2-5 %.
constexpr int kWarmPerXcd = 4;
template <int D, int KG, int THREADS>
__device__ __forceinline__ void warm_l2(const AttnParams& p) {
  constexpr int LINES = D * 4 / 128;     // 128-byte lines of a key and its value
  constexpr int AT_ONCE = 4;
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3, n_wg = p.n_warm >> 3;
  const int heads_apart = min(8, p.n_kv_heads & -p.n_kv_heads);      // of the kv heads that an XCD's row tiles have
  const int groups = min(n_wg, p.n_streams), parts = n_wg / groups, part = j / groups;
  if (part >= parts) return;
  uint32_t sum = 0;
  for (int s = j % groups; s < p.n_streams; s += groups) {
    const cs::u32x2 seen = p.ws_warm[s];
    const int rows = static_cast<int>(seen.y);
    const i32x2* own_t = reinterpret_cast<const i32x2*>(p.ws_own) + static_cast<int64_t>(s) * p.max_blocks;
    for (int kvh = xcd % heads_apart; kvh < p.n_kv_heads; kvh += heads_apart) {
      const uint16_t* kh = static_cast<const uint16_t*>(p.k) + static_cast<int64_t>(kvh) * p.stride_head;
      const uint16_t* vh = static_cast<const uint16_t*>(p.v) + static_cast<int64_t>(kvh) * p.stride_head;
      const int64_t own_at = static_cast<int64_t>(seen.x) * p.stride_slot + static_cast<int64_t>(kvh) * D;
      const uint16_t* kn = static_cast<const uint16_t*>(p.k_new) + own_at;
      const uint16_t* vn = static_cast<const uint16_t*>(p.v_new) + own_at;
      const int step = parts * THREADS;
      for (int i0 = KG * kBN * LINES + part * THREADS + static_cast<int>(threadIdx.x); i0 < rows * LINES; i0 += AT_ONCE * step) {
        i32x2 e[AT_ONCE];
        uint32_t got[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) e[u] = own_t[min((i0 + u * step) / LINES, rows - 1) / CS_KV_BLOCK];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
          const int row = min((i0 + u * step) / LINES, rows - 1), line = (i0 + u * step) % LINES, r = row % CS_KV_BLOCK;
          const OwnEntry at(static_cast<uint32_t>(e[u].x), static_cast<uint32_t>(e[u].y));
          const bool v = line >= LINES / 2;
          const uint16_t* src = at.own(r) ? (v ? vn : kn) + at.row_of(r) * p.stride_slot
                                          : (v ? vh : kh) + (static_cast<int64_t>(at.id) * CS_KV_BLOCK + r) * p.stride_slot;
          got[u] = *reinterpret_cast<const uint32_t*>(src + line % (LINES / 2) * 64);
        }
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) sum |= got[u];
      }
    }
  }
  asm volatile("" :: "v"(sum));          // (the loads are not to be left out)
}

template <int D, int ROWW, int KG, int STAGES, bool SPLIT = false, bool OWN = false>
__global__ __launch_bounds__(64 * ROWW * KG, D == 128 ? 2 : 4) void window_attn_bf16_tile_kernel(AttnParams p) {
  __shared__ TileStages<D, KG, STAGES> stages;
  int block = blockIdx.x;
  if constexpr (OWN && !SPLIT && KG > 1) {
    if (block < p.n_warm) {
      warm_l2<D, KG, 64 * ROWW * KG>(p);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (no scalar load is left in flight)
      return;
    }
    block -= p.n_warm;
  }
  attend_row_tile<D, ROWW, KG, STAGES, SPLIT, OWN>(p, block, stages);
}

// The parts of window_attn_own_rows_kernel, in workgroups.
constexpr int kListedStreams = 64;       // up to here a workgroup lists 16 row tiles of all kv heads, beyond one of one kv head
struct OwnParts {
  int64_t moves, entries, streams, row_tiles, tiles;
  __host__ __device__ __forceinline__ OwnParts(const AttnParams& p, int bm) {
    moves = (p.n_new * p.row_vecs + 63) / 64;
    entries = (static_cast<int64_t>(p.n_streams) * p.max_blocks + 3) / 4;
    streams = (p.n_streams + 63) / 64;
    row_tiles = p.n_q * p.group / bm + p.n_streams;       // of a kv head
    tiles = p.n_streams <= kListedStreams ? (row_tiles + 15) / 16 : row_tiles * p.n_kv_heads;
  }
};

// What the call that plans does for those that read their own rows, besides planning: the refresh write (of n_new rows, which
// it still needs itself), the table, and the row tiles of BM rows of a launch without a plan: first query token and
// rows of the stream (0: no tile), first row, kv head, frontier (the last cache entry that the last row sees, inside those
// that the stream defines; -1: none), stream.  Of every stream, its first query and the cache entries up to its last frontier.
// More than kRankedTiles row tiles of up to 64 streams are listed by their key tiles, longest first, so that what starts late or
// shares a CU is short (as find_row_tile has them, the last streams' longest sweeps start last).  us a step, by stream / by length,
// head_dim 64, 16 layers: 319 row tiles (14 streams, 8/1 heads) 423 / 368, 411 455 / 402, 420 (9 streams, 16/4) 424 / 408, 736 680 / 578,
// 1,491 (64 streams, 8/1) 1,058 / 908; head_dim 128: 368 of 64 rows 501 / 481, 500 525 / 481.  Fewer have a CU each, and are level
// (144 319 / 317, 304 of 64 rows 397 / 398) or faster by stream (204 333 / 339, 271 336 / 359, 288 of 64 rows 404 / 416).
// A tile's place is how many of the others go first: those of more key tiles, or of as many and ahead of it, which makes each
// place one tile's whatever the positions are.  A workgroup has the numbers to compare in LDS, and each lane counts a quarter of them for one
// of 16 tiles.  us that a call which plans takes more than refresh write and attention, a workgroup for each tile and kv head / this,
// head_dim 64: 64 streams of 8/1 heads 1,792 row tiles 15 / 10.5, 3,260 46 / 24, 9,655 174 / 47, of 16/4 7,168 34 / 2, 16 of 8/1 353 3.0 / 2.0.
constexpr int kRankedTiles = 300;
constexpr int kRankKeys = 1024;          // numbers in LDS at once
template <int BM>
__global__ __launch_bounds__(64) void window_attn_own_rows_kernel(AttnParams p) {
  __shared__ int s_tiles[64];
  struct Listed { int first, q0, rows, cap; };
  __shared__ Listed s_list[kListedStreams];
  __shared__ __attribute__((aligned(16))) uint32_t s_key[kRankKeys];
  const int lane = threadIdx.x, l16 = lane & 15, group16 = lane >> 4;
  // The parts are chains of dependent loads, so they go to workgroups of their own: the refresh write to the first, then four
  // entries of the table a workgroup, then the streams, then the row tiles (round again where the grid is smaller than that).
  // One after the other in each workgroup, and an entry a lane with a binary search, they took 7.9
  // us for one stream and 12.1 for 12 streams of head_dim 64 instead of 4.8 to 6.7 and 7.7 (a step 531 / 527 and 650 / 646).
  const OwnParts parts(p, BM);
  auto first_of = [&](int64_t before) { return (blockIdx.x + gridDim.x - before % gridDim.x) % gridDim.x; };
  OwnMove<64>().all(p);
  const int64_t n_entries = static_cast<int64_t>(p.n_streams) * p.max_blocks;
  for (int64_t e = first_of(parts.moves); e < parts.entries; e += gridDim.x) {
    const int64_t i = min(4 * e + group16, n_entries - 1);
    const int s = static_cast<int>(i / p.max_blocks), first = static_cast<int>(i - static_cast<int64_t>(s) * p.max_blocks) * CS_KV_BLOCK;
    const int len = p.kv_len[s] - first;
    const bool there = len > 0 && 4 * e + group16 < n_entries;     // (otherwise the stream's row of the block table ends before)
    const int q0 = p.cu_q[s], q1 = p.cu_q[s + 1];
    int lo = q0, hi = there ? q1 : q0;   // the first query at or past the block: 16 places at once, then between two of them
    while (__any(lo < hi)) {
      const int step = (hi - lo + 15) / 16, at = lo + l16 * step;
      const bool below = lo < hi && at < hi && p.q_pos[at] < first;
      const int n_below = __popc(static_cast<uint32_t>(__ballot(below) >> (16 * group16)) & 0xffffu);
      if (n_below == 0) {
        hi = lo;
      } else {
        hi = min(hi, lo + n_below * step);
        lo += (n_below - 1) * step + 1;
      }
    }
    uint32_t mask = 0;
    if (there && lo + l16 < q1) {
      // (a row without a slot, its position pulled back to the last that the stream's table covers, is not that entry's)
      const int at = p.q_pos[lo + l16] - first;
      mask = at < CS_KV_BLOCK && (!p.new_slot || p.new_slot[lo + l16] >= 0) ? 1u << at : 0u;
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) mask |= __shfl_xor(mask, off);
    if (there && l16 == 0) p.ws_own[i] = OwnEntry::packed(p.block_table[i], lo - q0, mask);
  }
  for (int64_t w = first_of(parts.moves + parts.entries); w < parts.streams; w += gridDim.x) {
    const int64_t s = 64 * w + lane;
    if (s >= p.n_streams) continue;
    const int q0 = p.cu_q[s], q1 = p.cu_q[s + 1];
    const int seen = q1 > q0 ? min(p.q_pos[q1 - 1] + 1, min(p.kv_len[s], p.max_blocks * CS_KV_BLOCK)) : 0;
    p.ws_warm[s] = cs::u32x2{static_cast<uint32_t>(q0), static_cast<uint32_t>(seen)};
  }
  const int64_t first_tile = first_of(parts.moves + parts.entries + parts.streams);
  auto list = [&](int64_t place, int q0, int rows, int r_tile, int kvh, int frontier, int s) {
    i32x4* d = reinterpret_cast<i32x4*>(p.ws_tiles + place * 8);
    d[0] = i32x4{q0, rows, r_tile, kvh};
    d[1] = i32x4{frontier, s, 0, 0};
  };
  if (p.n_streams > kListedStreams) {
    for (int64_t b = first_tile; b < parts.tiles; b += gridDim.x) {
      RowTile t = {};
      int frontier = -1;
      if (find_row_tile<BM, 1>(p, static_cast<int>(b), s_tiles, t)) frontier = tile_frontier<BM>(p, t);
      if (lane == 0) list(b, t.q0, t.rows_total, t.r_tile, t.kvh, frontier, t.s);
      __syncthreads();
    }
  } else if (first_tile < parts.tiles) {
    Listed mine = {};
    if (lane < p.n_streams) {
      mine.q0 = p.cu_q[lane];
      mine.rows = (p.cu_q[lane + 1] - mine.q0) * p.group;
      mine.cap = min(p.kv_len[lane], p.max_blocks * CS_KV_BLOCK) - 1;
    }
    const int tiles = (mine.rows + BM - 1) / BM;
    int incl = tiles;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int below = __shfl_up(incl, off);
      incl += lane >= off ? below : 0;
    }
    mine.first = incl - tiles;
    s_list[lane] = mine;
    const int row_tiles = static_cast<int>(parts.row_tiles), n_found = min(__shfl(incl, 63), row_tiles);
    const bool ranked = static_cast<int64_t>(n_found) * p.n_kv_heads > kRankedTiles;
    __syncthreads();
    // the query of the last row of the tile that begins at r_tile
    auto last_query = [&](int q0, int rows, int r_tile) { return q0 + (min(r_tile + BM, rows) - 1) / p.group; };
    struct Found { int s, q0, rows, r_tile, frontier; };
    auto find = [&](int x) {               // row tile x of all streams, the last of a stream's rows first
      int s = 0;                           // the last stream that begins at or before x
#pragma unroll
      for (int step = 32; step > 0; step >>= 1) s += s + step < p.n_streams && s_list[s + step].first <= x ? step : 0;
      const Listed l = s_list[s];
      const int r_tile = (l.first + (l.rows + BM - 1) / BM - 1 - x) * BM;
      return Found{s, l.q0, l.rows, r_tile, min(p.q_pos[last_query(l.q0, l.rows, r_tile)], l.cap)};
    };
    // to rank: tile j of stream i % lanes is number i of its round, j going up with i / lanes
    const int lanes = p.n_streams > 1 ? 1 << (32 - __clz(p.n_streams - 1)) : 1, apart = 64 / lanes;
    const Listed of = s_list[lane % lanes];
    const int of_tiles = (of.rows + BM - 1) / BM;
    int most = of_tiles;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off));
    // (ranked: row tiles times key tiles are below 2^20, own_row_tile)
    auto key_of = [](int x, int frontier) { return static_cast<uint32_t>(max(frontier, -1) / kBN) << 20 | (0xfffffu - x); };
    for (int64_t b = first_tile; b < parts.tiles; b += gridDim.x) {
      const int x = static_cast<int>(b) * 16 + l16;
      Found t = {0, 0, 0, 0, -1};
      if (x < n_found) t = find(x);
      int place = x;
      if (ranked) {
        constexpr int AT_ONCE = 4;
        const uint32_t key = key_of(x, t.frontier);
        int ahead = 0;
        for (int j0 = 0; j0 < most; j0 += kRankKeys / lanes) {
          const int n = min(kRankKeys, (most - j0) * lanes);
          __syncthreads();
          for (int i = lane; i < n + lane; i += 64 * AT_ONCE) {      // (all positions asked for before the first store)
            int its[AT_ONCE];
#pragma unroll
            for (int u = 0; u < AT_ONCE; ++u) {
              const int j = j0 + i / lanes + u * apart;
              its[u] = p.q_pos[j < of_tiles ? last_query(of.q0, of.rows, (of_tiles - 1 - j) * BM) : 0];
            }
#pragma unroll
            for (int u = 0; u < AT_ONCE; ++u) {
              const int j = j0 + i / lanes + u * apart, o = of.first + j;
              if (i + 64 * u < kRankKeys) s_key[i + 64 * u] = j < of_tiles && o < n_found ? key_of(o, min(its[u], of.cap)) : 0u;
            }
          }
          __syncthreads();
#pragma unroll 4
          for (int i = 4 * group16; i < n; i += 16) {
            const cs::u32x4 o = *reinterpret_cast<const cs::u32x4*>(s_key + i);
            ahead += (o.x > key ? 1 : 0) + (o.y > key ? 1 : 0) + (o.z > key ? 1 : 0) + (o.w > key ? 1 : 0);
          }
        }
        ahead += __shfl_xor(ahead, 16);
        ahead += __shfl_xor(ahead, 32);
        if (x < n_found) place = ahead;
      }
      for (int kvh = group16; kvh < p.n_kv_heads && x < row_tiles; kvh += 4)
        list(static_cast<int64_t>(place) * p.n_kv_heads + kvh, t.q0, t.rows, t.r_tile, kvh, t.frontier, t.s);
    }
  }
  wait_scalar();                         // (no scalar load is left in flight)
}

// =============================================================================================
// bf16 / head_dim 128: planned, persistent kernel
//
// A small planning kernel turns (cu_q, q_pos) into a list of work items, an item being one
// (stream, kv head, 128-row tile, key range), and deals the items to the 8 XCDs: all items of one
// (stream, kv head) pair go to one XCD (their K/V tiles then meet in that XCD's L2), pairs are
// dealt to XCDs in boustrophedon order of decreasing work, and every XCD's list is sorted by
// decreasing key-range length.  The plan depends only on cu_q and q_pos, so one plan serves
// every decoder layer of a step.
//
// The attention kernel is persistent: workgroup b serves XCD b % 8 (workgroups are dealt to XCDs round robin by the
// hardware) and follows its chain of items.  It takes the two row tiles of a unit, which follow each other there and begin at
// the same key tile, as ONE job of 256 rows: every K/V tile that it fetches, and every fragment
// that a wave reads from LDS, then serves twice the rows (see window_attn_bf16_stream_kernel).  The plan makes
// chains of units: two neighbouring row tiles of a stream counted from its end, or, of a pair whose row tiles go
// to all XCDs, two that the same XCD takes.  For streams of few rows a kernel with two workgroups per CU takes every row tile
// as a job of its own (window_attn_bf16_rows32_kernel).

// Item descriptor: 8 ints.  [0] first query token of the stream, [1] rows of the stream (tokens x
// heads per kv group), [2] first row of the tile, [3] kv head | stream << 8, [4] highest visible
// cache index among the tile's rows, [5] key tiles [begin, end) as begin | end << 16, [6] index of
// the item the same workgroup takes next (-1: none), [7] first row of the item's partial result in the workspace (an even
// number), or -2 when the item covers the whole sweep and writes `out`; plus 1, unless it is the second of its unit.
// Plan header (ints): [0..8] list offsets per XCD, [9] row tiles, [16..23] end item,
// then one 32-int entry per workgroup j of XCD x at [32 + 32 (64 x + j)]: [0] its first item (-1: none),
// [8..15] a copy of that item's descriptor (all that the workgroup reads of its entry).
// Entries from kWorkgroupsPerXcd on name no item but where two workgroups share a CU (window_attn_bf16_rows32_kernel).
constexpr int kSlotsPerXcd = 64;      // header entries per XCD
constexpr int kWorkgroupsPerXcd = 32; // persistent workgroups per XCD: one per CU
constexpr int kHdrEndItem = 16, kHdrHeads = 32;
constexpr int kHdrEntryInts = 32;
constexpr int kHdrStatus = 14;        // status word of the fused launch's launch-wide wait
// Behind the entries, the counters of that wait, 256 bytes apart so that they sit in different
// memory channels: kSyncGroups group counters, the counter of finished groups, the release word.
constexpr int kSyncGroups = 16, kSyncPitch = 64;
constexpr int kHdrSyncBase = (kHdrHeads + kHdrEntryInts * 8 * kSlotsPerXcd + kSyncPitch - 1) / kSyncPitch * kSyncPitch;
constexpr int kSyncInts = (kSyncGroups + 2) * kSyncPitch;
constexpr int kPlanHeaderInts = kHdrSyncBase + kSyncInts;
// What a job costs besides its key tiles, in half tiles, for the planner's balance: measured 7,300-8,900 cycles (results of
// the job before, queries, first scores) beside 1,510-1,730 for a half tile.  3 instead: 2,100 tokens over 17,600 keys 258 against
// 244 us a layer, over 6,000 keys 111 against 104.
constexpr int kItemFixedCostHalves = 5;
constexpr int kPlanThreads = 1024;
constexpr int kSoloFixedCostHalves = 3;  // ... and an item of the kernel of 32 rows a wave
constexpr int kDealAtOnce = 72;       // units of an XCD that are dealt by length over the whole list (at most two a lane)
constexpr int kSortMax = 2048;        // streams sorted by work in LDS; beyond, stream order is kept

struct PlanParams {
  const int32_t* __restrict__ cu_q;
  const int32_t* __restrict__ q_pos;
  const int32_t* __restrict__ kv_len;
  int32_t max_blocks;
  int32_t n_streams, group, n_kv_heads, max_tiles, r_cap, bm, n_slots, hist_pitch;   // n_slots: workgroups per XCD
  int32_t solo;         // 1: every row tile is a unit of its own (window_attn_bf16_rows32_kernel)
  int32_t* header;      // [kPlanHeaderInts]
  int32_t* items;       // [items_cap][8]
  int32_t* rt_desc;     // [r_cap * n_kv_heads][8]: q0, rows_total, r_tile, kvh, n_split
  int32_t* st_toff;     // [n_streams + 1] first row tile of each stream
  int32_t* st_uoff;     // [n_streams] first unit of each stream
  int32_t* st_work;     // [n_streams] key tiles summed over the stream's row tiles
  int32_t* st_rank;     // [n_streams] rank by decreasing work
  int32_t* rt_stream;   // [r_cap]
  int32_t* rt_wgmax;    // [r_cap]
  int32_t* un_head;     // [r_cap] first row tile of each unit
  int32_t* hist;        // [8][hist_pitch] items per (XCD, bucket), then list cursors
  int32_t span;         // 1: sweeps are cut into contiguous spans of equal cost (few, long sweeps)
  int32_t pref_pitch;   // ints per XCD in sw_pref
  int32_t* sw_pref;     // [8][pref_pitch] span plan: cost prefix of each XCD's sweeps
};

// Exclusive prefix sum over the THREADS threads of the planning workgroup.
template <int THREADS>
__device__ __forceinline__ int plan_block_scan(int v, int* s_wave, int& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(incl, off);
    if (lane >= off) incl += t;
  }
  __syncthreads();                       // s_wave may still be read from a previous call
  if (lane == 63) s_wave[w] = incl;
  __syncthreads();
  int base = 0, sum = 0;
  for (int i = 0; i < THREADS / 64; ++i) {
    const int t = s_wave[i];
    if (i < w) base += t;
    sum += t;
  }
  total = sum;
  return base + incl - v;
}

// Rows (query tokens x query heads of one kv group) of a stream; a stream whose block-table row
// defines no entry (kv_len <= 0) has nothing to attend to and gets no row tiles.
__device__ __forceinline__ int plan_stream_rows(const PlanParams& pp, int s) {
  return pp.kv_len[s] > 0 ? (pp.cu_q[s + 1] - pp.cu_q[s]) * pp.group : 0;
}

__device__ __forceinline__ int plan_xcd_of_pair(int pair) {
  const int round = pair >> 3, pos = pair & 7;
  return (round & 1) ? 7 - pos : pos;
}

// Span plan, for launches with few (row tile, kv head) sweeps, some of them long (one stream with
// a long window; any small batch).  Dealing whole sweeps, or fixed key ranges of them, to workgroups
// leaves the workgroups with unequal totals because the pieces are coarse next to a workgroup's
// share.  Here every XCD gets every eighth sweep (sweep = row tile * kv heads + kv head, so with
// four or eight kv heads an XCD serves one kv head), lays its sweeps end to end, and the sequence
// is cut into one contiguous span per workgroup, of equal COST: 2 n_kt + kItemFixedCostHalves per
// sweep, in half key tiles.  A sweep is that of a unit of two row tiles, the longer one's; the shorter one
// takes part as far as it goes.  A sweep that a cut crosses becomes
// several items whose partial results the merge kernel combines; cuts closer than kMinPieceTiles to
// a sweep's end move onto it.  Items of a workgroup are consecutive in the list, pieces of a sweep
// are consecutive too, and the position of an item in the list also names its partial-result slot.
constexpr int kMinSpanTiles = 3;     // fewer workgroups are used rather than give one less than this
constexpr int kMinPieceTiles = 2;

constexpr int kSpanPrefInLds = 8 * 136;   // the span plan runs with fewer than 1,024 sweeps: at most 130 ints per XCD

// What a unit's items need to know: first query token, rows of the stream, first row and stream of its first row tile, the
// frontiers of its two (-1: there is no second).
struct PlanUnit { int q0, rows, r_tile, stream, wg_max, wg_max2; };
constexpr int kSpanUnits = 1024;         // the span plan runs with fewer than 1,024 row tiles

__device__ void plan_spans(const PlanParams& pp, int n_rt, int n_un, int* s_wave, int (*s_cut)[kSlotsPerXcd + 1], int* s_pref, PlanUnit* s_unit) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n_kv = pp.n_kv_heads;
  const int n_sw = n_un * n_kv;
  auto tiles_of = [&](int wg_max) { return wg_max < 0 ? 0 : wg_max / kBN + 1; };
  for (int u = tid; u < n_un; u += kPlanThreads) {
    const int r = pp.un_head[u], st = pp.rt_stream[r], t = r - pp.st_toff[st];
    s_unit[u] = PlanUnit{pp.cu_q[st], plan_stream_rows(pp, st), t * pp.bm, st, pp.rt_wgmax[r], t > 0 ? pp.rt_wgmax[r - 1] : -1};
  }
  __syncthreads();
  auto sweep_tiles = [&](int sw) { return tiles_of(s_unit[sw / n_kv].wg_max); };
  // ---- cost prefix of every XCD's sweeps (one wave per XCD)
  if (w < 8) {
    int32_t* pref = pp.sw_pref + w * pp.pref_pitch;
    const int n_x = (n_sw - w + 7) >> 3;
    int run = 0;
    if (lane == 0) pref[0] = 0;
    for (int i0 = 0; i0 < n_x; i0 += 64) {
      const int i = i0 + lane;
      const int v = i < n_x ? 2 * sweep_tiles(8 * i + w) + kItemFixedCostHalves : 0;
      int incl = v;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(incl, off);
        if (lane >= off) incl += t;
      }
      if (i < n_x) pref[i + 1] = run + incl;
      run += __shfl(incl, 63);
    }
  }
  __threadfence_block();
  __syncthreads();
  // the searches below read the prefixes many times: keep them in LDS when they fit (they do for
  // every launch the host routes here; the global copy serves the general case)
  const bool in_lds = 8 * pp.pref_pitch <= kSpanPrefInLds;
  if (in_lds)
    for (int i = tid; i < 8 * pp.pref_pitch; i += kPlanThreads)
      s_pref[i] = __hip_atomic_load(&pp.sw_pref[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  // Position helpers of XCD x.  A position is a tile count from the start of the XCD's sequence.
  auto n_of = [&](int x) { return (n_sw - x + 7) >> 3; };
  auto cost_pref = [&](int x, int i) {
    return in_lds ? s_pref[x * pp.pref_pitch + i]
                  : __hip_atomic_load(&pp.sw_pref[x * pp.pref_pitch + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto tile_pref = [&](int x, int i) { return (cost_pref(x, i) - kItemFixedCostHalves * i) >> 1; };
  auto sweep_at_tile = [&](int x, int pos) {      // largest i with tile_pref(i) <= pos (pos < total tiles)
    int lo = 0, hi = n_of(x);
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (tile_pref(x, mid) <= pos) lo = mid; else hi = mid;
    }
    return lo;
  };
  // ---- cuts: thread (x, j) places the start of workgroup j's span
  const int x = tid >> 6, j = tid & 63;          // threads 0..511: one per (XCD, workgroup)
  const int n_wg = pp.n_slots;
  if (tid < 512) {
    const int n_x = n_of(x);
    const int total_tiles = n_x > 0 ? tile_pref(x, n_x) : 0;
    const int total_cost = n_x > 0 ? cost_pref(x, n_x) : 0;
    const int spans = total_tiles > 0 ? max(1, min(n_wg, total_tiles / kMinSpanTiles)) : 0;
    int cut = total_tiles;
    if (j < spans) {
      const int64_t c = static_cast<int64_t>(total_cost) * j / spans;   // cost position
      int lo = 0, hi = n_x;                       // largest i with cost_pref(i) <= c
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cost_pref(x, mid) <= c) lo = mid; else hi = mid;
      }
      const int len = sweep_tiles(8 * lo + x);
      int o = static_cast<int>(c - cost_pref(x, lo) - kItemFixedCostHalves + 1) >> 1;
      o = max(0, min(o, len));
      if (o < kMinPieceTiles) o = 0;
      if (len - o < kMinPieceTiles) o = len;
      cut = j == 0 ? 0 : tile_pref(x, lo) + o;
    }
    s_cut[x][j] = cut;
    if (j == 0) s_cut[x][kSlotsPerXcd] = total_tiles;
  }
  __syncthreads();
  // ---- items per workgroup, their positions in the list
  int i_lo = 0, i_hi = -1, lo_t = 0, hi_t = 0;
  if (tid < 512) {
    lo_t = s_cut[x][j];
    hi_t = s_cut[x][j + 1];
    if (hi_t > lo_t) {
      i_lo = sweep_at_tile(x, lo_t);
      i_hi = sweep_at_tile(x, hi_t - 1);
    }
  }
  // the piece [kb, ke) of sweep i that belongs to this workgroup, and the key tiles of its second row tile (0: none)
  auto piece = [&](int i, int& kb, int& ke, int& n_kt, int& n_kt2) {
    const int begin = tile_pref(x, i);
    n_kt = tile_pref(x, i + 1) - begin;
    kb = max(lo_t, begin) - begin;
    ke = min(hi_t, begin + n_kt) - begin;
    n_kt2 = tiles_of(s_unit[(8 * i + x) / n_kv].wg_max2);
  };
  int count = 0;
  for (int i = i_lo; i <= i_hi; ++i) {
    int kb, ke, n_kt, n_kt2;
    piece(i, kb, ke, n_kt, n_kt2);
    count += kb < n_kt2 ? 2 : 1;
  }
  int total_items;
  const int first = plan_block_scan<kPlanThreads>(tid < 512 ? count : 0, s_wave, total_items);
  if (tid < 512 && j == 0) pp.header[x] = first;
  if (tid == 0) {
    pp.header[8] = total_items;
    pp.header[9] = n_rt * n_kv;
    for (int i = 10; i < kHdrHeads; ++i) pp.header[i] = 0;
    pp.header[kHdrEndItem + 4] = -1;                    // end item: no key tiles, nothing visible
    pp.header[kHdrEndItem + 6] = -1;
    pp.header[kHdrEndItem + 7] = -1;
  }
  for (int i = tid; i < kSyncInts; i += kPlanThreads) pp.header[kHdrSyncBase + i] = 0;
  for (int i = n_rt * n_kv + tid; i < pp.r_cap * n_kv; i += kPlanThreads)
    pp.rt_desc[static_cast<int64_t>(i) * 8 + 4] = 0;
  if (tid >= 512) return;
  // ---- write the items of workgroup (x, j) and its header entry
  int32_t d_first[8] = {0, 0, 0, 0, -1, 0, -1, -1};     // the end item
  int pos = first;
  for (int i = i_lo; i <= i_hi; ++i) {
    const int sw = 8 * i + x;
    const int u = sw / n_kv, kvh = sw - u * n_kv;
    const PlanUnit un = s_unit[u];
    const int s = un.stream;
    int kb, ke, n_kt, n_kt2;
    piece(i, kb, ke, n_kt, n_kt2);
    const bool two = kb < n_kt2;
    int pieces = 1, pieces2 = 1;                         // of the sweep's two row tiles
    if (kb == 0 && ke < n_kt) {
      const int begin = tile_pref(x, i);
      for (int k = j + 1; k < kSlotsPerXcd; ++k) {
        const int c = s_cut[x][k];
        if (c >= begin + n_kt) break;
        if (c <= begin || c == s_cut[x][k - 1]) continue;
        ++pieces;
        pieces2 += c < begin + n_kt2 ? 1 : 0;
      }
    }
    for (int second = 0; second < (two ? 2 : 1); ++second) {
      const int n_mine = second ? n_kt2 : n_kt, ke_mine = min(ke, n_mine);
      const bool split = kb > 0 || ke_mine < n_mine;
      int32_t d[8] = {un.q0, un.rows, un.r_tile - second * pp.bm, kvh | (s << 8), second ? un.wg_max2 : un.wg_max, kb | (ke_mine << 16),
                      i < i_hi || second < (two ? 1 : 0) ? pos + 1 : -1, (split ? pos * pp.bm : -2) | (second ? 0 : 1)};
      int32_t* it = pp.items + static_cast<int64_t>(pos) * 8;
#pragma unroll
      for (int k = 0; k < 8; ++k) it[k] = d[k];
      if (pos == first) {
#pragma unroll
        for (int k = 0; k < 8; ++k) d_first[k] = d[k];
      }
      // the sweep's first piece describes it to the merge kernel: piece c of either row tile stands at the list
      // position [5] + c + min(c, [6]), since the pieces of the two alternate until the second's are used up
      if (kb == 0) {
        int32_t* rd = pp.rt_desc + static_cast<int64_t>((pp.un_head[u] - second) * n_kv + kvh) * 8;
        rd[0] = un.q0; rd[1] = un.rows; rd[2] = un.r_tile - second * pp.bm; rd[3] = kvh; rd[4] = second ? pieces2 : pieces; rd[5] = pos;
        rd[6] = n_kt2 > 0 ? pieces2 : 0;
      }
      ++pos;
    }
  }
  int32_t* hd = pp.header + kHdrHeads + kHdrEntryInts * (x * kSlotsPerXcd + j);
  hd[0] = count > 0 ? first : -1;
  for (int i = 0; i < 8; ++i) hd[8 + i] = d_first[i];
}

// What planning keeps in LDS.
struct PlanLds {
  unsigned long long key[kSortMax];
  int wave[kPlanThreads / 64];
  int list_off[9];
  int left_tiles[8], left_end[8];   // pairs left over by whole rounds: row tiles; last row tile + pair
  int by_rank[8][64];      // deal: lane (and length) of the item of each rank, per XCD
  int units[8];            // units in each XCD's list
  int deal[8][128];        // deal at once: units by length
};
static_assert(kDealAtOnce <= 128 && sizeof(int4) * 8 * 128 <= sizeof(PlanLds::key), "the deal keeps its units there");
// ... and the span plan besides
struct SpanLds {
  PlanUnit unit[kSpanUnits];
  int cut[8][kSlotsPerXcd + 1];     // first tile position of every workgroup's span
};

template <int THREADS, bool SPAN>
__device__ __forceinline__ void plan_work(const PlanParams& pp, PlanLds& lds, SpanLds* span_lds) {
  auto& s_key = lds.key;
  auto& s_wave = lds.wave;
  auto& s_list_off = lds.list_off;
  auto& s_left_tiles = lds.left_tiles;
  auto& s_left_end = lds.left_end;
  auto& s_by_rank = lds.by_rank;
  auto& s_units = lds.units;
  auto& s_deal = lds.deal;
  const int tid = threadIdx.x;
  const int hist_pitch = pp.hist_pitch;

  // ---- clear counters; row tiles per stream
  if (tid < 8) s_units[tid] = 0;
  for (int i = tid; i < 8 * hist_pitch; i += THREADS) pp.hist[i] = 0;
  int* s_toff = reinterpret_cast<int*>(s_key);           // the streams' first row tiles are searched in LDS if they fit
  const bool in_lds = pp.n_streams <= 2 * kSortMax;
  int* s_work = &s_deal[0][0];                           // ... and their work is summed up there
  const bool work_in_lds = pp.n_streams <= 8 * 128;
  int carry = 0;
  for (int s0 = 0; s0 < pp.n_streams; s0 += THREADS) {
    const int s = s0 + tid;
    int tiles = 0;
    if (s < pp.n_streams) {
      const int rows = plan_stream_rows(pp, s);
      tiles = (rows + pp.bm - 1) / pp.bm;
      if (work_in_lds) s_work[s] = 0;
      else pp.st_work[s] = 0;
    }
    int total;
    const int excl = plan_block_scan<THREADS>(tiles, s_wave, total);
    if (s < pp.n_streams) pp.st_toff[s] = carry + excl;
    if (s < pp.n_streams && in_lds) s_toff[s] = carry + excl;
    carry += total;
  }
  const int n_rt = carry;                // row tiles per kv head
  if (tid == 0) pp.st_toff[pp.n_streams] = n_rt;
  // units: two neighbouring row tiles of a stream, counted from its end (an odd one out is the stream's first)
  int n_un = 0;
  for (int s0 = 0; s0 < pp.n_streams; s0 += THREADS) {
    const int s = s0 + tid;
    const int tiles = s < pp.n_streams ? (plan_stream_rows(pp, s) + pp.bm - 1) / pp.bm : 0;
    int total;
    const int excl = plan_block_scan<THREADS>((tiles + 1) >> 1, s_wave, total);
    if (s < pp.n_streams) pp.st_uoff[s] = n_un + excl;
    n_un += total;
  }
  __threadfence_block();
  __syncthreads();

  // ---- per row tile: its stream, its causal frontier; work per stream
  for (int r = tid; r < n_rt; r += THREADS) {
    int lo = 0, hi = pp.n_streams;       // last stream whose first row tile is <= r
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if ((in_lds ? s_toff[mid] : pp.st_toff[mid]) <= r) lo = mid; else hi = mid;
    }
    const int s = lo;
    const int t = r - pp.st_toff[s];
    const int q0 = pp.cu_q[s];
    const int rows = plan_stream_rows(pp, s);
    const int last_row = min((t + 1) * pp.bm, rows) - 1;
    // the tile's frontier, kept inside the entries the stream's block-table row defines
    const int wg_max = max(0, min(pp.q_pos[q0 + last_row / pp.group], min(pp.kv_len[s], pp.max_blocks * CS_KV_BLOCK) - 1));
    pp.rt_stream[r] = s;
    pp.rt_wgmax[r] = wg_max;
    const int tiles_s = pp.st_toff[s + 1] - pp.st_toff[s];
    if (((tiles_s - 1 - t) & 1) == 0) pp.un_head[pp.st_uoff[s] + (t >> 1)] = r;
    if (work_in_lds) atomicAdd(&s_work[s], max(wg_max, 0) / kBN + 1);
    else atomicAdd(&pp.st_work[s], max(wg_max, 0) / kBN + 1);
  }
  __threadfence_block();
  __syncthreads();

  if constexpr (SPAN) {
    if (pp.span) {
      plan_spans(pp, n_rt, n_un, s_wave, span_lds->cut, reinterpret_cast<int*>(s_key), span_lds->unit);    // s_key is unused on this route
      return;
    }
  }

  // ---- rank streams by decreasing work (ties: stream order)
  if (pp.n_streams <= kSortMax) {
    int n_sort = 1;
    while (n_sort < pp.n_streams) n_sort <<= 1;
    for (int i = tid; i < n_sort; i += THREADS)
      s_key[i] = i < pp.n_streams
                     ? (static_cast<unsigned long long>(0x7fffffff - (work_in_lds ? s_work[i] : __hip_atomic_load(&pp.st_work[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) << 32) | static_cast<unsigned>(i)
                     : ~0ull;
    __syncthreads();
    for (int k = 2; k <= n_sort; k <<= 1)
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = tid; i < n_sort; i += THREADS) {
          const int partner = i ^ j;
          if (partner > i) {
            const unsigned long long a = s_key[i], b = s_key[partner];
            const bool up = (i & k) == 0;
            if ((a > b) == up) { s_key[i] = b; s_key[partner] = a; }
          }
        }
        __syncthreads();
      }
    for (int i = tid; i < pp.n_streams; i += THREADS)
      pp.st_rank[static_cast<unsigned>(s_key[i] & 0xffffffffu)] = i;
  } else {
    for (int i = tid; i < pp.n_streams; i += THREADS) pp.st_rank[i] = i;
  }
  __threadfence_block();
  __syncthreads();

  // ---- order of an XCD's list.  With enough (stream, kv head) pairs to give every XCD two, a pair
  //      goes to one XCD whole (boustrophedon deal by rank) and its row tiles stay together in the
  //      list, pairs by rank, longest row tile first: the workgroups of an XCD then sweep the K/V
  //      of few pairs at a time and share them in its L2 (an order by length alone re-read K/V
  //      2.5 times from HBM).  Otherwise items are dealt round robin and ordered by length.
  //      bucket = position class in the list (counting sort), XCD chosen alongside.
  //      Pairs beyond the last whole round of eight (the ones with the least work) have their row
  //      tiles dealt to all XCDs instead, behind the whole pairs: one XCD's list would carry a pair
  //      more than another's (20 pairs: three against two).  On its XCD a row tile's place among
  //      them goes by its distance from its stream's end, longest first.  us a layer without /
  //      with: 5 streams of 3,200 keys, 4 kv heads 171.9 / 151.1; 25 streams of 2,900 keys, one
  //      kv head 165.0 / 155.9; 21 streams of 1,000 keys, 4 kv heads 98.4 / 96.1.
  const int n_pairs = pp.n_streams * pp.n_kv_heads, whole_pairs = n_pairs & ~7;
  const bool grouped = n_pairs >= 16;
  if (grouped && tid < n_pairs - whole_pairs) {
    const int rank = (whole_pairs + tid) / pp.n_kv_heads;
    const int s = pp.n_streams <= kSortMax ? static_cast<int>(s_key[rank] & 0xffffffffu) : rank;
    s_left_tiles[tid] = pp.st_toff[s + 1] - pp.st_toff[s];
    s_left_end[tid] = pp.st_toff[s + 1] - 1 + whole_pairs + tid;
  }
  __syncthreads();
  // the row tiles of these pairs that XCD x takes before the given one (`level` from its stream's end)
  auto left_before = [&](int pair, int level, int x) {
    int at = 0;
    for (int i = 0; i < n_pairs - whole_pairs; ++i) {
      const int nearer = min(s_left_tiles[i], level + (i < pair - whole_pairs ? 1 : 0));
      const int first = (s_left_end[i] - x) & 7;           // level of the pair's first tile on this XCD; every eighth follows
      at += nearer > first ? (nearer - first + 7) >> 3 : 0;
    }
    return at;
  };
  auto place = [&](int r, int s, int kvh, int& bucket) {
    if (grouped) {
      const int pair = pp.st_rank[s] * pp.n_kv_heads + kvh;
      bucket = pair >> 3;
      return pair < whole_pairs ? plan_xcd_of_pair(pair) : (r + pair) & 7;
    }
    // (both row tiles of a unit by the longer one)
    const int head = r + ((pp.st_toff[s + 1] - 1 - r) & 1);
    bucket = pp.max_tiles + 1 - min(max(pp.rt_wgmax[head], 0) / kBN + 1, pp.max_tiles + 1);
    return ((pp.st_uoff[s] + ((head - pp.st_toff[s]) >> 1)) * pp.n_kv_heads + kvh) & 7;
  };
  for (int r = tid; r < n_rt; r += THREADS)
    for (int kvh = 0; kvh < pp.n_kv_heads; ++kvh) {
      int bucket;
      const int x = place(r, pp.rt_stream[r], kvh, bucket);
      atomicAdd(&pp.hist[x * hist_pitch + bucket], 1);
    }
  __threadfence_block();
  __syncthreads();

  // ---- per XCD (one wave each): first list position of every bucket
  {
    const int lane = tid & 63;
    for (int w = tid >> 6; w < 8; w += THREADS / 64) {
      int* hx = pp.hist + w * hist_pitch;
      int run = 0;
      for (int k0 = 0; k0 < hist_pitch; k0 += 64) {
        const int k = k0 + lane;
        const int v = k < hist_pitch ? __hip_atomic_load(&hx[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        int incl = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int t = __shfl_up(incl, off);
          if (lane >= off) incl += t;
        }
        if (k < hist_pitch) hx[k] = run + incl - v;
        run += __shfl(incl, 63);
      }
      if (lane == 0) s_list_off[w + 1] = run;          // list length for now
    }
  }
  __syncthreads();
  if (tid == 0) {
    s_list_off[0] = 0;
    for (int x = 0; x < 8; ++x) s_list_off[x + 1] += s_list_off[x];
    for (int x = 0; x < 9; ++x) pp.header[x] = s_list_off[x];
    pp.header[9] = n_rt * pp.n_kv_heads;
    for (int i = 10; i < kHdrHeads; ++i) pp.header[i] = 0;
    pp.header[kHdrEndItem + 4] = -1;                    // end item: no key tiles, nothing visible
    pp.header[kHdrEndItem + 6] = -1;
    pp.header[kHdrEndItem + 7] = -1;
  }
  for (int i = tid; i < kSyncInts; i += THREADS) pp.header[kHdrSyncBase + i] = 0;
  __threadfence_block();
  __syncthreads();

  // ---- write the items (row-tile slots beyond the planned ones are marked unsplit, so that the
  //      merge kernel needs no other bound than the size of its grid)
  for (int i = n_rt * pp.n_kv_heads + tid; i < pp.r_cap * pp.n_kv_heads; i += THREADS)
    pp.rt_desc[static_cast<int64_t>(i) * 8 + 4] = 0;
  for (int r = tid; r < n_rt; r += THREADS) {
    const int s = pp.rt_stream[r];
    const int t = r - pp.st_toff[s];
    const int q0 = pp.cu_q[s];
    const int rows = plan_stream_rows(pp, s);
    const int level = pp.st_toff[s + 1] - 1 - r;         // row tiles from the stream's end
    for (int kvh = 0; kvh < pp.n_kv_heads; ++kvh) {
      int32_t* rd = pp.rt_desc + static_cast<int64_t>(r * pp.n_kv_heads + kvh) * 8;
      rd[0] = q0; rd[1] = rows; rd[2] = t * pp.bm; rd[3] = kvh; rd[4] = 1;
      if (!grouped && (level & 1)) continue;             // written with the other row tile of its unit
      int bucket;
      const int x = place(r, s, kvh, bucket);
      int* cursor = &pp.hist[x * hist_pitch + bucket];
      // a pair's bucket holds its row tiles only, the last bucket those of the pairs left over: the longest (last)
      // row tile goes first; where buckets are shared by length, arrival order decides
      const int n_here = !grouped && t > 0 ? 2 : 1;
      const int pair = pp.st_rank[s] * pp.n_kv_heads + kvh;
      const int within = !grouped ? atomicAdd(cursor, n_here) : pair < whole_pairs ? level : left_before(pair, level, x);
      const int start = grouped ? __hip_atomic_load(cursor, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
      const int pos = s_list_off[x] + start + within;
      // units: the first item of one says where its second is ([6], for the deal below: -1 not a first one, -2 alone,
      // -3 - i with item i).  Of a whole pair two neighbours make a unit; of a pair left over the row tiles that this
      // XCD takes, two by two
      int unit = -1;
      if (grouped && pp.solo) {
        unit = -2;
      } else if (!grouped || pair < whole_pairs) {
        if ((level & 1) == 0) unit = t > 0 ? -4 - pos : -2;
      } else if ((level & 8) == 0) {
        unit = t >= 8 ? -3 - (s_list_off[x] + start + left_before(pair, level + 8, x)) : -2;
      }
      if (unit < -1) atomicAdd(&s_units[x], 1);
      for (int second = 0; second < n_here; ++second) {
        const int wg_max = pp.rt_wgmax[r - second];
        int32_t* it = pp.items + static_cast<int64_t>(pos + second) * 8;
        it[0] = q0; it[1] = rows; it[2] = (t - second) * pp.bm; it[3] = kvh | (s << 8); it[4] = wg_max;
        it[5] = (max(wg_max, 0) / kBN + 1) << 16; it[6] = second ? -1 : unit; it[7] = second || unit == -1 ? -2 : -1;
      }
    }
  }
  __threadfence_block();
  __syncthreads();

  // ---- deal every XCD's list to its workgroups (one wave per XCD, a lane per workgroup), a batch
  //      of as many items as there are workgroups at a time: within a batch the longest item goes
  //      to the workgroup with the least work so far, the second longest to the next one, ...
  //      (ranks by counting, 64 lane reads each).  This is close to the schedule a run-time queue
  //      would produce, fixed here so that the attention kernel needs no atomics.  Items of one
  //      workgroup are chained through their `next` field.
  {
    const int lane = tid & 63;
    for (int w = tid >> 6; w < 8; w += THREADS / 64) {
      const int begin = s_list_off[w], end = s_list_off[w + 1];
      const int n_wg = pp.n_slots;
      int load = lane < n_wg ? 0 : 0x7fffffff;          // half key tiles; lanes beyond the grid rank last
      int first_item = -1, last = -1;
      auto field = [&](int i, int k) {
        return __hip_atomic_load(&pp.items[static_cast<int64_t>(i) * 8 + k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      auto take = [&](int item, int second_item, int tiles) {
        for (int k = 0; k < (second_item >= 0 ? 2 : 1); ++k) {
          const int idx = k ? second_item : item;
          if (last >= 0) pp.items[static_cast<int64_t>(last) * 8 + 6] = idx;
          else first_item = idx;
          last = idx;
        }
        // (the second of two workgroups of a CU, which the issue arbiter serves less often, gets 3/4 of the first one's work)
        load += pp.solo ? (2 * tiles + kSoloFixedCostHalves) * (lane >= kWorkgroupsPerXcd ? 4 : 3) : 2 * tiles + kItemFixedCostHalves;
      };
      // A short pair-ordered list is dealt by length over the whole list: its pairs are under way together in any case, and
      // batches in list order let long units meet.  us a step in list order / by length: 12 streams of 1,000 keys (71 units an
      // XCD) 1,157 / 1,069, 11 (67) 1,847 / 1,713, 5 of 3,200 (71) 2,564 / 2,504, 5 ragged (54) 3,415 / 3,337, 9 and 10 of 1,000
      // (53, 57) 1,597 / 1,566, 963 / 947.  Longer lists keep their order, so that few pairs at a time share an L2: 12 of 1,000,
      // eight kv heads (81) 1,337 / 1,386, 15 of 1,000 (88) 2,177 / 2,182, 16 of 900 (90) 2,035 / 2,069, 9 of 2,000 (107) 2,595 /
      // 2,681.  The line at 72 lies above all that gained and below all that lost, but the number of units is not what decides:
      // the spread of their lengths against a round does, and lists of 92 and 100 would gain too (16 of 1,000 1,372 / 1,328, 25
      // of 2,900, one kv head 2,519 / 2,400).  Working both deals out tells which, but cost 15-30 us a plan.
      if (grouped && s_units[w] <= kDealAtOnce) {
        int4* unit_at = reinterpret_cast<int4*>(s_key) + w * 128;     // first item, second (or -1), key tiles
        int* by_len = s_deal[w];
        int n_units = 0;
        for (int base = begin; base < end; base += 64) {
          const int at = base + lane;
          const int unit = at < end ? field(at, 6) : -1;
          const unsigned long long firsts = __ballot(unit < -1);
          if (unit < -1)
            unit_at[n_units + __popcll(firsts & ((1ull << lane) - 1))] = make_int4(at, unit < -2 ? -3 - unit : -1, field(at, 5) >> 16, 0);
          n_units += __popcll(firsts);
        }
        __builtin_amdgcn_wave_barrier();
        const int len0 = lane < n_units ? unit_at[lane].z : -1, len1 = lane + 64 < n_units ? unit_at[lane + 64].z : -1;
        int rank0 = 0, rank1 = 0;                         // by decreasing length, ties in list order
#pragma unroll 8
        for (int j = 0; j < 64; ++j) {
          const int l0 = __builtin_amdgcn_readlane(len0, j);
          rank0 += l0 > len0 || (l0 == len0 && j < lane) ? 1 : 0;
          rank1 += l0 >= len1 ? 1 : 0;
        }
        for (int j = 0; j < n_units - 64; ++j) {
          const int l1 = __builtin_amdgcn_readlane(len1, j);
          rank0 += l1 > len0 ? 1 : 0;
          rank1 += l1 > len1 || (l1 == len1 && j < lane) ? 1 : 0;
        }
        if (lane < n_units) by_len[rank0] = lane;
        if (lane + 64 < n_units) by_len[rank1] = lane + 64;
        __builtin_amdgcn_wave_barrier();
        for (int dealt = 0; dealt < n_units; dealt += n_wg) {
          int load_rank = 0;
#pragma unroll 8
          for (int j = 0; j < n_wg; ++j) {
            const int wj = __builtin_amdgcn_readlane(load, j);
            load_rank += (wj < load || (wj == load && j < lane)) ? 1 : 0;
          }
          if (load_rank < min(n_wg, n_units - dealt)) {
            const int4 u = unit_at[by_len[dealt + load_rank]];
            take(u.x, u.y, u.z);
          }
        }
      } else {
        // (a pair-ordered list that is not a whole number of batches starts with the short batch:
        // the full batches that follow even the loads out again, which a short batch at the end
        // cannot.  A list ordered by length keeps its batches aligned instead: workgroups that start
        // equal-length items together sweep the same key ranges together and share them in L2,
        // which is worth more there: 6 % on the dense long-window case.)
        int n_batch = grouped && s_units[w] % n_wg ? s_units[w] % n_wg : n_wg;
        for (int base = begin; base < end; n_batch = n_wg) {
          // of whole pairs the next n_batch units lie within the next 64 items
          const int unit = base + lane < end ? field(base + lane, 6) : -1, keys = base + lane < end ? field(base + lane, 5) : 0;
          const bool first = unit < -1;
          const int second = unit < -2 ? -3 - unit : -1;
          const unsigned long long firsts = __ballot(first);
          const int rank = __popcll(firsts & ((1ull << lane) - 1)), n_seen = __popcll(firsts), n_here = min(n_seen, n_batch);
          const unsigned long long stop = __ballot(first && rank == n_batch);
          int len = -1;                                     // lanes without a unit rank last
          if (first && rank < n_batch) len = keys >> 16;
          int item_rank = 0, load_rank = 0;                 // by decreasing length / increasing load, ties by lane
#pragma unroll 8
          for (int j = 0; j < 64; ++j) {
            const int lj = __builtin_amdgcn_readlane(len, j);
            item_rank += (lj > len || (lj == len && j < lane)) ? 1 : 0;
          }
#pragma unroll 8
          for (int j = 0; j < n_wg; ++j) {
            const int wj = __builtin_amdgcn_readlane(load, j);
            load_rank += (wj < load || (wj == load && j < lane)) ? 1 : 0;
          }
          s_by_rank[w][item_rank] = lane | (len << 8);
          __builtin_amdgcn_wave_barrier();
          const int got = load_rank < n_here ? s_by_rank[w][load_rank] : 0;
          const int got_second = __shfl(second, got & 63);
          if (load_rank < n_here) take(base + (got & 63), got_second, got >> 8);
          __builtin_amdgcn_wave_barrier();
          base = stop ? base + __ffsll(stop) - 1 : min(base + 64, end);
        }
      }
      if (last >= 0) pp.items[static_cast<int64_t>(last) * 8 + 6] = -1;
      if (lane < kSlotsPerXcd) {
        int32_t* hd = pp.header + kHdrHeads + kHdrEntryInts * (w * kSlotsPerXcd + lane);
        int32_t d[8] = {0, 0, 0, 0, -1, 0, -1, -1};       // the end item
        if (first_item >= 0)
          for (int i = 0; i < 8; ++i) d[i] = field(first_item, i);
        hd[0] = first_item;
        for (int i = 0; i < 8; ++i) hd[8 + i] = d[i];
      }
    }
  }
}

__global__ __launch_bounds__(kPlanThreads) void window_attn_plan_kernel(PlanParams pp) {
  __shared__ __attribute__((aligned(16))) PlanLds lds;
  __shared__ SpanLds span_lds;
  plan_work<kPlanThreads, true>(pp, lds, &span_lds);
}

// A row tile to each workgroup but the first, which makes the plan of the calls that follow: a BUILD call of whole sweeps
// below 1,024 row tiles.  The planning launch ahead of the persistent kernel cost such a call 27-32 us, which the layers
// that reuse the plan repay after three to ten of them and a caller that plans in every call never.  us a BUILD call, with the
// planning launch / tile kernel alone, no plan / this one: 10 streams of 420 tokens, 900 keys 83.2 / 62.5 / 62.1, of 610 70.5 / 44.6 /
// 44.3; 20 of 200 tokens, 1,760 keys 124.7 / 112.3 / 114.6; 5 of 500 tokens, 610 keys 58.0 / 28.7 / 32.8 (planning takes 32 there, of
// 150 streams 45).  One workgroup more is one round more where the others fill the chip to the last slot: 64 streams of two
// row tiles and four kv heads, 930 keys 62.6 / 47.6 / 57.3.
template <int ROWW, int KG, int STAGES>
__global__ __launch_bounds__(64 * ROWW * KG, 2) void window_attn_bf16_tile_and_plan_kernel(AttnParams p, PlanParams pp) {
  __shared__ TileStages<128, KG, STAGES> stages;
  static_assert(sizeof(PlanLds) <= sizeof(stages), "the plan is made in the tile buffers");
  if (blockIdx.x == 0)
    plan_work<64 * ROWW * KG, false>(pp, *reinterpret_cast<PlanLds*>(&stages), nullptr);
  else
    attend_row_tile<128, ROWW, KG, STAGES>(p, blockIdx.x - 1, stages);
}


// 16-byte store that is written through the XCD's L2 to memory (agent scope), the cache policy an
// agent-scope atomic store carries: its acknowledgement (vmcnt) comes when the other XCDs can read
// the bytes, so a wait on vmcnt stands in for an L2 write-back.  The s_nop belongs to the store: a
// store of more than 8 bytes reads its data registers for a cycle after it issues, the compiler
// does not know that this statement is such a store, and it is free to reuse the data registers in
// the very next instruction (seen in an experiment: the next row's address landed in the first
// 8 bytes of a stored row).
__device__ __forceinline__ void store_agent(void* dst, const cs::u32x4& v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(dst), "v"(v) : "memory");
}
// Waits for the acknowledgements of this wave's stores.  Spelled out: the compiler does not know of
// stores issued from inline assembly, so a fence of its own may come without the wait.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

constexpr uint32_t kBarrierSpinLimit = 1u << 24;

// Launch-wide barrier of a grid whose workgroups are all resident (at most one per CU on 256 CUs, by
// construction of the persistent grid).  Arrivals are counted in two levels so that no counter takes
// more than n/16 + 16 read-modify-writes in a row (they execute at the memory side, one after the
// other per address): workgroup b adds to group counter b & 15; whoever completes a group resets it
// and adds to the counter of finished groups; whoever completes that resets it and bumps the release
// word.  Everybody else polls the release word against the value it read before arriving (it cannot
// have moved yet: a bump needs every arrival, the reader's included).  Which workgroup runs where
// plays no part in the counting.  The wait is bounded: after kBarrierSpinLimit polls the workgroup
// raises the status word and goes on, so every wave exits even if part of the grid never became
// resident; the results of such a launch are not valid and the status word says so.
//
// Visibility across the XCDs' L2s: the rows written before the barrier are stored write-through at
// agent scope (see store_agent) and every wave waits for its stores' acknowledgements, so no L2
// write-back is needed on arrival (one per workgroup measured 16 us per launch, one per wave 40 us);
// after the release one thread per workgroup invalidates the CU's vector cache and the XCD's L2
// (they are shared by the workgroup's waves), which costs nothing measurable.
__device__ __forceinline__ void launch_barrier(int32_t* sync, int32_t* status, int n_workgroups) {
  wait_stores();                                           // the row stores are acknowledged
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t* group = sync + (blockIdx.x % kSyncGroups) * kSyncPitch;
    int32_t* groups_done = sync + kSyncGroups * kSyncPitch;
    int32_t* release = sync + (kSyncGroups + 1) * kSyncPitch;
    const int in_group = (n_workgroups - static_cast<int>(blockIdx.x % kSyncGroups) + kSyncGroups - 1) / kSyncGroups;
    const int n_groups = n_workgroups < kSyncGroups ? n_workgroups : kSyncGroups;
    const int r0 = __hip_atomic_load(release, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool last = false;
    if (__hip_atomic_fetch_add(group, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == in_group - 1) {
      __hip_atomic_store(group, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__hip_atomic_fetch_add(groups_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_groups - 1) {
        __hip_atomic_store(groups_done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(release, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = true;
      }
    }
    if (!last) {
      uint32_t polls = 0;
      while (__hip_atomic_load(release, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == r0) {
        if (++polls > kBarrierSpinLimit) {                // never taken when the whole grid is resident
          __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(8);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}


// f(Begin), f(Begin + 1), ... f(End - 1) with the index as a compile-time constant.
template <int Begin, int End, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (Begin < End) {
    f(std::integral_constant<int, Begin>{});
    unrolled<Begin + 1, End>(f);
  }
}

// One matrix instruction that accumulates in the accumulation registers, spelled out so that they stay there.  The
// compiler does not know it for one and keeps no distances for it: whoever reads the accumulators waits first
// (mfma_settle), and a vector instruction that writes an operand stands two wait states or more before it by the order of
// the slots (tests/test_matrix_waits.py checks both in the built code).
__device__ __forceinline__ void mfma_acc(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_settle(f32x16 (&o)[2][4]) {
  asm volatile("s_nop 15\n\ts_nop 7"
               : "+a"(o[0][0]), "+a"(o[0][1]), "+a"(o[0][2]), "+a"(o[0][3]), "+a"(o[1][0]), "+a"(o[1][1]), "+a"(o[1][2]), "+a"(o[1][3]));
}

// The persistent kernel: 4 waves of 64 rows (two blocks of 32), one workgroup per CU, one wave per SIMD.
//
// What bounds it: power.  The matrix cores toggle enough for the device to run at 1.6-2.1 GHz instead of 2.4, so
// cycles saved by overlap alone come back as a lower clock, and what counts is work per matrix instruction.  Timing
// builds of the kernel before (32 rows a wave, 128 a workgroup, two workgroups per CU) with half the LDS reads, with
// half the tile requests and with both left out ran 13, 8 and 20 % shorter.  Hence 64 rows a wave
// (each K and V fragment read from LDS feeds two matrix instructions) and 256 a workgroup (each tile is fetched once
// for twice the rows).  The price is that no second wave hides anything: a half tile (32 keys) is laid out by hand as
// 32 slots of one matrix instruction, 16 for the scores of the NEXT half tile and 16 for P V of this one, and between
// them go the softmax of this half tile, the LDS reads two to three slots ahead and the next requests.  A tile (64 keys)
// takes 3,020 cycles in sweeps of 58 tiles and 3,460 in sweeps of 9, of which 2,048 are matrix instructions; a job takes
// 8,900 more with whole results, 7,300 with partial ones.
// * Registers: O (128) and Q (64) live in the accumulation registers, scores and weights in the others; the matrix
//   instructions of P V are spelled out so that O stays there.
// * Row sums: v_dot2 waits for the matrix pipe to drain (48 cycles instead of 32 per matrix instruction when one
//   follows each, and a second wave's stall it too); the 4x4 matrix instruction with ones sums the same rounded weights.
// * Requests run three slots ahead through four LDS stages of 32 KiB; queries come by the same way.  A tile takes one
//   barrier.  Sweeps inside a job change one index per slot; everything else (frontier tile, next job's queries, next
//   job) is set up when the walk enters it.
// * Frontiers: rows that see nothing more of a sweep get an infinite reference maximum once; only half tiles that hold
//   some row's frontier are masked score by score.
// * The scores of a job's first tile are formed ahead of its sweep, and again inside it: 8,000 of 462,000 cycles of a
//   workgroup at 64 streams.  The reference is then the maximum over 64 keys.  Over 32 the error against 64 bits was larger:
//   2.130e-3 instead of 2.111e-3 (32 streams of 860 keys), 2.161e-3 instead of 2.142e-3 (64 of 560).
// us a layer, two builds in turn (32 rows a wave / this one): 64 streams of 560 keys, 32/8 heads 244 / 235; 32 streams of
// 860 keys, 28/4 heads 127 / 117; 2,100 tokens over 6,000 keys 102 / 89, over 17,600 keys 249 / 214 (1.07 PFLOP/s); 5 ragged
// streams of 2,600 keys 109 / 110 (1.5 jobs a workgroup, the longest 1.4 times the mean: the cycles saved are not on it).
template <bool FUSE>
__global__ __launch_bounds__(256, 1) void window_attn_bf16_stream_kernel(AttnParams p) {
  constexpr int RB = 2;                 // 32-row blocks per wave
  constexpr int WROWS = 32 * RB;        // rows per wave
  constexpr int D = 128;
  constexpr int STEPS = D / 16, DB = D / 32;
  constexpr int TILE = kBN * D;         // elements of one K (or V) tile: 16 KiB, unpadded
  constexpr int IPW = 4;                // 1-KiB DMA instructions per wave, per tile, per tensor
  constexpr int STAGES = 4;
  constexpr int kStageBytes = 2 * TILE * 2, kHalfBytes = 32 * D * 2;

  __shared__ __attribute__((aligned(1024))) uint16_t s_kv[STAGES][2][TILE];
  __shared__ __attribute__((aligned(1024))) uint16_t s_sink[4][512];
  __shared__ int32_t s_pos[2][4][64];   // query positions of the waves' rows, every other job
  __shared__ __attribute__((aligned(1024))) uint16_t s_out[4][32 * 64];     // results of the waves on their way out

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;

  if constexpr (FUSE) {
    // ---- refresh write (Sec. 3.5: the K/V just computed go into the destination cache before
    //      attention reads it): the whole grid moves the new rows, 16 bytes of K and of V per
    //      thread four times a turn, then meets at a launch-wide barrier.  What bounds it is how much four waves a CU keep
    //      in flight: 19,200 tokens of eight kv heads (157 MB with both directions) take 58 us once a turn, 44 four times,
    //      43 eight times
    constexpr int TURN = 4;
    const int64_t n_units = p.n_new * p.row_vecs;
    const int apart = static_cast<int>(gridDim.x) * 256, apart_tok = apart / p.row_vecs, apart_rem = apart - apart_tok * p.row_vecs;
    const cs::u32x4* kn = static_cast<const cs::u32x4*>(p.k_new);
    const cs::u32x4* vn = static_cast<const cs::u32x4*>(p.v_new);
    uint16_t* kc = const_cast<uint16_t*>(static_cast<const uint16_t*>(p.k));
    uint16_t* vc = const_cast<uint16_t*>(static_cast<const uint16_t*>(p.v));
    int64_t unit = static_cast<int64_t>(blockIdx.x) * 256 + tid, tok = unit / p.row_vecs;
    int rem = static_cast<int>(unit - tok * p.row_vecs);
    while (unit < n_units) {
      int64_t dst[TURN];
      cs::u32x4 kv[TURN], vv[TURN];
#pragma unroll
      for (int i = 0; i < TURN; ++i) {     // (past the last unit: that one's data, for no slot)
        const int sl = unit < n_units ? p.new_slot[tok] : -1;
        const int64_t from = unit < n_units ? unit : n_units - 1;
        const int head = rem / p.head_vecs, c = rem - head * p.head_vecs;
        dst[i] = sl < 0 ? -1 : static_cast<int64_t>(sl) * p.stride_slot + head * p.stride_head + c * 8;
        kv[i] = __builtin_nontemporal_load(kn + from);
        vv[i] = __builtin_nontemporal_load(vn + from);
        unit += apart;
        tok += apart_tok;
        rem += apart_rem;
        if (rem >= p.row_vecs) {
          rem -= p.row_vecs;
          ++tok;
        }
      }
#pragma unroll
      for (int i = 0; i < TURN; ++i) {
        if (dst[i] < 0) continue;
        store_agent(kc + dst[i], kv[i]);
        store_agent(vc + dst[i], vv[i]);
      }
    }
    launch_barrier(p.ws_sync, p.ws_status, static_cast<int>(gridDim.x));
  }

  // ---- this workgroup's items: a chain through the `next` field of the descriptors, dealt by the planning kernel
  const int xcd = blockIdx.x & 7, slot_j = blockIdx.x >> 3;
  auto item_at = [&](int idx) -> const int32_t* {
    return idx >= 0 ? p.ws_items + static_cast<int64_t>(idx) * 8 : p.ws_plan + kHdrEndItem;
  };
  const int32_t* entry = p.ws_plan + kHdrHeads + kHdrEntryInts * (xcd * kSlotsPerXcd + slot_j);
  i32x8 d = const_load8(entry + 8);
  if ((d[5] >> 16) == 0) return;        // nothing for this workgroup

  // The two items of a unit follow each other in the chain and are taken as one job of 256 rows: waves 0-1 the second, waves
  // 2-3 the first.  The plan marks the second; what the items hold does not tell (a stream's odd first row tile, a unit of its
  // own, may stand before a later unit that ends in the same key tile), and comparing it took 0.8 % of a step.
  auto joins = [](const i32x8& b) { return (b[7] & 1) == 0; };
  auto mine = [&](const i32x8& a, const i32x8& b, bool both) { return wave < 2 && both ? b : a; };
  auto takes_part = [&](bool both) { return both || wave >= 2; };

  // ---- constants of the lane
  const uint32_t blk_bytes = static_cast<uint32_t>(CS_KV_BLOCK * 2 * p.stride_slot);     // (stride_slot < 2^26: the host checks)
  const uint32_t row_bytes = static_cast<uint32_t>(p.stride_slot * 2);
  const int l_row = lane >> 4, l_pos = lane & 15;
  // tile requests: instruction i of a tensor moves rows 4 i + l_row of this wave's cache block; which 16-byte chunk
  auto k_chunk = [&](int i) __attribute__((always_inline)) { return static_cast<uint32_t>((l_pos ^ (4 * i + l_row)) * 16); };
  auto v_chunk = [&](int i) __attribute__((always_inline)) { return static_cast<uint32_t>((l_pos ^ (4 * l_row + 2 * (i & 1))) * 16); };
  uint32_t k_addr[STEPS], v_addr[DB];   // LDS byte addresses of this lane's fragments in the current stage
#pragma unroll
  for (int st = 0; st < STEPS; ++st)
    k_addr[st] = lds_address(&s_kv[0][0][0]) + 2 * (n * D + (((2 * st + h) ^ (n & 15)) << 3));
  const int i16 = lane & 15, gid = (lane >> 4) & 1;
  const int v_row = 4 * h + (i16 >> 2);
  const int v_swz = 4 * (v_row & 3) + 2 * (v_row >> 2);
#pragma unroll
  for (int db = 0; db < DB; ++db)
    v_addr[db] = lds_address(&s_kv[0][1][0]) +
                 2 * (v_row * D + (((4 * db + 2 * gid + ((i16 & 3) >> 1)) ^ v_swz) << 3) + 4 * (i16 & 1));

  // ---- requests run three slots ahead of the computation, across jobs, on a walk of their own along the chain.  A slot
  // is a key tile, or 32 query rows of each wave: two of these stand ahead of a job's tiles.  Every wave fetches its own
  // queries, the first 16 rows of a slot to its share of the K half, the others to its share of the V half.  Each slot
  // takes a wave eight DMA instructions; past the last one they go to a sink, so that their number stays the same.
  struct Rows { int tok0, rem0, last; };                // of a wave's first row: token and head; rows after it
  const uint32_t group_inv = 65535u / p.group + 1;      // x * group_inv >> 16 = x / group for x < 80
  auto rows_of = [&](const i32x8& it) __attribute__((always_inline)) {
    const int r0 = min(it[2] + (wave & 1) * WROWS, it[1] - 1);
    const int t0 = r0 / p.group;
    return Rows{it[0] + t0, r0 - t0 * p.group, it[1] - 1 - r0};
  };
  auto row_offset = [&](const Rows& r, int row) __attribute__((always_inline)) {       // bytes from the first row's token and the kv head's first query head; past the last row, that row again
    const uint32_t x = r.rem0 + min(row, r.last);
    const uint32_t t = (x * group_inv) >> 16;
    return (t * p.n_q_heads + (x - t * p.group)) * (D * 2);
  };
  i32x8 r_cur = d, r_x1 = const_load8(item_at(d[6]));
  int r_q = 2, r_kt = 0, r_ke = 0, r_live = 1, r_stage = 0;    // r_q: query slots before the next tile
  int r_parity = 1;                     // the job's half of s_pos (the walk may be at the next but one before a job has read its own)
  int r_last = 0;                       // the cache block of the item's frontier
  uint32_t r_hi = 0;                    // the frontier's row in it
  const int32_t* r_row = nullptr;
  int r_id = 0;
  const char *r_k = nullptr, *r_v = nullptr;                      // the kv head's cache
  const char *src_k = nullptr, *src_v = nullptr;                  // the slot: base (of cache block 0)
  uint32_t src_id = 0;                                            // ... block ids count (all ones) or not (0)
  uint32_t req_off[2 * IPW];                                      // ... offsets of the lane
  const char *req_k = nullptr, *req_v = nullptr;
  uint32_t req_dst = 0, req_step = 0, req_v_at = 0;
  const uint32_t lds_mine = lds_address(&s_kv[0][0][wave * IPW * 512]);
  const uint32_t lds_sink = lds_address(&s_sink[wave][0]);
  auto enter_job = [&]() __attribute__((always_inline)) {
    r_kt = r_cur[5] & 0xffff; r_ke = r_cur[5] >> 16;
    r_last = max(r_cur[4], 0) >> 4;
    r_hi = (max(r_cur[4], 0) & 15) * row_bytes;
    r_row = p.block_table + static_cast<int64_t>(r_cur[3] >> 8) * p.max_blocks;
    const int64_t head = static_cast<int64_t>(r_cur[3] & 255) * p.stride_head * 2;
    r_k = static_cast<const char*>(p.k) + head;
    r_v = static_cast<const char*>(p.v) + head;
    r_q = 2;
    r_parity ^= 1;
  };
  auto enter_queries = [&]() __attribute__((always_inline)) {
    const i32x8 it = mine(r_cur, r_x1, joins(r_x1));
    const Rows r = rows_of(it);
    src_k = src_v = static_cast<const char*>(p.q) + (static_cast<int64_t>(r.tok0) * p.n_q_heads + (it[3] & 255) * p.group) * (D * 2);
    src_id = 0;
#pragma unroll
    for (int i = 0; i < 2 * IPW; ++i) req_off[i] = row_offset(r, (2 - r_q) * 32 + 4 * i + l_row) + k_chunk(i & 3);
    if (r_q == 2) {
      const uint32_t x = r.rem0 + min(lane, r.last);
      dma4_sa(((x * group_inv) >> 16) * 4, p.q_pos + r.tok0, lds_address(&s_pos[r_parity][wave][0]));
    }
  };
  // Rows past the item's frontier may be unallocated or hold anything: their lanes fetch the frontier row instead
  // (finite data, weight 0 after masking).
  auto enter_tile = [&]() __attribute__((always_inline)) {
    src_k = r_k; src_v = r_v; src_id = ~0u;
    const int blk = 4 * r_kt + wave;
    const uint32_t hi = blk < r_last ? 15 * row_bytes : r_hi, lo = blk > r_last ? r_hi : 0;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const uint32_t row = max(lo, min((4 * i + l_row) * row_bytes, hi));
      req_off[i] = row + k_chunk(i);
      req_off[IPW + i] = row + v_chunk(i);
    }
  };
  // addresses of the slot's request, in four parts for four slots of a block
  uint64_t r_at = 0;
  auto prepare = [&](int part) __attribute__((always_inline)) {
    if (part == 0) r_at = static_cast<uint64_t>(static_cast<uint32_t>(r_id) & src_id) * blk_bytes;
    if (part == 1) req_k = src_k + r_at;
    if (part == 2) req_v = src_v + r_at;
    if (part == 3) {
      req_dst = r_live ? lds_mine + r_stage * kStageBytes : lds_sink;
      req_step = r_live ? 1024 : 0;
      req_v_at = r_live ? TILE * 2 : 0;
    }
  };
  auto request_part = [&](int part) __attribute__((always_inline)) {
    if (part < IPW) dma16_sa(req_off[part], req_k, req_dst + part * req_step);
    else dma16_sa(req_off[part], req_v, req_dst + req_v_at + (part - IPW) * req_step);
  };
  // ... and on to the next slot: inside a sweep only the tile changes
  auto advance = [&]() __attribute__((always_inline)) {
    r_stage = (r_stage + 1) & (STAGES - 1);
    if (__builtin_expect(r_q == 0 && r_kt + 2 < r_ke, 1)) {
      ++r_kt;
    } else {
      if (r_q) {
        --r_q;
      } else if (r_kt + 1 < r_ke) {
        ++r_kt;
      } else if (r_live) {
        i32x8 to = r_x1;
        if (joins(r_x1)) {
          to = const_load8(item_at(r_x1[6]));
          wait_scalar();
        }
        if ((to[5] >> 16) > 0) {
          r_cur = to;
          r_x1 = const_load8(item_at(to[6]));
          wait_scalar();
          enter_job();
        } else {
          r_live = 0;
        }
      }
      if (r_live) {
        if (r_q) enter_queries();
        else enter_tile();
      }
    }
  };
  // the block id of the tile that the walker stands at: asked for in every slot, behind its request, and waited for at
  // the end of the slot (by hand, so that the waits for LDS reads in between need not be waits for it)
  auto ask = [&]() __attribute__((always_inline)) { r_id = sload1(r_row + min(4 * r_kt + wave, r_last)); };
  auto asked = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(r_id)); };
  auto send = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int part = 0; part < 4; ++part) prepare(part);
#pragma unroll
    for (int part = 0; part < 2 * IPW; ++part) request_part(part);
    advance();
    ask();
  };
  // waits until the tile after the current one has landed for every wave; after it every wave has left the previous one
  auto gate = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory"); };

  // ---- per-job state of the lane
  bf16x8 qf[RB][STEPS];
  int lim[RB];
  const s16x4 ones4 = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 o[RB][DB];
  f32x4 lacc[RB][2];
  float m_run[RB], m_scaled[RB], m_top[RB], t_max[RB];
  uint64_t need = 0;                    // rows whose maximum has to be raised before the next half tile
  int k_step = 0;                       // from this stage to the next
  const float slack = kMaxSlack / p.scale_log2e;
  f32x16 sa[RB], sb[RB];                // scores of the current and of the next half tile
  bf16x8 ka[4];                         // K fragments in flight
  typedef __attribute__((address_space(3))) const cs::u32x4 lds_u32x4;
  auto k_frag = [&](int st, int half) {
    ka[st & 3] = __builtin_bit_cast(bf16x8, reinterpret_cast<lds_u32x4*>(static_cast<uintptr_t>(k_addr[st]))[half * kHalfBytes / 16]);
  };
  // (a row with a score that is no number has no maximum either: see past_frontier)
  auto row_max = [&](const f32x16 (&s)[RB], int rb) __attribute__((always_inline)) {
    float t = kNegInf;
#pragma unroll
    for (int r = 0; r < 16; ++r) t = __builtin_elementwise_maximum(t, s[rb][r]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    t_max[rb] = __builtin_elementwise_maximum(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  auto mask = [&](f32x16 (&s)[RB], int half_tile) __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = 32 * half_tile + 8 * (r / 4) + 4 * h + (r % 4);
        if (key > lim[rb]) s[rb][r] = kNegInf;
      }
  };
  // The scores of a half tile past some row's frontier.  Rows that see none of its keys (nor any later one) are out of
  // the sweep: their reference maximum becomes infinite for the weights, which are 0 from here on as long as the scores
  // are finite.  Scores are masked one by one only where a frontier lies inside the half tile, or a score is infinite or
  // no number (the row maxima keep both).  One branch for the two: a second one, or masking every half tile past a
  // frontier, took 3-5 % of a long window's layer.  (A wave whose rows belong to two frames has frontiers thousands of
  // keys apart, and all half tiles between them pass through here.)
  auto past_frontier = [&](f32x16 (&s)[RB], int half_tile) __attribute__((always_inline)) {
    const int j0 = 32 * half_tile;
    bool one_by_one = false;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      if (lim[rb] < j0) m_scaled[rb] = m_top[rb] = INFINITY;
      one_by_one |= (lim[rb] >= j0 && lim[rb] < j0 + 31) || !(t_max[rb] < INFINITY);
    }
    if (__ballot(one_by_one)) {
      mask(s, half_tile);
      row_max(s, 0);
      row_max(s, 1);
    }
    need = __ballot(t_max[0] > m_top[0] || t_max[1] > m_top[1]);
  };
  // the reference maximum: in log2 units as the weights need it, and where it is raised
  auto set_max = [&](int rb, bool here, float m) __attribute__((always_inline)) {
    m_run[rb] = here ? m : m_run[rb];
    m_scaled[rb] = here ? (m == kNegInf ? 0.f : m) * p.scale_log2e : m_scaled[rb];
    m_top[rb] = here ? m + slack : m_top[rb];
  };
  auto raise_max = [&]() __attribute__((always_inline)) {
    if (__builtin_expect(need != 0, 0)) {
      mfma_settle(o);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const bool up = t_max[rb] > m_top[rb];
        const float m_new = up ? t_max[rb] : m_run[rb];
        const float alpha = up ? __builtin_amdgcn_exp2f((m_run[rb] - m_new) * p.scale_log2e) : 1.f;
        set_max(rb, up, m_new);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) lacc[rb][i][r] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
          for (int r = 0; r < 16; ++r) o[rb][db][r] *= alpha;
          asm volatile("" : "+a"(o[rb][db]));
        }
      }
    }
  };
#define FENCE() __builtin_amdgcn_sched_barrier(0)

  // One half tile (32 keys): softmax and P V of the scores `sc`, and the scores `sn` of the next half tile, as 32 slots
  // of one matrix instruction and what its 32 cycles leave room for.  The fences keep the slots as they are written.
  auto block = [&](auto half_c, const f32x16 (&sc)[RB], f32x16 (&sn)[RB]) __attribute__((always_inline)) {
    constexpr int HALF = decltype(half_c)::value;
    cs::u32x4 w[RB][2];
    // the weights, two at a time (unit u = 8 mm + 4 rb + c): v_fma, v_exp, pack, each some instructions behind the other
    float f[17][2], e[16][2];
    auto form = [&](int u, int i) {
      if (u < 16) f[u][i] = fmaf(sc[(u >> 2) & 1][8 * (u >> 3) + 2 * (u & 3) + i], p.scale_log2e, -m_scaled[(u >> 2) & 1]);
    };
    auto pack = [&](int u) { w[(u >> 2) & 1][u >> 3][u & 3] = pack_bf16x2(e[u][0], e[u][1]); };
    auto op = [&](int k) {
      const int u = k / 5, j = k % 5;
      if (j == 0 || j == 2) e[u][j >> 1] = __builtin_amdgcn_exp2f(f[u][j >> 1]);
      else if (j == 1 || j == 3) form(u + 1, j >> 1);
      else if (u > 0) pack(u - 1);
    };
    s16x4 vlo[4], vhi[4];
    auto v_frag = [&](int m) {
      const int g0 = HALF * kHalfBytes / 8 + 16 * (m >> 2) * D * 2 / 8, db = m & 3;
      vlo[m & 3] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(((lds_s16x4*)(static_cast<uintptr_t>(v_addr[db]))) + g0);
      vhi[m & 3] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(((lds_s16x4*)(static_cast<uintptr_t>(v_addr[db]))) + g0 + 8 * D * 2 / 8);
    };
    auto part_max = [&](int rb, int part) {
      float t = part ? t_max[rb] : kNegInf;
#pragma unroll
      for (int r = 0; r < 8; ++r) t = __builtin_elementwise_maximum(t, sn[rb][8 * part + r]);
      t_max[rb] = t;
    };
    auto swap_max = [&](int rb) {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(t_max[rb]), __float_as_uint(t_max[rb]), false, false);
      t_max[rb] = __builtin_elementwise_maximum(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    };
    FENCE();
    form(0, 0);
    form(0, 1);
    unrolled<0, 32>([&](auto slot_c) {
      constexpr int slot = decltype(slot_c)::value, rb = slot & 1, st = slot >> 1, m = st - 8;
      if (HALF == 0 && slot == 16) gate();
      if constexpr (slot < 16) {
        sn[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[st & 3], qf[rb][st & 7], st == 0 ? zero16 : sn[rb], 0, 0, 0);
        if (rb == 0 && st + 3 < STEPS) k_frag((st + 3) & 7, HALF ^ 1);
        if (slot >= 11 && rb == 1) v_frag((slot - 11) >> 1);
        if (HALF == 0 && slot >= 2 && slot < 6) prepare(slot - 2);
      } else {
        const s16x8 a = __builtin_shufflevector(vlo[m & 3], vhi[m & 3], 0, 1, 2, 3, 4, 5, 6, 7);
        mfma_acc(o[rb][m & 3], __builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, w[rb][(m >> 2) & 1]));
        if (rb == 0 && m + 3 < 8) v_frag(m + 3);
        if (HALF == 0 && rb == 1) request_part(m & 7);
        if (HALF == 0 && slot >= 20 && slot < 24) {
          k_addr[2 * (slot - 20)] += k_step;
          k_addr[2 * (slot - 20) + 1] += k_step;
        }
        if (HALF == 1 && slot >= 28) v_addr[slot - 28] += k_step;
        if (slot >= 24 && slot < 28) part_max((slot >> 1) & 1, slot & 1);
        if (slot == 28 || slot == 29) swap_max(slot & 1);
        if (slot == 30) need = __ballot(t_max[0] > m_top[0] || t_max[1] > m_top[1]);
        if (slot >= 26 && rb == 0) k_frag((slot - 26) >> 1, HALF);        // of the half tile after the next one
      }
      if constexpr (slot < 24) {
        unrolled<80 * slot / 24, 80 * (slot + 1) / 24>([&](auto k) { op(decltype(k)::value); });
        if constexpr (slot == 23) pack(15);
      }
      FENCE();
    });
    // row sums of the rounded weights: the 4x4 instruction with ones adds a lane's own four.  All at once: the change
    // from the large instruction and back costs 16 cycles
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int mm = 0; mm < 2; ++mm)
          lacc[rb][mm] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones4, __builtin_bit_cast(s16x4, cs::u32x2{w[rb][mm][2 * i], w[rb][mm][2 * i + 1]}), lacc[rb][mm], 0, 0, 0);
    FENCE();
  };

  // results on their way out: 32 rows of 64 columns at a time, chunk c of row r at r * 128 + 16 (c ^ (r & 7))
  typedef __attribute__((address_space(3))) cs::u32x4 lds_out;
  const uint32_t out_write = lds_address(&s_out[wave][0]) + n * 128 + 16 * (h ^ (n & 7));
  const uint32_t out_read = lds_address(&s_out[wave][0]) + (lane >> 3) * 128 + 16 * ((lane & 7) ^ (lane >> 3));
  bool out = false;                     // this wave holds results of the job before
  Rows out_rows = {0, 0, 0};
  int out_kvh = 0, out_part = -1;
  // Normalises and stores the rows of the finished job (or their un-normalised partial results when the key sweep is
  // shared).  The two halves of the wave exchange every other group of four, and the rows go through LDS, so that a store
  // writes 8 rows of 128 bytes.  Straight from the registers it wrote 32 rows of 32 bytes: a job's results took 3,100 and
  // 3,700 cycles (its two blocks of 32 rows, 64 streams of 560 keys) instead of 2,300 and 2,500, a layer of 64 streams with
  // its refresh write 264.5 us instead of 258.5, of 32 streams 127.8 instead of 124.6.
  // Partial results likewise: 1,800 and 2,050 cycles instead of 2,300 and 2,700 (2,100 tokens over 6,000 keys; a layer with
  // merge and refresh write 94.3 us instead of 97.1).
  auto finish = [&](int rb, const Rows& r, int kvh, int part, auto between) __attribute__((always_inline)) {
    const float l_half = lacc[rb][0][0] + lacc[rb][1][0];
    const auto lsw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_half), __float_as_uint(l_half), false, false);
    const float l_tot = __uint_as_float(lsw[0]) + __uint_as_float(lsw[1]);
    if (part >= 0) {
      const int64_t prow = static_cast<int64_t>(part) + (wave & 1) * WROWS + rb * 32 + n;
      if (h == 0) {
        p.ws_ml[prow * 2] = m_run[rb];
        p.ws_ml[prow * 2 + 1] = l_tot;
      }
      float* po = p.ws_o + (static_cast<int64_t>(part) + (wave & 1) * WROWS + rb * 32 + (lane >> 3)) * D + 4 * (lane & 7);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
#pragma unroll
        for (int rq = 0; rq < 4; ++rq)
          *reinterpret_cast<lds_out*>(static_cast<uintptr_t>(out_write ^ (32 * rq))) =
              cs::u32x4{__float_as_uint(o[rb][db][4 * rq + 0]), __float_as_uint(o[rb][db][4 * rq + 1]),
                        __float_as_uint(o[rb][db][4 * rq + 2]), __float_as_uint(o[rb][db][4 * rq + 3])};
        cs::u32x4 row[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) row[i] = reinterpret_cast<lds_out*>(static_cast<uintptr_t>(out_read))[i * 64];
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<cs::u32x4*>(po + i * 8 * D + 32 * db) = row[i];
      }
      unrolled<0, DB>(between);
    } else {
      // (a row past the stream's last one holds that row's result and stores it once more)
      const float inv = __builtin_amdgcn_rcpf(l_tot);      // 1 ulp: far below the bf16 result's rounding
      char* base = static_cast<char*>(p.out) + (static_cast<int64_t>(r.tok0) * p.n_q_heads + kvh * p.group) * (D * 2);
      uint32_t at[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) at[i] = row_offset(r, rb * 32 + 8 * i + (lane >> 3)) + 16 * (lane & 7);
      unrolled<0, DB>([&](auto db_c) {
        constexpr int db = decltype(db_c)::value;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          uint32_t w[2][2];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c)
              w[i][c] = pack_bf16x2(o[rb][db][8 * k + 4 * i + 2 * c] * inv, o[rb][db][8 * k + 4 * i + 2 * c + 1] * inv);
          const auto lo = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
          const auto hi = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
          // chunk 4 (db & 1) + 2 k + h of row n
          *reinterpret_cast<lds_out*>(static_cast<uintptr_t>(out_write ^ (64 * (db & 1) + 32 * k))) = cs::u32x4{lo[0], hi[0], lo[1], hi[1]};
        }
        between(db_c);
        if constexpr (db & 1) {
          cs::u32x4 row[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) row[i] = reinterpret_cast<lds_out*>(static_cast<uintptr_t>(out_read))[i * 64];
#pragma unroll
          for (int i = 0; i < 4; ++i) *reinterpret_cast<cs::u32x4*>(base + at[i] + 64 * (db - 1)) = row[i];
        }
      });
    }
  };
  auto send_between = [&](auto db) __attribute__((always_inline)) {
    request_part(2 * decltype(db)::value);
    request_part(2 * decltype(db)::value + 1);
  };
  auto results = [&](int rb) __attribute__((always_inline)) {           // with a slot's request between the stores
#pragma unroll
    for (int part = 0; part < 4; ++part) prepare(part);
    if (out) finish(rb, out_rows, out_kvh, out_part, send_between);
    else unrolled<0, DB>(send_between);
    advance();
    ask();
    asked();
  };

  // ---- prologue: the requests of the first three slots
  enter_job();
  enter_queries();
#pragma unroll 1
  for (int i = 0; i < STAGES - 1; ++i) {
    send();
    asked();
  }
  i32x8 x1 = const_load8(item_at(d[6]));
  int stage = 0;
  const uint32_t q_delta = wave * (IPW * 1024) + (n >> 4) * (TILE * 2 - IPW * 1024);
  uint32_t pos_at = lds_address(&s_pos[0][wave][n]), pos_next = lds_address(&s_pos[1][wave][n]);
  auto next_stage = [&](bool k, bool v) __attribute__((always_inline)) {
    k_step = stage == STAGES - 1 ? -(STAGES - 1) * kStageBytes : kStageBytes;
    if (k)
#pragma unroll
      for (int st = 0; st < STEPS; ++st) k_addr[st] += k_step;
    if (v)
#pragma unroll
      for (int db = 0; db < DB; ++db) v_addr[db] += k_step;
  };

  for (;;) {
    // ---- from job to job: the query slots (wave by wave: their regions are the wave's own), the results of the job
    // before, the requests of the second and third tile.  The second takes the last tile's stage: all waves have left it
    asm volatile("s_barrier" ::: "memory");
    mfma_settle(o);
    results(0);
    const bool stored = out && out_part < 0;            // 8 + 8 stores, then
    const bool paired = joins(x1);
    const i32x8 my = mine(d, x1, paired);
    const int kb = d[5] & 0xffff, ke = d[5] >> 16;
    const bool works = takes_part(paired) && my[2] + (wave & 1) * WROWS < my[1];
    // (the requests of queries are older than 16 others: the first tile's and the second's)
    asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
      for (int st = 0; st < STEPS; ++st)
        qf[rb][st] = __builtin_bit_cast(bf16x8, *reinterpret_cast<lds_u32x4*>(static_cast<uintptr_t>(k_addr[st] + q_delta)));
      if (rb == 0) {
        typedef __attribute__((address_space(3))) const int32_t lds_i32;
        lim[0] = reinterpret_cast<lds_i32*>(static_cast<uintptr_t>(pos_at))[0];
        lim[1] = reinterpret_cast<lds_i32*>(static_cast<uintptr_t>(pos_at))[32];
        asm volatile("" : "+v"(lim[0]), "+v"(lim[1]));
        const uint32_t t = pos_at;
        pos_at = pos_next;
        pos_next = t;
      }
#pragma unroll
      for (int st = 0; st < STEPS; ++st) asm volatile("" : "+a"(qf[rb][st]));
      next_stage(true, true);
      stage = (stage + 1) & (STAGES - 1);
      if (rb == 0) {
        results(1);
      }
    }
    // the first tile: its request is older than those of the next two and the stores
    if (stored) asm volatile("s_waitcnt vmcnt(32)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(16)\n\ts_barrier" ::: "memory");
    const i32x8 nd = const_load8(item_at(paired ? x1[6] : d[6]));     // the next job
    // positions do not decrease along the rows
    lim[0] = min(lim[0], my[4]);                          // my[4]: the row tile's frontier, already inside the stream's entries
    lim[1] = min(lim[1], my[4]);
    const int wave_min = __builtin_amdgcn_readlane(lim[0], 0), wave_max = __builtin_amdgcn_readlane(lim[1], 31);
    const int h_end = works && wave_max >= 0 ? min(2 * (my[5] >> 16), wave_max / 32 + 1) : 0;     // half tiles this wave computes
    const int h_plain = min(h_end, wave_min >= 31 ? (wave_min - 31) / 32 + 1 : 0);                // ... that all its rows see
    auto clear = [&](int i) __attribute__((always_inline)) {
      o[i >> 2][i & 3] = zero16;
      asm volatile("" : "+a"(o[i >> 2][i & 3]));
    };
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      lacc[rb][0] = lacc[rb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      set_max(rb, true, kNegInf);
    }
    if (2 * kb < h_end) {
      // the scores of the whole first tile: their maximum is the rows' reference (the weight of the largest is then
      // exact in bf16 for most of them)
#pragma unroll
      for (int st = 0; st < 3; ++st) k_frag(st, 0);
      unrolled<0, 2 * STEPS>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value, st = i & 7, half = i >> 3;
        constexpr int ahead = (i + 3) & 7;
        if constexpr (i + 3 < 2 * STEPS) k_frag(ahead, (i + 3) >> 3);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          f32x16& to = half ? sb[rb] : sa[rb];
          to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[st & 3], qf[rb][st], st == 0 ? zero16 : to, 0, 0, 0);
        }
        if constexpr (half == 0) clear(st);
        FENCE();
      });
      if (2 * kb + 1 >= h_plain) mask(sb, 2 * kb + 1);
      if (2 * kb >= h_plain) mask(sa, 2 * kb);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        row_max(sb, rb);
        const float t = t_max[rb];
        row_max(sa, rb);
        set_max(rb, true, fmaxf(t, t_max[rb]));
      }
#pragma unroll
      for (int st = 0; st < 3; ++st) k_frag(st, 1);
    } else {
      unrolled<0, 8>([&](auto i) { clear(decltype(i)::value); });
    }
    wait_scalar();
#pragma unroll 1
    for (int kt = kb; kt < ke; ++kt) {
      k_step = stage == STAGES - 1 ? -(STAGES - 1) * kStageBytes : kStageBytes;
      const int h0 = 2 * kt;
      if (__builtin_expect(h0 < h_end, 1)) {
        if (__builtin_expect(h0 >= h_plain, 0)) past_frontier(sa, h0);
        raise_max();
        block(std::integral_constant<int, 0>{}, sa, sb);
      } else {
#pragma unroll
        for (int part = 0; part < 4; ++part) prepare(part);
        gate();
#pragma unroll
        for (int st = 0; st < STEPS; ++st) k_addr[st] += k_step;
#pragma unroll
        for (int i = 0; i < 2 * IPW; ++i) request_part(i);
      }
      advance();
      ask();
      if (__builtin_expect(h0 + 1 < h_end, 1)) {
        if (__builtin_expect(h0 + 1 >= h_plain, 0)) past_frontier(sb, h0 + 1);
        raise_max();
        block(std::integral_constant<int, 1>{}, sb, sa);
      } else {
#pragma unroll
        for (int db = 0; db < DB; ++db) v_addr[db] += k_step;
      }
      stage = (stage + 1) & (STAGES - 1);
      asked();
    }
    out = works;
    out_rows = rows_of(my);
    out_kvh = my[3] & 255;
    out_part = my[7] & ~1;
    d = nd;
    if ((d[5] >> 16) <= 0) break;
    x1 = const_load8(item_at(d[6]));
  }
  mfma_settle(o);
  if (out) {
    auto nothing = [](auto) {};
    finish(0, out_rows, out_kvh, out_part, nothing);
    finish(1, out_rows, out_kvh, out_part, nothing);
  }
  // no request may land after the workgroup's LDS has been given on, no scalar load be left in flight
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// The persistent kernel for streams of few rows: 4 waves of 32 rows, a row tile a job, two workgroups per CU.  Jobs of 256
// rows (below) are too coarse there: a stream's last row tile is alone in every other job and leaves two waves without work,
// two units a workgroup and a few more take three rounds, and a job's own 8,900 cycles weigh on short sweeps.  Here the
// second workgroup of a CU fills what the first leaves idle.  What bounds it: the vector pipe beside the matrix pipe, and on
// the shortest sweeps K and V at memory rate.
// us a layer of REUSE calls, jobs of 256 rows / this kernel: 68 streams of 200 rows a kv head, 32/8 heads, 700 keys 86 / 56, 137 of 252,
// 28/4 heads 85 / 55, 34 of 448, 32/8 heads 97 / 69 (1,300 keys).  Where it runs and where not: solo_row_tiles.
// Tile requests run one tile ahead of the computation ACROSS item boundaries; item descriptors and cache-block ids arrive by
// scalar loads a tile ahead of their use, the queries of the next item are requested before the finished one is stored.
__global__ __launch_bounds__(256, 2) void window_attn_bf16_rows32_kernel(AttnParams p) {
  constexpr int D = 128;
  constexpr int STEPS = D / 16, DB = D / 32;
  constexpr int TILE = kBN * D;         // elements of one K (or V) tile: 16 KiB, unpadded
  constexpr int IPW = 4;                // 1-KiB DMA instructions per wave, per tile, per tensor

  __shared__ __attribute__((aligned(1024))) uint16_t sK[2][TILE];
  __shared__ __attribute__((aligned(1024))) uint16_t sV[2][TILE];
  __shared__ __attribute__((aligned(1024))) uint16_t s_sink[4][512];   // see request_part

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;

  // ---- this workgroup's items: a chain through the `next` field of the descriptors; three are kept loaded
  const int xcd = blockIdx.x & 7, slot_j = blockIdx.x >> 3;
  auto item_at = [&](int idx) -> const int32_t* {
    return idx >= 0 ? p.ws_items + static_cast<int64_t>(idx) * 8 : p.ws_plan + kHdrEndItem;
  };
  i32x8 d0 = sload8(p.ws_plan + kHdrHeads + kHdrEntryInts * (xcd * kSlotsPerXcd + slot_j) + 8);
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(d0));
  if ((d0[5] >> 16) == 0) return;       // nothing for this workgroup

  // ---- constants of the lane: DMA sources inside a cache block, LDS addresses of its fragments in stage 0
  const uint16_t* kall = static_cast<const uint16_t*>(p.k);
  const uint16_t* vall = static_cast<const uint16_t*>(p.v);
  const int64_t blk_stride = static_cast<int64_t>(CS_KV_BLOCK) * p.stride_slot;
  const int l_row = lane >> 4, l_pos = lane & 15;
  uint32_t k_off[IPW], v_off[IPW];      // byte offsets inside a cache block (the host checks the range)
  int k_chunk[IPW], v_chunk[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int trow = 4 * i + l_row;                         // row of this wave's block
    k_chunk[i] = l_pos ^ trow;
    v_chunk[i] = l_pos ^ (4 * (trow & 3) + 2 * ((trow >> 2) & 1));
    k_off[i] = static_cast<uint32_t>((trow * p.stride_slot + k_chunk[i] * 8) * 2);
    v_off[i] = static_cast<uint32_t>((trow * p.stride_slot + v_chunk[i] * 8) * 2);
  }
  uint32_t k_addr[STEPS], v_addr[DB];
#pragma unroll
  for (int st = 0; st < STEPS; ++st)
    k_addr[st] = lds_address(&sK[0][0]) + 2 * (n * D + (((2 * st + h) ^ (n & 15)) << 3));
  const int i16 = lane & 15, gid = (lane >> 4) & 1;
  const int v_row = 4 * h + (i16 >> 2);
  const int v_swz = 4 * (v_row & 3) + 2 * (v_row >> 2);
#pragma unroll
  for (int db = 0; db < DB; ++db)
    v_addr[db] = lds_address(&sV[0][0]) + 2 * (v_row * D + (((4 * db + 2 * gid + ((i16 & 3) >> 1)) ^ v_swz) << 3) + 4 * (i16 & 1));

  // ---- a slot of the tile stream: one key tile of one item, with the cache-block ids its request needs (this wave's
  //      quarter of the tile, and the block of the item's frontier)
  struct Slot {
    int kt, ke, wg_max, seq;
    const int32_t* row;  // the stream's block-table row
    int64_t head_off;    // element offset of the kv head inside a cache row
    int id, last_id;
    int live;            // an int: a bool would leave tail padding that struct copies drag through memory
  };
  i32x8 d1, d2;
  int seq0 = 0;                         // d0 is the seq0-th item of this workgroup
  auto first_slot = [&](const i32x8& d, int seq) {
    Slot s;
    s.kt = d[5] & 0xffff; s.ke = d[5] >> 16; s.wg_max = d[4]; s.seq = seq;
    s.row = p.block_table + static_cast<int64_t>(d[3] >> 8) * p.max_blocks;
    s.head_off = static_cast<int64_t>(d[3] & 255) * p.stride_head;
    s.id = 0; s.last_id = 0;
    s.live = (d[5] >> 16) > 0 ? 1 : 0;
    return s;
  };
  auto successor = [&](const Slot& c) {
    if (c.kt + 1 < c.ke) {
      Slot s = c;
      s.kt = c.kt + 1;
      return s;
    }
    const int rel = c.seq + 1 - seq0;                       // 1 or 2
    return first_slot(rel == 1 ? d1 : d2, c.seq + 1);
  };
  auto request_ids = [&](Slot& s) {
    const int last_blk = max(s.wg_max, 0) >> 4;           // CS_KV_BLOCK = 16
    s.id = sload1(s.row + min(s.kt * 4 + wave, last_blk));
    s.last_id = sload1(s.row + last_blk);
  };
  // A tile request is 8 DMA instructions per wave (4 for K, 4 for V), each moving 1 KiB.  Issued back to back they hold the
  // wave for hundreds of cycles: regular tiles are issued one instruction at a time between the matrix instructions of the S
  // phase, with a wave-uniform base and the lane's constant offset.  The S phase always issues its eight parts, so that no
  // branch splits it: when there is nothing to request (the next tile holds a frontier and went out at once, or there is
  // none) they re-read the current tile's cache block into a 1-KiB sink.
  const uint16_t *req_k = nullptr, *req_v = nullptr;
  uint32_t req_dst_k = 0, req_dst_v = 0, req_step = 0;
  const uint32_t lds_k0 = lds_address(&sK[0][wave * IPW * 512]), lds_v0 = lds_address(&sV[0][wave * IPW * 512]);
  const uint32_t lds_sink = lds_address(&s_sink[wave][0]);
  auto request_part = [&](int part) {
    const int i = part & 3;
    if (part < 4) dma16_sa(k_off[i], req_k, req_dst_k + i * req_step);
    else dma16_sa(v_off[i], req_v, req_dst_v + i * req_step);
  };
  auto prepare = [&](const Slot& s, uint32_t dst_k, uint32_t dst_v, uint32_t step) {
    // (a block spans fewer than 2^31 elements: the host checks the slot stride)
    const int64_t at = s.head_off + static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(s.id)) *
                                                         static_cast<uint32_t>(blk_stride));
    req_k = kall + at;
    req_v = vall + at;
    req_dst_k = dst_k;
    req_dst_v = dst_v;
    req_step = step;
  };
  auto prepare_sink = [&](const Slot& s) { prepare(s, lds_sink, lds_sink, 0); };
  auto prepare_regular = [&](const Slot& s, int stage) { prepare(s, lds_k0 + stage * (TILE * 2), lds_v0 + stage * (TILE * 2), 1024); };
  auto issue = [&](const Slot& s, int stage) {     // the whole request at once
    if (s.kt != s.wg_max / kBN) {
      prepare_regular(s, stage);
#pragma unroll
      for (int part = 0; part < 2 * IPW; ++part) request_part(part);
      return;
    }
    // the tile that holds the frontier of its item: rows past the frontier may be unallocated or hold anything, they
    // fetch the frontier row instead (finite data, weight 0 after masking)
    const uint16_t* kg = kall + s.head_off;
    const uint16_t* vg = vall + s.head_off;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int q = wave * IPW + i;
      const int j_un = s.kt * kBN + 4 * q + l_row;
      const bool over = j_un > s.wg_max;
      const int j = over ? s.wg_max : j_un;
      const int64_t slot = static_cast<int64_t>(over ? s.last_id : s.id) * CS_KV_BLOCK + j % CS_KV_BLOCK;
      dma16(kg + slot * p.stride_slot + k_chunk[i] * 8, &sK[stage][q * 512]);
      dma16(vg + slot * p.stride_slot + v_chunk[i] * 8, &sV[stage][q * 512]);
    }
  };

  // ---- per-item state of the lane
  bf16x8 qf[STEPS];
  int lim_raw = 0, it_tok_head = 0;
  bool it_valid = false;
  int it_rows_left = 0;                 // rows of the stream at and after this wave's first row
  auto load_item = [&](const i32x8& d) {
    it_rows_left = d[1] - (d[2] + wave * 32);
    const int row = d[2] + wave * 32 + n;
    it_valid = row < d[1];
    const int row_c = it_valid ? row : d[1] - 1;
    const int tq = row_c / p.group;
    const int tok = d[0] + tq;
    it_tok_head = tok * p.n_q_heads + (d[3] & 255) * p.group + (row_c - tq * p.group);
    const uint16_t* qrow = static_cast<const uint16_t*>(p.q) + static_cast<int64_t>(it_tok_head) * D;
#pragma unroll
    for (int st = 0; st < STEPS; ++st)
      qf[st] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const cs::u32x4*>(qrow + 16 * st + 8 * h));
    lim_raw = min(p.q_pos[tok], d[4]);      // d[4]: the tile's frontier, already inside the stream's entries
  };

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = zero16;
  float m_run = kNegInf, l_run = 0.f;
  int lim = -1, wave_min = -1, wave_max = -1;
  const float slack = kMaxSlack / p.scale_log2e;

  auto compute = [&](int kt, int stage) {
    const int j0 = kt * kBN;
    f32x16 sacc[2];
    constexpr int KPF = 2;        // K fragments are read two steps ahead of their matrix instructions
    bf16x8 ka[KPF + 1][2];
    typedef __attribute__((address_space(3))) const cs::u32x4 lds_u32x4;
    // LDS addresses of this tile's fragments: one add per address and tile; pinned in registers, so that every read folds
    // its row-group offset into the instruction's immediate field
    const uint32_t stage_off = static_cast<uint32_t>(stage) * (TILE * 2);
    uint32_t kad[STEPS], va[DB];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      kad[st] = k_addr[st] + stage_off;
      asm volatile("" : "+v"(kad[st]));
    }
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      va[db] = v_addr[db] + stage_off;
      asm volatile("" : "+v"(va[db]));
    }
    auto k_frag = [&](int st, int kb) {
      return __builtin_bit_cast(bf16x8, reinterpret_cast<lds_u32x4*>(static_cast<uintptr_t>(kad[st]))[kb * 32 * D * 2 / 16]);
    };
#pragma unroll
    for (int st = 0; st < KPF; ++st) {
      ka[st][0] = k_frag(st, 0);
      ka[st][1] = k_frag(st, 1);
    }
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      if (st + KPF < STEPS) {
        ka[(st + KPF) % (KPF + 1)][0] = k_frag(st + KPF, 0);
        ka[(st + KPF) % (KPF + 1)][1] = k_frag(st + KPF, 1);
      }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[st % (KPF + 1)][kb], qf[st], st == 0 ? zero16 : sacc[kb], 0, 0, 0);
      request_part(st);
    }
    // pin that order (the scheduler would otherwise pull each read back to just before its use)
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * KPF, 0);
#pragma unroll
    for (int st = 0; st < STEPS - KPF; ++st) {
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * KPF, 0);
    if (j0 + kBN - 1 > wave_min) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = j0 + 32 * kb + 8 * (r / 4) + 4 * h + (r % 4);
          if (key > lim) sacc[kb][r] = kNegInf;
        }
    }
    float t_max = kNegInf;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) t_max = fmaxf(t_max, sacc[kb][r]);
    // the two half-waves hold the same queries
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(t_max), __float_as_uint(t_max), false, false);
    t_max = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    if (__any(t_max > m_run + slack)) {
      const bool up = t_max > m_run + slack;
      const float m_new = up ? t_max : m_run;
      const float alpha = up ? __builtin_amdgcn_exp2f((m_run - m_new) * p.scale_log2e) : 1.f;
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    }
    const float m_scaled = (m_run == kNegInf ? 0.f : m_run) * p.scale_log2e;
    bf16x8 pb[2][2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        cs::u32x4 w;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float e0 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * mm + 2 * c], p.scale_log2e, -m_scaled));
          const float e1 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * mm + 2 * c + 1], p.scale_log2e, -m_scaled));
          const uint32_t pk = pack_bf16x2(e0, e1);
          l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), __builtin_bit_cast(bf16x2, 0x3f803f80u), l_run, false);
          w[c] = pk;
        }
        pb[kb][mm] = __builtin_bit_cast(bf16x8, w);
      }
    // 16 matrix instructions, m = (key block, key half, d block); V^T fragments are read VPF of them ahead
    constexpr int VPF = 3;
    s16x4 vlo[VPF + 1], vhi[VPF + 1];
    auto v_frag = [&](int m) {
      const int g0 = (32 * (m >> 3) + 16 * ((m >> 2) & 1)) * D;
      const uint32_t a = va[m & 3];
      vlo[m % (VPF + 1)] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(((lds_s16x4*)(static_cast<uintptr_t>(a))) + g0 * 2 / 8);
      vhi[m % (VPF + 1)] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(((lds_s16x4*)(static_cast<uintptr_t>(a))) + (g0 + 8 * D) * 2 / 8);
    };
#pragma unroll
    for (int m = 0; m < VPF; ++m) v_frag(m);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      if (m + VPF < 16) v_frag(m + VPF);
      const s16x8 a = __builtin_shufflevector(vlo[m % (VPF + 1)], vhi[m % (VPF + 1)], 0, 1, 2, 3, 4, 5, 6, 7);
      o[m & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pb[m >> 3][(m >> 2) & 1], o[m & 3], 0, 0, 0);
    }
  };

  // Normalises and stores the rows of the finished item, then clears the accumulators.
  auto finish_item = [&](int tok_head, bool valid) {
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (valid) {
      const float inv = __builtin_amdgcn_rcpf(l_tot);      // 1 ulp: far below the bf16 result's rounding
      uint16_t* orow = static_cast<uint16_t*>(p.out) + static_cast<int64_t>(tok_head) * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          cs::u32x2 w;
          w.x = pack_bf16x2(o[db][4 * rq + 0] * inv, o[db][4 * rq + 1] * inv);
          w.y = pack_bf16x2(o[db][4 * rq + 2] * inv, o[db][4 * rq + 3] * inv);
          *reinterpret_cast<cs::u32x2*>(orow + 32 * db + 8 * rq + 4 * h) = w;
        }
    }
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = zero16;
    m_run = kNegInf;
    l_run = 0.f;
  };

  // ---- prologue: first item, first tile request, the next two items, block ids of the second slot
  Slot cur = first_slot(d0, 0);
  request_ids(cur);
  d1 = sload8(item_at(d0[6]));
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(cur.id), "+s"(cur.last_id), "+s"(d1));
  issue(cur, 0);
  d2 = sload8(item_at(d1[6]));
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(d2));
  Slot nxt = successor(cur);
  request_ids(nxt);
  load_item(d0);
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(nxt.id), "+s"(nxt.last_id));
  bool new_item = true, ep_pending = false, ep_valid = false;
  int ep_tok_head = 0;
  int stage = 0;

  for (;;) {
    // everything requested so far has landed: the tile of `cur`, and at an item boundary the queries and frontier of its
    // item (telling the compiler so here keeps it from waiting for them later, when that wait would also cover the tile
    // request issued below)
    wait_vmcnt<0>();
#pragma unroll
    for (int st = 0; st < STEPS; ++st) asm volatile("" : "+v"(qf[st]));
    asm volatile("" : "+v"(lim_raw));
    __syncthreads();                     // every wave's share landed; every wave left the other stage
    if (new_item) {
      lim = it_valid ? lim_raw : -1;
      const int rows_here = min(32, it_rows_left);        // rows of this wave that exist; positions do not decrease along them
      wave_min = rows_here > 0 ? __builtin_amdgcn_readlane(lim, 0) : -1;
      wave_max = rows_here > 0 ? __builtin_amdgcn_readlane(lim, max(rows_here, 1) - 1) : -1;
      new_item = false;
    }
    // request the next tile: at once if it holds the frontier of its item or if this wave has nothing to compute in this
    // step, else spread over the S phase of this step
    const bool computes = cur.kt * kBN <= wave_max;
    if (nxt.live && computes && nxt.kt != nxt.wg_max / kBN) {
      prepare_regular(nxt, stage ^ 1);
    } else {
      if (nxt.live) issue(nxt, stage ^ 1);
      prepare_sink(cur);
    }
    // scalar requests for later steps: block ids of the slot after next; at the last tile of an item also the descriptor
    // three items ahead.  Always issued, towards harmless addresses when there is nothing to fetch: a conditional request
    // would let the compiler merge the pending register with another value before the wait
    const bool cur_last = cur.kt + 1 == cur.ke;
    Slot nn = nxt.live ? successor(nxt) : nxt;
    request_ids(nn);
    i32x8 d3 = sload8(cur_last ? item_at(d2[6]) : p.ws_plan + kHdrEndItem);

    if (ep_pending) {
      finish_item(ep_tok_head, ep_valid);
      ep_pending = false;
    }
    if (computes) compute(cur.kt, stage);

    asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(nn.id), "+s"(nn.last_id), "+s"(d3));
    if (cur_last) {
      ep_pending = true;
      ep_tok_head = it_tok_head;
      ep_valid = it_valid;
      if ((d1[5] >> 16) > 0) {
        load_item(d1);
        new_item = true;
      }
      d0 = d1; d1 = d2; d2 = d3;
      ++seq0;
    }
    if (!nxt.live) break;
    cur = nxt;
    nxt = nn;
    stage ^= 1;
  }
  finish_item(ep_tok_head, ep_valid);
  wait_vmcnt<0>();                       // no request may land after the workgroup's LDS has been given on
}

// Merges the partial results of split row tiles: out = sum_c w_c O_c / sum_c w_c l_c with
// w_c = 2^((m_c - max_c m_c) * scale * log2 e).  One workgroup per 8 rows; 32 threads per row.
__global__ __launch_bounds__(256) void window_attn_merge_kernel(AttnParams p) {
  constexpr int D = 128;
  const int groups = p.bm / 8;
  const int item = blockIdx.x / groups;              // < the row-tile capacity the grid was sized for
  const int32_t* d = p.ws_desc + item * 8;
  const int n_split = d[4];
  if (n_split <= 1) return;
  const int q0 = d[0], rows_total = d[1], r_tile = d[2], kvh = d[3];
  const int sub = threadIdx.x & 31;                    // 4 consecutive output dims
  const int rl = (blockIdx.x - item * groups) * 8 + (threadIdx.x >> 5);
  const int row = r_tile + rl;
  if (row >= rows_total) return;
  const int first = d[5], doubled = d[6];              // see plan_spans
  // one pass, four key ranges at a time: all loads of a batch are independent of each other and
  // of the running maximum (rows a range did not see hold m = -inf, l = 0, O = 0)
  float m_all = kNegInf, l_all = 0.f;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < n_split; c0 += 4) {
    float2 ml[4];
    float4 t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = min(c0 + u, n_split - 1);
      const int64_t pr = static_cast<int64_t>(first + c + min(c, doubled)) * p.bm + rl;
      ml[u] = *reinterpret_cast<const float2*>(p.ws_ml + pr * 2);
      t[u] = *reinterpret_cast<const float4*>(p.ws_o + pr * D + 4 * sub);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (c0 + u >= n_split || ml[u].x == kNegInf) continue;
      const float m_new = fmaxf(m_all, ml[u].x);
      const float a = m_all == kNegInf ? 0.f : __builtin_amdgcn_exp2f((m_all - m_new) * p.scale_log2e);
      const float w = __builtin_amdgcn_exp2f((ml[u].x - m_new) * p.scale_log2e);
      m_all = m_new;
      l_all = fmaf(w, ml[u].y, l_all * a);
      acc[0] = fmaf(w, t[u].x, acc[0] * a); acc[1] = fmaf(w, t[u].y, acc[1] * a);
      acc[2] = fmaf(w, t[u].z, acc[2] * a); acc[3] = fmaf(w, t[u].w, acc[3] * a);
    }
  }
  const float inv = 1.f / l_all;
  const int tok = q0 + row / p.group;
  const int head = kvh * p.group + row % p.group;
  uint16_t* orow = static_cast<uint16_t*>(p.out) + (static_cast<int64_t>(tok) * p.n_q_heads + head) * D;
  cs::u32x2 w2;
  w2.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
  w2.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
  *reinterpret_cast<cs::u32x2*>(orow + 4 * sub) = w2;
}

// ------------------------------------------------------------------------------------------
// fp32: a workgroup = 8 waves = 32 rows (query token, query head of one kv group) of one stream; the
// waves take every eighth tile of 32 keys and merge their partial results through LDS at the end, so
// that a short window still puts eight waves on its few row tiles and the sums over the keys stay
// short.  Both contractions run on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: products and
// sums in fp32), fed from global memory / L2 without staging: its operands are one float per lane and
// an instruction takes 64 cycles, so a wave's loads keep ahead of it.
//   S^T = K Q^T    half h of the wave contributes d = 8 i + 4 h + j (16-byte loads of K and Q rows),
//                  even and odd i in accumulators of their own (two chains of D/2 sums)
//   O^T += V^T P^T step r contracts the two keys that register r of S^T holds in the two halves
// A tile's P V is summed from zero and then added to the running output, so no chain of sums is longer
// than 32 + (tiles of the wave).  What bounds it: matrix instructions on long windows, the chain
// block table -> K -> S -> V of a wave's few tiles on short ones.
// Measured against one token and head per wave with the keys dealt to lanes (which read every K/V row
// once per query head, 64 rows scattered over the lanes of each load): 337 tokens, 2 heads of 64,
// 452 keys 41.5 -> 19.6 us; 424 tokens, 28 heads of 128, 919 keys 959 -> 58.7 us; 2,082 tokens, 6,033
// keys 30.1 -> 1.63 ms (83 TFLOP/s of the 157 the unit has).  Error against 64 bits 2.1e-7..3.0e-7
// before, 1.6e-7..2.1e-7 now.
constexpr int kF32Rows = 32, kF32Keys = 32, kF32Waves = 8;

template <int D>
__global__ __launch_bounds__(64 * kF32Waves, 2) void window_attn_f32_kernel(AttnParams p) {
  constexpr int DB = D / 32, VECS = D / 8;
  __shared__ float s_o[kF32Waves / 2][DB * 16][64];
  __shared__ float s_ml[kF32Waves / 2][2][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, h = lane >> 5;

  RowTile rt;
  if (!find_row_tile<kF32Rows, kF32Waves>(p, blockIdx.x, reinterpret_cast<int*>(&s_o[0][0][0]), rt)) return;
  const int s = __builtin_amdgcn_readfirstlane(rt.s), kvh = __builtin_amdgcn_readfirstlane(rt.kvh);
  const int q0 = __builtin_amdgcn_readfirstlane(rt.q0), rows_total = __builtin_amdgcn_readfirstlane(rt.rows_total);
  const int r_tile = __builtin_amdgcn_readfirstlane(rt.r_tile);
  const int32_t* bt = p.block_table + static_cast<int64_t>(s) * p.max_blocks;
  const int cap = min(p.kv_len[s], p.max_blocks * CS_KV_BLOCK) - 1;

  const int row = r_tile + n;
  const bool valid = row < rows_total;
  const int row_c = valid ? row : rows_total - 1;
  const int tok = q0 + row_c / p.group;
  const int head = kvh * p.group + row_c % p.group;
  const int lim = valid ? min(p.q_pos[tok], cap) : -1;
  int top = lim, low = valid ? lim : 0x7fffffff;         // highest and lowest frontier of the rows
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) {
    top = max(top, __shfl_xor(top, off));
    low = min(low, __shfl_xor(low, off));
  }
  top = __builtin_amdgcn_readfirstlane(top);
  low = __builtin_amdgcn_readfirstlane(low);
  if (top < 0) return;                    // no row sees a cache entry (the same in every wave): rows left untouched
  const int n_key_tiles = top / kF32Keys + 1;

  const int64_t q_at = (static_cast<int64_t>(tok) * p.n_q_heads + head) * D;
  const float* qrow = static_cast<const float*>(p.q) + q_at;
  float4 qv[VECS];
#pragma unroll
  for (int i = 0; i < VECS; ++i) qv[i] = *reinterpret_cast<const float4*>(qrow + 8 * i + 4 * h);

  f32x16 o[DB];
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = zero16;
  float m = kNegInf, l = 0.f;
  const float* kb = static_cast<const float*>(p.k) + kvh * p.stride_head;
  const float* vb = static_cast<const float*>(p.v) + kvh * p.stride_head;
  const int last_blk = top / CS_KV_BLOCK;

  for (int kt = wave; kt < n_key_tiles; kt += kF32Waves) {
    const int j0 = kt * kF32Keys;
    // rows past the highest frontier may be unallocated: their lanes take the frontier row (weight 0)
    const int64_t blk0 = bt[2 * kt], blk1 = bt[min(2 * kt + 1, last_blk)];
    auto slot_of = [&](int j) {                          // j inside this tile
      const int jc = min(j, top);
      return (jc - j0 < CS_KV_BLOCK ? blk0 : blk1) * CS_KV_BLOCK + jc % CS_KV_BLOCK;
    };
    const float* kr = kb + slot_of(j0 + n) * p.stride_slot + 4 * h;
    f32x16 sa = zero16, sb = zero16;
#pragma unroll
    for (int i = 0; i < VECS; ++i) {
      const float4 t = *reinterpret_cast<const float4*>(kr + 8 * i);
      f32x16& c = i & 1 ? sb : sa;
      if (i == VECS / 2) __builtin_amdgcn_sched_barrier(0);            // half of the row in registers at a time
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(t.x, qv[i].x, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(t.y, qv[i].y, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(t.z, qv[i].z, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(t.w, qv[i].w, c, 0, 0, 0);
    }
    // register r is key j0 + 8 (r / 4) + 4 h + r % 4 of query n
    float sc[16], t_max = kNegInf;
    const bool straddles = j0 + kF32Keys - 1 > low;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = (sa[r] + sb[r]) * p.scale;
      if (straddles && j0 + 8 * (r / 4) + 4 * h + r % 4 > lim) sc[r] = kNegInf;
      t_max = fmaxf(t_max, sc[r]);
    }
    t_max = fmaxf(t_max, __shfl_xor(t_max, 32));
    const float m_new = fmaxf(m, t_max);
    const float m_ref = m_new == kNegInf ? 0.f : m_new;  // a row that sees none of these keys
    const float alpha = expf(m - m_ref);                 // exp(-inf) = 0 on the first keys
    float l_tile = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = expf(sc[r] - m_ref);
      l_tile += sc[r];
    }
    l = fmaf(l, alpha, l_tile);
    m = m_new;
    // a value row that is masked for some of the queries takes part in the product with weight 0: one
    // that is not finite must not reach them
    bool finite = true;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      float vv[16];
#pragma unroll
      for (int r = 0; r < 16; ++r)
        vv[r] = vb[slot_of(j0 + 8 * (r / 4) + 4 * h + r % 4) * p.stride_slot + 32 * db + n];
      f32x16 t = zero16;
#pragma unroll
      for (int r = 0; r < 16; ++r) t = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[r], sc[r], t, 0, 0, 0);
      if (straddles) {
#pragma unroll
        for (int r = 0; r < 16; ++r) finite = finite && fabsf(vv[r]) < INFINITY;
        if (__any(!finite)) {
          t = zero16;
#pragma unroll 1
          for (int key = 0; key < kF32Keys; ++key) {
            const int r = 4 * (key / 8) + key % 4, hh = (key >> 2) & 1;
            float mine = 0.f;
#pragma unroll
            for (int k = 0; k < 16; ++k) mine = k == r ? sc[k] : mine;
            const float w = __shfl(mine, n + 32 * hh);
            const float* vr = vb + slot_of(j0 + key) * p.stride_slot + 32 * db;
            if (j0 + key <= lim) {
#pragma unroll
              for (int k = 0; k < 16; ++k) t[k] = fmaf(w, vr[8 * (k / 4) + 4 * h + k % 4], t[k]);
            }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] = fmaf(o[db][r], alpha, t[r]);
    }
  }

  // ---- the waves' partial results: the upper half of the waves hands over to the lower half, three times
  float l_all = l + __shfl_xor(l, 32);
#pragma unroll
  for (int half = kF32Waves / 2; half > 0; half >>= 1) {
    if (wave >= half && wave < 2 * half) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) s_o[wave - half][db * 16 + r][lane] = o[db][r];
      s_ml[wave - half][0][lane] = m;
      s_ml[wave - half][1][lane] = l_all;
    }
    __syncthreads();
    if (wave < half) {
      const float m_o = s_ml[wave][0][lane], l_o = s_ml[wave][1][lane];
      const float m_new = fmaxf(m, m_o);
      const float a = m == kNegInf ? 0.f : expf(m - m_new), b = m_o == kNegInf ? 0.f : expf(m_o - m_new);
      l_all = fmaf(l_all, a, l_o * b);
      m = m_new;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = fmaf(o[db][r], a, s_o[wave][db * 16 + r][lane] * b);
    }
    __syncthreads();
  }
  if (wave == 0 && lim >= 0) {            // register r of block db is d = 32 db + 8 (r / 4) + 4 h + r % 4
    const float inv = 1.f / l_all;
    float* orow = static_cast<float*>(p.out) + q_at;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq)
        *reinterpret_cast<float4*>(orow + 32 * db + 8 * rq + 4 * h) =
            make_float4(o[db][4 * rq] * inv, o[db][4 * rq + 1] * inv, o[db][4 * rq + 2] * inv, o[db][4 * rq + 3] * inv);
  }
}

// Launch shape and workspace layout of the bf16 / head_dim 128 path, shared by the workspace
// query and the call.
struct AttnPlan {
  int64_t r_cap;         // upper bound on row tiles per kv head
  int64_t rt_cap;        // ... times kv heads
  int64_t items_cap;     // upper bound on work items
  int max_tiles;         // key tiles of the longest sweep
  int grid;              // persistent workgroups: 8 XCDs x up to kWorkgroupsPerXcd, or twice as many
  int solo;              // whole sweeps in the kernel of 32 rows a wave
  int bm;                // rows per item
  int hist_pitch;        // buckets of the planner's counting sort, per XCD
  int span, pref_pitch;  // span plan (see plan_spans) and the ints per XCD of its prefix array
  size_t off_pref;
  size_t off_items, off_rt_desc, off_st_toff, off_st_work, off_st_rank, off_rt_stream, off_rt_wgmax,
      off_un_head, off_st_uoff, off_hist, off_ml, off_o, total;
};

// Launches that run whole sweeps from a plan, by 128-row tiles x kv heads and key tiles of the longest window (see
// tile_route_128).
bool whole_sweeps(int64_t row_tiles, int key_tiles, int n_kv_heads) {
  if (row_tiles >= 1024) return true;
  return row_tiles >= (n_kv_heads > 4 ? 768 : 512) && key_tiles > 8 && key_tiles <= 32;
}

// Of those from 1,024 row tiles on, launches whose row tiles are jobs of their own (window_attn_bf16_rows32_kernel), by the
// mean of the streams' rows, the row tiles T and the key tiles.  us a layer of REUSE calls, jobs of 256 rows / this kernel,
// streams alike (five head layouts) and, in brackets, of 0.4 to 1.6 times the rows and keys:
//   up to 260 rows, 300 keys  T 1,100 46.5 / 33 (41 / 33), T 2,600 72 / 60 (67 / 60); 700 keys T 1,100 78 / 56 (66 / 62),
//                             T 2,600 1.16 times as long (1.03), T 5,000 1.11 (1.01); 1,300 keys 1.26 to 1.11 (1.03 to 1.00);
//                             47 key tiles 1.08 to 0.98; 75 key tiles (1.00 to 0.95)
//   up to 400                 300 and 700 keys 1.37 to 1.11 (1.17 to 0.99), 1,300 keys 1.31 to 1.11 (1.02 to 0.98), 47 key tiles
//                             1.18 to 1.04, 75 (0.97 to 0.94)
//   up to 1,400               T below 2,000: 640 rows 1.23 to 1.10 (1.18 to 0.97), 1,000 rows 1.18 to 1.04 (1.08 to 0.97), 1,300 rows
//                             1.09 to 1.03 (1.03 to 0.92); 33 key tiles (1.00 to 0.92).  T above: 640 rows 1.13 to 1.03
//                             (1.04 to 0.96), 1,000 rows 1.03 to 0.97 (1.02 to 0.94).  Whole steps of 10 to 31 layers with 1,070 to
//                             1,400 rows, streams as they come: T 1,048 to 1,820 1.02 to 0.99, T 1,860 to 2,324 0.99 to 0.97
//   beyond                    1,700 rows 1.01 to 0.94, 2,400 rows 1.03 to 0.92
// (1,024 row tiles of at most 1,400 rows a stream are 86 pairs at least: the planner deals by pair.)
bool solo_row_tiles(int64_t n_q, int32_t n_streams, int32_t group, int64_t row_tiles, int key_tiles) {
  const int64_t rows = n_q * group;
  return row_tiles >= 1024 && ((rows <= 400ll * n_streams && key_tiles <= 48) || (rows <= 1400ll * n_streams && key_tiles <= 24 && row_tiles < 1800));
}

AttnPlan plan_attn(int64_t n_q, int32_t n_streams, int32_t group, int32_t n_kv_heads, int32_t max_blocks) {
  AttnPlan a;
  a.bm = kBM;
  a.r_cap = (n_q * group) / a.bm + n_streams;
  a.rt_cap = a.r_cap * n_kv_heads;
  a.max_tiles = static_cast<int>((static_cast<int64_t>(max_blocks) * CS_KV_BLOCK + kBN - 1) / kBN);
  // split long key sweeps when the row tiles alone cannot fill the chip a couple of times over
  a.span = !whole_sweeps(a.rt_cap, a.max_tiles, n_kv_heads) && a.max_tiles > 4 ? 1 : 0;
  static_assert(kSpanUnits >= 1024, "a split launch has fewer than 1,024 row tiles");
  // span plan: every cut adds an item to each row tile of a unit, and an item's list position names its partial-result slot
  a.items_cap = a.span ? a.rt_cap + 2 * 8 * kWorkgroupsPerXcd : a.rt_cap;
  a.pref_pitch = static_cast<int>(a.rt_cap / 8 + 2);
  const int64_t per_xcd = (a.items_cap + 7) / 8;
  a.solo = solo_row_tiles(n_q, n_streams, group, a.rt_cap, a.max_tiles) ? 1 : 0;
  const int64_t most = a.solo ? kSlotsPerXcd : kWorkgroupsPerXcd;
  a.grid = 8 * static_cast<int>(per_xcd < most ? per_xcd : most);
  size_t at = kPlanHeaderInts * sizeof(int32_t);
  auto take = [&](size_t bytes) {
    const size_t here = (at + 255) & ~static_cast<size_t>(255);
    at = here + bytes;
    return here;
  };
  a.off_items = take(static_cast<size_t>(a.items_cap) * 8 * sizeof(int32_t));
  a.off_rt_desc = take(static_cast<size_t>(a.rt_cap) * 8 * sizeof(int32_t));
  a.off_st_toff = take((static_cast<size_t>(n_streams) + 1) * sizeof(int32_t));
  a.off_st_work = take(static_cast<size_t>(n_streams) * sizeof(int32_t));
  a.off_st_rank = take(static_cast<size_t>(n_streams) * sizeof(int32_t));
  a.off_rt_stream = take(static_cast<size_t>(a.r_cap) * sizeof(int32_t));
  a.off_rt_wgmax = take(static_cast<size_t>(a.r_cap) * sizeof(int32_t));
  a.off_un_head = take(static_cast<size_t>(a.r_cap) * sizeof(int32_t));
  a.off_st_uoff = take(static_cast<size_t>(n_streams) * sizeof(int32_t));
  const int64_t pair_rounds = (static_cast<int64_t>(n_streams) * n_kv_heads + 7) / 8;
  a.hist_pitch = static_cast<int>((a.max_tiles + 2 > pair_rounds ? a.max_tiles + 2 : pair_rounds) + 1);
  a.off_hist = take(static_cast<size_t>(8) * a.hist_pitch * sizeof(int32_t));
  a.off_pref = take(static_cast<size_t>(8) * a.pref_pitch * sizeof(int32_t));
  a.off_ml = take(a.span ? static_cast<size_t>(a.items_cap) * a.bm * 2 * sizeof(float) : 0);
  a.off_o = take(a.span ? static_cast<size_t>(a.items_cap) * a.bm * 128 * sizeof(float) : 0);
  a.total = (at + 255) & ~static_cast<size_t>(255);
  return a;
}

// head_dim 128: which launches leave the plan and the persistent kernel for the tile kernel, by 128-row tiles x kv
// heads and key tiles of the longest window.  Both are the caller's upper bounds (n_q, max_blocks): the host knows no
// other sizes, and the route has to be the same for all calls of a shape.  The row tiles that a launch then has are
// fewer (in the runs below, with budgets 12-40 % above the rows, 0.6-0.85 of T), so a caller that budgets closer stays
// on a route up to more work.  Below the lines of whole_sweeps the persistent kernel splits its sweeps and needs the merge
// launch; its plan costs 15-50 us a step.
// us a layer in a step, plan not counted, persistent / tile kernel (28/4 heads unless noted; T: row tiles):
//   whole sweeps from T 1,024  T 1,044 48 / 51, T 1,076 with 50 key tiles 89 / 98.  A BUILD call below runs in the tile kernel all the same,
//                              with the planning as one workgroup more (see window_attn_bf16_tile_and_plan_kernel)
//   ... from T 512 (768 with   no merge, and short lists are dealt by length.  us a step, plan included: T 928 1,477 / 1,751,
//   more than four kv heads),  T 752 1,223 / 1,277, T 520 1,069 / 1,130, T 632 with 22 key tiles 1,312 / 1,398, 16/4 heads T 544
//   9 to 32 key tiles          1,154 / 1,283, one kv head T 811 (16 layers) 856 / 1,012, 32/8 heads T 1,016 (16 layers) 960 / 1,064, T 880
//                              912 / 948, but T 744 1,473 / 1,462 (32 layers), T 608 1,331 / 1,334.  Longer sweeps on few workgroups:
//                              T 564 with 48 key tiles 2,158 / 2,059, T 624 with 59 2,695 / 2,682.  Below: T 472 1,250 / 1,199, T 404
//                              1,050 / 1,000, T 460 with 40 1,935 / 1,822 (T 496 one kv head 1,100 / 1,183)
//   kRows128 (what is left     past 64 key tiles the split wins: T 508 with 89 91 / 112, T 564 with 121 (32 rows a wave) 137 / 167
//   to 1,023)
//   kRows64Keys2 (to 440)      T 288 31.3 / 22.4; at T 520 its twice as many workgroups (two fit a CU) no longer all run
//                              at once: 37.1 (kRows128 35.0); past 48 key tiles level
//   kRows64Keys4 (to 128)      T 116 20.2 / 17.4, with 28 key tiles 28.3 / 24.9 (two groups 18.1, 28.7): one workgroup
//                              per CU, all of them run at once and the longest sweep is the time; up to 8 key tiles two
//                              groups are enough (300 keys 11.0 / 12.2, persistent 16.3)
//   kSplit64Keys4: few row     each in pieces of its keys, a workgroup of four key groups to a piece, and a merge launch.  As many pieces as
//   tiles with long sweeps     let all workgroups run at once (one a CU), by the 64-row tiles U of streams that are alike, and no more than
//                              one trip of the groups has tiles for.  us a layer, persistent of 32 rows a wave (no longer here) / of 64 / this:
//                              18 tokens of 28/4 heads, 215 key tiles 36.0 / 32.5 / 26.4; 2 of 16/4, 21 key tiles 13.5 / 16.5 / 11.4; U 16 18 key
//                              tiles 14.5 / 16.1 / 13.4, 72 23.6 / 23.5 / 18.2; U 48 24 21.5 / 20.3 / 15.3, 237 86 / 85 / 70; U 60 118 48.8 / 58.9 / 43.7
//                              (without a plan either: 16 key tiles, U 64 16.9 / 15.8 / 15.2, 13 level, below a whole sweep is as fast).
//                              Three pieces: U 78 20 21.2 / 19.9 / 18.3, 33 25.6 / 25.3 / 21.5, but 13 17.0 / 16.0 / 17.4; U 80 101 36 / 41 / 33,
//                              113 38 / 43 / 50, and with 16 key tiles U 72 to 80 15.2 to 15.5 / 15.9 to 16.9 (of 64 / this).  Two: U 104 72 52 / 58 / 43, U 128 48 33 / 32 / 28, 20 23.9 / 23.3 / 22.0, but U 112 17 17.1 / 15.8 /
//                              17.5; past 80 key tiles two pieces lose but for up to 64 rows a stream (persistent of 64 / this: U 104 65 30.3 / 28.4,
//                              107 79 32.8 / 31.9, 118 84 35.0 / 35.8, 122 96 35.7 / 38.4, 98 94 32.4 / 38.8); of up to 64 rows a stream, U 72 239 122 / 115 / 109, U 80 148
//                              91 / 89 / 75, U 116 122 107 / 98 / 92.  A piece more than fit at once costs 10-50 %, one fewer 0-20 %, hence the
//                              mean of U and the most that n_q rows can make
//   what is left of them (2    split from a plan: F row tiles without the streams' part-filled ones, persistent of 64 / tile: F 88 48 key tiles
//   key tiles > T, > 20 + 3/8 F)  36.5 / 31.0, F 64 55 35.4 / (pieces 30.8)
//   long sweeps of streams     whole in one launch: 39 streams of 11 tokens, 16/4 heads, 53 key tiles 60 / 65 / 49, 50 of 5, 73 key tiles 112 / 109 /
//   of up to 64 rows           93 (of 96 rows 24 streams, 50 key tiles 41 / 46 / 50)
//   single_tiles: whole        Up to 128 rows a stream and kv head on average.  The persistent kernel's jobs of 256 rows then hold one row tile,
//   sweeps, but one row tile   two of its four waves, and a plan orders nothing.  us a layer, persistent of 32 rows a wave, two workgroups a CU
//   a stream (kRows128)        (no longer here) / of 64 / tile: 18 tokens of 28/4 heads, 263 streams of 290 keys 45 / 63 / 51, of 550 88.5 / 99 / 95,
//                              of 1,000 144 / 153 / 145, 65 of 900 37 / 52 / 37, 1,025 of 550 309 / 314 / 316; 32 tokens of 32/8, 64 of 900 49 / 56 / 46;
//                              5 tokens of 28/4, 263 of 550 65 / 89 / 68; 4,000 to 8,300 keys 1 to 8 % below either.  Plans of 27-38 us (1,025 streams 97
//                              and 129) are not counted.  160 streams, every eighth of 118 tokens, the others of 2: 900 keys 92 / 104 / 91.  From two row
//                              tiles a stream on the persistent kernel wins: 27 tokens, 129 streams of 550 keys 53 / 58 / 72
enum class TileRoute { kNone, kRows128, kRows64Keys2, kRows64Keys4, kSplit64Keys4 };

struct TileChoice {
  TileRoute route;
  int pieces;          // kSplit64Keys4: of a sweep
};

// REUSE calls that read their own rows (`own`), of up to 64 streams: no refresh write goes ahead of the tile kernel, and its row
// tiles are listed by length, so it stays the faster one further up.  us a layer, REUSE calls of two launches / kRows128 /
// kRows64Keys2, with budgets 2 and 35 % above the rows (the row tiles that are there decide which of the two is the faster, the host
// knows the budget):
//   kRows64Keys2 up to 510     K 23 to 41, T 440 to 504: tight budgets 0.80 to 0.95 of two launches / 0.83 to 0.98, loose ones 0.81 to 0.95 / 0.71 to
//   row tiles T, 20 key tiles  0.92 (16/4 heads T 448 49.0 / 42.6 / 34.8, one stream of 32/8 T 496 63.2 / 64.5 / 55.0); but K 7 to 15 tight 0.78 to 0.93 / 0.93
//   K and more                 to 1.08, loose 0.76 to 0.90 / 0.84 to 0.95, and T 512 to 590 tight 0.77 to 1.03 / 0.94 to 1.23 (8/1 heads T 588, K 15
//                              36.6 / 34.8 / 47.9), loose 0.78 to 0.99 / 0.81 to 1.09
//   kRows128 up to 850         K 7 and 8 0.74 to 0.99; K 15 T 590 to 850 tight 0.73 to 1.03, loose 0.78 to 1.01; K 24 tight 0.88 to 1.06 (16/2 heads T 750 56.0
//                              / 59.3), loose 0.79 to 1.02; K 37 to 41 tight 0.79 to 1.03, loose 0.79 to 0.97; but 28/4 T 928 of 900 keys 776 / 802 a step
//                              of 16 layers, 8/1 T 878 846 / 849, 32/8 T 952 866 / 923
TileChoice tile_route_128(int64_t n_q, int32_t n_streams, int32_t group, int32_t n_kv_heads, int64_t row_tiles, int key_tiles, bool own) {
  const bool listed = own && n_streams <= 64;
  const int64_t rows = (n_q + n_streams - 1) / n_streams * group;                  // of a stream and kv head, if all are alike
  // 64-row tiles: as many as alike streams have, at most n_q * group / 64 + n_streams a kv head; the mean of the two
  const int64_t tiles64 = (((rows + 63) / 64 * n_streams + n_q * group / 64 + n_streams) * n_kv_heads + 1) / 2;
  if (whole_sweeps(row_tiles, key_tiles, n_kv_heads) && !(listed && row_tiles <= 850))
    return {n_q * group <= static_cast<int64_t>(kBM) * n_streams ? TileRoute::kRows128 : TileRoute::kNone, 1};
  const int64_t trips = (key_tiles + 3) / 4;
  const int pieces = static_cast<int>(256 / tiles64 < trips ? 256 / tiles64 : trips);
  if (pieces >= 4 || (pieces > 1 && key_tiles > (pieces == 3 ? 16 : 20) && (key_tiles <= (pieces == 2 ? 80 : 112) || rows <= 64)))
    return {TileRoute::kSplit64Keys4, pieces};
  if (rows <= 64 && tiles64 <= 256 && key_tiles > 48) return {TileRoute::kRows64Keys4, 1};
  if (key_tiles > 64) return {TileRoute::kNone, 1};
  if (row_tiles <= 128) {
    const int64_t full_tiles = n_q * group / kBM * n_kv_heads;
    if (2 * key_tiles > row_tiles && key_tiles > 20 + 3 * full_tiles / 8) return {TileRoute::kNone, 1};
    return {key_tiles > 8 ? TileRoute::kRows64Keys4 : TileRoute::kRows64Keys2, 1};
  }
  if (row_tiles <= (listed && key_tiles >= 20 ? 510 : 440) && key_tiles <= 48) return {TileRoute::kRows64Keys2, 1};
  if (row_tiles <= 440) return {TileRoute::kNone, 1};
  return {TileRoute::kRows128, 1};
}

template <int D, int ROWW, int KG, int STAGES>
int launch_tiles(const AttnParams& p, hipStream_t st) {
  const int64_t tiles = ((p.n_q * p.group) / (32 * ROWW) + p.n_streams) * p.n_kv_heads;      // upper bound
  if (tiles > 0x7fffffffll) return CS_EUNSUPPORTED;
  const dim3 grid(static_cast<unsigned>(tiles)), block(64 * ROWW * KG);
  if (p.ws_own) {
    // workgroups that run at once: two a CU, with four key groups one
    constexpr int kAtOnce = KG > 2 ? 256 : 512;
    const int idle = tiles < kAtOnce ? static_cast<int>(kAtOnce - tiles) / 8 : 0;
    AttnParams own = p;
    own.n_warm = KG > 1 ? 8 * (idle < kWarmPerXcd ? idle : kWarmPerXcd) : 0;
    hipLaunchKernelGGL((window_attn_bf16_tile_kernel<D, ROWW, KG, STAGES, false, true>), dim3(grid.x + own.n_warm), block, 0, st, own);
  } else hipLaunchKernelGGL((window_attn_bf16_tile_kernel<D, ROWW, KG, STAGES>), grid, block, 0, st, p);
  return cs::note_hip(hipGetLastError());
}

int launch_own_rows(const AttnParams& p, int bm, hipStream_t st) {
  const OwnParts parts(p, bm);
  const int64_t grid = parts.moves + parts.entries + parts.streams + parts.tiles;
  const dim3 blocks(static_cast<unsigned>(grid < (1 << 16) ? grid : 1 << 16));
  if (bm == 128) hipLaunchKernelGGL(window_attn_own_rows_kernel<128>, blocks, dim3(64), 0, st, p);
  else hipLaunchKernelGGL(window_attn_own_rows_kernel<64>, blocks, dim3(64), 0, st, p);
  return cs::note_hip(hipGetLastError());
}

int launch_split_tiles(const AttnParams& p, hipStream_t st) {
  const int64_t tiles = ((p.n_q * p.group) / p.bm + p.n_streams) * p.n_kv_heads;
  const dim3 grid(static_cast<unsigned>(tiles * p.pieces));
  if (p.ws_own) hipLaunchKernelGGL((window_attn_bf16_tile_kernel<128, 2, 4, 1, true, true>), grid, dim3(512), 0, st, p);
  else hipLaunchKernelGGL((window_attn_bf16_tile_kernel<128, 2, 4, 1, true>), grid, dim3(512), 0, st, p);
  const int e = cs::note_hip(hipGetLastError());
  if (e != CS_OK) return e;
  hipLaunchKernelGGL(window_attn_merge_kernel, dim3(static_cast<unsigned>(tiles * (p.bm / 8))), dim3(256), 0, st, p);
  return cs::note_hip(hipGetLastError());
}

}  // namespace

extern "C" size_t cs_window_prefill_attn_workspace(int64_t n_q, int32_t n_streams, int32_t n_q_heads,
                                                   int32_t n_kv_heads, int32_t head_dim,
                                                   int32_t max_blocks, int32_t dtype) {
  if (dtype != CS_BF16 || head_dim != 128 || n_q <= 0 || n_streams <= 0 || n_kv_heads < 1 ||
      n_q_heads < n_kv_heads || max_blocks <= 0)
    return 0;
  if (n_q_heads % n_kv_heads || n_q * n_q_heads >= (1ll << 31)) return 0;
  return plan_attn(n_q, n_streams, n_q_heads / n_kv_heads, n_kv_heads, max_blocks).total;
}

namespace {

// What calls with CS_ATTN_OWN_ROWS keep behind the workspace of the others: the table of own rows, then the row tiles of a
// launch without a plan (of 64 rows or more), then a pair of words a stream.  Where the others need no workspace (head_dim 64),
// a header goes ahead of it that holds the status word.
constexpr size_t kOwnHeaderBytes = 256;
static_assert(kHdrStatus * sizeof(int32_t) == CS_ATTN_STATUS_OFFSET && CS_ATTN_STATUS_OFFSET < kOwnHeaderBytes, "the status word is in the header");
size_t own_offset(size_t attn_bytes) { return attn_bytes ? attn_bytes : kOwnHeaderBytes; }

// REUSE calls with the flag read their own rows in shapes that run without a plan, as long as T row tiles of 128 times K key
// tiles are no more than this: the row tiles then hide a launch of 2-4 us and the refresh write, but ask for the place of every
// cache block's rows, about 2 % of a sweep.  us a layer of REUSE calls, own rows / refresh write and attention:
//   head_dim 128, streams of one row tile  T 1,968 with K 16 132.6 / 134.8, T 968 with 63 184 / 191, T 7,708 with 9 290 / 298 (69,000), but T
//                 1,968 with 63 438 / 432 (124,000), with 125 837 / 825
//   head_dim 64   64 streams of 8/1 heads T 5,244 with 47 210 / 220, 9,655 with 47 532 / 564 (454,000), T 7,168 of 16/4 with 24 253 / 264, 5,048 of 4/4
//                 with 47 313 / 359, but 19,247 with 94 2,095 / 1,826, 19,436 of 16/4 with 47 1,142 / 1,058, 21,232 of 32/8 with 32 897 / 866 (680,000),
//                 one stream, 1,579 with 470 719 / 690
constexpr int64_t kOwnWork128 = 100000, kOwnWork64 = 1 << 19;

// Rows of the row tiles that such calls list; 0: a call with the flag attends as one without.
int own_row_tile(int64_t n_q, int32_t n_streams, int32_t group, int32_t n_kv_heads, int32_t head_dim, int32_t max_blocks) {
  const int64_t row_tiles = (n_q * group / kBM + n_streams) * n_kv_heads;
  const int64_t key_tiles = (static_cast<int64_t>(max_blocks) * CS_KV_BLOCK + kBN - 1) / kBN;
  if (row_tiles * key_tiles > (head_dim == 128 ? kOwnWork128 : kOwnWork64)) return 0;
  if (head_dim == 64) return kBM;
  const TileRoute route = tile_route_128(n_q, n_streams, group, n_kv_heads, row_tiles, static_cast<int>(key_tiles), true).route;
  return route == TileRoute::kNone ? 0 : route == TileRoute::kRows128 ? 128 : 64;
}
size_t own_table_bytes(int32_t n_streams, int32_t max_blocks) {
  return (static_cast<size_t>(n_streams) * max_blocks * sizeof(cs::u32x2) + 255) & ~static_cast<size_t>(255);
}
size_t own_tiles_bytes(int64_t n_q, int32_t n_streams, int32_t group, int32_t n_kv_heads) {
  return static_cast<size_t>((n_q * group / 64 + n_streams) * n_kv_heads) * 8 * sizeof(int32_t);
}
size_t own_bytes(int64_t n_q, int32_t n_streams, int32_t group, int32_t n_kv_heads, int32_t max_blocks) {
  return own_table_bytes(n_streams, max_blocks) + own_tiles_bytes(n_q, n_streams, group, n_kv_heads) + static_cast<size_t>(n_streams) * sizeof(cs::u32x2);
}

// The attention call; with k_new != nullptr the launch first writes the new K/V rows into the cache
// (bf16 / head_dim 128: inside the same launch; other shapes: the caller has already queued the
// refresh write as a launch of its own).
// The argument checks of the attention call that need no device: an error code, CS_OK (go on), or
// kAttnNothingToDo (valid arguments, empty launch).
constexpr int kAttnNothingToDo = 1;

int attn_validate(const void* q, const void* k_cache_layer, const void* v_cache_layer,
                  const int32_t* cu_q, const int32_t* q_pos, const int32_t* kv_len,
                  const int32_t* block_table, int32_t max_blocks, int32_t block_size,
                  const void* out, int64_t n_q, int32_t n_streams, int32_t n_q_heads,
                  int32_t n_kv_heads, int32_t head_dim, int64_t stride_slot,
                  int64_t stride_head, float softmax_scale, int32_t dtype, int32_t plan_mode) {
  if (n_q < 0 || n_streams < 0 || n_q_heads < 1 || n_kv_heads < 1 || max_blocks < 0) return CS_EINVAL;
  if (stride_slot < 0 || stride_head < 0) return CS_EINVAL;
  if (n_q_heads % n_kv_heads) return CS_EINVAL;
  if (!(softmax_scale > 0.f) || !isfinite(softmax_scale)) return CS_EINVAL;   // also rejects NaN
  if (dtype != CS_F32 && dtype != CS_BF16) return CS_EUNSUPPORTED;
  if (head_dim != 64 && head_dim != 128) return CS_EUNSUPPORTED;
  if (block_size != CS_KV_BLOCK) return CS_EUNSUPPORTED;
  if (n_q_heads / n_kv_heads > 16) return CS_EUNSUPPORTED;
  const int elems = dtype == CS_BF16 ? 8 : 4;
  if (stride_slot % elems || stride_head % elems) return CS_EUNSUPPORTED;
  if (n_q == 0 || n_streams == 0) return kAttnNothingToDo;
  const bool plan_only = plan_mode == CS_ATTN_PLAN_ONLY && dtype == CS_BF16 && head_dim == 128;
  if (!cu_q || !q_pos || !kv_len || !block_table) return CS_EINVAL;
  if (!plan_only && (!q || !k_cache_layer || !v_cache_layer || !out)) return CS_EINVAL;
  if (!cs::aligned16(q) || !cs::aligned16(out) || !cs::aligned16(k_cache_layer) ||
      !cs::aligned16(v_cache_layer))
    return CS_EUNSUPPORTED;
  if (n_q * n_q_heads >= (1ll << 31)) return CS_EUNSUPPORTED;
  if (dtype == CS_BF16 && head_dim == 64 && max_blocks > kMaxBlocks64) return CS_EUNSUPPORTED;
  return CS_OK;
}

int attn_call(const void* q, const void* k_cache_layer, const void* v_cache_layer,
              const int32_t* cu_q, const int32_t* q_pos, const int32_t* kv_len,
              const int32_t* block_table, int32_t max_blocks, int32_t block_size,
              void* out, int64_t n_q, int32_t n_streams, int32_t n_q_heads,
              int32_t n_kv_heads, int32_t head_dim, int64_t stride_slot,
              int64_t stride_head, float softmax_scale, int32_t dtype,
              void* workspace, size_t workspace_bytes, int32_t plan_mode,
              const void* k_new, const void* v_new, const int32_t* new_slot, int64_t n_new, bool own,
              void* stream) {
  const int checked = attn_validate(q, k_cache_layer, v_cache_layer, cu_q, q_pos, kv_len, block_table, max_blocks,
                                    block_size, out, n_q, n_streams, n_q_heads, n_kv_heads, head_dim, stride_slot,
                                    stride_head, softmax_scale, dtype, plan_mode);
  if (checked == kAttnNothingToDo) return CS_OK;
  if (checked != CS_OK) return checked;
  const int group = n_q_heads / n_kv_heads;

  AttnParams p;
  p.q = q;
  p.k = k_cache_layer;
  p.v = v_cache_layer;
  p.out = out;
  p.cu_q = cu_q;
  p.q_pos = q_pos;
  p.block_table = block_table;
  p.kv_len = kv_len;
  p.stride_slot = stride_slot;
  p.stride_head = stride_head;
  p.max_blocks = max_blocks;
  p.n_streams = n_streams;
  p.n_q_heads = n_q_heads;
  p.n_kv_heads = n_kv_heads;
  p.group = group;
  p.scale = softmax_scale;
  p.scale_log2e = softmax_scale * 1.4426950408889634f;
  p.n_q = n_q;
  const bool fuse = k_new != nullptr;
  p.k_new = k_new;
  p.v_new = v_new;
  p.new_slot = new_slot;
  p.n_new = n_new;
  p.head_vecs = head_dim / 8;
  p.row_vecs = n_kv_heads * p.head_vecs;
  p.ws_own = nullptr;
  p.ws_tiles = nullptr;
  p.ws_warm = nullptr;
  p.n_warm = 0;
  p.ws_sync = nullptr;
  p.ws_status = nullptr;
  p.clear_status = 0;
  hipStream_t st = cs::as_stream(stream);
  // before a call with own rows
  const int own_bm = own ? own_row_tile(n_q, n_streams, group, n_kv_heads, head_dim, max_blocks) : 0;
  auto own_rows = [&](size_t attn_bytes) -> int {
    char* table = static_cast<char*>(workspace) + own_offset(attn_bytes);
    char* tiles = table + own_table_bytes(n_streams, max_blocks);
    p.ws_own = reinterpret_cast<cs::u32x2*>(table);
    p.ws_tiles = reinterpret_cast<int32_t*>(tiles);
    p.ws_warm = reinterpret_cast<cs::u32x2*>(tiles + own_tiles_bytes(n_q, n_streams, group, n_kv_heads));
    if (plan_mode == CS_ATTN_PLAN_REUSE) return CS_OK;
    if (plan_mode == CS_ATTN_PLAN_ONLY && head_dim == 128) p.n_new = 0;
    const int e = launch_own_rows(p, own_bm, st);
    p.ws_own = nullptr;                  // (its own attention reads the cache)
    return e;
  };
  if (dtype == CS_BF16) {
    if (head_dim == 128) {
      if (n_kv_heads > 256 || n_streams >= (1 << 23)) return CS_EUNSUPPORTED;
      if (plan_mode != CS_ATTN_PLAN_BUILD && plan_mode != CS_ATTN_PLAN_REUSE && plan_mode != CS_ATTN_PLAN_ONLY)
        return CS_EINVAL;
      const AttnPlan a = plan_attn(n_q, n_streams, group, n_kv_heads, max_blocks);
      // (a call that plans attends, and plans, as without own rows: any REUSE call may follow it)
      const bool reads_own = own_bm && plan_mode == CS_ATTN_PLAN_REUSE;
      const TileChoice choice = tile_route_128(n_q, n_streams, group, n_kv_heads, a.rt_cap, a.max_tiles, reads_own);
      const TileRoute route = choice.route;
      if (a.items_cap * a.bm >= (1ll << 31)) return CS_EUNSUPPORTED;
      if (stride_slot >= (1ll << 26) || a.max_tiles >= (1 << 15)) return CS_EUNSUPPORTED;      // 32-bit byte offsets inside a cache block
      if (!workspace || workspace_bytes < a.total || !cs::aligned16(workspace)) return CS_EWORKSPACE;
      char* w = static_cast<char*>(workspace);
      p.bm = a.bm;
      p.ws_plan = reinterpret_cast<const int32_t*>(w);
      p.ws_sync = reinterpret_cast<int32_t*>(w) + kHdrSyncBase;
      p.ws_status = reinterpret_cast<int32_t*>(w) + kHdrStatus;
      p.ws_items = reinterpret_cast<const int32_t*>(w + a.off_items);
      p.ws_desc = reinterpret_cast<int32_t*>(w + a.off_rt_desc);
      p.ws_ml = reinterpret_cast<float*>(w + a.off_ml);
      p.ws_o = reinterpret_cast<float*>(w + a.off_o);
      // Without a plan the refresh write is a launch of its own, and so it is for whole sweeps of few row tiles: the launch-wide
      // barrier takes 4-9 us more than that launch (10 streams of 420 tokens, 610 keys, us a layer of a graph 47.9 / 42.0).
      const bool few = a.rt_cap < 1024;
      const bool one_launch = fuse && !own && route == TileRoute::kNone && (a.span || !few) && !a.solo;
      if (own_bm) {
        const int e = own_rows(a.total);
        if (e != CS_OK) return e;
      } else if (fuse && !one_launch && plan_mode != CS_ATTN_PLAN_ONLY) {
        const int e = cs_kv_refresh_scatter(k_new, v_new, new_slot, const_cast<void*>(k_cache_layer),
                                            const_cast<void*>(v_cache_layer), n_new, n_kv_heads, head_dim, stride_slot,
                                            stride_head, dtype, stream);
        if (e != CS_OK) return e;
      }
      if (route != TileRoute::kNone && plan_mode != CS_ATTN_PLAN_ONLY) {
        // (the plan is neither needed nor made; the status word of a BUILD call still starts at zero)
        p.clear_status = plan_mode == CS_ATTN_PLAN_BUILD ? 1 : 0;
        if (route == TileRoute::kRows128) return launch_tiles<128, 4, 1, 2>(p, st);
        if (route == TileRoute::kRows64Keys2) return launch_tiles<128, 2, 2, 1>(p, st);
        if (route == TileRoute::kSplit64Keys4) {
          // (row tiles and pieces of them: at most twice those of alike streams, so 256 and 512; the workspace has place for
          // the items of a plan, 512 and more, and for the partial results of as many 128-row tiles)
          p.bm = 64;
          p.pieces = choice.pieces;
          p.ws_desc = reinterpret_cast<int32_t*>(w + a.off_items);      // (no plan: its items' place is free)
          return launch_split_tiles(p, st);
        }
        return launch_tiles<128, 2, 4, 1>(p, st);
      }
      PlanParams pp;
      pp.cu_q = cu_q;
      pp.q_pos = q_pos;
      pp.kv_len = kv_len;
      pp.max_blocks = max_blocks;
      pp.n_streams = n_streams;
      pp.group = group;
      pp.n_kv_heads = n_kv_heads;
      pp.max_tiles = a.max_tiles;
      pp.r_cap = static_cast<int32_t>(a.r_cap);
      pp.bm = a.bm;
      pp.n_slots = a.grid / 8;
      pp.solo = a.solo;
      pp.hist_pitch = a.hist_pitch;
      pp.header = reinterpret_cast<int32_t*>(w);
      pp.items = reinterpret_cast<int32_t*>(w + a.off_items);
      pp.rt_desc = reinterpret_cast<int32_t*>(w + a.off_rt_desc);
      pp.st_toff = reinterpret_cast<int32_t*>(w + a.off_st_toff);
      pp.st_work = reinterpret_cast<int32_t*>(w + a.off_st_work);
      pp.st_rank = reinterpret_cast<int32_t*>(w + a.off_st_rank);
      pp.rt_stream = reinterpret_cast<int32_t*>(w + a.off_rt_stream);
      pp.rt_wgmax = reinterpret_cast<int32_t*>(w + a.off_rt_wgmax);
      pp.un_head = reinterpret_cast<int32_t*>(w + a.off_un_head);
      pp.st_uoff = reinterpret_cast<int32_t*>(w + a.off_st_uoff);
      pp.hist = reinterpret_cast<int32_t*>(w + a.off_hist);
      pp.span = a.span;
      pp.pref_pitch = a.pref_pitch;
      pp.sw_pref = reinterpret_cast<int32_t*>(w + a.off_pref);
      if (plan_mode == CS_ATTN_PLAN_BUILD && few && !a.span) {
        const int64_t tiles = ((n_q * group) / kBM + n_streams) * n_kv_heads;
        hipLaunchKernelGGL((window_attn_bf16_tile_and_plan_kernel<4, 1, 2>), dim3(static_cast<unsigned>(tiles) + 1), dim3(256), 0, st, p, pp);
        return cs::note_hip(hipGetLastError());
      }
      if (plan_mode != CS_ATTN_PLAN_REUSE) {
        hipLaunchKernelGGL(window_attn_plan_kernel, dim3(1), dim3(kPlanThreads), 0, st, pp);
        const int e = cs::note_hip(hipGetLastError());
        if (e != CS_OK) return e;
        if (plan_mode == CS_ATTN_PLAN_ONLY) return CS_OK;
      }
      if (a.solo)
        hipLaunchKernelGGL(window_attn_bf16_rows32_kernel, dim3(static_cast<unsigned>(a.grid)), dim3(256), 0, st, p);
      else if (one_launch)
        hipLaunchKernelGGL((window_attn_bf16_stream_kernel<true>), dim3(static_cast<unsigned>(a.grid)), dim3(256), 0, st, p);
      else
        hipLaunchKernelGGL((window_attn_bf16_stream_kernel<false>), dim3(static_cast<unsigned>(a.grid)), dim3(256), 0, st, p);
      if (a.span) {
        const int e = cs::note_hip(hipGetLastError());
        if (e != CS_OK) return e;
        hipLaunchKernelGGL(window_attn_merge_kernel, dim3(static_cast<unsigned>(a.rt_cap * (a.bm / 8))),
                           dim3(256), 0, st, p);
      }
    } else {
      // Two key groups while the launch is so small that its longest sweep is what it takes (all of its row tiles
      // are resident together, 1,024 of them with one group).  One group / two, us a step of 16 layers (own rows): bound of 364 row tiles
      // 426 / 336, 752 509 / 453, 992 571 / 578 (of 1,000 with 55 key tiles 1,519 / 1,434), 1,200 640 / 662, 1,408 750 / 776, 3,552 1,638 /
      // 1,793.  One group with two stages, not one: the same order 1,200 730 / 640, 1,408 781 / 750, 1,856 1,005 / 953, 3,552 1,669 /
      // 1,638 (one stage / two; without own rows 740 / 720, 831 / 831, 1,064 / 1,067, 1,787 / 1,744).
      const int64_t tiles = ((n_q * group) / kBM + n_streams) * n_kv_heads;
      if (own_bm) {
        const int e = own_rows(0);
        if (e != CS_OK) return e;
        p.ws_status = static_cast<int32_t*>(workspace) + kHdrStatus;
        p.clear_status = plan_mode == CS_ATTN_PLAN_REUSE ? 0 : 1;
      }
      if (tiles <= 1024) return launch_tiles<64, 4, 2, 2>(p, st);
      return launch_tiles<64, 4, 1, 2>(p, st);
    }
  } else {
    const int64_t tiles = ((n_q * group) / kF32Rows + n_streams) * n_kv_heads;       // upper bound on row tiles
    if (tiles > 0x7fffffffll) return CS_EUNSUPPORTED;
    const dim3 grid(static_cast<unsigned>(tiles)), block(64 * kF32Waves);
    if (head_dim == 128)
      hipLaunchKernelGGL(window_attn_f32_kernel<128>, grid, block, 0, st, p);
    else
      hipLaunchKernelGGL(window_attn_f32_kernel<64>, grid, block, 0, st, p);
  }
  return cs::note_hip(hipGetLastError());
}

}  // namespace

extern "C" int cs_window_prefill_attn(const void* q, const void* k_cache_layer, const void* v_cache_layer,
                                      const int32_t* cu_q, const int32_t* q_pos, const int32_t* kv_len,
                                      const int32_t* block_table, int32_t max_blocks, int32_t block_size,
                                      void* out, int64_t n_q, int32_t n_streams, int32_t n_q_heads,
                                      int32_t n_kv_heads, int32_t head_dim, int64_t stride_slot,
                                      int64_t stride_head, float softmax_scale, int32_t dtype,
                                      void* workspace, size_t workspace_bytes, int32_t plan_mode,
                                      void* stream) {
  return attn_call(q, k_cache_layer, v_cache_layer, cu_q, q_pos, kv_len, block_table, max_blocks, block_size, out,
                   n_q, n_streams, n_q_heads, n_kv_heads, head_dim, stride_slot, stride_head, softmax_scale, dtype,
                   workspace, workspace_bytes, plan_mode, nullptr, nullptr, nullptr, 0, false, stream);
}

extern "C" size_t cs_refresh_prefill_attn_workspace(int64_t n_q, int32_t n_streams, int32_t n_q_heads,
                                                    int32_t n_kv_heads, int32_t head_dim, int32_t max_blocks,
                                                    int32_t dtype) {
  const size_t attn = cs_window_prefill_attn_workspace(n_q, n_streams, n_q_heads, n_kv_heads, head_dim, max_blocks, dtype);
  if (dtype != CS_BF16 || (head_dim != 64 && head_dim != 128) || n_q <= 0 || n_streams <= 0 || max_blocks <= 0 || n_kv_heads < 1 ||
      n_q_heads < n_kv_heads || n_q_heads % n_kv_heads || n_q * n_q_heads >= (1ll << 31))
    return attn;
  if (!own_row_tile(n_q, n_streams, n_q_heads / n_kv_heads, n_kv_heads, head_dim, max_blocks)) return attn;
  return own_offset(attn) + own_bytes(n_q, n_streams, n_q_heads / n_kv_heads, n_kv_heads, max_blocks);
}

extern "C" int cs_refresh_prefill_attn(const void* k_new, const void* v_new, const int32_t* slot, int64_t n_tok,
                                       const void* q, void* k_cache_layer, void* v_cache_layer,
                                       const int32_t* cu_q, const int32_t* q_pos, const int32_t* kv_len,
                                       const int32_t* block_table, int32_t max_blocks, int32_t block_size,
                                       void* out, int64_t n_q, int32_t n_streams, int32_t n_q_heads,
                                       int32_t n_kv_heads, int32_t head_dim, int64_t stride_slot,
                                       int64_t stride_head, float softmax_scale, int32_t dtype,
                                       void* workspace, size_t workspace_bytes, int32_t plan_mode,
                                       void* stream) {
  if (n_tok < 0) return CS_EINVAL;
  // The rows are the queries' own: what finds them is made by the call that plans and read by those that follow it.  Where the
  // cache is laid out as the rows are, so that the same offsets serve both; otherwise the call is as without the flag.
  const int32_t mode = plan_mode & ~CS_ATTN_OWN_ROWS;
  bool own = mode != plan_mode && (mode == CS_ATTN_PLAN_BUILD || mode == CS_ATTN_PLAN_REUSE || mode == CS_ATTN_PLAN_ONLY);
  if (own) plan_mode = mode;
  own = own && dtype == CS_BF16 && n_tok == n_q && n_tok > 0 && n_streams > 0 && max_blocks > 0 && stride_head == head_dim &&
        stride_slot == static_cast<int64_t>(n_kv_heads) * head_dim && n_tok * stride_slot < (1ll << 34) &&
        max_blocks <= (1 << kOwnRowBits) / CS_KV_BLOCK;
  if (own) {
    const int checked = attn_validate(q, k_cache_layer, v_cache_layer, cu_q, q_pos, kv_len, block_table, max_blocks,
                                      block_size, out, n_q, n_streams, n_q_heads, n_kv_heads, head_dim, stride_slot,
                                      stride_head, softmax_scale, dtype, plan_mode);
    if (checked < 0) return checked;
    own = head_dim == 128 || own_row_tile(n_q, n_streams, n_q_heads / n_kv_heads, n_kv_heads, head_dim, max_blocks);
  }
  if (own) {
    if (!workspace || !cs::aligned16(workspace) ||
        workspace_bytes < cs_refresh_prefill_attn_workspace(n_q, n_streams, n_q_heads, n_kv_heads, head_dim, max_blocks, dtype))
      return CS_EWORKSPACE;
    const bool only = plan_mode == CS_ATTN_PLAN_ONLY && head_dim == 128;
    if (!only && (!k_new || !v_new || !slot)) return CS_EINVAL;
    if (!cs::aligned16(k_new) || !cs::aligned16(v_new)) return CS_EUNSUPPORTED;
    return attn_call(q, k_cache_layer, v_cache_layer, cu_q, q_pos, kv_len, block_table, max_blocks, block_size, out, n_q,
                     n_streams, n_q_heads, n_kv_heads, head_dim, stride_slot, stride_head, softmax_scale, dtype, workspace,
                     workspace_bytes, plan_mode, k_new, v_new, slot, n_tok, true, stream);
  }
  const bool one_launch = dtype == CS_BF16 && head_dim == 128;
  const bool plan_only = plan_mode == CS_ATTN_PLAN_ONLY && one_launch;
  if (n_tok > 0 && !plan_only && (!k_new || !v_new || !slot)) return CS_EINVAL;
  if (!cs::aligned16(k_new) || !cs::aligned16(v_new)) return CS_EUNSUPPORTED;
  if (!one_launch || n_tok == 0 || n_q == 0 || n_streams == 0) {
    // shapes without a persistent kernel (fp32 caches, head_dim 64), or nothing to attend: the
    // refresh write as a launch of its own, then the attention call (whose arguments are checked
    // first, so that a call that fails has moved nothing)
    const int checked = attn_validate(q, k_cache_layer, v_cache_layer, cu_q, q_pos, kv_len, block_table, max_blocks,
                                      block_size, out, n_q, n_streams, n_q_heads, n_kv_heads, head_dim, stride_slot,
                                      stride_head, softmax_scale, dtype, plan_mode);
    if (checked < 0) return checked;
    if (n_tok > 0) {
      const int e = cs_kv_refresh_scatter(k_new, v_new, slot, k_cache_layer, v_cache_layer, n_tok, n_kv_heads,
                                          head_dim, stride_slot, stride_head, dtype, stream);
      if (e != CS_OK) return e;
    }
    return attn_call(q, k_cache_layer, v_cache_layer, cu_q, q_pos, kv_len, block_table, max_blocks, block_size, out,
                     n_q, n_streams, n_q_heads, n_kv_heads, head_dim, stride_slot, stride_head, softmax_scale, dtype,
                     workspace, workspace_bytes, plan_mode, nullptr, nullptr, nullptr, 0, false, stream);
  }
  return attn_call(q, k_cache_layer, v_cache_layer, cu_q, q_pos, kv_len, block_table, max_blocks, block_size, out,
                   n_q, n_streams, n_q_heads, n_kv_heads, head_dim, stride_slot, stride_head, softmax_scale, dtype,
                   workspace, workspace_bytes, plan_mode, k_new, v_new, slot, n_tok, false, stream);
}
