// Residual proxy.  Paper Sec. 4 (Codec Processing): the decoder hands out no residuals, so they
// are approximated from pixels: the previous decoded frame is shifted by the motion vectors,
// compared with the current frame, and a patch is scored by the average absolute pixel difference
// inside it (the per-patch counterpart of the block residual of Eq. 2; input of the rescue rule, Eq. 4).
//
// One launch where a patch is small enough (at most 128 source rows and 512 columns): a workgroup owns a run of
// whole patches of one patch row, as many as its lanes take in one turn, sums them in LDS and writes their scores.
// Larger patches keep three launches, the output array doubling as the accumulator: clear the sums, a workgroup per
// run of source rows with one global atomic per workgroup and patch, then sum -> score.  In both a thread owns a
// 4-pixel group of columns (consecutive lanes, consecutive groups: every load of a wave is one contiguous span) and
// walks down the rows a cell row of the motion field at a time: one vector, then for four pixel rows at once the
// current pixels (one dword) and the reference pixels (one 8-byte load and a byte permute that also clamps columns
// outside the frame), eight independent loads in flight.  |a - b| over four pixels is one v_sad_u8; a group that
// straddles a patch border is split by byte masks fixed per thread, so the row loop has no patch arithmetic at all.
// HBM bound.  Runs of patches that share lines of the planes go to one XCD, so that its L2 serves the second, and in
// large batches a run is a whole patch row (512 lanes), read front to back.  us for 1920 x 1080, 16 x 16 patches, with
// short runs dealt round the XCDs / as three launches / now: cell 4, 32 frames, 149 MB 42.2 / 47.0 / 41.7; 96 frames,
// 448 MB 110 / 105 / 98.6 (4.5 TB/s); 200 frames 223 / 186 / 184 (5.1 TB/s); cell 16, 96 frames 140 / 125 / 91.4.
// Integer adds commute, so the result is bit exact whatever the order.
#include "common.h"

namespace {

constexpr int kNumeratorBits = 29;

struct ExactDiv {                // q = (n * mul) >> shift == n / d for every n < 2^kNumeratorBits
  uint32_t mul;
  uint32_t shift;
};

ExactDiv exact_div(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  const uint64_t two = 1ull << (kNumeratorBits + l);
  ExactDiv e;
  e.mul = static_cast<uint32_t>((two + d - 1) / d);
  e.shift = kNumeratorBits + l;
  return e;
}

__device__ __forceinline__ uint32_t div_by(uint32_t n, ExactDiv e) {
  return static_cast<uint32_t>((static_cast<uint64_t>(n) * e.mul) >> e.shift);
}

struct ResidualParams {
  const uint8_t* __restrict__ cur;
  const uint8_t* __restrict__ prev;
  const uint32_t* __restrict__ field;     // [F][cells_h][cells_w] packed (dx, dy), quarter pixels
  uint32_t* __restrict__ res;             // [F][P]: sums, then scores
  int64_t pitch, frame_stride;
  int32_t n_frames, src_w, src_h, cell_shift, cells_w, cells_h;
  uint32_t in_w, in_h, den_x, den_y;      // den = patch * src size
  ExactDiv div_x;
  int32_t grid_h, grid_w, n_sub, n_parts;
};

typedef cs::u32x2 __attribute__((aligned(4))) dword_pair;

// first source coordinate of patch index i along an axis: ceil(i * den / n_in), capped at n_src
__device__ __forceinline__ int first_coord(int i, uint32_t den, uint32_t n_in, int n_src) {
  const unsigned long long v = (static_cast<unsigned long long>(i) * den + n_in - 1) / n_in;
  return v < static_cast<unsigned long long>(n_src) ? static_cast<int>(v) : n_src;
}

__global__ __launch_bounds__(256) void clear_sums_kernel(uint32_t* p, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// 256 times the sum of a patch over its number of source pixels.
__device__ __forceinline__ uint32_t patch_mean(const ResidualParams& p, int r, int c, uint32_t sum) {
  const int64_t wide = first_coord(c + 1, p.den_x, p.in_w, p.src_w) - first_coord(c, p.den_x, p.in_w, p.src_w);
  const int64_t tall = first_coord(r + 1, p.den_y, p.in_h, p.src_h) - first_coord(r, p.den_y, p.in_h, p.src_h);
  const unsigned long long n = static_cast<unsigned long long>(wide * tall);
  return n ? static_cast<uint32_t>((256ull * sum) / n) : 0u;
}

// kWhole: a workgroup of T threads owns a run of whole patches of one patch row (n_sub runs per row) and writes their
// means: one launch.  Its waves are n_parts parts of the row's source rows times T / 64 / n_parts shares of the columns.
// Otherwise a workgroup owns the source rows of one n_sub-th of a patch row and adds to sums that a launch before
// this one clears and a launch after it divides.
template <bool kWhole, int T>
__global__ __launch_bounds__(T) void residual_sum_kernel(ResidualParams p) {
  extern __shared__ uint32_t s_sum[];                       // [patches of the workgroup]
  const int tid = threadIdx.x;
  // workgroups go to the XCDs round robin: an XCD's workgroups take consecutive runs
  const int xcd = blockIdx.x & 7;
  const int run = kWhole ? (blockIdx.x >> 3) + xcd * (gridDim.x >> 3) + min(xcd, static_cast<int>(gridDim.x & 7)) : blockIdx.x;
  const int sub = run % p.n_sub;
  const int band = (run / p.n_sub) % p.grid_h;
  const int frame = run / (p.n_sub * p.grid_h);
  const int col_lo = kWhole ? static_cast<int>(static_cast<int64_t>(p.grid_w) * sub / p.n_sub) : 0;
  const int col_hi = kWhole ? static_cast<int>(static_cast<int64_t>(p.grid_w) * (sub + 1) / p.n_sub) : p.grid_w;
  const int n_parts = kWhole ? p.n_parts : p.n_sub;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = kWhole ? wave % n_parts : sub;
  const int y_lo = first_coord(band, p.den_y, p.in_h, p.src_h);
  const int y_hi = first_coord(band + 1, p.den_y, p.in_h, p.src_h);
  // the band's rows in quads (rows 4q .. 4q+3, the unit of the row loop), dealt to its parts
  const int q_lo = y_lo >> 2, n_quads = ((y_hi - 1) >> 2) + 1 - q_lo;
  const int q_begin = q_lo + static_cast<int>(static_cast<int64_t>(n_quads) * part / n_parts);
  const int q_end = q_lo + static_cast<int>(static_cast<int64_t>(n_quads) * (part + 1) / n_parts);
  const int y_begin = max(y_lo, 4 * q_begin), y_end = min(y_hi, 4 * q_end);
  if (!kWhole && (y_lo >= y_hi || y_begin >= y_end)) return;          // uniform for the workgroup

  for (int i = tid; i < col_hi - col_lo; i += T) s_sum[i] = 0u;
  __syncthreads();

  const int W = p.src_w, H = p.src_h;
  const int all_groups = (W + 3) / 4;                                // 4-pixel groups along a row
  const int k_lo = kWhole ? first_coord(col_lo, p.den_x, p.in_w, W) >> 2 : 0;
  const int groups = kWhole ? min(all_groups, (first_coord(col_hi, p.den_x, p.in_w, W) + 3) >> 2) : all_groups;
  const int k_step = kWhole ? T / n_parts : T;
  const int k_first = kWhole ? k_lo + 64 * (wave / n_parts) + (tid & 63) : tid;
  const uint8_t* cur = p.cur + static_cast<int64_t>(frame) * p.frame_stride;
  const uint8_t* prev = p.prev + static_cast<int64_t>(frame) * p.frame_stride;
  const uint32_t* field = p.field + static_cast<int64_t>(frame) * p.cells_h * p.cells_w;
  const int cell = 1 << p.cell_shift;

  for (int k = k_first; k < groups && y_begin < y_end; k += k_step) {
    // ---- the group's patch column(s) and the byte masks that split it between them
    const int x = 4 * k;
    int col_a = static_cast<int>(div_by(static_cast<uint32_t>(x) * p.in_w, p.div_x)), col_b = 0;
    uint32_t mask_a = 0u, mask_b = 0u;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (x + t < W) {
        const int c = static_cast<int>(div_by(static_cast<uint32_t>(x + t) * p.in_w, p.div_x));
        if (c == col_a) mask_a |= 0xffu << (8 * t);
        else { mask_b |= 0xffu << (8 * t); col_b = c; }     // columns are at least 4 pixels wide: one other column at most
      }
    }
    if (col_a < col_lo || col_a >= col_hi) mask_a = 0u;
    if (col_b < col_lo || col_b >= col_hi) mask_b = 0u;
    uint32_t acc_a = 0u, acc_b = 0u;
    // ---- down the rows, one cell row of the motion field at a time, four pixel rows per batch
    const int yc_last = (y_end - 1) >> p.cell_shift;
    const uint32_t* fcol = field + (x >> p.cell_shift);
    uint32_t mv_next = fcol[static_cast<int64_t>(y_begin >> p.cell_shift) * p.cells_w];
    for (int yc = y_begin >> p.cell_shift; yc <= yc_last; ++yc) {
      const uint32_t mv = mv_next;
      mv_next = fcol[static_cast<int64_t>(min(yc + 1, yc_last)) * p.cells_w];     // one cell row ahead
      const int ox = (static_cast<int>(static_cast<int16_t>(mv & 0xffffu)) + 2) >> 2;
      const int oy = (static_cast<int>(static_cast<int16_t>(mv >> 16)) + 2) >> 2;
      const int xs = x + ox;
      // the reference group's four bytes, columns clamped to the frame, lie in one 8-byte load inside the row's pitch
      // and are picked out of it by one byte permute
      const int a0 = min(max(min(xs, W - 1) & ~3, 0), static_cast<int>(p.pitch) - 8);
      uint32_t pick = 0x03020100u + 0x01010101u * static_cast<uint32_t>(xs - a0);
      if (xs < 0 || xs + 3 > W - 1) {
        pick = 0u;
#pragma unroll
        for (int t = 0; t < 4; ++t) pick |= static_cast<uint32_t>(min(max(xs + t, 0), W - 1) - a0) << (8 * t);
      }
      const int y_cell = yc << p.cell_shift;                 // (a part may begin and end inside a cell row)
      for (int r4 = max((y_begin & ~3) - y_cell, 0); r4 < min(y_end - y_cell, cell); r4 += 4) {
        uint32_t c4[4];
        dword_pair ref[4];
        bool live[4];
#pragma unroll
        for (int dy = 0; dy < 4; ++dy) {
          const int y = y_cell + r4 + dy;
          live[dy] = y >= y_begin && y < y_end;
          const int yv = min(max(y, y_begin), y_end - 1);    // a row of this workgroup in any case
          const int yy = min(max(yv + oy, 0), H - 1);
          const uint8_t* prow = prev + static_cast<int64_t>(yy) * p.pitch;
          c4[dy] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(cur + static_cast<int64_t>(yv) * p.pitch + x));
          ref[dy] = *reinterpret_cast<const dword_pair*>(prow + a0);
        }
#pragma unroll
        for (int dy = 0; dy < 4; ++dy) {
          const uint32_t pred = __builtin_amdgcn_perm(ref[dy].y, ref[dy].x, pick);
          const uint32_t ma = live[dy] ? mask_a : 0u, mb = live[dy] ? mask_b : 0u;
          acc_a = __builtin_amdgcn_sad_u8(c4[dy] & ma, pred & ma, acc_a);
          acc_b = __builtin_amdgcn_sad_u8(c4[dy] & mb, pred & mb, acc_b);
        }
      }
    }
    if (acc_a) atomicAdd(&s_sum[col_a - col_lo], acc_a);
    if (acc_b) atomicAdd(&s_sum[col_b - col_lo], acc_b);
  }
  __syncthreads();
  uint32_t* out = p.res + (static_cast<int64_t>(frame) * p.grid_h + band) * p.grid_w;
  for (int i = tid; i < col_hi - col_lo; i += T) {
    if constexpr (kWhole) out[col_lo + i] = patch_mean(p, band, col_lo + i, s_sum[i]);
    else if (s_sum[i]) atomicAdd(out + i, s_sum[i]);
  }
}

__global__ __launch_bounds__(256) void residual_mean_kernel(ResidualParams p) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int n_patch = p.grid_h * p.grid_w;
  if (i >= static_cast<int64_t>(p.n_frames) * n_patch) return;
  const int cell = static_cast<int>(i % n_patch);
  const int r = cell / p.grid_w, c = cell - r * p.grid_w;
  p.res[i] = patch_mean(p, r, c, p.res[i]);
}

}  // namespace

extern "C" int cs_residual_proxy(const uint8_t* cur, const uint8_t* prev, const int16_t* mv_field,
                                 int32_t n_frames, int32_t src_w, int32_t src_h, int64_t pitch,
                                 int64_t frame_stride, int32_t cell, int32_t in_w, int32_t in_h,
                                 int32_t patch, int32_t grid_h, int32_t grid_w, uint32_t* res,
                                 void* stream) {
  if (n_frames < 0 || src_w < 1 || src_h < 1 || in_w < 1 || in_h < 1 || patch < 1 || grid_h < 1 || grid_w < 1)
    return CS_EINVAL;
  if (pitch < src_w || frame_stride < pitch * src_h) return CS_EINVAL;
  if (n_frames == 0) return CS_OK;
  if (!cur || !prev || !mv_field || !res) return CS_EINVAL;
  if (cell != 4 && cell != 8 && cell != 16) return CS_EUNSUPPORTED;
  if (src_w > 16384 || src_h > 16384 || in_w > 16384 || in_h > 16384 || patch > 1024) return CS_EUNSUPPORTED;
  if (grid_w > 8192 || static_cast<int64_t>(n_frames) * grid_h * grid_w >= (1ll << 31)) return CS_EUNSUPPORTED;
  if (pitch % 16 || frame_stride % 16 || pitch < ((src_w + 15) / 16) * 16) return CS_EUNSUPPORTED;
  if (!cs::aligned16(cur) || !cs::aligned16(prev) || (reinterpret_cast<uintptr_t>(mv_field) & 3u) ||
      (reinterpret_cast<uintptr_t>(res) & 3u))
    return CS_EUNSUPPORTED;
  // a 4-pixel group may touch two patch columns at most: columns at least 4 source pixels wide
  if (static_cast<int64_t>(patch) * src_w < 4ll * in_w) return CS_EUNSUPPORTED;

  ResidualParams p;
  p.cur = cur;
  p.prev = prev;
  p.field = reinterpret_cast<const uint32_t*>(mv_field);
  p.res = res;
  p.pitch = pitch;
  p.frame_stride = frame_stride;
  p.n_frames = n_frames;
  p.src_w = src_w;
  p.src_h = src_h;
  p.cell_shift = cell == 4 ? 2 : cell == 8 ? 3 : 4;
  p.cells_w = (src_w + cell - 1) / cell;
  p.cells_h = (src_h + cell - 1) / cell;
  p.in_w = in_w;
  p.in_h = in_h;
  p.den_x = static_cast<uint32_t>(patch) * src_w;
  p.den_y = static_cast<uint32_t>(patch) * src_h;
  p.div_x = exact_div(p.den_x);
  p.grid_h = grid_h;
  p.grid_w = grid_w;
  const int64_t bands = static_cast<int64_t>(n_frames) * grid_h;
  const int64_t band_rows = (static_cast<int64_t>(p.den_y) + in_h - 1) / in_h + 1;
  hipStream_t st = cs::as_stream(stream);
  const int64_t col_groups = (static_cast<int64_t>(p.den_x) + 4ll * in_w - 1) / (4ll * in_w);    // of one patch
  if (band_rows <= 128 && col_groups <= 128) {
    // patches small enough for a workgroup of their own.  A run is as many of them as the lanes of a part's waves take
    // in one turn.
    auto runs = [&](int64_t lanes) {
      const int64_t cols = col_groups >= lanes ? 1 : (lanes - 1) / col_groups;
      return (grid_w + cols - 1) / cols;
    };
    // Large batches: 512 lanes and one part, where a row keeps three quarters of them busy and there are three such
    // workgroups per CU.  us with 256 threads / 512, 1920 x 1080, cell 4, 16 x 16 patches: 16 frames (256 workgroups)
    // 24.0 / 25.7, 32 41.7 / 42.4, 64 73.7 / 68.7, 96 104.1 / 98.6; 1280 x 720 (320 lanes of 512) 52.1 / 55.0.
    const int64_t wide_sub = runs(512);
    const bool wide = bands * wide_sub >= 768 && (src_w + 3) / 4 >= 384 * wide_sub;
    if (wide) {
      p.n_parts = 1;
      p.n_sub = static_cast<int32_t>(wide_sub);
    } else {
      // at least four quads of rows per part: the set-up of a thread is paid once
      p.n_parts = band_rows >= 64 ? 4 : band_rows >= 32 ? 2 : 1;
      p.n_sub = static_cast<int32_t>(runs(256 / p.n_parts));
    }
    if (bands * p.n_sub >= (1ll << 31)) return CS_EUNSUPPORTED;
    const dim3 grid(static_cast<unsigned>(bands * p.n_sub));
    const size_t lds = static_cast<size_t>((grid_w + p.n_sub - 1) / p.n_sub) * sizeof(uint32_t);
    if (wide) hipLaunchKernelGGL((residual_sum_kernel<true, 512>), grid, dim3(512), lds, st, p);
    else hipLaunchKernelGGL((residual_sum_kernel<true, 256>), grid, dim3(256), lds, st, p);
    return cs::note_hip(hipGetLastError());
  }
  // larger ones: enough workgroups to fill the chip, a patch row's source rows split among n_sub workgroups
  int64_t n_sub = (8192 + bands - 1) / bands;               // a few rounds of workgroups per CU
  if (n_sub > band_rows / 16) n_sub = band_rows / 16;        // at least four quads of rows each: the per-thread set-up is paid once per workgroup
  if (n_sub < 1) n_sub = 1;
  p.n_sub = static_cast<int32_t>(n_sub);
  if (bands * n_sub >= (1ll << 31)) return CS_EUNSUPPORTED;

  const int64_t n_out = static_cast<int64_t>(n_frames) * grid_h * grid_w;
  hipLaunchKernelGGL(clear_sums_kernel, dim3(static_cast<unsigned>((n_out + 255) / 256)), dim3(256), 0, st, res, n_out);
  hipLaunchKernelGGL((residual_sum_kernel<false, 256>), dim3(static_cast<unsigned>(bands * n_sub)), dim3(256),
                     static_cast<size_t>(grid_w) * sizeof(uint32_t), st, p);
  hipLaunchKernelGGL(residual_mean_kernel, dim3(static_cast<unsigned>((n_out + 255) / 256)), dim3(256), 0, st, p);
  return cs::note_hip(hipGetLastError());
}
