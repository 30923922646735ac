// Block-to-patch projection.  Paper Sec. 3.3.1 (paragraph on mapping codec changes to ViT
// patches): block rectangles are in source-frame pixels, patches in model-input pixels; the
// rectangles are rescaled and every patch gets the strongest motion (Eq. 1) among the blocks that
// land on it.  Sec. 3.3.2: a patch touched by an intra-coded block is flagged.
//
// A workgroup per band of patch rows of a frame (one band in large batches and for small frames).  The band's patch table
// lives in LDS as 64-bit keys
//     key = |v|^2 << 32 | (dx + 32768) << 16 | (dy + 32768)
// so that "largest magnitude, ties to the lexicographically largest vector" is an unsigned
// maximum and the winning vector comes back out of the key: blocks are streamed once (one 16-byte
// load each), each computes its patch range with exact integer arithmetic and raises the keys of
// the patches it overlaps (ds_max_u64; a plain read first skips the atomic when the patch already
// holds at least as much, which is the common case inside a moving region).  The order in which
// blocks arrive cannot change the result.  Divisions by the two launch constants
// patch * src_w and patch * src_h are multiplications by a precomputed reciprocal that is exact for
// the numerators that can occur (below 2^29).
//
// A record's patch range, key and raises are some 150 vector instructions, 13 us for a 1920 x 1080
// frame's 14 k blocks on one CU: with at most half as many frames as the chip has CUs the bands of a frame are
// separate workgroups.  Each reads all of the frame's records (from L2 after the first) but leaves a
// record after one comparison when it does not reach the band; blocks arrive in raster order, so
// whole wavefronts leave together.  32 frames of 1920 x 1080: 13.7 us with a workgroup per frame,
// 8.3 with eight.  With one band a record is read once and past the caches: 1,376 frames, 304 MB,
// 60.4 us (5.0 TB/s), 68.3 with the cached loads and the comparison that bands need.
#include "common.h"

namespace {

constexpr int kProjectThreads = 1024;
constexpr int kBatch = 4;
constexpr int kNumeratorBits = 29;

struct ExactDiv {                // q = (n * mul) >> shift == n / d for every n < 2^kNumeratorBits
  uint32_t mul;
  uint32_t shift;
};

ExactDiv exact_div(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;                                  // l = ceil(log2 d)
  const uint64_t two = 1ull << (kNumeratorBits + l);
  ExactDiv e;
  e.mul = static_cast<uint32_t>((two + d - 1) / d);             // < 2^(kNumeratorBits + 1)
  e.shift = kNumeratorBits + l;
  return e;
}

__device__ __forceinline__ uint32_t div_by(uint32_t n, ExactDiv e) {
  return static_cast<uint32_t>((static_cast<uint64_t>(n) * e.mul) >> e.shift);
}

struct ProjectParams {
  const cs::u32x4* __restrict__ blocks;
  const int32_t* __restrict__ cu_blocks;
  uint32_t* __restrict__ mv;         // [F][P] packed (dx, dy)
  uint8_t* __restrict__ intra;       // [F][P]
  uint32_t src_w, src_h, in_w, in_h;
  uint32_t den_x, den_y;             // patch * src_w, patch * src_h
  ExactDiv div_x, div_y;
  int32_t grid_h, grid_w, n_patch;
  int32_t n_frames, n_bands;
};

// kBands: a workgroup owns one band of a frame, not all of it.
template <bool kBands>
__global__ __launch_bounds__(kProjectThreads) void project_blocks_kernel(ProjectParams p) {
  extern __shared__ unsigned long long s_key[];                         // [patches of the band]
  const int tid = threadIdx.x;
  // (the bands of a frame lie n_frames workgroups apart: with a multiple of 8 frames they share an XCD's L2)
  const int frame = kBands ? blockIdx.x % p.n_frames : blockIdx.x, band = kBands ? blockIdx.x / p.n_frames : 0;
  const int row_lo = kBands ? band * p.grid_h / p.n_bands : 0;
  const int row_hi = kBands ? (band + 1) * p.grid_h / p.n_bands : p.grid_h;
  const int n_cells = (row_hi - row_lo) * p.grid_w;
  uint32_t* s_intra = reinterpret_cast<uint32_t*>(s_key + n_cells);    // bitmap, n_cells bits
  for (int i = tid; i < n_cells; i += kProjectThreads) s_key[i] = 0ull;
  for (int i = tid; i < (n_cells + 31) / 32; i += kProjectThreads) s_intra[i] = 0u;
  __syncthreads();
  // source rows the band's patches overlap: a block reaches the band if hi_y > band_y0 and lo_y < band_y1
  const uint64_t lo_num = static_cast<uint64_t>(row_lo) * p.den_y, hi_num = static_cast<uint64_t>(row_hi) * p.den_y;
  const uint32_t band_y0 = static_cast<uint32_t>(min(lo_num / p.in_h, static_cast<uint64_t>(0xffffffffu)));
  const uint32_t band_y1 = static_cast<uint32_t>(min((hi_num + p.in_h - 1u) / p.in_h, static_cast<uint64_t>(0xffffffffu)));
  const int begin = p.cu_blocks[frame], end = p.cu_blocks[frame + 1];
  auto apply = [&](const cs::u32x4 rec) {
    const uint32_t x = rec.x & 0xffffu, y = rec.x >> 16, w = rec.y & 0xffffu, h = rec.y >> 16;
    const int dx = static_cast<int16_t>(rec.z & 0xffffu), dy = static_cast<int16_t>(rec.z >> 16);
    const bool is_intra = (rec.w & 1u) != 0;
    const uint32_t mag = static_cast<uint32_t>(dx * dx) + static_cast<uint32_t>(dy * dy);   // up to 2^31
    if (!is_intra && mag == 0u) return;                       // a zero vector changes no patch
    if (kBands && (y + h <= band_y0 || y >= band_y1)) return;
    // footprint clipped to the frame; nothing left -> no footprint
    const uint32_t lo_x = min(x, p.src_w), hi_x = min(x + w, p.src_w);
    const uint32_t lo_y = min(y, p.src_h), hi_y = min(y + h, p.src_h);
    if (hi_x <= lo_x || hi_y <= lo_y) return;
    // patch columns c with lo*in < (c+1)*den and hi*in > c*den (positive overlap), same for rows
    const int c0 = static_cast<int>(div_by(lo_x * p.in_w, p.div_x));
    const int c1 = min(static_cast<int>(div_by(hi_x * p.in_w + p.den_x - 1u, p.div_x)) - 1, p.grid_w - 1);
    const int r0 = max(static_cast<int>(div_by(lo_y * p.in_h, p.div_y)), row_lo);
    const int r1 = min(static_cast<int>(div_by(hi_y * p.in_h + p.den_y - 1u, p.div_y)), row_hi) - 1;
    const unsigned long long key = (static_cast<unsigned long long>(mag) << 32) |
                                   (static_cast<uint32_t>(dx + 32768) << 16) | static_cast<uint32_t>(dy + 32768);
    for (int r = r0; r <= r1; ++r)
      for (int c = c0; c <= c1; ++c) {
        const int cell = (r - row_lo) * p.grid_w + c;
        if (is_intra) {
          const uint32_t bit = 1u << (cell & 31);
          if (!(s_intra[cell >> 5] & bit)) atomicOr(&s_intra[cell >> 5], bit);
        } else if (s_key[cell] < key) {
          atomicMax(&s_key[cell], key);
        }
      }
  };
  // kBatch records in flight per thread (a record past the end is replaced by an empty one)
  for (int i0 = begin + tid; i0 < end; i0 += kProjectThreads * kBatch) {
    cs::u32x4 rec[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + u * kProjectThreads;
      // (only the other bands of a frame read a record again)
      rec[u] = i >= end ? cs::u32x4{0u, 0u, 0u, 0u} : kBands ? p.blocks[i] : __builtin_nontemporal_load(p.blocks + i);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) apply(rec[u]);
  }
  __syncthreads();

  const int64_t first = static_cast<int64_t>(frame) * p.n_patch + row_lo * p.grid_w;
  uint32_t* mv = p.mv + first;
  uint8_t* intra = p.intra + first;
  for (int i = tid; i < n_cells; i += kProjectThreads) {
    const unsigned long long key = s_key[i];                  // 0: no moving inter block here
    const uint32_t low = static_cast<uint32_t>(key);
    const uint32_t dx16 = key == 0ull ? 0u : ((low >> 16) - 32768u) & 0xffffu;
    const uint32_t dy16 = key == 0ull ? 0u : ((low & 0xffffu) - 32768u) & 0xffffu;
    mv[i] = dx16 | (dy16 << 16);
    intra[i] = (s_intra[i >> 5] >> (i & 31)) & 1u;
  }
}

}  // namespace

extern "C" int cs_project_blocks(const cs_block* blocks, const int32_t* cu_blocks, int32_t n_frames,
                                 int32_t src_w, int32_t src_h, int32_t in_w, int32_t in_h,
                                 int32_t patch, int32_t grid_h, int32_t grid_w, int16_t* mv,
                                 uint8_t* intra, void* stream) {
  static_assert(sizeof(cs_block) == 16, "block records are 16 bytes");
  if (n_frames < 0 || src_w < 1 || src_h < 1 || in_w < 1 || in_h < 1 || patch < 1 || grid_h < 1 || grid_w < 1)
    return CS_EINVAL;
  if (n_frames == 0) return CS_OK;
  if (!blocks || !cu_blocks || !mv || !intra) return CS_EINVAL;
  if (src_w > 16384 || src_h > 16384 || in_w > 16384 || in_h > 16384 || patch > 1024) return CS_EUNSUPPORTED;
  const int64_t n_patch = static_cast<int64_t>(grid_h) * grid_w;
  if (n_patch > 7168) return CS_EUNSUPPORTED;       // the frame's patch table stays in LDS (under 64 KB)
  if (!cs::aligned16(blocks) || (reinterpret_cast<uintptr_t>(mv) & 3u)) return CS_EUNSUPPORTED;

  ProjectParams p;
  p.blocks = reinterpret_cast<const cs::u32x4*>(blocks);
  p.cu_blocks = cu_blocks;
  p.mv = reinterpret_cast<uint32_t*>(mv);
  p.intra = intra;
  p.src_w = src_w; p.src_h = src_h; p.in_w = in_w; p.in_h = in_h;
  p.den_x = static_cast<uint32_t>(patch) * src_w;
  p.den_y = static_cast<uint32_t>(patch) * src_h;
  p.div_x = exact_div(p.den_x);
  p.div_y = exact_div(p.den_y);
  p.grid_h = grid_h; p.grid_w = grid_w;
  p.n_patch = static_cast<int32_t>(n_patch);
  // Bands: one workgroup per CU, at most eight (past that the records every band reads cost more than its share of
  // the work), one patch row at least.  us with one band / 256 / 512 workgroups in all, 1920 x 1080: 32 frames
  // 13.7 / 8.3 / 8.3, 96 14.2 / 12.6 / 13.5, 255 16.4 / 16.4 / 23.5.  A frame of few blocks and patches is one
  // band: 640 x 360 to 16 x 16 patches, 64 frames, 4.2 / 4.4 / 5.2 (to 26 x 46 5.3 / 5.1 / 6.0).
  int bands = n_frames < 256 ? 256 / n_frames : 1;
  if (static_cast<int64_t>(src_w) * src_h / 256 + 2 * n_patch < 2048) bands = 1;        // macroblocks + 2 patches
  if (bands > 8) bands = 8;
  if (bands > grid_h) bands = grid_h;
  p.n_frames = n_frames;
  p.n_bands = bands;
  const int64_t cells = static_cast<int64_t>((grid_h + bands - 1) / bands) * grid_w;
  const size_t lds = static_cast<size_t>(cells) * 8 + static_cast<size_t>((cells + 31) / 32) * 4;
  const dim3 grid(static_cast<unsigned>(n_frames) * bands), block(kProjectThreads);
  if (bands > 1) hipLaunchKernelGGL(project_blocks_kernel<true>, grid, block, lds, cs::as_stream(stream), p);
  else hipLaunchKernelGGL(project_blocks_kernel<false>, grid, block, lds, cs::as_stream(stream), p);
  return cs::note_hip(hipGetLastError());
}
