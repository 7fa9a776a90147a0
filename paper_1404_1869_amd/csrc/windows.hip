// Crop-before windows: the per-window baseline the paper measures its dense pyramid against (Sec. 3.4)
// and the "crop before" pipeline of Sec. 4.  Every region is cut out of its image in pixel space and
// warped on its own to the classifier's S x S input (bilinear, half-pixel centres, the box stretched
// onto the grid with no context margin), then mean-centred, so that each window can run through the
// conv stack as an independent plane.
//
// Output pixel (i, j) of box (x1, y1, x2, y2) samples the image at
//   sy = y1 + (i + 0.5) (y2 - y1) / S - 0.5,  sx = x1 + (j + 0.5) (x2 - x1) / S - 0.5,
// each clamped to the image ([0, H - 1], [0, W - 1]), so a box reaching outside the image repeats the
// edge pixel with interpolation weights in [0, 1); the top-left neighbour is floor(s), the other one
// lies one further (clamped).  Coordinates and fractions are fp64
// with + - * / only and contraction off, in the order written, so the taps are reproducible bit for
// bit; the blend is fp32.
//
// Bound by the stores of the windows (2000 windows of 227 x 227 in 16 bits are 0.63 GB); the image stays
// in the caches, but gathering a pixel's 12 bytes one by one issues more loads than the stores take time.
// So a workgroup walks down up to RB rows of a box, two neighbouring columns per thread: the
// horizontally blended source rows of the last output row are kept, an output row fetches only source
// rows it does not share with the one above (a box below 227 px high brings less than one new row per
// output row), ahead of the blend that needs them, and the taps of both columns of a channel are
// one 4-byte load (columns less than two source pixels apart; wider boxes load a 2-byte
// pair of taps per column).  2000 boxes on a
// 768 x 1024 image, bf16: 369 -> 155 us (4.1 TB/s written).
// Rows are `pitch` elements apart; the columns from S to pitch - 1 are written as zeros (a pitch that is a
// multiple of 8 lets conv1 load the rows straight into LDS).
#include <cmath>
#include <type_traits>

#include "common.h"

namespace dn {
namespace {

constexpr int RB = 16;   // most output rows per workgroup (12 and 16 within 2 %, 32 6 % slower)
constexpr int NT = 128;  // threads per workgroup, two columns each

struct Tap {
  int32_t i0, i1;
  float frac;
};

#pragma clang fp contract(off)
__device__ inline Tap warp_tap(double lo, double step, int o, int n) {
  double s = lo + (o + 0.5) * step - 0.5;
  s = fmin(fmax(s, 0.0), (double)(n - 1));
  const int i0 = (int)floor(s);
  Tap t;
  t.i0 = i0;
  t.i1 = min(i0 + 1, n - 1);
  t.frac = (float)(s - (double)i0);
  return t;
}

// rows_per: output rows per workgroup (at most RB).  PAIRS: rows and `out` let a thread's two values be
// stored at once.
template <typename T, bool PAIRS>
__global__ __launch_bounds__(NT) void warp_regions_kernel(const uint8_t* __restrict__ img, int n_img, int H,
                                                          int W, const float* __restrict__ boxes,
                                                          const int32_t* __restrict__ box_img, int S, int pitch,
                                                          int row_blocks, int rows_per, float m0,
                                                          float m1, float m2, T* __restrict__ out) {
  typedef uint32_t u32u __attribute__((aligned(1)));
  typedef uint16_t u16u __attribute__((aligned(1)));
  typedef T pair_t __attribute__((ext_vector_type(2)));
  __shared__ Tap s_row[RB];
  const int r = blockIdx.x / row_blocks, i_first = (blockIdx.x % row_blocks) * rows_per;
  const int rows = min(rows_per, S - i_first);
  const double x1 = boxes[4 * r + 0], y1 = boxes[4 * r + 1], x2 = boxes[4 * r + 2], y2 = boxes[4 * r + 3];
  const int b = box_img ? __builtin_amdgcn_readfirstlane(box_img[r]) : 0;
  const bool ok = isfinite(x1) && isfinite(y1) && isfinite(x2) && isfinite(y2) && x2 - x1 > 0 &&
                  y2 - y1 > 0 && b >= 0 && b < n_img;
  const int64_t SS = (int64_t)S * pitch;
  T* o = out + (int64_t)r * 3 * SS + (int64_t)i_first * pitch;
  auto store = [&](int64_t at, uint32_t j, float v0, float v1) {  // columns j, j + 1 of a row
    const pair_t p = from_f32x2<T>(v0, v1);
    T* row = o + at;
    if constexpr (PAIRS) {
      if (j < (uint32_t)pitch) *(pair_t*)(row + j) = p;
    } else {
      if (j < (uint32_t)pitch) row[j] = p[0];
      if (j + 1 < (uint32_t)pitch) row[j + 1] = p[1];
    }
  };
  if (!ok) {
    for (int i = 0; i < rows; ++i)
      for (int j = 2 * threadIdx.x; j < pitch; j += 2 * NT)
#pragma unroll
        for (int c = 0; c < 3; ++c) store(c * SS + (int64_t)i * pitch, j, 0.f, 0.f);
    return;
  }
  const double fx = (x2 - x1) / S, fy = (y2 - y1) / S;
  if ((int)threadIdx.x < rows) s_row[threadIdx.x] = warp_tap(y1, fy, i_first + threadIdx.x, H);
  __syncthreads();
  const int64_t HW = (int64_t)H * W;
  const uint8_t* I = img + (int64_t)b * 3 * HW;
  const float mean[3] = {m0, m1, m2};
  // BYTES fetched per channel: 4 for both columns, whose taps lie in four consecutive bytes when the
  // columns are less than two source pixels apart whatever the coordinates' rounding; 2 per column; 1 in
  // an image one pixel wide.
  auto columns = [&](auto bytes_c) {
    constexpr int BYTES = decltype(bytes_c)::value, NQ = BYTES == 2 ? 2 : 1;
    for (int j = 2 * threadIdx.x; j < pitch; j += 2 * NT) {
      const Tap tx[2] = {warp_tap(x1, fx, min(j, S - 1), W), warp_tap(x1, fx, min(j + 1, S - 1), W)};
      uint32_t at[NQ];           // first byte fetched
      uint32_t s0[2], s1[2];     // bit positions of the taps in the fetched words
#pragma unroll
      for (int k = 0; k < NQ; ++k) at[k] = (uint32_t)min(tx[k].i0, W - BYTES);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        s0[k] = 8u * ((uint32_t)tx[k].i0 - at[k % NQ]);
        s1[k] = 8u * ((uint32_t)tx[k].i1 - at[k % NQ]);
      }
      struct Raw {
        uint32_t q[NQ][3];
      };
      auto fetch = [&](int row) {
        Raw w;
        const uint8_t* p = I + (int64_t)row * W;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int k = 0; k < NQ; ++k) {
            const uint8_t* q = p + c * HW;  // the same for the whole workgroup
            if constexpr (BYTES == 4) w.q[k][c] = *(const u32u*)(q + at[k]);
            if constexpr (BYTES == 2) w.q[k][c] = *(const u16u*)(q + at[k]);
            if constexpr (BYTES == 1) w.q[k][c] = q[at[k]];
          }
        return w;
      };
      auto blend = [&](const Raw& w, float (&v)[2][3]) {  // the source row at both columns
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float a = (float)((w.q[k % NQ][c] >> s0[k]) & 255u), z = (float)((w.q[k % NQ][c] >> s1[k]) & 255u);
            v[k][c] = (1.f - tx[k].frac) * a + tx[k].frac * z;
          }
      };
      float top[2][3], bot[2][3];
      // Rows are the same for the whole workgroup: i0, i1 are the source rows in top and bot.
      auto row_of = [&](int i, int& i0, int& i1) {
        i0 = __builtin_amdgcn_readfirstlane(s_row[i].i0);
        i1 = __builtin_amdgcn_readfirstlane(s_row[i].i1);
      };
      int i0, i1;
      row_of(0, i0, i1);
      Raw raw0 = fetch(i0), raw1 = fetch(i1);
      bool new0 = true, new1 = true, down = false;
      for (int i = 0; i < rows; ++i) {
        if (down) {  // the row above's lower source row is this row's upper one
#pragma unroll
          for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) top[k][c] = bot[k][c];
        }
        if (new0) blend(raw0, top);
        if (new1) blend(raw1, bot);
        if (i + 1 < rows) {
          int n0, n1;
          row_of(i + 1, n0, n1);
          down = n0 != i0 && n0 == i1;
          new0 = n0 != i0 && n0 != i1;
          new1 = n1 != i1;
          if (new0) raw0 = fetch(n0);
          if (new1) raw1 = fetch(n1);
          i0 = n0;
          i1 = n1;
        }
        const float ly = s_row[i].frac;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          float v[2];
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            v[k] = (1.f - ly) * top[k][c] + ly * bot[k][c] - mean[c];
            if (j + k >= S) v[k] = 0.f;
          }
          store(c * SS + (int64_t)i * pitch, (uint32_t)j, v[0], v[1]);
        }
      }
    }
  };
  if (fx <= 1.9 && W >= 4)
    columns(std::integral_constant<int, 4>{});
  else if (W >= 2)
    columns(std::integral_constant<int, 2>{});
  else
    columns(std::integral_constant<int, 1>{});
}

}  // namespace

int launch_warp_regions(const uint8_t* d_img, int32_t n_img, int32_t H, int32_t W, const float* d_boxes,
                        const int32_t* d_box_img, int32_t n, int32_t S, int32_t pitch, const float* mean,
                        dn_dtype dt, void* d_out, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const int row_blocks = (S + RB - 1) / RB, rows_per = (S + row_blocks - 1) / row_blocks;
  const int64_t blocks = (int64_t)n * row_blocks;
  if (blocks <= 0 || blocks > 0x7fffffff) return (int)hipErrorInvalidValue;
  const bool pairs = pitch % 2 == 0 && ((uintptr_t)d_out & (2 * dtype_size(dt) - 1)) == 0;
  auto go = [&](auto tag) {
    using T = decltype(tag);
#define DN_WARP_ARGS \
  d_img, n_img, H, W, d_boxes, d_box_img, S, pitch, row_blocks, rows_per, mean[0], mean[1], mean[2], (T*)d_out
    if (pairs)
      warp_regions_kernel<T, true><<<(unsigned)blocks, NT, 0, s>>>(DN_WARP_ARGS);
    else
      warp_regions_kernel<T, false><<<(unsigned)blocks, NT, 0, s>>>(DN_WARP_ARGS);
#undef DN_WARP_ARGS
  };
  switch (dt) {
    case DN_F32: go(float{}); break;
    case DN_F16: go(_Float16{}); break;
    case DN_BF16: go(__bf16{}); break;
  }
  return (int)hipGetLastError();
}

}  // namespace dn
