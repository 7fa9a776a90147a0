// Convolution engine for conv1..conv5 of the AlexNet topology (the bulk of the path's work, Sec. 3),
// as implicit GEMMs on gfx950 MFMA (32x32x16 tiles, fp32 accumulation): fp16 / bf16 inputs, or fp32 inputs
// as three bf16 parts each.  Bias and ReLU are applied in the epilogue.
//
// GEMM view: rows = output pixels of a 2-D spatial tile, columns = output channels of one group,
// k = (input channel, kernel tap).  A workgroup stages the input tile with its halo in LDS once per
// chunk of 16 input channels and reuses it for every kernel tap, so each input element is read from
// L2 once per output-channel block instead of once per tap.
//
//  conv1 (11x11, stride 4, 3 channels) reads channel-major planes.  Per input channel its 144 k
//  values cover a 12 x 12 tap square (taps with ky = 11 or kx = 11 carry zero weights): k-step s
//  (16 k) covers rows 4 (s / 3) .. + 3 and columns 4 (s % 3) .. + 3, and each lane's 8 k values are
//  4 consecutive input pixels of one row and the 4 below them, read as two 8-byte LDS loads at
//  offsets that do not depend on the lane.
//  conv2..conv5 (stride 1, R x R, pad (R-1)/2, groups) read channels-last maps; k = (tap, channel),
//  each lane's 8 k values are 8 consecutive channels of one pixel (one 16-byte LDS load).
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace dn {
namespace {

// ------------------------------------------------------------------------------------------------
// Packed weight layout
//   conv1, fp32: [96][3][144], k = 16 s + 8 h + 4 j + e holds tap ky = 4 (s / 3) + 2 h + j,
//          kx = 4 (s % 3) + e (zero where ky or kx is 11)
//   conv2..5, fp32: [M][R*R][C/G] (tap-major, channels contiguous); both are read where values do not split
//   conv1, 16-bit types: see pack_conv1_resident_kernel
//   conv2..5, 16-bit types, stage-major for conv_s1_direct_kernel and conv_flat_kernel: per channel block
//          (group g, block of BM output channels) and stage (chunk of 16 input channels, kernel row ky), one
//          contiguous block of R * BM * 2 16-byte pieces, piece (kx BM + m) 2 + p holding input
//          channels 8 (p ^ ((m >> 4) & 1)) .. + 7 of the chunk at tap (ky, kx) of channel m: exactly
//          the order of the LDS weight-row buffer, so each direct load reads 1 KB of contiguous memory
//   conv1..5, fp32: split copies for conv1_f32_kernel and conv_f32_kernel, three bf16 parts of each weight:
//          per channel block of 64, chunk of 16 input channels and tap (conv1: per input channel and
//          k-step, all 96 channels) [3][channels][2 slots of 8 k], the slots swapped as above
//   biases: fp32 [M]
// ------------------------------------------------------------------------------------------------
constexpr int L_M[5] = {96, 256, 384, 384, 256};
constexpr int L_C[5] = {3, 96, 256, 384, 384};
constexpr int L_R[5] = {11, 5, 3, 3, 3};
constexpr int L_G[5] = {1, 2, 1, 2, 2};
constexpr int K1 = 144;  // conv1 packed k per input channel
__host__ __device__ constexpr int conv1_ky(int k) {
  return 4 * ((k >> 4) / 3) + 2 * ((k >> 3) & 1) + ((k >> 2) & 1);
}
__host__ __device__ constexpr int conv1_kx(int k) { return 4 * ((k >> 4) % 3) + (k & 3); }

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

__global__ void pack_conv1_kernel(const float* __restrict__ w, float* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 96 * 3 * K1) return;
  const int k = i % K1, mc = i / K1;  // mc = m * 3 + c
  const int ky = conv1_ky(k), kx = conv1_kx(k);
  float v = 0.f;
  if (ky < 11 && kx < 11) v = w[(mc * 11 + ky) * 11 + kx];
  out[i] = v;
}

__global__ void pack_conv_kernel(const float* __restrict__ w, float* __restrict__ out, int M, int Cg, int RR) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)M * Cg * RR) return;
  const int c = (int)(i % Cg);
  const int t = (int)((i / Cg) % RR);
  const int m = (int)(i / ((int64_t)Cg * RR));
  out[i] = w[((int64_t)m * Cg + c) * RR + t];
}

// conv1, 16-bit types, for conv1_resident_kernel: the 3 x 11 x 11 taps of an output channel as 99
// units of 4 taps (input channel c, kernel row r, columns 4 cb .. 4 cb + 3, the column 11 of the last
// block zero), unit u = 33 c + 11 cb + r, packed into 25 k-steps of 16: k-step j holds units 4 j .. 4 j
// + 3 (a zero unit past 98), k = 8 h + 4 s + e taking unit 4 j + 2 h + s, column 4 cb + e.  Layout
// [25][96][16] in the order of the kernel's LDS weights: the two 16-byte slots of a channel's k-step
// are swapped for channels 16..31 of every 32-channel group.
constexpr int C1_UNITS = 99, C1_KSTEPS = (C1_UNITS + 3) / 4;
template <typename T>
__global__ void pack_conv1_resident_kernel(const float* __restrict__ w, T* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= C1_KSTEPS * 96 * 16) return;
  const int j = i / (96 * 16), m = (i / 16) % 96, kk = i % 16;
  const int h = (kk / 8) ^ ((m >> 4) & 1), sx = (kk % 8) / 4, e = kk % 4;
  const int u = 4 * j + 2 * h + sx;
  float v = 0.f;
  if (u < C1_UNITS) {
    const int c = u / 33, cb = (u % 33) / 11, r = (u % 33) % 11, kx = 4 * cb + e;
    if (kx < 11) v = w[((m * 3 + c) * 11 + r) * 11 + kx];
  }
  out[i] = from_f32<T>(v);
}

template <typename T>
__global__ void pack_stage_kernel(const float* __restrict__ w, T* __restrict__ out, int Mg, int Cg,
                                  int R, int BM, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int e = (int)(i % 8), p = (int)((i / 8) % 2), m = (int)((i / 16) % BM);
  int64_t r = i / (16 * (int64_t)BM);
  const int kx = (int)(r % R);
  r /= R;
  const int ky = (int)(r % R);
  r /= R;
  const int nchunks = Cg / 16;
  const int chunk = (int)(r % nchunks);
  const int64_t blk = r / nchunks;  // channel block: group * (Mg / BM) + block within the group
  const int mpg = Mg / BM;
  const int g = (int)(blk / mpg), mb = (int)(blk % mpg);
  const int v = p ^ ((m >> 4) & 1);
  const int64_t oc = (int64_t)g * Mg + (int64_t)mb * BM + m;
  const int c = chunk * 16 + v * 8 + e;
  out[i] = from_f32<T>(w[((oc * Cg + c) * R + ky) * R + kx]);
}

// Values are split times 2^16: fp32's smallest step, 2^-149, is then 2^-133, bf16's smallest (the matrix
// cores keep bf16's subnormals), so the parts hold every fp32 value below the limit exactly.  Unscaled, the
// third part runs out of bf16's range below 2^-110 (1e-34 is off by 2e-7 of it, 1e-36 by 2e-5, 1.3e-38 by
// 2e-3).  UNSPLIT takes a sum of products back.
constexpr float SPLIT_SCALE = 0x1p16f, UNSPLIT = 0x1p-32f;
// Bits of |2^16 x| from which it rounds to a bf16 infinity (|x| from 5.2e33, infinities, NaN).
constexpr uint32_t SPLIT_LIMIT = 0x7f7f8000u;

// x (scaled) = h + m + l, each the nearest bf16 of the rest.
struct Split3 {
  __bf16 h, m, l;
};
__device__ inline Split3 split3(float x) {
  Split3 s;
  s.h = (__bf16)x;
  const float r = x - (float)s.h;
  s.m = (__bf16)r;
  s.l = (__bf16)(r - (float)s.m);
  return s;
}

// conv2..5, fp32 storage: the stage-major copy for conv_f32_kernel, one thread per weight.  Per channel
// block (group, 64 output channels), chunk of 16 input channels and tap: the weights' three bf16 parts
// [3][64][2 slots], the slots swapped for channels 16..31 of every 32.  *special is set when a weight does
// not split.
__global__ void pack_split_kernel(const float* __restrict__ w, __bf16* __restrict__ out,
                                  uint32_t* __restrict__ special, int Mg, int Cg, int RR, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int c = (int)(i % 16), m = (int)((i / 16) % 64);
  const int64_t r = i / (16 * 64);  // (block, chunk, tap)
  const int tap = (int)(r % RR), nchunks = Cg / 16, chunk = (int)((r / RR) % nchunks);
  const int64_t blk = r / RR / nchunks;
  const int64_t oc = blk * 64 + m;  // blocks run through the groups' channels in order
  const float x = SPLIT_SCALE * w[(oc * Cg + chunk * 16 + c) * RR + tap];
  if ((__builtin_bit_cast(uint32_t, x) & 0x7fffffffu) >= SPLIT_LIMIT) atomicOr(special, 1u);
  const Split3 s = split3(x);
  __bf16* d = out + r * (3 * 64 * 16) + m * 16 + ((c >> 3) ^ ((m >> 4) & 1)) * 8 + (c & 7);
  d[0] = s.h;
  d[64 * 16] = s.m;
  d[2 * 64 * 16] = s.l;
}

// conv1, fp32 storage: per input channel and k-step (K1's order) the weights' three bf16 parts [3][96][2
// slots], the slots swapped for channels 16..31 of every 32.
__global__ void pack_split1_kernel(const float* __restrict__ w, __bf16* __restrict__ out,
                                   uint32_t* __restrict__ special) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 3 * K1 * 96) return;
  const int kk = i % 16, m = (i / 16) % 96, cs = i / (16 * 96);  // cs = channel * 9 + k-step
  const int c = cs / (K1 / 16), k = (cs % (K1 / 16)) * 16 + kk, ky = conv1_ky(k), kx = conv1_kx(k);
  const float x = ky < 11 && kx < 11 ? SPLIT_SCALE * w[((m * 3 + c) * 11 + ky) * 11 + kx] : 0.f;
  if ((__builtin_bit_cast(uint32_t, x) & 0x7fffffffu) >= SPLIT_LIMIT) atomicOr(special, 1u);
  const Split3 s = split3(x);
  __bf16* d = out + cs * (3 * 96 * 16) + m * 16 + ((kk >> 3) ^ ((m >> 4) & 1)) * 8 + (kk & 7);
  d[0] = s.h;
  d[96 * 16] = s.m;
  d[2 * 96 * 16] = s.l;
}

__global__ void clear_words_kernel(uint32_t* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0u;
}

__global__ void copy_f32_kernel(const float* __restrict__ a, float* __restrict__ b, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = a[i];
}

// One 16-byte LDS fragment: 8 consecutive 16-bit values.
template <typename T>
__device__ inline typename Mfma<T>::frag lds_frag16(const T* p) {
  return *(const typename Mfma<T>::frag*)p;
}

// Compute units of the device current at the first call (256 if the query fails), queried once;
// the initialisation is thread-safe.
int device_cu_count() {
  static const int n = [] {
    int dev = 0, v = 0;
    const bool ok = hipGetDevice(&dev) == hipSuccess &&
                    hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess;
    return ok && v > 0 ? v : 256;
  }();
  return n;
}

// ------------------------------------------------------------------------------------------------
// Stride-1 R x R conv with zero padding (R-1)/2, grouped, channels-last: the tile geometry and LDS layout
// the kernels below share.
// Workgroup: TH x TW output pixels x BM output channels of one group.  The MFMA A operand is the
// weights and B the pixels, so each lane's accumulator holds 4 consecutive output channels of one pixel
// per register group.  LDS holds halos ((TH+R-1) x (TW+R-1) pixels) of 16 input channels at a time.
// ------------------------------------------------------------------------------------------------
// Slots (16 bytes) that collide modulo 512 bytes when the 32 lanes of a half-wave read pixels
// (r, c), r < 16, c < 2, of a halo whose rows are rs slots apart (two slots per pixel).
constexpr int colpair_collisions(int rs) {
  int n = 0;
  for (int a = 0; a < 32; ++a)
    for (int b = 0; b < a; ++b)
      if ((((a & 15) * rs + 2 * (a >> 4)) - ((b & 15) * rs + 2 * (b >> 4))) % 32 == 0) {
        ++n;
        break;
      }
  return n;
}
// Padding slots per 16-bit halo row: odd (so the two rows of a 2 x 16 MFMA tile fall on slots of
// opposite parity), and of 1 and 3 the one with fewer collisions for 16 x 2 MFMA tiles.
constexpr int halo_row_pad(int hw) {
  return colpair_collisions(2 * hw + 3) < colpair_collisions(2 * hw + 1) ? 3 : 1;
}

template <typename T, int R, int BM, int TM, int TS, int TN_ = 4>
struct ConvCfg {
  // Tile of TH x TW output pixels, TS = 100 TH + TW (TW 16 or 32, TH TW a multiple of 256).
  static constexpr int TH = TS / 100, TW = TS % 100, CC = 16;
  static_assert(sizeof(T) == 2, "MFMA operands are 16-bit");
  static_assert((TW == 16 || TW == 32) && TH % 2 == 0 && (TH * TW) % 256 == 0, "tile shape");
  static constexpr int TN = TN_;                   // 32-pixel MFMA tiles per wave (32 TN pixels)
  static constexpr int HH = TH + R - 1, HW = TW + R - 1;
  static constexpr int WM = BM / (32 * TM), WN = (TH * TW) / (32 * TN);
  static constexpr int NT = 64 * WM * WN;
  static constexpr int VEC = 8;                    // elements per 16-byte slot
  static_assert(WM * 32 * TM == BM, "channel block must be whole wave tiles");
  // LDS layout.  A pixel (or an output channel's weight row) is 32 bytes, two 16-byte slots.  The 32
  // lanes of a half-wave read 16 bytes each and must hit distinct slots modulo 512 bytes: a halo row
  // is padded by an odd number of slots (RP), so the two tile rows a half-wave reads land on slots of
  // opposite parity; the weight rows of channels 16..31 of a 32-channel group swap their two slots.
  static constexpr int PS = CC;                         // pixel stride (elements)
  static constexpr int RP = halo_row_pad(HW);           // halo row padding (16-byte slots)
  static constexpr int RSS = 2 * HW + RP;               // halo row stride (slots)
  static constexpr int RS = HW * PS + 8 * RP;           // halo row stride (elements)
  static constexpr int STAGE_E = WM * WN * 32 * TN * 64;  // epilogue staging of 64 channels per wave
  __device__ static inline int halo_off(int hy, int hx, int v) { return hy * RS + hx * PS + v * VEC; }
  // Tile pixel of index idx: each 32-pixel MFMA tile is 2 rows x 16 columns (the two rows a half-wave
  // reads then fall on LDS slots of opposite parity); with 32-column tiles, MFMA tiles 2 p and 2 p + 1
  // are the left and right halves of row pair p.
  __device__ static inline int pix_row(int idx) { return 2 * ((idx >> 5) / (TW / 16)) + ((idx >> 4) & 1); }
  __device__ static inline int pix_col(int idx) { return 16 * ((idx >> 5) % (TW / 16)) + (idx & 15); }
  __device__ static inline int w_off(int kx, int m, int v) {
    return (kx * BM + m) * PS + (v ^ ((m >> 4) & 1)) * VEC;
  }
};

template <typename T, int BM, int TM, int TS, int TN = 4>
constexpr int conv_threads() {
  return 64 * (BM / (32 * TM)) * (TS / 100) * (TS % 100) / (32 * TN);
}

// Sum of the ksplit partial copies of a split fp32 conv launch, in copy order, plus bias, then ReLU:
// run r has tiles_x workgroups of 256 four-channel groups per plane (Ho x Wo x M outputs).
__global__ __launch_bounds__(256) void split_reduce_kernel(const float* __restrict__ part,
                                                           int64_t part_slice, int ksplit,
                                                           const float* __restrict__ bias,
                                                           float* __restrict__ out, KRuns runs, int M) {
  int bid = blockIdx.x;
  const KRun& rn = runs.r[run_of(runs, bid)];
  bid -= rn.first;
  const int plane = bid / rn.tiles_x, v = (bid % rn.tiles_x) * 256 + (int)threadIdx.x;
  if ((int64_t)v * 4 >= (int64_t)rn.Ho * rn.Wo * M) return;
  const int64_t o = rn.out_off + plane * rn.out_stride + (int64_t)v * 4;
  f32x4 acc = *(const f32x4*)(part + o);
  for (int k = 1; k < ksplit; ++k) {
    const f32x4 p = *(const f32x4*)(part + k * part_slice + o);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += p[e];
  }
  const f32x4 b = *(const f32x4*)(bias + (v * 4) % M);
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] = fmaxf(acc[e] + b[e], 0.f);
  *(f32x4*)(out + o) = acc;
}

// ------------------------------------------------------------------------------------------------
// Stride-1 conv for 16-bit storage with direct global->LDS loads.  Waves: BM/(32 TM) along channels x
// (TH TW)/(32 TN) along pixels.  Pipeline: a stage is (chunk of 16 input channels, kernel row ky).  LDS
// holds two halo buffers (one per chunk) and two weight-row buffers (R taps x BM x 16).  While a stage
// computes, the next stage's weight row (and, during a chunk's first row, the next chunk's halo) is
// loaded by buffer_load_dwordx4 ... lds: one wave instruction writes 64 consecutive 16-byte LDS slots,
// each lane choosing the global address of its slot (padding slots and halo pixels outside the map use
// an offset past the buffer's end, which the hardware returns as zeros).  No registers hold staged data
// and no LDS store instructions are issued; a stage's loads are waited for (vmcnt) just before the
// barrier that publishes them.
// ------------------------------------------------------------------------------------------------
template <int BYTES>
struct Pieces {  // 1 KB LDS pieces, rounded up to a whole number per wave
  static constexpr int count(int slots, int waves) { return ((slots + 63) / 64 + waves - 1) / waves; }
};

// Wait until every vector-memory access of this wave has completed (vmcnt 0; other counters left
// free), as an instruction the compiler's own wait bookkeeping sees.
__device__ inline void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Output stores are non-temporal: the next layer reads a batch's maps only after this launch has
// written all of them, so they need not stay in the caches next to this layer's inputs.
template <typename V>
__device__ inline void store_out(const V& v, V* p) {
  __builtin_nontemporal_store(v, p);
}

__device__ inline void lds_direct16(__amdgpu_buffer_rsrc_t rsrc, void* lds_piece, uint32_t voff,
                                    uint32_t soff = 0) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds_piece,
                                           16, voff, soff, 0, 0);
}

// BMP: the channel block the stage-major weight copy is cut in (a multiple of BM); a workgroup's BM
// channels are a sub-block of one such block.  TN_: 32-pixel MFMA tiles per wave.  MULTI: the launch
// holds several runs (else run 0 only).
template <typename T, int R, int BM, int TM, int OCC, int TS, int BMP, int TN_, bool MULTI>
__global__ __launch_bounds__((conv_threads<T, BM, TM, TS, TN_>()), OCC) void conv_s1_direct_kernel(
    const T* __restrict__ in, T* __restrict__ out, const T* __restrict__ wp,
    const float* __restrict__ bias, KRuns runs, int C, int Cg, int M, int Mg, int mblocks) {
  using Cf = ConvCfg<T, R, BM, TM, TS, TN_>;
  using Op = Mfma<T>;
  static_assert(TM == 2 || TM == 3, "epilogues for 64 or 96 channels per wave");
  constexpr int pad = (R - 1) / 2;
  constexpr int TN = Cf::TN, NW = Cf::WM * Cf::WN;
  static_assert(BMP % BM == 0, "a channel block is a sub-block of the weight copy's block");
  constexpr int HSLOTS = Cf::HH * Cf::RSS, WSLOTS = R * BM * 2, WSLOTS_P = R * BMP * 2;
  constexpr int DH = Pieces<16>::count(HSLOTS, NW), DW = Pieces<16>::count(WSLOTS, NW);
  constexpr int HALO_E = DH * NW * 512, W_E = DW * NW * 512;  // elements (2 bytes)
  constexpr int PIPE_E = 2 * HALO_E + 2 * W_E;
  // TM = 2: the epilogue stages 16 KB per wave; when that would set the LDS size, it runs in two
  // rounds of half the waves each.  TM = 3 stages 32 pixels per wave at a time (below).
  constexpr int ROUNDS = (TM == 2 && Cf::STAGE_E > PIPE_E && NW % 2 == 0) ? 2 : 1;
  constexpr int STG_E = TM == 2 ? Cf::STAGE_E / ROUNDS : 0;
  constexpr int LDS_E = PIPE_E > STG_E ? PIPE_E : STG_E;
  typedef T out4_t __attribute__((ext_vector_type(4)));
  __shared__ __align__(1024) T s_mem[LDS_E];
  auto halo_buf = [&](int b) { return s_mem + b * HALO_E; };
  auto wrow_buf = [&](int b) { return s_mem + 2 * HALO_E + b * W_E; };

  const int nb = gridDim.x, xcd = blockIdx.x % 8, per = nb / 8, rem = nb % 8;
  int bid = xcd * per + min(xcd, rem) + blockIdx.x / 8;
  const KRun& rn = runs.r[run_of<MULTI>(runs, bid)];
  bid -= rn.first;
  const int H = rn.H, W = rn.W, tiles_x = rn.tiles_x, tiles_y = rn.tiles_y;
  const int64_t in_stride = rn.in_stride, out_stride = rn.out_stride;
  in += rn.in_off;
  out += rn.out_off;
  const int mb = bid % mblocks;
  bid /= mblocks;
  const int tx = bid % tiles_x;
  bid /= tiles_x;
  const int ty = bid % tiles_y;
  const int plane = bid / tiles_y;
  const int mpg = Mg / BM;
  const int g = mb / mpg, m0 = (mb % mpg) * BM;
  const int oy0 = ty * Cf::TH, ox0 = tx * Cf::TW;
  const T* src = in + plane * in_stride + g * Cg;
  // The stage-major weights of the enclosing BMP-channel block: per stage one contiguous block of
  // WSLOTS_P 16-byte pieces, [kernel column][BMP channels][2 slots]; this workgroup's channels start
  // msub channels into it.
  const int mbp = g * (Mg / BMP) + m0 / BMP, msub = m0 % BMP;
  const T* wg = wp + (int64_t)mbp * (Cg / Cf::CC) * R * (WSLOTS_P * 8);
  const __amdgpu_buffer_rsrc_t rsrc_in =
      uniform_rsrc(src, (uint32_t)(((int64_t)H * W * C - g * Cg) * sizeof(T)));
  const __amdgpu_buffer_rsrc_t rsrc_w = uniform_rsrc(wg, (uint32_t)((Cg / Cf::CC) * R * WSLOTS_P * 16));
  constexpr uint32_t OOB = 0x80000000u;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave % Cf::WM, wn = wave / Cf::WM;
  const int half = lane >> 5, l32 = lane & 31;
  // MFMA pixel tile t of wave wn is the tile's (t WN + wn)-th 32-pixel tile: the waves along pixels
  // take the tiles in turn, so a partly filled bottom band splits its rows over them.
  auto gtile = [&](int t) { return t * Cf::WN + wn; };
  // Two layouts of the tile's pixels over the MFMA tiles.  Row layout: each MFMA tile is 2 rows x 16
  // columns (pix_row / pix_col).  Column-pair layout, for a tile cut by the map's right edge (cv < TW
  // columns in the map): MFMA tile m is the 16 rows of columns 2 m and 2 m + 1 (lane l: row l % 16,
  // column 2 m + l / 16), so only ceil(cv / 2) MFMA tiles are computed instead of all TW / 16 column
  // blocks.  A tile takes the layout with fewer MFMA tiles holding a map pixel (ties: rows).
  const int cv = min(Cf::TW, W - ox0), rv = min(Cf::TH, H - oy0);
  const int n_rows = ((rv + 1) / 2) * (Cf::TW / 16), n_cols = (cv + 1) / 2;
  const bool colpair = Cf::TH == 16 && n_cols < n_rows;
  const int n_mt = colpair ? n_cols : n_rows;  // MFMA tiles holding a map pixel: tiles 0 .. n_mt - 1
  auto out_row = [&](int idx) { return colpair ? (idx & 15) : Cf::pix_row(idx); };
  auto out_col = [&](int idx) { return colpair ? 2 * (idx >> 5) + ((idx >> 4) & 1) : Cf::pix_col(idx); };
  // LDS offset of this lane's pixel in MFMA pixel tile t: pix0 + t DPIX (tile t of the wave lies
  // t WN tiles further: 2 t WN / (TW / 16) halo rows down, or 2 t WN columns right), so the reads
  // take immediate offsets.
  static_assert(Cf::WN % (Cf::TW / 16) == 0, "a wave's MFMA tiles are whole row pairs apart");
  constexpr int DPIX_R = 2 * (Cf::WN / (Cf::TW / 16)) * Cf::RS, DPIX_C = 2 * Cf::WN * Cf::PS;
  const int pix0 = Cf::halo_off(out_row(gtile(0) * 32 + l32), out_col(gtile(0) * 32 + l32), 0);
  // Byte offsets (chunk 0) of this lane's halo slot in each of its wave's LDS pieces; the chunk's
  // offset goes in the scalar offset (a lane past the plane keeps an offset the hardware drops).
  uint32_t hoff[DH];
#pragma unroll
  for (int i = 0; i < DH; ++i) {
    const int q = (wave * DH + i) * 64 + lane;
    const int row = q / Cf::RSS, r = q % Cf::RSS;
    const int iy = oy0 - pad + row, ix = ox0 - pad + r / 2;
    const bool ok = row < Cf::HH && r < 2 * Cf::HW && iy >= 0 && iy < H && ix >= 0 && ix < W;
    hoff[i] = ok ? (uint32_t)((((int64_t)iy * W + ix) * C + (r & 1) * 8) * sizeof(T)) : OOB;
  }
  auto load_halo = [&](int buf, int c0) {
#pragma unroll
    for (int i = 0; i < DH; ++i)
      lds_direct16(rsrc_in, halo_buf(buf) + (wave * DH + i) * 512, hoff[i], (uint32_t)(c0 * sizeof(T)));
  };
  // Weight piece p of a stage block lands in LDS piece p: lane offset 16 lane, the piece's and the
  // stage's offsets in the scalar offset; the wave skips pieces past the block.
  static_assert(WSLOTS % 64 == 0, "a stage's weights are whole 1 KB pieces");
  const uint32_t lane16 = (uint32_t)lane * 16u;
  // (the wave index as a scalar: the piece offsets go in the scalar offset operand)
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  auto load_w = [&](int buf, int c0, int ky) {  // stage (chunk c0 / 16, kernel row ky)
    const uint32_t add = (uint32_t)(((c0 / Cf::CC) * R + ky) * WSLOTS_P * 16);
#pragma unroll
    for (int i = 0; i < DW; ++i) {
      const int p = wave_s * DW + i;  // piece p: kernel column p / (BM / 32), channels 32 (p % (BM / 32))
      const uint32_t src = BMP == BM ? (uint32_t)p * 1024u
                                     : (uint32_t)(((p / (BM / 32)) * BMP + msub + 32 * (p % (BM / 32))) * 32);
      if (p * 64 < WSLOTS) lds_direct16(rsrc_w, wrow_buf(buf) + p * 512, lane16, add + src);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int t = 0; t < TN; ++t) acc[a][t] = f32x16{};

  const int nchunks = Cg / Cf::CC, nst = nchunks * R;
  // MFMA pixel tiles of this wave that hold a pixel of the map: a prefix of its TN tiles.  In a
  // tile cut by the map's bottom or right edge the wave runs a stage loop that skips the empty
  // tiles' reads and MFMAs; every wave still issues its share of the loads and reaches the same
  // barriers.
  int tnv = 0;
#pragma unroll
  for (int t = 0; t < TN; ++t) tnv += gtile(t) < n_mt ? 1 : 0;
  tnv = __builtin_amdgcn_readfirstlane(tnv);
  auto stage_loop = [&](auto tnv_c, auto dpix_c) {
    constexpr int TNV = decltype(tnv_c)::value, DPIX = decltype(dpix_c)::value;
    load_halo(0, 0);
    load_w(0, 0, 0);
    wait_vmem();
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
      const int chunk = st / R, ky = st - chunk * R;
      const bool next_w = st + 1 < nst, next_h = ky == 0 && chunk + 1 < nchunks;
      const int wbuf = (st + 1) & 1, wc0 = ((st + 1) / R) * Cf::CC, wky = (st + 1) % R;
      const int hbuf = (chunk + 1) & 1, hc0 = (chunk + 1) * Cf::CC;
      const T* hs = halo_buf(chunk & 1);
      const T* ws = wrow_buf(st & 1);
      if (next_w) load_w(wbuf, wc0, wky);
      if (next_h) load_halo(hbuf, hc0);
      if constexpr (TNV > 0) {
#pragma unroll
        for (int kx = 0; kx < R; ++kx) {
          typename Op::frag x[TNV], w[TM];
#pragma unroll
          for (int t = 0; t < TNV; ++t)
            x[t] = lds_frag16<T>(hs + pix0 + t * DPIX + ky * Cf::RS + kx * Cf::PS + half * 8);
#pragma unroll
          for (int mt = 0; mt < TM; ++mt)
            w[mt] = lds_frag16<T>(ws + Cf::w_off(kx, wm * 32 * TM + mt * 32 + l32, half));
#pragma unroll
          for (int mt = 0; mt < TM; ++mt)
#pragma unroll
            for (int t = 0; t < TNV; ++t) acc[mt][t] = Op::mma(w[mt], x[t], acc[mt][t]);
        }
      }
      wait_vmem();
      __syncthreads();
    }
  };
  static_assert(TN >= 1 && TN <= 4, "stage loop variants cover 0..4 tiles");
  using RowL = std::integral_constant<int, DPIX_R>;
  using ColL = std::integral_constant<int, DPIX_C>;
  auto run_layout = [&](auto layout) {
    switch (tnv) {
      case 4: if constexpr (TN >= 4) stage_loop(std::integral_constant<int, 4>{}, layout); break;
      case 3: if constexpr (TN >= 3) stage_loop(std::integral_constant<int, 3>{}, layout); break;
      case 2: if constexpr (TN >= 2) stage_loop(std::integral_constant<int, 2>{}, layout); break;
      case 1: stage_loop(std::integral_constant<int, 1>{}, layout); break;
      default: stage_loop(std::integral_constant<int, 0>{}, layout); break;
    }
  };
  if (colpair)
    run_layout(ColL{});
  else
    run_layout(RowL{});

  typedef T vec8_t __attribute__((ext_vector_type(8)));
  T* dst = out + plane * out_stride;
  if constexpr (TM == 2) {
    // Epilogue: stage each wave's pixels x 64 channels (one 128-byte line per pixel) in LDS, 16-byte
    // chunks XOR-swizzled by the pixel index, then write whole lines: 8 lanes per pixel.
    constexpr int WPR = NW / ROUNDS;  // waves staging per round
  #pragma unroll
    for (int round = 0; round < ROUNDS; ++round) {
      if (round) __syncthreads();
      const bool mine = wave / WPR == round;
      T* stg = s_mem + (wave % WPR) * (32 * TN * 64);
      if (mine) {
  #pragma unroll
        for (int mt = 0; mt < TM; ++mt)
  #pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int j = 4 * mt + q;
            const f32x4 bv = *(const f32x4*)(bias + g * Mg + m0 + wm * 64 + 8 * j + 4 * half);
  #pragma unroll
            for (int t = 0; t < TN; ++t) {
              const int p = t * 32 + l32;
              out4_t r;
  #pragma unroll
              for (int e = 0; e < 4; ++e)
                r[e] = from_f32<T>(fmaxf(acc[mt][t][4 * q + e] + bv[e], 0.f));
              const int key = (p & 7) ^ ((p >> 3) & 3);
              *(out4_t*)(stg + p * 64 + ((j ^ key) * 8) + 4 * half) = r;
            }
          }
      }
      __syncthreads();
      if (mine) {
        const int j = lane & 7;
  #pragma unroll
        for (int it = 0; it < (32 * TN) / 8; ++it) {
          const int p = it * 8 + (lane >> 3);
          const int key = (p & 7) ^ ((p >> 3) & 3);
          const vec8_t v = *(const vec8_t*)(stg + p * 64 + ((j ^ key) * 8));
          const int idx = gtile(p >> 5) * 32 + (p & 31);
          const int oy = oy0 + out_row(idx), ox = ox0 + out_col(idx);
          if (oy < H && ox < W)
            store_out(v, (vec8_t*)(dst + ((int64_t)oy * W + ox) * M + g * Mg + m0 + wm * 64 + 8 * j));
        }
      }
    }
  } else {
    // TM = 3: each wave owns 96 channels (192 bytes) of each of its 128 pixels.  After the loop's
    // last barrier no wave reads the stage buffers, so each wave stages one 32-pixel MFMA tile at a
    // time in a private LDS region (rows of 96 channels + one 16-byte slot: conflict-free 8-byte
    // writes), then writes each pixel's 192 bytes as 16-byte chunks.
    constexpr int SROW = 32 * TM + 8, NCH = 4 * TM;
    static_assert(NW * 32 * SROW <= LDS_E, "per-wave staging fits the stage buffers");
    T* stg = s_mem + wave * (32 * SROW);
    const int mw = g * Mg + m0 + wm * 32 * TM;  // this wave's first output channel
#pragma unroll
    for (int t = 0; t < TN; ++t) {
#pragma unroll
      for (int mt = 0; mt < TM; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = mt * 32 + 8 * q + 4 * half;
          const f32x4 bv = *(const f32x4*)(bias + mw + m);
          out4_t o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = from_f32<T>(fmaxf(acc[mt][t][4 * q + e] + bv[e], 0.f));
          *(out4_t*)(stg + l32 * SROW + m) = o;
        }
#pragma unroll
      for (int it = 0; it < NCH / 2; ++it) {  // 32 pixels x NCH chunks over 64 lanes
        const int u = it * 64 + lane, p = u / NCH, ch = u % NCH;
        const vec8_t v = *(const vec8_t*)(stg + p * SROW + 8 * ch);
        const int idx = gtile(t) * 32 + p;
        const int oy = oy0 + out_row(idx), ox = ox0 + out_col(idx);
        if (oy < H && ox < W) store_out(v, (vec8_t*)(dst + ((int64_t)oy * W + ox) * M + mw + 8 * ch));
      }
    }
  }
}

// Keeps the compiler from moving this wave's LDS accesses across it (a wave's own LDS operations
// execute in order).
__device__ inline void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// f(integral_constant<I>) for I = B .. E - 1, in order.
template <int B, int E, typename F>
__device__ inline void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// ------------------------------------------------------------------------------------------------
// Stride-1 conv for 16-bit storage on small maps: the pixels of a run's planes as one sequence.
// A 16 x 16 tile of a 13 x 13 map computes 7 MFMA pixel tiles for 169 pixels (5.3 tiles' worth), and its
// workgroup a whole map whatever its size.  Here a workgroup takes PT consecutive pixels of the
// sequence (plane, row, column), across row and plane boundaries, so that only the run's last MFMA
// tile has empty pixels.
// Halo: positions are numbered along padded planes, pad = (R - 1) / 2 zero columns left of each row and
// pad zero rows above each plane (the zeros right of a row and below a plane are the next row's and
// plane's), so a tap is a constant distance away and the halo of consecutive pixels is a contiguous
// range of positions.  LDS holds the 16-byte halves (channels 0..7 and 8..15 of the chunk) of HS
// positions in two planes: 32 consecutive pixels read 32 consecutive slots, conflict-free but for a
// slot or two where a row ends.  Stages, weights and the order of the sums are conv_s1_direct_kernel's, so
// the results are the same bit for bit.  Bound by the matrix cores: conv3 of 2000 windows (13 x 13 maps, bf16)
// 566 -> 453 us (1.32 PFLOP/s), conv4 470 -> 360, conv5 292 -> 245, their conv2 (27 x 27) 787 -> 719.
// ------------------------------------------------------------------------------------------------
// CHUNKED: a stage is a whole chunk (all R kernel rows' weights).
template <typename T, int R, int BM, int TM, int OCC, int BMP, int WN, int TN, int HS, bool CHUNKED, bool MULTI>
__global__ __launch_bounds__(64 * (BM / (32 * TM)) * WN, OCC) void conv_flat_kernel(
    const T* __restrict__ in, T* __restrict__ out, const T* __restrict__ wp, const float* __restrict__ bias,
    KRuns runs, int C, int Cg, int M, int Mg, int mblocks) {
  using Op = Mfma<T>;
  using frag = typename Op::frag;
  typedef T out4_t __attribute__((ext_vector_type(4)));
  typedef T vec8_t __attribute__((ext_vector_type(8)));
  constexpr int pad = (R - 1) / 2, WM = BM / (32 * TM), NW = WM * WN, PT = 32 * TN * WN;
  static_assert(WM * 32 * TM == BM && BMP % BM == 0 && HS % 64 == 0, "whole wave tiles and load pieces");
  constexpr int WSLOTS = R * BM * 2, WSLOTS_P = R * BMP * 2, DW = Pieces<16>::count(WSLOTS, NW);
  static_assert(WSLOTS % 64 == 0, "a stage's weights are whole 1 KB pieces");
  constexpr int DH = (HS / 64 + NW - 1) / NW;                     // groups of 64 positions per wave
  constexpr int HALF_E = HS * 8, HALO_E = 2 * HALF_E, ROW_E = DW * NW * 512, W_E = CHUNKED ? R * ROW_E : ROW_E;
  constexpr int SROW = 32 * TM + 8;                               // epilogue staging: a pixel's row
  static_assert(NW * 32 * SROW <= 2 * HALO_E + 2 * W_E, "per-wave staging fits the stage buffers");
  __shared__ __align__(1024) T s_mem[2 * HALO_E + 2 * W_E];
  auto halo_buf = [&](int b) { return s_mem + b * HALO_E; };
  auto wrow_buf = [&](int b) { return s_mem + 2 * HALO_E + b * W_E; };

  const int nb = gridDim.x, xcd = blockIdx.x % 8, per = nb / 8, rem = nb % 8;
  int bid = xcd * per + min(xcd, rem) + blockIdx.x / 8;
  const KRun& rn = runs.r[run_of<MULTI>(runs, bid)];
  bid -= rn.first;
  const int H = rn.H, W = rn.W, total = rn.tiles_y * H * W;  // tiles_y: planes; all pixels of the run
  const int mb = bid % mblocks, p0 = (bid / mblocks) * PT;   // channel block, first pixel
  const int mpg = Mg / BM, g = mb / mpg, m0 = (mb % mpg) * BM;
  const int mbp = g * (Mg / BMP) + m0 / BMP, msub = m0 % BMP;
  const int Wp = W + pad, Hp = H + pad, HW = H * W;
  // Padded position of pixel p; a pixel's first tap (0, 0) is pad (Wp + 1) positions before it.
  auto position = [&](int p) {
    const int pl = p / HW, r = p - pl * HW, y = r / W, x = r - y * W;
    return (pl * Hp + pad + y) * Wp + pad + x;
  };
  const int last = min(p0 + PT, total) - 1, pos0 = position(p0);
  const int first_tap = pos0 - pad * (Wp + 1);                             // halo slot 0
  const int nslots = position(last) - pos0 + 2 * pad * (Wp + 1) + 1;       // at most HS
  // Loads address the run from pixel `base` on, which no pixel of the halo precedes.
  const int base = max(p0 - pad * (Wp + 1), 0);
  const T* src = in + rn.in_off + (int64_t)base * C + g * Cg;
  const int64_t left = ((int64_t)(total - base) * C - g * Cg) * (int64_t)sizeof(T);
  const __amdgpu_buffer_rsrc_t rsrc_in = uniform_rsrc(src, (uint32_t)min(left, (int64_t)0x7fffffff));
  const T* wg = wp + (int64_t)mbp * (Cg / 16) * R * (WSLOTS_P * 8);
  const __amdgpu_buffer_rsrc_t rsrc_w = uniform_rsrc(wg, (uint32_t)((Cg / 16) * R * WSLOTS_P * 16));
  constexpr uint32_t OOB = 0x80000000u;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int wm = wave % WM, wn = wave / WM;
  const int half = lane >> 5, l32 = lane & 31;
  auto gtile = [&](int t) { return t * WN + wn; };  // MFMA pixel tile t of this wave
  // Groups of 64 halo positions go to the waves in turn; byte offset of this lane's position in each.
  uint32_t hoff[DH];
#pragma unroll
  for (int i = 0; i < DH; ++i) {
    const int s = (wave + NW * i) * 64 + lane, q = first_tap + s;
    const int row = q / Wp, x = q - row * Wp - pad, pl = row / Hp, y = row - pl * Hp - pad;
    const int p = pl * HW + y * W + x;
    const bool ok = s < nslots && x >= 0 && y >= 0 && p < total;
    hoff[i] = ok ? (uint32_t)(p - base) * (uint32_t)(C * (int)sizeof(T)) : OOB;
  }
  auto load_halo = [&](int buf, int c0) {
#pragma unroll
    for (int i = 0; i < DH; ++i) {
      const int grp = wave_s + NW * i;
      if (grp * 64 < nslots) {
        lds_direct16(rsrc_in, halo_buf(buf) + grp * 512, hoff[i], (uint32_t)(c0 * sizeof(T)));
        lds_direct16(rsrc_in, halo_buf(buf) + HALF_E + grp * 512, hoff[i], (uint32_t)(c0 * sizeof(T)) + 16u);
      }
    }
  };
  const uint32_t lane16 = (uint32_t)lane * 16u;
  auto load_w = [&](T* row, int c0, int ky) {  // as conv_s1_direct_kernel
    const uint32_t add = (uint32_t)(((c0 / 16) * R + ky) * WSLOTS_P * 16);
#pragma unroll
    for (int i = 0; i < DW; ++i) {
      const int p = wave_s * DW + i;
      const uint32_t from = BMP == BM ? (uint32_t)p * 1024u
                                      : (uint32_t)(((p / (BM / 32)) * BMP + msub + 32 * (p % (BM / 32))) * 32);
      if (p * 64 < WSLOTS) lds_direct16(rsrc_w, row + p * 512, lane16, add + from);
    }
  };

  int pix[TN];  // LDS element offset of this lane's pixel's first tap, in the half it reads
  int tnv = 0;  // MFMA pixel tiles of this wave with a pixel: a prefix
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    pix[t] = (position(min(p0 + gtile(t) * 32 + l32, last)) - pos0) * 8 + half * HALF_E;
    tnv += p0 + gtile(t) * 32 <= last ? 1 : 0;
  }
  tnv = __builtin_amdgcn_readfirstlane(tnv);
  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int t = 0; t < TN; ++t) acc[a][t] = f32x16{};

  const int nchunks = Cg / 16, nst = nchunks * R;
  auto stage_loop = [&](auto tnv_c) {
    constexpr int TNV = decltype(tnv_c)::value;
    auto row_taps = [&](const T* halo, const T* ws, int ky) {
      if constexpr (TNV > 0) {
        const T* hs = halo + ky * Wp * 8;
#pragma unroll
        for (int kx = 0; kx < R; ++kx) {
          frag x[TNV], w[TM];
#pragma unroll
          for (int t = 0; t < TNV; ++t) x[t] = lds_frag16<T>(hs + pix[t] + kx * 8);
#pragma unroll
          for (int mt = 0; mt < TM; ++mt) {
            const int m = wm * 32 * TM + mt * 32 + l32;
            w[mt] = lds_frag16<T>(ws + (kx * BM + m) * 16 + (half ^ ((m >> 4) & 1)) * 8);
          }
#pragma unroll
          for (int mt = 0; mt < TM; ++mt)
#pragma unroll
            for (int t = 0; t < TNV; ++t) acc[mt][t] = Op::mma(w[mt], x[t], acc[mt][t]);
        }
      }
    };
    if constexpr (CHUNKED) {
      auto load = [&](int chunk) {
        load_halo(chunk & 1, chunk * 16);
#pragma unroll
        for (int ky = 0; ky < R; ++ky) load_w(wrow_buf(chunk & 1) + ky * ROW_E, chunk * 16, ky);
      };
      load(0);
      wait_vmem();
      __syncthreads();
      for (int chunk = 0; chunk < nchunks; ++chunk) {
        if (chunk + 1 < nchunks) load(chunk + 1);
#pragma unroll
        for (int ky = 0; ky < R; ++ky) row_taps(halo_buf(chunk & 1), wrow_buf(chunk & 1) + ky * ROW_E, ky);
        wait_vmem();
        __syncthreads();
      }
    } else {
      load_halo(0, 0);
      load_w(wrow_buf(0), 0, 0);
      wait_vmem();
      __syncthreads();
      for (int st = 0; st < nst; ++st) {
        const int chunk = st / R, ky = st - chunk * R;
        if (st + 1 < nst) load_w(wrow_buf((st + 1) & 1), ((st + 1) / R) * 16, (st + 1) % R);
        if (ky == 0 && chunk + 1 < nchunks) load_halo((chunk + 1) & 1, (chunk + 1) * 16);
        row_taps(halo_buf(chunk & 1), wrow_buf(st & 1), ky);
        wait_vmem();
        __syncthreads();
      }
    }
  };
  static_assert(TN >= 1 && TN <= 4, "stage loop variants cover 0..4 tiles");
  switch (tnv) {
    case 4: if constexpr (TN >= 4) stage_loop(std::integral_constant<int, 4>{}); break;
    case 3: if constexpr (TN >= 3) stage_loop(std::integral_constant<int, 3>{}); break;
    case 2: if constexpr (TN >= 2) stage_loop(std::integral_constant<int, 2>{}); break;
    case 1: stage_loop(std::integral_constant<int, 1>{}); break;
    default: stage_loop(std::integral_constant<int, 0>{}); break;
  }

  // Epilogue: each wave stages one MFMA pixel tile at a time in a private LDS region and writes its
  // pixels' rows of 32 TM channels as 16-byte chunks.  The pixels' outputs are consecutive in memory.
  constexpr int NCH = 4 * TM;
  T* stg = s_mem + wave * (32 * SROW);
  const int mw = g * Mg + m0 + wm * 32 * TM;  // this wave's first output channel
  T* dst = out + rn.out_off + (int64_t)p0 * M + mw;
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    wave_lds_order();
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = mt * 32 + 8 * q + 4 * half;
        const f32x4 bv = *(const f32x4*)(bias + mw + m);
        out4_t o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = from_f32<T>(fmaxf(acc[mt][t][4 * q + e] + bv[e], 0.f));
        *(out4_t*)(stg + l32 * SROW + m) = o;
      }
    wave_lds_order();
#pragma unroll
    for (int it = 0; it < NCH / 2; ++it) {  // 32 pixels x NCH chunks over 64 lanes
      const int u = it * 64 + lane, p = u / NCH, ch = u % NCH;
      const vec8_t v = *(const vec8_t*)(stg + p * SROW + 8 * ch);
      const int idx = gtile(t) * 32 + p;
      if (p0 + idx <= last) store_out(v, (vec8_t*)(dst + (int64_t)idx * M + 8 * ch));
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Stride-1 conv for fp32 storage on the bf16 matrix cores, by the three-way bf16 split with six products of
// Henry, Tang and Heinecke ("Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision
// Computations", ARITH 2019).  A value is x = h + m + l, each the nearest bf16 of what is left: exact, with
// |m| <= 2^-8 |x| and |l| <= 2^-17 |x|.  A product x w is taken as h h' + (h m' + m h') + (m m' + h l' + l h');
// the dropped m l' + l m' + l l' are at most 2^-24 (1 + 2^-10) |x w| and of both signs, so one product may be
// off by about the half ulp that rounding it to fp32 would cost (an fp32 MFMA rounds its sum only).  Six bf16
// MFMAs replace eight fp32 ones of the same k, and run at 16 times their rate.  h h' and the five small terms
// are summed in accumulators of their own, so the sum of the large terms is rounded once per 16 k (the fp32
// MFMA rounds it once per 2 k): over a layer's K the error against 64 bits falls two to three times.
// Values that do not split (infinities, NaN, and finite values from 5.2e33) are seen as they are staged
// (inputs) or packed (weights), and products that pass fp32's range in the sums (there the products of the
// parts are infinities of both signs; as sums are 2^32 times too large, from 7.9e28).  A workgroup that meets
// one computes its sums from the fp32 data with fp32 MFMAs instead (after its split sums; at once where a
// weight is the cause).  An infinite weight: conv3 on 8 maps of 37 x 49 524 us, conv2 on 8 of 59 x 79 282, conv1
// on 8 planes of 480 x 640 199, against 164, 128 and 88 us where all values split, and 51, 47 and 12 ms with one
// thread per pixel.
//
// Workgroup: 16 x 16 output pixels x 64 channels of one group, four waves of 64 channels x 64 pixels.
// LDS holds one halo of 16 input channels as three bf16 planes, and two buffers of three taps' weights,
// streamed by direct loads from the split copy.  The next chunk's halo is loaded into registers while
// a chunk computes and is split between two barriers at its end.  72 MFMAs lie between two barriers, so
// the two workgroups of a CU (77 KB of LDS at R = 5) cover each other's waits.  Bound by the matrix cores.
// Against fp32 MFMAs (32x32x2, one 16-bit-sized pipeline per CU): conv3 on 8 maps of 37 x 49 596 -> 151 us
// (170 TFLOP/s of fp32 work, 1.02 PFLOP/s of bf16 products), conv2 of a 480 x 640 image's 8-scale pyramid
// 624 -> 141 us; error against 64 bits 7.1e-7 -> 2.6e-7 of the 2-norm.
// ------------------------------------------------------------------------------------------------
// One fp32 MFMA: two k, offset lane / 32; the accumulator's layout is the 16-bit tile's.
__device__ inline f32x16 mma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// The larger of m and every |v|; NaN when any is NaN (two values per v_maximum3_f32).
__device__ inline float max_or_nan(float m, const f32x16& v) {
  auto larger = [](float p, float q) { return __builtin_elementwise_maximum(p, q); };
  float a = m, b = 0.f;
#pragma unroll
  for (int e = 0; e < 16; e += 4) {
    a = larger(larger(a, __builtin_fabsf(v[e])), __builtin_fabsf(v[e + 1]));
    b = larger(larger(b, __builtin_fabsf(v[e + 2])), __builtin_fabsf(v[e + 3]));
  }
  return larger(a, b);
}

template <int R>
struct SplitCfg {
  using Cf = ConvCfg<__bf16, R, 64, 2, 1616, 2>;
  static constexpr int BM = 64, NT = 256, NW = 4, TM = 2, TN = 2;
  static constexpr int TS = 3, NS = (R * R + TS - 1) / TS;  // taps per stage, stages per chunk
  static constexpr int HALO_E = Cf::HH * Cf::RS;            // elements of one of the three halo planes
  static constexpr int TAP_E = 3 * BM * 16;                 // elements of one tap's weights
  static constexpr int W_OFF = (3 * HALO_E + 511) / 512 * 512;
  static constexpr int LDS_E = W_OFF + 2 * TS * TAP_E;
  static constexpr int HALO_V = Cf::HH * Cf::HW * 4, HALO_PER = (HALO_V + NT - 1) / NT;  // 4 channels each
  static_assert(NW * 64 * 64 * 2 <= LDS_E, "the fp32 epilogue staging fits the stage buffers");
  static_assert((size_t)LDS_E * 2 <= 80 * 1024, "two workgroups per CU");
};

// ksplit > 1 (launches too small to fill the chip): the launch is ksplit copies of its base workgroups;
// copy ks runs the input-channel chunks [ks nchunks / ksplit, (ks + 1) nchunks / ksplit) and writes its
// raw sums (no bias, no ReLU) to part + ks part_slice at the output's element offsets;
// split_reduce_kernel then adds the copies in order.
// wsplit: per block of 64 output channels, chunk of 16 input channels and tap: [3][64][2 slots] of bf16,
// in the order of the LDS buffer.  w: the fp32 weights [M][R R][Cg] and special: whether any of them
// does not split.  wide: fp32 MFMAs only (maps whose tiles exceed 32-bit byte offsets).
template <int R, bool MULTI>
__global__ __launch_bounds__(256, 2) void conv_f32_kernel(
    const float* __restrict__ in, float* __restrict__ out, const __bf16* __restrict__ wsplit,
    const float* __restrict__ w, const uint32_t* __restrict__ special, const float* __restrict__ bias,
    KRuns runs, int C, int Cg, int M, int Mg, int mblocks, int ksplit, int base, float* __restrict__ part,
    int64_t part_slice, int wide) {
  using P = SplitCfg<R>;
  using Cf = typename P::Cf;
  using Op = Mfma<__bf16>;
  using frag = typename Op::frag;
  const bool exact = *special || wide;  // no split at all
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  constexpr int pad = (R - 1) / 2, TM = P::TM, TN = P::TN, RR = R * R;
  __shared__ __align__(1024) __bf16 s_mem[P::LDS_E];

  // XCD-aware order, as conv_s1_direct_kernel
  const int nb = gridDim.x, xcd = blockIdx.x % 8, per = nb / 8, rem = nb % 8;
  int bid = xcd * per + min(xcd, rem) + blockIdx.x / 8;
  const int ks = bid / base;
  bid -= ks * base;
  const KRun& rn = runs.r[run_of<MULTI>(runs, bid)];
  bid -= rn.first;
  const int H = rn.H, W = rn.W, tiles_x = rn.tiles_x, tiles_y = rn.tiles_y;
  const int mb = bid % mblocks;
  bid /= mblocks;
  const int tx = bid % tiles_x;
  bid /= tiles_x;
  const int ty = bid % tiles_y;
  const int plane = bid / tiles_y;
  const int mpg = Mg / P::BM;
  const int g = mb / mpg, m0 = (mb % mpg) * P::BM;  // group, first output channel within it
  const int oy0 = ty * Cf::TH, ox0 = tx * Cf::TW;
  const float* src = in + rn.in_off + plane * rn.in_stride + g * Cg;
  const int nchunks = Cg / 16;
  const int c_lo = ks * nchunks / ksplit, c_hi = (ks + 1) * nchunks / ksplit;

  const int tid = threadIdx.x, lane = tid & 63, wn = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  constexpr uint32_t OOB = 0x80000000u;

  // Halo loads: 4 channels of a pixel each, at byte offsets from the tile's first halo row in the map
  // (a tile's rows span less than 2^31 bytes, or `wide` is set).
  const int iy_first = max(oy0 - pad, 0);
  const float* row0 = src + (int64_t)iy_first * W * C;
  const int64_t span = (int64_t)(min(oy0 + Cf::TH + pad, H) - iy_first) * W * C - g * Cg;
  const __amdgpu_buffer_rsrc_t rsrc_in = uniform_rsrc(row0, (uint32_t)(span * sizeof(float)));
  uint32_t hoff[P::HALO_PER];
#pragma unroll
  for (int i = 0; i < P::HALO_PER; ++i) {
    const int e = tid + i * P::NT, v = e & 3, p = e >> 2;
    const int iy = oy0 - pad + p / Cf::HW, ix = ox0 - pad + p % Cf::HW;
    const bool ok = e < P::HALO_V && iy >= 0 && iy < H && ix >= 0 && ix < W;
    hoff[i] = ok ? (((uint32_t)(iy - iy_first) * (uint32_t)W + (uint32_t)ix) * (uint32_t)C + 4u * v) * 4u : OOB;
  }
  u32x4_t hreg[P::HALO_PER];
  auto load_halo = [&](int chunk) {
#pragma unroll
    for (int i = 0; i < P::HALO_PER; ++i)
      hreg[i] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc_in, hoff[i], chunk * 64, 0));
  };
  // Scales the loaded values; called where MFMAs are in flight.
  uint32_t top = 0;  // largest |2^16 x|, as bits
  auto scale_halo = [&] {
#pragma unroll
    for (int i = 0; i < P::HALO_PER; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float v = SPLIT_SCALE * __builtin_bit_cast(float, (uint32_t)hreg[i][q]);
        const uint32_t bits = __builtin_bit_cast(uint32_t, v);
        hreg[i][q] = bits;
        top = max(top, bits & 0x7fffffffu);
      }
  };
  auto store_halo = [&] {
    typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < P::HALO_PER; ++i) {
      const int e = tid + i * P::NT, v = e & 3, p = e >> 2;
      if (e < P::HALO_V) {
        bf4 h, m, l;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const Split3 sp = split3(__builtin_bit_cast(float, (uint32_t)hreg[i][q]));
          h[q] = sp.h, m[q] = sp.m, l[q] = sp.l;
        }
        __bf16* d = s_mem + Cf::halo_off(p / Cf::HW, p % Cf::HW, v >> 1) + 4 * (v & 1);
        *(bf4*)d = h;
        *(bf4*)(d + P::HALO_E) = m;
        *(bf4*)(d + 2 * P::HALO_E) = l;
      }
    }
  };
  // Weights of stage s (taps 3 s ..) of a chunk: whole 1 KB pieces, dealt to the waves in turn.
  const __bf16* wg = wsplit + (int64_t)(g * mpg + m0 / P::BM) * nchunks * RR * P::TAP_E;
  const __amdgpu_buffer_rsrc_t rsrc_w =
      uniform_rsrc(wg, (uint32_t)(nchunks * RR * P::TAP_E * (int)sizeof(__bf16)));
  const int wave_s = __builtin_amdgcn_readfirstlane(wn);
  const uint32_t lane16 = (uint32_t)lane * 16u;
  auto load_w = [&](int buf, int chunk, auto sc) {
    constexpr int S = decltype(sc)::value;
    constexpr int TAPS = RR - P::TS * S < P::TS ? RR - P::TS * S : P::TS, PIECES = TAPS * P::TAP_E / 512;
    const uint32_t from = (uint32_t)((chunk * RR + P::TS * S) * P::TAP_E) * 2u;
#pragma unroll
    for (int i = 0; i < (PIECES + P::NW - 1) / P::NW; ++i) {
      const int q = wave_s + P::NW * i;
      if (q < PIECES)
        lds_direct16(rsrc_w, s_mem + P::W_OFF + buf * (P::TS * P::TAP_E) + q * 512, lane16, from + q * 1024u);
    }
  };

  // Pixel layouts and skipped MFMA tiles at the map's edges as in conv_s1_direct_kernel.
  auto gtile = [&](int t) { return t * Cf::WN + wn; };
  const int cv = min(Cf::TW, W - ox0), rv = min(Cf::TH, H - oy0);
  const int n_rows = (rv + 1) / 2, n_cols = (cv + 1) / 2;
  const bool colpair = n_cols < n_rows;
  const int n_mt = colpair ? n_cols : n_rows;
  auto out_row = [&](int idx) { return colpair ? (idx & 15) : Cf::pix_row(idx); };
  auto out_col = [&](int idx) { return colpair ? 2 * (idx >> 5) + ((idx >> 4) & 1) : Cf::pix_col(idx); };
  int pix[TN];
  int tnv = 0;
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    const int idx = gtile(t) * 32 + l32;
    pix[t] = Cf::halo_off(out_row(idx), out_col(idx), half);
    tnv += gtile(t) < n_mt ? 1 : 0;
  }
  tnv = __builtin_amdgcn_readfirstlane(tnv);

  f32x16 big[TM][TN], small[TM][TN];  // sums of h h', and of the five small terms
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int t = 0; t < TN; ++t) big[a][t] = f32x16{}, small[a][t] = f32x16{};

  auto chunks = [&](auto tnv_c) {
    constexpr int TNV = decltype(tnv_c)::value;
    load_halo(c_lo);
    load_w(0, c_lo, std::integral_constant<int, 0>{});
    scale_halo();
    store_halo();
    wait_vmem();
    __syncthreads();
    int buf = 0;
    for (int chunk = c_lo; chunk < c_hi; ++chunk) {
      const bool next = chunk + 1 < c_hi;
      if (next) load_halo(chunk + 1);
      static_for<0, P::NS>([&](auto sc) {
        constexpr int S = decltype(sc)::value;
        if constexpr (S + 1 < P::NS)
          load_w(buf ^ 1, chunk, std::integral_constant<int, S + 1>{});
        else if (next)
          load_w(buf ^ 1, chunk + 1, std::integral_constant<int, 0>{});
        if (S + 1 == P::NS && next) scale_halo();  // loaded by the first stage's end
        if constexpr (TNV > 0) {
          const __bf16* ws = s_mem + P::W_OFF + buf * (P::TS * P::TAP_E);
          static_for<P::TS * S, (P::TS * (S + 1) < RR ? P::TS * (S + 1) : RR)>([&](auto tc) {
            constexpr int TAP = decltype(tc)::value, KY = TAP / R, KX = TAP % R;
            frag x[3][TNV], wf[3][TM];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
#pragma unroll
              for (int t = 0; t < TNV; ++t)
                x[k][t] = *(const frag*)(s_mem + pix[t] + k * P::HALO_E + KY * Cf::RS + KX * Cf::PS);
#pragma unroll
              for (int mt = 0; mt < TM; ++mt)
                wf[k][mt] = *(const frag*)(ws + (TAP - P::TS * S) * P::TAP_E + k * (P::BM * 16) +
                                           Cf::w_off(0, mt * 32 + l32, half));
            }
            auto term = [&](int kw, int kx, f32x16 (&acc)[TM][TN]) {
#pragma unroll
              for (int mt = 0; mt < TM; ++mt)
#pragma unroll
                for (int t = 0; t < TNV; ++t) acc[mt][t] = Op::mma(wf[kw][mt], x[kx][t], acc[mt][t]);
            };
            term(0, 0, big);
            term(2, 0, small);
            term(0, 2, small);
            term(1, 1, small);
            term(1, 0, small);
            term(0, 1, small);
          });
        }
        wait_vmem();
        if constexpr (S + 1 == P::NS) {
          if (next) {
            __syncthreads();  // every wave is done with this chunk's halo
            store_halo();
          }
        }
        __syncthreads();
        buf ^= 1;
      });
    }
  };
  if (!exact) switch (tnv) {
    case 2: chunks(std::integral_constant<int, 2>{}); break;
    case 1: chunks(std::integral_constant<int, 1>{}); break;
    default: chunks(std::integral_constant<int, 0>{}); break;
  }

  float peak = 0.f;  // largest |sum|, or NaN
#pragma unroll
  for (int mt = 0; mt < TM; ++mt)
#pragma unroll
    for (int t = 0; t < TN; ++t) {
#pragma unroll
      for (int e = 0; e < 16; ++e) big[mt][t][e] += small[mt][t][e];
      peak = max_or_nan(peak, big[mt][t]);
    }
  float unsplit = UNSPLIT;
  if (__syncthreads_or(top >= SPLIT_LIMIT || !(peak < INFINITY)) || exact) {
    unsplit = 1.f;
    // Some value or sum does not split: this workgroup's sums on the fp32 matrix cores (32x32x2), from the fp32
    // data with 64-bit addresses.  Per chunk the halo is staged as floats; each lane takes 8 channels of
    // its pixel (LDS) and of its output channel (weights, from L2), one per MFMA.
    typedef float v4 __attribute__((ext_vector_type(4)));
    float* s_halo = (float*)s_mem;
    constexpr int PSF = 20;  // floats per halo pixel: 16 channels, padded so that pixels fall on other banks
    static_assert(Cf::HH * Cf::HW * PSF * 2 <= P::LDS_E, "the fp32 halo fits the stage buffers");
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int t = 0; t < TN; ++t) big[mt][t] = f32x16{};
    const float* wl = w + (int64_t)(g * Mg + m0 + l32) * RR * Cg + 8 * half;
    for (int c0 = 16 * c_lo; c0 < 16 * c_hi; c0 += 16) {
      __syncthreads();
      for (int e = tid; e < P::HALO_V; e += P::NT) {
        const int v = e & 3, p = e >> 2;
        const int iy = oy0 - pad + p / Cf::HW, ix = ox0 - pad + p % Cf::HW;
        v4 x = v4{};
        if (iy >= 0 && iy < H && ix >= 0 && ix < W) {
          const float* q = src + ((int64_t)iy * W + ix) * C + c0 + 4 * v;
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = q[i];
        }
        *(v4*)(s_halo + p * PSF + 4 * v) = x;
      }
      __syncthreads();
#pragma unroll R
      for (int tap = 0; tap < RR; ++tap) {
        v4 xv[TN][2], wv[TM][2];
#pragma unroll
        for (int t = 0; t < TN; ++t) {
          const int idx = gtile(t) * 32 + l32;
          const float* q = s_halo + ((out_row(idx) + tap / R) * Cf::HW + out_col(idx) + tap % R) * PSF + 8 * half;
          xv[t][0] = *(const v4*)q, xv[t][1] = *(const v4*)(q + 4);
        }
#pragma unroll
        for (int mt = 0; mt < TM; ++mt) {
          const float* q = wl + ((int64_t)mt * 32 * RR + tap) * Cg + c0;
          wv[mt][0] = *(const v4*)q, wv[mt][1] = *(const v4*)(q + 4);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int mt = 0; mt < TM; ++mt)
#pragma unroll
            for (int t = 0; t < TN; ++t)
              big[mt][t] = mma_f32(wv[mt][i >> 2][i & 3], xv[t][i >> 2][i & 3], big[mt][t]);
      }
    }
    __syncthreads();
  }

  const bool raw = ksplit > 1;  // raw sums of this copy
  float* dst = (raw ? part + ks * part_slice : out) + rn.out_off + plane * rn.out_stride;
  const int mw = g * Mg + m0;  // first output channel
  // Epilogue: each wave stages its 64 pixels x 64 channels (256-byte rows, 16-byte chunks swizzled by
  // the pixel) and writes whole rows, 16 lanes per pixel.
  float* stg = (float*)s_mem + wn * (64 * 64);
#pragma unroll
  for (int mt = 0; mt < TM; ++mt)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const int p = t * 32 + l32, j = 8 * mt + 2 * q + half;
        f32x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = big[mt][t][4 * q + e] * unsplit;
        *(f32x4*)(stg + p * 64 + ((j ^ (p & 15)) * 4)) = r;
      }
  wave_lds_order();
  const int j = lane & 15;
  const f32x4 bv = *(const f32x4*)(bias + mw + 4 * j);
#pragma unroll
  for (int it = 0; it < 16; ++it) {
    const int p = it * 4 + (lane >> 4);
    f32x4 r = *(const f32x4*)(stg + p * 64 + ((j ^ (p & 15)) * 4));
    const int idx = gtile(p >> 5) * 32 + (p & 31);
    const int oy = oy0 + out_row(idx), ox = ox0 + out_col(idx);
    if (oy < H && ox < W) {
      float* d = dst + ((int64_t)oy * W + ox) * M + mw + 4 * j;
      if (raw) {
        *(f32x4*)d = r;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = fmaxf(r[e] + bv[e], 0.f);
        __builtin_nontemporal_store(r, (f32x4*)d);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// conv1 for fp32 storage, on bf16 matrix cores as conv_f32_kernel: three bf16 parts of each value, six
// products.  Workgroup: 16 x 16 output pixels x 96 channels, four waves of 96 channels x 64 pixels.
// Per input channel its 72 x 72 input halo sits in LDS as three bf16 planes and nine k-steps (12 x 12
// taps, zero weights at 11) run over it; the weights stream through two buffers of two k-steps.  The
// next channel's halo is loaded into registers meanwhile.  With 3 x 2 MFMA tiles per wave there is no
// room for two accumulators each at two waves per SIMD, so one takes all terms: 162 roundings of a sum,
// against 216 with fp32 MFMAs of two k.  Bound by the matrix cores, 10 % of it the zero taps; against
// fp32 MFMAs, conv1 of a 480 x 640 image's 8-scale pyramid 295 -> 95 us.
// ------------------------------------------------------------------------------------------------
struct Split1 {
  static constexpr int NT = 256, NW = 4, TM = 3, TN = 2, HR = 72, HS = 80;
  static constexpr int NK = K1 / 16, TS = 2, NS = (NK + TS - 1) / TS;  // k-steps per channel and stage, stages
  static constexpr int HALO_E = HR * HS, KSE = 3 * 96 * 16;            // elements of a plane, of a k-step
  static constexpr int W_OFF = (3 * HALO_E + 511) / 512 * 512;
  static constexpr int LDS_E = W_OFF + 2 * TS * KSE;
  static constexpr int HALO_V = HR * HR / 4, HALO_PER = (HALO_V + NT - 1) / NT;
  static_assert(NW * 32 * 96 * 2 <= LDS_E, "the fp32 epilogue staging (32 pixels per wave) fits");
  static_assert((size_t)LDS_E * 2 <= 80 * 1024, "two workgroups per CU");
};

// wsplit: per input channel and k-step [3][96][2 slots] of bf16, in LDS order; w: [96][3][144] fp32.
// ksplit > 1: as conv_f32_kernel's split, over the three input channels; wide: as conv_f32_kernel's.
template <bool MULTI>
__global__ __launch_bounds__(256, 2) void conv1_f32_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                           const __bf16* __restrict__ wsplit,
                                                           const float* __restrict__ w,
                                                           const uint32_t* __restrict__ special,
                                                           const float* __restrict__ bias, KRuns runs, int ksplit,
                                                           int base, float* __restrict__ part,
                                                           int64_t part_slice, int wide) {
  using P = Split1;
  using Op = Mfma<__bf16>;
  using frag = Op::frag;
  using hfrag = Op::half_frag;
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  constexpr int TM = P::TM, TN = P::TN;
  const bool exact = *special || wide;  // no split at all
  __shared__ __align__(1024) __bf16 s_mem[P::LDS_E];

  const int nb = gridDim.x, xcd = blockIdx.x % 8, per = nb / 8, rem = nb % 8;
  int bid = xcd * per + min(xcd, rem) + blockIdx.x / 8;
  const int copy = bid / base;  // split copy: input channels [3 copy / ksplit, 3 (copy + 1) / ksplit)
  bid -= copy * base;
  const KRun& rn = runs.r[run_of<MULTI>(runs, bid)];
  bid -= rn.first;
  const int H = rn.H, W = rn.W, pitch = rn.pitch, Ho = rn.Ho, Wo = rn.Wo, tiles_x = rn.tiles_x;
  const int tx = bid % tiles_x;
  bid /= tiles_x;
  const int ty = bid % rn.tiles_y, plane = bid / rn.tiles_y;
  const int oy0 = ty * 16, ox0 = tx * 16, iy0 = 4 * oy0, ix0 = 4 * ox0;
  const float* src = in + rn.in_off + plane * rn.in_stride;
  const int c_lo = copy * 3 / ksplit, c_hi = (copy + 1) * 3 / ksplit;

  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  constexpr uint32_t OOB = 0x80000000u;

  // Halo loads: four pixels of a row each, at byte offsets from the tile's first row (the rows of one
  // channel, less than 2^31 bytes, or `wide` is set; 16-byte loads at 4-byte alignment).  Columns from W on
  // are replaced by zeros.
  const int rows = min(P::HR, H - iy0);
  uint32_t hoff[P::HALO_PER];
#pragma unroll
  for (int i = 0; i < P::HALO_PER; ++i) {
    const int e = tid + i * P::NT, r = e / 18, x = ix0 + 4 * (e % 18);
    hoff[i] = e < P::HALO_V && r < rows && x < W ? ((uint32_t)r * (uint32_t)pitch + (uint32_t)x) * 4u : OOB;
  }
  u32x4_t hreg[P::HALO_PER];
  auto load_halo = [&](int c) {
    const __amdgpu_buffer_rsrc_t rsrc =
        uniform_rsrc(src + ((int64_t)c * H + iy0) * pitch, (uint32_t)((int64_t)rows * pitch * sizeof(float)));
#pragma unroll
    for (int i = 0; i < P::HALO_PER; ++i)
      hreg[i] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, hoff[i], 0, 0));
  };
  // Scales the loaded values and drops those past the row; called where MFMAs are in flight.
  uint32_t top = 0;  // largest |2^16 x|, as bits
  auto scale_halo = [&] {
#pragma unroll
    for (int i = 0; i < P::HALO_PER; ++i) {
      const int x = ix0 + 4 * ((tid + i * P::NT) % 18);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float v = SPLIT_SCALE * __builtin_bit_cast(float, (uint32_t)hreg[i][q]);
        const uint32_t bits = x + q < W ? __builtin_bit_cast(uint32_t, v) : 0u;
        hreg[i][q] = bits;
        top = max(top, bits & 0x7fffffffu);
      }
    }
  };
  auto store_halo = [&] {
    typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < P::HALO_PER; ++i) {
      const int e = tid + i * P::NT, r = e / 18, xc = 4 * (e % 18);
      if (e < P::HALO_V) {
        bf4 h, m, l;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const Split3 sp = split3(__builtin_bit_cast(float, (uint32_t)hreg[i][q]));
          h[q] = sp.h, m[q] = sp.m, l[q] = sp.l;
        }
        __bf16* d = s_mem + r * P::HS + xc;
        *(bf4*)d = h;
        *(bf4*)(d + P::HALO_E) = m;
        *(bf4*)(d + 2 * P::HALO_E) = l;
      }
    }
  };
  const __amdgpu_buffer_rsrc_t rsrc_w = uniform_rsrc(wsplit, (uint32_t)(3 * P::NK * P::KSE * (int)sizeof(__bf16)));
  const uint32_t lane16 = (uint32_t)lane * 16u;
  auto load_w = [&](int buf, int c, auto sc) {  // stage sc of channel c: k-steps TS sc ..
    constexpr int S = decltype(sc)::value;
    constexpr int STEPS = P::NK - P::TS * S < P::TS ? P::NK - P::TS * S : P::TS, PIECES = STEPS * P::KSE / 512;
    const uint32_t from = (uint32_t)((c * P::NK + P::TS * S) * P::KSE) * 2u;
#pragma unroll
    for (int i = 0; i < (PIECES + P::NW - 1) / P::NW; ++i) {
      const int q = wv + P::NW * i;
      if (q < PIECES)
        lds_direct16(rsrc_w, s_mem + P::W_OFF + buf * (P::TS * P::KSE) + q * 512, lane16, from + q * 1024u);
    }
  };

  // MFMA pixel tile t of wave wv: tile rows 2 (4 t + wv) and the next, 16 columns each
  auto gtile = [&](int t) { return t * P::NW + wv; };
  int lpix[TN];
  int tnv = 0;
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    const int idx = gtile(t) * 32 + l32;
    lpix[t] = (4 * (idx / 16) + 2 * half) * P::HS + 4 * (idx % 16);
    tnv += 2 * gtile(t) < Ho - oy0 ? 1 : 0;
  }
  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int t = 0; t < TN; ++t) acc[a][t] = f32x16{};

  auto channels = [&](auto tnv_c) {
    constexpr int TNV = decltype(tnv_c)::value;
    load_halo(c_lo);
    load_w(0, c_lo, std::integral_constant<int, 0>{});
    scale_halo();
    store_halo();
    wait_vmem();
    __syncthreads();
    int buf = 0;
    for (int c = c_lo; c < c_hi; ++c) {
      const bool next = c + 1 < c_hi;
      if (next) load_halo(c + 1);
      static_for<0, P::NS>([&](auto sc) {
        constexpr int S = decltype(sc)::value;
        if constexpr (S + 1 < P::NS)
          load_w(buf ^ 1, c, std::integral_constant<int, S + 1>{});
        else if (next)
          load_w(buf ^ 1, c + 1, std::integral_constant<int, 0>{});
        if (S + 1 == P::NS && next) scale_halo();  // loaded by the first stage's end
        if constexpr (TNV > 0) {
          const __bf16* ws = s_mem + P::W_OFF + buf * (P::TS * P::KSE);
          static_for<P::TS * S, (P::TS * (S + 1) < P::NK ? P::TS * (S + 1) : P::NK)>([&](auto jc) {
            constexpr int J = decltype(jc)::value, O = 4 * (J / 3) * P::HS + 4 * (J % 3);
            frag x[3][TNV], wf[3][TM];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
#pragma unroll
              for (int t = 0; t < TNV; ++t) {
                const __bf16* q = s_mem + lpix[t] + k * P::HALO_E + O;
                const hfrag lo = *(const hfrag*)q, hi = *(const hfrag*)(q + P::HS);
                x[k][t] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
              }
#pragma unroll
              for (int mt = 0; mt < TM; ++mt)
                wf[k][mt] = *(const frag*)(ws + (J - P::TS * S) * P::KSE + k * (96 * 16) + (mt * 32 + l32) * 16 +
                                           (half ^ ((l32 >> 4) & 1)) * 8);
            }
            auto term = [&](int kw, int kx) {
#pragma unroll
              for (int mt = 0; mt < TM; ++mt)
#pragma unroll
                for (int t = 0; t < TNV; ++t) acc[mt][t] = Op::mma(wf[kw][mt], x[kx][t], acc[mt][t]);
            };
            term(2, 0);
            term(0, 2);
            term(1, 1);
            term(1, 0);
            term(0, 1);
            term(0, 0);
          });
        }
        wait_vmem();
        if constexpr (S + 1 == P::NS) {
          if (next) {
            __syncthreads();  // every wave is done with this channel's halo
            store_halo();
          }
        }
        __syncthreads();
        buf ^= 1;
      });
    }
  };
  if (!exact) switch (tnv) {
    case 2: channels(std::integral_constant<int, 2>{}); break;
    case 1: channels(std::integral_constant<int, 1>{}); break;
    default: channels(std::integral_constant<int, 0>{}); break;
  }

  float peak = 0.f;  // largest |sum|, or NaN
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int t = 0; t < TN; ++t) peak = max_or_nan(peak, acc[a][t]);
  float unsplit = UNSPLIT;
  if (__syncthreads_or(top >= SPLIT_LIMIT || !(peak < INFINITY)) || exact) {
    unsplit = 1.f;
    // Some value or sum does not split: this workgroup's sums on the fp32 matrix cores, as conv_f32_kernel's.  The
    // zero-weight taps take zeros, whatever the plane holds there.
    typedef float v4 __attribute__((ext_vector_type(4)));
    float* s_halo = (float*)s_mem;
    constexpr int HSF = 76;  // floats per halo row
    static_assert(P::HR * HSF * 2 <= P::LDS_E, "the fp32 halo fits the stage buffers");
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int t = 0; t < TN; ++t) acc[a][t] = f32x16{};
    for (int c = c_lo; c < c_hi; ++c) {
      __syncthreads();
      for (int e = tid; e < P::HR * P::HR; e += P::NT) {
        const int r = e / P::HR, x = e % P::HR;
        s_halo[r * HSF + x] = iy0 + r < H && ix0 + x < W ? src[((int64_t)c * H + iy0 + r) * pitch + ix0 + x] : 0.f;
      }
      __syncthreads();
#pragma unroll 3
      for (int k = 0; k < P::NK; ++k) {  // rows 4 (k / 3) .. + 3, columns 4 (k % 3) .. + 3
        v4 xv[TN][2], wv[TM][2];
#pragma unroll
        for (int t = 0; t < TN; ++t) {
          const int idx = gtile(t) * 32 + l32;
          const float* q = s_halo + (4 * (idx / 16) + 4 * (k / 3) + 2 * half) * HSF + 4 * (idx % 16) + 4 * (k % 3);
          xv[t][0] = *(const v4*)q, xv[t][1] = *(const v4*)(q + HSF);
          if (k % 3 == 2) xv[t][0][3] = 0.f, xv[t][1][3] = 0.f;
          if (k / 3 == 2 && half) xv[t][1] = v4{};
        }
#pragma unroll
        for (int mt = 0; mt < TM; ++mt) {
          const float* q = w + ((mt * 32 + l32) * 3 + c) * K1 + 16 * k + 8 * half;
          wv[mt][0] = *(const v4*)q, wv[mt][1] = *(const v4*)(q + 4);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int mt = 0; mt < TM; ++mt)
#pragma unroll
            for (int t = 0; t < TN; ++t)
              acc[mt][t] = mma_f32(wv[mt][i >> 2][i & 3], xv[t][i >> 2][i & 3], acc[mt][t]);
      }
    }
    __syncthreads();
  }

  const bool raw = ksplit > 1;
  float* dst = (raw ? part + copy * part_slice : out) + rn.out_off + plane * rn.out_stride;
  // Epilogue: per MFMA pixel tile each wave stages 32 pixels x 96 channels (384-byte rows, 16-byte chunks
  // swizzled by the pixel) and writes whole rows, 24 lanes per pixel.
  float* stg = (float*)s_mem + wv * (32 * 96);
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    wave_lds_order();
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = 8 * mt + 2 * q + half;
        f32x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = acc[mt][t][4 * q + e] * unsplit;
        *(f32x4*)(stg + l32 * 96 + ((j ^ ((l32 >> 2) & 7)) * 4)) = r;
      }
    wave_lds_order();
#pragma unroll
    for (int it = 0; it < 12; ++it) {
      const int u = it * 64 + lane, p = u / 24, j = u % 24;
      f32x4 r = *(const f32x4*)(stg + p * 96 + ((j ^ ((p >> 2) & 7)) * 4));
      const int idx = gtile(t) * 32 + p, oy = oy0 + idx / 16, ox = ox0 + idx % 16;
      if (oy < Ho && ox < Wo) {
        float* d = dst + ((int64_t)oy * Wo + ox) * 96 + 4 * j;
        if (raw) {
          *(f32x4*)d = r;
        } else {
          const f32x4 bv = *(const f32x4*)(bias + 4 * j);
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = fmaxf(r[e] + bv[e], 0.f);
          __builtin_nontemporal_store(r, (f32x4*)d);
        }
      }
    }
  }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int OUT_CPOL = 2;  // cache policy of conv1's output stores: non-temporal
// conv1's MFMA pixel tiles per wave (Conv1R): 2, chosen by timing on the 96-plane batch (4, one wave per
// SIMD with 30 % fewer LDS bytes per MFMA, took 0.82-0.84 ms against 0.646: a lone wave does not hide
// its own LDS and load latency).
#ifndef DN_CONV1_PT
#define DN_CONV1_PT 2
#endif
// Wait until at most N (< 64) vector-memory accesses of this wave are outstanding.
template <int N>
__device__ inline void wait_vmem_upto() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// ------------------------------------------------------------------------------------------------
// conv1 for 16-bit storage with direct global->LDS loads (DIRECT: rows that start on 16 bytes), weights
// resident, one independent pipeline per wave.  A workgroup of 8 waves (one per CU, two waves per SIMD) loads
// all weights (75 KB) into LDS once, as 25 k-steps of 16 (the 363 taps of an output channel as 99 units of
// 4 taps: see pack_conv1_resident_kernel) x 96 channels x
// two 16-byte slots, the slots swapped for channels 16..31 of every 32-channel group, so that the 32
// lanes of a half-wave reading one k-step's 16 bytes of 32 channels hit distinct slots modulo 512
// bytes.  After that every wave is its own worker with no workgroup barrier: it walks wave tiles of 4
// x 16 output pixels x 96 channels, and per stage (one input channel of one tile) loads the tile's 24
// x 72 input halo (rows of nine 16-byte slots of plane data and one zero slot) into one of its two
// private LDS buffers while it computes from the other, reading k-step j + 1's fragments while k-step
// j's MFMAs run.  Stage c runs k-steps 0..7, 8..15 or 16..24; k-steps 8 and 16 hold units of two
// input channels, so they run first in their stage, from both buffers, before the next stage's halo
// load reuses the older one.  A wave that writes out a tile, or waits for a load, stalls only
// itself; the other wave on its SIMD keeps the MFMAs busy.  A tile's outputs leave through LDS, as
// whole 192-byte pixel rows.
// DIRECT = false, for rows at any alignment (pitches that are not multiples of 8, unaligned pointers,
// planes beyond 2^31 bytes): the halo is loaded into registers, 16 bytes at 2-byte alignment, and
// written to LDS where the direct loads are waited for, with the columns past the row's end zeroed.
// 64 planes of 227 x 227 in fp16: 22.3 us (0.60 PFLOP/s), against 82 for a kernel of 16 x 16 tiles per
// workgroup that loaded such rows value by value.
// ------------------------------------------------------------------------------------------------
// PT: 32-pixel MFMA tiles per wave (2: wave tiles of 4 x 16 pixels, 8 waves per workgroup, two per
// SIMD; 4: 8 x 16 pixels, 4 waves, one per SIMD, 30 % fewer LDS bytes per MFMA).
template <int PT>
struct Conv1R {
  static constexpr int NWV = PT == 2 ? 8 : 4;    // waves (workers) per workgroup
  static constexpr int TH = 2 * PT, TW = 16, HR = 4 * (TH - 1) + 12;  // wave tile; halo rows (k 0..11)
  static constexpr int EPI_STORES = PT * 6;      // 16-byte stores per lane in a tile's epilogue
  static constexpr int HSL = 10, HS = HSL * 8;   // halo row: slots, elements
  static constexpr int NH = (HR * HSL + 63) / 64;  // 1 KB pieces of a halo
  static constexpr int KSE = 96 * 16;            // elements of one k-step's weights
  static constexpr int WP = C1_KSTEPS * KSE / 512;  // 1 KB pieces of all weights
  static constexpr int DWL = (WP + NWV - 1) / NWV;  // weight pieces per wave (all weights, once)
  static constexpr int HALO_E = NH * 512;
  static constexpr int SROW = 104, SPX = 16;     // staging: elements per pixel row, pixels per round
  static constexpr int HALO_OFF = WP * 512, BIAS_OFF = HALO_OFF + NWV * 2 * HALO_E;
  static constexpr int LDS_E = BIAS_OFF + 2 * 96;  // the biases as 96 floats
  // unit u of a tile's k-steps: input channel, and its LDS offset (row r, columns 4 cb ..) in the halo
  __host__ __device__ static constexpr int uchan(int u) { return u < C1_UNITS ? u / 33 : 2; }
  __host__ __device__ static constexpr int uoff(int u) {
    return u < C1_UNITS ? ((u % 33) % 11) * HS + 4 * ((u % 33) / 11) : uoff(C1_UNITS - 1);
  }
  __host__ __device__ static constexpr int kchan(int j) { return j < 8 ? 0 : (j < 16 ? 1 : 2); }  // stage
};
static_assert(Conv1R<2>::WP * 512 == C1_KSTEPS * Conv1R<2>::KSE, "the weights are whole pieces");
static_assert(Conv1R<2>::uchan(4 * 8) == 0 && Conv1R<2>::uchan(4 * 8 + 1) == 1 &&
                  Conv1R<2>::uchan(4 * 16 + 1) == 1 && Conv1R<2>::uchan(4 * 16 + 2) == 2,
              "k-steps 8 and 16 are the only ones that span two input channels");
static_assert(Conv1R<2>::SPX * Conv1R<2>::SROW <= Conv1R<2>::HALO_E, "epilogue staging fits a halo buffer");
static_assert((size_t)Conv1R<2>::LDS_E * 2 <= 160 * 1024, "one workgroup's LDS fits the CU");
static_assert((size_t)Conv1R<4>::LDS_E * 2 <= 160 * 1024, "one workgroup's LDS fits the CU");

template <typename T, int PT, bool MULTI, bool DIRECT>
__global__ __launch_bounds__(64 * Conv1R<PT>::NWV, 1) void conv1_resident_kernel(
    const T* __restrict__ in, T* __restrict__ out, const T* __restrict__ wp,
    const float* __restrict__ bias, KRuns runs, int ntiles) {
  using P = Conv1R<PT>;
  constexpr int NWV = P::NWV;
  using Op = Mfma<T>;
  using frag = typename Op::frag;
  using hfrag = typename Op::half_frag;
  typedef T out4_t __attribute__((ext_vector_type(4)));
  typedef T vec8_t __attribute__((ext_vector_type(8)));
  __shared__ __align__(1024) T s_mem[P::LDS_E];
  float* s_bias = (float*)(s_mem + P::BIAS_OFF);
  if (threadIdx.x < 96) s_bias[threadIdx.x] = bias[threadIdx.x];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  constexpr uint32_t OOB = 0x80000000u;

  // Workers: workgroups are dispatched round-robin over the 8 XCDs, and rank r = x * (workgroups
  // per XCD) + i of XCD x has the workers NWV r .. NWV r + NWV - 1; worker w takes wave tiles w,
  // w + NWV G, ...: the workers in flight on one XCD hold neighbouring tiles, whose halos overlap in
  // its L2.  The tiles left after the last whole round go to the workgroups in turn, one wave of each
  // first (a wave alone on its SIMD takes little more than half the time of one of two), instead of
  // eight to a workgroup and none to the others: one image's 8550 tiles (4.2 rounds) 49 -> 44 us, the 2870 tiles
  // of a 480 x 640 image's pyramid 21 -> 16.5 us.
  const int G = gridDim.x, xcd = blockIdx.x % 8, per = G / 8, rem = G % 8;
  const int rank = xcd * per + min(xcd, rem) + blockIdx.x / 8;
  const int NWK = NWV * G, wk = NWV * rank + wave;
  const int rounds = ntiles / NWK, tail = rounds * NWK + wave * G + rank;
  const int ntile = rounds + (tail < ntiles ? 1 : 0);
  auto tile_at = [&](int j) { return j < rounds ? wk + j * NWK : tail; };

  // All weights, once: piece q of the k-step blob lands in LDS piece q.
  {
    const __amdgpu_buffer_rsrc_t rsrc_w = uniform_rsrc(wp, (uint32_t)(C1_KSTEPS * P::KSE * sizeof(T)));
#pragma unroll
    for (int i = 0; i < P::DWL; ++i) {
      const int q = wave + NWV * i;
      if (q < P::WP) lds_direct16(rsrc_w, s_mem + q * 512, (uint32_t)(q * 1024 + lane * 16));
    }
  }
  auto hbuf = [&](int b) { return s_mem + P::HALO_OFF + (2 * wave + b) * P::HALO_E; };
  // The current tile's input.  DIRECT: a descriptor of its plane and byte offsets of this lane's halo
  // slots in channel 0.  Otherwise: its plane, the tile's first row and column, and the loaded slots.
  uint32_t chan_bytes = 0;  // bytes of one input channel of the plane
  uint32_t hoff[DIRECT ? P::NH : 1];
  __amdgpu_buffer_rsrc_t rsrc_in;
  const T* tsrc = in;
  int tH = 0, tW = 0, tpitch = 0, ty0 = 0, tx0 = 0;
  vec8_t hreg[DIRECT ? 1 : P::NH];
  // Column W of the plane is the zero-weight tap (kx = 11) of the last output column when
  // (W - 11) % 4 == 0.  With W % 8 != 0 its 16-byte slot starts inside the row and is loaded, so when
  // rows are padded (pitch > W) the padding value would enter as 0 * x; zcol is then that column's
  // position in the tile's halo (else -1) and the halo copy of it is overwritten with zeros.
  int zcol = -1;
  auto set_tile = [&](int t) {  // wave tile t is the current tile
    const KRun& rn = runs.r[run_of<MULTI>(runs, t)];
    const int H = rn.H, W = rn.W, pitch = rn.pitch, tl = t - rn.first;
    const int tx = tl % rn.tiles_x, rr = tl / rn.tiles_x, ty = rr % rn.tiles_y, plane = rr / rn.tiles_y;
    const int iy0 = 4 * P::TH * ty, ix0 = 4 * P::TW * tx;
    if constexpr (DIRECT) {
      chan_bytes = (uint32_t)((int64_t)H * pitch * sizeof(T));
      rsrc_in = uniform_rsrc(in + rn.in_off + plane * rn.in_stride, 3 * chan_bytes);
      const bool zero_col_w = W % 8 != 0 && pitch > W;
      zcol = __builtin_amdgcn_readfirstlane(zero_col_w && W >= ix0 && W < ix0 + 72 ? W - ix0 : -1);
#pragma unroll
      for (int i = 0; i < P::NH; ++i) {
        const int q = i * 64 + lane;
        const int row = q / P::HSL, r = q % P::HSL;
        const int iy = iy0 + row, ix = ix0 + 8 * r;
        const bool ok = row < P::HR && r < 9 && iy < H && ix < W;
        hoff[i] = ok ? (uint32_t)(((int64_t)iy * pitch + ix) * sizeof(T)) : OOB;
      }
    } else {
      tsrc = in + rn.in_off + plane * rn.in_stride;
      tH = H, tW = W, tpitch = pitch, ty0 = iy0, tx0 = ix0;
    }
  };
  // load_halo: channel c of the current tile on its way to buffer b; land: it is there.
  auto load_halo = [&](int b, int c) {
    if constexpr (DIRECT) {
#pragma unroll
      for (int i = 0; i < P::NH; ++i) lds_direct16(rsrc_in, hbuf(b) + i * 512, hoff[i], c * chan_bytes);
    } else {
      typedef T vec8_any __attribute__((ext_vector_type(8), aligned(2)));
      const int64_t end = (int64_t)(3 - c) * tH * tpitch;  // elements from channel c's start to the plane's end
      const T* src = tsrc + (int64_t)c * tH * tpitch;
#pragma unroll
      for (int i = 0; i < P::NH; ++i) {
        const int q = i * 64 + lane;
        const int row = q / P::HSL, r = q % P::HSL;
        const int iy = ty0 + row, ix = tx0 + 8 * r;
        vec8_t v = vec8_t{};
        if (row < P::HR && r < 9 && iy < tH && ix < tW) {
          const int64_t at = (int64_t)iy * tpitch + ix;
          if (at + 8 <= end) {
            v = *(const vec8_any*)(src + at);
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (ix + e < tW) v[e] = src[at + e];
          }
        }
        hreg[i] = v;
      }
    }
  };
  auto zero_col = [&](int b) {  // after buffer b's direct loads have landed
    if (zcol >= 0) {
      wave_lds_order();
      if (lane < P::HR) hbuf(b)[lane * P::HS + zcol] = from_f32<T>(0.f);
      wave_lds_order();
    }
  };
  auto land = [&](int b) {
    if constexpr (DIRECT) {
      wait_vmem();
      zero_col(b);
    } else {
      wave_lds_order();
#pragma unroll
      for (int i = 0; i < P::NH; ++i) {
        const int q = i * 64 + lane, ix = tx0 + 8 * (q % P::HSL);
        vec8_t v = hreg[i];
        if (tx0 + 72 > tW) {  // what follows the row in a slot that crosses its end
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = ix + e < tW ? v[e] : from_f32<T>(0.f);
        }
        *(vec8_t*)(hbuf(b) + q * 8) = v;
      }
      wave_lds_order();
    }
  };

  int lpix[PT], lpix2[PT];
#pragma unroll
  for (int b = 0; b < PT; ++b) {
    const int idx = b * 32 + l32;
    lpix[b] = 4 * (idx / P::TW) * P::HS + 4 * (idx % P::TW);
    lpix2[b] = lpix[b] + 2 * half * P::HS;
  }
  const int lw = 16 * l32 + 8 * (half ^ ((l32 >> 4) & 1));
  // Lane bases: this lane's pixel (input row 4 prow, column 4 pcol) per pixel tile (lpix2: two rows
  // further in the upper half-wave), and its output channel's weight slot (half ^ swap).  k-step J:
  // lane half h reads units 4 J + 2 h (the fragment's low 8 bytes) and 4 J + 2 h + 1 (high); hp holds
  // the previous input channel's halo, hs the stage's.
  auto read = [&](auto jc, const T* hp, const T* hs, frag* x, frag* w) {
    constexpr int J = decltype(jc)::value, CS = P::kchan(J);
    hfrag hv[PT][2];
#pragma unroll
    for (int sx = 0; sx < 2; ++sx) {
      const int u0 = 4 * J + sx, u1 = 4 * J + 2 + sx;
      const bool p0 = P::uchan(u0) != CS, p1 = P::uchan(u1) != CS;
      const int o0 = P::uoff(u0), o1 = P::uoff(u1);
      if (!p0 && !p1 && o1 - o0 == 2 * P::HS) {  // the usual case: the upper half two rows down
#pragma unroll
        for (int b = 0; b < PT; ++b) hv[b][sx] = *(const hfrag*)(hs + lpix2[b] + o0);
      } else {
        const T* bh = half ? (p1 ? hp : hs) + o1 : (p0 ? hp : hs) + o0;
#pragma unroll
        for (int b = 0; b < PT; ++b) hv[b][sx] = *(const hfrag*)(bh + lpix[b]);
      }
    }
#pragma unroll
    for (int b = 0; b < PT; ++b) x[b] = __builtin_shufflevector(hv[b][0], hv[b][1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
    for (int mt = 0; mt < 3; ++mt) w[mt] = *(const frag*)(s_mem + J * P::KSE + 512 * mt + lw);
  };

  f32x16 acc[3][PT];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < PT; ++b) acc[a][b] = f32x16{};

  if (ntile > 0) {
    set_tile(tile_at(0));
    load_halo(0, 0);
  }
  wait_vmem();
  __syncthreads();  // weights and biases are in LDS; from here on each wave runs on its own
  if (ntile > 0) land(0);
  // One tile per iteration, its three stages in straight-line code.  Channel 0 and channel 2 of tile
  // j sit in buffer X = j & 1, channel 1 in the other, Y; a stage's load of the next stage's channel
  // goes to the buffer its own k-steps no longer read.
  for (int j = 0; j < ntile; ++j) {
    T* hx = hbuf(j & 1);
    T* hy = hbuf((j + 1) & 1);
    // k-steps J0 .. J1 - 1 of stage J0's channel (halo in hs, the previous channel's in hp); the next
    // stage's load (issue) follows k-step J0's MFMAs, which have then consumed any fragment of hp.
    auto ksteps = [&](auto j0c, auto j1c, const T* hp, const T* hs, auto&& issue) {
      constexpr int J0 = decltype(j0c)::value, J1 = decltype(j1c)::value;
      frag xr[2][PT], wr[2][3];
      read(std::integral_constant<int, J0>{}, hp, hs, xr[0], wr[0]);
      auto body = [&](auto jc) {
        constexpr int J = decltype(jc)::value, B = (J - J0) & 1;
        if constexpr (J + 1 < J1) read(std::integral_constant<int, J + 1>{}, hp, hs, xr[B ^ 1], wr[B ^ 1]);
        // raised wave priority while this k-step's MFMAs issue: the SIMD's other wave then issues
        // its LDS reads, loads and epilogue work in between rather than ahead of them
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int mt = 0; mt < 3; ++mt)
#pragma unroll
          for (int b = 0; b < PT; ++b) acc[mt][b] = Op::mma(wr[B][mt], xr[B][b], acc[mt][b]);
        __builtin_amdgcn_s_setprio(0);
        if constexpr (J == J0) {
          wave_lds_order();
          issue();
        }
      };
      static_for<J0, J1>(body);
    };
    // stage 0: channel 0 in X; channel 1 loads into Y
    ksteps(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{}, hy, hx,
           [&] { load_halo((j + 1) & 1, 1); });
    land((j + 1) & 1);
    // stage 1: channel 1 in Y (k-step 8 also reads channel 0 in X); channel 2 loads into X
    ksteps(std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{}, hx, hy, [&] { load_halo(j & 1, 2); });
    land(j & 1);
    // stage 2: channel 2 in X (k-step 16 also reads channel 1 in Y); the next tile's channel 0
    // loads into Y, the next tile's X
    ksteps(std::integral_constant<int, 16>{}, std::integral_constant<int, C1_KSTEPS>{}, hy, hx, [&] {
      if (j + 1 < ntile) {
        set_tile(tile_at(j + 1));
        load_halo((j + 1) & 1, 0);
      }
    });
    {
      // Epilogue of the tile: bias + ReLU; per 32-pixel MFMA tile, two rounds of 16 pixels staged
      // in X, just consumed (rows of 104 channels), read back as whole pixel rows and written with
      // 16-byte buffer stores that every lane issues (a pixel outside the map stores at an offset
      // past the plane, which the hardware drops): P::EPI_STORES stores per lane.
      T* hs = hx;
      const int t = tile_at(j);
      const KRun& rn = runs.r[run_of<MULTI>(runs, t)];
      const int Ho = rn.Ho, Wo = rn.Wo, tl = t - rn.first;
      const int tx = tl % rn.tiles_x, rr = tl / rn.tiles_x, ty = rr % rn.tiles_y, plane = rr / rn.tiles_y;
      T* dst = out + rn.out_off + plane * rn.out_stride;
      const __amdgpu_buffer_rsrc_t rsrc_out =
          uniform_rsrc(dst, DIRECT ? (uint32_t)((int64_t)Ho * Wo * 96 * sizeof(T)) : 0u);
#pragma unroll
      for (int b = 0; b < PT; ++b) {
        out4_t v[3][4];
#pragma unroll
        for (int mt = 0; mt < 3; ++mt)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 bv = *(const f32x4*)(s_bias + mt * 32 + 8 * q + 4 * half);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[mt][q][e] = from_f32<T>(fmaxf(acc[mt][b][4 * q + e] + bv[e], 0.f));
          }
#pragma unroll
        for (int ph = 0; ph < 2; ++ph) {
          wave_lds_order();
          if ((l32 >> 4) == ph) {
#pragma unroll
            for (int mt = 0; mt < 3; ++mt)
#pragma unroll
              for (int q = 0; q < 4; ++q)
                *(out4_t*)(hs + (l32 & 15) * P::SROW + mt * 32 + 8 * q + 4 * half) = v[mt][q];
          }
          wave_lds_order();
#pragma unroll
          for (int it = 0; it < 3; ++it) {  // 16 pixels x 12 chunks of 8 channels
            const int u = it * 64 + lane, p = u / 12, ch = u % 12;
            const vec8_t o = *(const vec8_t*)(hs + p * P::SROW + 8 * ch);
            const int idx = b * 32 + 16 * ph + p;
            const int oy = ty * P::TH + idx / P::TW, ox = tx * P::TW + idx % P::TW;
            const int64_t at = ((int64_t)oy * Wo + ox) * 96 + 8 * ch;
            if constexpr (DIRECT) {
              const uint32_t off = oy < Ho && ox < Wo ? (uint32_t)(at * sizeof(T)) : OOB;
              __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rsrc_out, off, 0, OUT_CPOL);
            } else if (oy < Ho && ox < Wo) {
              *(vec8_t*)(dst + at) = o;
            }
          }
        }
      }
      wave_lds_order();
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < PT; ++b) acc[a][b] = f32x16{};
      // Vector-memory operations retire in issue order: once no more than the epilogue's stores
      // are outstanding, the next tile's halo loads (issued before them) have landed in LDS.
      if constexpr (DIRECT) wait_vmem_upto<P::EPI_STORES>();
    }
    if (j + 1 < ntile) {
      if constexpr (DIRECT)
        zero_col((j + 1) & 1);
      else
        land((j + 1) & 1);
    }
  }
}

// Copies an fp32 launch of `blocks` workgroups splits its input channels over (at most max_copies): the ks
// minimising rounds(ks) / ks + 0.15 [ks > 1] + 0.02 ks blocks / slots, rounds(ks) = ceil(ks blocks / slots)
// with two workgroups resident per CU: the launch's rounds of shorter workgroups, plus the reduction
// and the partial sums' traffic, which grows with the copies and the launch's output.  Launches of at
// least one round do not split: a lone workgroup's whole K loop sets a small launch's time, not a large
// one's.  Timed at 1, 2, 3, 4, 6, 8, 12 and 16 copies: conv3 of two 13 x 13 and 9 x 9 maps (12
// workgroups) takes 92 us unsplit, 28 at 6, 23 at 16 (chosen: 16); conv4 of the 480 x 640 pyramid's eight
// maps (378 workgroups) 110 us unsplit, 100 at 4 (chosen), 134 at 8.
int split_copies(int64_t blocks, int max_copies) {
  const int64_t slots = 2LL * device_cu_count();
  int ks = 1;
  if (blocks < slots) {
    double best = 1.0;
    for (int k = 2; k <= max_copies; ++k) {
      const double cost = (double)((k * blocks + slots - 1) / slots) / k + 0.15 + 0.02 * k * (double)blocks / slots;
      if (cost < best) best = cost, ks = k;
    }
  }
  return ks;
}

// Elements of one partial copy of a launch over `runs`: its output extent, rounded to 64.
int64_t split_span(const MapRun* runs, int n_runs) {
  int64_t span = 0;
  for (int i = 0; i < n_runs; ++i) span = std::max(span, runs[i].out_off + runs[i].n * runs[i].out_stride);
  return (span + 63) / 64 * 64;
}

// Stride-1 layers, fp32 storage.  part / part_bytes: workspace for the partial sums of a split launch (may
// be NULL: no split); part_need non-NULL: only report the bytes this launch would use there (0 without
// a split).
template <int R>
int run_conv_f32(const float* in, float* out, const float* wp, const __bf16* wsplit, const uint32_t* special,
                 const float* bias, const MapRun* runs, int n_runs, int C, int G, int M, float* part,
                 size_t part_bytes, size_t* part_need, hipStream_t s) {
  using P = SplitCfg<R>;
  using Cf = typename P::Cf;
  const int Cg = C / G, Mg = M / G;
  if (Mg % P::BM || Cg % 16) return (int)hipErrorInvalidValue;  // whole channel blocks and chunks per group
  const int mblocks = M / P::BM;
  KRuns kr;
  const int64_t blocks = fill_kruns(runs, n_runs, kr, [&](KRun& k) {
    k.Ho = k.H, k.Wo = k.W;
    k.tiles_x = (k.W + Cf::TW - 1) / Cf::TW, k.tiles_y = (k.H + Cf::TH - 1) / Cf::TH;
    return (int64_t)k.tiles_x * k.tiles_y * mblocks;
  });
  if (blocks <= 0) return (int)hipErrorInvalidValue;
  // a tile's halo rows are addressed with 32-bit byte offsets (maps up to 77,000 columns wide)
  int wide = 0;
  for (int i = 0; i < n_runs; ++i)
    if ((int64_t)Cf::HH * runs[i].W * C * (int64_t)sizeof(float) >= 0x7fffffffLL) wide = 1;
  int ks = split_copies(blocks, Cg / 16);
  const int64_t span = split_span(runs, n_runs);  // elements of one partial copy
  const size_t need = ks > 1 ? (size_t)ks * (size_t)span * sizeof(float) : 0;
  if (part_need) {
    *part_need = need;
    return 0;
  }
  if (ks > 1 && (!part || part_bytes < need)) ks = 1;
  if (blocks * ks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
#define DN_F32_ARGS in, out, wsplit, wp, special, bias, kr, C, Cg, M, Mg, mblocks, ks, (int)blocks, part, span, \
                    wide
  if (n_runs == 1)
    conv_f32_kernel<R, false><<<(unsigned)(blocks * ks), P::NT, 0, s>>>(DN_F32_ARGS);
  else
    conv_f32_kernel<R, true><<<(unsigned)(blocks * ks), P::NT, 0, s>>>(DN_F32_ARGS);
#undef DN_F32_ARGS
  if (ks > 1) {
    KRuns rr;
    const int64_t rb = fill_kruns(runs, n_runs, rr, [&](KRun& k) {
      k.Ho = k.H, k.Wo = k.W;
      k.tiles_x = (int)(((int64_t)k.H * k.W * M / 4 + 255) / 256), k.tiles_y = 1;
      return (int64_t)k.tiles_x;
    });
    if (rb <= 0) return (int)hipErrorInvalidValue;
    split_reduce_kernel<<<(unsigned)rb, 256, 0, s>>>(part, span, ks, bias, out, rr, M);
  }
  return (int)hipGetLastError();
}

// Stride-1 layers, 16-bit storage.
template <typename T, int R, int BM, int TM, int OCC, int TS, int BMP = BM, int TN = 4>
int run_conv_s1(const T* in, T* out, const T* wstage, const float* bias, const MapRun* runs, int n_runs, int C,
                int G, int M, hipStream_t s) {
  using Cf = ConvCfg<T, R, BM, TM, TS, TN>;
  const int Cg = C / G, Mg = M / G;
  if (Mg % BM) return (int)hipErrorInvalidValue;  // whole channel blocks per group
  const int mblocks = G * (Mg / BM);
  KRuns kr;
  const int64_t blocks = fill_kruns(runs, n_runs, kr, [&](KRun& k) {
    k.Ho = k.H, k.Wo = k.W;
    k.tiles_x = (k.W + Cf::TW - 1) / Cf::TW, k.tiles_y = (k.H + Cf::TH - 1) / Cf::TH;
    return (int64_t)k.tiles_x * k.tiles_y * mblocks;
  });
  if (blocks <= 0) return (int)hipErrorInvalidValue;
  if (n_runs == 1)
    conv_s1_direct_kernel<T, R, BM, TM, OCC, TS, BMP, TN, false><<<(unsigned)blocks, Cf::NT, 0, s>>>(
        in, out, wstage, bias, kr, C, Cg, M, Mg, mblocks);
  else
    conv_s1_direct_kernel<T, R, BM, TM, OCC, TS, BMP, TN, true><<<(unsigned)blocks, Cf::NT, 0, s>>>(
        in, out, wstage, bias, kr, C, Cg, M, Mg, mblocks);
  return (int)hipGetLastError();
}

// Halo positions of PT pixels of a run's sequence, at most: the pixels, the pads of the row and plane
// ends between them, and the taps of the first and the last.
template <int R>
int64_t flat_positions(const MapRun& r, int64_t PT) {
  constexpr int64_t pad = (R - 1) / 2;
  const int64_t HW = (int64_t)r.H * r.W, rows = (PT - 2) / r.W + 1, planes = r.n > 1 ? (PT - 2) / HW + 1 : 0;
  return PT + rows * pad + planes * pad * (r.W + pad) + 2 * pad * (r.W + pad + 1) + 1;
}

// Whether conv_flat_kernel can take a launch's runs in workgroups of PT pixels with HS halo positions: the
// planes of a run follow one another, the padded positions count in 32 bits, and the halos fit.
template <int R, int PT, int HS>
bool flat_fits(const MapRun* runs, int n_runs, int C, int M) {
  constexpr int64_t pad = (R - 1) / 2;
  for (int i = 0; i < n_runs; ++i) {
    const MapRun& r = runs[i];
    const int64_t HW = (int64_t)r.H * r.W;
    if (r.n <= 0 || r.n > 0x3fffffffLL / ((r.H + pad) * (r.W + pad)) ||
        (r.n > 1 && (r.in_stride != HW * C || r.out_stride != HW * M)) ||
        flat_positions<R>(r, PT) > HS)
      return false;
  }
  return true;
}

// Whether TS tiles would compute at least a tenth more MFMA pixel tiles than the pixels as sequences (where
// both compute about the same, the 2-D tiles' smaller halos win: one image's 74 x 74 maps, conv3 58 us in
// tiles and 73 as sequences).
template <int TS>
bool flat_fills_better(const MapRun* runs, int n_runs) {
  constexpr int TH = TS / 100, TW = TS % 100;
  // MFMA pixel tiles of a tile holding rv x cv pixels of the map
  auto mfma_tiles = [](int rv, int cv) {
    const int64_t rows = (rv + 1) / 2 * (TW / 16), cols = (cv + 1) / 2;
    return TH == 16 ? std::min(rows, cols) : rows;
  };
  int64_t tiled = 0, flat = 0;
  for (int i = 0; i < n_runs; ++i) {
    const MapRun& r = runs[i];
    const int64_t ty = r.H / TH, tx = r.W / TW;  // whole tiles down and across; then what is left of each
    const int rv = r.H % TH, cv = r.W % TW;
    const int64_t one = ty * tx * mfma_tiles(TH, TW) + (cv ? ty * mfma_tiles(TH, cv) : 0) +
                        (rv ? tx * mfma_tiles(rv, TW) : 0) + (rv && cv ? mfma_tiles(rv, cv) : 0);
    tiled += one * r.n;
    flat += ((int64_t)r.n * r.H * r.W + 31) / 32;
  }
  return 10 * tiled >= 11 * flat;
}

// Workgroups of PT pixels x BM channels of a launch's runs as sequences.
int64_t flat_blocks(const MapRun* runs, int n_runs, int M, int PT, int BM) {
  int64_t tiles = 0;
  for (int i = 0; i < n_runs; ++i) tiles += ((int64_t)runs[i].n * runs[i].H * runs[i].W + PT - 1) / PT;
  return tiles * (M / BM);
}

template <typename T, int R, int BM, int TM, int OCC, int BMP, int WN, int TN, int HS, bool CHUNKED = false>
int run_conv_flat(const T* in, T* out, const T* wstage, const float* bias, const MapRun* runs, int n_runs, int C,
                  int G, int M, hipStream_t s) {
  constexpr int PT = 32 * TN * WN, NT = 64 * (BM / (32 * TM)) * WN;
  const int Cg = C / G, Mg = M / G;
  if (Mg % BM || n_runs <= 0 || n_runs > MAX_RUNS) return (int)hipErrorInvalidValue;
  const int mblocks = G * (Mg / BM);
  MapRun one[MAX_RUNS];  // each run as one sequence
  for (int i = 0; i < n_runs; ++i) one[i] = runs[i], one[i].n = 1;
  KRuns kr;
  int i = 0;
  const int64_t blocks = fill_kruns(one, n_runs, kr, [&](KRun& k) {
    k.Ho = k.H, k.Wo = k.W;
    k.tiles_y = runs[i++].n;
    k.tiles_x = (int)(((int64_t)k.tiles_y * k.H * k.W + PT - 1) / PT);
    return (int64_t)k.tiles_x * mblocks;
  });
  if (blocks <= 0) return (int)hipErrorInvalidValue;
  if (n_runs == 1)
    conv_flat_kernel<T, R, BM, TM, OCC, BMP, WN, TN, HS, CHUNKED, false><<<(unsigned)blocks, NT, 0, s>>>(
        in, out, wstage, bias, kr, C, Cg, M, Mg, mblocks);
  else
    conv_flat_kernel<T, R, BM, TM, OCC, BMP, WN, TN, HS, CHUNKED, true><<<(unsigned)blocks, NT, 0, s>>>(
        in, out, wstage, bias, kr, C, Cg, M, Mg, mblocks);
  return (int)hipGetLastError();
}

// Per layer: channel block BM, MFMA tiles per wave along channels TM, waves per SIMD requested, and
// the tile shape (100 rows + columns).  Chosen by timing each layer at the 96-plane batch shapes: two waves per
// SIMD matter most; conv3/conv5 run best at three waves per SIMD; conv4's 192 channels per group run
// best as one block of 3 x 32 channels per wave (7 LDS fragment reads per 12 MFMAs instead of 6 per 8).
// conv2 takes 16 x 32 tiles of 64 channels (four waves of 64 channels x 128 pixels): each stage's
// weight row then serves 512 pixels, which halves the weight loads per output against 16 x 16 tiles
// of 128 channels (2 % faster; with 128 channels, eight waves per workgroup, 10 % slower).  On the
// 74-wide maps of conv3..conv5, 32-wide tiles waste 20 % more MFMA work and were 25-30 % slower.
#ifndef DN_CONV2_CFG
#define DN_CONV2_CFG 64, 2, 2, 1632
#endif
#ifndef DN_CONV3_CFG
#define DN_CONV3_CFG 128, 2, 3, 1616
#endif
#ifndef DN_CONV5_CFG
#define DN_CONV5_CFG 128, 2, 3, 1616
#endif
#ifndef DN_CONV4_CFG
#define DN_CONV4_CFG 192, 3, 2, 1616
#endif

template <int BM_, int TM_, int OCC_, int TS_>
struct CfgBM {
  static constexpr int BM = BM_;
};
// Channel block of the direct-load kernel per layer (the stage-major weight copy is cut in these).
constexpr int L_BM[5] = {0, CfgBM<DN_CONV2_CFG>::BM, CfgBM<DN_CONV3_CFG>::BM, CfgBM<DN_CONV4_CFG>::BM,
                         CfgBM<DN_CONV5_CFG>::BM};

// A launch of the per-layer configuration with fewer workgroups than two rounds of the chip's
// resident slots (CUs x workgroups per CU) leaves CUs idle; such launches (one image's planes) take
// 64-channel blocks of 16 x 16 pixels instead, three to six times as many workgroups.
// Small launches: 64-channel blocks of 16 x 16 pixels whose waves own DN_SMALL_TN MFMA pixel tiles.
#ifndef DN_SMALL_TN
#define DN_SMALL_TN 2
#endif
#ifndef DN_SMALL_OCC
#define DN_SMALL_OCC 3
#endif
template <int BM_, int TM_, int OCC_, int TS_>
bool small_launch(const MapRun* runs, int n_runs, int M) {
  int64_t blocks = 0;
  for (int i = 0; i < n_runs; ++i)
    blocks += (int64_t)((runs[i].W + TS_ % 100 - 1) / (TS_ % 100)) *
              ((runs[i].H + TS_ / 100 - 1) / (TS_ / 100)) * (M / BM_) * runs[i].n;
  const int per_cu = OCC_ * 4 / (BM_ / (32 * TM_) * (TS_ / 100) * (TS_ % 100) / 128);
  return blocks < 2LL * device_cu_count() * (per_cu > 0 ? per_cu : 1);
}

template <typename T>
int conv_dispatch(int layer, const void* d_in, const MapRun* runs, int n_runs, const void* d_packed,
                  void* d_out, float* part, size_t part_bytes, size_t* part_need, const PackedLayout& L,
                  hipStream_t s) {
  const T* in = (const T*)d_in;
  T* out = (T*)d_out;
  const T* wp = (const T*)((const char*)d_packed + L.w_off[layer - 1]);  // fp32 only
  const T* ws = (const T*)((const char*)d_packed + L.s_off[layer - 1]);
  const float* bias = (const float*)((const char*)d_packed + L.b_off[layer - 1]);
  if (layer == 1) {
    if (part_need) *part_need = 0;
    KRuns kr;
    auto tiles16 = [](KRun& k) {  // tiles of 16 x 16 output pixels
      k.Ho = (k.H - 11) / 4 + 1, k.Wo = (k.W - 11) / 4 + 1;
      k.tiles_x = (k.Wo + 15) / 16, k.tiles_y = (k.Ho + 15) / 16;
      return (int64_t)k.tiles_x * k.tiles_y;
    };
    if constexpr (std::is_same<T, float>::value) {
      const int64_t blocks = fill_kruns(runs, n_runs, kr, tiles16);
      if (blocks <= 0) return (int)hipErrorInvalidValue;
      // launches too small to fill the chip split the three input channels (as conv2-5 do)
      int ks = split_copies(blocks, 3);
      const int64_t span = split_span(runs, n_runs);
      const size_t need = ks > 1 ? (size_t)ks * (size_t)span * sizeof(float) : 0;
      if (part_need) {
        *part_need = need;
        return 0;
      }
      if (ks > 1 && (!part || part_bytes < need)) ks = 1;
      const __bf16* wsplit = (const __bf16*)ws;
      const uint32_t* special = (const uint32_t*)((const char*)d_packed + L.special_off);
      // a tile's halo rows are addressed with 32-bit byte offsets (rows up to 7.4 million values apart)
      int wide = 0;
      for (int i = 0; i < n_runs; ++i)
        if ((int64_t)Split1::HR * std::max(runs[i].pitch, runs[i].W) * 4 >= 0x7fffffffLL) wide = 1;
      if (n_runs == 1)
        conv1_f32_kernel<false><<<(unsigned)(blocks * ks), 256, 0, s>>>(in, out, wsplit, wp, special, bias, kr, ks,
                                                                         (int)blocks, part, span, wide);
      else
        conv1_f32_kernel<true><<<(unsigned)(blocks * ks), 256, 0, s>>>(in, out, wsplit, wp, special, bias, kr, ks,
                                                                        (int)blocks, part, span, wide);
      if (ks > 1) {
        KRuns rr;
        const int64_t rb = fill_kruns(runs, n_runs, rr, [](KRun& k) {
          k.Ho = (k.H - 11) / 4 + 1, k.Wo = (k.W - 11) / 4 + 1;
          k.tiles_x = (int)(((int64_t)k.Ho * k.Wo * 96 / 4 + 255) / 256), k.tiles_y = 1;
          return (int64_t)k.tiles_x;
        });
        if (rb <= 0) return (int)hipErrorInvalidValue;
        split_reduce_kernel<<<(unsigned)rb, 256, 0, s>>>(part, span, ks, bias, (float*)out, rr, 96);
      }
    } else {
      if (part_need) return 0;
      // Direct loads take 16-byte slots of plane rows at 32-bit byte offsets within one plane.
      bool direct = ((uintptr_t)in & 15) == 0;
      for (int i = 0; i < n_runs; ++i) {
        const MapRun& r = runs[i];
        const int64_t Ho = (r.H - 11) / 4 + 1, Wo = (r.W - 11) / 4 + 1;
        const int64_t pitch = r.pitch > 0 ? r.pitch : r.W;
        direct = direct && pitch % 8 == 0 && r.in_stride % 8 == 0 && r.in_off % 8 == 0 &&
                 3 * r.H * pitch * (int64_t)sizeof(T) < 0x7fffffffLL &&
                 Ho * Wo * 96 * (int64_t)sizeof(T) < 0x7fffffffLL;
      }
      // wave tiles of 4 x 16 output pixels, 8 workers per workgroup, one workgroup per CU
      using R1 = Conv1R<DN_CONV1_PT>;
      const int64_t wtiles = fill_kruns(runs, n_runs, kr, [](KRun& k) {
        k.Ho = (k.H - 11) / 4 + 1, k.Wo = (k.W - 11) / 4 + 1;
        k.tiles_x = (k.Wo + R1::TW - 1) / R1::TW, k.tiles_y = (k.Ho + R1::TH - 1) / R1::TH;
        return (int64_t)k.tiles_x * k.tiles_y;
      });
      if (wtiles <= 0) return (int)hipErrorInvalidValue;
      const int grid = (int)std::min<int64_t>(wtiles, device_cu_count());
      auto go = [&](auto multi, auto dir) {
        conv1_resident_kernel<T, DN_CONV1_PT, decltype(multi)::value, decltype(dir)::value>
            <<<grid, 64 * R1::NWV, 0, s>>>(in, out, ws, bias, kr, (int)wtiles);
      };
      if (direct)
        n_runs == 1 ? go(std::false_type{}, std::true_type{}) : go(std::true_type{}, std::true_type{});
      else
        n_runs == 1 ? go(std::false_type{}, std::false_type{}) : go(std::true_type{}, std::false_type{});
    }
    return (int)hipGetLastError();
  }
  const int li = layer - 1;
  if constexpr (std::is_same<T, float>::value) {
    const __bf16* wsplit = (const __bf16*)((const char*)d_packed + L.s_off[li]);
    const uint32_t* special = (const uint32_t*)((const char*)d_packed + L.special_off) + li;
#define DN_RUN_ARGS \
  in, out, wp, wsplit, special, bias, runs, n_runs, L_C[li], L_G[li], L_M[li], part, part_bytes, part_need, s
    return layer == 2 ? run_conv_f32<5>(DN_RUN_ARGS) : run_conv_f32<3>(DN_RUN_ARGS);
#undef DN_RUN_ARGS
  } else {
    if (part_need) {
      *part_need = 0;
      return 0;
    }
    // The 16-bit kernels address one plane with 32-bit byte offsets.  Refused first: the counts below are
    // then of maps below 2^31 bytes.
    const int64_t most = 0x7ffffffeLL / (L_C[li] * (int64_t)sizeof(T));  // pixels
    for (int i = 0; i < n_runs; ++i)
      if ((int64_t)runs[i].H * runs[i].W > most) return (int)hipErrorInvalidValue;
#define DN_RUN_ARGS in, out, ws, bias, runs, n_runs, L_C[li], L_G[li], L_M[li], s
#define DN_SMALL_CFG(l) 3, 64, 2, DN_SMALL_OCC, 1616, L_BM[l], DN_SMALL_TN
#define DN_FLAT_ARGS runs, n_runs, L_C[li], L_M[li]
    // Maps that fill their tiles badly go as sequences where the launch keeps the chip busy that way (2000,
    // 350 and 100 windows' 13 x 13 maps: conv3 566 -> 453, 112 -> 91 and 37 -> 32 us; 200 windows' 27 x 27
    // maps: conv2 85 -> 79 us).  With fewer workgroups than the limits the tiles' larger number wins (100
    // windows: conv5 25 us as sequences, 22 in tiles; 60 windows: conv2 30 against 27).
    const int64_t cus = device_cu_count();
    const bool fills = layer == 2 ? flat_fills_better<1632>(runs, n_runs) : flat_fills_better<1616>(runs, n_runs);
    switch (layer) {
      case 2:
        if (fills && flat_fits<5, 512, 832>(DN_FLAT_ARGS) && flat_blocks(runs, n_runs, 256, 512, 64) >= 4 * cus)
          return run_conv_flat<T, 5, 64, 2, 2, L_BM[1], 4, 4, 832>(DN_RUN_ARGS);
        return run_conv_s1<T, 5, DN_CONV2_CFG>(DN_RUN_ARGS);
      // Layers 3 to 5: launches of at most two small workgroups (128 pixels x 64 channels, waves of 32
      // pixels, whole chunks per stage) per CU take those, which spread the pixels evenly over the
      // CUs: the eight maps of a 480 x 640 image's pyramid (49 x 65 .. 15 x 20) 30 -> 25, 25 -> 20 and 19.5 ->
      // 17.5 us, 20 windows' maps 23 -> 13, 18 -> 11 and 18 -> 10 us against 16 x 16 tiles.
#define DN_LAYER3(l, cfg, ...)                                                                              \
  if (flat_blocks(runs, n_runs, L_M[li], 128, 64) <= 2 * cus && flat_fits<3, 128, 320>(DN_FLAT_ARGS))       \
    return run_conv_flat<T, 3, 64, 2, 2, L_BM[l], 4, 1, 320, true>(DN_RUN_ARGS);                            \
  if (fills && flat_fits<3, 256, 384>(DN_FLAT_ARGS)) {                                                      \
    if (!small_launch<cfg>(runs, n_runs, L_M[li]))                                                          \
      return run_conv_flat<T, 3, __VA_ARGS__, L_BM[l], 2, 4, 384>(DN_RUN_ARGS);                             \
    if (2 * flat_blocks(runs, n_runs, L_M[li], 256, 64) >= 3 * cus)                                         \
      return run_conv_flat<T, 3, 64, 2, 3, L_BM[l], 4, 2, 384>(DN_RUN_ARGS);                                \
  }                                                                                                         \
  if (small_launch<cfg>(runs, n_runs, L_M[li])) return run_conv_s1<T, DN_SMALL_CFG(l)>(DN_RUN_ARGS);        \
  return run_conv_s1<T, 3, cfg>(DN_RUN_ARGS);
      case 3:
        DN_LAYER3(2, DN_CONV3_CFG, 128, 2, 3)
      case 4:
        DN_LAYER3(3, DN_CONV4_CFG, 192, 3, 2)
      case 5:
        DN_LAYER3(4, DN_CONV5_CFG, 128, 2, 3)
#undef DN_LAYER3
    }
#undef DN_FLAT_ARGS
#undef DN_SMALL_CFG
#undef DN_RUN_ARGS
    return (int)hipErrorInvalidValue;
  }
}

}  // namespace

PackedLayout packed_layout(dn_dtype dt) {
  PackedLayout L{};
  size_t off = 0;
  for (int l = 0; l < 5 && dt == DN_F32; ++l) {
    L.w_off[l] = off;
    const size_t n = l == 0 ? (size_t)96 * 3 * K1
                            : (size_t)L_M[l] * (L_C[l] / L_G[l]) * L_R[l] * L_R[l];
    off = align256(off + n * sizeof(float));
  }
  for (int l = 0; l < 5; ++l) {
    L.b_off[l] = off;
    off = align256(off + (size_t)L_M[l] * 4);
  }
  for (int l = 0; l < 5; ++l) {
    L.s_off[l] = off;
    const size_t n = l == 0 ? (size_t)(dt == DN_F32 ? 3 * K1 : C1_KSTEPS * 16) * 96
                            : (size_t)L_M[l] * (L_C[l] / L_G[l]) * L_R[l] * L_R[l];
    off = align256(off + n * (dt == DN_F32 ? 3 * 2 : dtype_size(dt)));
  }
  if (dt == DN_F32) {
    L.special_off = off;
    off = align256(off + 5 * sizeof(uint32_t));
  }
  L.total = off;
  return L;
}

int launch_pack_weights(const float* const* d_w, const float* const* d_b, dn_dtype dt, void* d_packed,
                        void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const PackedLayout L = packed_layout(dt);
  char* base = (char*)d_packed;
  uint32_t* special = (uint32_t*)(base + L.special_off);
  if (dt == DN_F32) clear_words_kernel<<<1, 64, 0, s>>>(special, 5);
  for (int l = 0; l < 5; ++l) {
    void* wd = base + L.w_off[l];
    void* sd = base + L.s_off[l];
    if (l == 0) {
      const int n = 96 * 3 * K1, nr = C1_KSTEPS * 96 * 16;
      if (dt == DN_F32) {
        pack_conv1_kernel<<<(n + 255) / 256, 256, 0, s>>>(d_w[0], (float*)wd);
        pack_split1_kernel<<<(n + 255) / 256, 256, 0, s>>>(d_w[0], (__bf16*)sd, special);
      }
      if (dt == DN_F16) pack_conv1_resident_kernel<_Float16><<<(nr + 255) / 256, 256, 0, s>>>(d_w[0], (_Float16*)sd);
      if (dt == DN_BF16) pack_conv1_resident_kernel<__bf16><<<(nr + 255) / 256, 256, 0, s>>>(d_w[0], (__bf16*)sd);
    } else {
      const int Cg = L_C[l] / L_G[l], Mg = L_M[l] / L_G[l], R = L_R[l];
      const int64_t n = (int64_t)L_M[l] * Cg * R * R;
      const unsigned nb = (unsigned)((n + 255) / 256);
      if (dt == DN_F32) {
        pack_conv_kernel<<<nb, 256, 0, s>>>(d_w[l], (float*)wd, L_M[l], Cg, R * R);
        pack_split_kernel<<<nb, 256, 0, s>>>(d_w[l], (__bf16*)sd, special + l, Mg, Cg, R * R, n);
      }
      if (dt == DN_F16) pack_stage_kernel<_Float16><<<nb, 256, 0, s>>>(d_w[l], (_Float16*)sd, Mg, Cg, R, L_BM[l], n);
      if (dt == DN_BF16) pack_stage_kernel<__bf16><<<nb, 256, 0, s>>>(d_w[l], (__bf16*)sd, Mg, Cg, R, L_BM[l], n);
    }
    copy_f32_kernel<<<(L_M[l] + 255) / 256, 256, 0, s>>>(d_b[l], (float*)(base + L.b_off[l]), L_M[l]);
  }
  return (int)hipGetLastError();
}

// One launch per MAX_RUNS runs (the partial-sum workspace is reused by each in turn), or with
// part_need: the largest workspace any of them would use.
static int conv_part_bytes_or_launch(int layer, const void* d_in, const MapRun* runs, int32_t n_runs,
                                     dn_dtype dt, const void* d_packed, void* d_out, void* d_part,
                                     size_t part_bytes, size_t* part_need, void* stream) {
  const PackedLayout L = packed_layout(dt);
  hipStream_t s = (hipStream_t)stream;
  if (layer < 1 || layer > 5 || n_runs <= 0) return (int)hipErrorInvalidValue;
  if (part_need) *part_need = 0;
  float* part = (float*)d_part;
  for (int i0 = 0; i0 < n_runs; i0 += MAX_RUNS) {
    const int nr = std::min(MAX_RUNS, n_runs - i0);
    size_t need = 0;
    size_t* q = part_need ? &need : nullptr;
    int st = (int)hipErrorInvalidValue;
    switch (dt) {
      case DN_F32:
        st = conv_dispatch<float>(layer, d_in, runs + i0, nr, d_packed, d_out, part, part_bytes, q, L, s);
        break;
      case DN_F16:
        st = conv_dispatch<_Float16>(layer, d_in, runs + i0, nr, d_packed, d_out, part, part_bytes, q, L, s);
        break;
      case DN_BF16:
        st = conv_dispatch<__bf16>(layer, d_in, runs + i0, nr, d_packed, d_out, part, part_bytes, q, L, s);
        break;
    }
    if (st) return st;
    if (part_need) *part_need = std::max(*part_need, need);
  }
  return 0;
}

int launch_conv(int layer, const void* d_in, const MapRun* runs, int32_t n_runs, dn_dtype dt,
                const void* d_packed, void* d_out, void* d_part, size_t part_bytes, void* stream) {
  return conv_part_bytes_or_launch(layer, d_in, runs, n_runs, dt, d_packed, d_out, d_part, part_bytes,
                                   nullptr, stream);
}

size_t conv_part_bytes(int layer, const MapRun* runs, int32_t n_runs, dn_dtype dt) {
  size_t need = 0;
  if (conv_part_bytes_or_launch(layer, nullptr, runs, n_runs, dt, nullptr, nullptr, nullptr, 0, &need,
                                nullptr))
    return 0;
  return need;
}

}  // namespace dn
