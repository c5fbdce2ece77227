// U-Net surrogate kernels for gfx950: implicit-GEMM convolutions on the BF16
// matrix cores (v_mfma_f32_32x32x16_bf16, FP32 accumulation), pooling,
// transposed convolution, the sigmoid head with a masked cross-entropy loss,
// and Adam.  C ABI in include/unet.h.
//
// MFMA operand layout (one wave, 32x32 output tile, K = 16 per instruction):
//   A fragment, lane l: A[row = l % 32][k = 8 * (l / 32) + j], j = 0..7
//   B fragment, lane l: B[k = 8 * (l / 32) + j][col = l % 32]
//   C, lane l, register r: C[row = 8 * (r / 4) + 4 * (l / 32) + r % 4][col = l % 32]
#include <hip/hip_runtime.h>

#include <mutex>
#include <stdint.h>

#include "../../include/unet.h"

namespace unet {

typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef float floatx16 __attribute__((__vector_size__(16 * sizeof(float))));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f2bf(float v) {
  uint32_t u = __float_as_uint(v);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ bf16x8 load8(const uint16_t *p) {
  const uint4 v = *reinterpret_cast<const uint4 *>(p);
  return __builtin_bit_cast(bf16x8, v);
}
// Eight channels at an address that need not be a multiple of 16 bytes (gfx950 reads and
// writes such vectors in one instruction too; the type says that they may come).
__device__ __forceinline__ uint4 load_any16(const uint16_t *p) {
  uint4 v;
  __builtin_memcpy(&v, p, sizeof v);
  return v;
}
__device__ __forceinline__ void store_any16(uint16_t *p, const uint4 &v) { __builtin_memcpy(p, &v, sizeof v); }
__device__ __forceinline__ bf16x8 zero8() { return __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0)); }
__device__ __forceinline__ bf16x8 pack8(const uint16_t (&v)[8]) {
  uint4 u;
  u.x = v[0] | ((uint32_t)v[1] << 16);
  u.y = v[2] | ((uint32_t)v[3] << 16);
  u.z = v[4] | ((uint32_t)v[5] << 16);
  u.w = v[6] | ((uint32_t)v[7] << 16);
  return __builtin_bit_cast(bf16x8, u);
}

// Buffer loads: a wave-uniform base, a byte offset per lane, and zeros from
// offsets beyond the buffer.  Loads masked this way are issued by every lane on
// every path, so the compiler can wait for the oldest of several in flight.
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
constexpr uint32_t kWholeBuffer = 0x80000000u;  // bytes reachable from a base
constexpr uint32_t kOutside = 0xc0000000u;      // offset of a masked lane (a scalar offset keeps it outside)
// Buffer loads take multiples of four bytes; the kernels that load by plain addresses
// serve other operands.
static bool dword_aligned(const uint16_t *a, const uint16_t *b) {
  return (reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) % 4 == 0;
}
__device__ __forceinline__ uint4 buffer_load16(const uint16_t *base, uint32_t bytes, uint32_t offset) {
  // the caller's base is wave-uniform: say so, for a descriptor in scalar registers
  const uint64_t v = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  uint16_t *const p = reinterpret_cast<uint16_t *>(((uint64_t)hi << 32) | lo);
  auto r = __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00027000);
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)offset, 0, 0));
}

__device__ __forceinline__ floatx16 mfma(bf16x8 a, bf16x8 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int c_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// ---------------------------------------------------------------------------
// one MFMA, for checking the operand layout: C(32x32) = A(32x16) B(16x32),
// row-major, A/B BF16, C FP32
// ---------------------------------------------------------------------------
__global__ void mfma_probe_kernel(const uint16_t *A, const uint16_t *B, float *C) {
  const int l = threadIdx.x;
  uint16_t a[8], b[8];
  for (int j = 0; j < 8; ++j) {
    a[j] = A[(l % 32) * 16 + 8 * (l / 32) + j];
    b[j] = B[(8 * (l / 32) + j) * 32 + (l % 32)];
  }
  floatx16 acc = {};
  acc = mfma(pack8(a), pack8(b), acc);
  for (int r = 0; r < 16; ++r) C[c_row(r, l) * 32 + (l % 32)] = acc[r];
}

// ---------------------------------------------------------------------------
// Implicit-GEMM forward: C[p][co] = sum_k A(p, k) B(k, co).  Block = 4 waves,
// 64 x 64 output tile (2 x 2 waves of 32 x 32).
//   MODE 0, 3x3 convolution:  k = (tap, ci), A = x[p + off(tap)][ci] (zero
//          outside), B = w[co][tap][ci]; output at p.
//   MODE 1, transposed 2x2 convolution, tap = blockIdx.z: k = ci,
//          A = x[p][ci], B = w[co][tap][ci]; output at 2p + tap (grid 2h x 2w).
//   MODE 2, data gradient of the transposed convolution: k = (tap, co'),
//          A = dy[2p + tap][co'], B = wt[ci][tap][co'] (here the output
//          channel is ci, the reduction channel co').
// K chunks of 8 never straddle a tap because channel counts are multiples of 8.
// ---------------------------------------------------------------------------
struct GemmArgs {
  const uint16_t *x;  // A source
  int n, h, w;        // A-source grid for MODE 0/1 (= output grid for MODE 0); input grid for MODE 2
  int kc;             // reduction channels (cin for MODE 0/1, cout' for MODE 2)
  int x_cs, x_co;
  const uint16_t *wgt;
  const float *bias;
  int nout;           // output channels
  uint16_t *y;
  int y_cs, y_co;
  int relu;
  // data gradients: zero where this activation (of the output's grid and channels,
  // a ReLU's output) is not positive; NULL for none
  const uint16_t *act;
  int act_cs, act_co;
};

// Wave tile TM x TN MFMA tiles (32 x 32 each): per K step a lane loads TM A
// fragments and TN B fragments for TM * TN products.  The four waves of a
// block are stacked along the pixels: block tile (128 TM) x (32 TN).
template <int MODE, int TM, int TN>
__global__ __launch_bounds__(256) void igemm_fwd(GemmArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t P = (int64_t)a.n * a.h * a.w;  // rows of A (pixels of the A grid)
  const int64_t pix0 = ((int64_t)blockIdx.x * 4 + wave) * (32 * TM);
  const int col0 = blockIdx.y * (32 * TN);
  const int tap_z = MODE == 1 ? (int)blockIdx.z : 0;
  const int half = lane >> 5;
  const int ntap = MODE == 0 ? 9 : (MODE == 2 ? 4 : 1);
  const int wtap = MODE == 1 ? 4 : ntap;  // taps per weight row
  const int K = ntap * a.kc;
  int pn[TM], py[TM], px[TM];
  bool prow[TM];
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int64_t pix = pix0 + 32 * t + (lane & 31);
    prow[t] = pix < P;
    pn[t] = py[t] = px[t] = 0;
    if (prow[t]) {
      pn[t] = (int)(pix / ((int64_t)a.h * a.w));
      const int r = (int)(pix - (int64_t)pn[t] * a.h * a.w);
      py[t] = r / a.w;
      px[t] = r - py[t] * a.w;
    }
  }
  floatx16 acc[TM][TN];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int u = 0; u < TN; ++u) acc[t][u] = floatx16{};
  for (int k0 = 0; k0 < K; k0 += 16) {
    const int kk = k0 + 8 * half;
    bf16x8 A[TM], B[TN];
#pragma unroll
    for (int t = 0; t < TM; ++t) A[t] = zero8();
#pragma unroll
    for (int u = 0; u < TN; ++u) B[u] = zero8();
    if (kk < K) {
      const int tap = MODE == 1 ? tap_z : kk / a.kc;
      const int ch = kk - (MODE == 1 ? 0 : tap * a.kc);
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        if (!prow[t]) continue;
        if constexpr (MODE == 0) {
          const int yy = py[t] + tap / 3 - 1, xx = px[t] + tap % 3 - 1;
          if (yy >= 0 && yy < a.h && xx >= 0 && xx < a.w)
            A[t] = load8(a.x + ((int64_t)pn[t] * a.h * a.w + (int64_t)yy * a.w + xx) * a.x_cs + a.x_co + ch);
        } else if constexpr (MODE == 1) {
          const int64_t pix = pix0 + 32 * t + (lane & 31);
          A[t] = load8(a.x + pix * a.x_cs + a.x_co + ch);
        } else {
          const int H2 = 2 * a.h, W2 = 2 * a.w;
          const int yy = 2 * py[t] + (tap >> 1), xx = 2 * px[t] + (tap & 1);
          A[t] = load8(a.x + ((int64_t)pn[t] * H2 * W2 + (int64_t)yy * W2 + xx) * a.x_cs + a.x_co + ch);
        }
      }
#pragma unroll
      for (int u = 0; u < TN; ++u) {
        const int col = col0 + 32 * u + (lane & 31);
        if (col < a.nout) B[u] = load8(a.wgt + ((int64_t)col * wtap + tap) * a.kc + ch);
      }
    }
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) acc[t][u] = mfma(A[t], B[u], acc[t][u]);
  }
#pragma unroll
  for (int u = 0; u < TN; ++u) {
    const int col = col0 + 32 * u + (lane & 31);
    if (col >= a.nout) continue;
    const float bv = a.bias ? a.bias[col] : 0.f;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t p = pix0 + 32 * t + c_row(r, lane);
        if (p >= P) continue;
        float v = acc[t][u][r] + bv;
        if (a.relu) v = v > 0.f ? v : 0.f;
        int64_t o;
        if constexpr (MODE == 1) {
          const int qn = (int)(p / ((int64_t)a.h * a.w));
          const int rr = (int)(p - (int64_t)qn * a.h * a.w);
          const int qy = rr / a.w, qx = rr - qy * a.w;
          const int H2 = 2 * a.h, W2 = 2 * a.w;
          o = (int64_t)qn * H2 * W2 + (int64_t)(2 * qy + (tap_z >> 1)) * W2 + 2 * qx + (tap_z & 1);
        } else {
          o = p;
        }
        a.y[o * a.y_cs + a.y_co + col] = f2bf(v);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// 3x3 convolution with LDS staging.  The reduction runs over 16-channel
// groups, and within a group over the nine taps (k = (group, tap, channel)):
// per group the block stages its input rows with a one-pixel halo (zero
// outside the image) and the group's weights of its output channels in LDS
// once, and all nine taps of all four waves read their MFMA fragments from
// there.  Wave tile TM x TN MFMA tiles (32 x 32 each); the four waves are
// stacked along the pixels, so a block covers 128 TM consecutive pixels --
// whole image rows (16 <= w <= 256, w divides the block, h * w a multiple of
// it) -- and 32 TN output channels.  Needs the reduction channels to be a
// multiple of 16.  For images 16 columns wide and outputs that cannot be stored as
// vectors; the rest goes to conv3x3_rows.  512 pixels by 32 channels for outputs of
// at most 32 channels once there is such a block per CU, 256 by 64 otherwise (us,
// 512 x 32 / 256 x 64: 32 -> 12 at 16 x 128 x 128 13.5 / 18.2, 64 -> 32 at 512 x 32 x 16
// 20.5 / 28.0; 64 -> 20 at two 256 x 256 images, 256 blocks, 24.7 / 29.9; 32 -> 12
// at 64 x 32 x 32, 128 blocks, 10.5 / 8.2).
// ---------------------------------------------------------------------------
// largest staged region over the allowed widths: (pixels / w + 2) rows of w + 2
constexpr int conv_halo_pix(int block_pix) {
  int m = 0;
  for (int w = 16; w <= 256; w *= 2) {
    const int v = (block_pix / w + 2) * (w + 2);
    m = v > m ? v : m;
  }
  return m;
}

template <int TM, int TN>
__global__ __launch_bounds__(256) void conv3x3_lds(GemmArgs a) {
  constexpr int BP = 128 * TM, BC = 32 * TN;
  __shared__ uint4 sA[conv_halo_pix(BP) * 2];  // [region pixel][channel half of the group]
  __shared__ uint4 sB[BC * 9 * 2];             // [output channel][tap][channel half]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5;
  const int w = a.w, h = a.h, rw = w + 2;
  const int64_t p0 = (int64_t)blockIdx.x * BP;
  const int img = (int)(p0 / ((int64_t)h * w));
  const int y0 = (int)((p0 - (int64_t)img * h * w) / w);  // first image row of the block
  const int rows = BP / w + 2;                            // staged rows, halo included
  const int col0 = blockIdx.y * BC;
  const int64_t img_base = (int64_t)img * h * w;
  floatx16 acc[TM][TN];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int u = 0; u < TN; ++u) acc[t][u] = floatx16{};
  // this lane's pixels within the block (row-major over the block's rows)
  int pr[TM], pc[TM];
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int q = wave * 32 * TM + 32 * t + (lane & 31);
    pr[t] = q / w;
    pc[t] = q - pr[t] * w;
  }
  // Software pipeline over the 16-channel groups: the next group's global
  // loads go to registers before this group's taps run, and are parked in
  // LDS after the barrier that ends them.  Each thread's staged elements
  // keep their place from group to group; only the channel offset moves.
  constexpr int KA = (conv_halo_pix(BP) * 2 + 255) / 256, KB = (BC * 9 * 2 + 255) / 256;
  const int nA = rows * rw * 2;
  constexpr uint32_t kNone = 0xffffffffu;  // element outside the image or the weights
  uint32_t offA[KA], offB[KB];              // element offsets (host keeps them below 2^32 - 1)
#pragma unroll
  for (int i = 0; i < KA; ++i) {
    const int e = tid + 256 * i, q = e >> 1, hf = e & 1;
    const int ry = q / rw, rx = q - ry * rw;
    const int y = y0 - 1 + ry, x = rx - 1;
    offA[i] = (e < nA && y >= 0 && y < h && x >= 0 && x < w)
                  ? (uint32_t)((img_base + (int64_t)y * w + x) * a.x_cs + a.x_co + 8 * hf)
                  : kNone;
  }
#pragma unroll
  for (int i = 0; i < KB; ++i) {
    const int e = tid + 256 * i, co = e / 18, rem = e - co * 18;
    const int tap = rem >> 1, hf = rem & 1;
    offB[i] = (e < BC * 9 * 2 && col0 + co < a.nout) ? (uint32_t)(((int64_t)(col0 + co) * 9 + tap) * a.kc + 8 * hf)
                                                     : kNone;
  }
  uint4 ra[KA], rb[KB];
  auto fetch = [&](int ch) {
#pragma unroll
    for (int i = 0; i < KA; ++i)
      ra[i] = offA[i] != kNone ? *reinterpret_cast<const uint4 *>(a.x + offA[i] + ch) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < KB; ++i)
      rb[i] = offB[i] != kNone ? *reinterpret_cast<const uint4 *>(a.wgt + offB[i] + ch) : make_uint4(0, 0, 0, 0);
  };
  const int groups = a.kc / 16;
  fetch(0);
  for (int g = 0; g < groups; ++g) {
#pragma unroll
    for (int i = 0; i < KA; ++i)
      if (tid + 256 * i < nA) sA[tid + 256 * i] = ra[i];
#pragma unroll
    for (int i = 0; i < KB; ++i)
      if (tid + 256 * i < BC * 9 * 2) sB[tid + 256 * i] = rb[i];
    __syncthreads();
    if (g + 1 < groups) fetch((g + 1) * 16);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int dy = tap / 3, dx = tap % 3;
      bf16x8 A[TM], B[TN];
#pragma unroll
      for (int t = 0; t < TM; ++t)
        A[t] = __builtin_bit_cast(bf16x8, sA[((pr[t] + dy) * rw + pc[t] + dx) * 2 + half]);
#pragma unroll
      for (int u = 0; u < TN; ++u)
        B[u] = __builtin_bit_cast(bf16x8, sB[((32 * u + (lane & 31)) * 9 + tap) * 2 + half]);
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u) acc[t][u] = mfma(A[t], B[u], acc[t][u]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < TN; ++u) {
    const int col = col0 + 32 * u + (lane & 31);
    if (col >= a.nout) continue;
    const float bv = a.bias ? a.bias[col] : 0.f;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t p = p0 + wave * 32 * TM + 32 * t + c_row(r, lane);
        float v = acc[t][u][r] + bv;
        if (a.relu) v = v > 0.f ? v : 0.f;
        a.y[p * a.y_cs + a.y_co + col] = f2bf(v);
      }
    }
  }
}

// Can the LDS-staged kernel with blocks of bp pixels run this convolution?
static bool conv_lds_fits(const GemmArgs &a, int bp) {
  // element offsets of the input and the weights must fit 32 bits
  const bool small = (int64_t)a.n * a.h * a.w * a.x_cs < ((int64_t)1 << 32) - 1 &&
                     (int64_t)a.nout * 9 * a.kc < ((int64_t)1 << 32) - 1;
  return small && a.kc % 16 == 0 && a.w >= 16 && a.w <= 256 && bp % a.w == 0 &&
         ((int64_t)a.h * a.w) % bp == 0;
}

// Two floats rounded to BF16 (to nearest even, as f2bf; a NaN stays a quiet NaN).
__device__ __forceinline__ uint32_t f2bf_pair(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float floatx2 __attribute__((ext_vector_type(2)));
  const floatx2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// v, zero where the ReLU output y is not positive.
__device__ __forceinline__ uint4 relu_masked(const uint4 &v, const uint4 &y) {
  const uint32_t yy[4] = {y.x, y.y, y.z, y.w};
  uint32_t gg[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!(bf2f((uint16_t)(yy[k] & 0xffffu)) > 0.f)) gg[k] &= 0xffff0000u;
    if (!(bf2f((uint16_t)(yy[k] >> 16)) > 0.f)) gg[k] &= 0x0000ffffu;
  }
  return make_uint4(gg[0], gg[1], gg[2], gg[3]);
}

// Output of a transposed 32 x 32 product tile: this lane holds channels
// c0 + 8 q + 4 half + 0..3 of pixel o in registers 4 q .. 4 q + 3.  Bias (loaded
// beforehand: a load between two tiles' stores would wait for the first's), ReLU
// and rounding to BF16; then the lane halves trade registers, so that each stores
// 16-byte runs of channels (channel counts, strides and offsets multiples of
// 8, y 16-byte aligned).
struct BiasRun {
  float4 b[4];
};
// buffer: of the biases, empty for none
__device__ __forceinline__ BiasRun load_bias(__amdgpu_buffer_rsrc_t buffer, int c0, int half) {
  BiasRun r;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    r.b[q] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(buffer, 4 * (c0 + 8 * q + 4 * half), 0, 0));
  return r;
}

// The activation of the runs store_pixel writes (loaded beforehand, as the bias).
struct ActRun {
  uint4 y[2];
};
__device__ __forceinline__ ActRun load_act(const GemmArgs &a, bool in, int64_t o, int c0, int half) {
  ActRun r = {};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c = c0 + 16 * q + 8 * half;
    if (in && c < a.nout) r.y[q] = *reinterpret_cast<const uint4 *>(a.act + o * a.act_cs + a.act_co + c);
  }
  return r;
}

template <bool ACT>
__device__ __forceinline__ void store_pixel(const GemmArgs &a, const BiasRun &bias, const ActRun &act, const floatx16 &acc,
                                            bool in, int64_t o, int c0, int half) {
  uint32_t w[8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float bv[4] = {bias.b[q].x, bias.b[q].y, bias.b[q].z, bias.b[q].w};
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = acc[4 * q + k] + bv[k];
      if (a.relu) v[k] = v[k] > 0.f ? v[k] : 0.f;
    }
    w[2 * q] = f2bf_pair(v[0], v[1]);
    w[2 * q + 1] = f2bf_pair(v[2], v[3]);
  }
  // lower half: channels 0..7 and 16..23; upper half: 8..15 and 24..31
  uint16_t *const y = a.y + o * a.y_cs + a.y_co + c0;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const auto s0 = __builtin_amdgcn_permlane32_swap(w[4 * q], w[4 * q + 2], false, false);
    const auto s1 = __builtin_amdgcn_permlane32_swap(w[4 * q + 1], w[4 * q + 3], false, false);
    const int c = 16 * q + 8 * half;
    uint4 v = make_uint4(s0[0], s1[0], s0[1], s1[1]);
    if (ACT && a.act) v = relu_masked(v, act.y[q]);
    if (in && c0 + c < a.nout) *reinterpret_cast<uint4 *>(y + c) = v;
  }
}

// ---------------------------------------------------------------------------
// Implicit GEMM straight from memory: a wave computes 32 TM pixels by 32 TN
// output channels with no LDS and no barrier; its operand fragments are 16-byte
// buffer loads (zeros outside the image and the channels) that run kRing steps of
// 16 reduction channels ahead of the products.  The products are transposed,
// C[channel][pixel], so a lane ends with runs of channels of one pixel and
// stores vectors.  For problems too small to fill the chip with the staged
// convolution's blocks, where the length of one wave's chain is what counts,
// and for the layers whose operands have little reuse.
//   ORDER 0, 3x3: reduction by (16-channel group, tap, channel), as in the staged
//     convolution; the ring is one group's nine taps.
//   ORDER 1, 3x3: by (tap, channel).
//   ORDER 2, 3x3 over 8 channels: two taps a step, the whole reduction in flight.
//   ORDER 3, transposed 2x2: by channel; TN = 4 is the four taps of 32 channels.
//   ORDER 4, its data gradient: by (tap, channel).
// Orders 0, 1 and 4 need kc to be a multiple of 16, order 3 too.
// Both orders of the 3x3 reduction stay because a change of order changes
// results in the last place, which a whole network carries on.
// One 256 x 256 image through the network: 341 us with the staged and gathering
// kernels alone, 207 us with this one for all that they left idle, 161 us with
// conv3x3_rows from 64 tiles on; the same bits.
// ---------------------------------------------------------------------------
template <int ORDER, int TM, int TN, int GP = 1>
__global__ __launch_bounds__(256) void igemm_direct(GemmArgs a, int pix_tiles) {
  constexpr bool kConv = ORDER <= 2;
  constexpr int kRing = ORDER == 0 ? 9 * GP : (ORDER == 2 ? 5 : (ORDER == 3 || (ORDER == 4 && TM * TN >= 4) ? 4 : 8));
  const int lane = threadIdx.x & 63, half = lane >> 5, l31 = lane & 31;
  const int64_t wid = (int64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t P = (int64_t)a.n * a.h * a.w;
  const int ctiles = ORDER == 3 ? (a.nout + 31) / 32 : (a.nout + 32 * TN - 1) / (32 * TN);
  if (wid >= (int64_t)pix_tiles * ctiles) return;
  // the four waves of a block share their pixels where they can
  const int ct = (int)(wid % ctiles);
  const int64_t pix0 = wid / ctiles * (32 * TM);
  const int col0 = ct * (ORDER == 3 ? 32 : 32 * TN);
  const int taps = kConv ? 9 : 4;
  // A (pixels): byte offsets from a base at or before the wave's first pixel
  const int W2 = 2 * a.w;
  int py[TM], px[TM];
  bool in[TM];
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int64_t p = pix0 + 32 * t + l31;
    in[t] = p < P;
    const int64_t q = in[t] ? p : P - 1;
    const int64_t r = q / a.w;
    px[t] = (int)(q - r * a.w);
    py[t] = (int)(r % a.h);
  }
  const uint16_t *abase;
  uint32_t arow[TM];  // this lane's pixel, byte offset from abase
  const uint32_t cs2 = 2u * (uint32_t)a.x_cs;
  if constexpr (ORDER == 4) {
    // dy pixel (2y, 2x); rows of the 2h x 2w grid, linear over images
    const int64_t r0 = pix0 / a.w;
    abase = a.x + a.x_co + 2 * r0 * W2 * a.x_cs;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int64_t p = in[t] ? pix0 + 32 * t + l31 : P - 1;
      const int64_t r = p / a.w;
      arow[t] = in[t] ? (uint32_t)((2 * (r - r0) * W2 + 2 * (p - r * a.w)) * cs2) + 16u * half : kOutside;
    }
  } else {
    abase = a.x + a.x_co + (pix0 - (kConv ? a.w + 1 : 0)) * a.x_cs;
#pragma unroll
    for (int t = 0; t < TM; ++t) arow[t] = in[t] ? (uint32_t)(32 * t + l31) * cs2 + 16u * half : kOutside;
  }
  // offset of tap (dy, dx) of a 3x3 window, masked outside the image
  auto tap_offset = [&](int t, int tap, uint32_t base) {
    const int dy = tap / 3, dx = tap % 3;
    const int y = py[t] + dy - 1, x = px[t] + dx - 1;
    const bool ok = in[t] && tap < 9 && y >= 0 && y < a.h && x >= 0 && x < a.w;
    return ok ? base + (uint32_t)(dy * a.w + dx) * cs2 : kOutside;
  };
  // B (weights, [channel][tap][kc])
  const uint16_t *const bbase = a.wgt + (int64_t)col0 * taps * a.kc;
  uint32_t brow[TN];
#pragma unroll
  for (int u = 0; u < TN; ++u) {
    const int c = ORDER == 3 ? l31 : 32 * u + l31;
    brow[u] = col0 + c < a.nout
                  ? 2u * (uint32_t)((c * taps + (ORDER == 3 ? u : 0)) * a.kc) + (ORDER == 2 ? 0u : 16u * half)
                  : kOutside;
  }
  const auto ar = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(abase), 0, (int)kWholeBuffer, 0x00027000);
  const auto br = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(bbase), 0, (int)kWholeBuffer, 0x00027000);
  auto get = [](auto r, uint32_t off, int s) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, s, 0));
  };
  const auto bias = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.bias), 0, a.bias ? 4 * a.nout : 0, 0x00027000);
  constexpr int NB = ORDER == 3 ? 1 : TN;
  BiasRun b[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) b[u] = load_bias(bias, col0 + 32 * u, half);
  floatx16 acc[TM][TN];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int u = 0; u < TN; ++u) acc[t][u] = floatx16{};
  bf16x8 A[kRing][TM], B[kRing][TN];
  auto products = [&](int i) {
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) acc[t][u] = mfma(B[i][u], A[i][t], acc[t][u]);
  };
  if constexpr (ORDER == 0) {
    uint32_t off[9][TM];
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
      for (int t = 0; t < TM; ++t) off[k][t] = tap_offset(t, k, arow[t]);
    // GP groups at a time: their loads share cache lines
    const int groups = a.kc / 16;
    auto load = [&](int k, int g) {
#pragma unroll
      for (int t = 0; t < TM; ++t) A[k][t] = get(ar, off[k % 9][t], 32 * g);
#pragma unroll
      for (int u = 0; u < TN; ++u) B[k][u] = get(br, brow[u], 2 * (k % 9) * a.kc + 32 * g);
    };
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
      for (int v = 0; v < GP; ++v) load(9 * v + k, v);
    for (int g = GP; g < groups; g += GP) {
#pragma unroll
      for (int v = 0; v < GP; ++v)
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          products(9 * v + k);
          if (v == GP - 1) {
#pragma unroll
            for (int x = 0; x < GP; ++x) load(9 * x + k, g + x);
          }
        }
    }
#pragma unroll
    for (int k = 0; k < 9 * GP; ++k) products(k);
  } else if constexpr (ORDER == 2) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const int tap = 2 * k + half;
#pragma unroll
      for (int t = 0; t < TM; ++t) A[k][t] = get(ar, tap_offset(t, tap, arow[t] - 16u * half), 0);
#pragma unroll
      for (int u = 0; u < TN; ++u) B[k][u] = get(br, tap < 9 ? brow[u] + 16u * tap : kOutside, 0);
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) products(k);
  } else {
    // steps in order; the step being loaded is (tap, 16-channel group)
    const int groups = a.kc / 16, steps = (ORDER == 1 ? 9 : (ORDER == 4 ? 4 : 1)) * groups;
    int ltap = 0, lg = 0;
    uint32_t off[TM];
    auto at_tap = [&]() {
#pragma unroll
      for (int t = 0; t < TM; ++t) off[t] = ORDER == 1 ? tap_offset(t, ltap, arow[t]) : arow[t];
    };
    at_tap();
    auto load = [&](int i) {
      const int as = 32 * lg + (ORDER == 4 ? ((ltap >> 1) * W2 + (ltap & 1)) * (int)cs2 : 0);
      const int bs = 2 * ltap * a.kc + 32 * lg;
#pragma unroll
      for (int t = 0; t < TM; ++t) A[i][t] = get(ar, off[t], as);
#pragma unroll
      for (int u = 0; u < TN; ++u) B[i][u] = get(br, brow[u], bs);
      if (++lg == groups) {
        lg = 0;
        ++ltap;
        if (ORDER == 1) at_tap();
      }
    };
    // past the last step the loads repeat the first one
    auto load_next = [&](int i, int s) {
      if (s >= steps) { ltap = 0; lg = 0; }
      load(i);
    };
#pragma unroll
    for (int i = 0; i < kRing; ++i) load_next(i, i);
    int s = 0;
    for (; s + kRing <= steps; s += kRing) {
#pragma unroll
      for (int i = 0; i < kRing; ++i) {
        products(i);
        load_next(i, s + i + kRing);
      }
    }
#pragma unroll
    for (int i = 0; i < kRing - 1; ++i)
      if (s + i < steps) products(i);
  }
  // C[channel 8 (r / 4) + 4 half + r % 4][pixel l31]
  ActRun act[ORDER == 3 ? 1 : TM][ORDER == 3 ? 1 : TN] = {};
  if (ORDER != 3 && a.act) {
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int u = 0; u < TN; ++u) {
        const int64_t p = pix0 + 32 * t + l31;
        act[ORDER == 3 ? 0 : t][ORDER == 3 ? 0 : u] = load_act(a, p < P, p, col0 + 32 * u, half);
      }
  }
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int64_t p = pix0 + 32 * t + l31;
#pragma unroll
    for (int u = 0; u < TN; ++u) {
      int64_t o = p;
      if constexpr (ORDER == 3) {
        const int64_t r = p / a.w;  // rows are linear over images on both grids
        o = (2 * r + (u >> 1)) * W2 + 2 * (p - r * a.w) + (u & 1);
      }
      const int c0 = col0 + (ORDER == 3 ? 0 : 32 * u);
      store_pixel<ORDER != 3>(a, b[ORDER == 3 ? 0 : u], act[ORDER == 3 ? 0 : t][ORDER == 3 ? 0 : u], acc[t][u], p < P, o, c0, half);
    }
  }
}

// ---------------------------------------------------------------------------
// 3x3 convolution through LDS.  The reduction runs over 16-channel groups, and
// within a group over the nine taps: k = (group, tap, channel).  A block takes
// tiles of 512 pixels (rows of min(w, 128) columns) by 32 TN output channels in
// turn; per group it stages the tile's input with a one-pixel halo (zero outside
// the image) and the group's weights.
// Four waves multiply and four stage, one of each per SIMD: the staging waves fill
// one of two buffers while the other is read, their loads two groups further on,
// and go straight on to the next tile, so the products wait for one barrier a
// group and nothing else.  A multiplying wave owns 32 columns by four rows; with eight
// products per six fragment reads LDS stays below the matrix cores (four per
// four: level with them).  LDS holds [channel half][pixel] and [tap][channel
// half][output channel], so that fragment reads are runs of 512 bytes.  The
// products are transposed, as in the kernel above, for 16-byte stores.
// Tiles are dealt to the XCDs in contiguous ranges (blocks go round the XCDs): a
// range's channel tiles and halos meet in one L2.
// 64 -> 64 channels, 16 x 128 x 128: 43 us with blocks of four waves that stage and
// multiply in turn (256 pixels), 31 us so; 32 -> 32, 16 x 256 x 256: 65 us and 34 us
// (its bytes: 28 us).  256 -> 128, 16 x 64 x 64: 49 and 40 us, 28 us without the
// loads: 32-byte pieces of a pixel are what staging is bound by.  Loading two
// groups at a time, so that the pieces of a line follow each other, gained nothing.
// ---------------------------------------------------------------------------
constexpr int kConvThreads = 512;
constexpr int kConvTilePix = 512;

template <int TN, bool ACT>
__global__ __launch_bounds__(kConvThreads, TN == 1 ? 4 : 2) void conv3x3_rows(GemmArgs a, int items) {
  constexpr int TM = 4, BC = 32 * TN;
  constexpr int kPix = (TM + 2) * 130;  // staged pixels, most for 128 columns
  // strides that keep the two channel halves, and the 18 weight planes, of a
  // staging wave's writes on different banks
  constexpr int kPlane = (kPix * 16 + 127) / 256 * 256 + 128, kWPlane = BC * 16 + 16;
  constexpr int kW = 2 * kPlane, kBuf = kW + 18 * kWPlane;
  __shared__ __attribute__((aligned(16))) char smem[2 * kBuf + 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = a.w, h = a.h;
  const int tw = w < 128 ? w : 128, th = kConvTilePix / tw, rw = tw + 2;
  const int ctiles = (a.nout + BC - 1) / BC, xtiles = w / tw, ytiles = (h + th - 1) / th;
  const int groups = a.kc / 16;
  // this block's tiles: every (grid / 8)-th of its XCD's range
  const int xcd = blockIdx.x & 7, step = gridDim.x >> 3;
  const int first = (int)((int64_t)items * xcd / 8) + (int)(blockIdx.x >> 3);
  const int end = (int)((int64_t)items * (xcd + 1) / 8);
  if (first >= end) return;
  const int stages = ((end - first - 1) / step + 1) * groups;
  struct Tile {
    int col0, x0, y0, img;
  };
  auto tile_of = [&](int item) {
    Tile t;
    int q = item / ctiles;
    t.col0 = (item - q * ctiles) * BC;
    int r = q / xtiles;
    t.x0 = (q - r * xtiles) * tw;
    t.img = r / ytiles;
    t.y0 = (r - t.img * ytiles) * th;
    return t;
  };

  if (wave >= 4) {
    const int t0 = tid - 256;
    constexpr int KA = (kPix * 2 + 255) / 256, KB = (BC * 18 + 255) / 256;
    const uint32_t cs2 = 2u * (uint32_t)a.x_cs;
    // piece i: 8 channels of a staged pixel, row ay column ax of the tile's halo,
    // or of one output channel's tap; past the last, a spare place
    int ay[KA], ax[KA], la[KA], lb[KB], bco[KB];
    uint32_t offa[KA], offb[KB];
#pragma unroll
    for (int i = 0; i < KA; ++i) {
      const int e = t0 + 256 * i, q = e >> 1, hf = e & 1;
      const bool in = q < (th + 2) * rw;
      ay[i] = in ? q / rw - 1 : -(1 << 30);
      ax[i] = q % rw - 1;
      offa[i] = (uint32_t)((q / rw) * w + q % rw) * cs2 + 16u * hf;
      la[i] = in ? hf * kPlane + q * 16 : -1;
    }
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const int e = t0 + 256 * i, co = e / 18, rem = e - 18 * co;
      bco[i] = e < BC * 18 ? co : 1 << 30;
      offb[i] = 2u * (uint32_t)((co * 9 + (rem >> 1)) * a.kc) + 16u * (rem & 1);
      lb[i] = e < BC * 18 ? kW + rem * kWPlane + co * 16 : -1;
    }
    struct Staged {
      uint4 a[KA], b[KB];
    } st[2];
    int item = first, g = 0;  // of the next stage to load
    auto load = [&](Staged &s) __attribute__((always_inline)) {
      const Tile t = tile_of(item);
      const uint16_t *const xp = a.x + a.x_co + (((int64_t)t.img * h + t.y0 - 1) * w + t.x0 - 1) * a.x_cs + 16 * g;
      const uint16_t *const wp = a.wgt + (int64_t)t.col0 * 9 * a.kc + 16 * g;
#pragma unroll
      for (int i = 0; i < KA; ++i) {
        const bool in = (unsigned)(t.y0 + ay[i]) < (unsigned)h && (unsigned)(t.x0 + ax[i]) < (unsigned)w;
        s.a[i] = buffer_load16(xp, kWholeBuffer, in ? offa[i] : kOutside);
      }
#pragma unroll
      for (int i = 0; i < KB; ++i) s.b[i] = buffer_load16(wp, kWholeBuffer, bco[i] < a.nout - t.col0 ? offb[i] : kOutside);
      if (++g == groups) {  // past the last stage: the last tile again, not used
        g = 0;
        item = item + step < end ? item + step : item;
      }
    };
    auto put = [&](int odd, const Staged &s) __attribute__((always_inline)) {
      // (no branch may part these waits from the loads they count)
#pragma unroll
      for (int i = 0; i < KA; ++i)
        *reinterpret_cast<uint4 *>(smem + (la[i] >= 0 ? la[i] + odd * kBuf : 2 * kBuf)) = s.a[i];
#pragma unroll
      for (int i = 0; i < KB; ++i)
        *reinterpret_cast<uint4 *>(smem + (lb[i] >= 0 ? lb[i] + odd * kBuf : 2 * kBuf)) = s.b[i];
    };
    load(st[0]);
    load(st[1]);
    put(0, st[0]);
    load(st[0]);
    __syncthreads();
    for (int i = 0; i < stages; i += 2) {
      put(1, st[1]);
      load(st[1]);
      __syncthreads();
      put(0, st[0]);
      load(st[0]);
      __syncthreads();
    }
    return;
  }

  const int half = lane >> 5, l31 = lane & 31;
  const int strips = tw >> 5, row0 = wave / strips * TM, x = (wave % strips) * 32 + l31;
  const auto bias = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.bias), 0, a.bias ? 4 * a.nout : 0, 0x00027000);
  int arow[TM + 2];
#pragma unroll
  for (int r = 0; r < TM + 2; ++r) arow[r] = half * kPlane + ((row0 + r) * rw + x) * 16;
  const int brow = kW + half * kWPlane + l31 * 16;
  floatx16 acc[TM][TN] = {};
  int item = first, g = 0;
  __syncthreads();
  for (int i = 0; i < stages; ++i) {
    const int buf = (i & 1) * kBuf;
    bf16x8 A[2][TM], B[2][TN];
    auto fetch = [&](int tap) __attribute__((always_inline)) {
      const int k = tap & 1, dy = tap / 3, dx = tap % 3;
#pragma unroll
      for (int u = 0; u < TN; ++u)
        B[k][u] = *reinterpret_cast<const bf16x8 *>(smem + buf + brow + 2 * tap * kWPlane + 512 * u);
#pragma unroll
      for (int t = 0; t < TM; ++t) A[k][t] = *reinterpret_cast<const bf16x8 *>(smem + buf + arow[t + dy] + 16 * dx);
    };
    fetch(0);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      if (tap < 8) fetch(tap + 1);
      __builtin_amdgcn_sched_barrier(0);  // the fetches stay ahead of the products
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u) acc[t][u] = mfma(B[tap & 1][u], A[tap & 1][t], acc[t][u]);
    }
    __syncthreads();
    if (++g < groups) continue;
    g = 0;
    const Tile q = tile_of(item);
    item += step;
    BiasRun b[TN];
#pragma unroll
    for (int u = 0; u < TN; ++u) b[u] = load_bias(bias, q.col0 + 32 * u, half);
    const int y0 = q.y0 + row0;
    const int64_t o = ((int64_t)q.img * h + y0) * w + q.x0 + x;
#pragma unroll
    for (int u = 0; u < TN; ++u) {
      constexpr int TA = TN == 1 ? 2 : TM;  // rows whose activations the registers hold
#pragma unroll
      for (int t0 = 0; t0 < TM; t0 += TA) {
        ActRun act[TA] = {};
        if constexpr (ACT) {
#pragma unroll
          for (int t = 0; t < TA; ++t)
            act[t] = load_act(a, y0 + t0 + t < h, o + (int64_t)(t0 + t) * w, q.col0 + 32 * u, half);
        }
#pragma unroll
        for (int t = t0; t < t0 + TA; ++t) {
          store_pixel<ACT>(a, b[u], act[t - t0], acc[t][u], y0 + t < h, o + (int64_t)t * w, q.col0 + 32 * u, half);
          acc[t][u] = floatx16{};
        }
      }
    }
  }
  if (stages & 1) __syncthreads();  // the staging waves go in pairs
}

// The general kernel's launch: reduction channels not a multiple of 16 (8 has
// its own form), outputs the direct kernel cannot store as vectors, or offsets
// beyond its window.
template <int MODE>
static void launch_gather(const GemmArgs &a, int64_t P, int taps_z, hipStream_t s) {
  if (a.nout >= 64) {
    dim3 g((unsigned)((P + 255) / 256), (unsigned)((a.nout + 63) / 64), (unsigned)taps_z);
    igemm_fwd<MODE, 2, 2><<<g, 256, 0, s>>>(a);
  } else {
    dim3 g((unsigned)((P + 511) / 512), (unsigned)((a.nout + 31) / 32), (unsigned)taps_z);
    igemm_fwd<MODE, 4, 1><<<g, 256, 0, s>>>(a);
  }
}

template <int ORDER, int TM, int TN, int GP = 1>
static void launch_direct(const GemmArgs &a, int64_t P, hipStream_t s) {
  const int64_t pt = (P + 32 * TM - 1) / (32 * TM);
  const int64_t ct = (a.nout + (ORDER == 3 ? 32 : 32 * TN) - 1) / (ORDER == 3 ? 32 : 32 * TN);
  // one wave per block while the waves do not fill the chip: every CU gets one,
  // and with the channel tile counted fastest an XCD meets few of them
  const int wpb = pt * ct <= 4096 ? 1 : 4;
  igemm_direct<ORDER, TM, TN, GP><<<dim3((unsigned)((pt * ct + wpb - 1) / wpb)), 64 * wpb, 0, s>>>(a, (int)pt);
}

// Tile by the number of 32 x 32 tiles: a larger one reads its operands less often, in
// 32-byte pieces that are what these kernels are bound by; a small one has the shorter
// chain and the more waves.  us with the smaller / the larger:
//   order 0, 256 -> 256: two 32 x 32 images (512 tiles) 18.2 / 15.1 (64 x 32; 20.3 with
//     64 x 64), three (768) 26.6 / 20.9 (64 x 64); 32 -> 64, 128 x 128 (1024) 4.9 / 5.2;
//   order 1, 64 -> 64: 92 x 100 (576) 8.6 / 8.0; 256 -> 256: 40 x 60 (600) 26.1 / 19.0,
//     two of 60 x 90 (2704) 81.5 / 54.6; 64 -> 32: two of 100 x 180 (1125) 13.0 / 12.2;
//   order 4, 64 channels, 1 x 128 x 128 (1024) 8.1 / 7.0; 256, 8 x 32 x 32 (2048)
//     22.6 / 14.9; 64 x 128 tiles for 256, 16 x 32 x 32 (4096) 25.7 / 21.2 and for 128,
//     16 x 64 x 64 (8192) 28.8 / 23.5.
template <int ORDER>
static void launch_direct_tiles(const GemmArgs &a, int64_t P, hipStream_t s) {
  const int64_t t = ((P + 31) / 32) * ((a.nout + 31) / 32);
  if constexpr (ORDER == 0) {
    if (a.kc > 32 && a.nout > 32 && t >= 768) launch_direct<0, 2, 2>(a, P, s);
    else if (t >= (a.kc > 32 ? 512 : 2048)) launch_direct<0, 2, 1>(a, P, s);
    else if (a.kc % 32 == 0) launch_direct<0, 1, 1, 2>(a, P, s);
    else launch_direct<0, 1, 1>(a, P, s);
  } else if constexpr (ORDER == 1) {
    if (a.nout > 32 && t >= 512) launch_direct<1, 2, 2>(a, P, s);
    else if (t >= 1024) launch_direct<1, 2, 1>(a, P, s);
    else launch_direct<1, 1, 1>(a, P, s);
  } else {
    if (a.nout > 64 && t >= 4096) launch_direct<4, 2, 4>(a, P, s);
    else if (a.nout > 32 && t >= 1024) launch_direct<4, 2, 2>(a, P, s);
    else if (t >= 2048) launch_direct<4, 2, 1>(a, P, s);
    else launch_direct<4, 1, 1>(a, P, s);
  }
}

// Can the direct kernel run this?  Its stores are vectors of 8 channels; the
// offsets of a wave (its pixels, the rows above and below them) have to stay
// within the buffer window, and its tiles within a grid.
static bool direct_fits(const GemmArgs &a, int64_t P, int taps) {
  if (!dword_aligned(a.x, a.wgt)) return false;
  if (reinterpret_cast<uintptr_t>(a.y) % 16 || a.y_cs % 8 || a.y_co % 8 || a.nout % 8) return false;
  if (a.act && (reinterpret_cast<uintptr_t>(a.act) % 16 || a.act_cs % 8 || a.act_co % 8)) return false;
  const int64_t reach = (taps == 9 ? 64 + 2 * (int64_t)a.w + 2 : 2 * (64 + 2 * (int64_t)a.w) * 2) * a.x_cs * 2;
  const int64_t wbytes = (int64_t)64 * taps * a.kc * 2;
  return reach < kWholeBuffer && wbytes < ((int64_t)1 << 29) && ((P + 31) / 32) * ((a.nout + 31) / 32) < ((int64_t)1 << 31);
}

// Tiles of conv3x3_rows, and can it run this?
static int64_t conv_rows_tiles(const GemmArgs &a, int bc) {
  const int tw = a.w < 128 ? a.w : 128, th = kConvTilePix / tw;
  return (int64_t)a.n * ((a.h + th - 1) / th) * (a.w / tw) * ((a.nout + bc - 1) / bc);
}
static bool conv_rows_fits(const GemmArgs &a, int64_t P) {
  const int64_t rows = a.w < 128 ? kConvTilePix / a.w + 2 : kConvTilePix / 128 + 2;
  return a.w >= 32 && conv_lds_fits(a, 256) && direct_fits(a, P, 9) && rows * a.w * a.x_cs * 2 < kWholeBuffer;
}

template <int TN>
static void launch_conv_rows(const GemmArgs &a, hipStream_t s) {
  // one tile of 64 channels, two of 32 per CU at a time
  const int64_t tiles = conv_rows_tiles(a, 32 * TN), most = TN == 1 ? 512 : 256;
  const dim3 g((unsigned)(tiles < most ? (tiles + 7) / 8 * 8 : most));
  if (a.act) conv3x3_rows<TN, true><<<g, kConvThreads, 0, s>>>(a, (int)tiles);
  else conv3x3_rows<TN, false><<<g, kConvThreads, 0, s>>>(a, (int)tiles);
}

// (Returns whether an activation's mask has been applied.)
// Group by group where the staged kernels can run (a rule on the shape alone: the
// order of the sums may not change with the number of images), tap by tap elsewhere.
// Within the first, by tiles of 512 pixels x 32 channels, us direct / through LDS:
//   64 -> 32 at 1 x 128 x 128 (32 tiles) 6.5 / 9.5, at two images (64) 10.6 / 9.4;
//   128 -> 128 at 1 x 64 x 64 (32) 10.3 / 12.8, at two (64) 18.5 / 13.0;
//   32 -> 32 at 1 x 256 x 256 (128) 7.1 / 7.9, at two (256) 11.1 / 9.1.
// 64-channel tiles once there is one per CU: 64 -> 64 at 4 x 128 x 128 13.9 (13.1
// with 32), at eight images 18.7 (21.5).
static bool launch_conv3x3(const GemmArgs &a, int64_t P, hipStream_t s) {
  const bool direct = direct_fits(a, P, 9);
  if (direct && a.kc == 8) {
    if (P >= 2 * 32 * 1024) launch_direct<2, 2, 1>(a, P, s);
    else launch_direct<2, 1, 1>(a, P, s);
  } else if (conv_rows_fits(a, P) && conv_rows_tiles(a, 32) >= (a.kc > 32 ? 64 : 192)) {
    if (a.nout > 32 && conv_rows_tiles(a, 64) >= 256) launch_conv_rows<2>(a, s);
    else launch_conv_rows<1>(a, s);
  } else if (conv_lds_fits(a, 256)) {
    // sixteen columns wide, or too few tiles, or outputs that are not whole
    // vectors: 64 blocks of the staged kernel leave most CUs idle
    const dim3 g((unsigned)(P / 256), (unsigned)((a.nout + 63) / 64));
    if (direct && (a.w >= 32 || (int64_t)g.x * g.y <= 64)) launch_direct_tiles<0>(a, P, s);
    else {
      if (a.nout <= 32 && P >= 256 * 512 && conv_lds_fits(a, 512)) conv3x3_lds<4, 1><<<(unsigned)(P / 512), 256, 0, s>>>(a);
      else conv3x3_lds<2, 2><<<g, 256, 0, s>>>(a);
      return false;
    }
  } else if (direct && a.kc % 16 == 0) {
    launch_direct_tiles<1>(a, P, s);
  } else {
    launch_gather<0>(a, P, 1, s);
    return false;
  }
  return true;
}

// ---------------------------------------------------------------------------
// Weight gradients (split over pixels): partial[kb][tap][m][n] = sum over the
// kb-th share of the pixels of A(m, p) B(p, n).
//   MODE 0, 3x3: m = co, n = (tap, ci): A = dy[p][co], B = x[p + off(tap)][ci]
//   MODE 1, transposed 2x2: m = co, n = ci:
//          A = dy[2p + tap][co], B = x[p][ci]  (p over the input grid)
// Channel counts, strides and offsets are multiples of 8.
// ---------------------------------------------------------------------------
constexpr int kWgradPix = 4096;  // pixels per partial sum

struct WgradArgs {
  const uint16_t *x;
  int n, h, w, cin, x_cs, x_co;   // x grid (input grid for MODE 1)
  const uint16_t *dy;
  int cout, dy_cs, dy_co;
  float *partial;                 // [kblocks][ntap][cout][ncol]
  int ncol;                       // MODE 0: 9 * cin; MODE 1: cin
  float *bpartial;                // [kblocks][ntap][cout] bias partial sums, or NULL
};

// ---------------------------------------------------------------------------
// Weight gradients by gathered pixels, for the grids where whole rows or 16-column
// segments leave the kernels below little to work on.  A block sums its 4096
// pixels for one tile of (output channel, tap and input channel); MODE 1 has a block per
// tap.  Per stage of 128 pixels in memory order, whatever the width, each thread
// loads an 8-pixel x 8-channel block of one operand (eight 16-byte vectors),
// transposes it in registers (byte permutes) and writes it channel-major to LDS, so
// an MFMA operand fragment (8 consecutive pixels of one channel) is one 128-bit
// LDS read and neither side of LDS sees bank conflicts.
// ---------------------------------------------------------------------------
constexpr int kStagePix = 128;  // pixels per LDS stage
constexpr int kStageLd = kStagePix + 8;

// 8 x 8 transpose of 16-bit values: in[p] holds channels 0..7 of pixel p,
// out[c] receives pixels 0..7 of channel c.
__device__ __forceinline__ void transpose8x8(const uint4 (&in)[8], uint4 (&out)[8]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t lo[4], hi[4];  // channel 2j and 2j + 1, pixel pairs i
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t a = (&in[2 * i].x)[j], b = (&in[2 * i + 1].x)[j];
      lo[i] = __builtin_amdgcn_perm(b, a, 0x05040100u);
      hi[i] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    }
    out[2 * j] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    out[2 * j + 1] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  }
}

// Block tile (32 MT) x (32 NT) of C with MT * NT = 4 waves, each one 32 x 32
// MFMA tile: (2, 2) in general, (1, 4) when the output channels fit 32.
template <int MODE, int MT, int NT>
__global__ __launch_bounds__(256) void wgrad_gather(WgradArgs a) {
  static_assert(MT * NT == 4, "four waves");
  __shared__ __attribute__((aligned(16))) uint16_t sA[32 * MT][kStageLd];  // [m][pixel]
  __shared__ __attribute__((aligned(16))) uint16_t sB[32 * NT][kStageLd];  // [n][pixel]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % MT, wn = wave / MT;
  const int half = lane >> 5;
  const int64_t P = (int64_t)a.n * a.h * a.w;
  const int64_t p_begin = (int64_t)blockIdx.x * kWgradPix;
  const int m0 = blockIdx.y * 32 * MT;  // output channel block
  const int tapz = MODE == 1 ? (int)(blockIdx.z % 4) : 0;
  const int nblk = MODE == 1 ? (int)(blockIdx.z / 4) : (int)blockIdx.z;
  const int n0 = nblk * 32 * NT;        // column block
  floatx16 acc = {};
  // the blocks of the first column block also sum dy over their pixels (bias)
  const bool bias_blk = a.bpartial && nblk == 0 && tid < 32 * MT;
  float bacc = 0.f;
  const int64_t p_end = p_begin + kWgradPix < P ? p_begin + kWgradPix : P;
  // staging: 8-pixel x 8-channel blocks, 64 MT of A then 64 NT of B; a
  // thread owns entries tid and tid + 256.  The next stage's loads go to
  // registers before this stage's products run; the transpose and the LDS
  // stores follow the barrier that ends them.
  constexpr int kEntries = 64 * (MT + NT), NE = (kEntries + 255) / 256;
  uint4 v[NE][8];
  auto load_stage = [&](int64_t pcs) {
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      const int e = tid + 256 * j;
      const bool stage_b = e >= 64 * MT;
      const int eo = stage_b ? e - 64 * MT : e;
      const int cg = eo >> 4, pb = eo & 15;
      // image, row and column of the first of the 8 consecutive pixels; the
      // others follow by increments (wrapping at row and image ends)
      const int64_t pfirst = pcs + pb * 8;
      int pn = (int)(pfirst / ((int64_t)a.h * a.w));
      const int rr0 = (int)(pfirst - (int64_t)pn * a.h * a.w);
      int py = rr0 / a.w, px = rr0 - py * a.w;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int64_t p = pfirst + r;
        if (r > 0 && ++px == a.w) {
          px = 0;
          if (++py == a.h) {
            py = 0;
            ++pn;
          }
        }
        v[j][r] = make_uint4(0, 0, 0, 0);
        if (e >= kEntries || p >= p_end) continue;
        if (!stage_b) {
          const int m = m0 + cg * 8;
          if (m < a.cout) {
            int64_t q;
            if constexpr (MODE == 0) {
              q = p;
            } else {
              const int H2 = 2 * a.h, W2 = 2 * a.w;
              q = (int64_t)pn * H2 * W2 + (int64_t)(2 * py + (tapz >> 1)) * W2 + 2 * px + (tapz & 1);
            }
            v[j][r] = *reinterpret_cast<const uint4 *>(a.dy + q * a.dy_cs + a.dy_co + m);
          }
        } else {
          const int nn = n0 + cg * 8;
          if (nn < a.ncol) {
            if constexpr (MODE == 0) {
              const int tap = nn / a.cin, ci = nn - tap * a.cin;
              const int yy = py + tap / 3 - 1, xx = px + tap % 3 - 1;
              if (yy >= 0 && yy < a.h && xx >= 0 && xx < a.w)
                v[j][r] = *reinterpret_cast<const uint4 *>(
                    a.x + ((int64_t)pn * a.h * a.w + (int64_t)yy * a.w + xx) * a.x_cs + a.x_co + ci);
            } else {
              v[j][r] = *reinterpret_cast<const uint4 *>(a.x + p * a.x_cs + a.x_co + nn);
            }
          }
        }
      }
    }
  };
  if (p_begin < p_end) load_stage(p_begin);
  for (int64_t pc = p_begin; pc < p_end; pc += kStagePix) {
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      const int e = tid + 256 * j;
      if (e >= kEntries) continue;
      const bool stage_b = e >= 64 * MT;
      const int eo = stage_b ? e - 64 * MT : e;
      const int cg = eo >> 4, pb = eo & 15;
      uint4 t[8];
      transpose8x8(v[j], t);
      uint16_t(*dst)[kStageLd] = stage_b ? sB : sA;
#pragma unroll
      for (int c = 0; c < 8; ++c) *reinterpret_cast<uint4 *>(&dst[cg * 8 + c][pb * 8]) = t[c];
    }
    __syncthreads();
    if (pc + kStagePix < p_end) load_stage(pc + kStagePix);
    if (bias_blk) {
#pragma unroll
      for (int q = 0; q < kStagePix; q += 8) {
        const uint4 u = *reinterpret_cast<const uint4 *>(&sA[tid][q]);
        const uint32_t w4[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) bacc += bf2f((uint16_t)(w4[k] & 0xffffu)) + bf2f((uint16_t)(w4[k] >> 16));
      }
    }
#pragma unroll
    for (int ks = 0; ks < kStagePix; ks += 16) {
      const uint4 av = *reinterpret_cast<const uint4 *>(&sA[wm * 32 + (lane & 31)][ks + 8 * half]);
      const uint4 bv = *reinterpret_cast<const uint4 *>(&sB[wn * 32 + (lane & 31)][ks + 8 * half]);
      acc = mfma(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv), acc);
    }
    __syncthreads();
  }
  const int ntap = MODE == 1 ? 4 : 1;
  if (bias_blk && m0 + tid < a.cout)
    a.bpartial[((int64_t)blockIdx.x * ntap + tapz) * a.cout + m0 + tid] = bacc;
  const int nn = n0 + wn * 32 + (lane & 31);
  if (nn >= a.ncol) return;
  float *out = a.partial + ((int64_t)blockIdx.x * ntap + tapz) * (int64_t)a.cout * a.ncol;
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + wm * 32 + c_row(r, lane);
    if (m < a.cout) out[(int64_t)m * a.ncol + nn] = acc[r];
  }
}

// ---------------------------------------------------------------------------
// Weight gradients with all taps in one wave, for images of any width.  A wave owns a
// 32 x 32 tile of (output, input) channels and marches down image rows, 16 pixels of a row
// at a time, accumulating every tap of that tile: a row of x enters three
// products per column shift (with the dy rows above, at and below it), so its
// fragments stay in registers for three steps and an LDS read feeds more than
// one product.  Both operands pass through LDS as they lie in memory, [pixel][32
// channels], in a piece of LDS of the wave's own (no barrier in the loop):
// ds_read_b64_tr_b16 turns eight pixels of a channel into an MFMA fragment, and
// a column shift is an offset of one pixel.  Global loads run kDepth rows ahead.
//   MODE 0, 3x3: steps run over 16-column segments, images and rows, with one
//     zero row after every image (it supplies the zero row above and below;
//     its own products are skipped).
//   MODE 1, transposed 2x2: a step is 16 input pixels and their four dy pixels.
// The order of a sum is thus by segments of columns, then images and rows, in eight
// ranges: the eight waves of a block take consecutive step ranges and add their sums
// through LDS at the end, in wave order; a block writes one partial sum.
// ---------------------------------------------------------------------------
constexpr int kWgThreads = 512;  // eight waves
constexpr int kPixBytes = 64;    // a staged pixel: 32 channels

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) short4v lds_short4;

// MFMA fragment of 16 consecutive staged pixels by 32 channels from two reads.
// Within 16 lanes, lane i receives element i % 4 of the 8-byte words that lanes
// i / 4, 4 + i / 4, 8 + i / 4 and 12 + i / 4 address; so lane l addresses pixel
// 8 (l / 32) + (l % 16) / 4, channels 16 (l / 16 % 2) + 4 (l % 4), first, and the
// same four pixels further on, second.
__device__ __forceinline__ int tr_pixel(int lane) { return 8 * (lane >> 5) + ((lane & 15) >> 2); }
__device__ __forceinline__ int tr_channel_bytes(int lane) { return (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2; }
__device__ __forceinline__ bf16x8 tr_fragment(lds_char *first, lds_char *second) {
  const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)first);
  const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)second);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Steps of a weight gradient: segments of 16 columns by (image, row) slots.
template <int MODE> __host__ __device__ inline int64_t wg_rows(const WgradArgs &a) {
  return (int64_t)a.n * (MODE == 0 ? a.h + 1 : a.h);
}

// Between a wave's LDS writes and other lanes' reads of them, and back: LDS operations of
// a wave are done in order, so no wait is needed, only that the compiler keeps
// the order (it sees one lane, whose addresses need not meet).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Block -> (share of the pixels, channel tile), tiles fastest: each XCD takes a
// contiguous range (blocks go round the XCDs), so the tiles of a share meet in one
// L2, or in few.  False past the last; the grid is wg_grid's.  Transposed 2x2,
// 512 -> 512 channels at 16 x 33 x 100 (13 shares): 1190 us with the blocks of a share
// dealt round the XCDs, 508 us so; 256 -> 256 262 and 141 us.
__device__ __forceinline__ bool wg_block(int kb, int tiles, int &ck, int &tile) {
  const int total = kb * tiles, id = (int)(blockIdx.x & 7) * ((total + 7) / 8) + (int)(blockIdx.x >> 3);
  ck = id / tiles;
  tile = id - ck * tiles;
  return id < total;
}
static unsigned wg_grid(int kb, int tiles) { return (unsigned)(((int64_t)kb * tiles + 7) / 8 * 8); }

template <int MODE>
__global__ __launch_bounds__(kWgThreads) void wgrad_taps(WgradArgs a, int kb, int64_t steps_per_wave, int ci_tiles,
                                                         int tiles) {
  constexpr int NT = MODE == 0 ? 9 : 4;  // taps
  constexpr int NA = MODE == 0 ? 1 : 4;  // dy tiles per step
  constexpr int kDepth = 2;              // steps whose loads are in flight
  constexpr int kXPix = MODE == 0 ? 18 : 16;
  // a wave's LDS: x, three zero pixels, dy
  constexpr int kZero = kXPix * kPixBytes, kDy = kZero + 3 * kPixBytes;
  constexpr int kWave = kDy + NA * 16 * kPixBytes;
  constexpr int kRed = 8 * 1024 * 4;  // eight waves' sums of one tap
  constexpr int kBytes = 8 * kWave > kRed ? 8 * kWave : kRed;
  __shared__ __attribute__((aligned(16))) char smem[kBytes];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  char *const sw = smem + wave * kWave;
  lds_char *const lw = (lds_char *)sw;
  int ck, tile;
  if (!wg_block(kb, tiles, ck, tile)) return;
  const int m0 = (tile / ci_tiles) * 32, n0 = (tile % ci_tiles) * 32;
  const bool bias = a.bpartial && n0 == 0;
  const int rows = MODE == 0 ? a.h + 1 : a.h;
  const int64_t rows_all = wg_rows<MODE>(a);
  const int64_t total = rows_all * ((a.w + 15) / 16);
  const int64_t u0 = ((int64_t)ck * 8 + wave) * steps_per_wave;
  const int64_t u1 = u0 + steps_per_wave < total ? u0 + steps_per_wave : total;
  // this lane stages channels ch .. ch + 7 of pixel px of the 16
  const int px = lane >> 2, ch = 8 * (lane & 3);
  const bool xc = n0 + ch < a.cin, dc = m0 + ch < a.cout;
  const uint16_t *const xg = a.x + a.x_co + n0;
  const uint16_t *const dg = a.dy + a.dy_co + m0;

  // the step being loaded: segment, slot row within its image, real row over
  // all images; it starts one step early in MODE 0 (the zero row before the
  // first image where u0 = 0)
  const int64_t first = MODE == 0 ? u0 - 1 : u0;
  int seg, row;
  int64_t lrow, slots_left;  // slots left in the segment
  if (first < 0) {
    seg = -1; row = rows - 1; lrow = 0; slots_left = 1;
  } else {
    seg = (int)(first / rows_all);
    const int64_t r = first - seg * rows_all;
    const int64_t img = r / rows;
    row = (int)(r - img * rows);
    lrow = img * a.h + row;
    slots_left = rows_all - r;
  }
  // byte offsets of this lane's pieces from the segment's first pixel (x: one
  // pixel before it in MODE 0)
  uint32_t xoff, hoff, doff;
  auto columns = [&]() {
    const int c = 16 * seg + px - (MODE == 0 ? 1 : 0);
    xoff = xc && c >= 0 && c < a.w ? 2u * (uint32_t)(px * a.x_cs + ch) : kOutside;
    hoff = xc && lane < 8 && c + 16 < a.w ? 2u * (uint32_t)((px + 16) * a.x_cs + ch) : kOutside;
    doff = dc && 16 * seg + px < a.w ? 2u * (uint32_t)((MODE == 0 ? px : 2 * px) * a.dy_cs + ch) : kOutside;
  };
  columns();
  struct Staged {  // this lane's pieces of one step, on their way to LDS
    uint4 x, xh, dy[NA];
    int seg;
    bool real;
  } st[kDepth];
  int64_t u = first;
  auto load = [&](Staged &g) __attribute__((always_inline)) {
    const bool on = (MODE == 1 || row < a.h) && seg >= 0 && u <= u1;
    const uint32_t bytes = on ? kWholeBuffer : 0;
    g.real = on && u >= u0 && u < u1;
    g.seg = seg;
    const int64_t pix = lrow * a.w + 16 * seg;
    const uint16_t *const xp = xg + (pix - (MODE == 0 ? 1 : 0)) * a.x_cs;
    g.x = buffer_load16(xp, bytes, xoff);
    if constexpr (MODE == 0) g.xh = buffer_load16(xp, bytes, hoff);
#pragma unroll
    for (int t = 0; t < NA; ++t) {
      const int64_t dpix = MODE == 0 ? pix : (2 * lrow + (t >> 1)) * 2 * a.w + 32 * seg + (t & 1);
      g.dy[t] = buffer_load16(dg + dpix * a.dy_cs, bytes, doff);
    }
    // on to the next step
    ++u;
    if (MODE == 1 || row < a.h) ++lrow;
    if (++row == rows) row = 0;
    if (--slots_left == 0) {
      slots_left = rows_all;
      lrow = 0;
      ++seg;
      columns();
    }
  };
  lds_char *p0 = lw, *p1 = lw;  // this lane's x fragment pixels
  int pseg = -2;                // the segment they are set for
  const int j0 = tr_pixel(lane), tc = tr_channel_bytes(lane);
  floatx16 acc[NT];
  float bsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // of this lane's dy channels
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = floatx16{};
  bf16x8 A[2][NA], B[3][MODE == 0 ? 3 : 1];
  bool real[2] = {false, false};
  if (lane < 12) *reinterpret_cast<uint4 *>(sw + kZero + 16 * lane) = make_uint4(0, 0, 0, 0);
  // an iteration brings in one step and runs the products of the one before it;
  // a few more than needed run at the end, on zeros
  const int iters = u0 < u1 ? (int)(u1 - first + 1) : 0;
  if (iters > 0) {
#pragma unroll
    for (int v = 0; v < kDepth; ++v) load(st[v]);
  }
  auto iterate = [&](Staged &g, bf16x8 (&An)[NA], const bf16x8 (&Ac)[NA], bool &real_n, bool real_c,
                     bf16x8 (&Bu)[MODE == 0 ? 3 : 1], const bf16x8 (&Bm)[MODE == 0 ? 3 : 1],
                     bf16x8 (&Bd)[MODE == 0 ? 3 : 1]) __attribute__((always_inline)) {
    wave_lds_fence();  // the last step's reads come first
    *reinterpret_cast<uint4 *>(sw + 16 * lane) = g.x;
    if (MODE == 0 && lane < 8) *reinterpret_cast<uint4 *>(sw + 16 * kPixBytes + 16 * lane) = g.xh;
#pragma unroll
    for (int t = 0; t < NA; ++t) *reinterpret_cast<uint4 *>(sw + kDy + t * 16 * kPixBytes + 16 * lane) = g.dy[t];
    wave_lds_fence();
    if (g.seg != pseg) {
      // columns outside the image read a zero pixel: their dy is zero, but zero
      // times an infinite x is not
      pseg = g.seg;
      const bool o0 = 16 * pseg + j0 >= a.w, o1 = 16 * pseg + j0 + 4 >= a.w;
      p0 = lw + (o0 ? kZero : j0 * kPixBytes + tc);
      p1 = lw + (o1 ? kZero : (j0 + 4) * kPixBytes + tc);
    }
    real_n = g.real;
    if (bias && g.real) {
#pragma unroll
      for (int t = 0; t < NA; ++t) {
        const uint32_t d4[4] = {g.dy[t].x, g.dy[t].y, g.dy[t].z, g.dy[t].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          bsum[2 * k] += __uint_as_float(d4[k] << 16);
          bsum[2 * k + 1] += __uint_as_float(d4[k] & 0xffff0000u);
        }
      }
    }
    load(g);
#pragma unroll
    for (int c = 0; c < (MODE == 0 ? 3 : 1); ++c) Bd[c] = tr_fragment(p0 + c * kPixBytes, p1 + c * kPixBytes);
#pragma unroll
    for (int t = 0; t < NA; ++t) {
      lds_char *const q = lw + kDy + (t * 16 + j0) * kPixBytes + tc;
      An[t] = tr_fragment(q, q + 4 * kPixBytes);
    }
    if constexpr (MODE == 0) {
      if (real_c) {  // rows above, at, below
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[c] = mfma(Ac[0], Bu[c], acc[c]);
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[3 + c] = mfma(Ac[0], Bm[c], acc[3 + c]);
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[6 + c] = mfma(Ac[0], Bd[c], acc[6 + c]);
      }
    } else {
      if (real_c) {
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma(Ac[t], Bm[0], acc[t]);
      }
    }
  };
  for (int j = 0; j < iters; j += 6) {
#pragma unroll
    for (int v = 0; v < 6; ++v)
      iterate(st[v % kDepth], A[v & 1], A[(v + 1) & 1], real[v & 1], real[(v + 1) & 1], B[(v + 1) % 3],
              B[(v + 2) % 3], B[v % 3]);
  }
  // sums of the eight waves, tap by tap
  float *const red = reinterpret_cast<float *>(smem);
  const int ntap = MODE == 1 ? 4 : 1;
  float *const out = a.partial + (int64_t)ck * ntap * a.cout * a.ncol;
  auto sum_waves = [&](const floatx16 &v, float (&r)[2]) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) red[wave * 1024 + c_row(q, lane) * 32 + (lane & 31)] = v[q];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      r[k] = red[tid + 512 * k];
#pragma unroll
      for (int u = 1; u < 8; ++u) r[k] += red[u * 1024 + tid + 512 * k];
    }
  };
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    float r[2];
    sum_waves(acc[t], r);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int m = m0 + (tid >> 5) + 16 * k, n = n0 + (tid & 31);
      if (m >= a.cout || n >= a.cin) continue;
      if constexpr (MODE == 0) out[(int64_t)m * a.ncol + t * a.cin + n] = r[k];
      else out[((int64_t)t * a.cout + m) * a.ncol + n] = r[k];
    }
  }
  if (bias) {  // uniform over the block; the sum over the taps counts as tap 0's
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k) red[(8 * (lane & 3) + k) * 128 + 16 * wave + px] = bsum[k];
    __syncthreads();
    if (tid < 32 && m0 + tid < a.cout) {
      float r = 0.f;
      for (int k = 0; k < 128; ++k) r += red[tid * 128 + (k + tid) % 128];
      for (int t = 0; t < ntap; ++t) a.bpartial[((int64_t)ck * ntap + t) * a.cout + m0 + tid] = t ? 0.f : r;
    }
  }
}

// ---------------------------------------------------------------------------
// Weight gradients in pixel order, for images of whole 16-pixel segments up to
// 256 (MODE 1: 128) columns.  One accumulator takes a tap's products of a share of the
// pixels in the order they lie in memory, and the bias its pixel pairs.  Where the
// width divides 4096 a share is 4096 pixels, as in wgrad_gather, whatever the number
// of images, and the two give the same bits (Adam's first steps turn a last-place
// change of a vanishing gradient into a whole learning rate); elsewhere it is
// ceil(rows / shares) whole rows, with ceil(pixels / 4096) shares.
// A block owns a share of the pixels and a 32 x 32 channel tile.  Rows of
// x and dy go through LDS in stages of at most SP pixels, whole rows with a zero
// column on both sides, x in a ring that also holds the rows above and below the
// stage; a row outside its image is read from a block of zeros.
// The sums are serial chains, so what counts is that nothing else delays them:
// four waves multiply and four stage, one of each per SIMD, a stage ahead and its
// loads two further.  MODE 0: a wave owns the three taps of a row (three reads of
// four pixels serve all three: the outer two taps are register pairs of them, the
// middle one is shifted by half a register) and a fourth adds up the bias.
// MODE 1: a wave per tap.
// 64 -> 64 channels, 16 x 128 x 128: 118 us with a block per tap, 32 us so (45 us
// with ten waves that each stage, multiply one tap and read both operands).  The
// chain of 256 steps of three products is 10 us, staging alone 17 us.
// ---------------------------------------------------------------------------
constexpr int kWgRowsThreads = 512;

template <int MODE, int SP, int SEGS>
__global__ __launch_bounds__(kWgRowsThreads) void wgrad_rows(WgradArgs a, int kb, int chunk_rows, int stage_rows,
                                                             int ci_tiles, int tiles) {
  constexpr int NA = MODE == 0 ? 1 : 4;  // dy tiles per stage
  constexpr int NT = MODE == 0 ? 3 : 1;  // taps of a wave
  constexpr int kPass = 64;              // pixels the staging waves take at a time
  constexpr int NP = SP / kPass;         // pieces of a tile a thread stages
  constexpr int kTile = SP * kPixBytes;
  constexpr int U = SEGS < 4 ? 4 : SEGS;  // steps per turn of the loop
  // x: MODE 0 a ring of 2 stage_rows + 2 rows of w + 2 pixels (largest for
  // one-row stages; its last row is read two pixels further), MODE 1 two stages
  constexpr int kX = MODE == 0 ? 4 * (SP + 2) * kPixBytes : 2 * kTile;
  constexpr int kZeroPix = 16 * SEGS + 4;  // a unit of zero pixels
  constexpr int kZero = kX + 2 * NA * kTile;
  constexpr int kSpare = kZero + kZeroPix * kPixBytes;
  __shared__ __attribute__((aligned(16))) char smem[kSpare + 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  lds_char *const lds = (lds_char *)smem;
  int ck, tile;
  if (!wg_block(kb, tiles, ck, tile)) return;
  const int m0 = (tile / ci_tiles) * 32, n0 = (tile % ci_tiles) * 32;
  const bool bias = a.bpartial && n0 == 0;
  const int w = a.w, G = stage_rows, ring = 2 * G + 2, pitch = (w + 2) * kPixBytes;
  const int rows_all = a.n * a.h;
  const int r0 = ck * chunk_rows, r1 = r0 + chunk_rows < rows_all ? r0 + chunk_rows : rows_all;
  const int stages = r1 > r0 ? (r1 - r0 + G - 1) / G : 0;
  const uint16_t *const xg = a.x + a.x_co + n0, *const dg = a.dy + a.dy_co + m0;

  // zero columns, the block of zeros, and the rows above the first stage and its
  // first one (ring rows 0 and 1)
  const uint4 zero = make_uint4(0, 0, 0, 0);
  for (int e = tid; e < 4 * kZeroPix; e += kWgRowsThreads) *reinterpret_cast<uint4 *>(smem + kZero + 16 * e) = zero;
  if constexpr (MODE == 0) {
    for (int e = tid; e < ring * 8; e += kWgRowsThreads)
      *reinterpret_cast<uint4 *>(smem + (e >> 3) * pitch + ((e >> 2) & 1) * (w + 1) * kPixBytes + 16 * (e & 3)) = zero;
    if (stages > 0)
      for (int e = tid; e < 2 * w * 4; e += kWgRowsThreads) {
        const int p = e >> 2, q = p / w;
        const int64_t r = r0 - 1 + q;
        uint4 v = zero;
        if (n0 + 8 * (e & 3) < a.cin && r >= 0)
          v = *reinterpret_cast<const uint4 *>(xg + (r * w + p - q * w) * a.x_cs + 8 * (e & 3));
        *reinterpret_cast<uint4 *>(smem + q * pitch + (1 + p - q * w) * kPixBytes + 16 * (e & 3)) = v;
      }
  }

  if (wave >= 4) {  // staging: piece k of this thread is 8 channels (ch) of one pixel of a stage
    const int t0 = tid - 256, ch = 8 * (t0 & 3);
    const bool xc = n0 + ch < a.cin, dc = m0 + ch < a.cout;
    uint32_t xoff[NP], doff[NP];
    int lx[NP], ld[NP];  // LDS addresses; a piece past the stage's pixels goes to a spare one
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int p = (t0 >> 2) + kPass * k;
      const bool in = p < G * w;
      const int prow = p / w, col = p - prow * w;
      // MODE 0: stage 0 goes to ring rows 2 .. (G = 1: 2 and 3 of 4)
      lx[k] = !in ? kSpare : (MODE == 0 ? (2 + prow) * pitch + (1 + col) * kPixBytes : p * kPixBytes) + 2 * ch;
      ld[k] = !in ? kSpare : kX + p * kPixBytes + 2 * ch;
      xoff[k] = xc && in ? 2u * (uint32_t)(p * a.x_cs + ch) : kOutside;
      doff[k] = dc && in ? 2u * (uint32_t)((MODE == 0 ? p : 4 * w * prow + 2 * col) * a.dy_cs + ch) : kOutside;
    }
    struct Staged {
      uint4 x[NP], dy[NA][NP];
    } st[2];
    // stage i: dy rows r0 + i G ..; x rows the same (MODE 1) or one further on.
    // Rows past the share's last (x: the one below it) lie beyond the buffer.
    const uint32_t xrow = 2u * (uint32_t)(w * a.x_cs), drow = 2u * (uint32_t)((MODE == 0 ? w : 4 * w) * a.dy_cs);
    const int xlast = MODE == 0 && r1 < rows_all ? r1 + 1 : r1;
    auto load = [&](int i, Staged &g) __attribute__((always_inline)) {
      const int dr = r0 + i * G, xr = dr + (MODE == 0 ? 1 : 0);
      const int dn = r1 - dr, xn = xlast - xr;
      const uint32_t xbytes = (uint32_t)(xn < 0 ? 0 : xn < G ? xn : G) * xrow;
      const uint32_t dbytes = (uint32_t)(dn < 0 ? 0 : dn < G ? dn : G) * drow;
      const uint16_t *const xp = xg + (int64_t)xr * (xrow / 2);
      const uint16_t *const dp = dg + (int64_t)dr * (drow / 2);
#pragma unroll
      for (int k = 0; k < NP; ++k) g.x[k] = buffer_load16(xp, xbytes, xoff[k]);
#pragma unroll
      for (int t = 0; t < NA; ++t) {
        const int tap = MODE == 0 ? 0 : (2 * w * (t >> 1) + (t & 1)) * a.dy_cs;
#pragma unroll
        for (int k = 0; k < NP; ++k) g.dy[t][k] = buffer_load16(dp + tap, dbytes, doff[k]);
      }
    };
    auto put = [&](int odd, const Staged &g) __attribute__((always_inline)) {
      // (no branch may part these waits from the loads they count)
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const bool in = ld[k] != kSpare;
        *reinterpret_cast<uint4 *>(smem + lx[k] + (MODE == 1 && in ? odd * kTile : 0)) = g.x[k];
#pragma unroll
        for (int t = 0; t < NA; ++t)
          *reinterpret_cast<uint4 *>(smem + ld[k] + (in ? (odd * NA + t) * kTile : 0)) = g.dy[t][k];
        if (MODE == 0 && in) {  // G rows on in the ring
          lx[k] += G * pitch;
          lx[k] = lx[k] >= ring * pitch ? lx[k] - ring * pitch : lx[k];
        }
      }
    };
    load(0, st[0]);
    load(1, st[1]);
    put(0, st[0]);
    load(2, st[0]);
    __syncthreads();
    for (int i = 0; i < stages; i += 2) {  // stages past the last are zeros
      put(1, st[1]);
      load(i + 3, st[1]);
      __syncthreads();
      put(0, st[0]);
      load(i + 4, st[0]);
      __syncthreads();
    }
    return;
  }

  const int lo = tr_pixel(lane) * kPixBytes + tr_channel_bytes(lane);
  const int segs = w >> 4, steps = G * segs;
  // bias: a chain of pixel pairs per channel; both lane halves hold the same sum
  float bsum = 0.f;
  auto add_bias = [&](const bf16x8 &F) __attribute__((always_inline)) {
    const uint4 v = __builtin_bit_cast(uint4, F);
    const uint32_t d4[4] = {v.x, v.y, v.z, v.w};
    float lo8[4], hi8[4];  // pairs of pixels 0 .. 7 and 8 .. 15
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t s = __float_as_uint(__uint_as_float(d4[q] << 16) + __uint_as_float(d4[q] & 0xffff0000u));
      const auto h = __builtin_amdgcn_permlane32_swap(s, s, false, false);
      lo8[q] = __uint_as_float(h[0]);
      hi8[q] = __uint_as_float(h[1]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) bsum += lo8[q];
#pragma unroll
    for (int q = 0; q < 4; ++q) bsum += hi8[q];
  };
  const int ntap = MODE == 1 ? 4 : 1;
  const int64_t share = (int64_t)ck * ntap;

  if (MODE == 0 && wave == 3) {
    __syncthreads();
    for (int i = 0; i < stages; i += 2) {
#pragma unroll
      for (int odd = 0; odd < 2; ++odd) {
        if (bias) {
          bf16x8 F[2][4];
          int s = 0;
          auto fetch4 = [&](bf16x8 (&f)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < 4; ++v, ++s) {
              lds_char *const p = lds + (s < steps ? kX + odd * kTile + s * 16 * kPixBytes : kZero) + lo;
              f[v] = tr_fragment(p, p + 4 * kPixBytes);
            }
          };
          fetch4(F[0]);
          for (int u = 0; u < steps; u += 8) {
            fetch4(F[1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < 4; ++v) add_bias(F[0][v]);
            fetch4(F[0]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < 4; ++v) add_bias(F[1][v]);
          }
        }
        __syncthreads();
      }
    }
    if (bias && lane < 32 && m0 + lane < a.cout) a.bpartial[share * a.cout + m0 + lane] = bsum;
    return;
  }

  floatx16 acc[NT] = {};
  int xr = 0;        // ring row of the row above the stage's first
  int y = r0 % a.h;  // row within its image
  __syncthreads();
  auto stage = [&](int i, int odd) __attribute__((always_inline)) {
    const int nr = r1 - (r0 + i * G) < G ? r1 - (r0 + i * G) : G;
    // position of the next unit of SEGS steps to fetch
    const int parts = MODE == 0 ? segs / SEGS : 1;
    int part = 0, row = 0, yy = y, slot = 0, done = 0;
    auto row_start = [&]() {  // this wave's window row of image row yy
      if constexpr (MODE == 0) {
        const int s = xr + row + wave;
        const bool in = yy + wave - 1 >= 0 && yy + wave - 1 < a.h && row < nr;
        slot = in ? (s >= ring ? s - ring : s) * pitch : -1;
      }
    };
    row_start();
    const int dy0 = kX + (odd * NA + (MODE == 0 ? 0 : wave)) * kTile;
    int ua = 0, ub = 0;  // the unit's LDS addresses
    auto next_unit = [&]() __attribute__((always_inline)) {
      ua = done < steps ? dy0 + done * 16 * kPixBytes : kZero;
      if constexpr (MODE == 0) {
        ub = slot < 0 ? kZero : slot + part * (SEGS * 16 * kPixBytes);
        if (++part == parts) {
          part = 0;
          ++row;
          if (++yy == a.h) yy = 0;
          row_start();
        }
      } else {
        ub = done < steps ? odd * kTile + done * 16 * kPixBytes : kZero;
      }
      done += SEGS;
    };
    // Fragments are fetched kAhead steps early, with no condition, so that the
    // wait before a product is for its own fragments only.
    constexpr int kAhead = 2, kSlots = 4;
    bf16x8 A[kSlots];
    short4v B[kSlots][MODE == 0 ? 3 : 2];
    auto fetch = [&](int k) __attribute__((always_inline)) {
      if (k % SEGS == 0) next_unit();
      lds_char *const p = lds + ua + lo + (k % SEGS) * 16 * kPixBytes;
      A[k % kSlots] = tr_fragment(p, p + 4 * kPixBytes);
      lds_char *const q = lds + ub + lo + (k % SEGS) * 16 * kPixBytes;
#pragma unroll
      for (int j = 0; j < (MODE == 0 ? 3 : 2); ++j)
        B[k % kSlots][j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(q + 4 * j * kPixBytes));
    };
    auto product = [&](int v) __attribute__((always_inline)) {
      const bf16x8 f = __builtin_bit_cast(bf16x8, __builtin_shufflevector(B[v][0], B[v][1], 0, 1, 2, 3, 4, 5, 6, 7));
      acc[0] = mfma(A[v], f, acc[0]);
      if constexpr (MODE == 0) {  // pixels -1 .. 6 so far; 0 .. 7 and 1 .. 8
        const short4v b0 = B[v][0], b1 = B[v][1], b2 = B[v][2];
        const auto r0 = __builtin_bit_cast(uint2, b0), r1 = __builtin_bit_cast(uint2, b1), r2 = __builtin_bit_cast(uint2, b2);
        const uint4 g = make_uint4(__builtin_amdgcn_alignbit(r0.y, r0.x, 16), __builtin_amdgcn_alignbit(r1.x, r0.y, 16),
                                   __builtin_amdgcn_alignbit(r1.y, r1.x, 16), __builtin_amdgcn_alignbit(r2.x, r1.y, 16));
        acc[1] = mfma(A[v], __builtin_bit_cast(bf16x8, g), acc[1]);
        const uint4 h = make_uint4(r0.y, r1.x, r1.y, r2.x);
        acc[2] = mfma(A[v], __builtin_bit_cast(bf16x8, h), acc[2]);
      } else if (bias) {
        add_bias(A[v]);
      }
    };
#pragma unroll
    for (int v = 0; v < kAhead; ++v) fetch(v);
    for (int s = 0; s < steps; s += U) {
#pragma unroll
      for (int v = 0; v < U; ++v) {
        fetch((v + kAhead) % U);
        __builtin_amdgcn_sched_barrier(0);  // the fetches stay ahead of the products
        product(v % kSlots);
      }
    }
    __syncthreads();
    xr += G;
    xr = xr >= ring ? xr - ring : xr;
    y += G;
    if (y >= a.h) y %= a.h;
  };
  for (int i = 0; i < stages; i += 2) {
    stage(i, 0);
    stage(i + 1, 1);  // past the last: zeros
  }
  const int n = n0 + (lane & 31);
  float *const out = a.partial + share * a.cout * a.ncol;
  if (n < a.cin) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + c_row(r, lane);
        if (m >= a.cout) continue;
        if constexpr (MODE == 0) out[(int64_t)m * a.ncol + (3 * wave + t) * a.cin + n] = acc[t][r];
        else out[((int64_t)wave * a.cout + m) * a.ncol + n] = acc[t][r];
      }
  }
  if (MODE == 1 && bias && lane < 32 && m0 + lane < a.cout) a.bpartial[(share + wave) * a.cout + m0 + lane] = bsum;
}

template <int MODE, int SP>
static void launch_wgrad_rows(const WgradArgs &a, int kb, hipStream_t s) {
  const int64_t rows = (int64_t)a.n * a.h;
  const int chunk = kWgradPix % a.w == 0 ? kWgradPix / a.w : (int)((rows + kb - 1) / kb);
  const int G = SP / a.w;
  const int ci_tiles = (a.cin + 31) / 32, tiles = ci_tiles * ((a.cout + 31) / 32);
  const dim3 g(wg_grid(kb, tiles));
  const int segs = MODE == 0 ? a.w / 16 : G * a.w / 16;
  if (segs % 8 == 0) wgrad_rows<MODE, SP, 8><<<g, kWgRowsThreads, 0, s>>>(a, kb, chunk, G, ci_tiles, tiles);
  else if (segs % 4 == 0) wgrad_rows<MODE, SP, 4><<<g, kWgRowsThreads, 0, s>>>(a, kb, chunk, G, ci_tiles, tiles);
  else if (segs % 2 == 0) wgrad_rows<MODE, SP, 2><<<g, kWgRowsThreads, 0, s>>>(a, kb, chunk, G, ci_tiles, tiles);
  else wgrad_rows<MODE, SP, 1><<<g, kWgRowsThreads, 0, s>>>(a, kb, chunk, G, ci_tiles, tiles);
}

// Whole 16-pixel segments, rows that fit a stage, and a stage's pixels within
// the buffer window.
static bool wgrad_rows_fits(const WgradArgs &a, int sp) {
  const int64_t cs = a.x_cs > 4 * (int64_t)a.dy_cs ? a.x_cs : 4 * (int64_t)a.dy_cs;
  return a.w % 16 == 0 && a.w <= sp && (int64_t)a.n * a.h < ((int64_t)1 << 31) - 512 && 2 * (sp + 2) * cs < kWholeBuffer;
}

template <int MODE>
static void launch_wgrad_taps(const WgradArgs &a, int kb, hipStream_t s) {
  const int64_t total = wg_rows<MODE>(a) * ((a.w + 15) / 16);
  const int64_t per_wave = (total + 8 * (int64_t)kb - 1) / (8 * (int64_t)kb);
  const int ci_tiles = (a.cin + 31) / 32, tiles = ci_tiles * ((a.cout + 31) / 32);
  wgrad_taps<MODE><<<wg_grid(kb, tiles), kWgThreads, 0, s>>>(a, kb, per_wave, ci_tiles, tiles);
}

template <int MODE>
static void launch_wgrad_gather(const WgradArgs &a, int kb, hipStream_t s) {
  const unsigned taps = MODE == 1 ? 4 : 1;
  if (a.cout <= 32) {
    wgrad_gather<MODE, 1, 4><<<dim3((unsigned)kb, 1, taps * (unsigned)((a.ncol + 127) / 128)), 256, 0, s>>>(a);
  } else {
    const dim3 g((unsigned)kb, (unsigned)((a.cout + 63) / 64), taps * (unsigned)((a.ncol + 63) / 64));
    wgrad_gather<MODE, 2, 2><<<g, 256, 0, s>>>(a);
  }
}

// The kernel of a weight gradient, by measurement over 4493 (MODE 1: 4294) shapes from
// 1 x 1 x 1 to 16 x 300 x 300 pixels and 8 to 1024 channels.  wgrad_gather where
//   - a stage or two of its 128 pixels is all there is (us, it / the other, 64 -> 64: 1 x 5 x 17
//     10.6 / 12.8; 1 x 16 x 16 12.5 / 11.8 in MODE 0);
//   - images have few columns: a 16-column segment is mostly empty (64 -> 64: 16 x 1000 x 1
//     85 / 258, 16 x 300 x 2 84 / 111, 1 x 300 x 3 26.5 / 30.6, 1 x 300 x 4 31.0 / 30.6, MODE 1
//     31.1 / 35.9; MODE 1, 256 -> 256: 16 x 300 x 8 99 / 139), the more so the fuller the chip;
//   - MODE 1 fills it with blocks that waste a quarter of a stage (256 -> 256 at 16 x 32 x 96
//     103 / 134; with fewer shares not: 512 -> 512 at 2 x 48 x 48 90 / 51) or read dy eight times
//     as wide as x (64 -> 1024 at 16 x 33 x 100 162 / 211).
template <int MODE>
static bool gather_wins(const WgradArgs &a, int kb, bool rows) {
  if (!dword_aligned(a.x, a.dy)) return true;
  const int64_t P = (int64_t)a.n * a.h * a.w, tiles = (int64_t)((a.cin + 31) / 32) * ((a.cout + 31) / 32);
  const int64_t blocks = kb * tiles;
  if (rows) return MODE == 0 ? P <= 128 : kb >= 3 && blocks >= 512 && 128 / a.w * a.w <= 96;
  if (P <= 128 || (P <= 256 && (a.cout > 32 || a.w <= 8))) return true;
  if (MODE == 0) return a.w <= 2 || (a.w == 3 && a.cout > 32) || (a.w <= 4 && P <= 1024);
  return a.w <= 4 || (a.w <= 6 && (P <= 512 || blocks >= 256)) || (a.w <= 12 && kb >= 3 && blocks >= 512) ||
         (blocks >= 512 && a.cout >= 8 * a.cin) || (tiles >= 1024 && P <= 2048);
}

template <int MODE>
static void launch_wgrad(const WgradArgs &a, int kb, hipStream_t s) {
  constexpr int SP = MODE == 0 ? 256 : 128;
  const bool rows = wgrad_rows_fits(a, SP);
  if (gather_wins<MODE>(a, kb, rows)) launch_wgrad_gather<MODE>(a, kb, s);
  else if (rows) launch_wgrad_rows<MODE, SP>(a, kb, s);
  else launch_wgrad_taps<MODE>(a, kb, s);
}

// sum_{k < count} p[k * stride] in a fixed order: eight interleaved partial
// sums (k mod 8) combined pairwise, so the loads of a thread overlap.
__device__ __forceinline__ float strided_sum(const float *p, int64_t count, int64_t stride) {
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int64_t k = 0;
  for (; k + 8 <= count; k += 8)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] += p[(k + j) * stride];
  for (int j = 0; k + j < count; ++j) acc[j] += p[(k + j) * stride];
  return ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
}

// Weight and bias gradients from the partial sums, in one launch:
//   dw[m][tap][n] (+)= sum over kblocks of partial[kb][tap][m][n]
//     (MODE 0: ntap = 1 and n = (tap, ci) already),
//   db[c] (+)= sum over the bparts bias partials, by the last ceil(cout / 32) blocks.
// The sums are strided_sum's.  SPLIT: eight threads share an element, one per partial
// sum, so that the few elements of the wide layers (9216 by 256 partials) have
// enough loads in flight: 5 us, with a thread per element and a launch for the
// biases 13.5 and 9.8 us.
template <bool SPLIT>
__global__ __launch_bounds__(256) void wgrad_reduce(const float *partial, int kblocks, int ntap, int cout, int ncol,
                                                    float *dw, int accumulate, int wblocks, const float *bpartial,
                                                    int64_t bparts, float *db) {
  const int64_t total = (int64_t)ntap * cout * ncol;
  const int tid = threadIdx.x;
  const bool bias = blockIdx.x >= (unsigned)wblocks;
  float s;
  int64_t e;
  if (SPLIT || bias) {
    __shared__ float part[8][33];
    const int j = tid >> 5, i = tid & 31;
    e = (bias ? blockIdx.x - wblocks : blockIdx.x) * (int64_t)32 + i;
    const float *const p = bias ? bpartial : partial;
    const int64_t count = bias ? bparts : kblocks, stride = bias ? cout : total;
    float v = 0.f;
    if (e < stride) {
      int64_t k = j;
      for (; k + 24 < count; k += 32) {
        float u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = p[(k + 8 * q) * stride + e];
#pragma unroll
        for (int q = 0; q < 4; ++q) v += u[q];
      }
      for (; k < count; k += 8) v += p[k * stride + e];
    }
    part[j][i] = v;
    __syncthreads();
    if (tid >= 32 || e >= stride) return;
    s = ((part[0][i] + part[1][i]) + (part[2][i] + part[3][i])) + ((part[4][i] + part[5][i]) + (part[6][i] + part[7][i]));
  } else {
    e = blockIdx.x * (int64_t)256 + tid;
    if (e >= total) return;
    s = strided_sum(partial + e, kblocks, total);
  }
  if (bias) {
    db[e] = accumulate ? db[e] + s : s;
    return;
  }
  const int tap = (int)(e / ((int64_t)cout * ncol));
  const int64_t rem = e - (int64_t)tap * cout * ncol;
  const int m = (int)(rem / ncol), n = (int)(rem - (int64_t)m * ncol);
  const int64_t o = ((int64_t)m * ntap + tap) * ncol + n;  // [co][tap][ci]
  dw[o] = accumulate ? dw[o] + s : s;
}

static void launch_wgrad_reduce(const float *partial, int kb, int ntap, int cout, int ncol, float *dw, int accumulate,
                                const float *bpartial, int64_t bparts, float *db, hipStream_t s) {
  const int64_t total = (int64_t)ntap * cout * ncol;
  const bool split = kb >= 32;  // (fewer partials are in flight at once anyway)
  const int wblocks = (int)((total + (split ? 31 : 255)) / (split ? 32 : 256));
  const int blocks = wblocks + (db ? (cout + 31) / 32 : 0);
  if (split) wgrad_reduce<true><<<blocks, 256, 0, s>>>(partial, kb, ntap, cout, ncol, dw, accumulate, wblocks, bpartial, bparts, db);
  else wgrad_reduce<false><<<blocks, 256, 0, s>>>(partial, kb, ntap, cout, ncol, dw, accumulate, wblocks, bpartial, bparts, db);
}

// wt[ci][ky][kx][co] = w[co][2-ky][2-kx][ci]
__global__ void conv_flip(const uint16_t *w, int cout, int cin, uint16_t *wt) {
  const int64_t total = (int64_t)cout * 9 * cin;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int co = (int)(e / (9 * cin));
    const int r = (int)(e - (int64_t)co * 9 * cin);
    const int tap = r / cin, ci = r - tap * cin;
    wt[((int64_t)ci * 9 + (8 - tap)) * cout + co] = w[e];
  }
}

// wt[ci][tap][co] = w[co][tap][ci] (2x2 taps)
__global__ void up_rearrange(const uint16_t *w, int cout, int cin, uint16_t *wt) {
  const int64_t total = (int64_t)cout * 4 * cin;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int co = (int)(e / (4 * cin));
    const int r = (int)(e - (int64_t)co * 4 * cin);
    const int tap = r / cin, ci = r - tap * cin;
    wt[((int64_t)ci * 4 + tap) * cout + co] = w[e];
  }
}

__global__ void relu_bwd_kernel(const uint16_t *y, int64_t n_pix, int c, int y_cs, int y_co, uint16_t *dy,
                                int dy_cs, int dy_co) {
  const int64_t total = n_pix * c;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = e / c;
    const int ch = (int)(e - p * c);
    if (!(bf2f(y[p * y_cs + y_co + ch]) > 0.f)) dy[p * dy_cs + dy_co + ch] = 0;
  }
}

__global__ void maxpool_fwd_kernel(const uint16_t *x, int n, int h, int w, int c, int x_cs, int x_co, uint16_t *y,
                                   int y_cs, int y_co) {
  const int h2 = h / 2, w2 = w / 2;
  const int64_t total = (int64_t)n * h2 * w2 * c;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int ch = (int)(e % c);
    const int64_t q = e / c;
    const int qn = (int)(q / ((int64_t)h2 * w2));
    const int r = (int)(q - (int64_t)qn * h2 * w2);
    const int qy = r / w2, qx = r - qy * w2;
    float m = -INFINITY;
    uint16_t best = 0;
    for (int a = 0; a < 2; ++a)
      for (int b = 0; b < 2; ++b) {
        const uint16_t v = x[((int64_t)qn * h * w + (int64_t)(2 * qy + a) * w + 2 * qx + b) * x_cs + x_co + ch];
        if (bf2f(v) > m) { m = bf2f(v); best = v; }
      }
    y[q * y_cs + y_co + ch] = best;
  }
}

// Pooling by vectors of eight channels, a window's eight channels per thread (channel
// counts, strides and offsets multiples of 8, fewer than 2^31 vectors).  Bound by
// memory: 16 x 256 x 256 x 32 in a slice of 64 channels, forward 27 us (37 us with a
// channel per thread); backward 64 us both ways, at 64 x 64 x 128 13 us (20 us).
struct Window {
  int64_t p;  // its first pixel
  int64_t q;  // its pixel of the half-size grid
  int ch;
};
__device__ __forceinline__ Window pool_window(unsigned e, unsigned w2, unsigned c8, int w) {
  const unsigned q = e / c8, row = q / w2;  // rows are linear over images on both grids
  return {(int64_t)row * 2 * w + 2 * (int64_t)(q - row * w2), (int64_t)q, (int)(e - q * c8) * 8};
}
__device__ __forceinline__ void unpack8(const uint4 &v, uint16_t (&o)[8]) {
  const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    o[2 * k] = (uint16_t)(u[k] & 0xffffu);
    o[2 * k + 1] = (uint16_t)(u[k] >> 16);
  }
}

__global__ __launch_bounds__(256) void maxpool_fwd_vec(const uint16_t *x, unsigned total, int w, int c8, int x_cs,
                                                       int x_co, uint16_t *y, int y_cs, int y_co) {
  const unsigned e = blockIdx.x * 256u + threadIdx.x;
  if (e >= total) return;
  const Window o = pool_window(e, (unsigned)w / 2, (unsigned)c8, w);
  const uint16_t *const px = x + o.p * x_cs + x_co + o.ch;
  uint4 v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const uint4 *>(px + (int64_t)((k >> 1) * w + (k & 1)) * x_cs);
  uint16_t best[8] = {};
  float m[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) m[j] = -INFINITY;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint16_t t[8];
    unpack8(v[k], t);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (bf2f(t[j]) > m[j]) {
        m[j] = bf2f(t[j]);
        best[j] = t[j];
      }
  }
  *reinterpret_cast<bf16x8 *>(y + o.q * y_cs + y_co + o.ch) = pack8(best);
}

__global__ __launch_bounds__(256) void maxpool_bwd_vec(const uint16_t *x, unsigned total, int w, int c8, int x_cs,
                                                       int x_co, const uint16_t *dy, int dy_cs, int dy_co, uint16_t *dx,
                                                       int dx_cs, int dx_co, int accumulate, int relu) {
  const unsigned e = blockIdx.x * 256u + threadIdx.x;
  if (e >= total) return;
  const Window o = pool_window(e, (unsigned)w / 2, (unsigned)c8, w);
  const uint16_t *const px = x + o.p * x_cs + x_co + o.ch;
  uint16_t *const pd = dx + o.p * dx_cs + dx_co + o.ch;
  uint4 v[4], d[4] = {};
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const uint4 *>(px + (int64_t)((k >> 1) * w + (k & 1)) * x_cs);
  uint16_t g[8];
  unpack8(*reinterpret_cast<const uint4 *>(dy + o.q * dy_cs + dy_co + o.ch), g);
  if (accumulate) {
#pragma unroll
    for (int k = 0; k < 4; ++k) d[k] = *reinterpret_cast<const uint4 *>(pd + (int64_t)((k >> 1) * w + (k & 1)) * dx_cs);
  }
  float m[8];
  int arg[8] = {};
#pragma unroll
  for (int j = 0; j < 8; ++j) m[j] = -INFINITY;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint16_t t[8];
    unpack8(v[k], t);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (bf2f(t[j]) > m[j]) {
        m[j] = bf2f(t[j]);
        arg[j] = k;
      }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint16_t t[8];
    unpack8(d[k], t);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (k == arg[j]) t[j] = accumulate ? f2bf(bf2f(t[j]) + bf2f(g[j])) : g[j];
    uint4 r = __builtin_bit_cast(uint4, pack8(t));
    if (relu) r = relu_masked(r, v[k]);
    *reinterpret_cast<uint4 *>(pd + (int64_t)((k >> 1) * w + (k & 1)) * dx_cs) = r;
  }
}

// Vector form (channel counts, strides and offsets multiples of 8): one
// 16-byte vector of 8 channels per thread.
__global__ void relu_bwd_vec(const uint16_t *y, int64_t n_pix, int c8, int y_cs, int y_co, uint16_t *dy, int dy_cs,
                             int dy_co) {
  const int64_t total = n_pix * c8;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = e / c8;
    const int ch = (int)(e - p * c8) * 8;
    uint16_t *const dp = dy + p * dy_cs + dy_co + ch;
    store_any16(dp, relu_masked(load_any16(dp), load_any16(y + p * y_cs + y_co + ch)));
  }
}

__global__ void maxpool_bwd_kernel(const uint16_t *x, int n, int h, int w, int c, int x_cs, int x_co,
                                   const uint16_t *dy, int dy_cs, int dy_co, uint16_t *dx, int dx_cs, int dx_co,
                                   int accumulate) {
  const int h2 = h / 2, w2 = w / 2;
  const int64_t total = (int64_t)n * h2 * w2 * c;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int ch = (int)(e % c);
    const int64_t q = e / c;
    const int qn = (int)(q / ((int64_t)h2 * w2));
    const int r = (int)(q - (int64_t)qn * h2 * w2);
    const int qy = r / w2, qx = r - qy * w2;
    float m = -INFINITY;
    int arg = 0;
    for (int k = 0; k < 4; ++k) {
      const float v = bf2f(x[((int64_t)qn * h * w + (int64_t)(2 * qy + k / 2) * w + 2 * qx + k % 2) * x_cs + x_co + ch]);
      if (v > m) { m = v; arg = k; }
    }
    const uint16_t g = dy[q * dy_cs + dy_co + ch];
    for (int k = 0; k < 4; ++k) {
      uint16_t *d = dx + ((int64_t)qn * h * w + (int64_t)(2 * qy + k / 2) * w + 2 * qx + k % 2) * dx_cs + dx_co + ch;
      if (accumulate) {
        if (k == arg) *d = f2bf(bf2f(*d) + bf2f(g));
      } else {
        *d = k == arg ? g : 0;
      }
    }
  }
}

__device__ __forceinline__ float head_logit(const uint16_t *x, int64_t p, int c, int x_cs, const float *w, float b) {
  float z = b;
  if ((c & 7) == 0 && (x_cs & 7) == 0) {  // 16-byte vectors of 8 channels
    for (int c8 = 0; c8 < c; c8 += 8) {
      const uint4 v = load_any16(x + p * x_cs + c8);
      const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        z += w[c8 + 2 * k] * bf2f((uint16_t)(u[k] & 0xffffu));
        z += w[c8 + 2 * k + 1] * bf2f((uint16_t)(u[k] >> 16));
      }
    }
    return z;
  }
  for (int ch = 0; ch < c; ++ch) z += w[ch] * bf2f(x[p * x_cs + ch]);
  return z;
}

__global__ void head_fwd_kernel(const uint16_t *x, int64_t n_pix, int c, int x_cs, const float *w, const float *b,
                                float *sat) {
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n_pix; p += (int64_t)gridDim.x * blockDim.x)
    sat[p] = 1.f / (1.f + __expf(-head_logit(x, p, c, x_cs, w, b[0])));
}

// Per pixel: logit z, loss term l = softplus(z) - t z (binary cross-entropy
// written on the logit), gradient g = (sigmoid(z) - t) * scale on masked
// pixels (0 elsewhere), and dx = g w.  g and l go to scratch for the sums.
__global__ void head_loss_pix(const uint16_t *x, int64_t n_pix, int c, int x_cs, const float *w, const float *b,
                              const float *t, const uint8_t *mask, float scale, uint16_t *dx, float *g_out,
                              float *l_out) {
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n_pix; p += (int64_t)gridDim.x * blockDim.x) {
    const float z = head_logit(x, p, c, x_cs, w, b[0]);
    const bool on = mask[p] != 0;
    const float sp = fmaxf(z, 0.f) + log1pf(__expf(-fabsf(z)));
    const float s = 1.f / (1.f + __expf(-z));
    const float g = on ? (s - t[p]) * scale : 0.f;
    g_out[p] = g;
    l_out[p] = on ? (sp - t[p] * z) * scale : 0.f;
    if (dx && (c & 7) == 0) {
      for (int c8 = 0; c8 < c; c8 += 8) {
        uint32_t u[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          u[k] = (uint32_t)f2bf(g * w[c8 + 2 * k]) | ((uint32_t)f2bf(g * w[c8 + 2 * k + 1]) << 16);
        store_any16(dx + p * c + c8, make_uint4(u[0], u[1], u[2], u[3]));
      }
    } else if (dx) {
      for (int ch = 0; ch < c; ++ch) dx[p * c + ch] = f2bf(g * w[ch]);
    }
  }
}

// The same by vectors (c a power of two from 8 to 64, x_cs a multiple of 8, x and dx
// 16-byte aligned): 256 pixels pass through LDS, so that global accesses are runs of
// whole pixels while a thread still adds up one pixel's channels in order.  Bound by
// memory: 16 x 256 x 256 pixels of 32 channels 34 us (71 us with a pixel per thread).
__global__ __launch_bounds__(256) void head_loss_pix_v(const uint16_t *x, int64_t n_pix, int c, int x_cs,
                                                       const float *w, const float *b, const float *t,
                                                       const uint8_t *mask, float scale, uint16_t *dx, float *g_out,
                                                       float *l_out, int relu) {
  __shared__ __attribute__((aligned(16))) char sx[256 * (64 * 2 + 16)];
  __shared__ float sw[64], sg[256];
  const int tid = threadIdx.x, c8 = c / 8, pitch = 2 * c + 16;  // (the odd 16 bytes spread pixels over the banks)
  const int64_t p0 = blockIdx.x * (int64_t)256;
  if (tid < c) sw[tid] = w[tid];
  for (int e = tid; e < 256 * c8; e += 256) {
    const int q = e / c8, k = e - q * c8;
    if (p0 + q < n_pix)
      *reinterpret_cast<uint4 *>(sx + q * pitch + 16 * k) = *reinterpret_cast<const uint4 *>(x + (p0 + q) * x_cs + 8 * k);
  }
  __syncthreads();
  const int64_t p = p0 + tid;
  if (p < n_pix) {
    float z = b[0];
    for (int k = 0; k < c8; ++k) {
      uint16_t v[8];
      const uint4 q = *reinterpret_cast<const uint4 *>(sx + tid * pitch + 16 * k);
      const uint32_t u[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[2 * j] = (uint16_t)(u[j] & 0xffffu);
        v[2 * j + 1] = (uint16_t)(u[j] >> 16);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) z += sw[8 * k + j] * bf2f(v[j]);
    }
    const bool on = mask[p] != 0;
    const float sp = fmaxf(z, 0.f) + log1pf(__expf(-fabsf(z)));
    const float s = 1.f / (1.f + __expf(-z));
    const float g = on ? (s - t[p]) * scale : 0.f;
    g_out[p] = g;
    l_out[p] = on ? (sp - t[p] * z) * scale : 0.f;
    sg[tid] = g;
  }
  if (!dx) return;
  __syncthreads();
  for (int e = tid; e < 256 * c8; e += 256) {
    const int q = e / c8, k = e - q * c8;
    if (p0 + q >= n_pix) break;
    uint32_t u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = f2bf_pair(sg[q] * sw[8 * k + 2 * j], sg[q] * sw[8 * k + 2 * j + 1]);
    uint4 r = make_uint4(u[0], u[1], u[2], u[3]);
    if (relu) r = relu_masked(r, *reinterpret_cast<const uint4 *>(sx + q * pitch + 16 * k));
    *reinterpret_cast<uint4 *>(dx + (p0 + q) * c + 8 * k) = r;
  }
}

// Block partials over a pixel chunk: threads = (256 / c) pixel lanes x c
// channels.  out[block] = {sum l, sum g, sum g x[.][0..c)}.
constexpr int kHeadPix = 4096;
__global__ void head_loss_sums(const uint16_t *x, int64_t n_pix, int c, int x_cs, const float *g, const float *l,
                               float *partial) {
  __shared__ float red[256];
  __shared__ float red_l[256], red_g[256];
  const int lanes = 256 / c;
  const int pl = threadIdx.x / c, ch = threadIdx.x - pl * c;
  const int64_t p0 = (int64_t)blockIdx.x * kHeadPix;
  float a = 0.f, sl = 0.f, sg = 0.f;
  for (int k = pl; k < kHeadPix; k += lanes) {
    const int64_t p = p0 + k;
    if (p >= n_pix) break;
    a += g[p] * bf2f(x[p * x_cs + ch]);
    if (ch == 0) { sl += l[p]; sg += g[p]; }
  }
  red[threadIdx.x] = a;
  red_l[threadIdx.x] = sl;
  red_g[threadIdx.x] = sg;
  __syncthreads();
  if (threadIdx.x < (unsigned)c) {
    float s = 0.f;
    for (int q = 0; q < lanes; ++q) s += red[q * c + threadIdx.x];
    partial[(int64_t)blockIdx.x * (2 + c) + 2 + threadIdx.x] = s;
  }
  if (threadIdx.x == 0) {
    float s1 = 0.f, s2 = 0.f;
    for (int q = 0; q < lanes; ++q) { s1 += red_l[q * c]; s2 += red_g[q * c]; }
    partial[(int64_t)blockIdx.x * (2 + c)] = s1;
    partial[(int64_t)blockIdx.x * (2 + c) + 1] = s2;
  }
}

// Vector form of head_loss_sums (c and x_cs multiples of 8): threads =
// (256 / (c / 8)) pixel lanes x (c / 8) channel groups of eight, each with
// eight accumulators fed by one 16-byte load per pixel.
__global__ void head_loss_sums_v(const uint16_t *x, int64_t n_pix, int c, int x_cs, const float *g, const float *l,
                                 float *partial) {
  __shared__ float red[256 * 8];
  __shared__ float red_l[256], red_g[256];
  const int groups = c / 8, lanes = 256 / groups;
  const int pl = threadIdx.x / groups, cg = threadIdx.x - pl * groups;
  const int64_t p0 = (int64_t)blockIdx.x * kHeadPix;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float sl = 0.f, sg = 0.f;
  // whole chunks: eight pixels' loads in flight (15 us for 16 x 256 x 256 pixels of 32
  // channels; one at a time 34 us)
  const int64_t end = p0 + kHeadPix < n_pix ? p0 + kHeadPix : n_pix;
  int64_t p = p0 + pl;
  auto add = [&](float gv, float lv, const uint4 &v) {
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[2 * q] += gv * bf2f((uint16_t)(u[q] & 0xffffu));
      a[2 * q + 1] += gv * bf2f((uint16_t)(u[q] >> 16));
    }
    if (cg == 0) { sl += lv; sg += gv; }
  };
  for (; p + 7 * lanes < end; p += 8 * lanes) {
    float gv[8], lv[8];
    uint4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      gv[i] = g[p + i * lanes];
      lv[i] = l[p + i * lanes];
      v[i] = load_any16(x + (p + i * lanes) * x_cs + cg * 8);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) add(gv[i], lv[i], v[i]);
  }
  for (; p < end; p += lanes) add(g[p], l[p], load_any16(x + p * x_cs + cg * 8));
#pragma unroll
  for (int j = 0; j < 8; ++j) red[threadIdx.x * 8 + j] = a[j];
  red_l[threadIdx.x] = sl;
  red_g[threadIdx.x] = sg;
  __syncthreads();
  if (threadIdx.x < (unsigned)c) {
    const int ch = threadIdx.x, g8 = ch >> 3, j = ch & 7;
    float s = 0.f;
    for (int q = 0; q < lanes; ++q) s += red[(q * groups + g8) * 8 + j];
    partial[(int64_t)blockIdx.x * (2 + c) + 2 + ch] = s;
  }
  if (threadIdx.x == 0) {
    float s1 = 0.f, s2 = 0.f;
    for (int q = 0; q < lanes; ++q) { s1 += red_l[q * groups]; s2 += red_g[q * groups]; }
    partial[(int64_t)blockIdx.x * (2 + c)] = s1;
    partial[(int64_t)blockIdx.x * (2 + c) + 1] = s2;
  }
}

// (eight threads per sum, one per partial of strided_sum's order)
__global__ __launch_bounds__(256) void head_loss_final(const float *partial, int blocks, int c, float *loss, float *dw,
                                                       float *db) {
  __shared__ float part[8][33];
  const int j = threadIdx.x >> 5, i = threadIdx.x & 31, k = blockIdx.x * 32 + i;
  float v = 0.f;
  if (k < 2 + c)
    for (int q = j; q < blocks; q += 8) v += partial[(int64_t)q * (2 + c) + k];
  part[j][i] = v;
  __syncthreads();
  if (threadIdx.x >= 32 || k >= 2 + c) return;
  const float s =
      ((part[0][i] + part[1][i]) + (part[2][i] + part[3][i])) + ((part[4][i] + part[5][i]) + (part[6][i] + part[7][i]));
  if (k == 0) loss[0] = s;
  else if (k == 1) { if (db) db[0] = s; }
  else if (dw) dw[k - 2] = s;
}

__global__ void adam_kernel(float *p, const float *g, float *m, float *v, uint16_t *pb, int64_t n, float lr, float b1,
                            float b2, float eps, float c1, float c2) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    if (pb) pb[i] = f2bf(pi);
  }
}

__global__ void to_bf16_kernel(const float *x, uint16_t *y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = f2bf(x[i]);
}
__global__ void to_f32_kernel(const uint16_t *x, float *y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = bf2f(x[i]);
}

static int grid1d(int64_t n) {
  int64_t b = (n + 255) / 256;
  return (int)(b < 1 ? 1 : (b > 16384 ? 16384 : b));
}
static int launched() { return hipGetLastError() == hipSuccess ? 0 : -100; }
static bool ok8(int v) { return v > 0 && v % 8 == 0; }
// channels co .. co + c of a pixel are whole aligned vectors of eight
static bool vec8(const uint16_t *p, int c, int cs, int co) {
  return reinterpret_cast<uintptr_t>(p) % 16 == 0 && c % 8 == 0 && cs % 8 == 0 && co % 8 == 0;
}

}  // namespace unet

using namespace unet;

// Split-K partial sums of the allocation-free weight gradient: a file-scope
// device array, one copy per GPU, held until the process ends.  Host code
// never uses its name as an address: the address comes from
// hipGetSymbolAddress, once per device, with that device current.
constexpr int64_t kStaticScratchFloats = (int64_t)4 << 20;  // 16 MiB
static __device__ __align__(256) float scratch[kStaticScratchFloats];

static float *scratch_ptr_current_device() {
  static std::mutex mu;
  static float *ptrs[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptrs[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    ptrs[dev] = static_cast<float *>(p);
  }
  return ptrs[dev];
}

// A channel slice [co, co + c) of a tensor with cs channels per pixel lies
// inside the tensor.
static bool slice_ok(int co, int c, int cs) { return co >= 0 && c >= 1 && (int64_t)co + c <= cs; }

extern "C" {

int unet_mfma_probe(const uint16_t *A, const uint16_t *B, float *C, void *s) {
  mfma_probe_kernel<<<1, 64, 0, (hipStream_t)s>>>(A, B, C);
  return launched();
}

int unet_conv3x3_fwd(const uint16_t *x, int n, int h, int w, int cin, int x_cs, int x_co, const uint16_t *wgt,
                     const float *bias, int cout, uint16_t *y, int y_cs, int y_co, int relu, void *s) {
  if (!x || !wgt || !y || n < 1 || h < 1 || w < 1 || !ok8(cin) || x_cs % 8 || x_co % 8 ||
      !slice_ok(x_co, cin, x_cs) || !slice_ok(y_co, cout, y_cs))
    return -1;
  GemmArgs a{x, n, h, w, cin, x_cs, x_co, wgt, bias, cout, y, y_cs, y_co, relu};
  launch_conv3x3(a, (int64_t)n * h * w, (hipStream_t)s);
  return launched();
}

static void launch_relu_bwd(const uint16_t *y, int64_t n_pix, int c, int y_cs, int y_co, uint16_t *dy, int dy_cs,
                            int dy_co, hipStream_t s) {
  if (c % 8 == 0 && y_cs % 8 == 0 && y_co % 8 == 0 && dy_cs % 8 == 0 && dy_co % 8 == 0)
    relu_bwd_vec<<<grid1d(n_pix * (c / 8)), 256, 0, s>>>(y, n_pix, c / 8, y_cs, y_co, dy, dy_cs, dy_co);
  else
    relu_bwd_kernel<<<grid1d(n_pix * c), 256, 0, s>>>(y, n_pix, c, y_cs, y_co, dy, dy_cs, dy_co);
}

int unet_conv3x3_relu_bwd_data(const uint16_t *dy, int n, int h, int w, int cout, int dy_cs, int dy_co,
                               const uint16_t *wt, int cin, uint16_t *dx, int dx_cs, int dx_co, const uint16_t *act,
                               int act_cs, int act_co, void *s) {
  if (!dy || !wt || !dx || !act || n < 1 || h < 1 || w < 1 || !ok8(cout) || dy_cs % 8 || dy_co % 8 ||
      !slice_ok(dy_co, cout, dy_cs) || !slice_ok(dx_co, cin, dx_cs) || !slice_ok(act_co, cin, act_cs))
    return -1;
  GemmArgs a{dy, n, h, w, cout, dy_cs, dy_co, wt, nullptr, cin, dx, dx_cs, dx_co, 0, act, act_cs, act_co};
  const int64_t P = (int64_t)n * h * w;
  if (!launch_conv3x3(a, P, (hipStream_t)s))
    launch_relu_bwd(act, P, cin, act_cs, act_co, dx, dx_cs, dx_co, (hipStream_t)s);
  return launched();
}

int unet_conv3x3_flip(const uint16_t *wgt, int cout, int cin, uint16_t *wt, void *s) {
  if (!wgt || !wt || cout < 1 || cin < 1) return -1;
  conv_flip<<<grid1d((int64_t)cout * 9 * cin), 256, 0, (hipStream_t)s>>>(wgt, cout, cin, wt);
  return launched();
}

int64_t unet_wgrad_scratch_floats(int n, int h, int w, int cin, int cout, int taps) {
  const int64_t P = (int64_t)n * h * w;
  const int64_t kb = (P + kWgradPix - 1) / kWgradPix;
  const int64_t wpart = kb * (int64_t)cout * cin * taps;
  const int64_t bpart = kb * (taps == 4 ? 4 : 1) * (int64_t)cout;  // bias partials follow
  return wpart + bpart;
}

int unet_conv3x3_wgrad(const uint16_t *x, int n, int h, int w, int cin, int x_cs, int x_co, const uint16_t *dy,
                       int cout, int dy_cs, int dy_co, float *dw, float *db, float *partial, int accumulate,
                       void *s) {
  if (!x || !dy || !dw || !partial || n < 1 || h < 1 || w < 1 || !ok8(cin) || !ok8(cout) || x_cs % 8 ||
      x_co % 8 || dy_cs % 8 || dy_co % 8 || x_co + cin > x_cs || dy_co + cout > dy_cs)
    return -1;
  const int64_t P = (int64_t)n * h * w;
  const int kb = (int)((P + kWgradPix - 1) / kWgradPix);
  const int64_t wpart = (int64_t)kb * cout * 9 * cin;
  WgradArgs a{x, n, h, w, cin, x_cs, x_co, dy, cout, dy_cs, dy_co, partial, 9 * cin, db ? partial + wpart : nullptr};
  launch_wgrad<0>(a, kb, (hipStream_t)s);
  launch_wgrad_reduce(partial, kb, 1, cout, 9 * cin, dw, accumulate, partial + wpart, kb, db, (hipStream_t)s);
  return launched();
}

int unet_conv3x3_wgrad_noalloc(const uint16_t *x, int n, int h, int w, int cin, int x_cs, int x_co,
                               const uint16_t *dy, int cout, int dy_cs, int dy_co, float *dw, float *db,
                               int accumulate, void *s) {
  if (!x || !dy || !dw || n < 1 || h < 1 || w < 1 || !ok8(cin) || !ok8(cout) || x_cs % 8 || x_co % 8 ||
      dy_cs % 8 || dy_co % 8 || !slice_ok(x_co, cin, x_cs) || !slice_ok(dy_co, cout, dy_cs))
    return -1;
  if (unet_wgrad_scratch_floats(n, h, w, cin, cout, 9) > kStaticScratchFloats) return -2;
  float *part = scratch_ptr_current_device();
  if (!part) return -100;
  return unet_conv3x3_wgrad(x, n, h, w, cin, x_cs, x_co, dy, cout, dy_cs, dy_co, dw, db, part, accumulate, s);
}

int unet_relu_bwd(const uint16_t *y, int n_pix, int c, int y_cs, int y_co, uint16_t *dy, int dy_cs, int dy_co,
                  void *s) {
  if (!y || !dy || n_pix < 1 || !slice_ok(y_co, c, y_cs) || !slice_ok(dy_co, c, dy_cs)) return -1;
  launch_relu_bwd(y, n_pix, c, y_cs, y_co, dy, dy_cs, dy_co, (hipStream_t)s);
  return launched();
}

int unet_maxpool_fwd(const uint16_t *x, int n, int h, int w, int c, int x_cs, int x_co, uint16_t *y, int y_cs,
                     int y_co, void *s) {
  if (!x || !y || n < 1 || h < 2 || w < 2 || (h & 1) || (w & 1) || !slice_ok(x_co, c, x_cs) ||
      !slice_ok(y_co, c, y_cs))
    return -1;
  const int64_t vectors = (int64_t)n * h * w * c / 32;
  if (vec8(x, c, x_cs, x_co) && vec8(y, c, y_cs, y_co) && vectors < ((int64_t)1 << 31))
    maxpool_fwd_vec<<<(unsigned)((vectors + 255) / 256), 256, 0, (hipStream_t)s>>>(x, (unsigned)vectors, w, c / 8, x_cs,
                                                                                   x_co, y, y_cs, y_co);
  else
    maxpool_fwd_kernel<<<grid1d((int64_t)n * h * w * c / 4), 256, 0, (hipStream_t)s>>>(x, n, h, w, c, x_cs, x_co, y,
                                                                                       y_cs, y_co);
  return launched();
}

static int maxpool_bwd(const uint16_t *x, int n, int h, int w, int c, int x_cs, int x_co, const uint16_t *dy, int dy_cs,
                       int dy_co, uint16_t *dx, int dx_cs, int dx_co, int accumulate, int relu, void *s) {
  if (!x || !dy || !dx || n < 1 || h < 2 || w < 2 || (h & 1) || (w & 1) || !slice_ok(x_co, c, x_cs) ||
      !slice_ok(dy_co, c, dy_cs) || !slice_ok(dx_co, c, dx_cs))
    return -1;
  const int64_t vectors = (int64_t)n * h * w * c / 32;
  if (vec8(x, c, x_cs, x_co) && vec8(dy, c, dy_cs, dy_co) && vec8(dx, c, dx_cs, dx_co) && vectors < ((int64_t)1 << 31)) {
    maxpool_bwd_vec<<<(unsigned)((vectors + 255) / 256), 256, 0, (hipStream_t)s>>>(
        x, (unsigned)vectors, w, c / 8, x_cs, x_co, dy, dy_cs, dy_co, dx, dx_cs, dx_co, accumulate, relu);
    return launched();
  }
  maxpool_bwd_kernel<<<grid1d((int64_t)n * h * w * c / 4), 256, 0, (hipStream_t)s>>>(
      x, n, h, w, c, x_cs, x_co, dy, dy_cs, dy_co, dx, dx_cs, dx_co, accumulate);
  if (relu) launch_relu_bwd(x, (int64_t)n * h * w, c, x_cs, x_co, dx, dx_cs, dx_co, (hipStream_t)s);
  return launched();
}

int unet_maxpool_bwd(const uint16_t *x, int n, int h, int w, int c, int x_cs, int x_co, const uint16_t *dy,
                     int dy_cs, int dy_co, uint16_t *dx, int dx_cs, int dx_co, int accumulate, void *s) {
  return maxpool_bwd(x, n, h, w, c, x_cs, x_co, dy, dy_cs, dy_co, dx, dx_cs, dx_co, accumulate, 0, s);
}

int unet_maxpool_relu_bwd(const uint16_t *x, int n, int h, int w, int c, int x_cs, int x_co, const uint16_t *dy,
                          int dy_cs, int dy_co, uint16_t *dx, int dx_cs, int dx_co, int accumulate, void *s) {
  return maxpool_bwd(x, n, h, w, c, x_cs, x_co, dy, dy_cs, dy_co, dx, dx_cs, dx_co, accumulate, 1, s);
}

int unet_upconv_fwd(const uint16_t *x, int n, int h, int w, int cin, int x_cs, int x_co, const uint16_t *wgt,
                    const float *bias, int cout, uint16_t *y, int y_cs, int y_co, void *s) {
  if (!x || !wgt || !y || n < 1 || h < 1 || w < 1 || !ok8(cin) || x_cs % 8 || x_co % 8 ||
      !slice_ok(x_co, cin, x_cs) || !slice_ok(y_co, cout, y_cs))
    return -1;
  GemmArgs a{x, n, h, w, cin, x_cs, x_co, wgt, bias, cout, y, y_cs, y_co, 0};
  const int64_t P = (int64_t)n * h * w;
  if (cin % 16 == 0 && direct_fits(a, P, 4)) {
    // 64 pixels a wave once that leaves 512 waves: weights read half as often.  64 -> 32
    // channels on 16 x 128 x 128 47 us with 32 pixels, 35 us with 64 (22 us for its
    // bytes); 256 -> 128 on 8 x 32 x 32 (1024 tiles of 32 x 32) 15 and 12 us.
    if ((P + 31) / 32 * ((cout + 31) / 32) >= 1024) launch_direct<3, 2, 4>(a, P, (hipStream_t)s);
    else launch_direct<3, 1, 4>(a, P, (hipStream_t)s);
  } else {
    launch_gather<1>(a, P, 4, (hipStream_t)s);
  }
  return launched();
}

static int upconv_bwd_data(const uint16_t *dy, int n, int h, int w, int cout, int dy_cs, int dy_co,
                           const uint16_t *wgt, int cin, uint16_t *wt, uint16_t *dx, int dx_cs, int dx_co,
                           const uint16_t *act, int act_cs, int act_co, void *s) {
  if (!dy || !wgt || !wt || !dx || n < 1 || h < 1 || w < 1 || !ok8(cout) || dy_cs % 8 || dy_co % 8 ||
      !slice_ok(dy_co, cout, dy_cs) || !slice_ok(dx_co, cin, dx_cs))
    return -1;
  up_rearrange<<<grid1d((int64_t)cout * 4 * cin), 256, 0, (hipStream_t)s>>>(wgt, cout, cin, wt);
  // A = dy over the 2h x 2w grid gathered at 2p + tap, output grid h x w
  GemmArgs a{dy, n, h, w, cout, dy_cs, dy_co, wt, nullptr, cin, dx, dx_cs, dx_co, 0, act, act_cs, act_co};
  const int64_t P = (int64_t)n * h * w;
  if (cout % 16 == 0 && direct_fits(a, P, 4)) {
    launch_direct_tiles<4>(a, P, (hipStream_t)s);
  } else {
    launch_gather<2>(a, P, 1, (hipStream_t)s);
    if (act) launch_relu_bwd(act, P, cin, act_cs, act_co, dx, dx_cs, dx_co, (hipStream_t)s);
  }
  return launched();
}

int unet_upconv_bwd_data(const uint16_t *dy, int n, int h, int w, int cout, int dy_cs, int dy_co,
                         const uint16_t *wgt, int cin, uint16_t *wt, uint16_t *dx, int dx_cs, int dx_co, void *s) {
  return upconv_bwd_data(dy, n, h, w, cout, dy_cs, dy_co, wgt, cin, wt, dx, dx_cs, dx_co, nullptr, 0, 0, s);
}

int unet_upconv_relu_bwd_data(const uint16_t *dy, int n, int h, int w, int cout, int dy_cs, int dy_co,
                              const uint16_t *wgt, int cin, uint16_t *wt, uint16_t *dx, int dx_cs, int dx_co,
                              const uint16_t *act, int act_cs, int act_co, void *s) {
  if (!act || !slice_ok(act_co, cin, act_cs)) return -1;
  return upconv_bwd_data(dy, n, h, w, cout, dy_cs, dy_co, wgt, cin, wt, dx, dx_cs, dx_co, act, act_cs, act_co, s);
}

int unet_upconv_wgrad(const uint16_t *x, int n, int h, int w, int cin, int x_cs, int x_co, const uint16_t *dy,
                      int cout, int dy_cs, int dy_co, float *dw, float *db, float *partial, void *s) {
  if (!x || !dy || !dw || !partial || n < 1 || h < 1 || w < 1 || !ok8(cin) || !ok8(cout) || x_cs % 8 ||
      x_co % 8 || dy_cs % 8 || dy_co % 8 || x_co + cin > x_cs || dy_co + cout > dy_cs)
    return -1;
  const int64_t P = (int64_t)n * h * w;
  const int kb = (int)((P + kWgradPix - 1) / kWgradPix);
  const int64_t wpart = (int64_t)kb * 4 * cout * cin;
  WgradArgs a{x, n, h, w, cin, x_cs, x_co, dy, cout, dy_cs, dy_co, partial, cin, db ? partial + wpart : nullptr};
  launch_wgrad<1>(a, kb, (hipStream_t)s);
  launch_wgrad_reduce(partial, kb, 4, cout, cin, dw, 0, partial + wpart, (int64_t)kb * 4, db, (hipStream_t)s);
  return launched();
}

int unet_head_fwd(const uint16_t *x, int n_pix, int c, int x_cs, const float *w, const float *b, float *sat,
                  void *s) {
  if (!x || !w || !b || !sat || n_pix < 1 || c < 1 || c > 256 || 256 % c || c > x_cs) return -1;
  head_fwd_kernel<<<grid1d(n_pix), 256, 0, (hipStream_t)s>>>(x, n_pix, c, x_cs, w, b, sat);
  return launched();
}

int64_t unet_head_scratch_floats(int n_pix, int c) {
  const int64_t blocks = ((int64_t)n_pix + kHeadPix - 1) / kHeadPix;
  return 2 * (int64_t)n_pix + blocks * (2 + c);
}

static int head_loss_bwd(const uint16_t *x, int n_pix, int c, int x_cs, const float *w, const float *b,
                       const float *target, const uint8_t *mask, float scale, float *loss, uint16_t *dx,
                       float *dw, float *db, float *partial, int relu, void *s) {
  if (!x || !w || !b || !target || !mask || !loss || !partial || n_pix < 1 || c < 1 || c > 256 || 256 % c ||
      c > x_cs)
    return -1;
  float *g = partial, *l = partial + n_pix, *sums = partial + 2 * (int64_t)n_pix;
  const int blocks = (int)(((int64_t)n_pix + kHeadPix - 1) / kHeadPix);
  if (c <= 64 && vec8(x, c, x_cs, 0) && (!dx || vec8(dx, c, c, 0)))
    head_loss_pix_v<<<(unsigned)(((int64_t)n_pix + 255) / 256), 256, 0, (hipStream_t)s>>>(
        x, n_pix, c, x_cs, w, b, target, mask, scale, dx, g, l, relu);
  else {
    head_loss_pix<<<grid1d(n_pix), 256, 0, (hipStream_t)s>>>(x, n_pix, c, x_cs, w, b, target, mask, scale, dx, g, l);
    if (relu && dx) launch_relu_bwd(x, n_pix, c, x_cs, 0, dx, c, 0, (hipStream_t)s);
  }
  if ((c & 7) == 0 && (x_cs & 7) == 0)
    head_loss_sums_v<<<blocks, 256, 0, (hipStream_t)s>>>(x, n_pix, c, x_cs, g, l, sums);
  else
    head_loss_sums<<<blocks, 256, 0, (hipStream_t)s>>>(x, n_pix, c, x_cs, g, l, sums);
  head_loss_final<<<(2 + c + 31) / 32, 256, 0, (hipStream_t)s>>>(sums, blocks, c, loss, dw, db);
  return launched();
}

int unet_head_loss_bwd(const uint16_t *x, int n_pix, int c, int x_cs, const float *w, const float *b,
                       const float *target, const uint8_t *mask, float scale, float *loss, uint16_t *dx,
                       float *dw, float *db, float *partial, void *s) {
  return head_loss_bwd(x, n_pix, c, x_cs, w, b, target, mask, scale, loss, dx, dw, db, partial, 0, s);
}

int unet_head_loss_relu_bwd(const uint16_t *x, int n_pix, int c, int x_cs, const float *w, const float *b,
                       const float *target, const uint8_t *mask, float scale, float *loss, uint16_t *dx,
                       float *dw, float *db, float *partial, void *s) {
  return head_loss_bwd(x, n_pix, c, x_cs, w, b, target, mask, scale, loss, dx, dw, db, partial, 1, s);
}

int unet_adam(float *p, const float *g, float *m, float *v, uint16_t *p_bf16, int64_t count, float lr, float beta1,
              float beta2, float eps, int step, void *s) {
  if (!p || !g || !m || !v || count < 1 || step < 1) return -1;
  const float c1 = 1.f - powf(beta1, (float)step), c2 = 1.f - powf(beta2, (float)step);
  adam_kernel<<<grid1d(count), 256, 0, (hipStream_t)s>>>(p, g, m, v, p_bf16, count, lr, beta1, beta2, eps, c1, c2);
  return launched();
}

int unet_to_bf16(const float *x, uint16_t *y, int64_t count, void *s) {
  if (!x || !y || count < 1) return -1;
  to_bf16_kernel<<<grid1d(count), 256, 0, (hipStream_t)s>>>(x, y, count);
  return launched();
}

int unet_to_f32(const uint16_t *x, float *y, int64_t count, void *s) {
  if (!x || !y || count < 1) return -1;
  to_f32_kernel<<<grid1d(count), 256, 0, (hipStream_t)s>>>(x, y, count);
  return launched();
}

}  // extern "C"
