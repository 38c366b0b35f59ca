// Surrogate MLP 7 -> 256 -> 256 -> 1 (GELU, erf form) on gfx950.
//
// Numerics: FP32 master weights; BF16 (round to nearest even) copies of the
// weights and of every layer input enter the products, which accumulate in
// FP32.  The forward 256x256 product runs on the BF16 matrix cores
// (v_mfma_f32_32x32x16_bf16).  The backward products keep the gradient
// signals in FP32 and run on the FP32 matrix cores (v_mfma_f32_16x16x4_f32);
// the BF16-valued weights and activations enter them exactly.  Rounding an
// activation to BF16 is treated as the identity in the backward pass.
//
// Kernels of one training step (all on the caller's stream):
//   k_mlp<.., true>  forward and, in the same block, backward of a tile of
//                    rows: layer 1 (VALU), layer 2 (MFMA), output and its
//                    gradient, dz2, dh1 = dz2 W1^T (MFMA), dz1, and the tile's
//                    partial sums of the small gradients
//   k_mlp_wgrad      parts of gW1 = a1^T dz2 (MFMA) over ranges of rows, and the
//                    fixed-order sums of the tiles' partials
//   k_mlp_adam       adds gW1's parts; Adam with bias correction, elementwise
// The forward pass is k_mlp<.., false> alone.
// Every sum has a fixed order, so results are bitwise reproducible.
#include <algorithm>

#include "common.h"

namespace sl {
namespace {

constexpr int kIn = SL_MLP_IN;
constexpr int kH = SL_MLP_HID;
constexpr int kNetT = 512;     // threads of a forward / backward block: wave w owns hidden columns [32 w, 32 w + 32)
constexpr int kThr = 256;      // threads of the other blocks
constexpr int kMaxSplit = 16;  // row ranges of gW1
constexpr int kMaxBatch = SL_MLP_MAX_BATCH;

// parameter offsets (floats) in the packed vector
constexpr int oW0 = 0;
constexpr int oB0 = oW0 + kIn * kH;
constexpr int oW1 = oB0 + kH;
constexpr int oB1 = oW1 + kH * kH;
constexpr int oW2 = oB1 + kH;
constexpr int oB2 = oW2 + kH;
static_assert(oB2 + 1 == SL_MLP_NPARAM, "parameter layout");

// per-tile partial sums written by k_mlp<.., true>: gW0 | gb0 | gb1 | gW2 | gb2
constexpr int pW0 = 0;
constexpr int pB0 = pW0 + kIn * kH;
constexpr int pB1 = pB0 + kH;
constexpr int pW2 = pB1 + kH;
constexpr int pB2 = pW2 + kH;
constexpr int kPart = pB2 + kH;   // gb2 sits in the first slot of its 256-wide group

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Round to the nearest BF16 value, ties to even (finite inputs).
__device__ __forceinline__ unsigned short bf16_bits(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16r(float f) { return __uint_as_float((unsigned)bf16_bits(f) << 16); }

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
// d/dz [z Phi(z)] = Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// Rows per block: few rows where the batch would leave CUs idle otherwise, as
// many as an MFMA tile where it fills them (16 instead of 32 rows: 14.0 against
// 13.3 us for the forward pass of 8190 rows, 78 against 69 us for a step).  A
// row's result does not depend on it (the rows of an MFMA tile are
// independent, and every sum over a row's columns has the same order).
int rows_per_block(int batch) { return batch <= 2048 ? 8 : batch <= 4096 ? 16 : 32; }
int row_tiles(int batch) { return (batch + rows_per_block(batch) - 1) / rows_per_block(batch); }
// Tiles that a workspace of this batch has room for: the most of any batch up to
// it.  A caller may size one workspace for its largest batch and train smaller
// ones in it (the calls take no size), and 2048 rows have more tiles than 2049.
int tile_room(int batch) { return batch <= 2048 ? row_tiles(batch) : std::max(row_tiles(2048), row_tiles(batch)); }
static_assert(4096 / 16 <= 2048 / 8, "16-row tiles never outnumber the 8-row tiles of 2048 rows");
// Row ranges of gW1: 128 rows or more each (64: 31.4 against 29.9 us for a step on 1024 rows).
int row_splits(int batch) { return std::min(kMaxSplit, std::max(1, batch / 128)); }

// Workspace of the training step (the forward pass needs none).
struct Ws {
  unsigned short* a1;       // [B][256] BF16 bits of h1
  float* dz2;               // [B][256]
  float* part;              // [tiles][kPart]
  float* small;             // [kPart] their sums
  float* gw1;               // [kMaxSplit][256][256] parts of gW1
  double* lossp;            // [tiles]
  double* loss;             // [1]
};

size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

size_t carve(int batch, unsigned char* base, Ws* w) {
  const size_t B = (size_t)(batch > 0 ? batch : 0);
  const size_t tiles = (size_t)tile_room(batch);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align256(bytes);
    return base ? base + o : nullptr;
  };
  Ws t;
  t.a1 = reinterpret_cast<unsigned short*>(take(sizeof(unsigned short) * B * kH));
  t.dz2 = reinterpret_cast<float*>(take(sizeof(float) * B * kH));
  t.part = reinterpret_cast<float*>(take(sizeof(float) * tiles * kPart));
  t.small = reinterpret_cast<float*>(take(sizeof(float) * kPart));
  t.gw1 = reinterpret_cast<float*>(take(sizeof(float) * (size_t)kMaxSplit * kH * kH));
  t.lossp = reinterpret_cast<double*>(take(sizeof(double) * tiles));
  t.loss = reinterpret_cast<double*>(take(sizeof(double)));
  if (w) *w = t;
  return off;
}

struct NetArgs {
  const float* params;
  const float* x;
  const float* ytrue;   // training only
  int B, tiles;
  float inv_b2;         // 2 / B
  float* y;             // forward output
  Ws w;
};

// Forward and, with TRAIN, backward of tiles of R rows.  Wave w owns the hidden
// columns [32 w, 32 w + 32) in layer 2 (one 32 x 32 MFMA tile per 16 inputs, of
// which the first R rows count) and the inputs [32 w, 32 w + 32) of dh1.
//
// What bounds it is latency (a step of the search trains on 1024 rows and
// screens 8190): the error functions of a thread's rows, the reads of W1 and
// the barriers between the layers.  So the block reads W1 itself, in FP32 and
// rounding as it goes, into registers that the tiles it walks share, with the
// reads issued before layer 1 (a separate kernel wrote BF16 and FP32
// transposes first: 5 us and a launch in front of every call); eight waves
// share a tile's error functions (four did); and the backward pass follows in
// the same block, where the activations and derivatives are still in LDS and
// registers (they went through memory to a second kernel, 16 B x 256 a row).
// Forward of 8190 rows: 24 (5 + 19) -> 14 us; forward and backward of 1024
// rows: 64 (6 + 28 + 30) -> 20 us.
template <int R, bool TRAIN>
__global__ void __launch_bounds__(kNetT) k_mlp(NetArgs a) {
  constexpr int kPitch = kH + 8;   // BF16 elements per LDS row
  constexpr int kP = kH + 4;       // floats per LDS row of dz2
  constexpr int RP = R < 16 ? 16 : R;   // rows of the FP32 MFMA tiles
  constexpr int NR = R / 2;        // accumulator elements that hold rows below R
  __shared__ __attribute__((aligned(16))) unsigned short A1s[32 * kPitch];
  __shared__ __attribute__((aligned(16))) float D2s[TRAIN ? RP * kP : 1];
  __shared__ float G1s[TRAIN ? R * kH : 1];   // gelu'(z1)
  __shared__ float xs[R * kIn], yp[8][32], g3s[32];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int li = lane & 31, lg = lane >> 5;
  const int j = 32 * wv + li;      // this lane's hidden column of layer 2
  // layer 2's B operand, lane: column j, inputs 16 kk + 8 lg + e
  union Frag {
    bf16x8 v;
    unsigned u[4];
  };
  Frag bw[kH / 16];
#pragma unroll
  for (int kk = 0; kk < kH / 16; ++kk)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* W = a.params + oW1 + (16 * kk + 8 * lg + 2 * e) * kH + j;
      bw[kk].u[e] = (unsigned)bf16_bits(W[0]) | ((unsigned)bf16_bits(W[kH]) << 16);
    }
  const int n = tid & (kH - 1);    // this thread's hidden column of layer 1
  float w0[kIn];
#pragma unroll
  for (int k = 0; k < kIn; ++k) w0[k] = bf16r(a.params[oW0 + k * kH + n]);
  const float b0 = a.params[oB0 + n];
  const float b1 = a.params[oB1 + j];
  const float w2 = bf16r(a.params[oW2 + j]);
  const float b2 = a.params[oB2];
  for (int tile = blockIdx.x; tile < a.tiles; tile += gridDim.x) {
    const int row0 = tile * R;
    const int nrow = min(R, a.B - row0);
    for (int e = tid; e < R * kIn; e += kNetT) xs[e] = e < nrow * kIn ? bf16r(a.x[(size_t)row0 * kIn + e]) : 0.0f;
    __syncthreads();   // (also: the last tile's readers of A1s and yp are done)
    // ---- layer 1: z1 = bf16(x) bf16(W0) + b0, a1 = bf16(gelu(z1))
#pragma unroll 4
    for (int q = 0; q < R / 2; ++q) {
      const int r = 2 * q + (tid >> 8);
      float z = b0;
#pragma unroll
      for (int k = 0; k < kIn; ++k) z = fmaf(xs[r * kIn + k], w0[k], z);
      const unsigned short hb = r < nrow ? bf16_bits(gelu(z)) : (unsigned short)0;
      A1s[r * kPitch + n] = hb;
      if constexpr (TRAIN) {
        G1s[r * kH + n] = gelu_grad(z);
        if (r < nrow) a.w.a1[(size_t)(row0 + r) * kH + n] = hb;
      }
    }
    __syncthreads();
    // ---- layer 2 on the BF16 matrix cores: z2 = a1 W1 (+ b1 below)
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    const unsigned short* arow = A1s + li * kPitch + 8 * lg;
#pragma unroll
    for (int kk = 0; kk < kH / 16; ++kk) {
      const bf16x8 av = *reinterpret_cast<const bf16x8*>(arow + 16 * kk);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bw[kk].v, acc, 0, 0, 0);
    }
    // ---- a2 = bf16(gelu(z2 + b1)) and the partial y over this wave's columns.
    // Accumulator element r of a 32x32 tile sits at row 8(r/4) + 4 lg + r%4,
    // column li.
    float h2[TRAIN ? NR : 1], g2[TRAIN ? NR : 1];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const float z = acc[r] + b1;
      const float h = bf16r(gelu(z));
      if constexpr (TRAIN) {
        h2[r] = h;
        g2[r] = gelu_grad(z);
      }
      float v = h * w2;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);   // the 32 columns (lanes sharing lg)
      if (li == 0) yp[wv][8 * (r >> 2) + 4 * lg + (r & 3)] = v;
    }
    __syncthreads();
    if (tid < 64) {
      double lp = 0.0;
      float g3 = 0.0f;
      if (tid < nrow) {
        const float yv = ((((b2 + yp[0][tid]) + yp[1][tid]) + (yp[2][tid] + yp[3][tid])) + (yp[4][tid] + yp[5][tid])) +
                         (yp[6][tid] + yp[7][tid]);
        const size_t b = (size_t)row0 + tid;
        if constexpr (TRAIN) {
          const float d = yv - a.ytrue[b];
          g3 = a.inv_b2 * d;
          lp = (double)d * (double)d;
        } else {
          a.y[b] = yv;
        }
      }
      if constexpr (TRAIN) {
        if (tid < 32) g3s[tid] = g3;
        lp = wave_sum(lp);   // fixed order
        if (tid == 0) a.w.lossp[tile] = lp;
      }
    }
    if constexpr (TRAIN) {
      __syncthreads();
      float* part = a.w.part + (size_t)tile * kPart;
      // ---- dz2 = g3 bf16(W2) gelu'(z2); partial gb1 and gW2 of this tile (rows past nrow have g3 = 0)
      float sb1 = 0.0f, sw2 = 0.0f;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int i = 8 * (r >> 2) + 4 * lg + (r & 3);
        const float g3 = g3s[i];
        const float d = i < nrow ? g3 * w2 * g2[r] : 0.0f;
        if (i < nrow) {
          a.w.dz2[(size_t)(row0 + i) * kH + j] = d;
          sw2 = fmaf(h2[r], g3, sw2);
        }
        sb1 += d;
        D2s[i * kP + j] = d;
      }
      sb1 += __shfl_xor(sb1, 32, 64);
      sw2 += __shfl_xor(sw2, 32, 64);
      if (lg == 0) {
        part[pB1 + j] = sb1;
        part[pW2 + j] = sw2;
      }
      if (tid == 0) {
        float s = 0.0f;
        for (int r = 0; r < nrow; ++r) s += g3s[r];
        part[pB2] = s;
      }
      __syncthreads();
      // ---- dh1[i][k] = sum_j dz2[i][j] W1[k][j] on the FP32 matrix cores.
      // f32 16x16x4: A element (row l%16, inner l/16); B element (inner l/16, column
      // l%16); accumulator element r at row 4(l/16) + r, column l%16.  Both operands
      // take the inner index 16 s + 4 (l/16) + m in step (s, m), so that a lane's
      // four steps are one 16-byte read of each.
      const int lc = lane & 15, lq = lane >> 4;
      constexpr int MT = RP / 16;
      f32x4 dh[MT][2];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) dh[m][c][r] = 0.0f;
      const float* Wr = a.params + oW1 + (size_t)(32 * wv + lc) * kH + 4 * lq;
#pragma unroll 8
      for (int s = 0; s < kH / 16; ++s) {
        f32x4 av[MT], bv[2];
#pragma unroll
        for (int m = 0; m < MT; ++m) av[m] = *reinterpret_cast<const f32x4*>(&D2s[(16 * m + lc) * kP + 16 * s + 4 * lq]);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) bv[c][e] = bf16r(Wr[(size_t)16 * c * kH + 16 * s + e]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int c = 0; c < 2; ++c)
              dh[m][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[m][e], bv[c][e], dh[m][c], 0, 0, 0);
      }
      // ---- dz1 = dh1 gelu'(z1); partial gb0 and gW0 of this tile
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int k = 32 * wv + 16 * c + lc;
        float sb0 = 0.0f, sw0[kIn];
#pragma unroll
        for (int q = 0; q < kIn; ++q) sw0[q] = 0.0f;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = 16 * m + 4 * lq + r;
            if (i < nrow) {   // (nrow <= R)
              const float dz1 = dh[m][c][r] * G1s[i * kH + k];
              sb0 += dz1;
#pragma unroll
              for (int q = 0; q < kIn; ++q) sw0[q] = fmaf(xs[i * kIn + q], dz1, sw0[q]);
            }
          }
        // add the four row groups (lanes lc, lc+16, lc+32, lc+48)
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
          sb0 += __shfl_xor(sb0, o, 64);
#pragma unroll
          for (int q = 0; q < kIn; ++q) sw0[q] += __shfl_xor(sw0[q], o, 64);
        }
        if (lq == 0) {
          part[pB0 + k] = sb0;
#pragma unroll
          for (int q = 0; q < kIn; ++q) part[pW0 + q * kH + k] = sw0[q];
        }
      }
      __syncthreads();   // xs, G1s and D2s are read before the next tile writes them
    }
  }
}

struct WgradArgs {
  int B, tiles, splits;
  Ws w;
};

// Blocks below 64 x splits: a 32 x 32 tile (inputs x outputs) of gW1 = a1^T dz2
// over one range of rows; the four waves take interleaved groups of 4 rows,
// summed in a fixed order, and k_mlp_adam adds the ranges' parts in order.  The
// ranges fill the chip (64 blocks walked the whole batch, one group's reads at
// a time, before: 25 us for 1024 rows; 7 us so).
// The other blocks: 64 columns of the tiles' partial sums each, the four waves
// a quarter of the tiles each; the first of them also sums the loss.
__global__ void __launch_bounds__(kThr) k_mlp_wgrad(WgradArgs a) {
  __shared__ float red[4][32][33];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if ((int)blockIdx.x < 64 * a.splits) {
    const int split = blockIdx.x / 64, t64 = blockIdx.x % 64;
    const int k0 = 32 * (t64 / 8), j0 = 32 * (t64 % 8);
    const int per = ((a.B + a.splits - 1) / a.splits + 15) / 16 * 16;
    const int lo = split * per, hi = min(a.B, lo + per);
    const int lc = lane & 15, lq = lane >> 4;
    f32x4 acc[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[m][n][r] = 0.0f;
    constexpr int U = 8;   // groups of rows in flight
    for (int b0 = lo + 4 * wv; b0 < hi; b0 += 16 * U) {
      float av[U][2], bv[U][2];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int b = b0 + 16 * u + lq;
        const bool on = b < hi;
        const unsigned short* a1r = a.w.a1 + (size_t)(on ? b : lo) * kH + k0 + lc;
        const float* d2r = a.w.dz2 + (size_t)(on ? b : lo) * kH + j0 + lc;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          av[u][m] = __uint_as_float(on ? (unsigned)a1r[16 * m] << 16 : 0u);
          bv[u][m] = on ? d2r[16 * m] : 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int n = 0; n < 2; ++n)
            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][m], bv[u][n], acc[m][n], 0, 0, 0);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wv][16 * m + 4 * lq + r][16 * n + lc] = acc[m][n][r];
    __syncthreads();
    float* g = a.w.gw1 + (size_t)split * kH * kH;
    for (int e = tid; e < 32 * 32; e += kThr) {
      const int i = e / 32, j = e % 32;
      g[(k0 + i) * kH + j0 + j] = (red[0][i][j] + red[1][i][j]) + (red[2][i][j] + red[3][i][j]);
    }
    return;
  }
  const int q = blockIdx.x - 64 * a.splits;
  const int c = q * 64 + lane;   // column of the partial table (kPart is a multiple of 64)
  const int per = (a.tiles + 3) / 4, t0 = wv * per, t1 = min(a.tiles, t0 + per);
  float s = 0.0f;
#pragma unroll 8
  for (int t = t0; t < t1; ++t) s += a.w.part[(size_t)t * kPart + c];
  float* sums = &red[0][0][0];
  sums[wv * 64 + lane] = s;
  __syncthreads();
  if (wv == 0) a.w.small[c] = (sums[lane] + sums[64 + lane]) + (sums[128 + lane] + sums[192 + lane]);
  if (q == 0 && wv == 1) {
    double l = 0.0;
    for (int t = lane; t < a.tiles; t += 64) l += a.w.lossp[t];
    l = wave_sum(l);
    if (lane == 0) *a.w.loss = l / (double)a.B;
  }
}

__global__ void __launch_bounds__(kThr) k_mlp_adam(float* __restrict__ p, float* __restrict__ m,
                                                   float* __restrict__ v, Ws w, int splits, float lr, float c1,
                                                   float c2, float* __restrict__ grads_out,
                                                   float* __restrict__ loss_out) {
  // 1 - beta written out: 1.0f - 0.999f is 1.0000467e-3 in FP32, not 1e-3
  constexpr float b1 = 0.9f, omb1 = 0.1f, b2 = 0.999f, omb2 = 0.001f, eps = 1e-8f;
  const int i = blockIdx.x * kThr + threadIdx.x;
  if (i == 0 && loss_out) *loss_out = (float)*w.loss;
  if (i >= SL_MLP_NPARAM) return;
  const float m0 = m[i], v0 = v[i], p0 = p[i];
  float gi;
  if (i >= oW1 && i < oB1) {
    float x[kMaxSplit];
#pragma unroll
    for (int s = 0; s < kMaxSplit; ++s) x[s] = s < splits ? w.gw1[(size_t)s * kH * kH + (i - oW1)] : 0.0f;
    gi = x[0];
#pragma unroll
    for (int s = 1; s < kMaxSplit; ++s)
      if (s < splits) gi += x[s];
  } else {
    gi = w.small[i < oB0 ? pW0 + i : i < oW1 ? pB0 + i - oB0 : i < oW2 ? pB1 + i - oB1 : i < oB2 ? pW2 + i - oW2 : pB2];
  }
  if (grads_out) grads_out[i] = gi;
  const float mi = b1 * m0 + omb1 * gi;
  const float vi = b2 * v0 + omb2 * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] = p0 - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// Blocks of the forward pass: the register copy of W1 is read once per block,
// so no more blocks than fit on the chip at once, each walking its tiles.
template <bool TRAIN>
int launch_net(const NetArgs& a, hipStream_t st) {
  const int blocks = std::min(a.tiles, TRAIN ? a.tiles : 2 * device_cus());
  switch (rows_per_block(a.B)) {
    case 8: k_mlp<8, TRAIN><<<blocks, kNetT, 0, st>>>(a); break;
    case 16: k_mlp<16, TRAIN><<<blocks, kNetT, 0, st>>>(a); break;
    default: k_mlp<32, TRAIN><<<blocks, kNetT, 0, st>>>(a); break;
  }
  return check_launch("k_mlp");
}

int validate(const void* params, const float* x, int batch, const void* ws) {
  SL_REQUIRE(batch >= 1 && batch <= kMaxBatch, "batch %d outside [1, %d]", batch, kMaxBatch);
  SL_REQUIRE(params && x && ws, "null pointer argument");
  return SL_OK;
}

}  // namespace
}  // namespace sl

using namespace sl;

extern "C" {

size_t sl_mlp_workspace_size(int batch) {
  if (batch < 0 || batch > kMaxBatch) {
    set_error("batch %d outside [0, %d]", batch, kMaxBatch);
    return 0;
  }
  return carve(batch, nullptr, nullptr);
}

int sl_mlp_forward(const float* params, const float* x, int batch, float* y, void* workspace, void* stream) {
  if (int rc = validate(params, x, batch, workspace)) return rc;
  SL_REQUIRE(y, "null output");
  return launch_net<false>(NetArgs{params, x, nullptr, batch, row_tiles(batch), 0.0f, y, Ws{}},
                           static_cast<hipStream_t>(stream));
}

int sl_mlp_forward_noalloc(const float* params, const float* x, int batch, float* y, void* stream) {
  SL_REQUIRE(batch >= 1 && batch <= kMaxBatch, "batch %d outside [1, %d]", batch, kMaxBatch);
  SL_REQUIRE(params && x && y, "null pointer argument");
  return launch_net<false>(NetArgs{params, x, nullptr, batch, row_tiles(batch), 0.0f, y, Ws{}},
                           static_cast<hipStream_t>(stream));
}

int sl_mlp_train_step(float* params, float* adam_m, float* adam_v, const float* x, const float* y, int batch,
                      float lr, int t, float* grads_out, float* loss_out, void* workspace, void* stream) {
  if (int rc = validate(params, x, batch, workspace)) return rc;
  SL_REQUIRE(adam_m && adam_v && y, "null pointer argument");
  SL_REQUIRE(t >= 1, "Adam step number t = %d must be >= 1", t);
  SL_REQUIRE(std::isfinite(lr) && lr > 0.0f, "learning rate must be finite and positive");
  hipStream_t st = static_cast<hipStream_t>(stream);
  Ws w;
  carve(batch, static_cast<unsigned char*>(workspace), &w);
  const int tiles = row_tiles(batch), splits = row_splits(batch);
  if (int rc = launch_net<true>(NetArgs{params, x, y, batch, tiles, (float)(2.0 / batch), nullptr, w}, st)) return rc;
  k_mlp_wgrad<<<64 * splits + kPart / 64, kThr, 0, st>>>(WgradArgs{batch, tiles, splits, w});
  if (int rc = check_launch("k_mlp_wgrad")) return rc;
  const double c1 = 1.0 / (1.0 - std::pow(0.9, t)), c2 = 1.0 / (1.0 - std::pow(0.999, t));
  k_mlp_adam<<<(SL_MLP_NPARAM + kThr - 1) / kThr, kThr, 0, st>>>(params, adam_m, adam_v, w, splits, lr, (float)c1,
                                                                 (float)c2, grads_out, loss_out);
  return check_launch("k_mlp_adam");
}

}  // extern "C"
