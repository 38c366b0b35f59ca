// Operator-level entry points: lens tracing, L, L^T, B, B^T and H^T H.
//
// These are the building blocks of the semilinear model (Rogers & Fiege 2011,
// Sec. 2.1-2.2, Eq. 7) exposed one call per operator.  The batched solver in
// solve.hip fuses the same operators into one persistent kernel.  Here one
// launch covers up to kBatch members (blockIdx.y), whose grid sides and packed
// offsets travel as a kernel argument: one launch per member left most of the
// chip idle and cost 16 members of a 128 x 128 image 48 launches per operator
// chain (trace 74, L 58, L^T 285 and H^T H 63 us in all).
#include <algorithm>
#include <climits>
#include <cstdarg>
#include <vector>

#include "common.h"

namespace sl {

static thread_local char g_err[512];

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}

// Members of one launch: grid sides and starts in the packed source vectors.
constexpr int kBatch = 64;
struct Batch {
  int ns[kBatch];
  long off[kBatch];
};

// The same for a launch of some members of the call, and which ones they are.
struct Picked {
  int ns[kBatch], id[kBatch];
  long off[kBatch];
};

// A subpixel's (u, v): 16 bytes in one access, 8-byte aligned as the caller's array.
struct alignas(8) UV {
  double u, v;
};

// ------------------------------------------------------------------ trace
// Bound by the FP64 trace (atan, atanh, two square roots and the divisions of
// one subpixel per thread); the lens's sines and cosines are taken once per
// block.  16 members of a 128 x 128 image with 2 x 2 subpixels: 27 us (16
// launches of 4.6 before).
__global__ void __launch_bounds__(256) k_trace(const double* __restrict__ genome, int nx, int ny, double pix, int nsub,
                                               Batch mb, double R, int rep, double* __restrict__ uv) {
  __shared__ Lens Ls;
  __shared__ int valid;
  const int m = blockIdx.y, ns = mb.ns[m];
  const int n2 = nsub * nsub;
  const long total = (long)nx * ny * n2;
  if (threadIdx.x == 0) {
    double g[7];
    for (int i = 0; i < 7; ++i) g[i] = genome[7 * m + i];
    valid = lens_valid(g);
    Ls = make_lens(g);
  }
  __syncthreads();
  const Lens L = Ls;
  const double h = 2.0 * R / (ns - 1);
  for (int i = 0; i < rep; ++i) {
    const long t = ((long)blockIdx.x * rep + i) * 256 + threadIdx.x;
    if (t >= total) return;
    double u = NAN, v = NAN;
    if (valid) {
      const int j = (int)(t / n2), k = (int)(t % n2);
      const int r = j / nx, c = j % nx;
      double x, y, bx, by;
      subpixel_xy(r, c, k / nsub, k % nsub, nx, ny, pix, nsub, x, y);
      lens_map(L, x, y, bx, by);
      const double uu = (bx + R) / h, vv = (by + R) / h;
      if (uu >= 0.0 && uu <= ns - 1 && vv >= 0.0 && vv <= ns - 1) {
        u = uu;
        v = vv;
      }
    }
    reinterpret_cast<UV*>(uv)[(long)m * total + t] = UV{u, v};
  }
}

// ------------------------------------------------------------------ L, L^T
// One thread per pixel; bound by the 16 n^2 bytes of positions it reads.
template <typename T>
__global__ void __launch_bounds__(256) k_apply_L(const double* __restrict__ uv, int J, int nsub, Batch mb,
                                                 const T* __restrict__ s_all, T* __restrict__ img) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x, m = blockIdx.y, ns = mb.ns[m];
  if (j >= J) return;
  const int n2 = nsub * nsub;
  const T* s = s_all + mb.off[m];
  const UV* p = reinterpret_cast<const UV*>(uv) + ((long)m * J + j) * n2;
  T acc = 0;
  for (int k = 0; k < n2; ++k) {
    const UV q = p[k];
    int cell;
    double fx, fy;
    if (!grid_cell(q.u, q.v, ns, cell, fx, fy)) continue;
    const T tx = (T)fx, ty = (T)fy;
    acc += (1 - tx) * (1 - ty) * s[cell] + tx * (1 - ty) * s[cell + 1] + (1 - tx) * ty * s[cell + ns] +
           tx * ty * s[cell + ns + 1];
  }
  img[(long)m * J + j] = acc / (T)n2;
}

// Adds the four terms of each of a pixel's subpixels to acc.
template <typename T, typename A>
__device__ __forceinline__ void add_pixel(const UV* __restrict__ p, int n2, int ns, T val, A* acc) {
  for (int k = 0; k < n2; ++k) {
    const UV q = p[k];
    int cell;
    double fx, fy;
    if (!grid_cell(q.u, q.v, ns, cell, fx, fy)) continue;
    const T tx = (T)fx, ty = (T)fy;
    atomicAdd(&acc[cell], (A)((1 - tx) * (1 - ty) * val));
    atomicAdd(&acc[cell + 1], (A)(tx * (1 - ty) * val));
    atomicAdd(&acc[cell + ns], (A)((1 - tx) * ty * val));
    atomicAdd(&acc[cell + ns + 1], (A)(tx * ty * val));
  }
}

// L^T of part of one member's pixels: the terms are added in an LDS copy of the
// member's source grid first and only its nonzero nodes go to memory, where
// atomics across the XCDs run at about 36 G/s (every term there: 285 us for 16
// members of a 128 x 128 image, 4.2 M terms; so 9 us).  The copy is FP64 for both
// types: ds_add_f32 takes two cycles a lane where ds_add_f64 takes a fraction of
// one (19 us for those 16 members with an FP32 copy, and one 64 x 64 image 22
// against 6 us).  The lanes of a wave take pixels n/64 apart, so that a magnified
// region's neighbouring pixels, which share nodes, do not meet in one LDS access.
constexpr int kLtT = 512;
template <typename T>
__global__ void __launch_bounds__(kLtT) k_apply_LT(const double* __restrict__ uv, int J, int nsub, Picked mb, int per,
                                                   const T* __restrict__ img, T* __restrict__ s_all) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int m = mb.id[blockIdx.y], ns = mb.ns[blockIdx.y], n2 = nsub * nsub, tid = threadIdx.x;
  T* s = s_all + mb.off[blockIdx.y];
  double* acc = reinterpret_cast<double*>(smem);
  for (int i = tid; i < ns * ns; i += kLtT) acc[i] = 0.0;
  __syncthreads();
  const int lo = (int)blockIdx.x * per;   // per: a multiple of 64
  for (int i = tid; i < per; i += kLtT) {
    const int j = lo + (i & 63) * (per >> 6) + (i >> 6);
    if (j >= J) continue;
    add_pixel(reinterpret_cast<const UV*>(uv) + ((long)m * J + j) * n2, n2, ns, img[(long)m * J + j] / (T)n2, acc);
  }
  __syncthreads();
  for (int i = tid; i < ns * ns; i += kLtT) {
    const double v = acc[i];
    if (v != 0.0) atomicAdd(&s[i], (T)v);   // (true for NaN)
  }
}

// The same for grids whose copy does not fit in LDS: a thread per pixel, every
// term to memory.  (About 256 blocks whose lanes took pixels far apart, as the
// LDS form's do, were slower than this: a 1024 x 1024 image with 512 x 512 nodes 867
// against 541 us.)
template <typename T>
__global__ void __launch_bounds__(256) k_apply_LT_mem(const double* __restrict__ uv, int J, int nsub, Picked mb,
                                                      const T* __restrict__ img, T* __restrict__ s_all) {
  const int j = blockIdx.x * 256 + threadIdx.x, m = mb.id[blockIdx.y], n2 = nsub * nsub;
  if (j >= J) return;
  add_pixel(reinterpret_cast<const UV*>(uv) + ((long)m * J + j) * n2, n2, mb.ns[blockIdx.y],
            img[(long)m * J + j] / (T)n2, s_all + mb.off[blockIdx.y]);
}

// Ordered L^T (fixed summation order).  A counting sort by node of the keys
// key = 4 t + corner (t = subpixel index j n^2 + k, corner 0..3 for the
// nodes cell, cell + 1, cell + ns, cell + ns + 1), then one wave per node puts
// its keys in ascending order, i.e. by pixel, subpixel, corner (the order of a
// sequential scatter over the pixels), and sums its terms in that order.

// Members of one launch: as Batch, and the start of each one's workspace (ints).
struct OrderedWs {
  int *cnt, *ptr, *cur, *keys;
};
__host__ __device__ inline long ordered_ints(long I_max, long keys) { return 3 * I_max + 1 + keys; }
__device__ __forceinline__ OrderedWs ordered_ws(int* ws, int m, long I_max, long keys) {
  int* w = ws + m * ordered_ints(I_max, keys);
  return {w, w + I_max, w + 2 * I_max + 1, w + 3 * I_max + 1};
}

// FILL = false: entries per node; true: the keys into their node's segment (in
// any order).  With LDS, a block counts its subpixels per node there first and
// takes each node's places with one atomic in memory.
template <bool FILL, bool LDS>
__global__ void __launch_bounds__(kLtT) k_lt_bin(const double* __restrict__ uv, long nsubpix, Picked mb, int per,
                                                 int* __restrict__ ws, long I_max) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int m = mb.id[blockIdx.y], ns = mb.ns[blockIdx.y], tid = threadIdx.x;
  const OrderedWs w = ordered_ws(ws, m, I_max, 4 * nsubpix);
  int* total = FILL ? w.cur : w.cnt;
  int* h = LDS ? reinterpret_cast<int*>(smem) : total;
  const UV* p = reinterpret_cast<const UV*>(uv) + m * nsubpix;
  const long lo = (long)blockIdx.x * per, hi = lo + per < nsubpix ? lo + per : nsubpix;
  if (LDS) {
    for (int i = tid; i < ns * ns; i += kLtT) h[i] = 0;
    __syncthreads();
  }
  if (LDS || !FILL) {
    for (long t = lo + tid; t < hi; t += kLtT) {
      const UV q = p[t];
      int cell;
      double fx, fy;
      if (!grid_cell(q.u, q.v, ns, cell, fx, fy)) continue;
      atomicAdd(&h[cell], 1);
      atomicAdd(&h[cell + 1], 1);
      atomicAdd(&h[cell + ns], 1);
      atomicAdd(&h[cell + ns + 1], 1);
    }
  }
  if (LDS) {
    __syncthreads();
    for (int i = tid; i < ns * ns; i += kLtT) {
      const int c = h[i];
      if (c) {
        const int at = atomicAdd(&total[i], c);
        if (FILL) h[i] = at;
      }
    }
    __syncthreads();
  }
  if (FILL) {
    for (long t = lo + tid; t < hi; t += kLtT) {
      const UV q = p[t];
      int cell;
      double fx, fy;
      if (!grid_cell(q.u, q.v, ns, cell, fx, fy)) continue;
      const int nd[4] = {cell, cell + 1, cell + ns, cell + ns + 1};
#pragma unroll
      for (int c = 0; c < 4; ++c) w.keys[atomicAdd(&h[nd[c]], 1)] = (int)(4 * t + c);
    }
  }
}

__global__ void __launch_bounds__(256) k_lt_zero(Batch mb, int* __restrict__ ws, long I_max, long nkeys) {
  const int i = blockIdx.x * 256 + threadIdx.x, ns = mb.ns[blockIdx.y];
  if (i < ns * ns) ordered_ws(ws, blockIdx.y, I_max, nkeys).cnt[i] = 0;
}

// Exclusive scan of cnt[0..I) into ptr[0..I] and the fill cursors cur (one block per member).
__global__ void __launch_bounds__(1024) k_lt_scan(Batch mb, int* __restrict__ ws, long I_max, long nkeys) {
  __shared__ int wsum[16];
  __shared__ int carry;
  const OrderedWs w = ordered_ws(ws, blockIdx.x, I_max, nkeys);
  const int I = mb.ns[blockIdx.x] * mb.ns[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if (tid == 0) carry = 0;
  __syncthreads();
  for (int i0 = 0; i0 < I; i0 += 1024) {
    const int i = i0 + tid;
    const int v = i < I ? w.cnt[i] : 0;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o, 64);
      if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int before = carry;
    for (int x = 0; x < wid; ++x) before += wsum[x];
    if (i < I) {
      w.ptr[i] = before + incl - v;
      w.cur[i] = before + incl - v;
    }
    __syncthreads();
    if (tid == 1023) carry = before + incl;
    __syncthreads();
  }
  if (tid == 0) w.ptr[I] = carry;
}

// One wave per node.  Its keys are distinct, so a key's rank is the count of
// smaller ones: up to kSortCap of them at a time in LDS.  A longer row is taken
// in ascending ranges of keys that hold no more than that, a range half as wide
// as one that held more and twice as wide after one that held less than half
// (each range scans the row: with widths that only shrank, a row of 3001 keys in
// one dense cluster among 4 M was scanned some 3000 times, 26.9 ms; 0.9 so).  (With one thread per
// node sorting its segment in memory by insertion, and five launches per member,
// a chain of operators with the ordered L^T took 81 ms for 16 members of a 128 x
// 128 image; 0.36 ms so.)
constexpr int kSortCap = 512, kGatherW = 4;

// What a row's gather reads, and this wave's LDS.
template <typename T>
struct RowView {
  const UV* p;
  const T* img;
  int ns, n2;
  int* ks;
  T *tw, *tv;
};

// Weight and value of a key's term.
template <typename T>
__device__ __forceinline__ void row_term(const RowView<T>& o, int key, T& w, T& v) {
  const long t = key >> 2;
  const UV q = o.p[t];
  int cell;
  double fx, fy;
  grid_cell(q.u, q.v, o.ns, cell, fx, fy);
  const T tx = (T)fx, ty = (T)fy;
  const int corner = key & 3;
  w = (corner & 1 ? tx : 1 - tx) * (corner & 2 ? ty : 1 - ty);
  v = o.img[t / o.n2] / (T)o.n2;
}

// The sum of the row of n keys by the whole wave (n, keys: the same in every lane).
template <typename T>
__device__ __forceinline__ T row_by_wave(const RowView<T>& o, const int* keys, int n, long all) {
  const int lane = threadIdx.x & 63;
  const auto wave_sync = [] {   // this wave's LDS accesses complete in order; keep the compiler's order too
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  T acc = 0;
  long width = n <= kSortCap ? all : all / ((n + kSortCap - 1) / kSortCap);
  for (long lo = 0; lo < all && n > 0;) {
    if (width < kSortCap) width = kSortCap;   // never more than that many distinct keys
    const long hi = lo + width < all ? lo + width : all;
    int c = 0;
    for (int e = 0; e < n && c <= kSortCap; e += 64) {
      const int k = e + lane < n ? keys[e + lane] : -1;
      const bool in = k >= lo && k < hi;
      const unsigned long long bal = __ballot(in);
      const int at = c + __builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
      if (in && at < kSortCap) o.ks[at] = k;
      c += __popcll(bal);
    }
    c = __builtin_amdgcn_readfirstlane(c);
    wave_sync();
    if (c > kSortCap) {
      width >>= 1;
      continue;
    }
    for (int e = lane; e < c; e += 64) {
      const int key = o.ks[e];
      int rank = 0;
      for (int x = 0; x < c; ++x) rank += o.ks[x] < key;
      T w, v;
      row_term(o, key, w, v);
      o.tw[rank] = w;
      o.tv[rank] = v;
    }
    wave_sync();
    for (int x = 0; x < c; ++x) acc += o.tw[x] * o.tv[x];
    wave_sync();
    lo = hi;
    if (c <= kSortCap / 2) width <<= 1;
  }
  return acc;
}

// On grids with more nodes than the image has subpixels (at most four keys a row
// on average) one lane takes a row of up to kShortRow keys, and the wave its 64
// rows' longer ones in turn.  (A wave per node there too: 512 x 512 pixels, 2 x 2
// subpixels, 2048 x 2048 nodes 5.7 ms in FP32, 6.3 in FP64; 4.7 so.)
constexpr int kShortRow = 8;
__host__ __device__ __forceinline__ bool rows_short(int ns, long nsubpix) { return (long)ns * ns >= nsubpix; }
template <typename T>
__global__ void __launch_bounds__(64 * kGatherW) k_lt_gather(const double* __restrict__ uv, int n2, long nsubpix,
                                                             Batch mb, int* __restrict__ ws, long I_max,
                                                             const T* __restrict__ img, T* __restrict__ s) {
  __shared__ int ks_[kGatherW][kSortCap];
  __shared__ T tw_[kGatherW][kSortCap], tv_[kGatherW][kSortCap];
  const int m = blockIdx.y, ns = mb.ns[m], lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const OrderedWs w = ordered_ws(ws, m, I_max, 4 * nsubpix);
  const RowView<T> o{reinterpret_cast<const UV*>(uv) + m * nsubpix, img + (long)m * (nsubpix / n2), ns, n2,
                     ks_[wid], tw_[wid], tv_[wid]};
  const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kGatherW + wid));
  if (!rows_short(ns, nsubpix)) {   // uniform
    if (wave >= ns * ns) return;
    const T acc = row_by_wave(o, w.keys + w.ptr[wave], w.ptr[wave + 1] - w.ptr[wave], 4 * nsubpix);
    if (lane == 0) s[mb.off[m] + wave] = acc;
    return;
  }
  const int i = 64 * wave + lane;
  const int e0 = i < ns * ns ? w.ptr[i] : 0, n = i < ns * ns ? w.ptr[i + 1] - e0 : 0;
  T acc = 0;
  if (n <= kShortRow) {
    int key[kShortRow];
#pragma unroll
    for (int e = 0; e < kShortRow; ++e) key[e] = e < n ? w.keys[e0 + e] : INT_MAX;   // (no key is that large)
    int last = -1;
    for (int r = 0; r < n; ++r) {   // the keys in ascending order
      int next = INT_MAX;
#pragma unroll
      for (int e = 0; e < kShortRow; ++e) next = key[e] > last ? min(next, key[e]) : next;
      T wt, v;
      row_term(o, next, wt, v);
      acc += wt * v;
      last = next;
    }
  }
  for (unsigned long long lng = __ballot(n > kShortRow); lng; lng &= lng - 1) {   // uniform
    const int l = __ffsll(lng) - 1;
    const T a = row_by_wave(o, w.keys + __builtin_amdgcn_readlane(e0, l), __builtin_amdgcn_readlane(n, l), 4 * nsubpix);
    if (lane == l) acc = a;
  }
  if (i < ns * ns) s[mb.off[m] + i] = acc;
}

template <typename T>
__global__ void k_fill(T* __restrict__ p, long n, T v) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ------------------------------------------------------------------ B, B^T
// TRANSPOSE=false: convolution, out(r, c) = sum P[a][b] x(r-a+ck, c-b+ck);
// true: correlation, x(r+a-ck, c+b-ck).  A block takes 32 rows x 8 N columns of
// one image, its input tile with the halo and the PSF in LDS.  A thread forms N
// consecutive outputs of one row from a register window, so that eight tap
// values from LDS (the same for every lane) and N + 7 input values serve 8 N
// products (two LDS reads per product in k_blur_small); a half-wave's lanes take consecutive rows,
// which the odd pitch puts in distinct banks.  Every output adds its taps in
// row-major order.  N = 8 reads less per product, N = 4 gives twice the waves;
// blur_cost estimates which is faster.
constexpr int kBlurT = 256, kBlurR = 32;
template <typename T, bool TRANSPOSE, int N>
__global__ void __launch_bounds__(kBlurT) k_blur(int nx, int ny, const double* __restrict__ psf, int K,
                                                 const T* __restrict__ in, T* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int W = 8 * N;   // columns of a block
  const int ck = (K - 1) / 2, KP = (K + 7) & ~7;
  const int tw = W + 2 * ck, pitch = tw | 1, th = kBlurR + 2 * ck;
  T* P = reinterpret_cast<T*>(smem);   // [K][KP], the pad zero
  T* tile = P + K * KP;
  const int bx = (nx + W - 1) / W, by = (ny + kBlurR - 1) / kBlurR;
  const int img = blockIdx.x / (bx * by), b = blockIdx.x % (bx * by);
  const int R0 = (b / bx) * kBlurR, C0 = (b % bx) * W;
  const T* src = in + (long)img * nx * ny;
  const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
  for (int a = ty; a < K; a += 8)
    for (int i = tx; i < KP; i += 32) P[a * KP + i] = i < K ? (T)psf[a * K + i] : (T)0;
  for (int j = tx; j < tw; j += 32) {
    const int cc = C0 - ck + j;
    const bool on = cc >= 0 && cc < nx;
    for (int i0 = ty; i0 < th; i0 += 64) {   // eight rows' loads in flight
      T v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int rr = R0 - ck + i0 + 8 * u;
        v[u] = on && i0 + 8 * u < th && rr >= 0 && rr < ny ? src[(long)rr * nx + cc] : (T)0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i0 + 8 * u < th) tile[(i0 + 8 * u) * pitch + j] = v[u];
    }
  }
  __syncthreads();
  const int r = R0 + tx, c0 = C0 + N * ty;
  if (r >= ny || c0 >= nx) return;
  T acc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = 0;
  // taps b0..b0+7 of PSF row a and the window x[i] they meet: the input b0 + i
  // after the thread's first (TRANSPOSE), or b0 + i before its last
  auto load = [&](int a, int b0, T (&x)[N + 7], T (&t)[8]) {
    const T* row = tile + (TRANSPOSE ? tx + a : tx + 2 * ck - a) * pitch + N * ty + (TRANSPOSE ? b0 : 2 * ck + N - 1 - b0);
    // the last chunk also reads up to seven values past the row, inside the LDS array, that no tap uses
#pragma unroll
    for (int i = 0; i < N + 7; ++i) x[i] = TRANSPOSE ? row[i] : row[-i];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = P[a * KP + b0 + u];
  };
  T x[N + 7], t[8];
  load(0, 0, x, t);
  for (int a = 0, b0 = 0; a < K;) {
    const int nb = K - b0;
    int a2 = a, b2 = b0 + 8;
    if (b2 >= K) {
      b2 = 0;
      ++a2;
    }
    T xn[N + 7], tn[8];
    load(min(a2, K - 1), b2, xn, tn);   // the next chunk, ahead of this one's products
    if (nb >= 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] += t[u] * x[TRANSPOSE ? u + i : u + N - 1 - i];
    } else {
#pragma unroll
      for (int u = 0; u < 7; ++u)
        if (u < nb) {   // uniform; a pad tap (zero) must not meet an infinite value
#pragma unroll
          for (int i = 0; i < N; ++i) acc[i] += t[u] * x[TRANSPOSE ? u + i : u + N - 1 - i];
        }
    }
#pragma unroll
    for (int i = 0; i < N + 7; ++i) x[i] = xn[i];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = tn[u];
    a = a2;
    b0 = b2;
  }
  T* o = out + (long)img * nx * ny + (long)r * nx + c0;
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (c0 + i < nx) o[i] = acc[i];
}

// The same for few outputs and small or thin images: one output per thread in
// 16 x 16 tiles, 256 threads a block, so that a single 200 x 200 image (K = 21) is
// 676 waves instead of the 196 of k_blur<4>: 12 against 22 us.
constexpr int kTile = 16;

template <typename T, bool TRANSPOSE>
__global__ void k_blur_small(int nx, int ny, const double* __restrict__ psf, int K,
                       const T* __restrict__ in, T* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem[];
  T* P = reinterpret_cast<T*>(smem);
  const int ck = (K - 1) / 2;
  const int tw = kTile + K - 1;
  T* tile = P + K * K;
  const long img_off = (long)blockIdx.z * nx * ny;
  const int R0 = blockIdx.y * kTile, C0 = blockIdx.x * kTile;
  const int tid = threadIdx.y * kTile + threadIdx.x;
  for (int i = tid; i < K * K; i += kTile * kTile) P[i] = (T)psf[i];
  for (int i = tid; i < tw * tw; i += kTile * kTile) {
    const int rr = R0 - ck + i / tw, cc = C0 - ck + i % tw;
    tile[i] = (rr >= 0 && rr < ny && cc >= 0 && cc < nx) ? in[img_off + (long)rr * nx + cc] : (T)0;
  }
  __syncthreads();
  const int r = R0 + threadIdx.y, c = C0 + threadIdx.x;
  if (r >= ny || c >= nx) return;
  T acc = 0;
  for (int a = 0; a < K; ++a)
    for (int b = 0; b < K; ++b) {
      // convolution reads x[r-a+ck][c-b+ck]; correlation reads z[r+a-ck][c+b-ck]
      const int tr = TRANSPOSE ? threadIdx.y + a : threadIdx.y + 2 * ck - a;
      const int tc = TRANSPOSE ? threadIdx.x + b : threadIdx.x + 2 * ck - b;
      acc += P[a * K + b] * tile[tr * tw + tc];
    }
  out[img_off + (long)r * nx + c] = acc;
}

// ------------------------------------------------------------------ H^T H
template <typename T>
__device__ __forceinline__ T node_at(const T* s, int ns, int r, int c) {
  return (r < 0 || c < 0 || r >= ns || c >= ns) ? (T)0 : s[r * ns + c];
}
template <typename T>
__device__ __forceinline__ T d2x_at(const T* s, int ns, int r, int c) {
  if (r < 0 || c < 0 || r >= ns || c >= ns) return (T)0;
  return node_at(s, ns, r, c - 1) - 2 * node_at(s, ns, r, c) + node_at(s, ns, r, c + 1);
}
template <typename T>
__device__ __forceinline__ T d2y_at(const T* s, int ns, int r, int c) {
  if (r < 0 || c < 0 || r >= ns || c >= ns) return (T)0;
  return node_at(s, ns, r - 1, c) - 2 * node_at(s, ns, r, c) + node_at(s, ns, r + 1, c);
}

template <typename T>
__global__ void __launch_bounds__(256) k_apply_HtH(int reg, Batch mb, const T* __restrict__ s_all,
                                                   T* __restrict__ out_all) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x, ns = mb.ns[blockIdx.y];
  if (i >= ns * ns) return;
  const T* s = s_all + mb.off[blockIdx.y];
  T* out = out_all + mb.off[blockIdx.y];
  if (reg == SL_H_IDENTITY) {
    out[i] = s[i];
    return;
  }
  const int r = i / ns, c = i % ns;
  out[i] = d2x_at(s, ns, r, c - 1) - 2 * d2x_at(s, ns, r, c) + d2x_at(s, ns, r, c + 1) +
           d2y_at(s, ns, r - 1, c) - 2 * d2y_at(s, ns, r, c) + d2y_at(s, ns, r + 1, c);
}

// ------------------------------------------------------------------ host helpers
static int check_grid(const sl_image_grid* img) {
  SL_REQUIRE(img != nullptr, "image grid is NULL");
  SL_REQUIRE(img->nx >= 1 && img->ny >= 1 && (long)img->nx * img->ny <= (1L << 28),
             "image size %d x %d out of range", img->nx, img->ny);
  SL_REQUIRE(std::isfinite(img->pix) && img->pix > 0.0, "pixel size must be positive");
  SL_REQUIRE(img->nsub >= 1 && img->nsub <= SL_MAX_NSUB, "nsub %d outside [1, %d]", img->nsub,
             SL_MAX_NSUB);
  return SL_OK;
}

static int check_ns(const int32_t* ns, int n_members) {
  SL_REQUIRE(n_members >= 1, "n_members must be >= 1");
  SL_REQUIRE(ns != nullptr, "ns is NULL");
  for (int m = 0; m < n_members; ++m)
    SL_REQUIRE(ns[m] >= 2 && ns[m] <= 4096, "ns[%d] = %d outside [2, 4096]", m, ns[m]);
  return SL_OK;
}

static inline unsigned nblocks(long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// Calls launch(first member, batch, members of the batch, largest side) for
// batches of at most kBatch members and 2^31 threads (threads(ns) of one member).
template <typename Threads, typename Launch>
static void for_batches(const int32_t* ns, int n_members, Threads threads, Launch launch) {
  long off = 0;
  for (int m0 = 0; m0 < n_members;) {
    Batch mb;
    int n = 0, big = 0;
    long most = 0;
    while (n < kBatch && m0 + n < n_members) {
      const int side = ns[m0 + n];
      const long t = std::max(most, (long)threads(side));
      if (n > 0 && t * (n + 1) > (1L << 31)) break;
      most = t;
      big = std::max(big, side);
      mb.ns[n] = side;
      mb.off[n] = off;
      off += (long)side * side;
      ++n;
    }
    launch(m0, mb, n, big);
    m0 += n;
  }
}

template <typename T>
static int apply_L_impl(const double* uv, int n_members, const sl_image_grid* img, const int32_t* ns,
                        const void* s, void* out, hipStream_t st) {
  const int J = img->nx * img->ny, n2 = img->nsub * img->nsub;
  for_batches(ns, n_members, [&](int) { return (long)J + 256; }, [&](int m0, const Batch& mb, int n, int) {
    hipLaunchKernelGGL(k_apply_L<T>, dim3(nblocks(J, 256), n), dim3(256), 0, st, uv + (long)m0 * J * n2 * 2, J,
                       img->nsub, mb, (const T*)s, (T*)out + (long)m0 * J);
  });
  return check_launch("k_apply_L");
}

// Calls launch(batch, members of the batch, largest side) for batches of the
// members whose side is at most `cut` (below = true) or more (false), each of at
// most kBatch members and 2^31 threads (`threads` of one member).
template <typename Launch>
static void for_picked(const int32_t* ns, int n_members, int cut, bool below, long threads, Launch launch) {
  const int most = (int)std::max(1L, std::min((long)kBatch, (1L << 31) / threads));
  long off = 0;
  Picked mb;
  int n = 0, big = 0;
  for (int m = 0; m < n_members; ++m) {
    if ((ns[m] <= cut) == below) {
      mb.ns[n] = ns[m];
      mb.id[n] = m;
      mb.off[n] = off;
      big = std::max(big, (int)ns[m]);
      if (++n == most) {
        launch(mb, n, big);
        n = big = 0;
      }
    }
    off += (long)ns[m] * ns[m];
  }
  if (n > 0) launch(mb, n, big);
}

// Largest side of a grid whose copy of `size` bytes per node fits in `lds` bytes.
static int side_that_fits(size_t lds, size_t size) {
  int n = 1;
  while (size * (n + 1) * (n + 1) <= lds) ++n;
  return n;
}

// Each member takes the form that its own grid allows: with the batch's largest
// grid deciding, one member of 150 nodes a side sent 62 of 40 to the memory
// atomics (128 x 128 image, 2 x 2 subpixels: 482 us; 44 so, and 2.7 -> 1.4 ms for the
// ordered form, which bins by the same rule).  Up to 78 KB of LDS two blocks of
// 512 threads share a CU, up to 158 KB (142 nodes) one has it alone, which still
// beats the atomics in memory.
constexpr size_t kLtLds = 158 * 1024;

template <typename T>
static int apply_LT_impl(const double* uv, int n_members, const sl_image_grid* img, const int32_t* ns,
                         const void* in, void* s, hipStream_t st) {
  const int J = img->nx * img->ny;
  long total = 0;
  for (int m = 0; m < n_members; ++m) total += (long)ns[m] * ns[m];
  hipLaunchKernelGGL(k_fill<T>, dim3(nblocks(total, 256)), dim3(256), 0, st, (T*)s, total, (T)0);
  SL_HIP(hipFuncSetAttribute((const void*)k_apply_LT<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLtLds));
  static const int cut = side_that_fits(kLtLds, sizeof(double));
  for_picked(ns, n_members, cut, true, (long)J + kLtT, [&](const Picked& mb, int n, int big) {
    // about 256 blocks over the batch, each with at least two pixels a thread: every block adds its nodes to
    // memory, so more of them cost more atomics than they save
    const int want = std::max(1, std::min((256 + n - 1) / n, (J + 2 * kLtT - 1) / (2 * kLtT)));
    const int per = ((J + want - 1) / want + 63) / 64 * 64;
    hipLaunchKernelGGL(k_apply_LT<T>, dim3(nblocks(J, per), n), dim3(kLtT), sizeof(double) * (size_t)big * big, st, uv,
                       J, img->nsub, mb, per, (const T*)in, (T*)s);
  });
  for_picked(ns, n_members, cut, false, (long)J + 256, [&](const Picked& mb, int n, int) {
    hipLaunchKernelGGL(k_apply_LT_mem<T>, dim3(nblocks(J, 256), n), dim3(256), 0, st, uv, J, img->nsub, mb,
                       (const T*)in, (T*)s);
  });
  return check_launch("k_apply_LT");
}

// Workspace of the ordered L^T: per member (I + 1) + 2 I ints of counts, row
// starts and cursors and 4 J n^2 keys, all sized for the largest grid, for as
// many members at a time as fit in `limit` bytes (at least one).
static long ordered_group(const sl_image_grid* img, const int32_t* ns, int n_members, size_t limit, long* I_max) {
  long I = 0;
  for (int m = 0; m < n_members; ++m) I = std::max(I, (long)ns[m] * ns[m]);
  *I_max = I;
  const size_t bytes = sizeof(int) * ordered_ints(I, 4L * img->nx * img->ny * img->nsub * img->nsub);
  return std::max(1L, std::min({(long)n_members, (long)kBatch, (long)(limit / bytes)}));
}

constexpr size_t kOrderedWs = 256u << 20;   // the most that the query asks for, beyond one member's

static size_t lt_ordered_ws(const sl_image_grid* img, const int32_t* ns, int n_members, size_t limit) {
  long I = 0;
  const long g = ordered_group(img, ns, n_members, limit, &I);
  return sizeof(int) * (size_t)(g * ordered_ints(I, 4L * img->nx * img->ny * img->nsub * img->nsub));
}

// Largest LDS histogram of a source grid (two blocks of 512 threads still fit on a CU).
constexpr size_t kBinLds = 78 * 1024;

// One pass of k_lt_bin over a group of members, each in the form its grid allows;
// a histogram of more nodes than there are subpixels costs more to clear and
// read out than the atomics in memory that it saves (one 32 x 32 image, 100 x 100
// nodes: the operator 40 -> 35 us).
template <bool FILL>
static void launch_bins(const double* uv, long nsp, const int32_t* ns, int n, int* ws, long I_max, hipStream_t st) {
  static const int fits = side_that_fits(kBinLds, sizeof(int));
  int cut = 1;
  while (cut < fits && (long)(cut + 1) * (cut + 1) <= nsp) ++cut;
  for (const bool lds : {true, false})
    for_picked(ns, n, cut, lds, nsp + kLtT, [&](const Picked& mb, int np, int big) {
      const int want = lds ? (int)std::max(1L, std::min((256L + np - 1) / np, (nsp + 8L * kLtT - 1) / (8L * kLtT)))
                           : (int)nblocks(nsp, kLtT);   // a thread per subpixel
      const int per = (int)((nsp + want - 1) / want);
      const dim3 grid(nblocks(nsp, per), np);
      if (lds)
        hipLaunchKernelGGL((k_lt_bin<FILL, true>), grid, dim3(kLtT), sizeof(int) * (size_t)big * big, st, uv, nsp, mb,
                           per, ws, I_max);
      else
        hipLaunchKernelGGL((k_lt_bin<FILL, false>), grid, dim3(kLtT), 0, st, uv, nsp, mb, per, ws, I_max);
    });
}

template <typename T>
static int apply_LT_ordered_impl(const double* uv, int n_members, const sl_image_grid* img, const int32_t* ns,
                                 const void* in, void* s, void* ws, size_t ws_bytes, hipStream_t st) {
  const int J = img->nx * img->ny, n2 = img->nsub * img->nsub;
  const long nsp = (long)J * n2;
  long I_max = 0;
  const int group = (int)ordered_group(img, ns, n_members, ws_bytes, &I_max);
  SL_HIP(hipFuncSetAttribute((const void*)k_lt_bin<false, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)kBinLds));
  SL_HIP(hipFuncSetAttribute((const void*)k_lt_bin<true, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)kBinLds));
  long off = 0;
  for (int m0 = 0; m0 < n_members; m0 += group) {
    const int n = std::min(group, n_members - m0);
    Batch mb;
    int big = 0;
    unsigned rows = 0;   // blocks of k_lt_gather that the member with the most needs
    for (int i = 0; i < n; ++i) {
      mb.ns[i] = ns[m0 + i];
      mb.off[i] = off;
      off += (long)ns[m0 + i] * ns[m0 + i];
      rows = std::max(rows, nblocks((long)ns[m0 + i] * ns[m0 + i],
                                    rows_short(ns[m0 + i], nsp) ? 64 * kGatherW : kGatherW));
      big = std::max(big, ns[m0 + i]);
    }
    const double* uvm = uv + (long)m0 * nsp * 2;
    int* w = (int*)ws;
    hipLaunchKernelGGL(k_lt_zero, dim3(nblocks((long)big * big, 256), n), dim3(256), 0, st, mb, w, I_max, 4 * nsp);
    launch_bins<false>(uvm, nsp, ns + m0, n, w, I_max, st);
    hipLaunchKernelGGL(k_lt_scan, dim3(n), dim3(1024), 0, st, mb, w, I_max, 4 * nsp);
    launch_bins<true>(uvm, nsp, ns + m0, n, w, I_max, st);
    hipLaunchKernelGGL(k_lt_gather<T>, dim3(rows, n), dim3(64 * kGatherW), 0, st, uvm, n2, nsp, mb, w, I_max,
                       (const T*)in + (long)m0 * J, (T*)s);
    if (int e = check_launch("ordered L^T")) return e;
  }
  return SL_OK;
}

// LDS of a blur block with N consecutive outputs a thread (1: k_blur_small).
template <typename T>
static size_t blur_lds(int N, int k) {
  if (N == 1) return sizeof(T) * ((size_t)k * k + (size_t)(kTile + k - 1) * (kTile + k - 1));
  return sizeof(T) * ((size_t)k * ((k + 7) & ~7) + (size_t)(kBlurR + k - 1) * ((8 * N + k - 1) | 1) + 8);
}

template <typename T, bool TR, int N>
static int blur_launch(int nx, int ny, int n_images, const double* psf, int k, const void* in, void* out,
                       hipStream_t st) {
  const size_t lds = blur_lds<T>(N, k);
  if (lds > 64 * 1024)
    SL_HIP(hipFuncSetAttribute((const void*)k_blur<T, TR, N>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const unsigned blocks = nblocks(nx, 8 * N) * nblocks(ny, kBlurR) * (unsigned)n_images;
  hipLaunchKernelGGL((k_blur<T, TR, N>), dim3(blocks), dim3(kBlurT), lds, st, nx, ny, psf, k, (const T*)in, (T*)out);
  return check_launch("k_blur");
}

// Estimated microseconds of one form, launch aside: rounds of blocks, each of a
// fixed part and one output's chain of products, and the products of the waves
// that hold outputs (on images narrower or flatter than a tile most of a
// register-tiled block's waves hold none; k_blur_small's tile fits closer).
// The constants are fits to 2010 measured launches of each form: 33 image
// shapes from 4 x 4 and 1 x 200 to 512 x 512, 2^17 to 2^21 outputs, K = 1 to 63,
// both types.  *bare: few blocks or few waves with outputs on a CU, which leave
// nothing to hide a block's staging and its chains behind.
template <typename T>
static double blur_cost(int N, int nx, int ny, int n_images, int k, double* bare) {
  struct Cost {
    double block, chain, wave;
  };
  static const Cost kCost[2][3] = {{{0.30, 0.0038, 0.0022}, {1.20, 0.020, 0.0021}, {0.54, 0.022, 0.0019}},
                                   {{0.10, 0.0105, 0.0028}, {3.20, 0.019, 0.0055}, {0.96, 0.021, 0.0043}}};
  const Cost& c = kCost[sizeof(T) == 8][N / 4];
  const int cus = device_cus(), fit = std::max(1, std::min(8, (int)(160 * 1024 / blur_lds<T>(N, k))));
  double blocks, waves, work;
  if (N == 1) {
    blocks = (double)nblocks(nx, kTile) * nblocks(ny, kTile);
    waves = (double)nblocks(nx, kTile) * nblocks(ny, 4);   // four rows of a tile per wave
    work = (double)k * k;
  } else {   // two column groups of N per wave
    blocks = (double)nblocks(nx, 8 * N) * nblocks(ny, kBlurR);
    waves = (nx / (8 * N) * 4 + (double)nblocks(nblocks(nx % (8 * N), N), 2)) * nblocks(ny, kBlurR);
    work = (double)k * ((k + 7) / 8) * 4 * (N / 4 + 1);
  }
  *bare = fit * waves <= 3 * blocks ? 1.6 : fit <= 2 ? 1.2 : 1.0;
  if (N > 1 && blocks * n_images * kBlurT >= 2147483648.0) return HUGE_VAL;   // its grid has one dimension
  const double rounds = std::max(1.0, blocks * n_images / ((double)cus * fit));
  return rounds * (c.block + c.chain * work) + c.wave * waves * n_images * work / cus;
}

// A register-tiled form has to be estimated a fifth faster than k_blur_small (more
// with few waves on a CU), so that the error of an estimate does not lose time.
// So chosen, 6 of the 2010 launches are more than 5 % slower than with
// k_blur_small, by 11 % at most, and the choice is within 3.5 % of the best of
// the three on average.  (The rule before counted full tiles only and took a
// register-tiled form from one or two blocks per CU up: 8192 images of 8 x 8, K =
// 63, 592 -> 3358 us; one 2000 x 2000 image in FP64, K = 3, 35 -> 44 us.)  Below K =
// 5 (FP64: 9) a tile's staging and the stores of N outputs per lane, a row apart
// from lane to lane, cost what the register window saves; at K = 5 only rows of
// whole groups of N win.  Where they win: K = 21, 64 images of 200 x 200, 72
// against 199 us; K = 63, 640 x 640, 143 against 301 us.
template <typename T, bool TR>
static int blur_impl(int nx, int ny, int n_images, const double* psf, int k, const void* in, void* out,
                     hipStream_t st) {
  if (k >= (sizeof(T) == 4 ? 5 : 9)) {
    double bare, bare4, bare8;
    const double small = 0.8 * blur_cost<T>(1, nx, ny, n_images, k, &bare);
    const double c4 = blur_cost<T>(4, nx, ny, n_images, k, &bare4), c8 = blur_cost<T>(8, nx, ny, n_images, k, &bare8);
    const bool ok4 = k > 5 || nx % 4 == 0, ok8 = k > 5 || nx % 8 == 0;
    if (ok4 && (c4 <= c8 || !ok8)) {
      if (bare4 * c4 < small) return blur_launch<T, TR, 4>(nx, ny, n_images, psf, k, in, out, st);
    } else if (ok8 && bare8 * c8 < small) {
      return blur_launch<T, TR, 8>(nx, ny, n_images, psf, k, in, out, st);
    }
  }
  const size_t lds = blur_lds<T>(1, k);
  if (lds > 64 * 1024)
    SL_HIP(hipFuncSetAttribute((const void*)k_blur_small<T, TR>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL((k_blur_small<T, TR>), dim3(nblocks(nx, kTile), nblocks(ny, kTile), n_images),
                     dim3(kTile, kTile), lds, st, nx, ny, psf, k, (const T*)in, (T*)out);
  return check_launch("k_blur");
}

}  // namespace sl

using namespace sl;

extern "C" {

const char* sl_last_error(void) { return g_err; }

const char* sl_version(void) { return "semilin 0.1 (gfx950)"; }

int sl_lens_trace(const double* lens, int n_members, const sl_image_grid* img, const int32_t* ns,
                  double half_width, double* uv, void* stream) {
  if (int e = check_grid(img)) return e;
  if (int e = check_ns(ns, n_members)) return e;
  SL_REQUIRE(lens && uv, "NULL device pointer");
  SL_REQUIRE(std::isfinite(half_width) && half_width > 0.0, "half_width must be positive");
  hipStream_t st = (hipStream_t)stream;
  const long per = (long)img->nx * img->ny * img->nsub * img->nsub;
  for_batches(ns, n_members, [&](int) { return per + 256; }, [&](int m0, const Batch& mb, int n, int) {
    // four subpixels a thread once that leaves four blocks per CU: the block's lens constants are one thread's work
    const int rep = nblocks(per, 1024) * (long)n >= 4L * device_cus() ? 4 : 1;
    hipLaunchKernelGGL(k_trace, dim3(nblocks(per, 256 * rep), n), dim3(256), 0, st, lens + 7L * m0, img->nx, img->ny,
                       img->pix, img->nsub, mb, half_width, rep, uv + 2 * per * m0);
  });
  return check_launch("k_trace");
}

int sl_apply_L(int dtype, const double* uv, int n_members, const sl_image_grid* img, const int32_t* ns,
               const void* s, void* img_out, void* stream) {
  if (int e = check_grid(img)) return e;
  if (int e = check_ns(ns, n_members)) return e;
  SL_REQUIRE(uv && s && img_out, "NULL device pointer");
  if (dtype == SL_F32) return apply_L_impl<float>(uv, n_members, img, ns, s, img_out, (hipStream_t)stream);
  if (dtype == SL_F64) return apply_L_impl<double>(uv, n_members, img, ns, s, img_out, (hipStream_t)stream);
  SL_REQUIRE(false, "unknown dtype %d", dtype);
}

int sl_apply_LT(int dtype, const double* uv, int n_members, const sl_image_grid* img, const int32_t* ns,
                const void* img_in, void* s_out, void* stream) {
  if (int e = check_grid(img)) return e;
  if (int e = check_ns(ns, n_members)) return e;
  SL_REQUIRE(uv && img_in && s_out, "NULL device pointer");
  if (dtype == SL_F32)
    return apply_LT_impl<float>(uv, n_members, img, ns, img_in, s_out, (hipStream_t)stream);
  if (dtype == SL_F64)
    return apply_LT_impl<double>(uv, n_members, img, ns, img_in, s_out, (hipStream_t)stream);
  SL_REQUIRE(false, "unknown dtype %d", dtype);
}

size_t sl_apply_LT_ordered_workspace_size(const sl_image_grid* img, const int32_t* ns, int n_members) {
  if (check_grid(img) != SL_OK || check_ns(ns, n_members) != SL_OK) return 0;
  return lt_ordered_ws(img, ns, n_members, kOrderedWs);
}

int sl_apply_LT_ordered(int dtype, const double* uv, int n_members, const sl_image_grid* img, const int32_t* ns,
                        const void* img_in, void* s_out, void* workspace, size_t workspace_bytes, void* stream) {
  if (int e = check_grid(img)) return e;
  if (int e = check_ns(ns, n_members)) return e;
  SL_REQUIRE(uv && img_in && s_out && workspace, "NULL device pointer");
  SL_REQUIRE(((uintptr_t)workspace & 3) == 0, "workspace must be 4-byte aligned");
  SL_REQUIRE(4L * img->nx * img->ny * img->nsub * img->nsub < (1L << 31), "image too large for 32-bit keys");
  const size_t need = lt_ordered_ws(img, ns, n_members, 0);   // one member at a time
  SL_REQUIRE(workspace_bytes >= need, "workspace too small: %zu < %zu bytes", workspace_bytes, need);
  if (dtype == SL_F32)
    return apply_LT_ordered_impl<float>(uv, n_members, img, ns, img_in, s_out, workspace, workspace_bytes,
                                        (hipStream_t)stream);
  if (dtype == SL_F64)
    return apply_LT_ordered_impl<double>(uv, n_members, img, ns, img_in, s_out, workspace, workspace_bytes,
                                        (hipStream_t)stream);
  SL_REQUIRE(false, "unknown dtype %d", dtype);
}

static int blur_args(int nx, int ny, int n_images, const double* psf, int k, const void* in, void* out) {
  SL_REQUIRE(nx >= 1 && ny >= 1 && n_images >= 1, "bad image sizes");
  SL_REQUIRE(k >= 1 && k <= SL_MAX_PSF && (k & 1), "PSF side %d must be odd and <= %d", k, SL_MAX_PSF);
  SL_REQUIRE(psf && in && out, "NULL device pointer");
  SL_REQUIRE(in != out, "in and out must differ");
  return SL_OK;
}

int sl_apply_B(int dtype, int nx, int ny, int n_images, const double* psf, int k, const void* in,
               void* out, void* stream) {
  if (int e = blur_args(nx, ny, n_images, psf, k, in, out)) return e;
  if (dtype == SL_F32) return blur_impl<float, false>(nx, ny, n_images, psf, k, in, out, (hipStream_t)stream);
  if (dtype == SL_F64) return blur_impl<double, false>(nx, ny, n_images, psf, k, in, out, (hipStream_t)stream);
  SL_REQUIRE(false, "unknown dtype %d", dtype);
}

int sl_apply_BT(int dtype, int nx, int ny, int n_images, const double* psf, int k, const void* in,
                void* out, void* stream) {
  if (int e = blur_args(nx, ny, n_images, psf, k, in, out)) return e;
  if (dtype == SL_F32) return blur_impl<float, true>(nx, ny, n_images, psf, k, in, out, (hipStream_t)stream);
  if (dtype == SL_F64) return blur_impl<double, true>(nx, ny, n_images, psf, k, in, out, (hipStream_t)stream);
  SL_REQUIRE(false, "unknown dtype %d", dtype);
}

int sl_apply_HtH(int dtype, int reg, int n_members, const int32_t* ns, const void* s, void* out,
                 void* stream) {
  if (int e = check_ns(ns, n_members)) return e;
  SL_REQUIRE(reg == SL_H_IDENTITY || reg == SL_H_CURVATURE, "unknown reg %d", reg);
  SL_REQUIRE(s && out && s != out, "bad device pointers");
  hipStream_t st = (hipStream_t)stream;
  SL_REQUIRE(dtype == SL_F32 || dtype == SL_F64, "unknown dtype %d", dtype);
  for_batches(ns, n_members, [](int side) { return (long)side * side + 256; },
              [&](int, const Batch& mb, int n, int big) {
    const dim3 grid(nblocks((long)big * big, 256), n);
    if (dtype == SL_F32)
      hipLaunchKernelGGL(k_apply_HtH<float>, grid, dim3(256), 0, st, reg, mb, (const float*)s, (float*)out);
    else
      hipLaunchKernelGGL(k_apply_HtH<double>, grid, dim3(256), 0, st, reg, mb, (const double*)s, (double*)out);
  });
  return check_launch("k_apply_HtH");
}

int sl_lcurve_corner(const double* reg, const double* chi2, int n, int32_t* k_star, double* kappa) {
  SL_REQUIRE(reg && chi2 && k_star, "NULL host pointer");
  SL_REQUIRE(n >= 4 && n <= SL_MAX_LAMBDA, "L-curve needs 4..%d points, got %d", SL_MAX_LAMBDA, n);
  std::vector<double> scratch(kLcurveScratch);
  const int k = lcurve_corner_impl(reg, chi2, n, kappa, scratch.data());
  SL_REQUIRE(k >= 0, "degenerate L-curve (non-positive values or fewer than 4 distinct points)");
  *k_star = k;
  return SL_OK;
}

}  // extern "C"
