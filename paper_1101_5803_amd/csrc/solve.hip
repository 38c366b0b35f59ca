// Batched matrix-free regularised source solve (Rogers & Fiege 2011, Sec. 2.1-2.6).
//
// One call scores n_members lens parameter sets against one data image:
//   k_setup   (1 block)          member offsets, XCD-sorted work queues, PSF
//                                factorisation (rank-1 test, 1-D taps, the
//                                banded B^T B coefficients and their image-edge
//                                corrections), sum of d^2
//   k_prep_*  (grid-wide)        FP64 subpixel trace (Eq. 1, Eqs. 10-11) of
//                                every pixel, compaction of the pixels that map
//                                onto the grid (Sec. 2.2: the others get no
//                                intensity), their bounding box, the transposed
//                                operator, and the right-hand side
//                                b = L^T B^T d in FP64
//   k_solve   (persistent, 1 block/CU)  each block pulls (member, lambda) items
//                                and runs CG on (L^T B^T B L + lambda H^T H) s = b
//                                from s = 0 (Eq. 7, Eq. 13-14, Sec. 2.2); the
//                                iterate s and residual r in global memory (each
//                                element touched only by its owner thread), p
//                                and q = A p in LDS, the image-space intermediate
//                                in an LDS frame over the mapped bounding box;
//                                ends with chi^2 (Eq. 4) and ||H s||^2 in FP64
//   k_split   (1 block)          moves the items that take the spectral
//                                preconditioner to their own queues (FP32,
//                                curvature H); k_solve<.., true> runs them as
//                                preconditioned CG on a side stream, beside
//                                the plain k_solve
//   k_corner  (1 block/member)   L-curve corner (Sec. 2.6, Eq. 20) in FP64 and
//                                the corner solution copy
//
// B^T B for a rank-1 PSF P = g_y g_x^T factorises as (C_y^T C_y) (x) (C_x^T C_x)
// with C the truncated 1-D "same" convolutions; each factor is a symmetric
// banded matrix equal to the autocorrelation of the 1-D taps except in the
// ck x ck corners next to the image edges, so B^T B y is two in-place banded
// passes over the frame (rows, then columns) with (4ck+1) taps plus a small
// correction for outputs within ck of the image edge.  A PSF that is not
// rank-1 takes the direct K x K path with an image-space buffer in global memory.
#include <algorithm>
#include <array>
#include <type_traits>
#include <map>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <vector>

#include "common.h"

namespace sl {

constexpr int kNT = 1024;     // threads per FP32 solve block (kNTof below)
constexpr int kWaves = kNT / kWave;
// Threads per solve block by bulk type: FP64 blocks run 512 threads, which
// leaves 256 VGPRs per lane and no spills; FP32 keeps 1024, whose extra waves
// hide the gathers' latency better than an unspilled 512-thread block does.
template <typename T>
constexpr int kNTof = sizeof(T) == 8 ? 512 : kNT;
constexpr int kSegR = 4;       // outputs per lane in a banded pass
constexpr int kUpd = 4;        // CG vector-update chunk (nodes per thread)
// The spectral preconditioner pays for its four n x n transforms only where
// lambda H^T H dominates the spectrum: it is used when lambda >= kPcTheta c.
constexpr int kPcThetaPct = 15;   // default theta = 0.15 (sl_tuning.pc_theta_pct = 0)
constexpr int kFillW = 16;     // waves that fill the transposed operator in parallel in k_prep_fill
constexpr int kHeavy = 4;      // default count of smallest lambdas of each member queued ahead of the rest
constexpr int kMaxCK = 31;

struct alignas(16) MemberInfo {
  int ns, I, M, r0, r1, c0, c1, status;   // M: interleaved table slots (>= mapped pixels)
  long long off;   // start in packed vectors
  int Mtrue;       // pixels with at least one subpixel on the grid
  int sell;        // transposed operator: CSR (0), sliced-ELL (1), sliced-ELL with paired 16-bit offsets (2)
  float pc_c;      // scale c of the spectral preconditioner (see k_prep_rhs)
  int lds_frame;   // where the solve keeps the member's image frame: Mem
  int pad_[2];
};

// Where a member's image frame and q live.  FP32: p, q and the frame in LDS
// at offsets for the largest grid, or the frame in global memory.  FP64, whose
// arrays are twice the size, places them by the member's own grid (LdsPlan),
// and q, which each iteration writes once and reads once by its owners, gives
// its place to the frame, which the gathers and the banded passes work in,
// where not both fit.
enum Mem { kMemGlobal = 0, kMemLds = 1, kMemLdsQGlobal = 2 };

// Device constants written by k_setup (one copy per workspace).
struct alignas(16) Consts {
  int qhead[8];
  int qcount[8];
  int pqhead[8];    // queues of the preconditioned items (filled by k_split)
  int pqcount[8];
  int sep;          // PSF is rank-1
  int mchead;       // next member of the Monte Carlo degrees-of-freedom pass
  int imhead;       // next member of the implicit-regularisation solve
  int pad0;
  double sum_d2;
  double sum_n2;    // sum of the squared Monte Carlo draws
};

struct Layout {
  size_t consts, lam, taps_d, taps_f, minfo, queues, pqueues, pix, cell, fx, fy, pmask, btd, pcpart, b, bh, dofk, s_all,
      gframe, gz, rbuf, mcbuf, ibuf, lt_ptr, lt_perm, lt_base, lt_cnt, lt_ent, total;
  long long lt_cap;
  int qcap, n_wg, I_max, J, n2, gframe_elems, slot_cap;
};

// Offsets (elements) inside the taps arrays, for a PSF of side K (ck = (K-1)/2).
struct TapIdx {
  int gx, gy, ax, ay, elx, erx, ely, ery, psf, total;
  __host__ __device__ TapIdx(int K) {
    const int ck = (K - 1) / 2;
    const int na = 4 * kMaxCK + 1;     // autocorrelation padded to the largest window
    gx = 0;
    gy = gx + K;
    ax = gy + K;
    ay = ax + na;
    elx = ay + na;
    erx = elx + ck * ck;
    ely = erx + ck * ck;
    ery = ely + ck * ck;
    psf = ery + ck * ck;
    total = psf + K * K;
  }
};

// One entry of the transposed lens operator: L^T w at a node is the sum of
// w[off] * weight over the node's entries (off = frame offset of the pixel).
template <typename T>
struct alignas(2 * sizeof(T) > 8 ? 16 : 8) LtEntry {
  int off;
  T w;
};

// Weights of the paired form's entries 2k and 2k + 1 of a row.
template <typename T>
struct alignas(2 * sizeof(T)) EntryPair {
  T x, y;
};

// ------------------------------------------------------------------ parameters
struct SolveArgs {
  int nx, ny, nsub, n2, K, ck, ckt, reg, n_members, n_lambda, max_ns, maxit, lds_frame_cap;
  int q_off, red_off, pc_off, frame_off;   // byte offsets in dynamic LDS
  int lds_bytes;                   // dynamic LDS of the solve kernels
  int frames_fit;                  // FP64: the whole image's frame fits in LDS beside the largest grid's vectors
  int one_vector;                  // k_chi2_src: no second vector, and one member only
  int gframe_elems;                // per-block global frame size (elements)
  int slot_cap;                    // trace-table slots per member (J + 64)
  double pix, R, sigma, tol;
  double* lamv;                    // workspace copy of the lambda grid
  const double* lens;
  const int32_t* ns;
  const double* d;
  const double* psf;
  // results
  double* s_corner;
  int64_t* s_off;
  double* chi2;
  double* regv;
  int32_t* iters;
  int32_t* status;
  int32_t* k_star;
  int32_t* corner_status;
  // workspace
  Consts* consts;
  double* taps_d;
  void* taps_t;   // taps in the bulk type
  MemberInfo* minfo;
  int* queues;
  int* pqueues;     // [8][qcap] items of the preconditioned solve
  int qcap;
  int32_t* pix_list;
  int32_t* cell;
  void* fx;
  void* fy;
  double* b;
  void* s_all;
  void* gframe;
  void* gz;
  void* rbuf;       // per-block CG residual
  int32_t* lt_ptr;  // [member][I_max + 65] slice (or row) starts of the transposed operator
  int32_t* lt_perm; // [member][I_max] nodes in slice order, packed (row << 16 | col)
  void* lt_ent;     // [member][lt_cap] LtEntry<T>
  long long lt_cap; // entries per member
  int I_max;
  int force_csr;    // variant: transposed operator as CSR rows
  int force_direct; // direct K x K blur only (variant, the hint that the PSF is not rank 1, or bicubic L)
  int psf_general;  // the caller's hint: the PSF is not rank 1
  int interp;       // SL_INTERP_BILINEAR | NEAREST (the fractions k_prep_trace stores) | BICUBIC
  int implicit;     // implicit regularisation: n_lambda unregularised CG iterations (k_implicit)
  int heavy;        // smallest lambdas of each member queued ahead of the rest
  float pc_theta;   // items with lambda >= pc_theta c take the spectral preconditioner
  int plain_cg;     // variant: no spectral preconditioner
  // Monte Carlo degrees of freedom (Sec. 2.5), when mcn is not NULL
  const double* mcn; // [ny*nx] Gaussian draws bhat
  double* dofv;      // [n_members] result: bhat^T (bhat - A xhat) at the corner
  double* bh;        // [member][I_max] A^T bhat (FP64)
  double* dofk;      // [member][n_lambda] implicit solve: the estimate after each iterate
  void* pmask;       // [member][slot_cap] first-occurrence mask of a slot's (subpixel, corner) pairs (PairMasks)
  double* btd;       // [2][J] B^T d and B^T bhat (FP64)
  double* pcpart;    // [member][rhs_blocks][2] parts of the preconditioner scale's two sums
  int rhs_blocks;    // blocks of k_prep_rhs per member
  int32_t* lt_base;  // [member][I_max] index of each node's first entry of the transposed operator
  int32_t* lt_cnt;   // [member][I_max] entries of each node
  void* mcbuf;       // [n_wg][5][I_max] r, xhat, rhat, phat, saved p of the pass
  void* ibuf;        // [n_wg][J] image residual e = d - A s of the implicit-regularisation solve
};

// ------------------------------------------------------------------ k_setup
struct LamList {
  double v[SL_MAX_LAMBDA];
};

// Inclusive sum over the block's 1024 threads of a 64-bit value; `sc` holds 17
// values of LDS.  Returns the inclusive prefix, *total the block's sum.
__device__ __forceinline__ long long block_scan64(long long v, long long* sc, long long* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const long long u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  if (lane == 63) sc[wid] = v;
  __syncthreads();
  long long before = 0, all = 0;
  for (int i = 0; i < 16; ++i) {
    if (i < wid) before += sc[i];
    all += sc[i];
  }
  __syncthreads();
  *total = all;
  return before + v;
}

// Lanes of this wave with the same key of up to 8 bits.
__device__ __forceinline__ unsigned long long match8(int key) {
  unsigned long long mk = ~0ull;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const unsigned long long bal = __ballot((key >> b) & 1);
    mk &= (key >> b) & 1 ? bal : ~bal;
  }
  return mk;
}

__device__ __forceinline__ int lanes_below(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// One block; what bounds it is the latency of its dependent steps, so each of
// them (offsets, sort, queues, factorisation, autocorrelations, edges) is
// spread over the threads, every value computed as one thread would compute
// it.  (One thread doing them in turn took 129 us for a 15 x 15 PSF and one
// member, 345 us for 256 members x 16 lambdas, 560 us for a 21 x 21 PSF and
// 24 lambdas.)
template <typename T>
__global__ void __launch_bounds__(1024) k_setup(SolveArgs a, LamList lams) {
  extern __shared__ __align__(16) unsigned char smem_setup[];
  double* tp = reinterpret_cast<double*>(smem_setup);   // the tap table, built here and copied out
  __shared__ double red[32];
  __shared__ long long scan64[16];
  __shared__ int start[256], wcnt[16][256], sh_sep, sh_am[16];
  __shared__ double sh_pm[16];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int M = a.n_members, K = a.K, ck = a.ck;
  const TapIdx ti(K);
  double* psh = tp + TapIdx(SL_MAX_PSF).total;   // the PSF
  if (tid < a.n_lambda) a.lamv[tid] = lams.v[tid];
  for (int i = tid; i < K * K; i += 1024) psh[i] = a.psf[i];
  for (int i = tid; i < ti.total; i += 1024) tp[i] = 0.0;
  if (tid < 256) start[tid] = 0;
  for (int i = tid; i < 16 * 256; i += 1024) (&wcnt[0][0])[i] = 0;
  if (tid == 0) sh_sep = 1;
  __syncthreads();
  // offsets of packed solutions (invalid ns contribute nothing) and the count of members per grid side
  long long off0 = 0;
  for (int m0 = 0; m0 < M; m0 += 1024) {
    const int m = m0 + tid;
    const int ns = m < M ? a.ns[m] : 0;
    const bool ok = ns >= 2 && ns <= a.max_ns;
    long long total;
    const long long I = ok ? (long long)ns * ns : 0;
    const long long off = off0 + block_scan64(I, scan64, &total) - I;
    if (m < M) {
      atomicAdd(&start[ok ? ns : 0], 1);
      a.s_off[m] = off;
      MemberInfo& mi = a.minfo[m];
      mi.ns = ok ? ns : 0;
      mi.I = (int)I;
      mi.off = off;
      mi.r0 = mi.c0 = INT_MAX;   // k_prep_trace widens the box
      mi.r1 = mi.c1 = INT_MIN;
    }
    off0 += total;
  }
  if (tid == 0) a.s_off[M] = off0;
  // largest |P| (the first of equals) for the rank-1 test
  double pm = 0.0;
  int pi = INT_MAX;
  for (int i = tid; i < K * K; i += 1024)
    if (fabs(psh[i]) > pm) {
      pm = fabs(psh[i]);
      pi = i;
    }
  for (int o = 32; o > 0; o >>= 1) {
    const double v = __shfl_xor(pm, o, 64);
    const int i = __shfl_xor(pi, o, 64);
    if (v > pm || (v == pm && i < pi)) {
      pm = v;
      pi = i;
    }
  }
  if (lane == 0) {
    sh_pm[wid] = pm;
    sh_am[wid] = pi;
  }
  __syncthreads();
  for (int w = 0; w < 16; ++w)
    if (sh_pm[w] > pm || (sh_pm[w] == pm && sh_am[w] < pi)) {
      pm = sh_pm[w];
      pi = sh_am[w];
    }
  const int am = pm > 0.0 ? pi / K : 0, bm = pm > 0.0 ? pi % K : 0;
  // start of every grid side in descending order (sides are at most 128)
  int above = 0;
  if (tid < 256)
    for (int v = tid + 1; v < 256; ++v) above += start[v];
  __syncthreads();
  if (tid < 256) start[tid] = above;
  // PSF factorisation P[a][b] = gy[a] * gx[b]
  for (int i = tid; i < K * K; i += 1024) tp[ti.psf + i] = psh[i];
  if (pm > 0.0 && tid < K) {
    tp[ti.gy + tid] = psh[tid * K + bm];
    tp[ti.gx + tid] = psh[am * K + tid] / psh[am * K + bm];
  }
  __syncthreads();
  for (int i = tid; i < K * K; i += 1024)
    if (fabs(psh[i] - tp[ti.gy + i / K] * tp[ti.gx + i % K]) > 1e-12 * pm) sh_sep = 0;
  // Counting sort of the members by descending ns, stable in member index:
  // rank r -> queue r % 8, position r / 8.  Within a queue the `heavy`
  // smallest lambdas of every member come first (their solves take the most
  // CG iterations, so starting them early shortens the tail of the launch),
  // then the other lambdas; both parts keep the members in order, so the
  // blocks of an XCD share few members at a time and their tables stay in its
  // L2.
  const int NL = a.n_lambda, H = min(NL, a.heavy);
  for (int m0 = 0; m0 < M; m0 += 1024) {
    const int m = m0 + tid;
    const int ns = m < M ? a.ns[m] : 0;
    const int key = m < M ? (ns >= 2 && ns <= a.max_ns ? ns : 0) : 255;   // 255: past the last member
    const unsigned long long same = match8(key);
    const int before = lanes_below(same);
    if (before == 0) wcnt[wid][key] = __popcll(same);
    __syncthreads();
    if (m < M) {
      int r = start[key] + before;
      for (int w = 0; w < wid; ++w) r += wcnt[w][key];
      const int q = r & 7, t = r >> 3;
      const int nmq = (M - q + 7) / 8;   // members in queue q
      int* Q = a.queues + q * a.qcap;
      for (int k = 0; k < H; ++k) Q[t * H + k] = m * NL + k;
      for (int k = H; k < NL; ++k) Q[nmq * H + t * (NL - H) + (k - H)] = m * NL + k;
    }
    __syncthreads();
    if (tid < 256) {
      int n = 0;
      for (int w = 0; w < 16; ++w) {
        n += wcnt[w][tid];
        wcnt[w][tid] = 0;
      }
      start[tid] += n;
    }
    __syncthreads();
  }
  if (tid < 8) {   // members with rank q + 8 t fill queue q densely
    const int nm = M > tid ? (M - tid + 7) / 8 : 0;
    a.consts->qcount[tid] = nm * NL;
    a.consts->qhead[tid] = 0;
    a.consts->pqcount[tid] = 0;
    a.consts->pqhead[tid] = 0;
  }
  // the banded path needs the kernel's window to cover +-2ck
  const bool sep = pm > 0.0 && sh_sep && ck <= a.ckt && !a.force_direct;
  if (tid == 0) a.consts->sep = sep;
  if (sep) {
    // autocorrelations a[d] = sum_i g[i] g[i-d], stored at index d + 2*kMaxCK
    for (int e = tid; e < 2 * (2 * K - 1); e += 1024) {
      const int dd = e / 2 - (K - 1), g0 = e & 1 ? ti.gy : ti.gx;
      double s = 0.0;
      for (int i = 0; i < K; ++i) {
        const int j = i - dd;
        if (j < 0 || j >= K) continue;
        s += tp[g0 + i] * tp[g0 + j];
      }
      tp[(e & 1 ? ti.ay : ti.ax) + dd + 2 * kMaxCK] = s;
    }
    // edge corrections: the truncated 1-D convolution C has (C^T C)[c][c']
    // = a[c'-c] - sum over intermediate indices k outside the image
    for (int e = tid; e < 4 * ck * ck; e += 1024) {
      const int p = (e >> 2) / ck, q = (e >> 2) % ck, g0 = e & 1 ? ti.gy : ti.gx;
      double s = 0.0;
      if (!(e & 2)) {
        for (int k = -ck; k < 0; ++k) {
          const int i1 = k - p + ck, i2 = k - q + ck;
          if (i1 >= 0 && i1 < K && i2 >= 0 && i2 < K) s += tp[g0 + i1] * tp[g0 + i2];
        }
        tp[(e & 1 ? ti.ely : ti.elx) + p * ck + q] = s;
      } else {
        // right edge: outputs c = n - ck + p, inputs c' = n - ck + q, k = n + kk
        for (int kk = 0; kk < ck; ++kk) {
          const int i1 = kk + 2 * ck - p, i2 = kk + 2 * ck - q;   // k - c + ck, k - c' + ck
          if (i1 >= 0 && i1 < K && i2 >= 0 && i2 < K) s += tp[g0 + i1] * tp[g0 + i2];
        }
        tp[(e & 1 ? ti.ery : ti.erx) + p * ck + q] = s;
      }
    }
  }
  __syncthreads();
  T* tt = reinterpret_cast<T*>(a.taps_t);
  for (int i = tid; i < ti.total; i += 1024) {
    a.taps_d[i] = tp[i];
    tt[i] = (T)tp[i];
  }
  // sums of d^2 and of the Monte Carlo draws squared, in FP64
  double acc = 0.0, accn = 0.0;
  const int J = a.nx * a.ny;
  for (int j = tid; j < J; j += 1024) {
    acc += a.d[j] * a.d[j];
    if (a.mcn) accn += a.mcn[j] * a.mcn[j];
  }
  acc = block_sum(acc, red);
  accn = block_sum(accn, red);
  if (tid == 0) {
    a.consts->sum_d2 = acc;
    a.consts->sum_n2 = accn;
    a.consts->mchead = 0;
    a.consts->imhead = 0;
  }
}

// Byte offsets of a member's arrays in dynamic LDS.
struct LdsPlan {
  int p, q, red, frame;
};
template <typename T>
__host__ __device__ __forceinline__ LdsPlan lds_plan(const SolveArgs& a, int I, int mem) {
  if (sizeof(T) == 4) return {0, a.q_off, a.red_off, a.frame_off};
  const int red = 64 * (int)sizeof(double), v = ((int)sizeof(T) * I + 255) & ~255;
  return {red, red + v, 0, red + (mem == kMemLdsQGlobal ? v : 2 * v)};
}

// Where q of a member with its frame in LDS lives: in LDS, but in global memory
// for FP64 with the wider windows, whose frames leave it no room more often
// than not.  (One place per kernel: an FP64 kernel with all three forms grew
// past what the compiler takes apart, its arguments stayed in scratch memory
// and every access through their pointers became a flat one.)
template <typename T>
__host__ __device__ constexpr int lds_mem(int ckt) {
  return sizeof(T) == 8 && ckt > 2 ? kMemLdsQGlobal : kMemLds;
}

// Where a launch's frames are not all sure to fit, FP64 members with more nodes
// keep a global frame, unless theirs fits at the offsets of the largest grid.  p
// alone takes 72 KB or more of theirs, so some members' frames would fit beside
// it and others' not, and the others' items, the longest of the launch, set its
// time: 64 members of 32..96 nodes per side on a 128 x 128 image with Monte Carlo
// degrees of freedom take the same time within its spread with the limit and
// without (1.67x and 1.64x of one earlier build's speed), so the line stays where
// the common offsets had it on such images (the global form is tested there, at
// 95 and 96 nodes).  Where all frames fit, LDS is the faster place: 64 members of
// 95..100 nodes on a 64 x 64 image, K = 15, 24.1 ms in global memory, 19.5 in LDS.
constexpr int kLdsNodesF64 = 9000;

// Elements of the frame of an h x w box.
__host__ __device__ __forceinline__ long frame_size(int h, int w, int ckt) {
  return (long)(h + 4 * ckt + kSegR) * ((w + 4 * ckt) | 1);
}

// Mem of a member whose frame has `elems` elements.
template <typename T>
__host__ __device__ __forceinline__ int mem_of(const SolveArgs& a, int I, long elems) {
  if (sizeof(T) == 4) return elems <= a.lds_frame_cap ? kMemLds : kMemGlobal;
  const int mem = a.one_vector ? (int)kMemLdsQGlobal : lds_mem<T>(a.ckt);
  if (lds_plan<T>(a, I, mem).frame + elems * (long)sizeof(T) > a.lds_bytes) return kMemGlobal;
  return I <= kLdsNodesF64 || a.frames_fit || elems <= a.lds_frame_cap ? mem : (int)kMemGlobal;
}

// ------------------------------------------------------------------ member set-up (k_prep_*)
// The tables of every member, by five grid-wide kernels (one block per member
// did all of it before: 2.9 ms for a single 128 x 128 lens, 4.0 ms for 256 of
// them, nearly all of it waves waiting on one another's cursors and on one
// wave's ordered sums; the five take 0.14 and 0.95 ms):
//   k_prep_trace   the FP64 subpixel trace, once, and B^T d once per call
//   k_prep_place   compaction into the interleaved trace table
//   k_prep_layout  row lengths of L^T, their order and the storage layout
//   k_prep_fill    L^T's entries in their fixed order
//   k_prep_rhs     entries' offsets and weights, b = L^T B^T d row by row
// Everything that is summed keeps one fixed order, the same on every run and
// whatever the grid.

constexpr int kPrepT = 256;     // threads (pixels) per block of k_prep_trace and k_prep_place
constexpr int kFillBand = 2048; // nodes whose fill cursors (kFillW waves x 4 bytes each) one block holds in LDS

// The traced subpixels in pixel order, kept between k_prep_trace and
// k_prep_place in the member's L^T entry region (64 n^2 bytes or more per
// pixel, written only later): one mapped bit per pixel, then cells and fractions.
template <typename T>
struct PixTmp {
  unsigned long long* words;   // [ceil(J/64)]
  int32_t* cell;               // [J][n^2]
  T* fx;
  T* fy;
  __device__ PixTmp(const SolveArgs& a, int m) {
    const long J = (long)a.nx * a.ny;
    const long nw = ((J + 63) / 64 + 1) & ~1L;   // 16-byte alignment of what follows
    words = reinterpret_cast<unsigned long long*>(reinterpret_cast<LtEntry<T>*>(a.lt_ent) + (long)m * a.lt_cap);
    fx = reinterpret_cast<T*>(words + nw);
    fy = fx + ((J * a.n2 + 3) & ~3L);
    cell = reinterpret_cast<int32_t*>(fy + ((J * a.n2 + 3) & ~3L));
  }
};

// Bounds: FP64 arithmetic of the trace (atan, atanh and two square roots per
// subpixel) and, for a single member, launch latency.  One thread per pixel;
// every lane keeps its subpixels' cells and fractions for the compaction, so
// each subpixel is traced once (the counting, placing and writing passes each
// traced it again before).  The blocks past the members' compute B^T img
// (img = d, then the Monte Carlo draws) over the image once for all members.
template <typename T>
__global__ void __launch_bounds__(kPrepT) k_prep_trace(SolveArgs a) {
  __shared__ Lens Ls;
  __shared__ int valid, bb[4];
  const int tid = threadIdx.x, J = a.nx * a.ny, tiles = (J + kPrepT - 1) / kPrepT;
  const int m = blockIdx.x / tiles, j = (blockIdx.x % tiles) * kPrepT + tid;
  const int nx = a.nx, ny = a.ny, nsub = a.nsub, n2 = a.n2;
  const int r = j / nx, c = j % nx;
  if (m >= a.n_members) {   // correlation with the PSF: row of the PSF outer, column inner
    const double* img = m == a.n_members ? a.d : a.mcn;
    const int K = a.K, ck = a.ck;
    if (j >= J) return;
    double v = 0.0;
    for (int aa = 0; aa < K; ++aa) {
      const int rr = r + aa - ck;
      if (rr < 0 || rr >= ny) continue;
      for (int b0 = 0; b0 < K; b0 += 8) {   // eight taps in flight; a tap off the image adds zero
        double x[8], p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int cc = c + b0 + u - ck;
          const bool on = b0 + u < K && cc >= 0 && cc < nx;
          x[u] = on ? img[rr * nx + cc] : 0.0;
          p[u] = b0 + u < K ? a.psf[aa * K + b0 + u] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) v += p[u] * x[u];
      }
    }
    a.btd[(long)(m - a.n_members) * J + j] = v;
    return;
  }
  const int ns = a.minfo[m].ns;
  if (tid == 0) {
    double g[7];
    for (int i = 0; i < 7; ++i) g[i] = a.lens[7L * m + i];
    valid = ns >= 2 && lens_valid(g);
    Ls = make_lens(g);
    bb[0] = bb[2] = INT_MAX;
    bb[1] = bb[3] = INT_MIN;
  }
  __syncthreads();
  const PixTmp<T> tmp(a, m);
  bool mapped = false;
  if (valid && j < J) {
    const Lens L = Ls;
    const double h = 2.0 * a.R / (ns - 1);
    for (int k = 0; k < n2; ++k) {
      double x, y, bx, by, fx = 0.0, fy = 0.0;
      int cell;
      subpixel_xy(r, c, k / nsub, k % nsub, nx, ny, a.pix, nsub, x, y);
      lens_map(L, x, y, bx, by);
      const bool in = grid_cell((bx + a.R) / h, (by + a.R) / h, ns, cell, fx, fy);
      if (!in) {
        cell = -1;
        fx = fy = 0.0;
      } else if (a.interp == SL_INTERP_NEAREST) {   // the nearest of the cell's four nodes, weight 1
        fx = fx >= 0.5 ? 1.0 : 0.0;
        fy = fy >= 0.5 ? 1.0 : 0.0;
      }
      mapped |= in;
      tmp.cell[(long)j * n2 + k] = cell;
      tmp.fx[(long)j * n2 + k] = (T)fx;
      tmp.fy[(long)j * n2 + k] = (T)fy;
    }
  }
  const unsigned long long bal = __ballot(mapped);
  if ((tid & 63) == 0 && j < J) tmp.words[j >> 6] = bal;
  if (mapped) {
    atomicMin(&bb[0], r);
    atomicMax(&bb[1], r);
    atomicMin(&bb[2], c);
    atomicMax(&bb[3], c);
  }
  __syncthreads();
  if (tid == 0 && bb[1] >= 0) {
    MemberInfo& mi = a.minfo[m];
    atomicMin(&mi.r0, bb[0]);
    atomicMax(&mi.r1, bb[1]);
    atomicMin(&mi.c0, bb[2]);
    atomicMax(&mi.c1, bb[3]);
  }
}

// A member's masks (below): 16 bits each hold those of up to 2 x 2 subpixels.
__host__ __device__ __forceinline__ size_t mask_bytes(int n2) { return n2 <= 4 ? 2 : 8; }
struct PairMasks {
  void* p;
  bool narrow;
  __device__ PairMasks(const SolveArgs& a, int m)
      : p(static_cast<unsigned char*>(a.pmask) + mask_bytes(a.n2) * (size_t)m * a.slot_cap), narrow(a.n2 <= 4) {}
  __device__ unsigned long long operator[](int t) const {
    return narrow ? static_cast<const unsigned short*>(p)[t] : static_cast<const unsigned long long*>(p)[t];
  }
  __device__ void set(int t, unsigned long long mask) const {
    if (narrow) static_cast<unsigned short*>(p)[t] = (unsigned short)mask;
    else static_cast<unsigned long long*>(p)[t] = mask;
  }
};

// First-occurrence mask of a pixel's 4 n^2 (subpixel, corner) pairs: bit 4 k +
// corner is set when subpixel k lies on the grid and no earlier subpixel
// reaches that node.  (corner 0..3: nodes c, c + 1, c + ns, c + ns + 1)
__device__ __forceinline__ int corner_node(int cell, int corner, int ns) {
  return cell + (corner & 1) + (corner >> 1) * ns;
}
__device__ __forceinline__ unsigned long long pair_mask(const int32_t* cell, int n2, int ns) {
  unsigned long long mask = 0;
  for (int k = 0; k < n2; ++k) {
    const int ck = cell[k];
    if (ck < 0) continue;
    unsigned f = 15u;
    for (int l = 0; l < k; ++l) {
      const int cl = cell[l];
      if (cl < 0) continue;
      // corners of subpixel k that are corners of subpixel l: their cells differ by at most one row and column
      for (int q = 0; q < 4; ++q) {
        const int d = corner_node(ck, q, ns) - cl;
        if (d == 0 || d == 1 || d == ns || d == ns + 1) f &= ~(1u << q);
      }
    }
    mask |= (unsigned long long)f << (4 * k);
  }
  return mask;
}

// Compaction: entry pos (rank of the mapped pixel in row order) goes to slot
// (pos % S) * 64 + pos / S of the interleaved table, so that the 64 lanes of a
// wave take pixels spread over the whole mapped region; slots past the last
// entry hold -1.  Each block counts the mapped bits before its pixels itself
// (at most 1024 words), so no pass over the whole image is needed between the
// trace and this copy.  Bound by the record copies (48 bytes per pixel read
// and written in FP32 with 2 x 2 subpixels).
template <typename T>
__global__ void __launch_bounds__(kPrepT) k_prep_place(SolveArgs a) {
  __shared__ int red[2][kPrepT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int J = a.nx * a.ny, tiles = (J + kPrepT - 1) / kPrepT, nwords = (J + 63) / 64;
  const int m = blockIdx.x / tiles, tile = blockIdx.x % tiles, j = tile * kPrepT + tid;
  const int n2 = a.n2;
  const PixTmp<T> tmp(a, m);
  const PairMasks pm(a, m);
  const int ns = a.minfo[m].ns;
  const int w0 = tile * (kPrepT / 64) + wid;   // this wave's word
  int before = 0, total = 0;
  for (int i = tid; i < nwords; i += kPrepT) {
    const int n = __popcll(tmp.words[i]);
    total += n;
    before += i < tile * (kPrepT / 64) ? n : 0;
  }
  total = wave_sum(total);
  before = wave_sum(before);
  if (lane == 0) {
    red[0][wid] = total;
    red[1][wid] = before;
  }
  __syncthreads();
  total = before = 0;
  for (int i = 0; i < kPrepT / 64; ++i) {
    total += red[0][i];
    before += red[1][i];
  }
  const int Mtrue = total, S = (Mtrue + 63) / 64, slots = 64 * S;
  int32_t* pix = a.pix_list + (long)m * a.slot_cap;
  int32_t* cellp = a.cell + (long)m * a.slot_cap * n2;
  T* fxp = reinterpret_cast<T*>(a.fx) + (long)m * a.slot_cap * n2;
  T* fyp = reinterpret_cast<T*>(a.fy) + (long)m * a.slot_cap * n2;
  if (tile == 0) {
    if (tid < 64 && Mtrue + tid < slots) {   // fewer than 64 empty slots
      const int p = Mtrue + tid, slot = (p % S) * 64 + p / S;
      pix[slot] = -1;
      pm.set(slot, 0ull);
      for (int k = 0; k < n2; ++k) {
        cellp[(long)slot * n2 + k] = -1;
        fxp[(long)slot * n2 + k] = (T)0;
        fyp[(long)slot * n2 + k] = (T)0;
      }
    }
    if (tid == 0) {   // the trace kernel has left the bounding box in r0..c1
      MemberInfo mi = a.minfo[m];
      double g[7];
      for (int i = 0; i < 7; ++i) g[i] = a.lens[7L * m + i];
      mi.M = slots;
      mi.Mtrue = Mtrue;
      mi.status = !(ns >= 2 && lens_valid(g)) ? SL_ST_INVALID : Mtrue > 0 ? SL_ST_OK : SL_ST_EMPTY;
      if (Mtrue == 0) {
        mi.r0 = mi.c0 = 0;
        mi.r1 = mi.c1 = -1;
      }
      mi.lds_frame = mem_of<T>(a, mi.I, frame_size(mi.r1 - mi.r0 + 1, mi.c1 - mi.c0 + 1, a.ckt));
      mi.sell = 0;
      mi.pc_c = 0.0f;
      a.minfo[m] = mi;
    }
  }
  if (j >= J) return;
  const unsigned long long word = tmp.words[w0];
  if (!((word >> lane) & 1ull)) return;
  for (int i = tile * (kPrepT / 64); i < w0; ++i) before += __popcll(tmp.words[i]);
  const int pos = before + __popcll(word & ((1ull << lane) - 1ull));
  const int slot = (pos % S) * 64 + pos / S;
  pix[slot] = ((j / a.nx) << 16) | (j % a.nx);   // packed row/column of the mapped pixel
  if (n2 == 4) {
    const int4 c4 = reinterpret_cast<const int4*>(tmp.cell)[j];
    reinterpret_cast<int4*>(cellp)[slot] = c4;
    if constexpr (sizeof(T) == 4) {
      reinterpret_cast<float4*>(fxp)[slot] = reinterpret_cast<const float4*>(tmp.fx)[j];
      reinterpret_cast<float4*>(fyp)[slot] = reinterpret_cast<const float4*>(tmp.fy)[j];
    } else {
      for (int k = 0; k < 4; ++k) {
        fxp[4L * slot + k] = tmp.fx[4L * j + k];
        fyp[4L * slot + k] = tmp.fy[4L * j + k];
      }
    }
    const int32_t cl[4] = {c4.x, c4.y, c4.z, c4.w};
    pm.set(slot, pair_mask(cl, 4, ns));
  } else {
    for (int k = 0; k < n2; ++k) {
      cellp[(long)slot * n2 + k] = tmp.cell[(long)j * n2 + k];
      fxp[(long)slot * n2 + k] = tmp.fx[(long)j * n2 + k];
      fyp[(long)slot * n2 + k] = tmp.fy[(long)j * n2 + k];
    }
    pm.set(slot, pair_mask(tmp.cell + (long)j * n2, n2, ns));
  }
}

// Cubic convolution kernel (Keys 1981, a = -1/2) at distance d >= 0 from a
// node; the tap at offset o (-1..2) from a cell's first node lies at
// distance |f - o| for the fraction f in [0, 1].
template <typename F>
__device__ __forceinline__ F keys_w(F d) {
  return d <= F(1) ? (F(1.5) * d - F(2.5)) * d * d + F(1)
                   : (d < F(2) ? ((F(-0.5) * d + F(2.5)) * d - F(4)) * d + F(2) : F(0));
}

// Pair q of mapped slot t: the node it adds to, -1 for none.
//
// Bilinear and nearest: q = 4 k + corner (q < 4 n^2), the pair of a node that
// an earlier subpixel of the pixel already reaches being folded into that one
// (pmask).  Bicubic: q = 16 k + 4 (j + 1) + (i + 1) (q < 16 n^2), the tap at row
// offset j and column offset i from subpixel k's cell; taps outside the grid
// are left out (the source is zero there), and pairs are not folded.
__device__ __forceinline__ int pair_node(bool cubic, int q, int ns, unsigned long long mask, const int32_t* cell) {
  if (!cubic) return (mask >> q) & 1ull ? corner_node(cell[q >> 2], q & 3, ns) : -1;
  const int c = cell[q >> 4];
  if (c < 0) return -1;
  const int r = c / ns + ((q >> 2) & 3) - 1, col = c % ns + (q & 3) - 1;
  return r < 0 || r >= ns || col < 0 || col >= ns ? -1 : r * ns + col;
}

// The weight below for 2 x 2 subpixels with cells cl and fractions f, g.
template <typename T>
__device__ __forceinline__ double pair_weight4(int node, int ns, const int32_t* cl, const T* f, const T* g) {
  double w = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double fx = (double)f[k], fy = (double)g[k];
    const int d = node - cl[k];
    const double wx = d == 0 || d == ns ? 1 - fx : fx, wy = d == 0 || d == 1 ? 1 - fy : fy;
    const double wk = wx * wy * 0.25;
    w += cl[k] >= 0 && (d == 0 || d == 1 || d == ns || d == ns + 1) ? wk : 0.0;
  }
  return w;
}

// FP64 weight of mapped slot t's pair q at `node`, the 1/n^2 subpixel average
// included: for bilinear and nearest L the weights of all the pixel's
// subpixels at the node, added in subpixel order.
template <typename T>
__device__ __forceinline__ double pair_weight(bool cubic, int t, int q, int node, int ns, int n2, const int32_t* cellp,
                                              const T* fxp, const T* fyp) {
  if (cubic) {
    const int k = q >> 4, j = (q >> 2) & 3, i = q & 3;
    const double fx = (double)fxp[(long)t * n2 + k], fy = (double)fyp[(long)t * n2 + k];
    return keys_w(fabs(fy - (j - 1))) * keys_w(fabs(fx - (i - 1))) / n2;
  }
  if (n2 == 4) {
    const int4 c4 = reinterpret_cast<const int4*>(cellp)[t];
    const int cl[4] = {c4.x, c4.y, c4.z, c4.w};
    return pair_weight4(node, ns, cl, fxp + 4L * t, fyp + 4L * t);
  }
  const double inv = 1.0 / n2;
  double w = 0.0;
  for (int k = 0; k < n2; ++k) {
    const int c = cellp[(long)t * n2 + k], d = node - c;
    if (c < 0 || !(d == 0 || d == 1 || d == ns || d == ns + 1)) continue;
    const double fx = (double)fxp[(long)t * n2 + k], fy = (double)fyp[(long)t * n2 + k];
    const double ww = (d == 0 || d == ns ? 1 - fx : fx) * (d == 0 || d == 1 ? 1 - fy : fy);
    w += ww * inv;
  }
  return w;
}

// Quarter-octave bucket of a row length (0 for empty rows): rows in one
// bucket differ by less than 19%.
__device__ __forceinline__ int len_bucket(int c) {
  if (c <= 0) return 0;
  const int msb = 31 - __clz(c);
  const int frac = msb >= 2 ? (c >> (msb - 2)) & 3 : (c << (2 - msb)) & 3;
  return 4 * msb + frac + 1;
}

// Layout of L^T for one member (node-major form, sliced-ELL with rows sorted
// by length: SELL-C-sigma with C = 64, one slice per wave): nodes are ordered
// by descending length bucket (stable in node index) into perm[] = packed
// (row << 16 | col); entry j of the node at position p sits at ptr[p/64] + 64 j
// + p%64, every slice padded to its longest row with entries (offset 0, weight
// 0) -- offset 0 is a frame halo element, always zero.  Falls back to plain CSR
// in node order (ptr = row starts) when the padded form exceeds the capacity.
// Members whose frame fits in LDS (frame offsets below 2^16) store the
// sliced-ELL entries in pairs: slices of even length, one dword holding the
// 16-bit offsets of entries 2k and 2k + 1 of a lane and one EntryPair their
// weights (6 bytes per entry instead of 8 in FP32, 10 instead of 16 in FP64).
//
// One block per member: the row lengths are counted with LDS atomics, which a
// grid-wide count would have to do in memory, and the sixteen waves place
// contiguous node ranges (a histogram per wave and an exclusive scan over the
// waves keep the order that of the node index).
// dynamic LDS: cnt[I], pcnt[I + 64], whist[16][128], slen[SL]; SL = slices + 1.
template <typename T>
__global__ void __launch_bounds__(1024) k_prep_layout(SolveArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int hist[128], scan[16], totals;
  const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, n2 = a.n2;
  const MemberInfo mi = a.minfo[m];
  if (__builtin_amdgcn_readfirstlane(mi.status) != SL_ST_OK) return;
  const int ns = mi.ns, I = mi.I, slots = mi.M, ngroups = (I + 63) / 64;
  int* cnt = reinterpret_cast<int*>(smem);   // row lengths
  int* pcnt = cnt + I;                       // row lengths in sorted order (positions past I: 0)
  int* whist = pcnt + I + 64;                // per-wave bucket histograms, later positions
  int* slen = whist + 16 * 128;              // slice lengths, then slice starts
  const int32_t* cellp = a.cell + (long)m * a.slot_cap * n2;
  const PairMasks pm(a, m);
  int32_t* rp = a.lt_ptr + (long)m * (a.I_max + 65);
  int32_t* perm = a.lt_perm + (long)m * a.I_max;
  int32_t* lbase = a.lt_base + (long)m * a.I_max;
  int32_t* lcnt = a.lt_cnt + (long)m * a.I_max;
  const bool cubic = a.interp == SL_INTERP_BICUBIC;
  for (int i = tid; i < I; i += 1024) cnt[i] = 0;
  for (int i = tid; i < 16 * 128; i += 1024) whist[i] = 0;
  if (tid < 64) pcnt[I + tid] = 0;
  if (tid == 0) totals = 0;
  __syncthreads();
  for (int t = tid; t < slots; t += 1024) {
    if (cubic) {
      for (int q = 0; q < 16 * n2; ++q) {
        const int nd = pair_node(true, q, ns, 0ull, cellp + (long)t * n2);
        if (nd >= 0) atomicAdd(&cnt[nd], 1);
      }
    } else if (n2 == 4) {
      const unsigned mask = (unsigned)pm[t];
      const int4 c4 = reinterpret_cast<const int4*>(cellp)[t];
      const int cl[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if ((mask >> q) & 1u) atomicAdd(&cnt[corner_node(cl[q >> 2], q & 3, ns)], 1);
    } else {
      for (unsigned long long mask = pm[t]; mask; mask &= mask - 1) {
        const int q = __ffsll((unsigned long long)mask) - 1;
        atomicAdd(&cnt[corner_node(cellp[(long)t * n2 + (q >> 2)], q & 3, ns)], 1);
      }
    }
  }
  __syncthreads();
  // stable placement: wave w takes the node groups [w G / 16, (w + 1) G / 16)
  const int g0 = (wid * ngroups) / 16, g1 = ((wid + 1) * ngroups) / 16;
  for (int g = g0; g < g1; ++g) {
    const int i = 64 * g + lane;
    if (i < I) {
      const int c = cnt[i];
      atomicAdd(&whist[wid * 128 + len_bucket(c)], 1);
      lcnt[i] = c;
    }
  }
  __syncthreads();
  if (tid < 128) {
    int s = 0;
    for (int w = 0; w < 16; ++w) {
      const int c = whist[w * 128 + tid];
      whist[w * 128 + tid] = s;   // nodes of this bucket in the waves before w
      s += c;
    }
    hist[tid] = s;
  }
  __syncthreads();
  int above = 0;
  if (tid < 128)
    for (int b = tid + 1; b < 128; ++b) above += hist[b];   // descending buckets
  if (tid < 128)
    for (int w = 0; w < 16; ++w) whist[w * 128 + tid] += above;
  __syncthreads();
  for (int g = g0; g < g1; ++g) {
    const int i = 64 * g + lane, c = i < I ? cnt[i] : 0;
    const int b = i < I ? len_bucket(c) : 127;   // 127: no row length reaches it
    const unsigned long long same = match8(b);
    int* pos = &whist[wid * 128 + b];
    const int p = *pos + lanes_below(same);
    if (i < I) {
      perm[p] = ((i / ns) << 16) | (i % ns);
      pcnt[p] = c;
      lbase[i] = p;
    }
    // every lane has read its bucket's position before the bucket's last lane advances it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (i < I && (same >> lane) == 1ull) *pos = p + 1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  __syncthreads();
  const bool pair_ok =
      mi.lds_frame != kMemGlobal && frame_size(mi.r1 - mi.r0 + 1, mi.c1 - mi.c0 + 1, a.ckt) <= 65536;
  for (int g = wid; g < ngroups; g += 16) {
    int mx = pcnt[64 * g + lane];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o, 64));
    if (pair_ok) mx = (mx + 1) & ~1;
    if (lane == 0) {
      slen[g] = 64 * mx;
      atomicAdd(&totals, 64 * mx);
    }
  }
  __syncthreads();
  const int sell = __builtin_amdgcn_readfirstlane((int)(!a.force_csr && (long long)totals <= a.lt_cap));
  // exclusive scan over units: slices for sliced-ELL, rows for CSR
  const int nunits = sell ? ngroups : I;
  const int* size = sell ? slen : cnt;
  const int chunk = (nunits + 1023) / 1024;
  const int u0 = min(nunits, tid * chunk), u1 = min(nunits, u0 + chunk);
  int local = 0;
  for (int u = u0; u < u1; ++u) local += size[u];
  int incl = local;
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  if (lane == 63) scan[wid] = incl;
  __syncthreads();
  int run = incl - local;
  for (int i = 0; i < wid; ++i) run += scan[i];
  for (int u = u0; u < u1; ++u) {
    const int n = size[u];
    rp[u] = run;
    if (sell) slen[u] = run;
    else lbase[u] = run;
    run += n;
  }
  if (tid == 1023) rp[nunits] = run;
  __syncthreads();
  if (sell)   // entry base of every node
    for (int i = tid; i < I; i += 1024) {
      const int p = lbase[i];
      lbase[i] = slen[p >> 6] + (p & 63);
    }
  if (tid == 0) a.minfo[m].sell = sell && pair_ok ? 2 : sell;
}

// Position of entry j of the node with entry base `base` in the arrays of each layout.
__device__ __forceinline__ long paired_index(int base, int j) {   // index into the 16-bit offsets and the weights
  return 2 * (((long)(base & ~63) >> 1) + 64L * (j >> 1) + (base & 63)) + (j & 1);
}

// The entries of L^T as codes (slot << 8 | pair), placed in their fixed order:
// a node's entries are ordered by (slot group of 64, pair, lane), the order
// of one wave walking all groups pair by pair.  One block takes the nodes
// [kFillBand b, kFillBand (b + 1)) of one member and all of its slots; wave w
// takes the slot groups [w G / 16, (w + 1) G / 16).  A first pass counts every
// node's entries per wave, an exclusive scan over the waves gives each wave
// the position after the groups before its range, and the second pass places
// them: within a step (one pair of 64 slots) each lane draws its position
// with an LDS atomic, and where lanes share a node they are ranked in lane
// order.  The cursors live in LDS: from global memory each step waited on a
// round trip to L2 (2.1 ms for a 128 x 128 lens on one wave, 20 us here).
// Folded pairs of other than 2 x 2 subpixels are ordered by their rank among
// the pixel's pairs.
template <typename T>
__global__ void __launch_bounds__(1024) k_prep_fill(SolveArgs a, int bands) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int m = blockIdx.x / bands, n0 = (blockIdx.x % bands) * kFillBand;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, n2 = a.n2;
  const MemberInfo mi = a.minfo[m];
  if (__builtin_amdgcn_readfirstlane((int)(mi.status != SL_ST_OK || n0 >= mi.I))) return;
  const int ns = mi.ns, nb = min(kFillBand, mi.I - n0), G = mi.M / 64, sell = mi.sell;
  const int cap = min(kFillBand, a.I_max);
  int* cur = reinterpret_cast<int*>(smem) + (long)wid * cap;   // this wave's cursors
  int* all = reinterpret_cast<int*>(smem);
  int* base = all + (long)kFillW * cap;
  const int32_t* cellp = a.cell + (long)m * a.slot_cap * n2;
  const PairMasks pm(a, m);
  const int32_t* lbase = a.lt_base + (long)m * a.I_max;
  LtEntry<T>* ent = reinterpret_cast<LtEntry<T>*>(a.lt_ent) + (long)m * a.lt_cap;
  const int E = a.lt_ptr[(long)m * (a.I_max + 65) + (mi.I + 63) / 64];   // sliced-ELL entries
  T* w2 = reinterpret_cast<T*>(reinterpret_cast<unsigned short*>(ent) + E);   // the paired form's weights
  const bool cubic = a.interp == SL_INTERP_BICUBIC;
  for (int i = tid; i < kFillW * cap; i += 1024) all[i] = 0;
  for (int i = tid; i < nb; i += 1024) base[i] = lbase[n0 + i];
  __syncthreads();
  const int g0 = (wid * G) / kFillW, g1 = ((wid + 1) * G) / kFillW;
  const int nq = cubic ? 16 * n2 : 4 * n2;
  for (int g = g0; g < g1; ++g) {
    const int t = g * 64 + lane;
    const unsigned long long mask = pm[t];
    if (n2 == 4 && !cubic) {
      const int4 c4 = reinterpret_cast<const int4*>(cellp)[t];
      const int cl[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const unsigned nd = (unsigned)(corner_node(cl[q >> 2], q & 3, ns) - n0);
        if (((unsigned)mask >> q) & 1u && nd < (unsigned)nb) atomicAdd(&cur[nd], 1);
      }
    } else {
      for (int q = 0; q < nq; ++q) {
        const int nd = pair_node(cubic, q, ns, mask, cellp + (long)t * n2) - n0;
        if ((unsigned)nd < (unsigned)nb && nd + n0 >= 0) atomicAdd(&cur[nd], 1);
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < nb; i += 1024) {   // exclusive scan over the waves
    int run = 0;
    for (int w = 0; w < kFillW; ++w) {
      const int c = all[(long)w * cap + i];
      all[(long)w * cap + i] = run;
      run += c;
    }
  }
  __syncthreads();
  // nd: node within the band, -1 for none
  auto place = [&](int nd, int code) {
    if (!__builtin_amdgcn_readfirstlane((int)(__ballot(nd >= 0) != 0ull))) return;   // uniform
    int j = 0, after = 1;
    if (nd >= 0) j = atomicAdd(&cur[nd], 1);
    // one wave's LDS accesses complete in order: the read sees every lane's add
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (nd >= 0) after = *reinterpret_cast<volatile int*>(&cur[nd]) - j;
    // a lane that was not its node's last add sees more than its own: each such node's lanes are ranked
    unsigned long long clash = __ballot(nd >= 0 && after != 1);
    while (clash) {
      const int k0 = __builtin_amdgcn_readlane(nd, __ffsll((unsigned long long)clash) - 1);
      const unsigned long long same = __ballot(nd == k0);
      if (nd == k0) j = j + after - __popcll(same) + lanes_below(same);
      clash &= ~same;
    }
    if (nd >= 0) {
      if (sell == 2) *reinterpret_cast<int*>(&w2[paired_index(base[nd], j)]) = code;
      else ent[(long)base[nd] + (sell ? 64L : 1L) * j].off = code;
    }
    __builtin_amdgcn_wave_barrier();
  };
  for (int g = g0; g < g1; ++g) {   // uniform per wave
    const int t = g * 64 + lane;
    const unsigned long long mask = pm[t];
    if (n2 == 4 && !cubic) {
      const int4 c4 = reinterpret_cast<const int4*>(cellp)[t];
      const int cl[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const unsigned nd = (unsigned)(corner_node(cl[q >> 2], q & 3, ns) - n0);
        place(((unsigned)mask >> q) & 1u && nd < (unsigned)nb ? (int)nd : -1, (t << 8) | q);
      }
    } else if (cubic) {
      for (int q = 0; q < nq; ++q) {
        const int nd = pair_node(true, q, ns, 0ull, cellp + (long)t * n2);
        place(nd >= n0 && nd - n0 < nb ? nd - n0 : -1, (t << 8) | q);
      }
    } else {
      unsigned long long rest = mask;
      while (__builtin_amdgcn_readfirstlane((int)(__ballot(rest != 0ull) != 0ull))) {
        int nd = -1, q = 0;
        if (rest) {
          q = __ffsll(rest) - 1;
          rest &= rest - 1;
          nd = corner_node(cellp[(long)t * n2 + (q >> 2)], q & 3, ns) - n0;
          if (nd < 0 || nd >= nb) nd = -1;
        }
        place(nd, (t << 8) | q);
      }
    }
  }
}

// acc + w v with the product rounded first (no fused multiply-add).
__device__ __forceinline__ double add_product(double acc, double w, double v) {
#pragma clang fp contract(off)
  return acc + w * v;
}

// Replaces every entry's code by its frame offset and weight and forms
// b = L^T B^T d on the way (Eq. 7; and A^T bhat of the Monte Carlo degrees of
// freedom): one lane per row in slice order, so the entries are read and
// written coalesced and each node's sum runs over its entries in their fixed
// order, in FP64, from v = B^T d at the pixel and the FP64 weight.  Also the
// padding entries, and the scale of the spectral preconditioner,
// c = sum_i cov_i b_i^2 / sum_i b_i^2 with cov = L^T 1 (the weight each node
// receives), a cheap stand-in for the Rayleigh quotient <b, L^T B^T B L b> / <b, b>.
// Bound by the dependent reads entry -> record (48 bytes) -> v, one cache line
// each per lane.  One wave takes one slice, four slices a block (one block per
// member left most of the chip idle for a single 128 x 128 member, 153 -> 51
// us with rhs_row's batched reads, and ended with its slowest block for 256
// of them, 417 -> 330 us).  Each block leaves its part of c's two sums for
// k_split.
constexpr int kRhsT = 256;
__host__ __device__ __forceinline__ int rhs_blocks_of(int I) { return (I + kRhsT - 1) / kRhsT; }
// Blocks per member in a launch: no more than keep the grid under 2^30 threads.
static int rhs_grid(int I_max, int M) { return std::min(rhs_blocks_of(I_max), std::max(1, (1 << 22) / M)); }

// What k_prep_rhs's rows read and write.
template <typename T>
struct RhsView {
  const int32_t* pix;
  const int32_t* cellp;
  const T* fxp;
  const T* fyp;
  const double* v;    // B^T d
  const double* vh;   // B^T bhat, or NULL
  LtEntry<T>* ent;
  unsigned short* off16;   // the paired form's offsets and weights
  T* w2;
  int ns, n2, nx, off0, pitch;   // frame offset of image pixel (r, c): r pitch + c + off0
  bool cubic;
};

// One row: its n entries from index e0, and the padding up to len.  FAST: 2 x 2
// subpixels, bilinear or nearest, no Monte Carlo draws.  The reads of U
// entries are issued together, level by level (code, then pixel and record,
// then v), and the next codes ahead of their use: with the general form's
// branches between them every entry waited for its own three reads.
template <typename T, bool FAST, bool PAIRED>
__device__ __forceinline__ void rhs_row(const RhsView<T>& o, int node, int n, int e0, int len, long step, double& acc,
                                        double& acch, double& cov) {
  constexpr int U = FAST ? (sizeof(T) == 4 ? 8 : 4) : 1;
  int next[U];
  auto codes = [&](int j0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u;
      next[u] = -1;
      if (j < n) next[u] = PAIRED ? *reinterpret_cast<const int*>(&o.w2[paired_index(e0, j)]) : o.ent[e0 + step * j].off;
    }
  };
  codes(0);
  for (int j0 = 0; j0 < len; j0 += U) {
    int code[U], rc[U];
    double w[U], v[U], vh[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      code[u] = next[u];
      rc[u] = o.pix[max(code[u], 0) >> 8];   // slot 0 stands in for no entry
    }
    if constexpr (FAST) {
      int4 c4[U];
      T f[U][4], g[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = max(code[u], 0) >> 8;
        c4[u] = reinterpret_cast<const int4*>(o.cellp)[t];
        if constexpr (sizeof(T) == 4) {
          const float4 x = reinterpret_cast<const float4*>(o.fxp)[t], y = reinterpret_cast<const float4*>(o.fyp)[t];
          f[u][0] = x.x; f[u][1] = x.y; f[u][2] = x.z; f[u][3] = x.w;
          g[u][0] = y.x; g[u][1] = y.y; g[u][2] = y.z; g[u][3] = y.w;
        } else {
          const double2* x = reinterpret_cast<const double2*>(o.fxp) + 2L * t;
          const double2* y = reinterpret_cast<const double2*>(o.fyp) + 2L * t;
          const double2 x0 = x[0], x1 = x[1], y0 = y[0], y1 = y[1];
          f[u][0] = x0.x; f[u][1] = x0.y; f[u][2] = x1.x; f[u][3] = x1.y;
          g[u][0] = y0.x; g[u][1] = y0.y; g[u][2] = y1.x; g[u][3] = y1.y;
        }
      }
      codes(j0 + U);
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = o.v[(rc[u] >> 16) * o.nx + (rc[u] & 0xFFFF)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int cl[4] = {c4[u].x, c4[u].y, c4[u].z, c4[u].w};
        w[u] = pair_weight4(node, o.ns, cl, f[u], g[u]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = max(code[u], 0) >> 8, at = (rc[u] >> 16) * o.nx + (rc[u] & 0xFFFF);
        w[u] = pair_weight(o.cubic, t, code[u] & 255, node, o.ns, o.n2, o.cellp, o.fxp, o.fyp);
        v[u] = o.v[at];
        vh[u] = o.vh ? o.vh[at] : 0.0;
      }
      codes(j0 + U);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u;
      if (j >= len) continue;
      int off = 0;
      T wt = (T)0;
      if (code[u] >= 0) {
        acc = add_product(acc, w[u], v[u]);
        if (!FAST) acch = add_product(acch, w[u], vh[u]);
        cov += w[u];
        off = (rc[u] >> 16) * o.pitch + (rc[u] & 0xFFFF) + o.off0;
        wt = (T)w[u];
      }
      if (PAIRED) {
        const long e = paired_index(e0, j);
        o.off16[e] = (unsigned short)off;
        o.w2[e] = wt;
      } else {
        LtEntry<T> y;
        y.off = off;
        y.w = wt;
        o.ent[e0 + step * j] = y;
      }
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(kRhsT) k_prep_rhs(SolveArgs a) {
  __shared__ double red[2 * kRhsT / 64];
  // blocks go to the XCDs in turn: all of a member's blocks on one of them, whose L2 holds its records
  const int idx = blockIdx.x >> 3, m = (idx / a.rhs_blocks) * 8 + (blockIdx.x & 7), part = idx % a.rhs_blocks;
  if (m >= a.n_members) return;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, n2 = a.n2;
  const MemberInfo mi = a.minfo[m];
  if (__builtin_amdgcn_readfirstlane((int)(mi.status != SL_ST_OK || part >= rhs_blocks_of(mi.I)))) return;
  const int ns = mi.ns, I = mi.I, sell = __builtin_amdgcn_readfirstlane(mi.sell);
  const int32_t* rp = a.lt_ptr + (long)m * (a.I_max + 65);
  const int32_t* perm = a.lt_perm + (long)m * a.I_max;
  const int32_t* lcnt = a.lt_cnt + (long)m * a.I_max;
  double* bm = a.b + (long)m * a.I_max;
  double* bhm = a.bh + (long)m * a.I_max;
  const int halo = 2 * a.ckt, pitch = (mi.c1 - mi.c0 + 1 + 2 * halo) | 1;
  const int ngroups = (I + 63) / 64, E = sell ? rp[ngroups] : 0;
  RhsView<T> o;
  o.pix = a.pix_list + (long)m * a.slot_cap;
  o.cellp = a.cell + (long)m * a.slot_cap * n2;
  o.fxp = reinterpret_cast<const T*>(a.fx) + (long)m * a.slot_cap * n2;
  o.fyp = reinterpret_cast<const T*>(a.fy) + (long)m * a.slot_cap * n2;
  o.v = a.btd;
  o.vh = a.mcn ? a.btd + a.nx * a.ny : nullptr;
  o.ent = reinterpret_cast<LtEntry<T>*>(a.lt_ent) + (long)m * a.lt_cap;
  o.off16 = reinterpret_cast<unsigned short*>(o.ent);
  o.w2 = reinterpret_cast<T*>(o.off16 + E);
  o.ns = ns;
  o.n2 = n2;
  o.nx = a.nx;
  o.pitch = pitch;
  o.off0 = (halo - mi.r0) * pitch + halo - mi.c0;
  o.cubic = a.interp == SL_INTERP_BICUBIC;
  const bool fast = n2 == 4 && !o.cubic && !o.vh;
  double num = 0.0, den = 0.0;
  for (int g = part * (kRhsT / 64) + wid; g < ngroups; g += a.rhs_blocks * (kRhsT / 64)) {
    const int p = 64 * g + lane;
    int node = -1, n = 0;
    if (p < I) {
      node = sell ? (perm[p] >> 16) * ns + (perm[p] & 0xFFFF) : p;
      n = lcnt[node];
    }
    const int e0 = sell ? rp[g] + lane : (p < I ? rp[p] : 0);
    const int len = sell ? (rp[g + 1] - rp[g]) >> 6 : n;   // slice length (the row's own in CSR)
    const long step = sell ? 64L : 1L;
    double acc = 0.0, acch = 0.0, cov = 0.0;
    if (fast && sell == 2) rhs_row<T, true, true>(o, node, n, e0, len, step, acc, acch, cov);
    else if (fast) rhs_row<T, true, false>(o, node, n, e0, len, step, acc, acch, cov);
    else if (sell == 2) rhs_row<T, false, true>(o, node, n, e0, len, step, acc, acch, cov);
    else rhs_row<T, false, false>(o, node, n, e0, len, step, acc, acch, cov);
    if (node >= 0) {
      bm[node] = acc;
      if (a.mcn) bhm[node] = acch;
      num += cov * acc * acc;
      den += acc * acc;
    }
  }
  block_sum2(num, den, red);
  if (tid == 0) {
    double* pc = a.pcpart + 2L * ((long)m * a.rhs_blocks + part);
    pc[0] = num;
    pc[1] = den;
  }
}

// ------------------------------------------------------------------ banded pass
// In-place pass out(p) = sum_{|d|<=2ck} a[|d|] in(p+d) - edge corrections along
// `nlines` lines of length `len` of the frame interior.  The frame carries a
// zero halo of 2*CKT elements on every side, so windows need no bounds tests.
// `F0` points at interior element (0, 0).  ROW: element (line, p) at
// F0[line*pitch + p]; else F0[p*pitch + line].  Every line is handled by the
// lanes of one wave within one step, so all reads of a line precede its
// writes.  acoef[d + 2*kMaxCK] = a[d].
template <typename T, int CKT, bool ROW>
__device__ __forceinline__ void banded_pass(T* __restrict__ F0, int pitch, int nlines, int len,
                                            int img_off, int img_len, int ck,
                                            const T* __restrict__ acoef, const T* __restrict__ EL,
                                            const T* __restrict__ ER) {
  constexpr int W = kSegR + 4 * CKT;
  constexpr int NH = 2 * CKT;
  T ac[NH + 1];
#pragma unroll
  for (int x = 0; x <= NH; ++x) ac[x] = acoef[2 * kMaxCK + x];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int S = (len + kSegR - 1) / kSegR;
  const int LPW = 64 / S;
  // consecutive lanes walk consecutive lines (odd pitch / unit stride: no LDS
  // bank conflicts); the segments of one line stay in one wave step
  const int sub_line = lane % LPW, seg = lane / LPW;
  const int p0 = seg * kSegR;
  const int step = ROW ? 1 : pitch;          // distance between positions
  const int lstride = ROW ? pitch : 1;       // distance between lines
  const bool edges = img_off < ck || img_off + len > img_len - ck;
  for (int l0 = wv * LPW; l0 < nlines; l0 += (kNTof<T> / kWave) * LPW) {   // same trip count for the whole wave
    const int line = l0 + sub_line;
    const bool active = seg < S && line < nlines;
    const T* src = F0 + (active ? line * lstride + (p0 - NH) * step : 0);
    T win[W];
#pragma unroll
    for (int x = 0; x < W; ++x) win[x] = active ? src[x * step] : (T)0;
    T out[kSegR];
#pragma unroll
    for (int o = 0; o < kSegR; ++o) {
      T acc = ac[0] * win[o + NH];
#pragma unroll
      for (int d = 1; d <= NH; ++d) acc += ac[d] * (win[o + NH - d] + win[o + NH + d]);
      out[o] = acc;
    }
    if (active && edges) {
      // outputs within ck of the image border: subtract the part of the
      // autocorrelation that runs through intermediate pixels outside the image
#pragma unroll
      for (int o = 0; o < kSegR; ++o) {
        const int gpos = img_off + p0 + o;
        if (gpos < ck) {
          T corr = 0;
          for (int q = 0; q < ck; ++q) {
            const int pp = q - img_off;
            if (pp >= 0 && pp < len) corr += EL[gpos * ck + q] * F0[line * lstride + pp * step];
          }
          out[o] -= corr;
        }
        if (gpos >= img_len - ck) {
          const int pr = gpos - (img_len - ck);
          T corr = 0;
          for (int q = 0; q < ck; ++q) {
            const int pp = img_len - ck + q - img_off;
            if (pp >= 0 && pp < len) corr += ER[pr * ck + q] * F0[line * lstride + pp * step];
          }
          out[o] -= corr;
        }
      }
    }
    // every lane of the wave has read its window (and edge inputs) before any
    // lane overwrites the line: keep the compiler from sinking loads below here
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (active) {
      T* dst = F0 + line * lstride + p0 * step;
#pragma unroll
      for (int o = 0; o < kSegR; ++o)
        if (p0 + o < len) dst[o * step] = out[o];
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// An out-of-line function sees its pointer arguments without their address
// space, and every access through them becomes a flat one, which waits on both
// the vector memory and the LDS counters; such functions take these pointer
// types inside.  (A cast to one of them and back is folded away.)
template <typename T>
using Lds = __attribute__((address_space(3))) T*;
template <typename T>
using Global = __attribute__((address_space(1))) T*;
__device__ __forceinline__ float uniform(float x) {
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

// ------------------------------------------------------------------ k_solve
template <typename T>
__device__ __forceinline__ T lds_node(const T* P, int ns, int r, int c) {
  return (r < 0 || c < 0 || r >= ns || c >= ns) ? (T)0 : P[r * ns + c];
}

// H^T H p at node (r, c): D2 (x) I + I (x) D2 with the 1-D Dirichlet D2
// (rows [5,-4,1], [-4,6,-4,1], [1,-4,6,-4,1], ...).
template <typename T>
__device__ __forceinline__ T hth_node(const T* P, int ns, int r, int c) {
  const T ctr = P[r * ns + c];
  const T dgx = (T)(6 - (c == 0) - (c == ns - 1));
  const T dgy = (T)(6 - (r == 0) - (r == ns - 1));
  const T n1 = lds_node(P, ns, r, c - 1) + lds_node(P, ns, r, c + 1) + lds_node(P, ns, r - 1, c) +
               lds_node(P, ns, r + 1, c);
  const T n2 = lds_node(P, ns, r, c - 2) + lds_node(P, ns, r, c + 2) + lds_node(P, ns, r - 2, c) +
               lds_node(P, ns, r + 2, c);
  return (dgx + dgy) * ctr - (T)4 * n1 + n2;
}

template <typename T>
__device__ __forceinline__ double reg_node(const T* P, int ns, int r, int c, int reg) {
  const double ctr = (double)P[r * ns + c];
  if (reg == SL_H_IDENTITY) return ctr * ctr;
  const double dx = (double)lds_node(P, ns, r, c - 1) - 2.0 * ctr + (double)lds_node(P, ns, r, c + 1);
  const double dy = (double)lds_node(P, ns, r - 1, c) - 2.0 * ctr + (double)lds_node(P, ns, r + 1, c);
  return dx * dx + dy * dy;
}

// Block-wide FP64 sum with one barrier; consecutive calls must alternate `buf`
// (0/1) and be separated by at least one other barrier before a buffer is reused.
template <int NW = kWaves, typename SP>
__device__ __forceinline__ double block_sum1(double v, SP scratch, int buf) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  v = wave_sum(v);
  const SP sc = scratch + 16 * buf;
  if (lane == 0) sc[wid] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) t += sc[i];
  return t;
}

// ---------------------------------------------------------------- spectral preconditioner
// H^T H = D^2 (x) I + I (x) D^2 with D = tridiag(1, -2, 1) (Dirichlet second
// differences on an n x n grid).  The orthonormal sine transform S,
// S_jk = sqrt(2/(n+1)) sin(pi (j+1)(k+1) / (n+1)) (symmetric, S S = I),
// diagonalises D: D = S diag(-4 sin^2(pi (k+1) / (2(n+1)))) S, so
// M = c I + lambda H^T H = (S (x) S) diag(c + lambda (mu_j + mu_k)) (S (x) S)
// with mu_k the eigenvalues of D^2, and M^-1 x is two 2-D transforms and a
// division.  With x an n x n array X, (S (x) S) x = S X S.
typedef float f32x4 __attribute__((ext_vector_type(4)));

// C = S D (SA) or D S on the FP32 matrix cores, D and C n x n arrays in LDS
// with rows `pitch` apart; with `scale`, element (j, k) is divided by c +
// lambda (mu_j + mu_k).  S comes from the table tab[m] = sqrt(2/(n+1))
// sin(pi m / (n+1)), m = (j+1)(k+1) mod 2(n+1).  A wave takes 16 x 16 output
// tiles of one 16-row (SA) or 16-column block of S, NTL of them at a time
// sharing its values; the next four inner steps' operands are read before the
// current four's MFMAs, and only the last steps test the inner index: a step
// is NTL MFMAs, NTL + 1 LDS reads and as many address updates.
// v_mfma_f32_16x16x4f32: lane l supplies A[l%16][l/16] and B[l/16][l%16];
// accumulator element r is C[4 (l/16) + r][l%16].
template <bool SA, int NTL>
__device__ __forceinline__ void sine_tiles(Lds<const float> tab, Lds<const float> mu, int n, int pitch,
                                           Lds<const float> D, Lds<float> C, int blk, int o0, int ostep, bool scale,
                                           float c, float lam) {
  constexpr int G = 4;
  const int lane = threadIdx.x & 63, lc = lane & 15, lq = lane >> 4;
  const unsigned nn2 = 2 * (n + 1);
  const int si = 16 * blk + lc;                       // this lane's row (column) of S; past n it feeds no stored result
  const unsigned step = (4u * (si + 1)) % nn2;
  unsigned mi = ((si + 1u) * (lq + 1)) % nn2;
  // data operand of tile q, inner index t = 4 u + lq: SA: D[t][j], else D[i][t]; a lane past the edge repeats the last
  const int dstep = SA ? 4 * pitch : 4;
  Lds<const float> dp[NTL];
#pragma unroll
  for (int q = 0; q < NTL; ++q) {
    const int f = min(16 * (o0 + q * ostep) + lc, n - 1);
    dp[q] = D + (SA ? lq * pitch + f : f * pitch + lq);
  }
  f32x4 acc[NTL];
#pragma unroll
  for (int q = 0; q < NTL; ++q) acc[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  float sv[G], dv[NTL][G];
  int t0 = 0;   // inner index of the next read
  auto load = [&](float (&s)[G], float (&d)[NTL][G]) {
    if (t0 + 4 * G <= n) {   // uniform
#pragma unroll
      for (int g = 0; g < G; ++g) {
        s[g] = tab[mi];
        mi += step;
        mi = min(mi, mi - nn2);   // mod nn2
#pragma unroll
        for (int q = 0; q < NTL; ++q) {
          d[q][g] = *dp[q];
          dp[q] += dstep;
        }
      }
    } else {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const bool in = t0 + 4 * g + lq < n;   // inner indices past n enter as zeros
        s[g] = in ? tab[mi] : 0.0f;
        mi += step;
        mi = min(mi, mi - nn2);
#pragma unroll
        for (int q = 0; q < NTL; ++q) {
          d[q][g] = in ? *dp[q] : 0.0f;
          dp[q] += dstep;
        }
      }
    }
    t0 += 4 * G;
  };
  load(sv, dv);
  for (int k = 0; k < n; k += 4 * G) {
    float sn[G], dn[NTL][G];
    load(sn, dn);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int q = 0; q < NTL; ++q)
        acc[q] = SA ? __builtin_amdgcn_mfma_f32_16x16x4f32(sv[g], dv[q][g], acc[q], 0, 0, 0)
                    : __builtin_amdgcn_mfma_f32_16x16x4f32(dv[q][g], sv[g], acc[q], 0, 0, 0);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      sv[g] = sn[g];
#pragma unroll
      for (int q = 0; q < NTL; ++q) dv[q][g] = dn[q][g];
    }
  }
#pragma unroll
  for (int q = 0; q < NTL; ++q) {
    const int o = o0 + q * ostep;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * (SA ? blk : o) + 4 * lq + r, col = 16 * (SA ? o : blk) + lc;
      if (row < n && col < n) {
        float v = acc[q][r];
        if (scale) v = v / (c + lam * (mu[row] + mu[col]));
        C[row * pitch + col] = v;
      }
    }
  }
}

// The n x n product by the block's 16 waves: nt = ceil(n/16) blocks of S, each
// taken by floor(16/nt) waves that share its nt tiles out (n <= 128: at most
// four tiles a wave).
template <bool SA>
__device__ __forceinline__ void sine_mul(Lds<const float> tab, Lds<const float> mu, int n, int pitch, Lds<const float> D,
                                         Lds<float> C, bool scale, float c, float lam) {
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nt = (n + 15) >> 4, per = 16 / nt, blk = wv / per, o0 = wv % per;
  if (blk >= nt || o0 >= nt) return;
  switch ((nt - o0 + per - 1) / per) {
    case 1: sine_tiles<SA, 1>(tab, mu, n, pitch, D, C, blk, o0, per, scale, c, lam); break;
    case 2: sine_tiles<SA, 2>(tab, mu, n, pitch, D, C, blk, o0, per, scale, c, lam); break;
    case 3: sine_tiles<SA, 3>(tab, mu, n, pitch, D, C, blk, o0, per, scale, c, lam); break;
    default: sine_tiles<SA, 4>(tab, mu, n, pitch, D, C, blk, o0, per, scale, c, lam); break;
  }
}

// One preconditioned-CG direction update, all threads of the block:
// z = M^-1 r (r from r_g, the scratch in the Q region and the frame F),
// rz_new = <r, z>, p = z + beta p with beta = rz_new / rz_old (0 when
// `restart`), and the frame zeroed again.  Returns rz_new.  Kept out of line so
// that its registers do not add to the CG loop's pressure.
//
// Bound by the matrix cores' FP32 rate (four products of n^3) and the LDS reads
// that feed them.  With S on either side of the data no product needs a
// transposed copy.  Rows n apart put the sixteen rows of an operand in 1, 2 or
// 4 of the 32 banks when 8 divides n; there they are n + 2 apart where both
// arrays have the room (qcap, fcap floats).  (58k cycles at n = 64 and 168k at n
// = 100 when 16 x 48 strips left half the waves or two thirds of their tiles
// empty, the transposed stores met in one bank and every access was a flat
// one; 38k and 117k so.)
__device__ __attribute__((noinline)) double pc_apply(float* P_, float* Q_, float* F_, int qcap_, int fcap_,
                                                     const float* tab_, const float* mu_, int n_, const float* r_,
                                                     float c_, float lam_, double rz_old, int restart,
                                                     double* red_) {
  const Lds<float> P = (Lds<float>)P_, Q = (Lds<float>)Q_, F = (Lds<float>)F_;
  const Lds<const float> tab = (Lds<const float>)tab_, mu = (Lds<const float>)mu_;
  const Global<const float> r_g = (Global<const float>)r_;
  const Lds<double> red = (Lds<double>)red_;
  const int n = __builtin_amdgcn_readfirstlane(n_), qcap = __builtin_amdgcn_readfirstlane(qcap_),
            fcap = __builtin_amdgcn_readfirstlane(fcap_);
  const float c = uniform(c_), lam = uniform(lam_);
  const int tid = threadIdx.x, nn = n * n;
  int pitch = n & 7 ? n : n + 2;
  Lds<float> X = Q;
  const Lds<float> Tb = F;
  int used = n * pitch;   // floats of the frame
  if (pitch != n) {
    if (used > qcap && 2 * used <= fcap) {
      X = F + used;
      used *= 2;
    } else if (used > qcap || used > fcap) {
      pitch = n;
      used = nn;
    }
  }
  const float inv_n = 1.0f / n;
  const int pad = pitch - n;
  // node i at i + row(i) pad; (i + 1/2) / n in FP32 is exact enough for i < 2^14
  auto at = [&](int i) { return i + (int)((i + 0.5f) * inv_n) * pad; };
  for (int i = tid; i < nn; i += kNT) X[at(i)] = r_g[i];
  __syncthreads();
  sine_mul<false>(tab, mu, n, pitch, X, Tb, false, 0.0f, 0.0f);   // X S
  __syncthreads();
  sine_mul<true>(tab, mu, n, pitch, Tb, X, true, c, lam);         // Y = S X S over the eigenvalues of M
  __syncthreads();
  sine_mul<true>(tab, mu, n, pitch, X, Tb, false, 0.0f, 0.0f);    // S Y
  __syncthreads();
  sine_mul<false>(tab, mu, n, pitch, Tb, X, false, 0.0f, 0.0f);   // z = S Y S
  __syncthreads();
  double rzn = 0.0;
  for (int i = tid; i < nn; i += kNT) rzn += (double)r_g[i] * (double)X[at(i)];
  rzn = block_sum1(rzn, red, 2);
  const float beta = restart ? 0.0f : (float)(rzn / rz_old);
  for (int i = tid; i < nn; i += kNT) P[i] = X[at(i)] + beta * P[i];
  if (X != Q) __syncthreads();   // z lies in the frame too
  for (int e = tid; e < used; e += kNT) F[e] = 0.0f;
  return rzn;
}

// Bicubic value of the n x n subpixels of mapped pixel t: for each subpixel
// the 4 x 4 nodes about its cell, weighted by the cubic convolution kernel in
// x and y, nodes outside the grid left out.
template <typename T>
__device__ __forceinline__ T pixel_gather_cubic(const T* X, int ns, int n2, int t, const int32_t* cellp,
                                                const T* fxp, const T* fyp) {
  T acc = 0;
#pragma unroll 1
  for (int k = 0; k < n2; ++k) {
    const int c = cellp[(long)t * n2 + k];
    if (c < 0) continue;
    const T fx = fxp[(long)t * n2 + k], fy = fyp[(long)t * n2 + k];
    const int r = c / ns, col = c % ns;
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
      const int rr = r + j - 1;
      if (rr < 0 || rr >= ns) continue;
      T row = 0;
#pragma unroll 1
      for (int i = 0; i < 4; ++i) {
        const int cc = col + i - 1;
        if (cc >= 0 && cc < ns) row += keys_w(fabs(fx - (T)(i - 1))) * X[rr * ns + cc];
      }
      acc += keys_w(fabs(fy - (T)(j - 1))) * row;
    }
  }
  return acc;
}

// Interpolated value of the n x n subpixels of mapped pixel t: sum_k w_k . x[cell_k..]
// (bilinear weights, or the nearest node's weight 1; bicubic when `cubic`)
template <typename T>
__device__ __forceinline__ T pixel_gather(const T* X, int ns, int n2, int t, const int32_t* cellp, const T* fxp,
                                          const T* fyp, bool cubic) {
  if (cubic) return pixel_gather_cubic(X, ns, n2, t, cellp, fxp, fyp);
  T acc = 0;
  if (n2 == 4) {
    const int4 c4 = reinterpret_cast<const int4*>(cellp)[t];
    T fx[4], fy[4];
    if constexpr (sizeof(T) == 4) {
      const float4 a4 = reinterpret_cast<const float4*>(fxp)[t];
      const float4 b4 = reinterpret_cast<const float4*>(fyp)[t];
      fx[0] = a4.x; fx[1] = a4.y; fx[2] = a4.z; fx[3] = a4.w;
      fy[0] = b4.x; fy[1] = b4.y; fy[2] = b4.z; fy[3] = b4.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        fx[k] = fxp[4L * t + k];
        fy[k] = fyp[4L * t + k];
      }
    }
    const int cl[4] = {c4.x, c4.y, c4.z, c4.w};
    // branch-free: an off-grid subpixel (cell -1) reads node 0 and adds zero
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = max(cl[k], 0);
      const T v = (1 - fy[k]) * ((1 - fx[k]) * X[c] + fx[k] * X[c + 1]) +
                  fy[k] * ((1 - fx[k]) * X[c + ns] + fx[k] * X[c + ns + 1]);
      acc += cl[k] >= 0 ? v : (T)0;
    }
    return acc;
  }
  for (int k = 0; k < n2; ++k) {
    const int c = cellp[(long)t * n2 + k];
    if (c < 0) continue;
    const T fx = fxp[(long)t * n2 + k], fy = fyp[(long)t * n2 + k];
    acc += (1 - fy) * ((1 - fx) * X[c] + fx * X[c + 1]) + fy * ((1 - fx) * X[c + ns] + fx * X[c + ns + 1]);
  }
  return acc;
}

// Invalid or empty member: s = 0, chi^2 = sum d^2 / sigma^2 (no barriers).
template <typename T>
__device__ void trivial_item(const SolveArgs& a, const MemberInfo& mi, int m, int kl) {
  const long out_idx = (long)m * a.n_lambda + kl;
  T* s_dst = reinterpret_cast<T*>(a.s_all) + out_idx * a.I_max;
  for (int i = threadIdx.x; i < mi.I; i += kNTof<T>) s_dst[i] = (T)0;
  if (threadIdx.x == 0) {
    a.chi2[out_idx] = mi.status == SL_ST_INVALID ? NAN : a.consts->sum_d2 / (a.sigma * a.sigma);
    a.regv[out_idx] = mi.status == SL_ST_INVALID ? NAN : 0.0;
    a.iters[out_idx] = 0;
    a.status[out_idx] = mi.status;
  }
}

// One CG solve of a valid member.  Every branch that encloses a barrier
// depends only on block-uniform values made scalar with readfirstlane.
// LDS: P = search direction p, Q = A p accumulator, the image frame (LDSF)
// and reduction scratch.  The iterate s (in its output slot) and the
// residual r live in global memory, read and written by their owner thread.
// The operands of one item's regularised normal operator (see apply_normal).
template <typename T>
struct OpView {
  const int32_t* pix;        // mapped-pixel slots: packed (row << 16 | col), -1 past the end
  const int32_t* cellp;      // [slot][n^2] bilinear cell of each subpixel, -1 off the grid
  const T* fxp;
  const T* fyp;
  T* F;                      // image frame with its zero halo (LDS or global)
  T* F0;                     // frame interior (0, 0) = image pixel (r0, c0)
  T* Z;                      // per-block image buffer of the direct blur (z = B y on the dilated box)
  T* W;                      // per-block image buffer of the direct blur (B^T z on the bounding box)
  const T* taps;
  const int32_t* lt_rp;      // transposed operator: slice (or row) starts
  const LtEntry<T>* lt_e;    //                      entries
  const int32_t* perm;       //                      nodes in slice order
  int ns, I, M, r0, c0, h, w, pitch, fo, n2, nx, ny, K, ck, sell, Dr0, Dc0, Dh, Dw;
  bool sep, ident;
  T inv_n2, lamT;
  bool cubic;                // bicubic L (16 nodes per subpixel); else bilinear or nearest
};

// y = L p into the frame: every mapped pixel is written once (assignment, so
// the frame outside the mapped pixels keeps whatever it held, zero unless a
// banded pass wrote it).  Two pixels per thread and step so that their table
// loads are in flight together.
// The bicubic form, out of line: its 16 taps per subpixel stay out of the
// register budget of the persistent kernels that inline the other forms.
template <typename T, int NT>
__device__ __attribute__((noinline)) void gather_L_cubic(const int32_t* pix, const int32_t* cellp, const T* fxp,
                                                        const T* fyp, T* F0, const T* P, int M, int ns, int n2,
                                                        int pitch, int fo, T inv_n2) {
  for (int t = threadIdx.x; t < M; t += NT) {
    const int rc = pix[t];
    if (rc >= 0) F0[(rc >> 16) * pitch + (rc & 0xFFFF) + fo] = pixel_gather_cubic(P, ns, n2, t, cellp, fxp, fyp) * inv_n2;
  }
}

// CUBIC = false compiles the bicubic branch out (the banded-blur kernels: a
// bicubic problem always takes the direct form).
template <typename T, int NT, bool CUBIC = true>
__device__ __forceinline__ void gather_L(const OpView<T>& o, const T* __restrict__ P) {
  const int32_t* pix = o.pix;
  T* const F0 = o.F0;
  const int M = o.M, ns = o.ns, n2 = o.n2, pitch = o.pitch, fo = o.fo;
  const T inv_n2 = o.inv_n2;
  if constexpr (CUBIC) {
    if (o.cubic) {
      gather_L_cubic<T, NT>(pix, o.cellp, o.fxp, o.fyp, F0, P, M, ns, n2, pitch, fo, inv_n2);
      return;
    }
  }
  for (int t = threadIdx.x; t < M; t += 2 * NT) {
    const int t2 = t + NT;
    const int rc = pix[t];
    const int rc2 = t2 < M ? pix[t2] : -1;
    const T v1 = pixel_gather(P, ns, n2, t, o.cellp, o.fxp, o.fyp, false);
    const T v2 = t2 < M ? pixel_gather(P, ns, n2, t2, o.cellp, o.fxp, o.fyp, false) : (T)0;
    if (rc >= 0) F0[(rc >> 16) * pitch + (rc & 0xFFFF) + fo] = v1 * inv_n2;
    if (rc2 >= 0) F0[(rc2 >> 16) * pitch + (rc2 & 0xFFFF) + fo] = v2 * inv_n2;
  }
}

// z = B y over the dilated box (Dh x Dw, row-major) from the frame, whose
// entries off the mapped pixels are zero.  Returns this thread's part of
// ||z||^2.
// F0, taps and Z are o.F0, o.taps and the output (of any pointer type).
template <typename T, int CKT, int NT, typename FP, typename TP, typename ZP>
__device__ __forceinline__ double blur_box(const OpView<T>& o, FP F0, TP taps, ZP __restrict__ Z) {
  const TapIdx ti(o.K);
  const int K = o.K, ck = o.ck, r0 = o.r0, c0 = o.c0, h = o.h, w = o.w, pitch = o.pitch;
  const int Dr0 = o.Dr0, Dc0 = o.Dc0, Dh = o.Dh, Dw = o.Dw;
  double zz = 0.0;
  for (int e = threadIdx.x; e < Dh * Dw; e += NT) {
    const int rr_ = Dr0 + e / Dw, cc_ = Dc0 + e % Dw;
    T acc = 0;
    if (ck <= CKT) {
      // every tap of an output in the dilated region lands in the bounding
      // box or its zero halo (2 CKT >= 2 ck on each side): no bounds tests
      const auto yrow = F0 + (rr_ + ck - r0) * pitch + (cc_ + ck - c0);
      const auto tp = taps + ti.psf;
      for (int aa = 0; aa < K; ++aa) {
        const auto y = yrow - aa * pitch;
        for (int bb = 0; bb < K; ++bb) acc += tp[aa * K + bb] * y[-bb];
      }
    } else {   // PSFs wider than the widest compiled window: the halo is narrower than ck
      for (int aa = 0; aa < K; ++aa) {
        const int yr = rr_ - aa + ck - r0;
        if (yr < 0 || yr >= h) continue;
        for (int bb = 0; bb < K; ++bb) {
          const int yc = cc_ - bb + ck - c0;
          if (yc < 0 || yc >= w) continue;
          acc += taps[ti.psf + aa * K + bb] * F0[yr * pitch + yc];
        }
      }
    }
    Z[e] = acc;
    zz += (double)acc * (double)acc;
  }
  return zz;
}

// w = B^T z at the mapped pixels, into the frame; z lives on the dilated box.
template <typename T, int NT>
__device__ __forceinline__ void blur_T_mapped(const OpView<T>& o, const T* __restrict__ Z) {
  const int32_t* pix = o.pix;
  T* const F0 = o.F0;
  const T* taps = o.taps;
  const TapIdx ti(o.K);
  const int K = o.K, ck = o.ck, pitch = o.pitch, fo = o.fo, M = o.M;
  const int Dr0 = o.Dr0, Dc0 = o.Dc0, Dh = o.Dh, Dw = o.Dw;
  for (int t = threadIdx.x; t < M; t += NT) {
    if (pix[t] < 0) continue;
    const int rr_ = pix[t] >> 16, cc_ = pix[t] & 0xFFFF;
    T acc = 0;
    for (int aa = 0; aa < K; ++aa) {
      const int zr = rr_ + aa - ck - Dr0;
      if (zr < 0 || zr >= Dh) continue;
      for (int bb = 0; bb < K; ++bb) {
        const int zc = cc_ + bb - ck - Dc0;
        if (zc < 0 || zc >= Dw) continue;
        acc += taps[ti.psf + aa * K + bb] * Z[zr * Dw + zc];
      }
    }
    F0[rr_ * pitch + cc_ + fo] = acc;
  }
}

// q = L^T w + lambda H^T H p gathered per node from the transposed operator
// (no atomics, fixed order), stored in Q.  Returns this thread's part of
// <p, q>.  With GRAD, q = L^T w alone (no P term) and the return value is
// this thread's part of ||q||^2.
//
// Bound by the entries' way from L2 and the Infinity Cache and by the bank
// conflicts of the frame reads.  With PIPE the paired entries are read a batch
// ahead of their use: 31.0k -> 28.3k cycles per c3 iteration of 65k.  The CKT =
// 10 kernel has no registers left for it (88.0k -> 88.7k per c4 iteration) and
// FP64's wide entries gain nothing (9.6k -> 14.2k at 16 x 16 nodes): there,
// batches of eight pairs.
template <typename T, int NT, bool GRAD, bool PIPE = false>
__device__ __forceinline__ double gather_LT(const OpView<T>& o, const T* __restrict__ P, T* __restrict__ Q) {
  const int tid = threadIdx.x;
  const T* const F = o.F;
  const int32_t* lt_rp = o.lt_rp;
  const LtEntry<T>* lt_e = o.lt_e;
  const int32_t* perm = o.perm;
  const int ns = o.ns, I = o.I, sell = o.sell;
  const bool ident = o.ident;
  const T lamT = o.lamT;
  double pq = 0.0;
  if (sell) {
    // sliced-ELL in length-sorted node order: wave w takes slices w, w + 16, ...;
    // the slice bounds are wave-uniform (scalar loads) and every lane of a
    // slice has `len` entries (padding reads the zero halo), eight in flight
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int nslices = (I + 63) >> 6;
    const int lt_E = lt_rp[nslices];   // sliced-ELL entries of the member
    for (int sl = wid; sl < nslices; sl += NT / 64) {
      const int idx = sl * 64 + lane;
      const int b0 = lt_rp[sl];
      const int len = (lt_rp[sl + 1] - b0) >> 6;
      const int pk = idx < I ? perm[idx] : 0;
      T acc = 0;
      if (sell == 2) {
        // paired entries (even `len`, entries summed in the same order)
        const unsigned* op = reinterpret_cast<const unsigned*>(lt_e) + (b0 >> 1) + lane;
        const EntryPair<T>* wq = reinterpret_cast<const EntryPair<T>*>(reinterpret_cast<const unsigned*>(lt_e) + (lt_E >> 1)) +
                                 (b0 >> 1) + lane;
        const int npair = len >> 1;
        if (PIPE && npair >= 4) {
          // (rows shorter than a batch: one by one below)
          // the next U pairs are read while these U are added; past the row's
          // end the last pair again, unused.  (One path for the reads: with a
          // second, unclamped one the values met at the join and every read was
          // waited for there, 55k cycles instead of 28k.)
          constexpr int U = 4;
          unsigned on[U];
          EntryPair<T> wn[U];
          const int last = npair - 1;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int jj = min(u, max(last, 0));
            on[u] = npair ? op[64L * jj] : 0u;
            if (npair) wn[u] = wq[64L * jj];
          }
          for (int j = 0; j < npair; j += U) {
            unsigned ov[U];
            EntryPair<T> wv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              ov[u] = on[u];
              wv[u] = wn[u];
            }
            if (j + U < npair) {
#pragma unroll
              for (int u = 0; u < U; ++u) {
                const int jj = min(j + U + u, last);
                on[u] = op[64L * jj];
                wn[u] = wq[64L * jj];
              }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (j + u < npair) {   // uniform
                acc += wv[u].x * F[ov[u] & 0xFFFFu];
                acc += wv[u].y * F[ov[u] >> 16];
              }
          }
        } else {
          int j = 0;
          if constexpr (!PIPE) {
            constexpr int U = 8;
            for (; j + U <= npair; j += U) {   // 2 U entries in flight
              unsigned ov[U];
              EntryPair<T> wv[U];
#pragma unroll
              for (int u = 0; u < U; ++u) {
                ov[u] = op[64L * (j + u)];
                wv[u] = wq[64L * (j + u)];
              }
#pragma unroll
              for (int u = 0; u < U; ++u) {
                acc += wv[u].x * F[ov[u] & 0xFFFFu];
                acc += wv[u].y * F[ov[u] >> 16];
              }
            }
          }
          for (; j < npair; ++j) {
            const unsigned o0 = op[64L * j];
            const EntryPair<T> w0 = wq[64L * j];
            acc += w0.x * F[o0 & 0xFFFFu];
            acc += w0.y * F[o0 >> 16];
          }
        }
      } else {
        const LtEntry<T>* ep = lt_e + b0 + lane;
        int j = 0;
        for (; j + 7 < len; j += 8) {
          LtEntry<T> x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] = ep[64L * (j + u)];
#pragma unroll
          for (int u = 0; u < 8; ++u) acc += x[u].w * F[x[u].off];
        }
        for (; j < len; ++j) {
          const LtEntry<T> x0 = ep[64L * j];
          acc += x0.w * F[x0.off];
        }
      }
      if (idx < I) {
        const int rn_ = pk >> 16, cn_ = pk & 0xFFFF, i = rn_ * ns + cn_;
        if (GRAD) {
          Q[i] = acc;
          pq += (double)acc * (double)acc;
        } else {
          const T pv = P[i];
          const T qv = acc + lamT * (ident ? pv : hth_node(P, ns, rn_, cn_));
          Q[i] = qv;
          pq += (double)pv * (double)qv;
        }
      }
    }
  } else {
    for (int i = tid; i < I; i += NT) {
      T acc = 0;
      const int e0 = lt_rp[i], e1 = lt_rp[i + 1];
      for (int e = e0; e < e1; ++e) acc += lt_e[e].w * F[lt_e[e].off];
      if (GRAD) {
        Q[i] = acc;
        pq += (double)acc * (double)acc;
      } else {
        const int rn_ = i / ns, cn_ = i - rn_ * ns;
        const T pv = P[i];
        const T qv = acc + lamT * (ident ? pv : hth_node(P, ns, rn_, cn_));
        Q[i] = qv;
        pq += (double)pv * (double)qv;
      }
    }
  }
  return pq;
}

// Register-tiled direct K x K forms.  Each thread computes eight consecutive outputs of one row
// from a window of KT + 7 values per input row, so that one load serves up
// to eight products; consecutive lanes take consecutive rows, so with the
// odd frame pitch their LDS reads fall in distinct banks.  The last tile of a
// row starts at width - 8: tiles overlap there and write the same values
// twice.  Each output sums its taps in the order of the per-output forms
// (row of the PSF outer, column inner), so the results are the same.
// Usable when the window is the PSF's own (not one size up) and both the box
// and the dilated box are at least 8 wide (tiled_ok).  FULL: the PSF has
// exactly KT = 2 CKT + 1 taps per side; otherwise the taps past the window's
// narrowest PSF are guarded in pairs by uniform branches, and the values they
// would have met are read from the frame's zero halo (2 CKT wide).
// (They took the per-output forms before, each tap a load: 24 members of a
// 96 x 90 image at four lambdas, K = 7, 11, 19 in FP32 42.4, 83.5, 245 ms,
// now 11.9, 13.9, 23.6; K = 9, 13, 19 in FP64 111, 216, 474 ms, now 24.5,
// 32.1, 45.3; the widest sides' 15 and 21 take 16.4 and 25.3 ms in FP32.)
template <typename T>
__device__ constexpr int narrowest_ck(int ckt) {   // of the PSFs that take window ckt
  return ckt == 2 ? 0 : ckt == 10 ? 8 : ckt == 16 ? 11 : sizeof(T) == 8 || ckt == 4 ? 3 : 5;
}
template <typename T, int CKT>
__device__ __forceinline__ bool tiled_ok(const OpView<T>& o) {
  return o.ck <= CKT && o.ck >= narrowest_ck<T>(CKT) && o.w >= 8 && o.Dw >= 8;
}

// z = B y over the dilated box into Z (Dh x Dw, row-major), y in the frame
// with its zero halo.  Returns this thread's part of ||z||^2 (each output
// counted once).
template <typename T, int CKT, int NT, bool FULL, typename FP, typename TP, typename ZP>
__device__ __forceinline__ double blur_box_t8(const OpView<T>& o, FP F0, TP taps, ZP __restrict__ Z) {
  constexpr int KT = 2 * CKT + 1, NV = KT + 7, KMIN = FULL ? KT : 2 * narrowest_ck<T>(CKT) + 1;
  const int K = FULL ? KT : o.K, ck = FULL ? CKT : o.ck;
  const int Dh = o.Dh, Dw = o.Dw, pitch = o.pitch;
  const auto tp = taps + TapIdx(K).psf;
  // output (r, c) of the dilated box reads base[(r - aa) * pitch + (c - bb)]
  const auto base = F0 + (o.Dr0 + ck - o.r0) * pitch + (o.Dc0 + ck - o.c0);
  const int nct = (Dw + 7) >> 3;
  double zz = 0.0;
  for (int t = threadIdx.x; t < Dh * nct; t += NT) {
    const int r = t % Dh;
    const int cn = (t / Dh) * 8;          // nominal tile start
    const int c = min(cn, Dw - 8);
    T acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0;
    for (int aa = 0; aa < K; ++aa) {
      const auto row = base + (r - aa) * pitch + c - (KT - 1);
      T v[NV];
#pragma unroll
      for (int j = 0; j < NV; ++j) v[j] = row[j];
      const auto ta = tp + aa * K;
#pragma unroll
      for (int bb = 0; bb < KMIN; ++bb) {
        const T tv = ta[bb];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += tv * v[i - bb + KT - 1];
      }
#pragma unroll
      for (int b2 = KMIN; b2 < KT; b2 += 2)
        if (b2 < K) {
#pragma unroll
          for (int bb = b2; bb < b2 + 2; ++bb) {
            const T tv = ta[bb];
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] += tv * v[i - bb + KT - 1];
          }
        }
    }
    const auto zo = Z + r * Dw + c;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      zo[i] = acc[i];
      if (c + i >= cn) zz += (double)acc[i] * (double)acc[i];
    }
  }
  return zz;
}

// w = B^T z over the bounding box (h x w) into W (row-major, pitch w), z
// staged in the frame over the dilated box with zeros beyond it.
template <typename T, int CKT, int NT, bool FULL>
__device__ __forceinline__ void blurT_box_t8(const OpView<T>& o, T* __restrict__ W) {
  constexpr int KT = 2 * CKT + 1, NV = KT + 7, KMIN = FULL ? KT : 2 * narrowest_ck<T>(CKT) + 1;
  const int K = FULL ? KT : o.K, ck = FULL ? CKT : o.ck;
  const int h = o.h, w = o.w, pitch = o.pitch;
  const T* tp = o.taps + TapIdx(K).psf;
  // output (r, c) of the box reads base[(r + aa) * pitch + (c + bb)]
  const T* base = o.F0 - ck * pitch - ck;
  const int nct = (w + 7) >> 3;
  for (int t = threadIdx.x; t < h * nct; t += NT) {
    const int r = t % h;
    const int c = min((t / h) * 8, w - 8);
    T acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0;
    for (int aa = 0; aa < K; ++aa) {
      const T* row = base + (r + aa) * pitch + c;
      T v[NV];
#pragma unroll
      for (int j = 0; j < NV; ++j) v[j] = row[j];
      const T* ta = tp + aa * K;
#pragma unroll
      for (int bb = 0; bb < KMIN; ++bb) {
        const T tv = ta[bb];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += tv * v[i + bb];
      }
#pragma unroll
      for (int b2 = KMIN; b2 < KT; b2 += 2)
        if (b2 < K) {
#pragma unroll
          for (int bb = b2; bb < b2 + 2; ++bb) {
            const T tv = ta[bb];
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] += tv * v[i + bb];
          }
        }
    }
    T* wo = W + r * w + c;
#pragma unroll
    for (int i = 0; i < 8; ++i) wo[i] = acc[i];
  }
}

// frame over the dilated box = Z (Dh x Dw, row-major)
template <typename T, int NT>
__device__ __forceinline__ void stage_dilated(const OpView<T>& o, const T* __restrict__ Z) {
  const int Dw = o.Dw, pitch = o.pitch;
  T* const D0 = o.F0 + (o.Dr0 - o.r0) * pitch + (o.Dc0 - o.c0);
  for (int e = threadIdx.x; e < o.Dh * Dw; e += NT) D0[(e / Dw) * pitch + e % Dw] = Z[e];
}

// frame over the bounding box = W (h x w, row-major)
template <typename T, int NT>
__device__ __forceinline__ void stage_box(const OpView<T>& o, const T* __restrict__ W) {
  const int w = o.w, pitch = o.pitch;
  for (int e = threadIdx.x; e < o.h * w; e += NT) o.F0[(e / w) * pitch + e % w] = W[e];
}

// Frame = B^T z at (at least) the mapped pixels, z on the dilated box in Zs.
// The tiled form writes the whole dilated box (z there, B^T z over the
// bounding box), so afterwards the rows of the dilated box must be zeroed
// before the next L gather (clear_rows); the per-output form writes the
// mapped pixels only.  Ends with a barrier.
template <typename T, int CKT, int NT>
__device__ __forceinline__ void adjoint_blur(const OpView<T>& o, const T* __restrict__ Zs) {
  if (tiled_ok<T, CKT>(o)) {   // uniform: scalar member values
    stage_dilated<T, NT>(o, Zs);
    __syncthreads();
    if (o.ck == CKT) blurT_box_t8<T, CKT, NT, true>(o, o.W);
    else blurT_box_t8<T, CKT, NT, false>(o, o.W);
    __syncthreads();
    stage_box<T, NT>(o, o.W);
  } else {
    blur_T_mapped<T, NT>(o, Zs);
  }
  __syncthreads();
}

// z = B y over the dilated box into Z; with SUM returns this thread's part of
// ||z||^2.  Narrower PSFs than the window's widest add it up in the order of
// the per-output form, which they took before.
template <typename T, int CKT, int NT, bool SUM>
__device__ __forceinline__ double forward_blur(const OpView<T>& o, T* __restrict__ Z) {
  if (!tiled_ok<T, CKT>(o)) return blur_box<T, CKT, NT>(o, (const T*)o.F0, o.taps, Z);
  if (o.ck == CKT) return blur_box_t8<T, CKT, NT, true>(o, (const T*)o.F0, o.taps, Z);
  (void)blur_box_t8<T, CKT, NT, false>(o, (const T*)o.F0, o.taps, Z);
  double zz = 0.0;
  if (SUM) {
    __syncthreads();
    for (int e = threadIdx.x; e < o.Dh * o.Dw; e += NT) zz += (double)Z[e] * (double)Z[e];
  }
  return zz;
}

// The same, out of line, for the end of an item: its registers stay out of the
// CG loop's budget.  (A loop over the taps of one output at a time, each with
// its own bounds tests, took 420k cycles per c3 item, 6.5 CG iterations; the
// tiled form and the rest of the tail 65k.)
template <typename T, int CKT, int NT, bool LDSF>
__device__ __attribute__((noinline)) void model_image(const T* F0_, const T* taps_, T* Z_, int K, int r0, int c0, int h,
                                                      int w, int pitch, int Dr0, int Dc0, int Dh, int Dw) {
  using FP = std::conditional_t<LDSF, Lds<const T>, Global<const T>>;
  const FP F0 = (FP)F0_;
  const Global<const T> taps = (Global<const T>)taps_;
  const Global<T> Z = (Global<T>)Z_;
  OpView<T> o{};
  o.K = __builtin_amdgcn_readfirstlane(K);
  o.ck = (o.K - 1) / 2;
  o.r0 = __builtin_amdgcn_readfirstlane(r0);
  o.c0 = __builtin_amdgcn_readfirstlane(c0);
  o.h = __builtin_amdgcn_readfirstlane(h);
  o.w = __builtin_amdgcn_readfirstlane(w);
  o.pitch = __builtin_amdgcn_readfirstlane(pitch);
  o.Dr0 = __builtin_amdgcn_readfirstlane(Dr0);
  o.Dc0 = __builtin_amdgcn_readfirstlane(Dc0);
  o.Dh = __builtin_amdgcn_readfirstlane(Dh);
  o.Dw = __builtin_amdgcn_readfirstlane(Dw);
  if (!tiled_ok<T, CKT>(o)) (void)blur_box<T, CKT, NT>(o, F0, taps, Z);
  else if (o.ck == CKT) (void)blur_box_t8<T, CKT, NT, true>(o, F0, taps, Z);
  else (void)blur_box_t8<T, CKT, NT, false>(o, F0, taps, Z);
}

// Zero the frame rows that an operator application wrote, after every
// gather has read the frame: the bounding box's rows (full pitch), and after
// the tiled direct blur (DIR: the direct forms ran; the tiled one stages z
// there) also the ck rows above and below them.  The tiled form needs
// ck <= CKT, so those rows lie inside the frame's 2 CKT halo; the other forms
// write inside the box only.
template <typename T, int CKT, int NT, bool DIR>
__device__ __forceinline__ void clear_rows(const OpView<T>& o) {
  const int up = (DIR && tiled_ok<T, CKT>(o)) ? o.ck : 0;
  T* const R0 = o.F0 - (up * o.pitch + 2 * CKT);   // column 0 of frame row 2 CKT - up
  const int n = (o.h + 2 * up) * o.pitch;
  for (int e = threadIdx.x; e < n; e += NT) R0[e] = (T)0;
}

// Q = (L^T B^T B L + lambda H^T H) P for one item, all threads of the block:
// L as a gather into the frame (zero on entry), B^T B in place (banded passes
// for a rank-1 PSF, else the direct K x K form through Z), then L^T as a
// gather over the transposed operator (fixed order, no atomics) fused with
// lambda H^T H.  DIR selects the form (a kernel instantiation of each runs,
// the one that does not match the problem returning at entry, so that the
// banded kernels carry none of the direct form's registers).  On return the
// frame holds B^T B L P (the direct form also
// leaves z in the rows of the dilated box); the caller zeroes the rows of the
// dilated box (clear_rows) after a barrier.  Returns this thread's part of
// <P, Q>.
template <typename T, int CKT, int NT, bool DIR>
__device__ __forceinline__ double apply_normal(const OpView<T>& o, const T* __restrict__ P, T* __restrict__ Q) {
  gather_L<T, NT, DIR>(o, P);
  __syncthreads();
  if constexpr (!DIR) {   // the kernels of the banded form run only when the PSF is separable
    // w = B^T B y: banded pass along rows then along columns, in place
    const TapIdx ti(o.K);
    banded_pass<T, CKT, true>(o.F0, o.pitch, o.h, o.w, o.c0, o.nx, o.ck, o.taps + ti.ax, o.taps + ti.elx,
                              o.taps + ti.erx);
    __syncthreads();
    banded_pass<T, CKT, false>(o.F0, o.pitch, o.w, o.h, o.r0, o.ny, o.ck, o.taps + ti.ay, o.taps + ti.ely,
                               o.taps + ti.ery);
    __syncthreads();
  } else {
    forward_blur<T, CKT, NT, false>(o, o.Z);  // z = B y over the dilated region into global Z
    __syncthreads();
    adjoint_blur<T, CKT, NT>(o, o.Z);  // w = B^T z (at least) at the mapped pixels, in the frame
  }
  return gather_LT<T, NT, false, sizeof(T) == 4 && CKT <= 7>(o, P, Q);
}

// Where an FP64 solve with Monte Carlo draws keeps an item's step lengths for
// k_mcdof: (alpha, beta) of iteration i at p[1 + i], for up to `cap` iterations,
// and the count of iterations in p[0].x (cap -1: no room).  They lie in what the
// member's L^T entries leave free of its region, shared out among its lambdas:
// the region is sized for twice the entries without padding, so that at least
// three eighths of it are free where the entries are paired (128 x 128 pixels, 2 x
// 2 subpixels, 16 lambdas: 12000 iterations or more).
struct CoefRoom {
  double2* p;
  int cap;
};
template <typename T>
__device__ __forceinline__ CoefRoom coef_room(const SolveArgs& a, const MemberInfo& mi, int m, int kl) {
  const long size = (long)sizeof(LtEntry<T>) * a.lt_cap;
  const long E = a.lt_ptr[(long)m * (a.I_max + 65) + (mi.sell ? (mi.I + 63) / 64 : mi.I)];   // entries with padding
  const long used = (E * (long)(mi.sell == 2 ? sizeof(unsigned short) + sizeof(T) : sizeof(LtEntry<T>)) + 15) & ~15L;
  const int each = (int)((size - used) / (long)sizeof(double2) / a.n_lambda);
  return {reinterpret_cast<double2*>(reinterpret_cast<unsigned char*>(a.lt_ent) + m * size + used) + (long)kl * each,
          each - 1};
}

template <typename T, int CKT, int MEM, bool PC, bool DIR>
__device__ __forceinline__ void run_item(const SolveArgs& a, const MemberInfo& mi, int m, int kl, unsigned char* smem) {
  constexpr int NT = kNTof<T>;   // threads of this block
  const int tid = threadIdx.x;
  const long out_idx = (long)m * a.n_lambda + kl;
  T* __restrict__ s_g = reinterpret_cast<T*>(a.s_all) + out_idx * a.I_max;
  // per-block scratch: the preconditioned launch runs beside the plain one and
  // takes the second half of the slots
  const long slot = (long)blockIdx.x + (PC ? (long)gridDim.x : 0L);
  T* __restrict__ r_g = reinterpret_cast<T*>(a.rbuf) + slot * a.I_max;
  const int ns = mi.ns, I = mi.I, M = mi.M, r0 = mi.r0, c0 = mi.c0;
  const int h = mi.r1 - mi.r0 + 1, w = mi.c1 - mi.c0 + 1;
  constexpr int HALO = 2 * CKT;
  const int pitch = (w + 2 * HALO) | 1;
  // kSegR extra rows absorb the tail of the last column window
  const int frame_elems = (h + 2 * HALO + kSegR) * pitch;
  const int J = a.nx * a.ny, n2 = a.n2, nx = a.nx, ny = a.ny, K = a.K, ck = a.ck;
  const T lamT = (T)a.lamv[kl];
  const bool ident = a.reg == SL_H_IDENTITY;
  constexpr bool LDSF = MEM != kMemGlobal;
  const LdsPlan lp = lds_plan<T>(a, I, MEM);
  T* P = reinterpret_cast<T*>(smem + lp.p);
  T* Q;   // (the second half of rbuf is the preconditioned launch's, which FP64 has not)
  if (MEM == kMemLdsQGlobal)
    Q = reinterpret_cast<T*>(a.rbuf) + (slot + (long)gridDim.x) * a.I_max;
  else
    Q = reinterpret_cast<T*>(smem + lp.q);
  double* red = reinterpret_cast<double*>(smem + lp.red);
  T* F;
  if (LDSF)
    F = reinterpret_cast<T*>(smem + lp.frame);
  else
    F = reinterpret_cast<T*>(a.gframe) + (long)blockIdx.x * a.gframe_elems;
  T* const F0 = F + HALO * pitch + HALO;        // interior (0, 0) = image (r0, c0)
  T* const Frows = F + HALO * pitch;            // interior rows, contiguous
  T* Z = reinterpret_cast<T*>(a.gz) + slot * 2L * J;   // z, then W = B^T z (direct blur)
  const int32_t* pix = a.pix_list + (long)m * a.slot_cap;
  const int32_t* cellp = a.cell + (long)m * a.slot_cap * n2;
  const T* fxp = reinterpret_cast<const T*>(a.fx) + (long)m * a.slot_cap * n2;
  const T* fyp = reinterpret_cast<const T*>(a.fy) + (long)m * a.slot_cap * n2;
  const T* taps = reinterpret_cast<const T*>(a.taps_t);
  const TapIdx ti(K);
  const bool sep = a.consts->sep != 0;
  const T inv_n2 = (T)1 / (T)n2;
  const int fo = -r0 * pitch - c0;             // frame offset of image pixel (r, c): r*pitch + c + fo
  const int32_t* lt_rp = a.lt_ptr + (long)m * (a.I_max + 65);
  const int sell = __builtin_amdgcn_readfirstlane(mi.sell);
  const LtEntry<T>* lt_e = reinterpret_cast<const LtEntry<T>*>(a.lt_ent) + (long)m * a.lt_cap;
  // dilated region (direct-blur paths): rows/cols within ck of the bbox, inside the image
  const int Dr0 = max(mi.r0 - ck, 0), Dr1 = min(mi.r1 + ck, ny - 1);
  const int Dc0 = max(mi.c0 - ck, 0), Dc1 = min(mi.c1 + ck, nx - 1);
  const int Dh = Dr1 - Dr0 + 1, Dw = Dc1 - Dc0 + 1;

  // s = 0, r = p = b, Q = 0, frame (with its halo) = 0
  for (int e = tid; e < frame_elems; e += NT) F[e] = (T)0;
  double rr = 0.0;
  const double* bm = a.b + (long)m * a.I_max;
  for (int i = tid; i < I; i += NT) {
    const T bv = (T)bm[i];
    P[i] = bv;
    Q[i] = (T)0;
    s_g[i] = (T)0;
    r_g[i] = bv;
    rr += (double)bv * (double)bv;
  }
  rr = block_sum1<NT / kWave>(rr, red, 0);
  const double stop2 = a.tol * a.tol * rr;
  // PC: preconditioned CG with M = c I + lambda H^T H (FP32, curvature H; the
  // caller checks that the frame holds the n x n scratch): p0 = z0 = M^-1 b.
  double rz = rr;                                       // <r, z>
  if constexpr (PC && sizeof(T) == 4) {
    float* tab = reinterpret_cast<float*>(smem + a.pc_off);
    float* mu = tab + 2 * (ns + 1);
    const double nrm = sqrt(2.0 / (ns + 1)), pi = 3.14159265358979323846;
    for (int e = tid; e < 2 * (ns + 1); e += NT) tab[e] = (float)(nrm * sin(pi * e / (ns + 1)));
    for (int e = tid; e < ns; e += NT) {
      const double sn = sin(pi * (e + 1) / (2.0 * (ns + 1)));
      mu[e] = (float)(16.0 * sn * sn * sn * sn);
    }
    rz = pc_apply(reinterpret_cast<float*>(P), reinterpret_cast<float*>(Q), reinterpret_cast<float*>(F),
                  (a.red_off - a.q_off) / 4, a.lds_frame_cap, tab, mu, ns,
                  reinterpret_cast<const float*>(r_g), mi.pc_c, (float)a.lamv[kl], 0.0, 1, red);
    __syncthreads();
  }
  CoefRoom cf{nullptr, -1};
  if constexpr (sizeof(T) == 8)
    if (a.mcn) cf = coef_room<T>(a, mi, m, kl);
  int st = SL_ST_MAXIT, it = 0;
  for (it = 0; it < a.maxit; ++it) {
    if (__builtin_amdgcn_readfirstlane((int)(rr <= stop2))) {
      st = SL_ST_OK;
      break;
    }
    const OpView<T> ov{pix, cellp, fxp, fyp, F, F0, Z, Z + J, taps, lt_rp, lt_e, a.lt_perm + (long)m * a.I_max, ns,
                       I, M, r0, c0, h, w, pitch, fo, n2, nx, ny, K, ck, sell, Dr0, Dc0, Dh, Dw, sep, ident, inv_n2,
                       lamT, a.interp == SL_INTERP_BICUBIC};
    double pq = apply_normal<T, CKT, NT, DIR>(ov, P, Q);
    pq = block_sum1<NT / kWave>(pq, red, 0);
    // every gather has read the frame (barrier above): back to zero for the next iteration
    clear_rows<T, CKT, NT, DIR>(ov);
    if (__builtin_amdgcn_readfirstlane((int)!(pq > 0.0))) {
      st = SL_ST_BREAKDOWN;
      break;
    }
    const T alT = (T)((PC ? rz : rr) / pq);
    // Updates in chunks of kUpd nodes per thread: every global load of a chunk
    // is issued before the first use, and the updated residual stays in
    // registers for the direction update when the chunk covers all of I.
    double rn = 0.0;
    T rk[kUpd];
    for (int i0 = tid; i0 < I; i0 += kUpd * NT) {
      T sk[kUpd];
#pragma unroll
      for (int k = 0; k < kUpd; ++k) {
        const int i = i0 + k * NT;
        if (i < I) {
          sk[k] = s_g[i];
          rk[k] = r_g[i];
        }
      }
#pragma unroll
      for (int k = 0; k < kUpd; ++k) {
        const int i = i0 + k * NT;
        if (i < I) {
          s_g[i] = sk[k] + alT * P[i];
          rk[k] -= alT * Q[i];
          r_g[i] = rk[k];
          rn += (double)rk[k] * (double)rk[k];
        }
      }
    }
    rn = block_sum1<NT / kWave>(rn, red, 1);
    if constexpr (PC && sizeof(T) == 4) {
      float* tab = reinterpret_cast<float*>(smem + a.pc_off);
      rz = pc_apply(reinterpret_cast<float*>(P), reinterpret_cast<float*>(Q), reinterpret_cast<float*>(F),
                    (a.red_off - a.q_off) / 4, a.lds_frame_cap, tab, tab + 2 * (ns + 1), ns,
                    reinterpret_cast<const float*>(r_g), mi.pc_c, (float)a.lamv[kl], rz, 0, red);
    } else {
      const T beta = (T)(rn / rr);
      if constexpr (sizeof(T) == 8) {
        if (it < cf.cap) cf.p[1 + it] = make_double2((double)alT, (double)beta);   // the same value from every thread
      }
      if (I <= kUpd * NT) {
#pragma unroll
        for (int k = 0; k < kUpd; ++k) {
          const int i = tid + k * NT;
          if (i < I) P[i] = rk[k] + beta * P[i];
        }
      } else {
        for (int i0 = tid; i0 < I; i0 += kUpd * NT) {
#pragma unroll
          for (int k = 0; k < kUpd; ++k) {
            const int i = i0 + k * NT;
            if (i < I) rk[k] = r_g[i];
          }
#pragma unroll
          for (int k = 0; k < kUpd; ++k) {
            const int i = i0 + k * NT;
            if (i < I) P[i] = rk[k] + beta * P[i];
          }
        }
      }
    }
    rr = rn;
    __syncthreads();
  }
  if (st == SL_ST_MAXIT && rr <= stop2) st = SL_ST_OK;
  if constexpr (sizeof(T) == 8)
    if (cf.cap >= 0) cf.p[0] = make_double2((double)it, 0.0);
  // ---- chi^2 and ||H s||^2 from the explicit solution
  __syncthreads();
  for (int i = tid; i < I; i += NT) P[i] = s_g[i];
  for (int e = tid; e < h * pitch; e += NT) Frows[e] = (T)0;
  __syncthreads();
  for (int t = tid; t < M; t += NT) {
    const int rc = pix[t];
    if (rc >= 0)
      F0[(rc >> 16) * pitch + (rc & 0xFFFF) + fo] =
          pixel_gather(P, ns, n2, t, cellp, fxp, fyp, DIR && a.interp == SL_INTERP_BICUBIC) * inv_n2;
  }
  double regacc = 0.0;
  for (int i = tid; i < I; i += NT) regacc += reg_node(P, ns, i / ns, i % ns, a.reg);
  __syncthreads();
  model_image<T, CKT, NT, LDSF>(F0, taps, Z, K, r0, c0, h, w, pitch, Dr0, Dc0, Dh, Dw);
  __syncthreads();
  double cacc = 0.0;
  for (int e = tid; e < Dh * Dw; e += NT) {
    const double zd = (double)Z[e];
    cacc += zd * zd - 2.0 * zd * a.d[(Dr0 + e / Dw) * nx + Dc0 + e % Dw];
  }
  block_sum2(cacc, regacc, red);
  if (tid == 0) {
    a.chi2[out_idx] = (a.consts->sum_d2 + cacc) / (a.sigma * a.sigma);
    a.regv[out_idx] = regacc;
    a.iters[out_idx] = it;
    a.status[out_idx] = st;
  }
  __syncthreads();
}

// Next (member, lambda) item for this block, -1 when every queue is empty;
// thread 0 pops, the value is broadcast through LDS and made scalar.
template <bool PC>
__device__ __forceinline__ int fetch_item(const SolveArgs& a, int xcd, int* sh_item) {
  int* head = PC ? a.consts->pqhead : a.consts->qhead;
  const int* count = PC ? a.consts->pqcount : a.consts->qcount;
  const int* queues = PC ? a.pqueues : a.queues;
  if (threadIdx.x == 0) {
    int item = -1;
    for (int x = 0; x < 8 && item < 0; ++x) {
      const int q = (xcd + x) & 7;
      const int idx = atomicAdd(&head[q], 1);
      if (idx < count[q]) item = queues[q * a.qcap + idx];
    }
    *sh_item = item;
  }
  __syncthreads();
  const int item = __builtin_amdgcn_readfirstlane(*sh_item);
  __syncthreads();
  return item;
}

// Persistent CG kernel: each block pulls (member, lambda) items from its XCD's
// queue (then the others').  PC = true takes the preconditioned items that
// k_split selected (FP32 only); PC = false all the others.
template <typename T, int CKT, bool PC, bool DIR>
__global__ void __launch_bounds__(kNTof<T>) k_solve(SolveArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int sh_item;
  if (__builtin_amdgcn_readfirstlane(a.consts->sep) == (int)DIR) return;   // the other form's launch does the work
  const int xcd = blockIdx.x & 7;
  for (int item = fetch_item<PC>(a, xcd, &sh_item); item >= 0; item = fetch_item<PC>(a, xcd, &sh_item)) {
    const int m = item / a.n_lambda, kl = item % a.n_lambda;   // scalar
    const MemberInfo mi = a.minfo[m];                          // uniform address: scalar loads
    if constexpr (PC) {
      run_item<T, CKT, kMemLds, true, DIR>(a, mi, m, kl, smem);
    } else {
      const int status = __builtin_amdgcn_readfirstlane(mi.status);
      const int fits = __builtin_amdgcn_readfirstlane(mi.lds_frame);
      if (status != SL_ST_OK)
        trivial_item<T>(a, mi, m, kl);
      else if (fits == kMemGlobal)
        run_item<T, CKT, kMemGlobal, false, DIR>(a, mi, m, kl, smem);
      else
        run_item<T, CKT, lds_mem<T>(CKT), false, DIR>(a, mi, m, kl, smem);
    }
  }
}

// ------------------------------------------------------------------ k_mcdof
// Next member of the Monte Carlo pass for this block (thread 0 takes it, the
// value is broadcast through LDS and made scalar), as fetch_item does.
__device__ __forceinline__ int fetch_counter(int* counter, int* sh_m) {
  if (threadIdx.x == 0) *sh_m = atomicAdd(counter, 1);
  __syncthreads();
  const int m = __builtin_amdgcn_readfirstlane(*sh_m);
  __syncthreads();
  return m;
}

// Monte Carlo degrees of freedom of one member at its corner lambda (Sec. 2.5).
// FP64: the system with right-hand side A^T bhat is advanced with the data
// system's alpha_k and beta_k (not its own).  Where the solve had room for all of
// them (CoefRoom) they are read back; otherwise the data system's plain CG runs
// again in lockstep, with its p in LDS (P) and the second system's direction
// swapped into P for its operator application; both give the same bits.  FP32:
// the second system by its own CG (see below).  Then gamma = <A^T bhat, xhat>
// = bhat^T A xhat and dof = bhat^T bhat - gamma.  Per-block scratch (global):
// r, xhat, rhat, phat and the saved p.
template <typename T, int CKT, int MEM, bool DIR>
__device__ __forceinline__ void run_mc_item(const SolveArgs& a, const MemberInfo& mi, int m, int kl,
                                            unsigned char* smem) {
  constexpr int NT = kNTof<T>;
  const int tid = threadIdx.x;
  const long slot = (long)blockIdx.x;
  T* __restrict__ r_g = reinterpret_cast<T*>(a.mcbuf) + slot * 5L * a.I_max;
  T* __restrict__ xh_g = r_g + a.I_max;
  T* __restrict__ rh_g = xh_g + a.I_max;
  T* __restrict__ ph_g = rh_g + a.I_max;
  T* __restrict__ pd_g = ph_g + a.I_max;
  const int ns = mi.ns, I = mi.I, M = mi.M, r0 = mi.r0, c0 = mi.c0;
  const int h = mi.r1 - mi.r0 + 1, w = mi.c1 - mi.c0 + 1;
  constexpr int HALO = 2 * CKT;
  const int pitch = (w + 2 * HALO) | 1;
  const int frame_elems = (h + 2 * HALO + kSegR) * pitch;
  const int J = a.nx * a.ny, n2 = a.n2, nx = a.nx, ny = a.ny, K = a.K, ck = a.ck;
  const LdsPlan lp = lds_plan<T>(a, I, MEM);
  T* P = reinterpret_cast<T*>(smem + lp.p);
  T* Q = MEM == kMemLdsQGlobal ? reinterpret_cast<T*>(a.rbuf) + slot * a.I_max : reinterpret_cast<T*>(smem + lp.q);
  double* red = reinterpret_cast<double*>(smem + lp.red);
  T* F = MEM != kMemGlobal ? reinterpret_cast<T*>(smem + lp.frame)
                           : reinterpret_cast<T*>(a.gframe) + slot * a.gframe_elems;
  T* const F0 = F + HALO * pitch + HALO;
  const int Dr0 = max(mi.r0 - ck, 0), Dr1 = min(mi.r1 + ck, ny - 1);
  const int Dc0 = max(mi.c0 - ck, 0), Dc1 = min(mi.c1 + ck, nx - 1);
  const OpView<T> ov{a.pix_list + (long)m * a.slot_cap, a.cell + (long)m * a.slot_cap * n2,
                     reinterpret_cast<const T*>(a.fx) + (long)m * a.slot_cap * n2,
                     reinterpret_cast<const T*>(a.fy) + (long)m * a.slot_cap * n2, F, F0,
                     reinterpret_cast<T*>(a.gz) + slot * 2L * J, reinterpret_cast<T*>(a.gz) + slot * 2L * J + J,
                     reinterpret_cast<const T*>(a.taps_t), a.lt_ptr + (long)m * (a.I_max + 65),
                     reinterpret_cast<const LtEntry<T>*>(a.lt_ent) + (long)m * a.lt_cap, a.lt_perm + (long)m * a.I_max,
                     ns, I, M, r0, c0, h, w, pitch, -r0 * pitch - c0, n2, nx, ny, K, ck,
                     __builtin_amdgcn_readfirstlane(mi.sell), Dr0, Dc0, Dr1 - Dr0 + 1, Dc1 - Dc0 + 1,
                     a.consts->sep != 0, a.reg == SL_H_IDENTITY, (T)1 / (T)n2, (T)a.lamv[kl],
                     a.interp == SL_INTERP_BICUBIC};
  for (int e = tid; e < frame_elems; e += NT) F[e] = (T)0;
  const double* bm = a.b + (long)m * a.I_max;
  const double* bhm = a.bh + (long)m * a.I_max;
  if constexpr (sizeof(T) == 4) {
    // FP32: the lockstep recurrence is linear in the second system with fixed
    // coefficients, so FP32 rounding injected at one step grows with the data
    // polynomial's later factors; here the second system is solved by its own
    // CG instead (same operator, same stopping rule relative to ||A^T bhat||),
    // which estimates the same Tikhonov gamma (Eq. 19) once converged.
    double rr = 0.0;
    for (int i = tid; i < I; i += NT) {
      const T nv = (T)bhm[i];
      P[i] = nv;
      rh_g[i] = nv;
      xh_g[i] = (T)0;
      rr += (double)nv * (double)nv;
    }
    rr = block_sum1<NT / kWave>(rr, red, 0);
    const double stop2 = a.tol * a.tol * rr;
    for (int it = 0; it < a.maxit; ++it) {
      if (__builtin_amdgcn_readfirstlane((int)(rr <= stop2))) break;
      double pq = apply_normal<T, CKT, NT, DIR>(ov, P, Q);
      pq = block_sum1<NT / kWave>(pq, red, 0);
      clear_rows<T, CKT, NT, DIR>(ov);
      if (__builtin_amdgcn_readfirstlane((int)!(pq > 0.0))) break;
      const T alT = (T)(rr / pq);
      double rn = 0.0;
      for (int i = tid; i < I; i += NT) {
        xh_g[i] += alT * P[i];
        const T rk = rh_g[i] - alT * Q[i];
        rh_g[i] = rk;
        rn += (double)rk * (double)rk;
      }
      rn = block_sum1<NT / kWave>(rn, red, 1);
      const T beta = (T)(rn / rr);
      for (int i = tid; i < I; i += NT) P[i] = rh_g[i] + beta * P[i];
      rr = rn;
      __syncthreads();
    }
  } else {
    const CoefRoom cf = coef_room<T>(a, mi, m, kl);
    const int n_it = __builtin_amdgcn_readfirstlane(cf.cap >= 0 ? (int)cf.p[0].x : INT_MAX);
    if (n_it <= cf.cap) {
      // The data system's step lengths as k_solve left them: only the second
      // system is advanced (solving the data system again in lockstep, as below,
      // took twice the operator applications: 170 ms for 64 c3 members, 83 ms so).
      for (int i = tid; i < I; i += NT) {
        const T nv = (T)bhm[i];
        P[i] = nv;
        rh_g[i] = nv;
        xh_g[i] = (T)0;
      }
      __syncthreads();
      for (int it = 0; it < n_it; ++it) {
        (void)apply_normal<T, CKT, NT, DIR>(ov, P, Q);
        __syncthreads();   // every gather has read P and the frame
        clear_rows<T, CKT, NT, DIR>(ov);
        const T alT = (T)cf.p[1 + it].x, beta = (T)cf.p[1 + it].y;
        for (int i = tid; i < I; i += NT) {
          const T ph = P[i];
          xh_g[i] += alT * ph;
          const T rk = rh_g[i] - alT * Q[i];
          rh_g[i] = rk;
          P[i] = rk + beta * ph;
        }
        __syncthreads();
      }
    } else {
      double rr = 0.0;
      for (int i = tid; i < I; i += NT) {
        const T bv = (T)bm[i], nv = (T)bhm[i];
        P[i] = bv;
        r_g[i] = bv;
        rr += (double)bv * (double)bv;
        xh_g[i] = (T)0;
        rh_g[i] = nv;
        ph_g[i] = nv;
      }
      rr = block_sum1<NT / kWave>(rr, red, 0);
      const double stop2 = a.tol * a.tol * rr;
      for (int it = 0; it < a.maxit; ++it) {
        if (__builtin_amdgcn_readfirstlane((int)(rr <= stop2))) break;
        // data system: q = A p, alpha, r update, beta, new p (saved to global)
        double pq = apply_normal<T, CKT, NT, DIR>(ov, P, Q);
        pq = block_sum1<NT / kWave>(pq, red, 0);
        clear_rows<T, CKT, NT, DIR>(ov);
        if (__builtin_amdgcn_readfirstlane((int)!(pq > 0.0))) break;
        const T alT = (T)(rr / pq);
        double rn = 0.0;
        for (int i = tid; i < I; i += NT) {
          const T rk = r_g[i] - alT * Q[i];
          r_g[i] = rk;
          rn += (double)rk * (double)rk;
        }
        rn = block_sum1<NT / kWave>(rn, red, 1);
        const T beta = (T)(rn / rr);
        for (int i = tid; i < I; i += NT) {
          pd_g[i] = r_g[i] + beta * P[i];
          P[i] = ph_g[i];
        }
        __syncthreads();
        // second system with the same alpha and beta
        double pqh = apply_normal<T, CKT, NT, DIR>(ov, P, Q);
        pqh = block_sum1<NT / kWave>(pqh, red, 0);   // its barrier: every gather has read P and the frame
        (void)pqh;
        clear_rows<T, CKT, NT, DIR>(ov);
        for (int i = tid; i < I; i += NT) {
          const T ph = P[i];
          xh_g[i] += alT * ph;
          const T rk = rh_g[i] - alT * Q[i];
          rh_g[i] = rk;
          ph_g[i] = rk + beta * ph;
          P[i] = pd_g[i];
        }
        rr = rn;
        __syncthreads();
      }
    }
  }
  double g = 0.0;
  for (int i = tid; i < I; i += NT) g += bhm[i] * (double)xh_g[i];
  g = block_sum1<NT / kWave>(g, red, 1);
  // every thread stores the same value: no lane-predicated store in the member loop
  a.dofv[m] = a.consts->sum_n2 - g;
  __syncthreads();
}

// One member per item, in member order, at the member's L-curve corner; a
// member without a solve (invalid, or no pixel maps) gets NaN.  The member
// loop holds no lane-predicated code besides the fetch (the form k_solve
// uses): a store under `threadIdx.x == 0` followed by `continue` was compiled
// into an inner loop that thread 0's lane left to do the store while the
// other lanes went on re-reading an item index that only thread 0 advances.
template <typename T, int CKT, bool DIR>
__global__ void __launch_bounds__(kNTof<T>) k_mcdof(SolveArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int sh_m;
  if (__builtin_amdgcn_readfirstlane(a.consts->sep) == (int)DIR) return;   // the other form's launch does the work
  for (int m = fetch_counter(&a.consts->mchead, &sh_m); m < a.n_members;
       m = fetch_counter(&a.consts->mchead, &sh_m)) {
    const MemberInfo mi = a.minfo[m];
    const int status = __builtin_amdgcn_readfirstlane(mi.status);
    if (status != SL_ST_OK) {
      a.dofv[m] = NAN;   // the same value from every thread
    } else {
      const int kl = __builtin_amdgcn_readfirstlane(a.k_star[m]);
      const int mem = __builtin_amdgcn_readfirstlane(mi.lds_frame);
      if (mem == kMemGlobal)
        run_mc_item<T, CKT, kMemGlobal, DIR>(a, mi, m, kl, smem);
      else
        run_mc_item<T, CKT, lds_mem<T>(CKT), DIR>(a, mi, m, kl, smem);
    }
  }
}

// ------------------------------------------------------------------ k_implicit
// Implicit regularisation by the iteration count (Sec. 2.4, Sec. 2.6): CGLS
// on min ||A s - d|| (A = B L) from s = 0 with no lambda, for exactly
// n_lambda iterations.  Each iteration applies A once (L gather, then B over
// the dilated bounding box) and A^T once (B^T at the mapped pixels, then the
// L^T gather), as CGLS does: q = A p, alpha = ||g||^2 / ||q||^2,
// s += alpha p, e -= alpha q, g = A^T e, beta = ||g'||^2 / ||g||^2,
// p = g + beta p, with the image residual e = d - A s carried on the dilated
// box (pixels outside it keep e = d; A^T e reads only the box).  After
// iteration k the iterate goes to solution slot k of the member, with
// chi^2 = ||e||^2 / sigma^2 and the zeroth-order measure ||s_k||^2 (Sec. 2.6).
// g_0 = A^T d is the member's fixed-order right-hand side.  After a
// breakdown (A p = 0) the remaining slots repeat the last iterate.
//
// Monte Carlo degrees of freedom (Sec. 2.5; FP64 only, mcn not NULL): a
// second system with data bhat advanced with the data system's alpha_k and
// beta_k, not its own (xhat += alpha phat, ehat -= alpha A phat,
// phat = A^T ehat + beta phat, from xhat = 0, ehat = bhat, phat = A^T bhat),
// so that xhat_k is the data system's k-step filter applied to bhat; after
// every iteration bhat^T (bhat - A xhat_k) = ||bhat||^2 - <A^T bhat, xhat_k>
// goes to dofk, and k_corner takes the value at the corner.  Its vectors
// live in the block's global scratch: xhat, phat and A^T ehat in mcbuf, ehat
// on the dilated box in the second half of gz.
template <typename T, int CKT, int MEM>
__device__ __forceinline__ void run_implicit_item(const SolveArgs& a, const MemberInfo& mi, int m,
                                                  unsigned char* smem) {
  constexpr int NT = kNTof<T>;
  const int tid = threadIdx.x;
  const long slot = (long)blockIdx.x;
  const int K_it = a.n_lambda;
  const int ns = mi.ns, I = mi.I, M = mi.M, r0 = mi.r0, c0 = mi.c0;
  const int h = mi.r1 - mi.r0 + 1, w = mi.c1 - mi.c0 + 1;
  constexpr int HALO = 2 * CKT;
  const int pitch = (w + 2 * HALO) | 1;
  const int frame_elems = (h + 2 * HALO + kSegR) * pitch;
  const int J = a.nx * a.ny, n2 = a.n2, nx = a.nx, ny = a.ny, K = a.K, ck = a.ck;
  const LdsPlan lp = lds_plan<T>(a, I, MEM);
  T* P = reinterpret_cast<T*>(smem + lp.p);               // search direction p
  T* G = MEM == kMemLdsQGlobal ? reinterpret_cast<T*>(a.rbuf) + slot * a.I_max   // gradient g = A^T e
                               : reinterpret_cast<T*>(smem + lp.q);
  double* red = reinterpret_cast<double*>(smem + lp.red);
  T* F = MEM != kMemGlobal ? reinterpret_cast<T*>(smem + lp.frame)
                           : reinterpret_cast<T*>(a.gframe) + slot * a.gframe_elems;
  T* const F0 = F + HALO * pitch + HALO;
  const int Dr0 = max(mi.r0 - ck, 0), Dr1 = min(mi.r1 + ck, ny - 1);
  const int Dc0 = max(mi.c0 - ck, 0), Dc1 = min(mi.c1 + ck, nx - 1);
  const int Dh = Dr1 - Dr0 + 1, Dw = Dc1 - Dc0 + 1;
  T* __restrict__ Zq = reinterpret_cast<T*>(a.gz) + slot * 2L * J;   // q = A p on the dilated box, then W
  T* __restrict__ E = reinterpret_cast<T*>(a.ibuf) + slot * J;        // e on the dilated box
  const bool mc = sizeof(T) == 8 && a.mcn != nullptr;               // uniform: a kernel argument
  T* __restrict__ xh = reinterpret_cast<T*>(a.mcbuf) + slot * 5L * a.I_max;
  T* __restrict__ ph = xh + a.I_max;
  T* __restrict__ gh = ph + a.I_max;
  T* __restrict__ Eh = reinterpret_cast<T*>(a.gz) + ((long)gridDim.x + slot) * 2L * J;   // ehat on the dilated box
  const double* bhm = a.bh + (long)m * a.I_max;
  const OpView<T> ov{a.pix_list + (long)m * a.slot_cap, a.cell + (long)m * a.slot_cap * n2,
                     reinterpret_cast<const T*>(a.fx) + (long)m * a.slot_cap * n2,
                     reinterpret_cast<const T*>(a.fy) + (long)m * a.slot_cap * n2, F, F0, Zq, Zq + J,
                     reinterpret_cast<const T*>(a.taps_t), a.lt_ptr + (long)m * (a.I_max + 65),
                     reinterpret_cast<const LtEntry<T>*>(a.lt_ent) + (long)m * a.lt_cap, a.lt_perm + (long)m * a.I_max,
                     ns, I, M, r0, c0, h, w, pitch, -r0 * pitch - c0, n2, nx, ny, K, ck,
                     __builtin_amdgcn_readfirstlane(mi.sell), Dr0, Dc0, Dh, Dw,
                     a.consts->sep != 0, true, (T)1 / (T)n2, (T)0, a.interp == SL_INTERP_BICUBIC};
  // Frame: zero outside the mapped pixels whenever L p is gathered into it
  // (the adjoint blur's other writes are cleared after each L^T gather).
  for (int e = tid; e < frame_elems; e += NT) F[e] = (T)0;
  const double* bm = a.b + (long)m * a.I_max;
  double gg = 0.0, din = 0.0;
  for (int i = tid; i < I; i += NT) {
    const T bv = (T)bm[i];
    P[i] = bv;
    gg += (double)bv * (double)bv;
  }
  for (int e = tid; e < Dh * Dw; e += NT) {
    const double dv = a.d[(Dr0 + e / Dw) * nx + Dc0 + e % Dw];
    E[e] = (T)dv;
    din += dv * dv;
  }
  if (mc) {
    for (int i = tid; i < I; i += NT) {
      xh[i] = (T)0;
      ph[i] = (T)bhm[i];
    }
    for (int e = tid; e < Dh * Dw; e += NT) Eh[e] = (T)a.mcn[(Dr0 + e / Dw) * nx + Dc0 + e % Dw];
  }
  block_sum2(gg, din, red + 32);
  const double d_out = a.consts->sum_d2 - din;   // sum of d^2 outside the dilated box
  const double inv_s2 = 1.0 / (a.sigma * a.sigma);
  int k = 0, st = SL_ST_OK;
  double chi2_last = a.consts->sum_d2 * inv_s2, reg_last = 0.0, dof_last = a.consts->sum_n2;
  for (; k < K_it; ++k) {
    if (__builtin_amdgcn_readfirstlane((int)(gg <= 0.0))) break;
    gather_L<T, NT>(ov, P);                               // frame = L p
    __syncthreads();
    double qq = forward_blur<T, CKT, NT, true>(ov, Zq);         // q = B L p
    qq = block_sum1<NT / kWave>(qq, red, 0);
    if (__builtin_amdgcn_readfirstlane((int)!(qq > 0.0))) {
      st = SL_ST_BREAKDOWN;
      break;
    }
    const T alT = (T)(gg / qq);
    const T* s_prev = reinterpret_cast<const T*>(a.s_all) + ((long)m * K_it + (k > 0 ? k - 1 : 0)) * a.I_max;
    T* s_k = reinterpret_cast<T*>(a.s_all) + ((long)m * K_it + k) * a.I_max;
    double reg = 0.0, ee = 0.0;
    for (int i = tid; i < I; i += NT) {
      const T sv = (k ? s_prev[i] : (T)0) + alT * P[i];
      s_k[i] = sv;
      reg += (double)sv * (double)sv;
    }
    for (int e = tid; e < Dh * Dw; e += NT) {
      const T ev = E[e] - alT * Zq[e];
      E[e] = ev;
      ee += (double)ev * (double)ev;
    }
    block_sum2(reg, ee, red + 32);                        // also orders the E writes before B^T reads them
    chi2_last = (d_out + ee) * inv_s2;
    reg_last = reg;
    {   // every thread stores the same block-reduced values: no lane-predicated code in the loop
      const long o = (long)m * K_it + k;
      a.chi2[o] = chi2_last;
      a.regv[o] = reg_last;
      a.iters[o] = k + 1;
      a.status[o] = SL_ST_OK;
    }
    adjoint_blur<T, CKT, NT>(ov, E);                      // frame = B^T e at the mapped pixels
    double gn = gather_LT<T, NT, true>(ov, P, G);         // g = L^T B^T e
    gn = block_sum1<NT / kWave>(gn, red, 1);
    clear_rows<T, CKT, NT, true>(ov);                           // every gather has read the frame
    const T beta = (T)(gn / gg);
    for (int i = tid; i < I; i += NT) P[i] = G[i] + beta * P[i];
    gg = gn;
    if (mc) {   // the second system with this iteration's alpha and beta
      __syncthreads();                                    // the frame is clear again
      gather_L<T, NT>(ov, ph);
      __syncthreads();
      forward_blur<T, CKT, NT, false>(ov, Zq);                   // A phat
      __syncthreads();
      double gam = 0.0;
      for (int i = tid; i < I; i += NT) {
        const T xv = xh[i] + alT * ph[i];
        xh[i] = xv;
        gam += bhm[i] * (double)xv;
      }
      for (int e = tid; e < Dh * Dw; e += NT) Eh[e] -= alT * Zq[e];
      gam = block_sum1<NT / kWave>(gam, red, 0);          // its barrier: ehat complete
      adjoint_blur<T, CKT, NT>(ov, Eh);
      gather_LT<T, NT, true>(ov, ph, gh);                 // A^T ehat
      __syncthreads();
      clear_rows<T, CKT, NT, true>(ov);
      for (int i = tid; i < I; i += NT) ph[i] = gh[i] + beta * ph[i];
      dof_last = a.consts->sum_n2 - gam;
      a.dofk[(long)m * K_it + k] = dof_last;              // the same value from every thread
    }
    __syncthreads();
  }
  // slots past an early stop repeat the last iterate (s = 0 when there is none)
  for (int kk = k; kk < K_it; ++kk) {
    const T* s_prev = reinterpret_cast<const T*>(a.s_all) + ((long)m * K_it + (kk > 0 ? kk - 1 : 0)) * a.I_max;
    T* s_k = reinterpret_cast<T*>(a.s_all) + ((long)m * K_it + kk) * a.I_max;
    for (int i = tid; i < I; i += NT) s_k[i] = kk ? s_prev[i] : (T)0;
    const long o = (long)m * K_it + kk;
    a.chi2[o] = chi2_last;
    a.regv[o] = reg_last;
    a.iters[o] = k;
    a.status[o] = st;
    if (mc) a.dofk[o] = dof_last;
    __syncthreads();
  }
}

// One member per item; members without a solve get the trivial result.
template <typename T, int CKT>
__global__ void __launch_bounds__(kNTof<T>) k_implicit(SolveArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int sh_m;
  for (int m = fetch_counter(&a.consts->imhead, &sh_m); m < a.n_members; m = fetch_counter(&a.consts->imhead, &sh_m)) {
    const MemberInfo mi = a.minfo[m];
    const int status = __builtin_amdgcn_readfirstlane(mi.status);
    if (status != SL_ST_OK) {   // same values from every thread, as trivial_item writes them
      const double c2 = status == SL_ST_INVALID ? NAN : a.consts->sum_d2 / (a.sigma * a.sigma);
      for (int k = 0; k < a.n_lambda; ++k) {
        T* s_dst = reinterpret_cast<T*>(a.s_all) + ((long)m * a.n_lambda + k) * a.I_max;
        for (int i = threadIdx.x; i < mi.I; i += kNTof<T>) s_dst[i] = (T)0;
        const long o = (long)m * a.n_lambda + k;
        a.chi2[o] = c2;
        a.regv[o] = status == SL_ST_INVALID ? NAN : 0.0;
        a.iters[o] = 0;
        a.status[o] = status;
      }
    } else {
      const int mem = __builtin_amdgcn_readfirstlane(mi.lds_frame);
      if (mem == kMemGlobal)
        run_implicit_item<T, CKT, kMemGlobal>(a, mi, m, smem);
      else
        run_implicit_item<T, CKT, lds_mem<T>(CKT)>(a, mi, m, smem);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ k_chi2_src
// Image chi^2 of candidate sources for one lens: the fitness of the
// source-refinement search (Sec. 3.2), where every source node is a free
// parameter and the lens is held fixed.  chi2[p] = ||B L s_p - d||^2 / sigma^2
// over all J pixels (Eq. 4; pixels outside the dilated bounding box of the
// mapped pixels keep their data).  k_setup and k_prep_* have built member 0's
// trace table.  Persistent over the candidates: block b takes p = b, b +
// gridDim.x, ...; the source is staged in LDS (in the bulk type), L gathers
// it into the frame, B runs over the dilated box into Z, and the residual
// sum is FP64.  The frame holds values at the mapped pixels only, each of
// which every gather overwrites, so it is zeroed once.
template <typename T, int CKT, bool LDSF>
__device__ __forceinline__ void run_chi2_src(const SolveArgs& a, const MemberInfo& mi, const double* src, int n_src,
                                             double* chi2, unsigned char* smem) {
  constexpr int NT = kNTof<T>;
  const int tid = threadIdx.x;
  const double inv_s2 = 1.0 / (a.sigma * a.sigma);
  const int ns = mi.ns, I = mi.I, M = mi.M, r0 = mi.r0, c0 = mi.c0;
  const int h = mi.r1 - mi.r0 + 1, w = mi.c1 - mi.c0 + 1;
  constexpr int HALO = 2 * CKT;
  const int pitch = (w + 2 * HALO) | 1;
  const int frame_elems = (h + 2 * HALO + kSegR) * pitch;
  const int J = a.nx * a.ny, n2 = a.n2, nx = a.nx, ny = a.ny, K = a.K, ck = a.ck;
  const long slot = (long)blockIdx.x;
  const LdsPlan lp = lds_plan<T>(a, I, kMemLdsQGlobal);   // no second vector
  T* S = reinterpret_cast<T*>(smem + lp.p);
  double* red = reinterpret_cast<double*>(smem + lp.red);
  T* F = LDSF ? reinterpret_cast<T*>(smem + lp.frame) : reinterpret_cast<T*>(a.gframe) + slot * a.gframe_elems;
  T* const F0 = F + HALO * pitch + HALO;
  const int Dr0 = max(mi.r0 - ck, 0), Dr1 = min(mi.r1 + ck, ny - 1);
  const int Dc0 = max(mi.c0 - ck, 0), Dc1 = min(mi.c1 + ck, nx - 1);
  const int Dh = Dr1 - Dr0 + 1, Dw = Dc1 - Dc0 + 1;
  T* __restrict__ Z = reinterpret_cast<T*>(a.gz) + slot * 2L * J;
  const OpView<T> ov{a.pix_list, a.cell, reinterpret_cast<const T*>(a.fx), reinterpret_cast<const T*>(a.fy), F, F0,
                     Z, Z + J, reinterpret_cast<const T*>(a.taps_t), a.lt_ptr,
                     reinterpret_cast<const LtEntry<T>*>(a.lt_ent), a.lt_perm, ns, I, M, r0, c0, h, w, pitch,
                     -r0 * pitch - c0, n2, nx, ny, K, ck, __builtin_amdgcn_readfirstlane(mi.sell), Dr0, Dc0, Dh, Dw,
                     a.consts->sep != 0, true, (T)1 / (T)n2, (T)0, a.interp == SL_INTERP_BICUBIC};
  for (int e = tid; e < frame_elems; e += NT) F[e] = (T)0;
  double din = 0.0;
  for (int e = tid; e < Dh * Dw; e += NT) {
    const double dv = a.d[(Dr0 + e / Dw) * nx + Dc0 + e % Dw];
    din += dv * dv;
  }
  din = block_sum1<NT / kWave>(din, red, 0);
  const double d_out = a.consts->sum_d2 - din;   // data outside the dilated box
  for (int p = blockIdx.x; p < n_src; p += gridDim.x) {
    const double* sp = src + (long)p * I;
    for (int i = tid; i < I; i += NT) S[i] = (T)sp[i];
    __syncthreads();
    gather_L<T, NT>(ov, S);                      // frame = L s_p at the mapped pixels
    __syncthreads();
    forward_blur<T, CKT, NT, false>(ov, Z);             // Z = B L s_p over the dilated box
    __syncthreads();
    double acc = 0.0;
    for (int e = tid; e < Dh * Dw; e += NT) {
      const double r = (double)Z[e] - a.d[(Dr0 + e / Dw) * nx + Dc0 + e % Dw];
      acc += r * r;
    }
    acc = block_sum1<NT / kWave>(acc, red, 1);   // its barrier: every read of S, the frame and Z is done
    chi2[p] = (acc + d_out) * inv_s2;            // the same value from every thread
    __syncthreads();
  }
}

// The frame's place is a template argument: through a pointer that may be to
// either memory every access to the frame is a flat one.
template <typename T, int CKT>
__global__ void __launch_bounds__(kNTof<T>) k_chi2_src(SolveArgs a, const double* src, int n_src, double* chi2) {
  extern __shared__ __align__(16) unsigned char smem[];
  const MemberInfo mi = a.minfo[0];
  const int status = __builtin_amdgcn_readfirstlane(mi.status);
  if (status != SL_ST_OK) {   // no mapped pixel (chi^2 of s = 0) or invalid lens (NaN)
    const double c2 = status == SL_ST_INVALID ? NAN : a.consts->sum_d2 * (1.0 / (a.sigma * a.sigma));
    for (int p = blockIdx.x; p < n_src; p += gridDim.x) chi2[p] = c2;   // the same value from every thread
  } else if (__builtin_amdgcn_readfirstlane(mi.lds_frame) != kMemGlobal) {
    run_chi2_src<T, CKT, true>(a, mi, src, n_src, chi2, smem);
  } else {
    run_chi2_src<T, CKT, false>(a, mi, src, n_src, chi2, smem);
  }
}

// The candidate-source chi^2 kernel of the bulk type and window (the windows
// the solve kernels are compiled for).
using Chi2Kernel = void (*)(SolveArgs, const double*, int, double*);
template <typename T>
static Chi2Kernel pick_chi2_kernel(int ckt) {
  if (sizeof(T) == 4) {
    switch (ckt) {
      case 2: return k_chi2_src<float, 2>;
      case 4: return k_chi2_src<float, 4>;
      case 7: return k_chi2_src<float, 7>;
      case 10: return k_chi2_src<float, 10>;
      case 16: return k_chi2_src<float, 16>;
    }
  } else {
    switch (ckt) {
      case 2: return k_chi2_src<double, 2>;
      case 7: return k_chi2_src<double, 7>;
      case 10: return k_chi2_src<double, 10>;
    }
  }
  return nullptr;
}

// Finishes the preconditioner's scale of every member (the sums of
// k_prep_rhs's blocks, in block order) and moves the items that take the
// spectral preconditioner into their own queues (stable, per XCD queue): valid
// member, FP32, curvature H, frame in LDS with room for the n x n scratch, and
// lambda >= pc_theta c.  One block, one wave per queue, 64 items per step (a
// lane per queue took 190 us for 4096 items and 290 us for 6144).
template <typename T>
__global__ void __launch_bounds__(512) k_split(SolveArgs a) {
  for (int m = threadIdx.x; m < a.n_members; m += 512) {
    double num = 0.0, den = 0.0;
    const double* pc = a.pcpart + 2L * m * a.rhs_blocks;
    const int n = a.minfo[m].status == SL_ST_OK ? min(rhs_blocks_of(a.minfo[m].I), a.rhs_blocks) : 0;
    for (int i = 0; i < n; ++i) {
      num += pc[2 * i];
      den += pc[2 * i + 1];
    }
    a.minfo[m].pc_c = den > 0.0 ? (float)(num / den) : 0.0f;
  }
  __syncthreads();
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = a.consts->qcount[q];
  int* Q = a.queues + q * a.qcap;
  int* PQ = a.pqueues + q * a.qcap;
  int keep = 0, moved = 0;
  for (int k0 = 0; k0 < n; k0 += 64) {   // in place: what is written lies before the items still to be read
    const int k = k0 + lane;
    const int item = k < n ? Q[k] : -1;
    bool pc = false;
    if (item >= 0) {
      const MemberInfo mi = a.minfo[item / a.n_lambda];
      const double lam = a.lamv[item % a.n_lambda];
      pc = sizeof(T) == 4 && a.reg == SL_H_CURVATURE && !a.plain_cg && mi.status == SL_ST_OK && mi.lds_frame != 0 &&
           mi.ns * mi.ns <= a.lds_frame_cap && lam >= (double)a.pc_theta * mi.pc_c;
    }
    const unsigned long long mp = __ballot(pc), mk = __ballot(item >= 0 && !pc);
    const int jp = moved + lanes_below(mp), jk = keep + lanes_below(mk);
    if (pc) PQ[jp] = item;
    if (item >= 0 && !pc) Q[jk] = item;
    moved += __popcll(mp);
    keep += __popcll(mk);
  }
  if (lane == 0) {
    a.consts->qcount[q] = keep;
    a.consts->pqcount[q] = moved;
    a.consts->pqhead[q] = 0;
  }
}

// ------------------------------------------------------------------ k_corner
template <typename T>
__global__ void __launch_bounds__(256) k_corner(SolveArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* scratch = reinterpret_cast<double*>(smem);
  __shared__ int sh_k;
  const int m = blockIdx.x;
  const int nl = a.n_lambda;
  const MemberInfo mi = a.minfo[m];
  // the corner by the whole block (the condition is the same for every thread)
  const int kk = (mi.status == SL_ST_OK && nl >= 4)
                     ? lcurve_corner_block(a.regv + (long)m * nl, a.chi2 + (long)m * nl, nl, scratch)
                     : -1;
  if (threadIdx.x == 0) {
    int k = 0, cst = mi.status;
    if (mi.status == SL_ST_OK) {
      if (nl >= 4) {
        if (kk >= 0)
          k = kk;
        else
          cst = SL_ST_LCURVE;
      } else if (nl > 1) {
        cst = SL_ST_LCURVE;
      }
    }
    // a curve through an unconverged point is flagged (its corner is still computed)
    if (cst == SL_ST_OK)
      for (int j = 0; j < nl; ++j) {
        const int sj = a.status[(long)m * nl + j];
        if (sj == SL_ST_MAXIT || sj == SL_ST_BREAKDOWN) {
          cst = sj;
          break;
        }
      }
    a.k_star[m] = k;
    a.corner_status[m] = cst;
    if (a.implicit && a.dofv) a.dofv[m] = mi.status == SL_ST_OK ? a.dofk[(long)m * nl + k] : NAN;
    sh_k = k;
  }
  __syncthreads();
  const T* src = reinterpret_cast<const T*>(a.s_all) + ((long)m * nl + sh_k) * a.I_max;
  for (int i = threadIdx.x; i < mi.I; i += blockDim.x) a.s_corner[mi.off + i] = (double)src[i];
}

// ------------------------------------------------------------------ host side
static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// k_setup's dynamic LDS: the tap table and the PSF of the largest PSF size
// (65.5 + 31.8 KB at 63 x 63)
static const size_t kSetupLds = sizeof(double) * ((size_t)TapIdx(SL_MAX_PSF).total + SL_MAX_PSF * SL_MAX_PSF);

template <typename T>
static int setup_lds_attr() {
  static std::once_flag once;
  static hipError_t err = hipSuccess;
  std::call_once(once, [] {
    err = hipFuncSetAttribute((const void*)k_setup<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSetupLds);
  });
  SL_HIP(err);
  return SL_OK;
}

// Bytes after the solve's workspace that sl_chi2_sources uses: the device
// copy of ns, then the member offsets k_setup writes.
constexpr size_t kSrcTail = 512;

// *p = v, from a launch argument (so that the write can be captured).
__global__ void k_put_int(int32_t* p, int v) {
  if (threadIdx.x == 0) *p = v;
}

int device_cus() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (dev < 0 || dev >= 64) return 256;
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}

static Layout make_layout(const sl_problem* pb, int max_ns, int M, int NL, int n_wg) {
  Layout L{};
  const size_t sz = pb->dtype == SL_F64 ? 8 : 4;
  L.J = pb->img.nx * pb->img.ny;
  L.n2 = pb->img.nsub * pb->img.nsub;
  L.I_max = max_ns * max_ns;
  L.n_wg = n_wg;
  L.qcap = ((M + 7) / 8) * NL;
  const TapIdx ti(pb->k);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  L.consts = take(sizeof(Consts));
  L.lam = take(sizeof(double) * SL_MAX_LAMBDA);
  L.taps_d = take(sizeof(double) * ti.total);
  L.taps_f = take(sz * ti.total);
  L.minfo = take(sizeof(MemberInfo) * M);
  L.queues = take(sizeof(int) * 8 * (size_t)L.qcap);
  L.pqueues = take(sizeof(int) * 8 * (size_t)L.qcap);
  L.slot_cap = L.J + 64;
  L.pix = take(sizeof(int32_t) * (size_t)M * L.slot_cap);
  L.cell = take(sizeof(int32_t) * (size_t)M * L.slot_cap * L.n2);
  L.fx = take(sz * (size_t)M * L.slot_cap * L.n2);
  L.fy = take(sz * (size_t)M * L.slot_cap * L.n2);
  L.pmask = take(mask_bytes(L.n2) * (size_t)M * L.slot_cap);
  L.btd = take(sizeof(double) * 2 * (size_t)L.J);
  L.pcpart = take(2 * sizeof(double) * (size_t)M * rhs_grid(L.I_max, M));
  L.b = take(sizeof(double) * (size_t)M * L.I_max);
  L.bh = take(sizeof(double) * (size_t)M * L.I_max);   // A^T bhat (Monte Carlo degrees of freedom)
  L.dofk = take(sizeof(double) * (size_t)M * NL);      // per-iterate estimate of the implicit solve
  L.s_all = take(sz * (size_t)M * NL * L.I_max);
  L.gframe_elems = (pb->img.ny + 4 * 16 + kSegR) * ((pb->img.nx + 4 * 16) | 1);   // widest window's halo
  L.gframe = take(sz * (size_t)n_wg * L.gframe_elems);
  L.gz = take(sz * 4 * (size_t)n_wg * L.J);          // [plain | preconditioned launch][slot]: z, B^T z
  L.rbuf = take(sz * 2 * (size_t)n_wg * L.I_max);
  L.mcbuf = take(sz * 5 * (size_t)n_wg * L.I_max);
  L.ibuf = take(sz * (size_t)n_wg * L.J);   // image residual of the implicit-regularisation solve
  L.lt_ptr = take(sizeof(int32_t) * (size_t)M * (L.I_max + 65));
  L.lt_perm = take(sizeof(int32_t) * (size_t)M * L.I_max);
  L.lt_base = take(sizeof(int32_t) * (size_t)M * L.I_max);
  L.lt_cnt = take(sizeof(int32_t) * (size_t)M * L.I_max);
  // twice the unpadded bound (4 or, bicubic, 16 nodes per subpixel): room for slice padding
  L.lt_cap = (pb->interp == SL_INTERP_BICUBIC ? 32LL : 8LL) * L.n2 * L.slot_cap;
  L.lt_ent = take((sz == 8 ? 16 : 8) * (size_t)M * (size_t)L.lt_cap);
  L.total = off;
  return L;
}

static int check_problem(const sl_problem* pb, int max_ns, int M, int NL) {
  SL_REQUIRE(pb != nullptr, "problem is NULL");
  const sl_image_grid& g = pb->img;
  SL_REQUIRE(g.nx >= 1 && g.ny >= 1 && g.nx <= 256 && g.ny <= 256,
             "batched solve supports images up to 256 x 256 (got %d x %d)", g.nx, g.ny);
  SL_REQUIRE(std::isfinite(g.pix) && g.pix > 0.0, "pixel size must be positive");
  SL_REQUIRE(g.nsub >= 1 && g.nsub <= SL_MAX_NSUB, "nsub %d outside [1, %d]", g.nsub, SL_MAX_NSUB);
  SL_REQUIRE(pb->k >= 1 && pb->k <= SL_MAX_PSF && (pb->k & 1), "PSF side %d must be odd, <= %d", pb->k,
             SL_MAX_PSF);
  SL_REQUIRE(std::isfinite(pb->sigma) && pb->sigma > 0.0, "sigma must be positive");
  SL_REQUIRE(std::isfinite(pb->half_width) && pb->half_width > 0.0, "half_width must be positive");
  SL_REQUIRE(pb->reg == SL_H_IDENTITY || pb->reg == SL_H_CURVATURE, "unknown reg %d", pb->reg);
  SL_REQUIRE(pb->dtype == SL_F32 || pb->dtype == SL_F64, "unknown dtype %d", pb->dtype);
  SL_REQUIRE(pb->psf_general == 0 || pb->psf_general == 1, "psf_general must be 0 or 1");
  SL_REQUIRE(pb->interp == SL_INTERP_BILINEAR || pb->interp == SL_INTERP_NEAREST || pb->interp == SL_INTERP_BICUBIC,
             "unknown interp %d", pb->interp);
  SL_REQUIRE(max_ns >= 2 && max_ns <= 128, "max_ns %d outside [2, 128]", max_ns);
  SL_REQUIRE(M >= 1 && M <= (1 << 20), "n_members %d out of range", M);
  SL_REQUIRE(NL >= 1 && NL <= SL_MAX_LAMBDA, "n_lambda %d outside [1, %d]", NL, SL_MAX_LAMBDA);
  SL_REQUIRE((long)M * NL < (1L << 30), "too many (member, lambda) items");
  return SL_OK;
}

using SolveKernel = void (*)(SolveArgs);

// Kernel variants: bulk type T and banded half-width CKT (>= ck of the PSF).
// Compiled banded-window sizes (CKT >= ck).  `wide` takes the next size up;
// nullptr when that variant does not exist.
// pc selects the preconditioned kernel of the same window size.
template <bool DIR>
static SolveKernel pick_kernel_f(int ck, bool wide, int* ckt, bool pc = false) {
  static const int sizes[] = {2, 4, 7, 10, 16};
  static const SolveKernel ks[] = {k_solve<float, 2, false, DIR>, k_solve<float, 4, false, DIR>,
                                   k_solve<float, 7, false, DIR>, k_solve<float, 10, false, DIR>,
                                   k_solve<float, 16, false, DIR>};
  static const SolveKernel kp[] = {k_solve<float, 2, true, DIR>, k_solve<float, 4, true, DIR>,
                                   k_solve<float, 7, true, DIR>, k_solve<float, 10, true, DIR>,
                                   k_solve<float, 16, true, DIR>};
  const SolveKernel* k = pc ? kp : ks;
  int i = 0;
  while (i < 5 && sizes[i] < ck) ++i;
  if (i == 5) {   // wider PSFs: direct path only
    *ckt = 2;
    return wide ? nullptr : k[0];
  }
  if (wide && ++i == 5) return nullptr;
  *ckt = sizes[i];
  return k[i];
}

// The Monte Carlo degrees-of-freedom kernel of the same bulk type and window as the solve.
template <typename T, bool DIR>
static SolveKernel pick_mc_kernel(int ckt) {
  if (sizeof(T) == 4) {
    switch (ckt) {
      case 2: return k_mcdof<float, 2, DIR>;
      case 4: return k_mcdof<float, 4, DIR>;
      case 7: return k_mcdof<float, 7, DIR>;
      case 10: return k_mcdof<float, 10, DIR>;
      case 16: return k_mcdof<float, 16, DIR>;
    }
  } else {
    switch (ckt) {
      case 2: return k_mcdof<double, 2, DIR>;
      case 7: return k_mcdof<double, 7, DIR>;
      case 10: return k_mcdof<double, 10, DIR>;
    }
  }
  return nullptr;
}

// The implicit-regularisation kernel of the same bulk type and window as the solve.
template <typename T>
static SolveKernel pick_implicit_kernel(int ckt) {
  if (sizeof(T) == 4) {
    switch (ckt) {
      case 2: return k_implicit<float, 2>;
      case 4: return k_implicit<float, 4>;
      case 7: return k_implicit<float, 7>;
      case 10: return k_implicit<float, 10>;
      case 16: return k_implicit<float, 16>;
    }
  } else {
    switch (ckt) {
      case 2: return k_implicit<double, 2>;
      case 7: return k_implicit<double, 7>;
      case 10: return k_implicit<double, 10>;
    }
  }
  return nullptr;
}

template <bool DIR>
static SolveKernel pick_kernel_d(int ck, bool wide, int* ckt) {
  static const int sizes[] = {2, 7, 10};
  static const SolveKernel ks[] = {k_solve<double, 2, false, DIR>, k_solve<double, 7, false, DIR>,
                                   k_solve<double, 10, false, DIR>};
  int i = 0;
  while (i < 3 && sizes[i] < ck) ++i;
  if (i == 3) {
    *ckt = 2;
    return wide ? nullptr : ks[0];
  }
  if (wide && ++i == 3) return nullptr;
  *ckt = sizes[i];
  return ks[i];
}

// ------------------------------------------------------------------ profiling
struct ProfileState {
  std::mutex mu;
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
};
static ProfileState g_prof;

// Per-device side stream for the preconditioned launch and the events that
// fork it from, and join it to, the caller's stream; created on first use
// (default priority, non-blocking).
// Two side streams: the banded and the direct form of the preconditioned
// launch go on separate streams, so that the form that returns at entry
// never holds the other back while its blocks wait for CUs.
struct SideStream {
  hipStream_t s = nullptr, s2 = nullptr;
  hipEvent_t fork = nullptr, join = nullptr, join2 = nullptr;
};
static std::mutex g_side_mu;
static SideStream g_side[64];

static int side_stream(SideStream** out) {
  int dev = 0;
  SL_HIP(hipGetDevice(&dev));
  SL_REQUIRE(dev >= 0 && dev < 64, "device index %d out of range", dev);
  SideStream& x = g_side[dev];
  if (!x.s) {
    SL_HIP(hipStreamCreateWithFlags(&x.s, hipStreamNonBlocking));
    SL_HIP(hipStreamCreateWithFlags(&x.s2, hipStreamNonBlocking));
    SL_HIP(hipEventCreateWithFlags(&x.fork, hipEventDisableTiming));
    SL_HIP(hipEventCreateWithFlags(&x.join, hipEventDisableTiming));
    SL_HIP(hipEventCreateWithFlags(&x.join2, hipEventDisableTiming));
  }
  *out = &x;
  return SL_OK;
}

// Each solve kernel comes as a pair: the banded-blur form and the direct
// form (suffix d); both are launched and the one that does not match the
// problem returns at entry.
struct LaunchCfg {
  SolveKernel kim = nullptr;   // implicit-regularisation solve (replaces k_split / k_solve)
  SolveKernel ks = nullptr, ksd = nullptr;
  SolveKernel kpc = nullptr, kpcd = nullptr;   // preconditioned kernels, when some items may take them
  SolveKernel kmc = nullptr, kmcd = nullptr;   // Monte Carlo degrees-of-freedom pass, when requested
  size_t lds = 0, layout_lds = 0, fill_lds = 0, corner_lds = 0;
};

// Chooses the CG kernel of variant v and its LDS budget and sets the
// kernels' LDS attributes (host-side, outside any stream capture).
template <typename T>
static int configure(SolveArgs& A, const Layout& L, const sl_tuning& v, LaunchCfg* c) {
  const size_t sz = sizeof(T);
  int ckt = 2;
  SolveKernel ks = sizeof(T) == 4 ? pick_kernel_f<false>(A.ck, v.wide_window != 0, &ckt)
                                  : pick_kernel_d<false>(A.ck, v.wide_window != 0, &ckt);
  int ckt_d = 2;
  SolveKernel ksd = sizeof(T) == 4 ? pick_kernel_f<true>(A.ck, v.wide_window != 0, &ckt_d)
                                   : pick_kernel_d<true>(A.ck, v.wide_window != 0, &ckt_d);
  if (!ks) {
    set_error("kernel variant does not exist for this PSF size and dtype");
    return SL_ENOIMPL;
  }
  A.ckt = ckt;
  A.force_csr = v.lt_csr != 0;
  A.force_direct = v.blur_direct != 0 || A.psf_general != 0 || A.interp == SL_INTERP_BICUBIC;
  A.plain_cg = v.plain_cg != 0;
  A.pc_theta = (v.pc_theta_pct > 0 ? v.pc_theta_pct : kPcThetaPct) * 0.01f;
  A.heavy = v.heavy > 0 ? v.heavy : kHeavy;
  // dynamic LDS: source vector | reduction scratch | frame (up to the full image)
  A.q_off = (int)align256(sz * L.I_max);
  A.red_off = A.q_off + (int)align256(sz * L.I_max);
  A.pc_off = A.red_off + 64 * (int)sizeof(double);
  // sine table 2 (max_ns + 1) and eigenvalues max_ns of the spectral preconditioner
  A.frame_off = A.pc_off + (int)align256(sizeof(float) * (3 * A.max_ns + 8));
  const size_t fixed = (size_t)A.frame_off;
  size_t lds = fixed + sz * (size_t)frame_size(A.ny, A.nx, ckt);
  const size_t lds_max = 160 * 1024 - 1024;
  if (lds > lds_max) lds = lds_max;
  SL_REQUIRE(lds > fixed + 64 * sz, "source grid too large for LDS");
  A.lds_frame_cap = (int)((lds - fixed) / sz);
  A.lds_bytes = (int)lds;
  // the candidate-source kernel's one member has no launch to hold up: its own frame decides
  A.frames_fit = A.one_vector;
  if (sizeof(T) == 8 && !A.one_vector)
    A.frames_fit = lds_plan<T>(A, L.I_max, lds_mem<T>(ckt)).frame + frame_size(A.ny, A.nx, ckt) * (long)sz <= (long)lds;
  c->ks = ks;
  c->ksd = ksd;
  if (sizeof(T) == 4 && A.reg == SL_H_CURVATURE && !A.plain_cg && !A.implicit) {
    int ckt2 = 0;
    c->kpc = pick_kernel_f<false>(A.ck, v.wide_window != 0, &ckt2, true);
    c->kpcd = pick_kernel_f<true>(A.ck, v.wide_window != 0, &ckt2, true);
  }
  c->lds = lds;
  if (A.implicit) {
    c->kim = pick_implicit_kernel<T>(ckt);
    c->kpc = c->kpcd = nullptr;
    if (!c->kim) {
      set_error("no implicit-regularisation kernel for window %d", ckt);
      return SL_ENOIMPL;
    }
  }
  if (A.mcn && !A.implicit) {   // the implicit solve runs its own lockstep system
    c->kmc = pick_mc_kernel<T, false>(ckt);
    c->kmcd = pick_mc_kernel<T, true>(ckt);
    if (!c->kmc || !c->kmcd) {
      set_error("no Monte Carlo degrees-of-freedom kernel for window %d", ckt);
      return SL_ENOIMPL;
    }
  }
  c->layout_lds = sizeof(int) * (2 * (size_t)L.I_max + 64 + 16 * 128 + (L.I_max + 63) / 64);
  c->fill_lds = sizeof(int) * (kFillW + 1) * (size_t)std::min(kFillBand, L.I_max);
  // lcurve_corner_block: 12 n + 2 n^2 doubles (both spline systems at once)
  c->corner_lds = sizeof(double) * (2 * A.n_lambda * A.n_lambda + 12 * A.n_lambda + 16);
  static std::mutex mu;
  std::lock_guard<std::mutex> g(mu);
  for (SolveKernel k : {c->ks, c->ksd, c->kpc, c->kpcd, c->kmc, c->kmcd})
    if (k) SL_HIP(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  if (c->kim)
    SL_HIP(hipFuncSetAttribute((const void*)c->kim, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  SL_HIP(hipFuncSetAttribute((const void*)k_prep_layout<T>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)c->layout_lds));
  SL_HIP(hipFuncSetAttribute((const void*)k_prep_fill<T>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)c->fill_lds));
  // up to 72 KB at SL_MAX_LAMBDA points
  SL_HIP(hipFuncSetAttribute((const void*)k_corner<T>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)c->corner_lds));
  return SL_OK;
}

// Launches the banded and the direct form of a persistent kernel on st, the
// banded one first; the one that does not match the problem (the separability
// flag k_setup leaves in the workspace) returns at entry.
// With force_direct the device's separability flag is 0 and the banded form
// would return at entry, so only the direct form is launched.
template <typename T>
static int launch_pair(SolveKernel kb, SolveKernel kd, const Layout& L, const LaunchCfg& c, hipStream_t st,
                       const SolveArgs& A, const char* what) {
  if (!A.force_direct) {
    hipLaunchKernelGGL(kb, dim3(L.n_wg), dim3(kNTof<T>), c.lds, st, A);
    if (int e = check_launch(what)) return e;
  }
  hipLaunchKernelGGL(kd, dim3(L.n_wg), dim3(kNTof<T>), c.lds, st, A);
  return check_launch(what);
}

// Enqueues the member set-up: the trace tables and, with `adjoint`, L^T and the
// right-hand sides (the candidate-source chi^2 needs neither).
template <typename T>
static int enqueue_prep(const SolveArgs& A, const LaunchCfg& c, hipStream_t st, bool adjoint) {
  const unsigned tiles = (unsigned)((A.nx * A.ny + kPrepT - 1) / kPrepT), M = (unsigned)A.n_members;
  const unsigned images = adjoint ? (A.mcn ? 2u : 1u) : 0u;   // B^T d, B^T bhat
  hipLaunchKernelGGL(k_prep_trace<T>, dim3(tiles * (M + images)), dim3(kPrepT), 0, st, A);
  if (int e = check_launch("k_prep_trace")) return e;
  hipLaunchKernelGGL(k_prep_place<T>, dim3(tiles * M), dim3(kPrepT), 0, st, A);
  if (int e = check_launch("k_prep_place")) return e;
  if (!adjoint) return SL_OK;
  hipLaunchKernelGGL(k_prep_layout<T>, dim3(M), dim3(1024), c.layout_lds, st, A);
  if (int e = check_launch("k_prep_layout")) return e;
  const int bands = (A.I_max + kFillBand - 1) / kFillBand;
  hipLaunchKernelGGL(k_prep_fill<T>, dim3(M * bands), dim3(64 * kFillW), c.fill_lds, st, A, bands);
  if (int e = check_launch("k_prep_fill")) return e;
  hipLaunchKernelGGL(k_prep_rhs<T>, dim3((M + 7) / 8 * 8 * (unsigned)A.rhs_blocks), dim3(kRhsT), 0, st, A);
  return check_launch("k_prep_rhs");
}

// Enqueues the launches of one solve on st: k_setup, k_prep_*, [k_split], the
// plain k_solve [beside the preconditioned k_solve on the side stream, joined
// back to st], k_corner.  `profile` records HIP events on st around the CG
// phase when profiling is on (never inside a capture).
// `priv` (nullable): a side stream and events owned by the caller (a graph
// capture uses its own, so that no other thread's eager solve can fork onto
// a stream that is part of the capture); NULL takes the per-device one under
// its lock.
template <typename T>
static int enqueue(const SolveArgs& A, const LamList& lams, const Layout& L, const LaunchCfg& c, hipStream_t st,
                   bool profile, SideStream* priv = nullptr) {
  if (int e = setup_lds_attr<T>()) return e;
  hipLaunchKernelGGL(k_setup<T>, dim3(1), dim3(1024), kSetupLds, st, A, lams);
  if (int e = check_launch("k_setup")) return e;
  if (int e = enqueue_prep<T>(A, c, st, true)) return e;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (profile) {
    std::lock_guard<std::mutex> g(g_prof.mu);
    if (g_prof.on) {
      SL_HIP(hipEventCreate(&e0));
      SL_HIP(hipEventCreate(&e1));
      SL_HIP(hipEventRecord(e0, st));
    }
  }
  if (c.kim) {
    hipLaunchKernelGGL(c.kim, dim3(L.n_wg), dim3(kNTof<T>), c.lds, st, A);
    if (int e = check_launch("k_implicit")) return e;
  } else if (c.kpc) {
    hipLaunchKernelGGL(k_split<T>, dim3(1), dim3(512), 0, st, A);
    if (int e = check_launch("k_split")) return e;
    // The plain launch first on st, the preconditioned one on the side
    // stream: both are persistent, so its blocks take the CUs that the plain
    // launch's last long items leave idle.  They share no queue and no
    // per-block scratch.
    std::unique_lock<std::mutex> g(g_side_mu, std::defer_lock);
    SideStream* ss = priv;
    if (!ss) {
      g.lock();
      if (int e = side_stream(&ss)) return e;
    }
    SL_HIP(hipEventRecord(ss->fork, st));
    if (int e = launch_pair<T>(c.ks, c.ksd, L, c, st, A, "k_solve")) return e;
    SL_HIP(hipStreamWaitEvent(ss->s, ss->fork, 0));
    SL_HIP(hipStreamWaitEvent(ss->s2, ss->fork, 0));
    if (!A.force_direct) {
      hipLaunchKernelGGL(c.kpc, dim3(L.n_wg), dim3(kNTof<T>), c.lds, ss->s, A);
      if (int e = check_launch("k_solve (preconditioned)")) return e;
    }
    hipLaunchKernelGGL(c.kpcd, dim3(L.n_wg), dim3(kNTof<T>), c.lds, ss->s2, A);
    if (int e = check_launch("k_solve (preconditioned, direct blur)")) return e;
    SL_HIP(hipEventRecord(ss->join, ss->s));
    SL_HIP(hipEventRecord(ss->join2, ss->s2));
    SL_HIP(hipStreamWaitEvent(st, ss->join, 0));
    SL_HIP(hipStreamWaitEvent(st, ss->join2, 0));
  } else {
    if (int e = launch_pair<T>(c.ks, c.ksd, L, c, st, A, "k_solve")) return e;
  }
  if (e1) {
    SL_HIP(hipEventRecord(e1, st));
    std::lock_guard<std::mutex> g(g_prof.mu);
    g_prof.ev.emplace_back(e0, e1);
  }
  hipLaunchKernelGGL(k_corner<T>, dim3(A.n_members), dim3(256), c.corner_lds, st, A);
  if (int e = check_launch("k_corner")) return e;
  if (c.kmc) return launch_pair<T>(c.kmc, c.kmcd, L, c, st, A, "k_mcdof");
  return SL_OK;
}

static int configure_any(int dtype, SolveArgs& A, const Layout& L, const sl_tuning& v, LaunchCfg* c) {
  return dtype == SL_F32 ? configure<float>(A, L, v, c) : configure<double>(A, L, v, c);
}

static int enqueue_any(int dtype, const SolveArgs& A, const LamList& lams, const Layout& L, const LaunchCfg& c,
                       hipStream_t st, bool profile, SideStream* priv = nullptr) {
  return dtype == SL_F32 ? enqueue<float>(A, lams, L, c, st, profile, priv)
                         : enqueue<double>(A, lams, L, c, st, profile, priv);
}

// ------------------------------------------------------------------ autotuner table
using TuneKey = std::array<int, 9>;

static TuneKey tune_key(const sl_problem* pb, int max_ns, int n_members, int n_lambda) {
  return {pb->dtype, pb->img.nx, pb->img.ny, pb->img.nsub, pb->k, pb->reg, max_ns, n_members, n_lambda};
}

struct TuneTable {
  std::mutex mu;
  std::map<TuneKey, sl_tuning> best;
};
static TuneTable g_tune;

static sl_tuning resolve_tuning(const sl_problem* pb, int max_ns, int n_members, int n_lambda,
                                const sl_solve_opts* opt) {
  if (opt->tuning) return *opt->tuning;
  std::lock_guard<std::mutex> g(g_tune.mu);
  auto it = g_tune.best.find(tune_key(pb, max_ns, n_members, n_lambda));
  return it == g_tune.best.end() ? sl_tuning{0, 0, 0, 0, 0, 0} : it->second;
}

// The autotuner's search, in three stages.  Variants 0..7: the structural
// switches (window, L^T layout, blur form) at the default threshold and
// queue order.  8..11: the preconditioner threshold theta (percent of c) on
// the best of 0..7.  12..15: the count of smallest lambdas queued first on
// the best of 0..11.
static const int kThetaPct[4] = {5, 10, 25, 40};
static const int kHeavyN[4] = {2, 3, 6, 8};
static sl_tuning variant_of(int i, const sl_tuning& base) {
  if (i < 8) return sl_tuning{i & 1, (i >> 1) & 1, (i >> 2) & 1, 0, 0, 0};
  sl_tuning v = base;
  if (i < 12)
    v.pc_theta_pct = kThetaPct[i - 8];
  else
    v.heavy = kHeavyN[i - 12];
  return v;
}

// Validates the arguments of a solve and fills the kernel arguments.
static int prepare(const sl_problem* pb, const double* lens, const int32_t* ns, int max_ns, int n_members,
                   const double* lambdas, int n_lambda, const sl_solve_opts* opt, void* workspace,
                   size_t workspace_bytes, const sl_result* out, SolveArgs* Ap, Layout* Lp, LamList* lams) {
  if (int e = check_problem(pb, max_ns, n_members, n_lambda)) return e;
  SL_REQUIRE(lens && ns && pb->d && pb->psf, "NULL device input");
  SL_REQUIRE(lambdas != nullptr, "lambdas is NULL");
  for (int k = 0; k < n_lambda; ++k) {
    SL_REQUIRE(std::isfinite(lambdas[k]) && lambdas[k] > 0.0, "lambda[%d] must be positive", k);
    SL_REQUIRE(k == 0 || lambdas[k] > lambdas[k - 1], "lambdas must be strictly ascending");
  }
  SL_REQUIRE(opt != nullptr, "opts is NULL");
  SL_REQUIRE(std::isfinite(opt->tol) && opt->tol >= 0.0, "tol must be >= 0");
  SL_REQUIRE(opt->maxit >= 1, "maxit must be >= 1");
  SL_REQUIRE(out && out->s_corner && out->s_off && out->chi2 && out->reg && out->iters && out->status &&
                 out->k_star && out->corner_status,
             "NULL result pointer");
  SL_REQUIRE(!opt->mc_noise || out->dof, "mc_noise given but the result has no dof array");
  SL_REQUIRE(workspace != nullptr && ((uintptr_t)workspace & 255) == 0,
             "workspace must be non-NULL and 256-byte aligned");
  const Layout L = make_layout(pb, max_ns, n_members, n_lambda, device_cus());
  SL_REQUIRE(workspace_bytes >= L.total, "workspace too small: %zu < %zu bytes", workspace_bytes, L.total);
  SolveArgs A{};
  A.nx = pb->img.nx;
  A.ny = pb->img.ny;
  A.nsub = pb->img.nsub;
  A.n2 = L.n2;
  A.K = pb->k;
  A.ck = (pb->k - 1) / 2;
  A.reg = pb->reg;
  A.psf_general = pb->psf_general != 0;
  A.interp = pb->interp;
  A.n_members = n_members;
  A.n_lambda = n_lambda;
  A.max_ns = max_ns;
  A.maxit = opt->maxit;
  A.pix = pb->img.pix;
  A.R = pb->half_width;
  A.sigma = pb->sigma;
  A.tol = opt->tol;
  A.lens = lens;
  A.ns = ns;
  A.d = pb->d;
  A.psf = pb->psf;
  A.s_corner = out->s_corner;
  A.s_off = out->s_off;
  A.chi2 = out->chi2;
  A.regv = out->reg;
  A.iters = out->iters;
  A.status = out->status;
  A.k_star = out->k_star;
  A.corner_status = out->corner_status;
  unsigned char* ws = (unsigned char*)workspace;
  A.consts = (Consts*)(ws + L.consts);
  A.lamv = (double*)(ws + L.lam);
  A.taps_d = (double*)(ws + L.taps_d);
  A.taps_t = ws + L.taps_f;
  A.minfo = (MemberInfo*)(ws + L.minfo);
  A.queues = (int*)(ws + L.queues);
  A.pqueues = (int*)(ws + L.pqueues);
  A.qcap = L.qcap;
  A.pix_list = (int32_t*)(ws + L.pix);
  A.cell = (int32_t*)(ws + L.cell);
  A.fx = ws + L.fx;
  A.fy = ws + L.fy;
  A.b = (double*)(ws + L.b);
  A.bh = (double*)(ws + L.bh);
  A.dofk = (double*)(ws + L.dofk);
  A.pmask = ws + L.pmask;
  A.btd = (double*)(ws + L.btd);
  A.pcpart = (double*)(ws + L.pcpart);
  A.rhs_blocks = rhs_grid(L.I_max, n_members);
  A.lt_base = (int32_t*)(ws + L.lt_base);
  A.lt_cnt = (int32_t*)(ws + L.lt_cnt);
  A.mcbuf = ws + L.mcbuf;
  A.ibuf = ws + L.ibuf;
  A.mcn = opt->mc_noise;
  A.dofv = opt->mc_noise ? out->dof : nullptr;
  A.s_all = ws + L.s_all;
  A.gframe = ws + L.gframe;
  A.gframe_elems = L.gframe_elems;
  A.slot_cap = L.slot_cap;
  A.gz = ws + L.gz;
  A.rbuf = ws + L.rbuf;
  A.lt_ptr = (int32_t*)(ws + L.lt_ptr);
  A.lt_perm = (int32_t*)(ws + L.lt_perm);
  A.lt_ent = ws + L.lt_ent;
  A.lt_cap = L.lt_cap;
  A.I_max = L.I_max;
  *lams = LamList{};
  for (int k = 0; k < n_lambda; ++k) lams->v[k] = lambdas[k];
  *Ap = A;
  *Lp = L;
  return SL_OK;
}

}  // namespace sl

using namespace sl;

extern "C" {

int sl_solve_semilinear(const sl_problem* pb, const double* lens, const int32_t* ns, int max_ns,
                        int n_members, const double* lambdas, int n_lambda, const sl_solve_opts* opt,
                        void* workspace, size_t workspace_bytes, sl_result* out, void* stream) {
  SolveArgs A;
  Layout L;
  LamList lams;
  if (int e = prepare(pb, lens, ns, max_ns, n_members, lambdas, n_lambda, opt, workspace, workspace_bytes, out, &A,
                      &L, &lams))
    return e;
  LaunchCfg c;
  if (int e = configure_any(pb->dtype, A, L, resolve_tuning(pb, max_ns, n_members, n_lambda, opt), &c)) return e;
  return enqueue_any(pb->dtype, A, lams, L, c, (hipStream_t)stream, true);
}

int sl_solve_implicit(const sl_problem* pb, const double* lens, const int32_t* ns, int max_ns, int n_members,
                      int n_iter, const sl_solve_opts* opt, void* workspace, size_t workspace_bytes, sl_result* out,
                      void* stream) {
  SL_REQUIRE(n_iter >= 4 && n_iter <= SL_MAX_LAMBDA, "n_iter %d outside [4, %d]", n_iter, SL_MAX_LAMBDA);
  SL_REQUIRE(opt != nullptr, "opts is NULL");
  SL_REQUIRE(opt->mc_noise == nullptr || pb->dtype == SL_F64,
             "mc_noise with the implicit-regularisation solve needs FP64: its lockstep system amplifies FP32 "
             "rounding of the step lengths past the first few iterations");
  double idx[SL_MAX_LAMBDA];   // placeholders for the argument checks: one slot per iterate
  for (int k = 0; k < n_iter; ++k) idx[k] = k + 1.0;
  SolveArgs A;
  Layout L;
  LamList lams;
  if (int e = prepare(pb, lens, ns, max_ns, n_members, idx, n_iter, opt, workspace, workspace_bytes, out, &A, &L,
                      &lams))
    return e;
  A.implicit = 1;
  LaunchCfg c;
  const sl_tuning dflt{0, 0, opt->tuning ? opt->tuning->blur_direct : 0, 1, 0, 0};
  if (int e = configure_any(pb->dtype, A, L, dflt, &c)) return e;
  return enqueue_any(pb->dtype, A, lams, L, c, (hipStream_t)stream, true);
}

size_t sl_chi2_sources_workspace_size(const sl_problem* pb, int ns) {
  const size_t n = sl_solve_workspace_size(pb, ns, 1, 1);
  return n ? align256(n) + kSrcTail : 0;
}

int sl_chi2_sources(const sl_problem* pb, const double* lens, int ns, const double* sources, int n_sources,
                    void* workspace, size_t workspace_bytes, double* chi2, void* stream) {
  SL_REQUIRE(pb != nullptr, "problem is NULL");
  SL_REQUIRE(ns >= 2 && ns <= 128, "ns %d outside [2, 128]", ns);
  SL_REQUIRE(n_sources >= 1 && n_sources <= (1 << 24), "n_sources %d out of range", n_sources);
  SL_REQUIRE(lens && sources && chi2, "NULL device pointer");
  const size_t base = sl_solve_workspace_size(pb, ns, 1, 1);
  SL_REQUIRE(base != 0, "%s", sl_last_error());
  SL_REQUIRE(workspace_bytes >= align256(base) + kSrcTail, "workspace too small: %zu < %zu bytes", workspace_bytes,
             align256(base) + kSrcTail);
  // the tail holds the device copy of ns and the member offsets k_setup writes
  unsigned char* tail = static_cast<unsigned char*>(workspace) + align256(base);
  int32_t* ns_dev = reinterpret_cast<int32_t*>(tail);
  sl_result dummy{};
  dummy.s_off = reinterpret_cast<int64_t*>(tail + 256);
  dummy.s_corner = reinterpret_cast<double*>(tail + 256);
  dummy.chi2 = dummy.reg = dummy.s_corner;
  dummy.iters = dummy.status = dummy.k_star = dummy.corner_status = ns_dev;
  const double lam1 = 1.0;
  const sl_solve_opts opt{0.0, 1, nullptr, nullptr};
  SolveArgs A;
  Layout L;
  LamList lams;
  if (int e = prepare(pb, lens, ns_dev, ns, 1, &lam1, 1, &opt, workspace, base, &dummy, &A, &L, &lams)) return e;
  A.one_vector = 1;
  LaunchCfg c;
  const sl_tuning dflt{0, 0, 0, 1, 0, 0};
  if (int e = configure_any(pb->dtype, A, L, dflt, &c)) return e;
  hipStream_t st = (hipStream_t)stream;
  const int nb = std::min(L.n_wg, n_sources);
  const int nt = pb->dtype == SL_F32 ? kNTof<float> : kNTof<double>;
  const Chi2Kernel kc = pb->dtype == SL_F32 ? pick_chi2_kernel<float>(A.ckt) : pick_chi2_kernel<double>(A.ckt);
  if (!kc) {
    set_error("no candidate-source chi^2 kernel for window %d", A.ckt);
    return SL_ENOIMPL;
  }
  {
    static std::mutex mu;
    std::lock_guard<std::mutex> g(mu);
    SL_HIP(hipFuncSetAttribute((const void*)kc, hipFuncAttributeMaxDynamicSharedMemorySize, (int)c.lds));
  }
  hipLaunchKernelGGL(k_put_int, dim3(1), dim3(64), 0, st, ns_dev, ns);
  if (int e = check_launch("k_put_int")) return e;
  if (pb->dtype == SL_F32) {
    if (int e = setup_lds_attr<float>()) return e;
    hipLaunchKernelGGL(k_setup<float>, dim3(1), dim3(1024), kSetupLds, st, A, lams);
    if (int e = check_launch("k_setup")) return e;
    if (int e = enqueue_prep<float>(A, c, st, false)) return e;
  } else {
    if (int e = setup_lds_attr<double>()) return e;
    hipLaunchKernelGGL(k_setup<double>, dim3(1), dim3(1024), kSetupLds, st, A, lams);
    if (int e = check_launch("k_setup")) return e;
    if (int e = enqueue_prep<double>(A, c, st, false)) return e;
  }
  hipLaunchKernelGGL(kc, dim3(nb), dim3(nt), c.lds, st, A, sources, n_sources, chi2);
  return check_launch("k_chi2_src");
}

int sl_solve_autotune(const sl_problem* pb, const double* lens, const int32_t* ns, int max_ns, int n_members,
                      const double* lambdas, int n_lambda, const sl_solve_opts* opt, void* workspace,
                      size_t workspace_bytes, sl_result* out, void* stream, sl_tuning* best, double* ms) {
  SolveArgs A0;
  Layout L;
  LamList lams;
  if (int e = prepare(pb, lens, ns, max_ns, n_members, lambdas, n_lambda, opt, workspace, workspace_bytes, out,
                      &A0, &L, &lams))
    return e;
  hipStream_t st = (hipStream_t)stream;
  hipEvent_t e0, e1;
  SL_HIP(hipEventCreate(&e0));
  SL_HIP(hipEventCreate(&e1));
  double t_best = 1e300;
  int i_best = -1, i_last = -1;
  sl_tuning v_best{0, 0, 0, 0, 0, 0}, base{0, 0, 0, 0, 0, 0};
  // the threshold matters only where the preconditioner can run
  const bool pc_possible = pb->dtype == SL_F32 && pb->reg == SL_H_CURVATURE;
  // SL_AUTOTUNE_VERBOSE=1: one line per variant on stderr as it is timed
  const char* ve = std::getenv("SL_AUTOTUNE_VERBOSE");
  const bool verbose = ve && ve[0] == '1';
  int rc = SL_OK;
  for (int i = 0; i < SL_N_VARIANTS && rc == SL_OK; ++i) {
    if (ms) ms[i] = -1.0;
    if (i == 8 || i == 12) base = v_best;   // the next stage starts from the best so far
    if (i >= 8 && i < 12 && !pc_possible) continue;
    const sl_tuning vi = variant_of(i, base);
    SolveArgs A = A0;
    LaunchCfg c;
    const int ce = configure_any(pb->dtype, A, L, vi, &c);
    if (ce == SL_ENOIMPL) continue;
    if ((rc = ce) != SL_OK) break;
    if ((rc = enqueue_any(pb->dtype, A, lams, L, c, st, false)) != SL_OK) break;   // untimed
    float t = 1e30f;
    for (int rep = 0; rep < 2 && rc == SL_OK; ++rep) {   // the faster of two timed runs
      float tr = 0.0f;
      if (hipEventRecord(e0, st) != hipSuccess) { rc = SL_EHIP; break; }
      if ((rc = enqueue_any(pb->dtype, A, lams, L, c, st, false)) != SL_OK) break;
      if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
          hipEventElapsedTime(&tr, e0, e1) != hipSuccess) {
        set_error("autotune timing failed: %s", hipGetErrorString(hipGetLastError()));
        rc = SL_EHIP;
        break;
      }
      t = std::min(t, tr);
    }
    if (rc != SL_OK) break;
    if (ms) ms[i] = t;
    if (verbose) {
      std::fprintf(stderr, "sl_solve_autotune: variant %d {%d %d %d theta %d%% heavy %d}: %.2f ms\n", i,
                   vi.wide_window, vi.lt_csr, vi.blur_direct, vi.pc_theta_pct ? vi.pc_theta_pct : kPcThetaPct,
                   vi.heavy ? vi.heavy : kHeavy, t);
      std::fflush(stderr);
    }
    i_last = i;
    if (t < t_best) {
      t_best = t;
      i_best = i;
      v_best = vi;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != SL_OK) return rc;
  SL_REQUIRE(i_best >= 0, "no kernel variant exists for this problem");
  const sl_tuning v = v_best;
  {
    std::lock_guard<std::mutex> g(g_tune.mu);
    g_tune.best[tune_key(pb, max_ns, n_members, n_lambda)] = v;
  }
  if (best) *best = v;
  if (i_best != i_last) {   // leave the best variant's results in `out`
    SolveArgs A = A0;
    LaunchCfg c;
    if (int e = configure_any(pb->dtype, A, L, v, &c)) return e;
    if (int e = enqueue_any(pb->dtype, A, lams, L, c, st, false)) return e;
  }
  return SL_OK;
}

}  // extern "C"

struct sl_plan {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

extern "C" {

int sl_plan_create(const sl_problem* pb, const double* lens, const int32_t* ns, int max_ns, int n_members,
                   const double* lambdas, int n_lambda, const sl_solve_opts* opt, void* workspace,
                   size_t workspace_bytes, const sl_result* out, sl_plan** plan) {
  SL_REQUIRE(plan != nullptr, "plan is NULL");
  *plan = nullptr;
  SolveArgs A;
  Layout L;
  LamList lams;
  if (int e = prepare(pb, lens, ns, max_ns, n_members, lambdas, n_lambda, opt, workspace, workspace_bytes, out, &A,
                      &L, &lams))
    return e;
  LaunchCfg c;
  if (int e = configure_any(pb->dtype, A, L, resolve_tuning(pb, max_ns, n_members, n_lambda, opt), &c)) return e;
  // The capture forks onto a side stream of its own, created before the
  // capture starts (default priority) and destroyed once it has ended.
  SideStream own;
  if (c.kpc) {
    SL_HIP(hipStreamCreateWithFlags(&own.s, hipStreamNonBlocking));
    SL_HIP(hipStreamCreateWithFlags(&own.s2, hipStreamNonBlocking));
    SL_HIP(hipEventCreateWithFlags(&own.fork, hipEventDisableTiming));
    SL_HIP(hipEventCreateWithFlags(&own.join, hipEventDisableTiming));
    SL_HIP(hipEventCreateWithFlags(&own.join2, hipEventDisableTiming));
  }
  auto drop_own = [&]() {
    if (own.s) (void)hipStreamDestroy(own.s);
    if (own.s2) (void)hipStreamDestroy(own.s2);
    if (own.fork) (void)hipEventDestroy(own.fork);
    if (own.join) (void)hipEventDestroy(own.join);
    if (own.join2) (void)hipEventDestroy(own.join2);
  };
  hipStream_t cs;
  if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) {
    drop_own();
    set_error("hipStreamCreateWithFlags failed");
    return SL_EHIP;
  }
  hipGraph_t g = nullptr;
  int rc = SL_OK;
  if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    set_error("hipStreamBeginCapture failed: %s", hipGetErrorString(hipGetLastError()));
    rc = SL_EHIP;
  } else {
    rc = enqueue_any(pb->dtype, A, lams, L, c, cs, false, c.kpc ? &own : nullptr);
    const hipError_t ee = hipStreamEndCapture(cs, &g);
    if (rc == SL_OK && ee != hipSuccess) {
      set_error("hipStreamEndCapture failed: %s", hipGetErrorString(ee));
      rc = SL_EHIP;
    }
  }
  (void)hipStreamDestroy(cs);
  drop_own();
  hipGraphExec_t ge = nullptr;
  if (rc == SL_OK) {
    const hipError_t ie = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
    if (ie != hipSuccess) {
      set_error("hipGraphInstantiate failed: %s", hipGetErrorString(ie));
      rc = SL_EHIP;
    }
  }
  if (rc != SL_OK) {
    if (g) (void)hipGraphDestroy(g);
    return rc;
  }
  sl_plan* p = new sl_plan;
  p->graph = g;
  p->exec = ge;
  *plan = p;
  return SL_OK;
}

int sl_plan_launch(sl_plan* plan, void* stream) {
  SL_REQUIRE(plan && plan->exec, "invalid plan");
  SL_HIP(hipGraphLaunch(plan->exec, (hipStream_t)stream));
  return SL_OK;
}

int sl_plan_destroy(sl_plan* plan) {
  if (!plan) return SL_OK;
  hipError_t e1 = plan->exec ? hipGraphExecDestroy(plan->exec) : hipSuccess;
  hipError_t e2 = plan->graph ? hipGraphDestroy(plan->graph) : hipSuccess;
  delete plan;
  if (e1 != hipSuccess || e2 != hipSuccess) {
    set_error("graph destroy failed");
    return SL_EHIP;
  }
  return SL_OK;
}

size_t sl_solve_workspace_size(const sl_problem* pb, int max_ns, int n_members, int n_lambda) {
  if (check_problem(pb, max_ns, n_members, n_lambda) != SL_OK) return 0;
  return make_layout(pb, max_ns, n_members, n_lambda, device_cus()).total;
}


int sl_solve_member_info(const sl_problem* pb, int max_ns, int n_members, int n_lambda, const void* workspace,
                         int32_t* info_host) {
  if (int e = check_problem(pb, max_ns, n_members, n_lambda)) return e;
  SL_REQUIRE(workspace && info_host, "NULL pointer");
  const Layout L = make_layout(pb, max_ns, n_members, n_lambda, device_cus());
  std::vector<MemberInfo> mi(n_members);
  SL_HIP(hipDeviceSynchronize());
  SL_HIP(hipMemcpy(mi.data(), (const unsigned char*)workspace + L.minfo, sizeof(MemberInfo) * n_members,
                   hipMemcpyDeviceToHost));
  for (int m = 0; m < n_members; ++m) {
    int32_t* o = info_host + 10 * m;
    o[0] = mi[m].ns;
    o[1] = mi[m].I;
    o[2] = mi[m].Mtrue;
    o[3] = mi[m].r0;
    o[4] = mi[m].r1;
    o[5] = mi[m].c0;
    o[6] = mi[m].c1;
    o[7] = mi[m].status;
    o[8] = mi[m].status == SL_ST_OK ? mi[m].sell : -1;
    o[9] = mi[m].status == SL_ST_OK ? mi[m].lds_frame != kMemGlobal : -1;
  }
  return SL_OK;
}

int sl_profile_enable(int on) {
  std::lock_guard<std::mutex> g(g_prof.mu);
  for (auto& p : g_prof.ev) {
    (void)hipEventDestroy(p.first);
    (void)hipEventDestroy(p.second);
  }
  g_prof.ev.clear();
  g_prof.on = on != 0;
  return SL_OK;
}

int sl_profile_solve_ms(double* ms_total, int32_t* launches) {
  SL_REQUIRE(ms_total && launches, "NULL pointer");
  std::lock_guard<std::mutex> g(g_prof.mu);
  double tot = 0.0;
  for (auto& p : g_prof.ev) {
    SL_HIP(hipEventSynchronize(p.second));
    float ms = 0.f;
    SL_HIP(hipEventElapsedTime(&ms, p.first, p.second));
    tot += ms;
  }
  *ms_total = tot;
  *launches = (int32_t)g_prof.ev.size();
  return SL_OK;
}

}  // extern "C"
