// Shared pieces of the fit and its adjoint: Gram + Hadamard GEMMs, the
// FP64 Cholesky / inverse of C C^H, device state.  Everything here has
// internal linkage (anonymous namespace) so that each translation unit gets
// its own copy of the kernels.
#pragma once
#include <float.h>
#include <limits.h>

#include "gemm_mod.h"
#include "gemm_split.h"
#include "splitk.h"

namespace isdf {
namespace {

constexpr int NB = 64;  // Cholesky block

struct FitState {
  int abort;    // nonzero: later launches of this call are no-ops
  int pivot;    // first failing pivot (INT_MAX: none)
  int bad_idx;  // first invalid idx position (INT_MAX: none)
  int pad;
  double pmin, pmax;
  double loss;
};

// ------------------------------------------------------------ idx checks
__global__ void check_idx(const int32_t* __restrict__ idx, int n_mu, int64_t nr, int* __restrict__ marker,
                          FitState* st) {
  int mu = blockIdx.x * blockDim.x + threadIdx.x;
  if (mu >= n_mu) return;
  int v = idx[mu];
  bool bad = v < 0 || v >= nr;
  if (!bad) bad = atomicAdd(&marker[v], 1) != 0;
  if (bad) {
    atomicMin(&st->bad_idx, mu);
    atomicOr(&st->abort, 1);
  }
}

// Threads of a launch share out `total` elements.
template <class F>
__device__ __forceinline__ void each_of(int64_t total, const F& f) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) f(e);
}

// E[n][k], n = 32 b + 16 c + t -> column nu = 16 b + t, part c (0: Re A, 1: Im A);
// k = 2 i + comp multiplies (re, im) of orbital i of the grid row.
// With Phi_mu[nu][i] = a + i b:  Re A = sum x a + y b,  Im A = sum y a - x b.
template <class TS, class T>
__device__ __forceinline__ void pack_gram_each(const TS* __restrict__ phi, int64_t ld, int n,
                                               const int32_t* __restrict__ idx, int n_mu, int64_t nr, int rows,
                                               T* __restrict__ E) {
  each_of((int64_t)rows * 2 * n, [&](int64_t e) {
    const int r = (int)(e / (2 * n));
    const int k = (int)(e % (2 * n));
    const int b = r >> 5, c = (r >> 4) & 1, t = r & 15;
    const int nu = b * 16 + t;
    double v = 0.0;
    if (nu < n_mu) {
      int64_t p = idx[nu];
      if (p < 0 || p >= nr) p = 0;  // invalid entries are reported by check_idx
      const int i = k >> 1, comp = k & 1;
      double2 z = Cplx<TS>::load(phi + 2 * (p * ld + i));
      if (c == 0) v = comp == 0 ? z.x : z.y;
      else v = comp == 0 ? -z.y : z.x;
    }
    E[e] = (T)v;
  });
}
template <class TS, class T>
__global__ void pack_gram_rhs(const TS* __restrict__ phi, int64_t ld, int n, const int32_t* __restrict__ idx,
                              int n_mu, int64_t nr, int rows, T* __restrict__ E) {
  pack_gram_each<TS, T>(phi, ld, n, idx, n_mu, nr, rows, E);
}

// F[n][k] (n = 2 i + c', k = 2 nu + c): real form of right-multiplication by
// Phi_mu, (x + iy)(a + ib) = (xa - yb) + i(xb + ya) with Phi_mu[nu][i] = a + ib.
template <class TS, class T>
__device__ __forceinline__ void pack_adj_each(const TS* __restrict__ phi, int64_t ld, int n,
                                              const int32_t* __restrict__ idx, int n_mu, int64_t nr, T* __restrict__ F) {
  each_of((int64_t)2 * n * 2 * n_mu, [&](int64_t e) {
    const int row = (int)(e / (2 * n_mu)), k = (int)(e % (2 * n_mu));
    const int i = row >> 1, cp = row & 1, nu = k >> 1, c = k & 1;
    int64_t p = idx[nu];
    if (p < 0 || p >= nr) p = 0;
    const double2 z = Cplx<TS>::load(phi + 2 * (p * ld + i));
    double v;
    if (cp == 0) v = c == 0 ? z.x : -z.y;
    else v = c == 0 ? z.y : z.x;
    F[e] = (T)v;
  });
}
template <class TS, class T>
__global__ void pack_adj_rhs(const TS* __restrict__ phi, int64_t ld, int n, const int32_t* __restrict__ idx,
                             int n_mu, int64_t nr, T* __restrict__ F) {
  pack_adj_each<TS, T>(phi, ld, n, idx, n_mu, nr, F);
}

// Everything a fit or its adjoint sets up from the inputs, in one launch (the
// small boxes are a chain of launches, each 5 us of the host's time and 2 of the
// GPU's; 24^3 fit 292 -> 284 us, loss and gradient 692 -> 656): the state, the occupancy marker and `zeros` cleared, and per orbital
// set the packed right-hand sides E, F and the real rows X[mu][k] =
// Phi_real[idx[mu]][k] (null: not wanted).
template <class TS, class T>
struct BeginSet {
  const TS* phi;
  int64_t ld;
  int n;
  T *E, *F, *X;
};
template <class TS, class T>
__global__ void fit_begin(FitState* st, int* __restrict__ marker, int64_t nr, const int32_t* __restrict__ idx, int n_mu,
                          int rows, BeginSet<TS, T> a, BeginSet<TS, T> b, double* __restrict__ zeros, int64_t nzeros) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->abort = 0;
    st->pivot = INT_MAX;
    st->bad_idx = INT_MAX;
    st->pad = 0;
    st->pmin = INFINITY;
    st->pmax = 0.0;
    st->loss = 0.0;
  }
  if (marker) each_of(nr, [&](int64_t e) { marker[e] = 0; });
  if (zeros) each_of(nzeros, [&](int64_t e) { zeros[e] = 0.0; });
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const BeginSet<TS, T>& w = s ? b : a;
    if (w.E) pack_gram_each<TS, T>(w.phi, w.ld, w.n, idx, n_mu, nr, rows, w.E);
    if (w.F) pack_adj_each<TS, T>(w.phi, w.ld, w.n, idx, n_mu, nr, w.F);
    if (w.X)
      each_of((int64_t)n_mu * 2 * w.n, [&](int64_t e) {
        const int mu = (int)(e / (2 * w.n)), k = (int)(e % (2 * w.n));
        int64_t p = idx[mu];
        if (p < 0 || p >= nr) p = 0;
        w.X[e] = (T)w.phi[2 * p * w.ld + k];
      });
  }
}
template <class TS, class T>
static bool begin(FitState* st, int* marker, int64_t nr, const int32_t* idx, int n_mu, int nmu16, BeginSet<TS, T> a,
                  BeginSet<TS, T> b, double* zeros, int64_t nzeros, hipStream_t s) {
  int64_t most = (int64_t)2 * nmu16 * 2 * (a.n > b.n ? a.n : b.n);
  if (marker && nr > most) most = nr;
  if (zeros && nzeros > most) most = nzeros;
  const int64_t blocks = ceil_div(most, 256) < 4096 ? ceil_div(most, 256) : 4096;
  hipLaunchKernelGGL((fit_begin<TS, T>), dim3((unsigned)blocks), dim3(256), 0, s, st, marker, nr, idx, n_mu, 2 * nmu16, a,
                     b, zeros, nzeros);
  return launch_ok();
}

// Gram + Hadamard epilogue.  Accumulator pairs (j, j+1) of a wavefront hold
// Re and Im of the same column nu.
enum { G_REAL = 0, G_CPLX = 1, G_EMB = 2 };
struct EpiGram {
  double* G;  // may be null (only A / B wanted)
  int64_t ldg;  // doubles
  int M;
  int n_mu;
  int mode;
  double* Aout;  // optional: A (and B) as interleaved complex rows, ld ldab doubles
  double* Bout;
  int64_t ldab;
  template <class Cfg, class Acc>
  __device__ __forceinline__ void apply(const Acc (&acc)[Cfg::MI][Cfg::NI], const TileAt& at) const {
    // Psi = Phi: G = |A|^2 (real)
#pragma unroll
    for (int i = 0; i < Cfg::MI; ++i)
#pragma unroll
      for (int jp = 0; jp < Cfg::NI / 2; ++jp) {
        const int nu = ((at.n_wave + 32 * jp) >> 5) * 16 + (at.lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = at.m_wave + i * 16 + Cfg::orow(at.lane, r);
          if (m < M && nu < n_mu) {
            const double re = (double)acc[i][2 * jp][r], im = (double)acc[i][2 * jp + 1][r];
            if (G) G[(int64_t)m * ldg + nu] = re * re + im * im;
            if (Aout) *reinterpret_cast<double2*>(Aout + (int64_t)m * ldab + 2 * nu) = make_double2(re, im);
          }
        }
      }
  }
  template <class Cfg, class Acc>
  __device__ __forceinline__ void apply2(const Acc (&a)[Cfg::MI][Cfg::NI], const Acc (&b)[Cfg::MI][Cfg::NI],
                                         const TileAt& at) const {
    // G = A .* conj(B)
#pragma unroll
    for (int i = 0; i < Cfg::MI; ++i)
#pragma unroll
      for (int jp = 0; jp < Cfg::NI / 2; ++jp) {
        const int nu = ((at.n_wave + 32 * jp) >> 5) * 16 + (at.lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = at.m_wave + i * 16 + Cfg::orow(at.lane, r);
          if (m < M && nu < n_mu) {
            const double ar = (double)a[i][2 * jp][r], ai = (double)a[i][2 * jp + 1][r];
            const double br = (double)b[i][2 * jp][r], bi = (double)b[i][2 * jp + 1][r];
            const double x = ar * br + ai * bi, y = ai * br - ar * bi;
            if (Aout) *reinterpret_cast<double2*>(Aout + (int64_t)m * ldab + 2 * nu) = make_double2(ar, ai);
            if (Bout) *reinterpret_cast<double2*>(Bout + (int64_t)m * ldab + 2 * nu) = make_double2(br, bi);
            if (!G) continue;
            if (mode == G_CPLX) {
              *reinterpret_cast<double2*>(G + (int64_t)m * ldg + 2 * nu) = make_double2(x, y);
            } else {
              *reinterpret_cast<double2*>(G + (int64_t)(2 * m) * ldg + 2 * nu) = make_double2(x, y);
              *reinterpret_cast<double2*>(G + (int64_t)(2 * m + 1) * ldg + 2 * nu) = make_double2(-y, x);
            }
          }
        }
      }
  }
};

// ------------------------------------------------------------ Cholesky
// Factors the kb x kb diagonal block at (k0, k0) of X in place (lower) and
// writes its inverse (lower) into the same block of Y.
//
// A serial chain of 64 pivots, so what counts is the latency of a step: the
// block is taken in four 64 x 16 panels, each factored by one wavefront with a
// row per lane in registers (row j of the panel reaches the other lanes
// through v_readlane, no barrier and no LDS in a step), and the columns to the
// right are updated on the FP64 matrix cores.  The inverse follows from the
// four 16 x 16 diagonal inverses (a column per lane) by doubling.  Blocks
// smaller than 64 are continued by the unit matrix.  80 us a block with one
// workgroup-wide barrier per pivot, 19 us this way (a panel 2.6, the loads 2.7).
__device__ __forceinline__ double read_lane(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

constexpr int POTRF_LD = NB + 1;

// acc (16 x 16) += s A B with A(m, k) at pa[m POTRF_LD + k] and B(k, n) at
// pb[k POTRF_LD + n] (TB: pb[n POTRF_LD + k]), K a multiple of 4.
template <bool TB>
__device__ __forceinline__ void potrf_mma(const double* pa, const double* pb, int K, double s, int lane, d4v& acc) {
  const int x = lane & 15, q = lane >> 4;
#pragma unroll 4
  for (int kk = 0; kk < K; kk += 4) {
    const int k = kk + q;
    MfmaT<double>::mma(s * pa[x * POTRF_LD + k], TB ? pb[x * POTRF_LD + k] : pb[k * POTRF_LD + x], acc);
  }
}
__device__ __forceinline__ void potrf_put(double* p, int lane, const d4v& acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) p[((lane >> 4) + 4 * r) * POTRF_LD + (lane & 15)] = acc[r];
}

// Folds the first n pivots of a block into the smallest and largest (one wave).
__device__ __forceinline__ void potrf_extremes(const double* pivots, int n, int lane, FitState* st) {
  double lo = lane < n ? pivots[lane] : INFINITY, hi = lane < n ? pivots[lane] : 0.0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o, ISDF_WAVE));
    hi = fmax(hi, __shfl_xor(hi, o, ISDF_WAVE));
  }
  if (lane == 0 && n > 0) {
    atomic_min_pos(&st->pmin, lo);
    atomic_max_pos(&st->pmax, hi);
  }
}

__global__ __launch_bounds__(256) void potrf_diag(double* __restrict__ X, int64_t ldx, int k0, int kb,
                                                  double* __restrict__ Y, int64_t ldy, FitState* st) {
  __shared__ double a[NB * POTRF_LD];
  __shared__ double x[NB * POTRF_LD];
  __shared__ double inv[NB], pivots[NB];  // 1 / l_jj, l_jj^2
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int abort = st->abort;
  if (tid == 0) bad = -1;
  {  // all loads in flight before the first LDS write
    double v[16];
    const int j = lane, jc = j < kb ? j : kb - 1;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int i = wv + 4 * e;
      v[e] = X[(int64_t)(k0 + (i < kb ? i : kb - 1)) * ldx + k0 + jc];
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int i = wv + 4 * e;
      x[i * POTRF_LD + j] = 0.0;
      if (j > i) continue;
      const double w = i < kb ? v[e] : (i == j ? 1.0 : 0.0);
      a[i * POTRF_LD + j] = w;
      a[j * POTRF_LD + i] = w;
    }
  }
  if (abort) return;  // (uniform)
  __syncthreads();
  for (int p = 0; p < NB / 16; ++p) {
    if (wv == 0) {
      const int c0 = 16 * p;
      double v[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) v[c] = lane >= c0 ? a[lane * POTRF_LD + c0 + c] : 0.0;
      // columns stay unscaled and each lane keeps its own row's pivot, so that
      // the chain from pivot to pivot is one reciprocal (the hardware's estimate
      // and two Newton steps: 1.0 / piv to the bit for each of 1e9 random pivots
      // between 2^-500 and 2^500) and two operations; the
      // panel's square roots are then taken together, a lane each
      double pv = 1.0;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double piv = read_lane(v[j], c0 + j);
        double y = __builtin_amdgcn_rcp(piv);
        // the pivot row, read while the reciprocal is on its way
        double row[16];
#pragma unroll
        for (int c = j + 1; c < 16; ++c) row[c] = read_lane(v[c], c0 + j);
        pv = lane == c0 + j ? piv : pv;
        __builtin_amdgcn_sched_barrier(0);
        y = fma(y, fma(-piv, y, 1.0), y);
        y = fma(y, fma(-piv, y, 1.0), y);
        const double u = v[j] * y;
#pragma unroll
        for (int c = j + 1; c < 16; ++c) v[c] = fma(-u, row[c], v[c]);
        __builtin_amdgcn_sched_barrier(0);
      }
      const unsigned long long wrong = __ballot(!(pv > 0.0) || !(pv < INFINITY));
      const double l = sqrt(pv), il = 1.0 / l;
#pragma unroll
      for (int c = 0; c < 16; ++c) v[c] = lane == c0 + c ? l : v[c] * read_lane(il, c0 + c);
      if (lane >= c0 && lane < c0 + 16) {
        inv[lane] = il;
        pivots[lane] = pv;
      }
      if (lane == 0 && wrong) bad = __ffsll((long long)wrong) - 1;
      if (lane >= c0) {
#pragma unroll
        for (int c = 0; c < 16; ++c) a[lane * POTRF_LD + c0 + c] = lane >= c0 + c ? v[c] : 0.0;
      }
    }
    __syncthreads();
    if (bad >= 0) {
      if (wv == 0) potrf_extremes(pivots, bad, lane, st);
      if (tid == 0) {
        atomicMin(&st->pivot, k0 + bad);
        atomicOr(&st->abort, 1);
      }
      return;
    }
    // tiles (ti, tj) right of the panel, p < tj <= ti
    int n = 0;
    for (int tj = p + 1; tj < NB / 16; ++tj)
      for (int ti = tj; ti < NB / 16; ++ti, ++n) {
        if ((n & 3) != wv) continue;
        double* c = a + 16 * ti * POTRF_LD + 16 * tj;
        d4v acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = c[((lane >> 4) + 4 * r) * POTRF_LD + (lane & 15)];
        potrf_mma<true>(a + 16 * ti * POTRF_LD + 16 * p, a + 16 * tj * POTRF_LD + 16 * p, 16, -1.0, lane, acc);
        potrf_put(c, lane, acc);
      }
    __syncthreads();
  }
  if (wv == 1) potrf_extremes(pivots, kb, lane, st);
  // 16 x 16 diagonal inverses: lane (block q, column c) solves L_q y = e_c
  if (wv == 0) {
    const int q = 16 * (lane >> 4), c = lane & 15;
    double y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) y[i] = i == c ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      y[k] *= inv[q + k];
#pragma unroll
      for (int i = k + 1; i < 16; ++i) y[i] = fma(-a[(q + i) * POTRF_LD + q + k], y[k], y[i]);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) x[(q + i) * POTRF_LD + q + c] = y[i];
  }
  __syncthreads();
  // doubling: the lower-left block of an inverse pair is -C^-1 (L21 A^-1); the
  // products L21 A^-1 go through the unused upper part of `a`
  d4v acc;
  if (wv < 2) {
    const int o = 32 * wv;
    acc = d4v{0, 0, 0, 0};
    potrf_mma<false>(a + (o + 16) * POTRF_LD + o, x + o * POTRF_LD + o, 16, 1.0, lane, acc);
    potrf_put(a + o * POTRF_LD + o + 16, lane, acc);
  }
  __syncthreads();
  if (wv < 2) {
    const int o = 32 * wv;
    acc = d4v{0, 0, 0, 0};
    potrf_mma<false>(x + (o + 16) * POTRF_LD + o + 16, a + o * POTRF_LD + o + 16, 16, -1.0, lane, acc);
    potrf_put(x + (o + 16) * POTRF_LD + o, lane, acc);
  }
  __syncthreads();
  const int tr = 16 * (wv >> 1), tc = 16 * (wv & 1);
  acc = d4v{0, 0, 0, 0};
  potrf_mma<false>(a + (32 + tr) * POTRF_LD, x + tc, 32, 1.0, lane, acc);
  potrf_put(a + tr * POTRF_LD + 32 + tc, lane, acc);
  __syncthreads();
  acc = d4v{0, 0, 0, 0};
  potrf_mma<false>(x + (32 + tr) * POTRF_LD + 32, a + 32 + tc, 32, -1.0, lane, acc);
  potrf_put(x + (32 + tr) * POTRF_LD + tc, lane, acc);
  __syncthreads();
  // (Y's upper triangle is zero already)
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int i = wv + 4 * e, j = lane;
    if (i >= kb || j > i) continue;
    X[(int64_t)(k0 + i) * ldx + k0 + j] = a[i * POTRF_LD + j];
    Y[(int64_t)(k0 + i) * ldy + k0 + j] = x[i * POTRF_LD + j];
  }
}

__global__ void fit_finish(const FitState* st, isdf_fit_info* info, double* loss_out, int backward) {
  int status = ISDF_OK;
  if (st->bad_idx != INT_MAX) status = ISDF_E_BAD_IDX;
  else if (st->pivot != INT_MAX) status = ISDF_E_NOT_PD;
  else if (st->abort) status = ISDF_E_NONFINITE;
  info->status = status;
  info->pivot = st->pivot == INT_MAX ? -1 : st->pivot;
  info->bad_idx = st->bad_idx == INT_MAX ? -1 : st->bad_idx;
  info->reserved = 0;
  info->pivot_min = st->pmin == INFINITY ? 0.0 : st->pmin;
  info->pivot_max = st->pmax;
  info->loss = st->loss;
  if (backward && loss_out) *loss_out = st->loss;
}

// ------------------------------------------------------------ launches
template <class T, int BM, int BN, int BK, int WM, int WN, class TA, int LA, class TB, int LB, int NOPS,
          int FOLD = 0, class Epi>
static bool launch_gemm(int M, int N, int64_t K, Operand<TA> A0, Operand<TB> B0, Operand<TA> A1,
                        Operand<TB> B1, int64_t K1, const Epi& epi, int lower_only, const int* abort,
                        hipStream_t st, int splits = 1, int batch = 1, int64_t sa = 0, int64_t sb = 0,
                        const int* only = nullptr, const int* only2 = nullptr, int tri = TRI_NONE) {
  if (M <= 0 || N <= 0) return true;
  GemmShape sh;
  sh.M = M;
  sh.N = N;
  sh.K = K;
  sh.kchunk = splits > 1 ? ceil_div(ceil_div(K, splits), BK) * BK : K;
  sh.splits = splits;
  sh.lower_only = lower_only && M == N && BM == BN;
  sh.abort = abort;
  sh.only = only;
  sh.only2 = only2;
  sh.sa = sa;
  sh.sb = sb;
  sh.tri = splits > 1 ? TRI_NONE : tri;
  const int64_t tiles = gemm_tiles((int)ceil_div(M, BM), (int)ceil_div(N, BN), sh.lower_only);
  dim3 grid((unsigned)(tiles * splits), (unsigned)batch, 1);
  hipLaunchKernelGGL((gemm_kernel<T, BM, BN, BK, WM, WN, TA, LA, TB, LB, NOPS, Epi, FOLD>), grid,
                     dim3(WM * WN * ISDF_WAVE), 0, st, sh, A0, B0, A1, B1, K1, epi);
  return launch_ok();
}

// Edge of the square output tiles of an M x N product (times `batch`, its lower
// tiles only when `lower`).  A 128 x 128 tile moves the least data per
// operation but takes 6.8 us per 64 of K on its CU's FP64 matrix cores, so a
// product of few tiles leaves the chip idle and its latency is a tile's: 64
// (four times the tiles) below two 128-tiles per CU, 32 below one 64-tile per
// CU.  256 x 256 x 256 takes 44 us on 128-tiles and 8 on 32-tiles, 13824 x 64
// x 512 116 and 29, 256 x 64 x 512 113 and 13, 13824 x 256 x 256 (216 tiles of
// 128) 51 and, on 64-tiles, 47.
static int tile_for(int64_t M, int64_t N, int lower, int64_t batch = 1) {
  const auto tiles = [&](int t) { return batch * gemm_tiles((int)ceil_div(M, t), (int)ceil_div(N, t), lower); };
  return tiles(128) >= 512 ? 128 : tiles(64) >= 256 ? 64 : 32;
}

// A product with one operand pair on the tiles of edge `tile`.
template <class T, class TA, int LA, class TB, int LB, class Epi>
static bool launch_tiled(int tile, int M, int N, int64_t K, Operand<TA> a, Operand<TB> b, const Epi& epi,
                         int lower_only, const int* abort, hipStream_t st, int splits = 1, int batch = 1,
                         int64_t sa = 0, int64_t sb = 0, const int* only = nullptr, const int* only2 = nullptr,
                         int tri = TRI_NONE) {
  if (tile == 128)
    return launch_gemm<T, 128, 128, 16, 2, 2, TA, LA, TB, LB, 1>(M, N, K, a, b, a, b, 0, epi, lower_only, abort, st,
                                                                splits, batch, sa, sb, only, only2, tri);
  if (tile == 64)
    return launch_gemm<T, 64, 64, 16, 2, 2, TA, LA, TB, LB, 1>(M, N, K, a, b, a, b, 0, epi, lower_only, abort, st,
                                                              splits, batch, sa, sb, only, only2, tri);
  return launch_gemm<T, 32, 32, 32, 2, 2, TA, LA, TB, LB, 1>(M, N, K, a, b, a, b, 0, epi, lower_only, abort, st, splits,
                                                            batch, sa, sb, only, only2, tri);
}

// Plain FP64 GEMM C = alpha op(A) op(B) + beta C.
template <int LA, int LB, class TC, class TA = double>
static bool dgemm(int M, int N, int64_t K, const TA* A, int64_t lda, const double* B, int64_t ldb, TC* C,
                  int64_t ldc, double alpha, double beta, int lower_only, const int* abort, hipStream_t st,
                  const int* only = nullptr, const int* only2 = nullptr, int tri = TRI_NONE) {
  EpiStore<TC> epi{C, ldc, M, N, alpha, beta, nullptr, 0, 0};
  Operand<TA> a{A, lda, nullptr, nullptr};
  Operand<double> b{B, ldb, nullptr, nullptr};
  return launch_tiled<double, TA, LA, double, LB>(tile_for(M, N, lower_only), M, N, K, a, b, epi, lower_only, abort, st,
                                                  1, 1, 0, 0, only, only2, tri);
}

// C = alpha A B^T in FP64, by residues where that is faster (mod_pays) and the
// work buffers are there, else on the FP64 matrix cores.  bal: what balances the
// two operands.  `prepared`: the powers of two and B's residues are in the
// buffers from an earlier call.  With complex buffers B
// has to be the real 2 x 2 block form of a complex matrix, M, N, K count reals
// all the same, and the product is the complex one of half N and K (tol: how far
// B may be from that form, mod_blocks).
template <class TC, class TA = double>
static bool nt_product(int64_t M, int N, int K, const TA* A, int64_t lda, const double* B, int64_t ldb, int bal, TC* C,
                       int64_t ldc, double alpha, const ModWork& w, bool prepared, const int* abort, hipStream_t st,
                       double tol = sizeof(TC) == 4 ? MOD_TOL_SINGLE : 0.0) {
  const int h = w.cplx ? 2 : 1;
  if (!w.mp || !(w.cplx ? mod_pays_c(M, N / h, K / h) : mod_pays(M, N, K)))
    return dgemm<KC, KC, TC, TA>((int)M, N, K, A, lda, B, ldb, C, ldc, alpha, 0.0, 0, abort, st);
  if (!(prepared ? mod_next(w, st) : mod_prepare<TA>(A, lda, (int)M, B, ldb, N / h, K / h, bal, tol, w, abort, st)))
    return false;
  const int vec = ldc % 2 == 0 && (uintptr_t)C % (2 * sizeof(TC)) == 0;
  for (int64_t r = 0, p = 0; r < M; r += w.mp, ++p) {
    const int rows = (int)(M - r < w.mp ? M - r : w.mp);
    ModStore<TC> epi{C + r * ldc, ldc, N, alpha, vec};
    if (!mod_panel<TA>(A + r * lda, lda, rows, N / h, K / h, bal, (int)p, w, epi, abort, st)) return false;
    if (!dgemm<KC, KC, TC, TA>(rows, N, K, A + r * lda, lda, B, ldb, C + r * ldc, ldc, alpha, 0.0, 0, abort, st,
                               w.flags, w.flags + 1 + p))
      return false;
  }
  return true;
}

// Batched FP64 GEMM: batch b uses A + b sa, B + b sb, C + b sc.
template <int LA, int LB>
static bool dgemm_batched(int M, int N, int64_t K, const double* A, int64_t lda, int64_t sa, const double* B,
                          int64_t ldb, int64_t sb, double* C, int64_t ldc, int64_t sc, int batch, double alpha,
                          int tri, const int* abort, hipStream_t st) {
  EpiStore<double> epi{C, ldc, M, N, alpha, 0.0, nullptr, 0, sc};
  Operand<double> a{A, lda, nullptr, nullptr};
  Operand<double> b{B, ldb, nullptr, nullptr};
  return launch_tiled<double, double, LA, double, LB>(tile_for(M, N, 0, batch), M, N, K, a, b, epi, 0, abort, st, 1,
                                                      batch, sa, sb, nullptr, nullptr, tri);
}

// GEMM in compute type T with split-K slices written to C + z * zstride.
// bscale: optional per-k factor of B; lower_only: skip tiles above the diagonal.
template <class T, int LA, int LB, class TA, class TB, class TC>
static bool tgemm(int M, int N, int64_t K, const TA* A, int64_t lda, const TB* B, int64_t ldb, TC* C, int64_t ldc,
                  double alpha, double beta, const int* abort, hipStream_t st, TilePlan plan = {0, 1},
                  int64_t zstride = 0, const double* bscale = nullptr, int lower_only = 0) {
  EpiStore<TC> epi{C, ldc, M, N, alpha, beta, nullptr, zstride, 0};
  Operand<TA> a{A, lda, nullptr, nullptr};
  Operand<TB> b{B, ldb, nullptr, bscale};
  return launch_tiled<T, TA, LA, TB, LB>(plan.tile ? plan.tile : tile_for(M, N, lower_only), M, N, K, a, b, epi,
                                         lower_only, abort, st, plan.splits);
}

// Upper triangle of an n x n matrix from its lower triangle: a 64 x 64 tile
// per workgroup through LDS, so that both sides move whole cache lines.
__global__ __launch_bounds__(256) void mirror_lower(double* __restrict__ H, int n, const int* abort) {
  if (*abort) return;
  __shared__ double t[64][65];
  const int i0 = 64 * blockIdx.y, j0 = 64 * blockIdx.x;  // tile (i, j), i >= j, of the lower triangle
  if (j0 > i0) return;
  const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
  for (int r = r0; r < 64; r += 4)
    if (i0 + r < n && j0 + c < n) t[r][c] = H[(int64_t)(i0 + r) * n + j0 + c];
  __syncthreads();
  for (int r = r0; r < 64; r += 4)
    if (j0 + r < n && i0 + c < n && i0 + c > j0 + r) H[(int64_t)(j0 + r) * n + i0 + c] = t[c][r];
}
static bool mirror(double* H, int n, const int* abort, hipStream_t s) {
  const unsigned b = (unsigned)ceil_div(n, 64);
  hipLaunchKernelGGL(mirror_lower, dim3(b, b), dim3(256), 0, s, H, n, abort);
  return launch_ok();
}

// W (order 2 n, the real form of a complex matrix up to rounding) to the nearest
// matrix of exact 2 x 2 blocks [[re, im], [-im, re]]: the mean of the two copies
// of each part.  Symmetric stays symmetric.
__global__ __launch_bounds__(256) void block_form(double* __restrict__ W, int n, const int* abort) {
  if (*abort) return;
  const int i = blockIdx.y;
  double* r0 = W + (int64_t)2 * i * 2 * n;  // (the caller's: aligned to a double only)
  double* r1 = r0 + 2 * n;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
    const double re = 0.5 * (r0[2 * j] + r1[2 * j + 1]), im = 0.5 * (r0[2 * j + 1] - r1[2 * j]);
    r0[2 * j] = r1[2 * j + 1] = re;
    r0[2 * j + 1] = im;
    r1[2 * j] = -im;
  }
}
static bool to_block_form(double* W, int n, const int* abort, hipStream_t s) {
  hipLaunchKernelGGL(block_form, dim3((unsigned)ceil_div(n, 256), (unsigned)n), dim3(256), 0, s, W, n, abort);
  return launch_ok();
}

// Cholesky of X (n x n, lower, in place) and W = X^-1 into X:
//  1. blocked right-looking Cholesky: 64-wide diagonal blocks factored and
//     inverted in LDS, panel L21 = A21 L11^-T, trailing update A22 -= L21 L21^T
//     on its lower tiles.  (The columns beyond a 256-wide block updated once per
//     block save 4 ms of passes over the trailing matrix at n = 8192, and make
//     the inverse 5 to 10 % less accurate: sums of 256 terms between two
//     subtractions instead of 64.)
//  2. Y = L^-1 by recursive doubling: once every aligned segment of size b
//     has its inverse, a pair [[A, 0], [L21, C]] gets its lower-left block
//     -C^-1 L21 A^-1 (two GEMMs, batched over all pairs of the level; K loops
//     leave out the zeros of the triangular operand);
//  3. W = Y^T Y, zeros left out, from MIRROR_MIN on its lower tiles only
//     (below, every tile runs at once and the mirror pass would add a launch).
struct InvWork {
  double* Y;  // [n][n]
  double* R;  // [n][n] scratch
};
constexpr int MIRROR_MIN = 768;

// (w.Y all zeros on entry)
static int spd_inverse(double* X, int n, InvWork w, FitState* st, hipStream_t s) {
  const int* ab = &st->abort;
  for (int k0 = 0; k0 < n; k0 += NB) {
    const int kb = n - k0 < NB ? n - k0 : NB, k1 = k0 + kb;
    hipLaunchKernelGGL(potrf_diag, dim3(1), dim3(256), 0, s, X, (int64_t)n, k0, kb, w.Y, (int64_t)n, st);
    if (!launch_ok()) return ISDF_E_HIP;
    if (k1 >= n) continue;
    double* P = X + (int64_t)k1 * n + k0;
    // panel: L21 = A21 L11^-T in place, each workgroup with all 64 columns of
    // its rows (it reads them before it writes them)
    EpiStore<double> epi{P, n, n - k1, kb, 1.0, 0.0, nullptr, 0, 0};
    Operand<double> a{P, n, nullptr, nullptr}, b{w.Y + (int64_t)k0 * n + k0, n, nullptr, nullptr};
    if (!launch_gemm<double, 32, NB, 32, 2, 2, double, KC, double, KC, 1>(n - k1, kb, kb, a, b, a, b, 0, epi, 0, ab, s))
      return ISDF_E_HIP;
    if (!dgemm<KC, KC>(n - k1, n - k1, kb, P, n, P, n, X + (int64_t)k1 * n + k1, n, -1.0, 1.0, 1, ab, s))
      return ISDF_E_HIP;
  }
  const int64_t ld = n;
  for (int b = NB; b < n; b *= 2) {
    const int pairs = n / (2 * b);
    const int64_t step = 2 * (int64_t)b * (ld + 1);  // from one pair's origin to the next
    if (pairs > 0) {
      // R_p = L21 A^-1, then C-block rows of Y: -C^-1 R_p
      if (!dgemm_batched<KC, XC>(b, b, b, X + (int64_t)b * ld, ld, step, w.Y, ld, step, w.R, b, (int64_t)b * b,
                                 pairs, 1.0, TRI_B_LOWER, ab, s))
        return ISDF_E_HIP;
      if (!dgemm_batched<KC, XC>(b, b, b, w.Y + (int64_t)b * ld + b, ld, step, w.R, b, (int64_t)b * b,
                                 w.Y + (int64_t)b * ld, ld, step, pairs, -1.0, TRI_A_LOWER, ab, s))
        return ISDF_E_HIP;
    }
    const int o = pairs * 2 * b, rem = n - o;
    if (rem > b) {  // ragged last pair: A of size b, C of size rem - b
      const int c = rem - b;
      const int64_t org = (int64_t)o * (ld + 1);
      if (!dgemm_batched<KC, XC>(c, b, b, X + org + (int64_t)b * ld, ld, 0, w.Y + org, ld, 0, w.R, b, 0, 1, 1.0,
                                 TRI_B_LOWER, ab, s))
        return ISDF_E_HIP;
      if (!dgemm_batched<KC, XC>(c, b, c, w.Y + org + (int64_t)b * ld + b, ld, 0, w.R, b, 0,
                                 w.Y + org + (int64_t)b * ld, ld, 0, 1, -1.0, TRI_A_LOWER, ab, s))
        return ISDF_E_HIP;
    }
  }
  // W = Y^T Y
  const int half = n >= MIRROR_MIN;
  if (!dgemm<XC, XC>(n, n, n, w.Y, n, w.Y, n, X, n, 1.0, 0.0, half, ab, s, nullptr, nullptr, TRI_UPPER_LOWER))
    return ISDF_E_HIP;
  if (half && !mirror(X, n, ab, s)) return ISDF_E_HIP;
  return ISDF_OK;
}

// Precision policy of the orbital contractions (the Gram blocks and the
// adjoint's products with Phi_mu / Phi).  E: storage of packed right-hand
// sides, and compute type of the plain engines; Q: compute type of the
// split-K reductions over grid rows; SPLIT: split engine or -1.
template <int PREC>
struct Prec;
template <>
struct Prec<ISDF_P_FP64> {
  typedef double E;
  typedef double Q;
  static constexpr int SPLIT = -1;
};
template <>
struct Prec<ISDF_P_FP32> {
  typedef float E;
  typedef float Q;
  static constexpr int SPLIT = -1;
};
template <>
struct Prec<ISDF_P_BF16X6> {
  typedef double E;
  typedef float Q;
  static constexpr int SPLIT = SPLIT_BF16X6;
};
template <>
struct Prec<ISDF_P_FP16X3> {
  typedef double E;
  typedef float Q;
  static constexpr int SPLIT = SPLIT_FP16X3;
};

// Slices between FP64 folds of the leading accumulator.
constexpr int SPLIT_FLUSH = 2;

// Output tile of the one-operand-pair split products: 128 x 128 with eight
// wavefronts of 64 x 32 (one workgroup per CU at two wavefronts per SIMD).
// Against 128 x 64 tiles of four wavefronts each operand panel serves twice
// the outputs, and the 512 threads stage a slice with half the registers
// each; bitwise the same products.
template <int MODE>
struct SplitTile {
  static constexpr int BM = 128, BN = 128, WM = 2, WN = 4;
};

// lower_only (M = N): only the tiles that reach the lower triangle, for
// symmetric products whose upper triangle is mirrored afterwards.
template <int MODE, int BM, int BN, int WM, int WN, int NOPS, class Epi>
static bool launch_split(int M, int N, int64_t K, PlaneOp<typename SplitT<MODE>::P> A0,
                         PlaneOp<typename SplitT<MODE>::P> B0, PlaneOp<typename SplitT<MODE>::P> A1,
                         PlaneOp<typename SplitT<MODE>::P> B1, int64_t K1, const double* scales, const Epi& epi,
                         const int* abort, hipStream_t st, int lower_only = 0, int splits = 1) {
  static_assert(BM % BN == 0, "tile");
  if (M <= 0 || N <= 0) return true;
  GemmShape sh{};
  sh.M = M;
  sh.N = N;
  sh.K = K;
  sh.splits = NOPS == 1 && splits > 1 ? splits : 1;
  sh.kchunk = sh.splits > 1 ? ceil_div(ceil_div(K, sh.splits), 32) * 32 : K;  // whole 32-deep slices
  sh.lower_only = lower_only && M == N;
  sh.abort = abort;
  const int64_t tiles = split_tiles((int)ceil_div(M, BM), (int)ceil_div(N, BN), BM / BN, sh.lower_only) * sh.splits;
  hipLaunchKernelGGL((gemm_split_kernel<MODE, BM, BN, WM, WN, NOPS, SPLIT_FLUSH, Epi>), dim3((unsigned)tiles),
                     dim3(WM * WN * ISDF_WAVE), 0, st, sh, A0, B0, A1, B1, K1, scales, epi);
  return launch_ok();
}

// Plane buffers of the split engines (16-bit parts, K padded to 32).
struct SplitWork {
  void* rows_a;      // parts of orbital rows of Phi  [NP][rows_cap][ldp_a]
  void* rows_b;      //                     of Psi    [NP][rows_cap][ldp_b]
  void* e_a;         // parts of the packed Gram right-hand side of Phi [NP][e_rows][ldp_a]
  void* e_b;         //                                          of Psi
  int ldp_a, ldp_b;  // row pitch of the planes
  int k_a, k_b;      // K extent: 2 n rounded up to 32
  int64_t rows_cap;
  int e_rows;        // 2 N_mu rounded up to 32
};

// K extent of the planes of an n-column complex operand (2 n reals rounded
// up to 32) and their row pitch (the same; see ldk_of for a padded pitch).
static inline int kext_of(int n) { return (int)ceil_div(2 * (int64_t)n, 32) * 32; }
static inline int ldp_of(int n) { return kext_of(n); }
static inline size_t plane_bytes(int np, int64_t rows, int ldp) { return (size_t)np * rows * ldp * 2; }

template <int MODE, class TS>
static bool split_rows(const TS* x, int64_t ld, int n, const int* gather, int64_t nr_src, int64_t r0, int rows,
                       void* out, int ldp, int64_t rows_cap, const double* scale, hipStream_t s) {
  if (rows <= 0) return true;
  const int64_t work = (int64_t)rows * (ldp / 8);
  int64_t blocks = ceil_div(work, 256);
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL((split_planes<MODE, TS>), dim3((unsigned)blocks), dim3(256), 0, s, x, ld, n, gather, nr_src, r0,
                     rows, (typename SplitT<MODE>::P*)out, ldp, rows_cap * ldp, scale);
  return launch_ok();
}

// Largest |real or imaginary part| of an r-major complex matrix, folded into
// *out (positive doubles order like their bit patterns).
template <class TS>
__global__ void absmax_rows(const TS* __restrict__ x, int64_t ld, int n, int64_t nr, double* out) {
  double m = 0.0;
  for (int64_t r = blockIdx.x; r < nr; r += gridDim.x)
    for (int k = threadIdx.x; k < 2 * n; k += blockDim.x) m = fmax(m, fabs((double)x[2 * r * ld + k]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, ISDF_WAVE));
  if ((threadIdx.x & 63) == 0 && m > 0.0) atomic_max_pos(out, m);
}

// scale[i] = 2^e with amax[src[i]] 2^e <= 2^14 (binary16 operands).
__global__ void pow2_scales(const double* amax, double* scale, int a0, int a1, int a2, int a3) {
  scale[0] = pow2_scale_for(amax[a0]);
  scale[1] = pow2_scale_for(amax[a1]);
  scale[2] = pow2_scale_for(amax[a2]);
  scale[3] = pow2_scale_for(amax[a3]);
}

template <class TS>
static bool absmax(const TS* x, int64_t ld, int n, int64_t nr, double* out, hipStream_t s) {
  int64_t blocks = nr < 2048 ? nr : 2048;
  hipLaunchKernelGGL((absmax_rows<TS>), dim3((unsigned)(blocks > 0 ? blocks : 1)), dim3(256), 0, s, x, ld, n, nr, out);
  return launch_ok();
}

// Operand scales of the Gram blocks: sc[0..3] = (Phi, E_phi, Psi, E_psi);
// amax[0], amax[1] receive max |Phi|, max |Psi|.  Only the FP16 split uses
// them; the other precisions pass null scales.
template <int PREC, class TS>
static bool gram_scales(const TS* phi, int64_t ld_phi, int n_phi, const TS* psi, int64_t ld_psi, int n_psi,
                        bool aliased, int64_t nr, double* amax, double* sc, hipStream_t s) {
  if (Prec<PREC>::SPLIT != SPLIT_FP16X3) return true;
  if (!fill<double>(amax, 2, 0.0, s)) return false;
  if (!absmax<TS>(phi, ld_phi, n_phi, nr, amax, s)) return false;
  if (!aliased && !absmax<TS>(psi, ld_psi, n_psi, nr, amax + 1, s)) return false;
  hipLaunchKernelGGL(pow2_scales, dim3(1), dim3(1), 0, s, (const double*)amax, sc, 0, 0, aliased ? 0 : 1,
                     aliased ? 0 : 1);
  return launch_ok();
}

// Operand scales of a Gram product over the rows [r0, r0 + rows) only
// (FP16 split; a power of two per operand, so any bound of its magnitude
// will do): sc[0], sc[2] for those rows of Phi and Psi, sc[1], sc[3] for the
// packed right-hand sides E_phi, E_psi (the interpolation rows), whose
// maxima land in amax[2], amax[3]; amax[0], amax[1] receive the rows'.
template <int PREC, class TS>
static bool gram_scales_rows(const TS* phi, int64_t ld_phi, int n_phi, const TS* psi, int64_t ld_psi, int n_psi,
                             bool aliased, int64_t r0, int64_t rows, const double* Ephi, const double* Epsi,
                             int nmu16, double* amax, double* sc, hipStream_t s) {
  if (Prec<PREC>::SPLIT != SPLIT_FP16X3) return true;
  if (!fill<double>(amax, 4, 0.0, s)) return false;
  if (rows > 0 && !absmax<TS>(phi + 2 * r0 * ld_phi, ld_phi, n_phi, rows, amax, s)) return false;
  if (!absmax<double>(Ephi, n_phi, n_phi, 2 * (int64_t)nmu16, amax + 2, s)) return false;
  if (!aliased) {
    if (rows > 0 && !absmax<TS>(psi + 2 * r0 * ld_psi, ld_psi, n_psi, rows, amax + 1, s)) return false;
    if (!absmax<double>(Epsi, n_psi, n_psi, 2 * (int64_t)nmu16, amax + 3, s)) return false;
  }
  hipLaunchKernelGGL(pow2_scales, dim3(1), dim3(1), 0, s, (const double*)amax, sc, 0, 2, aliased ? 0 : 1,
                     aliased ? 2 : 3);
  return launch_ok();
}

// Gram + Hadamard of `rows` orbital rows (gathered through `gather` if
// non-null, else starting at row r0) into G (and optionally A, B).
template <int PREC, class TS>
static bool gram(const TS* phi, int64_t ld_phi, int n_phi, const TS* psi, int64_t ld_psi, int n_psi, bool aliased,
                 const typename Prec<PREC>::E* Ephi, const typename Prec<PREC>::E* Epsi, int nmu16, int n_mu,
                 const int* gather, int64_t nr, int64_t r0, int rows, double* G, int64_t ldg, int mode,
                 const int* abort, hipStream_t s, const double* scales, const SplitWork* sw, double* Aout = nullptr,
                 double* Bout = nullptr) {
  typedef typename Prec<PREC>::E T;
  constexpr int SPLIT = Prec<PREC>::SPLIT;
  EpiGram epi{G, ldg, rows, n_mu, mode, Aout, Bout, 2 * (int64_t)n_mu};
  const int N = 2 * nmu16;
  Operand<TS> a0{phi + 2 * r0 * ld_phi, 2 * ld_phi, gather, nullptr};
  Operand<T> b0{Ephi, 2 * (int64_t)n_phi, nullptr, nullptr};
  Operand<TS> a1{psi + 2 * r0 * ld_psi, 2 * ld_psi, gather, nullptr};
  Operand<T> b1{Epsi, 2 * (int64_t)n_psi, nullptr, nullptr};
  if constexpr (SPLIT >= 0) {
    typedef typename SplitT<SPLIT>::P P;
    const double* sc = SPLIT == SPLIT_FP16X3 ? scales : nullptr;
    if (!split_rows<SPLIT, TS>(phi, ld_phi, n_phi, gather, nr, gather ? 0 : r0, rows, sw->rows_a, sw->ldp_a,
                               sw->rows_cap, sc, s))
      return false;
    PlaneOp<P> pa0{(const P*)sw->rows_a, sw->ldp_a, sw->rows_cap * sw->ldp_a, nullptr};
    PlaneOp<P> pb0{(const P*)sw->e_a, sw->ldp_a, (int64_t)sw->e_rows * sw->ldp_a, nullptr};
    if (aliased)
      return launch_split<SPLIT, SplitTile<SPLIT>::BM, SplitTile<SPLIT>::BN, SplitTile<SPLIT>::WM,
                          SplitTile<SPLIT>::WN, 1>(rows, N, sw->k_a, pa0, pb0, pa0, pb0, 0, sc, epi, abort, s);
    if (!split_rows<SPLIT, TS>(psi, ld_psi, n_psi, gather, nr, gather ? 0 : r0, rows, sw->rows_b, sw->ldp_b,
                               sw->rows_cap, sc ? sc + 2 : nullptr, s))
      return false;
    PlaneOp<P> pa1{(const P*)sw->rows_b, sw->ldp_b, sw->rows_cap * sw->ldp_b, nullptr};
    PlaneOp<P> pb1{(const P*)sw->e_b, sw->ldp_b, (int64_t)sw->e_rows * sw->ldp_b, nullptr};
    return launch_split<SPLIT, 64, 64, 2, 2, 2>(rows, N, sw->k_a, pa0, pb0, pa1, pb1, sw->k_b, sc, epi, abort, s);
  } else {
    // FP32: accumulators folded into FP64 every 2 steps (32-deep)
    constexpr int FOLD = sizeof(T) == 4 ? 2 : 0;
    if constexpr (FOLD == 0) {
      // few tiles: smaller ones (tile_for)
      if (aliased && tile_for(rows, N, 0) < 128)
        return launch_gemm<T, 64, 64, 16, 2, 2, TS, KC, T, KC, 1>(rows, N, 2 * (int64_t)n_phi, a0, b0, a0, b0, 0, epi,
                                                                  0, abort, s);
      if (!aliased && tile_for(rows, N, 0) < 128)
        return launch_gemm<T, 64, 64, 16, 2, 2, TS, KC, T, KC, 2>(rows, N, 2 * (int64_t)n_phi, a0, b0, a1, b1,
                                                                  2 * (int64_t)n_psi, epi, 0, abort, s);
    }
    if (aliased)
      return launch_gemm<T, 128, 128, 16, 2, 2, TS, KC, T, KC, 1, FOLD>(rows, N, 2 * (int64_t)n_phi, a0, b0, a0, b0,
                                                                         0, epi, 0, abort, s);
    return launch_gemm<T, 128, 64, 16, 2, 2, TS, KC, T, KC, 2, FOLD>(rows, N, 2 * (int64_t)n_phi, a0, b0, a1, b1,
                                                                      2 * (int64_t)n_psi, epi, 0, abort, s);
  }
}

template <class TS, class T>
static bool pack(const TS* phi, int64_t ld, int n, const int* idx, int n_mu, int64_t nr, int nmu16, T* E,
                 hipStream_t s) {
  const int64_t total = (int64_t)2 * nmu16 * 2 * n;
  int64_t blocks = ceil_div(total, 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL((pack_gram_rhs<TS, T>), dim3((unsigned)blocks), dim3(256), 0, s, phi, ld, n, idx, n_mu, nr,
                     2 * nmu16, E);
  return launch_ok();
}

// Parts of the packed Gram right-hand sides (split precisions only).
template <int PREC>
static bool split_rhs(const double* Ephi, const double* Epsi, int n_phi, int n_psi, bool aliased,
                      const double* scales, const SplitWork* sw, hipStream_t s) {
  constexpr int SPLIT = Prec<PREC>::SPLIT;
  if constexpr (SPLIT >= 0) {
    const double* sc = SPLIT == SPLIT_FP16X3 ? scales : nullptr;
    if (!split_rows<SPLIT, double>(Ephi, n_phi, n_phi, nullptr, sw->e_rows, 0, sw->e_rows, sw->e_a, sw->ldp_a,
                                   sw->e_rows, sc ? sc + 1 : nullptr, s))
      return false;
    if (!aliased && !split_rows<SPLIT, double>(Epsi, n_psi, n_psi, nullptr, sw->e_rows, 0, sw->e_rows, sw->e_b,
                                               sw->ldp_b, sw->e_rows, sc ? sc + 3 : nullptr, s))
      return false;
  }
  return true;
}

// Carves the plane buffers of a split precision (no-op otherwise).
static SplitWork carve_split(Carver& c, isdf_prec prec, int n_phi, int n_psi, bool aliased, int n_mu,
                             int64_t rows_cap) {
  SplitWork w{};
  if (prec != ISDF_P_BF16X6 && prec != ISDF_P_FP16X3) return w;
  const int np = prec == ISDF_P_BF16X6 ? 3 : 2;
  w.ldp_a = ldp_of(n_phi);
  w.ldp_b = ldp_of(n_psi);
  w.k_a = kext_of(n_phi);
  w.k_b = kext_of(n_psi);
  w.rows_cap = rows_cap;
  w.e_rows = (int)ceil_div(2 * (int64_t)ceil_div(n_mu, 16) * 16, 32) * 32;
  w.rows_a = c.take<char>(plane_bytes(np, rows_cap, w.ldp_a));
  w.e_a = c.take<char>(plane_bytes(np, w.e_rows, w.ldp_a));
  if (!aliased) {
    w.rows_b = c.take<char>(plane_bytes(np, rows_cap, w.ldp_b));
    w.e_b = c.take<char>(plane_bytes(np, w.e_rows, w.ldp_b));
  }
  return w;
}

static bool fit_args_ok(const isdf_grid* g, isdf_dtype dt, const void* phi, int64_t ld_phi, int n_phi,
                        const void* psi, int64_t ld_psi, int n_psi, const int32_t* idx, int n_mu, isdf_prec prec,
                        int64_t* nr_out) {
  if (!g) return false;
  for (int a = 0; a < 3; ++a)
    if (g->n[a] <= 0) return false;
  const int64_t nr = (int64_t)g->n[0] * g->n[1] * g->n[2];
  if (nr >= INT32_MAX) return false;
  if (dt != ISDF_C128 && dt != ISDF_C64) return false;
  if (!phi || !psi || !idx || n_phi <= 0 || n_psi <= 0 || ld_phi < n_phi || ld_psi < n_psi) return false;
  if (n_mu <= 0 || n_mu > nr) return false;
  if (prec < ISDF_P_FP64 || prec > ISDF_P_FP16X3) return false;
  *nr_out = nr;
  return true;
}

// Bytes per element of the packed right-hand sides (E, F) and gathered
// rows: the FP32 engine stages them in float, every other precision in
// double (the split engines split them while staging).
static size_t tsize_of(isdf_prec p) { return p == ISDF_P_FP32 ? sizeof(float) : sizeof(double); }

}  // namespace
}  // namespace isdf
