// V_mu(r) = int zeta_mu(r') / |r - r'| dr' for every column of Theta
// (eq. V_mu of arXiv:2208.07731, the step after the fit in the paper's
// hybrid-DFT flow), on the periodic grid:
//
//   V-hat(G) = 4 pi zeta-hat(G) / |G|^2,  G = 0 dropped (neutral background).
//
// Theta is r-major [N_r][N_mu] (the fit's layout), so every grid line along
// an axis holds N_mu independent signals side by side.  Five line passes,
// each reading and writing the whole array once (the work is HBM-bound):
//   1. FFT along k   (Theta -> W)          4. inverse FFT along j (W -> W)
//   2. FFT along j   (W -> W)              5. inverse FFT along k (W -> V)
//   3. FFT along i, multiply by 4 pi / (N_r |G|^2), inverse FFT along i
// Where the (j, k) planes fit LDS, passes 1 + 2 and 4 + 5 are one each
// (fft_planes).  Otherwise:
// a workgroup loads one line of n points for 32, 16 or 8 columns (n <= 64,
// 128, 256) into LDS (one 32 KB buffer, passes in place) and runs a
// mixed-radix Stockham FFT (radices 8, 4, 2, 3, 5, 7) there.  Inverse
// transforms are conj(FFT(conj x)).  Real Theta (Psi = Phi) is packed two
// columns per complex signal: the operator is real and even in G, so the
// real and imaginary parts of the result are the two columns' potentials.
#include <type_traits>

#include "common.h"

namespace isdf {
namespace {

constexpr int FFT_CT = 32;         // column padding of the work array (tiles of 32, 16 or 8 columns)
constexpr int FFT_THREADS = 256;
constexpr int FFT_MAXPASS = 12;
constexpr int FFT_NMAX = 256;      // n x 8 columns x 16 B <= 32 KB of LDS

struct FftAxis {
  int n;
  int npass;
  int radix[FFT_MAXPASS];
  int ns[FFT_MAXPASS];     // sub-transform length before the pass
  int tw[FFT_MAXPASS];     // offset of the pass twiddles exp(-2 pi i x / (ns R)), x < ns R
};

struct FftPlan {
  FftAxis ax[3];
  int ntw;                 // table entries (double2)
};

static bool factor_axis(int n, FftAxis& a, int& off) {
  a.n = n;
  a.npass = 0;
  int ns = 1, m = n;
  static const int radices[] = {8, 4, 2, 3, 5, 7};
  while (m > 1) {
    int r = 0;
    for (int c : radices)
      if (m % c == 0) {
        r = c;
        break;
      }
    if (r == 0 || a.npass == FFT_MAXPASS) return false;
    a.radix[a.npass] = r;
    a.ns[a.npass] = ns;
    a.tw[a.npass] = off;
    off += ns * r;
    ++a.npass;
    ns *= r;
    m /= r;
  }
  return true;
}

static bool make_plan(const isdf_grid* g, FftPlan& p) {
  int off = 0;
  for (int a = 0; a < 3; ++a) {
    if (g->n[a] > FFT_NMAX || !factor_axis(g->n[a], p.ax[a], off)) return false;
  }
  p.ntw = off;
  return true;
}

// Twiddle tables of the three axes.
__global__ void fft_tables(FftPlan p, double2* __restrict__ tab) {
  for (int a = 0; a < 3; ++a) {
    const FftAxis& ax = p.ax[a];
    for (int s = 0; s < ax.npass; ++s) {
      const int m = ax.ns[s] * ax.radix[s];
      for (int x = threadIdx.x; x < m; x += blockDim.x) {
        double sn, cs;
        sincospi(-2.0 * x / m, &sn, &cs);
        tab[ax.tw[s] + x] = make_double2(cs, sn);
      }
    }
  }
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }  // a * (-i)

__device__ __forceinline__ void dft4(double2& v0, double2& v1, double2& v2, double2& v3) {
  const double2 a0 = cadd(v0, v2), a1 = csub(v0, v2), a2 = cadd(v1, v3), a3 = mul_mi(csub(v1, v3));
  v0 = cadd(a0, a2);
  v2 = csub(a0, a2);
  v1 = cadd(a1, a3);
  v3 = csub(a1, a3);
}

// cos and sin of 2 pi j / R, R = 3, 5 or 7.
template <int R>
struct OddRoot {
  static constexpr double C3 = -0.5, S3 = 0.86602540378443864676;
  static constexpr double C5[2] = {0.30901699437494742410, -0.80901699437494742410};
  static constexpr double S5[2] = {0.95105651629515357212, 0.58778525229247312917};
  static constexpr double C7[3] = {0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624};
  static constexpr double S7[3] = {0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048};
  __device__ __forceinline__ static constexpr double re(int j) {
    const int k = j > R / 2 ? R - j : j;
    return k == 0 ? 1.0 : R == 3 ? C3 : R == 5 ? C5[k - 1] : C7[k - 1];
  }
  __device__ __forceinline__ static constexpr double im(int j) {
    const int k = j > R / 2 ? R - j : j;
    const double s = k == 0 ? 0.0 : R == 3 ? S3 : R == 5 ? S5[k - 1] : S7[k - 1];
    return j > R / 2 ? -s : s;
  }
};

// Forward DFT of v[0..R), R a compile-time radix (values stay in registers).
template <int R>
__device__ __forceinline__ void dft(double2 (&v)[R]) {
  if constexpr (R == 2) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 4) {
    dft4(v[0], v[1], v[2], v[3]);
  } else if constexpr (R == 8) {
    double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    double2 o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4(e0, e1, e2, e3);
    dft4(o0, o1, o2, o3);
    const double h = 0.70710678118654752440;  // 1 / sqrt(2)
    // o_q *= exp(-2 pi i q / 8)
    o1 = make_double2(h * (o1.x + o1.y), h * (o1.y - o1.x));
    o2 = mul_mi(o2);
    o3 = make_double2(h * (o3.y - o3.x), -h * (o3.x + o3.y));
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1);
    v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3);
    v[7] = csub(e3, o3);
  } else {
    // odd R: pairs t = v_k + v_(R-k), u = v_k - v_(R-k); output q is
    // v_0 + sum_k cos(2 pi q k / R) t_k  -/+  i sum_k sin(2 pi q k / R) u_k
    constexpr int H = (R - 1) / 2;
    double2 t[H], u[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
      t[k] = cadd(v[k + 1], v[R - 1 - k]);
      u[k] = csub(v[k + 1], v[R - 1 - k]);
    }
    const double2 v0 = v[0];
#pragma unroll
    for (int k = 0; k < H; ++k) v[0] = cadd(v[0], t[k]);
#pragma unroll
    for (int q = 1; q <= H; ++q) {
      double2 a = v0, b = make_double2(0.0, 0.0);
#pragma unroll
      for (int k = 1; k <= H; ++k) {
        const double c = OddRoot<R>::re((q * k) % R), s = OddRoot<R>::im((q * k) % R);
        a.x += c * t[k - 1].x;
        a.y += c * t[k - 1].y;
        b.x += s * u[k - 1].x;
        b.y += s * u[k - 1].y;
      }
      v[q] = make_double2(a.x + b.y, a.y - b.x);
      v[R - q] = make_double2(a.x - b.y, a.y + b.x);
    }
  }
}

// One Stockham pass of radix R over the CT columns of LDS buffer `a`, in
// place: each thread reads its butterflies' inputs into registers, the
// workgroup synchronises, and the outputs go back into `a`.  A thread owns
// at most ceil(8 / R) butterflies (n CT <= 2048 elements over 256 threads).
template <int R, int CT>
__device__ __forceinline__ void stockham_pass(double2* a, int n, int ns, const double2* __restrict__ tw) {
  const int c = threadIdx.x % CT, grp = threadIdx.x / CT;
  constexpr int NGRP = FFT_THREADS / CT;
  constexpr int NB = (8 + R - 1) / R;
  const int m = n / R;
  double2 v[NB][R];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int j = grp + q * NGRP;
    if (j < m) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = a[(j + r * m) * CT + c];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int j = grp + q * NGRP;
    if (j < m) {
      const int k = j % ns;
      if (ns > 1) {
#pragma unroll
        for (int r = 1; r < R; ++r) v[q][r] = cmul(v[q][r], tw[k * r]);
      }
      dft<R>(v[q]);
      const int d = (j / ns) * ns * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) a[(d + r * ns) * CT + c] = v[q][r];
    }
  }
  __syncthreads();
}

// Forward FFT, in place, of the CT columns held in LDS buffer `a` (n points
// each, element (x, c) at a[x * CT + c]).
// POW2: every radix is 8, 4 or 2 (a kernel without the register-hungry
// generic radices).
template <int CT, bool POW2>
__device__ void fft_lds(double2* a, const FftAxis& ax, const double2* __restrict__ tab) {
  const int n = ax.n;
  for (int s = 0; s < ax.npass; ++s) {
    const double2* tw = tab + ax.tw[s];
    const int R = ax.radix[s];
    if (R == 8) stockham_pass<8, CT>(a, n, ax.ns[s], tw);
    else if (R == 4) stockham_pass<4, CT>(a, n, ax.ns[s], tw);
    else if (R == 2) stockham_pass<2, CT>(a, n, ax.ns[s], tw);
    else if constexpr (!POW2) {
      if (R == 3) stockham_pass<3, CT>(a, n, ax.ns[s], tw);
      else if (R == 5) stockham_pass<5, CT>(a, n, ax.ns[s], tw);
      else stockham_pass<7, CT>(a, n, ax.ns[s], tw);
    }
  }
}

// Line geometry: point x of line `line` along axis `axis`.
struct Lines {
  int n0, n1, n2;
  __device__ __forceinline__ int64_t point(int axis, int64_t line, int x) const {
    if (axis == 2) return line * n2 + x;                             // line = i n1 + j
    if (axis == 1) return (line / n2) * (int64_t)n1 * n2 + (int64_t)x * n2 + line % n2;  // line = i n2 + k
    return (int64_t)x * n1 * n2 + line;                              // line = j n2 + k
  }
};

// Consecutive logical workgroups on one XCD (they are dealt out to the 8 XCDs in turn).
__device__ __forceinline__ int xcd_order(int bid, int total) {
  const int full = (total / 8) * 8;
  if (bid >= full) return bid;
  return (bid % 8) * (total / 8) + bid / 8;
}

enum { SRC_W = 0, SRC_REAL = 1, SRC_CPLX = 2 };
enum { DST_W = 0, DST_REAL = 1, DST_CPLX = 2 };

// One line pass.  dir: 0 forward, 1 inverse, 2 forward + Poisson kernel +
// inverse (axis 0 only).  Source / destination: the work array W, stored in
// tiles of 32 columns ([ncols / 32][N_r][32] double2, so that a k-line of a
// tile is contiguous), or Theta / V as real pairs or complex of type TS.
template <class TS, int SRC, int DST, int CT, bool POW2>
__global__ __launch_bounds__(FFT_THREADS) void fft_pass(const void* __restrict__ src, int64_t lds, void* __restrict__ dst,
                                                        int64_t ldd, const double2* __restrict__ W_in,
                                                        double2* __restrict__ W_out, int64_t ncols, int n_mu,
                                                        Lines L, int axis, int dir, FftPlan plan,
                                                        const double2* __restrict__ tab, double3 gscale,
                                                        double inv_nr) {
  extern __shared__ double2 lds_buf[];
  const FftAxis& ax = plan.ax[axis];
  const int n = ax.n;
  double2* a = lds_buf;
  const int64_t line = blockIdx.x;
  const int64_t nr = (int64_t)L.n0 * L.n1 * L.n2;
  const int64_t c0 = (int64_t)blockIdx.y * CT;
  const bool conj_in = dir == 1;
  // load: at most 8 elements per thread (n CT <= 2048), all issued before
  // the LDS stores so that they are in flight together
  constexpr int PER = 8;
  const int total = n * CT;
  double2 t[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int e = threadIdx.x + q * FFT_THREADS;
    t[q] = make_double2(0.0, 0.0);
    if (e < total) {
      const int x = e / CT, c = e % CT;
      const int64_t p = L.point(axis, line, x), col = c0 + c;
      if (SRC == SRC_W) {
        t[q] = W_in[((col >> 5) * nr + p) * 32 + (col & 31)];
      } else if (SRC == SRC_REAL) {
        const TS* row = (const TS*)src + p * lds;
        if (2 * col < n_mu) t[q].x = (double)row[2 * col];
        if (2 * col + 1 < n_mu) t[q].y = (double)row[2 * col + 1];
      } else {
        if (col < n_mu) t[q] = Cplx<TS>::load((const TS*)src + 2 * (p * lds + col));
      }
    }
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int e = threadIdx.x + q * FFT_THREADS;
    if (e < total) a[e] = conj_in ? make_double2(t[q].x, -t[q].y) : t[q];
  }
  __syncthreads();
  fft_lds<CT, POW2>(a, ax, tab);
  double2* res = a;
  if (dir == 2) {
    // res holds the spectrum along axis 0 (all three axes transformed):
    // multiply by 4 pi / (N_r |G|^2), then conj for the inverse transform
    const int64_t j = line / L.n2, k = line % L.n2;
    const int mj = j < (L.n1 + 1) / 2 ? (int)j : (int)j - L.n1;
    const int mk = k < (L.n2 + 1) / 2 ? (int)k : (int)k - L.n2;
    const double gjk = (mj * gscale.y) * (mj * gscale.y) + (mk * gscale.z) * (mk * gscale.z);
    for (int e = threadIdx.x; e < n * CT; e += FFT_THREADS) {
      const int x = e / CT;
      const int mi = x < (n + 1) / 2 ? x : x - n;
      const double g2 = (mi * gscale.x) * (mi * gscale.x) + gjk;
      const double kv = g2 > 0.0 ? 4.0 * M_PI * inv_nr / g2 : 0.0;
      const double2 v = res[e];
      res[e] = make_double2(kv * v.x, -kv * v.y);
    }
    __syncthreads();
    fft_lds<CT, POW2>(res, ax, tab);
  }
  const bool conj_out = dir >= 1;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int e = threadIdx.x + q * FFT_THREADS;
    if (e < total) t[q] = res[e];
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int e = threadIdx.x + q * FFT_THREADS;
    if (e >= total) continue;
    const int x = e / CT, c = e % CT;
    const int64_t p = L.point(axis, line, x), col = c0 + c;
    double2 v = t[q];
    if (conj_out) v.y = -v.y;
    if (DST == DST_W) {
      W_out[((col >> 5) * nr + p) * 32 + (col & 31)] = v;
    } else if (DST == DST_REAL) {
      TS* row = (TS*)dst + p * ldd;
      if (2 * col < n_mu) row[2 * col] = (TS)v.x;
      if (2 * col + 1 < n_mu) row[2 * col + 1] = (TS)v.y;
    } else {
      if (col < n_mu) Cplx<TS>::store((TS*)dst + 2 * (p * ldd + col), v.x, v.y);
    }
  }
}

// ------------------------------------------------- two axes in one pass
// The (j, k) planes of a few columns fit LDS, so both of their axes are
// transformed in one read and one write of the array: three passes over memory
// (planes, axis i with the kernel, planes back) instead of five, which is what
// the work is bound by.  A plane of n1 x n2 points of `ct` columns (a power of
// two) holds at most 8 points per thread; its first radix pass takes the points
// from memory and its last one writes them there, both straight from registers.
// The work array is then [ncols / ct][N_r][ct], so that planes and runs of
// lines are contiguous.  Theta and V are touched ct columns (16 ct bytes of
// FP64) at a time: workgroups of neighbouring columns of a plane are given to
// one XCD, whose L2 joins them to whole cache lines.
// 64^3, 2048 real columns (4.3 GB each way): 8.7 ms in five passes of 1.75 at
// 4.9 TB/s, 7.2 in these (planes 2.7 each, axis i 1.9): one 144 KB workgroup per
// CU waits for its points before it transforms them, so a plane pass reaches
// 3.2 TB/s.

struct PlaneArgs {
  const void* theta;  // forward source
  void* V;            // inverse destination
  int64_t ld;         // of theta or V
  double2* W;
  int n_mu, cplx, vec;
  int lct;            // log2 ct
  int ntiles;         // column tiles
  Lines L;
  int pitch;          // LDS points per row of the plane
};

// a / n of 0 <= a < 2^14, n <= 2^8, inv = 1 / n: (a + 1/2) / n is at least
// 1 / (2 n) from an integer, far more than the product's rounding.
__device__ __forceinline__ int small_div(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

// One radix pass along k (ALONG_K) or j of the plane in LDS buffer `a`, T
// threads.  FIRST: the points come from memory, LAST: they go there.
template <class TS, int T, bool INV, int R, bool ALONG_K, bool FIRST, bool LAST>
__device__ __forceinline__ void plane_pass(double2* a, const PlaneArgs& A, const FftAxis& ax, int s,
                                           const double2* __restrict__ tab, int64_t p0, int64_t tile) {
  constexpr int NB = (8 + R - 1) / R;
  const double2* tw = tab + ax.tw[s];
  const int ns = ax.ns[s], m = ax.n / R, ct = 1 << A.lct;
  const int c = threadIdx.x & (ct - 1), step = T >> A.lct;
  const int n2 = A.L.n2, total = m * (ALONG_K ? A.L.n1 : n2);
  const float inv_line = 1.0f / (float)(ALONG_K ? m : n2), inv_ns = 1.0f / (float)ns;
  const int64_t nr = (int64_t)A.L.n0 * A.L.n1 * n2;
  const int col = (int)tile * ct + c;
  auto lds_at = [&](int line, int x) {
    const int y = ALONG_K ? line : x, k = ALONG_K ? x : line;
    return ((y * A.pitch + k + (k >> 3)) << A.lct) + c;
  };
  const int xstep = ALONG_K ? 1 : n2;  // grid points from one point of a line to the next
  auto point = [&](int line, int x) { return p0 + (ALONG_K ? line * n2 + x : x * n2 + line); };
  double2 v[NB][R];
  int ln[NB], jb[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int b = (int)(threadIdx.x >> A.lct) + q * step;
    const int d = small_div(b, inv_line), e = b - d * (ALONG_K ? m : n2);
    ln[q] = ALONG_K ? d : e;
    jb[q] = b < total ? (ALONG_K ? e : d) : -1;
    if (jb[q] < 0) continue;
    if constexpr (!FIRST) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = a[lds_at(ln[q], jb[q] + r * m)];
    } else if constexpr (INV) {
      const double2* w = A.W + ((tile * nr + point(ln[q], jb[q])) << A.lct) + c;
      const int64_t dw = (int64_t)(m * xstep) << A.lct;
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = w[r * dw];
    } else {
      const int64_t dr = (int64_t)(m * xstep) * A.ld;
      const int64_t at = point(ln[q], jb[q]) * A.ld;
      if (A.cplx) {
        const TS* row = (const TS*)A.theta + 2 * (at + (col < A.n_mu ? col : 0));
#pragma unroll
        for (int r = 0; r < R; ++r) v[q][r] = Cplx<TS>::load(row + 2 * r * dr);
        if (col >= A.n_mu) {
#pragma unroll
          for (int r = 0; r < R; ++r) v[q][r] = make_double2(0.0, 0.0);
        }
      } else if (A.vec && 2 * col + 1 < A.n_mu) {  // an aligned pair of columns
        const TS* row = (const TS*)A.theta + at + 2 * col;
#pragma unroll
        for (int r = 0; r < R; ++r) v[q][r] = Cplx<TS>::load(row + r * dr);
      } else {
        const TS* row = (const TS*)A.theta + at;
        const bool re = 2 * col < A.n_mu, im = 2 * col + 1 < A.n_mu;
#pragma unroll
        for (int r = 0; r < R; ++r)
          v[q][r] = make_double2(re ? (double)row[r * dr + 2 * col] : 0.0, im ? (double)row[r * dr + 2 * col + 1] : 0.0);
      }
    }
  }
  if constexpr (FIRST && INV) {
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r].y = -v[q][r].y;
  }
  if constexpr (!FIRST && !LAST) __syncthreads();
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    if (jb[q] < 0) continue;
    const int g = small_div(jb[q], inv_ns), k = jb[q] - g * ns;
    if (ns > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) v[q][r] = cmul(v[q][r], tw[k * r]);
    }
    dft<R>(v[q]);
    const int d = g * ns * R + k;
    if constexpr (!LAST) {
#pragma unroll
      for (int r = 0; r < R; ++r) a[lds_at(ln[q], d + r * ns)] = v[q][r];
    } else if constexpr (!INV) {
      double2* w = A.W + ((tile * nr + point(ln[q], d)) << A.lct) + c;
      const int64_t dw = (int64_t)(ns * xstep) << A.lct;
#pragma unroll
      for (int r = 0; r < R; ++r) w[r * dw] = v[q][r];
    } else {
      const int64_t dr = (int64_t)(ns * xstep) * A.ld;
      const int64_t at = point(ln[q], d) * A.ld;
      if (A.cplx) {
        TS* row = (TS*)A.V + 2 * (at + col);
        if (col < A.n_mu) {
#pragma unroll
          for (int r = 0; r < R; ++r) Cplx<TS>::store(row + 2 * r * dr, v[q][r].x, -v[q][r].y);
        }
      } else if (A.vec && 2 * col + 1 < A.n_mu) {
        TS* row = (TS*)A.V + at + 2 * col;
#pragma unroll
        for (int r = 0; r < R; ++r) Cplx<TS>::store(row + r * dr, v[q][r].x, -v[q][r].y);
      } else {
        TS* row = (TS*)A.V + at + 2 * col;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (2 * col < A.n_mu) row[r * dr] = (TS)v[q][r].x;
          if (2 * col + 1 < A.n_mu) row[r * dr + 1] = (TS)-v[q][r].y;
        }
      }
    }
  }
  if constexpr (!LAST) __syncthreads();
}

template <class TS, int T, bool INV, bool POW2, bool ALONG_K, bool FIRST, bool LAST>
__device__ __forceinline__ void plane_radix(double2* a, const PlaneArgs& A, const FftAxis& ax, int s,
                                            const double2* __restrict__ tab, int64_t p0, int64_t tile) {
  const int R = ax.radix[s];
  if (R == 8) plane_pass<TS, T, INV, 8, ALONG_K, FIRST, LAST>(a, A, ax, s, tab, p0, tile);
  else if (R == 4) plane_pass<TS, T, INV, 4, ALONG_K, FIRST, LAST>(a, A, ax, s, tab, p0, tile);
  else if (R == 2) plane_pass<TS, T, INV, 2, ALONG_K, FIRST, LAST>(a, A, ax, s, tab, p0, tile);
  else if constexpr (!POW2) {
    if (R == 3) plane_pass<TS, T, INV, 3, ALONG_K, FIRST, LAST>(a, A, ax, s, tab, p0, tile);
    else plane_pass<TS, T, INV, 5, ALONG_K, FIRST, LAST>(a, A, ax, s, tab, p0, tile);
  }
}

// The first axis of a plane, then the second.
template <class TS, int T, bool INV, bool POW2, bool ALONG_K, bool SECOND>
__device__ __forceinline__ void plane_axis(double2* a, const PlaneArgs& A, const FftAxis& ax,
                                           const double2* __restrict__ tab, int64_t p0, int64_t tile) {
  const int mid0 = SECOND ? 0 : 1, mid1 = SECOND ? ax.npass - 1 : ax.npass;
  if constexpr (!SECOND) plane_radix<TS, T, INV, POW2, ALONG_K, true, false>(a, A, ax, 0, tab, p0, tile);
  for (int s = mid0; s < mid1; ++s) plane_radix<TS, T, INV, POW2, ALONG_K, false, false>(a, A, ax, s, tab, p0, tile);
  if constexpr (SECOND) plane_radix<TS, T, INV, POW2, ALONG_K, false, true>(a, A, ax, ax.npass - 1, tab, p0, tile);
}

// Forward (Theta -> W: k, then j) or inverse (W -> V: j, then k) transform of
// one plane of one column tile.  LDS rows are padded by a point per 8, so that
// a radix pass along k writes its strided outputs to different banks.
template <class TS, int T, bool INV, bool POW2>
__global__ __launch_bounds__(T) void fft_planes(PlaneArgs A, FftPlan plan, const double2* __restrict__ tab) {
  __shared__ double2 a[9 * T];
  const int logical = xcd_order(blockIdx.x, gridDim.x);
  const int64_t tile = logical % A.ntiles, p0 = (int64_t)(logical / A.ntiles) * A.L.n1 * A.L.n2;
  constexpr bool K_FIRST = !INV;
  plane_axis<TS, T, INV, POW2, K_FIRST, false>(a, A, plan.ax[K_FIRST ? 2 : 1], tab, p0, tile);
  plane_axis<TS, T, INV, POW2, !K_FIRST, true>(a, A, plan.ax[K_FIRST ? 1 : 2], tab, p0, tile);
}

// Axis i of the planes' work array, forward, times the kernel, inverse, in
// place: CT signals (runs of points of a plane times its ct columns, all
// contiguous) per workgroup.
template <int CT, bool POW2>
__global__ __launch_bounds__(FFT_THREADS) void fft_axis0(double2* __restrict__ W, int lct, Lines L, FftPlan plan,
                                                         const double2* __restrict__ tab, double3 gscale,
                                                         double inv_nr) {
  extern __shared__ double2 lds_buf[];
  double2* a = lds_buf;
  const FftAxis& ax = plan.ax[0];
  const int n = ax.n;
  const int64_t plane = ((int64_t)L.n1 * L.n2) << lct;  // signals of a column tile
  const int c = threadIdx.x % CT;
  const int64_t sig = (int64_t)blockIdx.x * CT + c, q0 = sig < plane ? sig : plane - 1;
  double2* base = W + (int64_t)blockIdx.y * plane * n + q0;
  constexpr int PER = 8, GRP = FFT_THREADS / CT;
  double2 t[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int x = threadIdx.x / CT + q * GRP;
    t[q] = base[(x < n ? x : n - 1) * plane];
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int x = threadIdx.x / CT + q * GRP;
    if (x < n) a[x * CT + c] = t[q];
  }
  __syncthreads();
  fft_lds<CT, POW2>(a, ax, tab);
  const int pt = (int)(q0 >> lct);
  const int j = pt / L.n2, k = pt - j * L.n2;
  const int mj = j < (L.n1 + 1) / 2 ? j : j - L.n1, mk = k < (L.n2 + 1) / 2 ? k : k - L.n2;
  const double gjk = (mj * gscale.y) * (mj * gscale.y) + (mk * gscale.z) * (mk * gscale.z);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int x = threadIdx.x / CT + q * GRP;
    if (x >= n) continue;
    const int mi = x < (n + 1) / 2 ? x : x - n;
    const double g2 = (mi * gscale.x) * (mi * gscale.x) + gjk;
    const double kv = g2 > 0.0 ? 4.0 * M_PI * inv_nr / g2 : 0.0;
    const double2 v = a[x * CT + c];
    a[x * CT + c] = make_double2(kv * v.x, -kv * v.y);
  }
  __syncthreads();
  fft_lds<CT, POW2>(a, ax, tab);
  if (sig >= plane) return;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int x = threadIdx.x / CT + q * GRP;
    if (x < n) {
      const double2 v = a[x * CT + c];
      base[x * plane] = make_double2(v.x, -v.y);
    }
  }
}

// log2 of the columns per plane (at most 8: a whole cache line of Theta), or
// -1 where the five line passes run: the plane of one column does not fit, an
// axis of it has length 1 (no pass to load or store with) or a factor 7 (its
// butterflies would spill at 1024 threads).  The most columns that fit are the
// fastest: 64^3, 2048 columns 7.2 ms with 2 a plane, 8.1 with 1 (two
// workgroups per CU, but half the bytes of a cache line), 8.6 with the line
// passes; 60^3, 1500 columns 6.8, 7.7 and 9.1; 72^3, 1001 columns 10.6 with 1,
// 12.9 with the line passes.
static int plane_columns(const Lines& L) {
  if (L.n1 < 2 || L.n2 < 2 || L.n1 % 7 == 0 || L.n2 % 7 == 0) return -1;
  int lct = 3;
  while (lct >= 0 && (((int64_t)L.n1 * L.n2 << lct) > 8 * 1024 || ((int64_t)L.n1 * (L.n2 + L.n2 / 8) << lct) > 9 * 1024))
    --lct;
  return lct;
}

struct PoissonWork {
  double2* tab;
  double2* W;
  int64_t ncols;
  size_t bytes;
};

static PoissonWork plan_poisson(void* ws, size_t cap, int64_t nr, int n_mu, bool cplx, int ntw) {
  Carver c(ws, cap);
  PoissonWork w{};
  const int64_t cols = cplx ? n_mu : ceil_div(n_mu, 2);
  w.ncols = ceil_div(cols, FFT_CT) * FFT_CT;  // a multiple of both column tiles
  w.tab = c.take<double2>(ntw > 0 ? ntw : 1);
  w.W = c.take<double2>((size_t)nr * w.ncols);
  w.bytes = c.used;
  return w;
}

template <class TS>
static int poisson_run(const isdf_grid* g, const TS* theta, int64_t ld_theta, int n_mu, bool cplx, TS* V,
                       int64_t ld_v, const FftPlan& plan, const PoissonWork& w, hipStream_t s) {
  const Lines L{g->n[0], g->n[1], g->n[2]};
  const int64_t nr = (int64_t)L.n0 * L.n1 * L.n2;
  const double3 gs = make_double3(2.0 * M_PI / (L.n0 * g->h[0]), 2.0 * M_PI / (L.n1 * g->h[1]),
                                  2.0 * M_PI / (L.n2 * g->h[2]));
  const double inv_nr = 1.0 / (double)nr;
  hipLaunchKernelGGL(fft_tables, dim3(1), dim3(256), 0, s, plan, w.tab);
  if (!launch_ok()) return ISDF_E_HIP;
  // Columns per workgroup: 32 (512-byte row segments) for n <= 64, else 16
  // (n <= 128), else 8: n x columns <= 2048 elements, 32 KB of LDS.
  bool pow2 = true;
  for (int a = 0; a < 3; ++a)
    for (int q = 0; q < plan.ax[a].npass; ++q) pow2 = pow2 && (plan.ax[a].radix[q] % 2 == 0);
  // (column tiles are a grid's second dimension, planes times tiles its first in
  // workgroups of up to 1024: more than those hold go by lines)
  const int lct = plane_columns(L);
  if (lct >= 0 && w.ncols >> lct <= 65535 && (w.ncols >> lct) * L.n0 <= (int64_t)1 << 21) {
    const int64_t pts = (int64_t)L.n1 * L.n2 << lct, padded = (int64_t)L.n1 * (L.n2 + L.n2 / 8) << lct;
    const int nt = (int)(w.ncols >> lct);
    const auto vec = [&](const void* q, int64_t ld) { return ld % 2 == 0 && (uintptr_t)q % (2 * sizeof(TS)) == 0; };
    PlaneArgs A{theta, V, ld_theta, w.W, n_mu, cplx ? 1 : 0, vec(theta, ld_theta) ? 1 : 0, lct, nt, L,
                L.n2 + L.n2 / 8};
    PlaneArgs B = A;
    B.ld = ld_v;
    B.vec = vec(V, ld_v) ? 1 : 0;
    const dim3 grid((unsigned)(nt * (int64_t)L.n0));
    auto planes = [&](auto inv_tag, auto pow2_tag, const PlaneArgs& args) -> bool {
      constexpr bool I = decltype(inv_tag)::value, P2 = decltype(pow2_tag)::value;
      if (pts <= 8 * 512 && padded <= 9 * 512)
        hipLaunchKernelGGL((fft_planes<TS, 512, I, P2>), grid, dim3(512), 0, s, args, plan, (const double2*)w.tab);
      else
        hipLaunchKernelGGL((fft_planes<TS, 1024, I, P2>), grid, dim3(1024), 0, s, args, plan, (const double2*)w.tab);
      return launch_ok();
    };
    auto axis0 = [&](auto ct_tag, auto pow2_tag) -> bool {
      constexpr int CTV = decltype(ct_tag)::value;
      constexpr bool P2 = decltype(pow2_tag)::value;
      hipLaunchKernelGGL((fft_axis0<CTV, P2>), dim3((unsigned)ceil_div(pts, CTV), (unsigned)nt), dim3(FFT_THREADS),
                         (size_t)L.n0 * CTV * sizeof(double2), s, w.W, lct, L, plan, (const double2*)w.tab, gs, inv_nr);
      return launch_ok();
    };
    auto three = [&](auto p2) -> bool {
      return planes(std::false_type(), p2, A) &&
             (L.n0 <= 64 ? axis0(std::integral_constant<int, 32>(), p2)
                         : L.n0 <= 128 ? axis0(std::integral_constant<int, 16>(), p2)
                                       : axis0(std::integral_constant<int, 8>(), p2)) &&
             planes(std::true_type(), p2, B);
    };
    return (pow2 ? three(std::true_type()) : three(std::false_type())) ? ISDF_OK : ISDF_E_HIP;
  }
  auto launch = [&](auto src_tag, auto dst_tag, auto ct_tag, auto pow2_tag, int axis, int dir, const void* src,
                    int64_t lds_, void* dst, int64_t ldd) {
    constexpr int S = decltype(src_tag)::value, D = decltype(dst_tag)::value, CTV = decltype(ct_tag)::value;
    constexpr bool P2 = decltype(pow2_tag)::value;
    const int n = plan.ax[axis].n;
    hipLaunchKernelGGL((fft_pass<TS, S, D, CTV, P2>), dim3((unsigned)(nr / n), (unsigned)(w.ncols / CTV)),
                       dim3(FFT_THREADS), (size_t)n * CTV * sizeof(double2), s, src, lds_, dst, ldd,
                       (const double2*)w.W, w.W, w.ncols, n_mu, L, axis, dir, plan, (const double2*)w.tab, gs,
                       inv_nr);
  };
  auto run = [&](auto src_tag, auto dst_tag, int axis, int dir, const void* src, int64_t lds_, void* dst,
                 int64_t ldd) -> bool {
    const int n = plan.ax[axis].n;
    typedef std::integral_constant<int, 32> c32;
    typedef std::integral_constant<int, 16> c16;
    typedef std::integral_constant<int, 8> c8;
    if (pow2) {
      std::true_type p2;
      if (n <= 64) launch(src_tag, dst_tag, c32(), p2, axis, dir, src, lds_, dst, ldd);
      else if (n <= 128) launch(src_tag, dst_tag, c16(), p2, axis, dir, src, lds_, dst, ldd);
      else launch(src_tag, dst_tag, c8(), p2, axis, dir, src, lds_, dst, ldd);
    } else {
      std::false_type p2;
      if (n <= 64) launch(src_tag, dst_tag, c32(), p2, axis, dir, src, lds_, dst, ldd);
      else if (n <= 128) launch(src_tag, dst_tag, c16(), p2, axis, dir, src, lds_, dst, ldd);
      else launch(src_tag, dst_tag, c8(), p2, axis, dir, src, lds_, dst, ldd);
    }
    return launch_ok();
  };
  typedef std::integral_constant<int, SRC_W> sW;
  typedef std::integral_constant<int, DST_W> dW;
  // 1. forward along k, Theta -> W
  bool ok = cplx ? run(std::integral_constant<int, SRC_CPLX>(), dW(), 2, 0, theta, ld_theta, nullptr, 0)
                 : run(std::integral_constant<int, SRC_REAL>(), dW(), 2, 0, theta, ld_theta, nullptr, 0);
  // 2. forward along j; 3. along i with the kernel; 4. inverse along j
  ok = ok && run(sW(), dW(), 1, 0, nullptr, 0, nullptr, 0);
  ok = ok && run(sW(), dW(), 0, 2, nullptr, 0, nullptr, 0);
  ok = ok && run(sW(), dW(), 1, 1, nullptr, 0, nullptr, 0);
  // 5. inverse along k, W -> V
  ok = ok && (cplx ? run(sW(), std::integral_constant<int, DST_CPLX>(), 2, 1, nullptr, 0, V, ld_v)
                   : run(sW(), std::integral_constant<int, DST_REAL>(), 2, 1, nullptr, 0, V, ld_v));
  return ok ? ISDF_OK : ISDF_E_HIP;
}

}  // namespace
}  // namespace isdf

using namespace isdf;

extern "C" size_t isdf_poisson_workspace(const isdf_grid* grid, int32_t n_mu, int32_t is_complex) {
  if (!grid || n_mu <= 0) return 0;
  FftPlan plan{};
  for (int a = 0; a < 3; ++a)
    if (grid->n[a] <= 0) return 0;
  if (!make_plan(grid, plan)) return 0;
  const int64_t nr = (int64_t)grid->n[0] * grid->n[1] * grid->n[2];
  return plan_poisson(nullptr, 0, nr, n_mu, is_complex != 0, plan.ntw).bytes;
}

extern "C" int isdf_poisson(const isdf_grid* grid, int32_t dt_in, const void* theta, int64_t ld_theta, int32_t n_mu,
                            int32_t is_complex, void* V, int64_t ld_v, void* ws, size_t ws_bytes, void* stream) {
  if (!dtype_valid(dt_in)) return ISDF_E_ARG;
  const isdf_dtype dt = (isdf_dtype)dt_in;
  if (!grid || !theta || !V || n_mu <= 0 || ld_theta < n_mu || ld_v < n_mu) return ISDF_E_ARG;
  if (dt != ISDF_C128 && dt != ISDF_C64) return ISDF_E_ARG;
  for (int a = 0; a < 3; ++a)
    if (grid->n[a] <= 0 || !(grid->h[a] > 0.0)) return ISDF_E_ARG;
  FftPlan plan{};
  if (!make_plan(grid, plan)) return ISDF_E_UNSUPPORTED;  // an axis > 256 or with a prime factor > 7
  const int64_t nr = (int64_t)grid->n[0] * grid->n[1] * grid->n[2];
  const int64_t lines_max = nr / 1;
  if (lines_max > INT32_MAX) return ISDF_E_ARG;
  const bool cplx = is_complex != 0;
  PoissonWork w = plan_poisson(ws, ws_bytes, nr, n_mu, cplx, plan.ntw);
  if (!ws || w.bytes > ws_bytes) return ISDF_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  if (dt == ISDF_C128)
    return poisson_run<double>(grid, (const double*)theta, ld_theta, n_mu, cplx, (double*)V, ld_v, plan, w, s);
  return poisson_run<float>(grid, (const float*)theta, ld_theta, n_mu, cplx, (float*)V, ld_v, plan, w, s);
}
