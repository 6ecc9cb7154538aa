// ISDF-compressed exchange operator (eq. v2 of arXiv:2208.07731):
//
//   (V_X psi_j)(r) ~ - sum_mu V'_mu(r) sum_i phi_i(r) phi_i*(r_mu) psi_j(r_mu)
//                  = - [ (V' .* A) Psi_mu ](r, j),   A = Phi Phi_mu^H,
//
// with V'_mu = conj(V_mu) for V_mu the potential of the fit's Theta column
// (eq. v2 expands phi_i* psi_j, the conjugate of the pair density the fit
// interpolates).  Per r-block: conj(V) .* A by the Gram engine, then one
// product with the packed Psi_mu (by residues where that is faster), scaled by
// -1, into the caller's output.  FP64 results for either storage type.
#include "fitlib.h"

namespace isdf {
namespace {

// Gram epilogue: conj(V) .* A as interleaved complex rows, so that A itself is
// never stored.  64^3, 2048 points, 256 orbitals: a pass of its own over A (24
// bytes read and 16 written per entry) took 4.5 ms of 38.7 and the FP64 product
// behind it 17.2; this epilogue costs nothing that can be told from the clock's
// drift, and the residue product takes 14 (split 7.3, int8 products 5.8).
// Multiplying by V as the rows are split instead: 8.0 for the split, 34.5 in all
// against 32.8.
template <class TS>
struct EpiExch {
  double* out;
  int64_t ldo;
  const TS* V;  // row 0 of the block
  int64_t ld_v;
  int v_complex;
  int M, n_mu;
  // With V for all of a wave's tiles in flight the loads cost one latency instead
  // of one per tile (22.0 -> 21.0 ms for the whole product at 64^3 x 2048).
  template <class Cfg, bool CPLX, class Acc>
  __device__ __forceinline__ void scaled(const Acc (&acc)[Cfg::MI][Cfg::NI], const TileAt& at) const {
    constexpr int IG = CPLX ? 1 : Cfg::MI;  // rows of tiles in flight (complex V: twice the registers)
#pragma unroll
    for (int i0 = 0; i0 < Cfg::MI; i0 += IG) {
      double v[IG][Cfg::NI / 2][4], w[CPLX ? IG : 1][Cfg::NI / 2][4];
#pragma unroll
      for (int i = 0; i < IG; ++i)
#pragma unroll
        for (int jp = 0; jp < Cfg::NI / 2; ++jp)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int nu = ((at.n_wave + 32 * jp) >> 5) * 16 + (at.lane & 15);
            const int m = at.m_wave + (i0 + i) * 16 + Cfg::orow(at.lane, r);
            const int64_t e = (int64_t)(m < M ? m : M - 1) * ld_v + (nu < n_mu ? nu : n_mu - 1);
            if constexpr (CPLX) {
              const double2 z = Cplx<TS>::load(V + 2 * e);
              v[i][jp][r] = z.x;
              w[i][jp][r] = z.y;
            } else {
              v[i][jp][r] = (double)V[e];
            }
          }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < IG; ++i)
#pragma unroll
        for (int jp = 0; jp < Cfg::NI / 2; ++jp)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int nu = ((at.n_wave + 32 * jp) >> 5) * 16 + (at.lane & 15);
            const int m = at.m_wave + (i0 + i) * 16 + Cfg::orow(at.lane, r);
            if (m >= M || nu >= n_mu) continue;
            const double x = acc[i0 + i][2 * jp][r], y = acc[i0 + i][2 * jp + 1][r], a = v[i][jp][r];
            double2 o = make_double2(a * x, a * y);
            if constexpr (CPLX) {
              const double c = w[i][jp][r];
              o = make_double2(x * a + y * c, y * a - x * c);
            }
            *reinterpret_cast<double2*>(out + (int64_t)m * ldo + 2 * nu) = o;
          }
    }
  }
  template <class Cfg, class Acc>
  __device__ __forceinline__ void apply(const Acc (&acc)[Cfg::MI][Cfg::NI], const TileAt& at) const {
    if (v_complex) scaled<Cfg, true>(acc, at);
    else scaled<Cfg, false>(acc, at);
  }
};

struct ExchPlan {
  int* ab;
  double* Ephi;
  double* Fpsi;
  double* A;
  ModWork mod;  // residues of the product with Psi_mu
  size_t bytes;
};

static ExchPlan plan_exch(void* ws, size_t cap, int n_mu, int n_phi, int n_psi, int64_t rblock) {
  Carver c(ws, cap);
  ExchPlan P{};
  const int nmu16 = (int)ceil_div(n_mu, 16) * 16;
  P.ab = c.take<int>(64);
  P.Ephi = c.take<double>((size_t)2 * nmu16 * 2 * n_phi);
  P.Fpsi = c.take<double>((size_t)2 * n_psi * 2 * n_mu);
  P.A = c.take<double>((size_t)rblock * 2 * n_mu);
  P.mod = carve_mod_c(c, rblock, n_psi, n_mu);
  P.bytes = c.used;
  return P;
}

static unsigned grid_for(int64_t n) {
  int64_t b = ceil_div(n, 256);
  return (unsigned)(b > 8192 ? 8192 : (b < 1 ? 1 : b));
}

template <class TS>
static int exch_run(int64_t nr, const TS* phi, int64_t ld_phi, int n_phi, const TS* psi, int64_t ld_psi, int n_psi,
                    const int32_t* idx, int n_mu, const TS* V, int64_t ld_v, int v_complex, TS* W, int64_t ld_w,
                    int64_t rblock, const ExchPlan& P, hipStream_t s) {
  const int nmu16 = (int)ceil_div(n_mu, 16) * 16;
  if (!fill<int>(P.ab, 1, 0, s)) return ISDF_E_HIP;
  if (!pack<TS, double>(phi, ld_phi, n_phi, idx, n_mu, nr, nmu16, P.Ephi, s)) return ISDF_E_HIP;
  hipLaunchKernelGGL((pack_adj_rhs<TS, double>), dim3(grid_for((int64_t)4 * n_psi * n_mu)), dim3(256), 0, s, psi,
                     ld_psi, n_psi, idx, n_mu, nr, P.Fpsi);
  if (!launch_ok()) return ISDF_E_HIP;
  const int64_t two_mu = 2 * (int64_t)n_mu;
  for (int64_t r = 0; r < nr; r += rblock) {
    const int rows = (int)(nr - r < rblock ? nr - r : rblock);
    // conj(V) .* A, A rows = Phi(r) Phi_mu^H
    EpiExch<TS> epi{P.A, two_mu, V + (v_complex ? 2 : 1) * r * ld_v, ld_v, v_complex, rows, n_mu};
    Operand<TS> a{phi + 2 * r * ld_phi, 2 * ld_phi, nullptr, nullptr};
    Operand<double> b{P.Ephi, 2 * (int64_t)n_phi, nullptr, nullptr};
    const int64_t k = 2 * (int64_t)n_phi;
    const bool ok = tile_for(rows, 2 * nmu16, 0) < 128
                        ? launch_gemm<double, 64, 64, 16, 2, 2, TS, KC, double, KC, 1>(rows, 2 * nmu16, k, a, b, a, b, 0,
                                                                                       epi, 0, P.ab, s)
                        : launch_gemm<double, 128, 128, 16, 2, 2, TS, KC, double, KC, 1>(rows, 2 * nmu16, k, a, b, a, b,
                                                                                         0, epi, 0, P.ab, s);
    if (!ok) return ISDF_E_HIP;
    // W rows = -(conj(V) .* A) Psi_mu; the even rows of the packed Psi_mu are the
    // columns of conj(Psi_mu), so by residues it is the product with B^H
    if (!nt_product<TS>(rows, 2 * n_psi, (int)two_mu, (const double*)P.A, two_mu, (const double*)P.Fpsi, two_mu,
                        MOD_MEANS, W + 2 * r * ld_w, 2 * ld_w, -1.0, P.mod, r > 0, P.ab, s))
      return ISDF_E_HIP;
  }
  return ISDF_OK;
}

}  // namespace
}  // namespace isdf

using namespace isdf;

extern "C" size_t isdf_exchange_workspace(const isdf_grid* grid, int32_t n_mu, int32_t n_phi, int32_t n_psi,
                                          int64_t rblock) {
  if (!grid || n_mu <= 0 || n_phi <= 0 || n_psi <= 0 || rblock <= 0) return 0;
  for (int a = 0; a < 3; ++a)
    if (grid->n[a] <= 0) return 0;
  const int64_t nr = (int64_t)grid->n[0] * grid->n[1] * grid->n[2];
  if (rblock > nr) rblock = nr;
  return plan_exch(nullptr, 0, n_mu, n_phi, n_psi, rblock).bytes;
}

extern "C" int isdf_exchange(const isdf_grid* grid, int32_t dt_in, const void* phi, int64_t ld_phi, int32_t n_phi,
                             const void* psi, int64_t ld_psi, int32_t n_psi, const int32_t* idx, int32_t n_mu,
                             const void* V, int64_t ld_v, int32_t v_complex, void* W, int64_t ld_w, int64_t rblock,
                             void* ws, size_t ws_bytes, void* stream) {
  if (!dtype_valid(dt_in)) return ISDF_E_ARG;
  const isdf_dtype dt = (isdf_dtype)dt_in;
  int64_t nr = 0;
  if (!fit_args_ok(grid, dt, phi, ld_phi, n_phi, psi, ld_psi, n_psi, idx, n_mu, ISDF_P_FP64, &nr)) return ISDF_E_ARG;
  if (!V || !W || ld_v < n_mu || ld_w < n_psi || rblock <= 0) return ISDF_E_ARG;
  if (rblock > nr) rblock = nr;
  ExchPlan P = plan_exch(ws, ws_bytes, n_mu, n_phi, n_psi, rblock);
  if (!ws || P.bytes > ws_bytes) return ISDF_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  if (dt == ISDF_C128)
    return exch_run<double>(nr, (const double*)phi, ld_phi, n_phi, (const double*)psi, ld_psi, n_psi, idx, n_mu,
                            (const double*)V, ld_v, v_complex, (double*)W, ld_w, rblock, P, s);
  return exch_run<float>(nr, (const float*)phi, ld_phi, n_phi, (const float*)psi, ld_psi, n_psi, idx, n_mu,
                         (const float*)V, ld_v, v_complex, (float*)W, ld_w, rblock, P, s);
}
