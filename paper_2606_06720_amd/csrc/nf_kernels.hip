// HIP kernels (gfx950, FP64) of the per-time-step hot path:
//   * row passes   -- the x-direction real transforms, fused with the pointwise
//                     work that needs physical values (flux K grad p, activation,
//                     relaxation, energy terms), transposing to column-major;
//   * column passes -- the y-direction complex transforms of the packed
//                     half spectrum, fused with the spectral multipliers
//                     (gradient, divergence, preconditioner, heat kernel) and the
//                     PCG vector updates / inner products.
//
// Data layout (2D, n = Nx*Ny, H = Nx/2):
//   physical   f[y][x]                 (double, x fastest, caller-owned)
//   mixed      M[kx][y]  kx < H        (complex, after the x transform)
//   spectral   F[kx][ky] kx < H        (complex, after both transforms)
// Column kx = 0 packs the real kx = 0 and kx = Nx/2 columns as X0 + i X_{Nx/2}.
// Every multiplier used on it (first-derivative wavenumbers with the Nyquist
// entry zeroed, preconditioner) is identical for both packed halves; the heat
// kernel, which differs, unpacks the pair (ky, -ky) first.
//
// Spectral vectors hold the unnormalised DFT of the physical field.  Inner
// products are sum_k w_k Re(a conj b) with w = 1 on the packed column and 2
// elsewhere, which is n times the physical Euclidean product (Parseval).
#include <hip/hip_runtime.h>

#include <climits>

#include "nf_fft.hpp"
#include "nf_internal.h"
#include "nf_tiles.hpp"

namespace nf {

// ================================================================ small kernels
__device__ __forceinline__ void k_status_reset_one(DevStatus* st, int full) {
  if (threadIdx.x == 0) {
    if (full) st->sticky = 0;
    for (int i = 0; i < 8; ++i) st->kbar[i] = 0.0;
    st->bb = 0.0;
    st->rho[0] = st->rho[1] = 0.0;
    st->alpha[0] = st->alpha[1] = 0.0;
    st->rr[0] = st->rr[1] = 0.0;
    st->rr0 = 0.0;
    st->orr = st->obb = st->rscale = 0.0;
    st->orr_prev = __builtin_inf();
    st->outer_done = 0;
    st->itot = 0;
    st->budget = INT_MAX;
    for (int i = 0; i < 16; ++i) st->out[i] = 0.0;
    st->conv_at = INT_MAX;
    st->converged = 0;
    st->iters = 0;
    st->flags = 0;
    st->team = TEAM_NONE;
    st->lost = 0;
  }
}
// open the formation of the team a loop start may be followed by
__device__ __forceinline__ void team_open(const Geo& g) {
  if (g.team == nullptr) return;
  ((TeamCtl*)g.team)->tickets = 0;
  ((TeamCtl*)g.team)->state = TEAM_OPEN;
  g.st->team = TEAM_NONE;
  g.st->lost = 0;
}

__global__ void k_status_reset(DevStatus* st, int full) {
  if (blockIdx.x == 0) k_status_reset_one(st, full);
}
__global__ void kb_status_reset(DevStatus* st0, int full) { k_status_reset_one(st0 + blockIdx.x, full); }
__global__ void k_zero(cd* p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = mk<double>(0.0, 0.0);
}

__device__ __forceinline__ void sum_slot_body(const double* __restrict__ slot, int K, int n, int o, DevStatus* st) {
  __shared__ double scratch[8 * 4];
  double v[8];
  for (int k = 0; k < 8; ++k) v[k] = 0.0;
  for (int k = 0; k < K; ++k)
    for (int i = threadIdx.x; i < n; i += 256) v[k] += slot[(size_t)k * MAX_WG + i];
  block_sum<256, 8>(v, scratch);
  if (threadIdx.x == 0)
    for (int k = 0; k < K; ++k) st->out[o + k] = v[k];
}
__global__ void __launch_bounds__(256) k_sum_slot(const double* __restrict__ slot, int K, int n, int o, DevStatus* st) {
  sum_slot_body(slot, K, n, o, st);
}
__global__ void __launch_bounds__(256) kb_sum_slot(const SumArgs* __restrict__ A, int K, int n, int o) {
  sum_slot_body(A[blockIdx.y].slot, K, n, o, A[blockIdx.y].st);
}

// ================================================================ row kernels
// physical -> mixed; optional partials sum f, sum |f| (compatibility of S)
template <int NX>
__device__ __forceinline__ void row_r2c_body(Geo g, const double* __restrict__ f, cd* __restrict__ out,
                                                 double* schk) {
  using C = Row2D<NX, 1>;
  __shared__ cd buf[C::NB * C::LS];
  __shared__ double red[2 * (C::NT / 64)];
  const cd* tw = (const cd*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  double2 v[C::EP];
  rowP_gload<C>(v, f, y0, nrow);
  double s[2] = {0.0, 0.0};
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    if (p < C::RH) {
      buf[(p / C::H) * C::LS + p % C::H] = mk<double>(v[i].x, v[i].y);
      s[0] += v[i].x + v[i].y;
      s[1] += fabs(v[i].x) + fabs(v[i].y);
    }
  }
  __syncthreads();
  lds_fft<double, -1, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  rfft_post<double, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  rowT_store<C, 1>(buf, out, nullptr, nullptr, g.ny, y0, nrow);
  if (schk) {
    block_sum<C::NT, 2>(s, red);
    write_partials<C::NT>(schk, s, 2);
  }
}
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 1>::NT)) k_row_r2c(Geo g, const double* __restrict__ f, cd* __restrict__ out,
                                                 double* schk) {
  row_r2c_body<NX>(g, f, out, schk);
}
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 1>::NT)) kb_row_r2c(const RowR2cArgs* __restrict__ A) {
  const RowR2cArgs& a = A[blockIdx.y];
  row_r2c_body<NX>(a.g, (const double*)a.f, (cd*)a.out, (double*)a.schk);
}

// mixed -> physical (unnormalised inverse: the caller folds 1/n into the spectral side)
template <int NX>
__device__ __forceinline__ void row_c2r_body(Geo g, const cd* __restrict__ in, double* __restrict__ f) {
  using C = Row2D<NX, 1>;
  __shared__ cd buf[C::NB * C::LS];
  const cd* tw = (const cd*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  cd tv[C::ET];
  rowT_gload<C>(tv, in, nullptr, nullptr, g.ny, y0, nrow);
  rowT_put<C>(buf, tv);
  __syncthreads();
  irfft_pre<double, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  lds_fft<double, +1, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  for (int p = threadIdx.x; p < C::RH; p += C::NT) {
    const int rr = p / C::H, j = p % C::H;
    if (rr < nrow) {
      const cd v = buf[rr * C::LS + j];
      *(double2*)(f + (size_t)(y0 + rr) * NX + 2 * j) = make_double2(v.x, v.y);
    }
  }
}
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 1>::NT)) k_row_c2r(Geo g, const cd* __restrict__ in, double* __restrict__ f) {
  row_c2r_body<NX>(g, in, f);
}
// the pressure of a split update written out on its own (see launch_row_split)
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 1>::NT)) kb_row_split_p(const SplitArgs* __restrict__ A) {
  const SplitArgs& a = A[blockIdx.y];
  row_c2r_body<NX>(a.g, (const cd*)a.P, (double*)a.p_out);
}

// Split update, pointwise part: p = F^-1 x_hat (written out), g = grad p,
// exact activation then exact relaxation of m, forward x transform of the
// result.  In place: P, Gx hold the transformed m_x, m_y on exit.
// WITHP: the three fields (P, Gx, Gy) in one tile, p written here; otherwise
// only Gx, Gy (p is written by a pass of its own before), in the two-row tile
// SplitCfg: rows of 2048 and more hold one row per workgroup with three fields
// (16-byte runs through the mixed layout) but two with two.
template <int NX>
using SplitCfg = RowCfg<NX, 2, NX, 0, ((NX / 8) * 2 >= 1024 ? 2 : 1)>;
template <int NX>
constexpr bool split_separate_p() { return Row2D<NX, 3>::R < 2 && (NX & (NX - 1)) == 0; }
template <int NX, bool WITHP>
using SplitTile = typename std::conditional<WITHP, Row2D<NX, 3>, SplitCfg<NX>>::type;
template <int NX, bool WITHP>
__device__ __forceinline__ void row_split_body(Geo g, cd* P, cd* Gx, const cd* __restrict__ Gy,
                                                   const double* __restrict__ m, double* __restrict__ p_out,
                                                   double c2dt, double gamma, double dt, double relax1) {
  using C = SplitTile<NX, WITHP>;
  constexpr int OFF = WITHP ? C::R : 0;  // first line of Gx
  __shared__ cd buf[C::NB * C::LS];
  const cd* tw = (const cd*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  const size_t n = (size_t)g.nx * g.ny;
  cd tv[C::ET];
  if constexpr (WITHP)
    rowT_gload<C>(tv, P, Gx, Gy, g.ny, y0, nrow);
  else
    rowT_gload<C>(tv, Gx, Gy, nullptr, g.ny, y0, nrow);
  double2 mxv[C::EP], myv[C::EP];
  rowP_gload<C>(mxv, m, y0, nrow);
  rowP_gload<C>(myv, m + n, y0, nrow);
  rowT_put<C>(buf, tv);
  __syncthreads();
  irfft_pre<double, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  lds_fft<double, +1, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);

  const double e1 = 1.0 - gamma;
  bool bad = false;
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int rr = p / C::H, j = p % C::H;
    if (p < C::RH && rr < nrow) {
      // m_x and m_y replace the first two fields' lines
      cd* pp = buf + rr * C::LS + j;
      cd* px = buf + (C::R + rr) * C::LS + j;
      const cd gxv = buf[(OFF + rr) * C::LS + j], gyv = buf[(OFF + C::R + rr) * C::LS + j];
      if constexpr (WITHP) {
        const cd pv = *pp;
        *(double2*)(p_out + (size_t)(y0 + rr) * NX + 2 * j) = make_double2(pv.x, pv.y);
      }
      double mx[2] = {mxv[i].x, mxv[i].y}, my[2] = {myv[i].x, myv[i].y};
      const double gxa[2] = {gxv.x, gxv.y}, gya[2] = {gyv.x, gyv.y};
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        // activation: m + c^2 dt phi1(c^2 dt |g|^2) (g.m) g, phi1(z) = expm1(z)/z
        const double g2 = gxa[t] * gxa[t] + gya[t] * gya[t];
        const double z = c2dt * g2;
        const double phi = z > 0.0 ? expm1(z) / z : 1.0;
        const double coef = c2dt * phi * (gxa[t] * mx[t] + gya[t] * my[t]);
        double qx = fma(coef, gxa[t], mx[t]);
        double qy = fma(coef, gya[t], my[t]);
        // relaxation: exact decay of |m| along m/|m|
        double fac;
        if (gamma == 1.0) {
          fac = relax1;
        } else {
          const double s2 = qx * qx + qy * qy;
          if (s2 == 0.0) {
            fac = 1.0;
          } else {
            const double u = 2.0 * e1 * dt * exp(-e1 * log(s2));
            fac = (u >= 1.0) ? 0.0 : exp(log1p(-u) / (2.0 * e1));
          }
        }
        qx *= fac;
        qy *= fac;
        if (!isfinite(qx) || !isfinite(qy)) bad = true;
        mx[t] = qx;
        my[t] = qy;
      }
      *pp = mk<double>(mx[0], mx[1]);
      *px = mk<double>(my[0], my[1]);
    }
  }
  if (bad) atomicOr(&g.st->sticky, (int)FLAG_NONFINITE);
  __syncthreads();
  lds_fft<double, -1, C::H, 2 * C::R, C::LS, C::NT>(buf, tw, g.twn);
  rfft_post<double, C::H, 2 * C::R, C::LS, C::NT>(buf, tw, g.twn);
  rowT_store<C, 2>(buf, P, Gx, nullptr, g.ny, y0, nrow);
}
template <int NX, bool WITHP>
__global__ void __launch_bounds__((SplitTile<NX, WITHP>::NT)) k_row_split(Geo g, cd* P, cd* Gx, const cd* __restrict__ Gy,
                                                   const double* __restrict__ m, double* __restrict__ p_out,
                                                   double c2dt, double gamma, double dt, double relax1) {
  row_split_body<NX, WITHP>(g, P, Gx, Gy, m, p_out, c2dt, gamma, dt, relax1);
}
template <int NX, bool WITHP>
__global__ void __launch_bounds__((SplitTile<NX, WITHP>::NT)) kb_row_split(const SplitArgs* __restrict__ A) {
  const SplitArgs& a = A[blockIdx.y];
  row_split_body<NX, WITHP>(a.g, (cd*)a.P, (cd*)a.Gx, (const cd*)a.Gy, (const double*)a.m, (double*)a.p_out, a.c2dt, a.gamma, a.dt, a.relax1);
}

// Last pass of the step: inverse x transform of the diffused m, written over
// m; partials sum (m_new - m_old)^2 and sum m_old^2.
template <int NX>
__device__ __forceinline__ void row_final_body(Geo g, const cd* __restrict__ Mx, const cd* __restrict__ My,
                                                   double* m, double* dslot) {
  using C = Row2D<NX, 2>;
  __shared__ cd buf[C::NB * C::LS];
  __shared__ double red[2 * (C::NT / 64)];
  const cd* tw = (const cd*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  const size_t n = (size_t)g.nx * g.ny;
  cd tv[C::ET];
  rowT_gload<C>(tv, Mx, My, nullptr, g.ny, y0, nrow);
  double2 o0[C::EP], o1[C::EP];
  rowP_gload<C>(o0, m, y0, nrow);
  rowP_gload<C>(o1, m + n, y0, nrow);
  rowT_put<C>(buf, tv);
  __syncthreads();
  irfft_pre<double, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  lds_fft<double, +1, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  double s[2] = {0.0, 0.0};
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int rr = p / C::H, j = p % C::H;
    if (p < C::RH && rr < nrow) {
      const cd a0 = buf[rr * C::LS + j], a1 = buf[(C::R + rr) * C::LS + j];
      const size_t idx = (size_t)(y0 + rr) * NX + 2 * j;
      const double d0 = a0.x - o0[i].x, d1 = a0.y - o0[i].y;
      const double d2 = a1.x - o1[i].x, d3 = a1.y - o1[i].y;
      s[0] += d0 * d0 + d1 * d1 + d2 * d2 + d3 * d3;
      s[1] += o0[i].x * o0[i].x + o0[i].y * o0[i].y + o1[i].x * o1[i].x + o1[i].y * o1[i].y;
      *(double2*)(m + idx) = make_double2(a0.x, a0.y);
      *(double2*)(m + n + idx) = make_double2(a1.x, a1.y);
    }
  }
  if (dslot) {
    block_sum<C::NT, 2>(s, red);
    write_partials<C::NT>(dslot, s, 2);
  }
}
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 2>::NT)) k_row_final(Geo g, const cd* __restrict__ Mx, const cd* __restrict__ My,
                                                   double* m, double* dslot) {
  row_final_body<NX>(g, Mx, My, m, dslot);
}
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 2>::NT)) kb_row_final(const FinalArgs* __restrict__ A) {
  const FinalArgs& a = A[blockIdx.y];
  row_final_body<NX>(a.g, (const cd*)a.Mx, (const cd*)a.My, (double*)a.m, (double*)a.dslot);
}

// Pointwise energy terms: sum r|g|^2, sum (m.g)^2, sum |m|^{2 gamma}
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 2>::NT)) k_row_energy(Geo g, const cd* __restrict__ Gx, const cd* __restrict__ Gy,
                                                    const double* __restrict__ m, const double* __restrict__ r,
                                                    double gamma, double* eslot) {
  using C = Row2D<NX, 2>;
  __shared__ cd buf[C::NB * C::LS];
  __shared__ double red[3 * (C::NT / 64)];
  const cd* tw = (const cd*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  const size_t n = (size_t)g.nx * g.ny;
  cd tv[C::ET];
  rowT_gload<C>(tv, Gx, Gy, nullptr, g.ny, y0, nrow);
  double2 mx[C::EP], my[C::EP], rv[C::EP];
  rowP_gload<C>(mx, m, y0, nrow);
  rowP_gload<C>(my, m + n, y0, nrow);
  rowP_gload<C>(rv, r, y0, nrow);
  rowT_put<C>(buf, tv);
  __syncthreads();
  irfft_pre<double, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  lds_fft<double, +1, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int rr = p / C::H, j = p % C::H;
    if (p < C::RH && rr < nrow) {
      const cd gxv = buf[rr * C::LS + j], gyv = buf[(C::R + rr) * C::LS + j];
      const double gxa[2] = {gxv.x, gxv.y}, gya[2] = {gyv.x, gyv.y};
      const double mxa[2] = {mx[i].x, mx[i].y}, mya[2] = {my[i].x, my[i].y}, ra[2] = {rv[i].x, rv[i].y};
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const double mg = mxa[t] * gxa[t] + mya[t] * gya[t];
        s[0] += ra[t] * (gxa[t] * gxa[t] + gya[t] * gya[t]);
        s[1] += mg * mg;
        const double mm = mxa[t] * mxa[t] + mya[t] * mya[t];
        s[2] += (mm == 0.0) ? 0.0 : exp(gamma * log(mm));
      }
    }
  }
  block_sum<C::NT, 3>(s, red);
  write_partials<C::NT>(eslot, s, 3);
}

// ================================================================ adjoint row kernels
// phi1'(z) = (e^z (z - 1) + 1) / z^2, by its Taylor series near 0
__device__ __forceinline__ double dphi1(double z) {
  if (fabs(z) < 1e-3) return 0.5 + z * (1.0 / 3.0 + z * (0.125 + z * (1.0 / 30.0)));
  return (expm1(z) * (z - 1.0) + z) / (z * z);
}

// Reverse of the pointwise part of the split update at one grid point.
// In: m (= m^k), g (= grad p^k), lam2 (= H^T lam^{k+1}, the adjoint after the
// diffusion stage).  Out: lam_m (adjoint of m through activation and
// relaxation) and lam_g (adjoint of g).
__device__ __forceinline__ void adjoint_point(double mx, double my, double gx, double gy, double lx, double ly,
                                              double c2dt, double gamma, double dt, double relax1, double& lmx,
                                              double& lmy, double& lgx, double& lgy) {
  // forward activation intermediates
  const double g2 = gx * gx + gy * gy;
  const double z = c2dt * g2;
  const double kap = c2dt * (z > 0.0 ? expm1(z) / z : 1.0);
  const double dkap = c2dt * dphi1(z);
  const double gm = gx * mx + gy * my;
  const double sx = fma(kap * gm, gx, mx), sy = fma(kap * gm, gy, my);  // m*
  // relaxation Jacobian (symmetric): fac (I - u u^T) + rho' u u^T
  double ax, ay;
  if (gamma == 1.0) {
    ax = relax1 * lx;
    ay = relax1 * ly;
  } else {
    const double s2 = sx * sx + sy * sy;
    const double e1 = 1.0 - gamma;
    if (s2 == 0.0) {
      ax = gamma > 1.0 ? lx : 0.0;
      ay = gamma > 1.0 ? ly : 0.0;
    } else {
      const double u = 2.0 * e1 * dt * exp(-e1 * log(s2));
      if (u >= 1.0) {
        ax = ay = 0.0;
      } else {
        const double fac = exp(log1p(-u) / (2.0 * e1));   // rho / s
        const double drho = exp((1.0 - 2.0 * e1) * log(fac));  // rho'(s) = (s/rho)^{2e-1}
        const double is = 1.0 / sqrt(s2);
        const double ux = sx * is, uy = sy * is;
        const double ul = ux * lx + uy * ly;
        ax = fac * (lx - ux * ul) + drho * ul * ux;
        ay = fac * (ly - uy * ul) + drho * ul * uy;
      }
    }
  }
  // activation: d m*/d m = I + kap g g^T;  d m*/d g as in the oracle
  const double gl = gx * ax + gy * ay;
  lmx = fma(kap * gl, gx, ax);
  lmy = fma(kap * gl, gy, ay);
  const double t = 2.0 * c2dt * dkap * gm * gl;
  lgx = t * gx + kap * gl * mx + kap * gm * ax;
  lgy = t * gy + kap * gl * my + kap * gm * ay;
}

// Adjoint, first pass: c2r of (H lam_x, H lam_y, grad_x p, grad_y p); the
// pointwise reverse of relaxation and activation; lam_m written to lam_out,
// lam_g transformed forward back into A0 / A1 (in place).
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 4>::NT)) k_row_adj1(Geo g, cd* A0, cd* A1, const cd* __restrict__ G0,
                                                      const cd* __restrict__ G1, const double* __restrict__ m,
                                                      double* __restrict__ lam_out, double c2dt, double gamma,
                                                      double dt, double relax1) {
  using C = Row2D<NX, 4>;
  __shared__ cd buf[C::NB * C::LS];
  const cd* tw = (const cd*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  const size_t n = (size_t)g.nx * g.ny;
  cd tv[C::ET];
#pragma unroll
  for (int i = 0; i < C::ET; ++i) {
    const int e = threadIdx.x + i * C::NT;
    const int f = e / C::RH, ee = e % C::RH;
    const int rr = ee % C::R, kx = ee / C::R;
    const cd* src = f == 0 ? A0 : (f == 1 ? A1 : (f == 2 ? G0 : G1));
    tv[i] = (e < 4 * C::RH && rr < nrow) ? src[(size_t)kx * g.ny + y0 + rr] : mk<double>(0.0, 0.0);
  }
  double2 mx[C::EP], my[C::EP];
  rowP_gload<C>(mx, m, y0, nrow);
  rowP_gload<C>(my, m + n, y0, nrow);
  rowT_put<C>(buf, tv);
  __syncthreads();
  irfft_pre<double, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  lds_fft<double, +1, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int rr = p / C::H, j = p % C::H;
    if (p < C::RH && rr < nrow) {
      cd* plx = buf + rr * C::LS + j;
      cd* ply = buf + (C::R + rr) * C::LS + j;
      const cd lx = *plx, ly = *ply;
      const cd gxv = buf[(2 * C::R + rr) * C::LS + j], gyv = buf[(3 * C::R + rr) * C::LS + j];
      double lm[2][2], lg[2][2];
      adjoint_point(mx[i].x, my[i].x, gxv.x, gyv.x, lx.x, ly.x, c2dt, gamma, dt, relax1, lm[0][0], lm[1][0], lg[0][0],
                    lg[1][0]);
      adjoint_point(mx[i].y, my[i].y, gxv.y, gyv.y, lx.y, ly.y, c2dt, gamma, dt, relax1, lm[0][1], lm[1][1], lg[0][1],
                    lg[1][1]);
      const size_t idx = (size_t)(y0 + rr) * NX + 2 * j;
      *(double2*)(lam_out + idx) = make_double2(lm[0][0], lm[0][1]);
      *(double2*)(lam_out + n + idx) = make_double2(lm[1][0], lm[1][1]);
      *plx = mk<double>(lg[0][0], lg[0][1]);
      *ply = mk<double>(lg[1][0], lg[1][1]);
    }
  }
  __syncthreads();
  lds_fft<double, -1, C::H, 2 * C::R, C::LS, C::NT>(buf, tw, g.twn);
  rfft_post<double, C::H, 2 * C::R, C::LS, C::NT>(buf, tw, g.twn);
  rowT_store<C, 2>(buf, A0, A1, nullptr, g.ny, y0, nrow);
}

// Adjoint, second pass: c2r of (grad mu, grad p); with mu (physical) and m:
// dL/dS += mu, dL/dr -= grad mu . grad p, and
// lam -= (m.grad p) grad mu + (m.grad mu) grad p.
template <int NX>
__global__ void __launch_bounds__((Row2D<NX, 4>::NT)) k_row_adj2(Geo g, const cd* __restrict__ M1, const cd* __restrict__ M2,
                                                      const cd* __restrict__ P1, const cd* __restrict__ P2,
                                                      const double* __restrict__ m, const double* __restrict__ mu,
                                                      double* lam, double* grad_r, double* grad_S) {
  using C = Row2D<NX, 4>;
  __shared__ cd buf[C::NB * C::LS];
  const cd* tw = (const cd*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  const size_t n = (size_t)g.nx * g.ny;
  cd tv[C::ET];
#pragma unroll
  for (int i = 0; i < C::ET; ++i) {
    const int e = threadIdx.x + i * C::NT;
    const int f = e / C::RH, ee = e % C::RH;
    const int rr = ee % C::R, kx = ee / C::R;
    const cd* src = f == 0 ? M1 : (f == 1 ? M2 : (f == 2 ? P1 : P2));
    tv[i] = (e < 4 * C::RH && rr < nrow) ? src[(size_t)kx * g.ny + y0 + rr] : mk<double>(0.0, 0.0);
  }
  double2 mx[C::EP], my[C::EP], muv[C::EP];
  rowP_gload<C>(mx, m, y0, nrow);
  rowP_gload<C>(my, m + n, y0, nrow);
  rowP_gload<C>(muv, mu, y0, nrow);
  rowT_put<C>(buf, tv);
  __syncthreads();
  irfft_pre<double, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  lds_fft<double, +1, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int rr = p / C::H, j = p % C::H;
    if (p < C::RH && rr < nrow) {
      const cd umx = buf[rr * C::LS + j], umy = buf[(C::R + rr) * C::LS + j];
      const cd upx = buf[(2 * C::R + rr) * C::LS + j], upy = buf[(3 * C::R + rr) * C::LS + j];
      const size_t idx = (size_t)(y0 + rr) * NX + 2 * j;
      double2 gS = *(const double2*)(grad_S + idx);
      double2 gr = *(const double2*)(grad_r + idx);
      double2 l0 = *(const double2*)(lam + idx);
      double2 l1 = *(const double2*)(lam + n + idx);
      gS.x += muv[i].x;
      gS.y += muv[i].y;
      gr.x -= umx.x * upx.x + umy.x * upy.x;
      gr.y -= umx.y * upx.y + umy.y * upy.y;
      const double mgp0 = mx[i].x * upx.x + my[i].x * upy.x, mgp1 = mx[i].y * upx.y + my[i].y * upy.y;
      const double mgm0 = mx[i].x * umx.x + my[i].x * umy.x, mgm1 = mx[i].y * umx.y + my[i].y * umy.y;
      l0.x -= mgp0 * umx.x + mgm0 * upx.x;
      l0.y -= mgp1 * umx.y + mgm1 * upx.y;
      l1.x -= mgp0 * umy.x + mgm0 * upy.x;
      l1.y -= mgp1 * umy.y + mgm1 * upy.y;
      *(double2*)(grad_S + idx) = gS;
      *(double2*)(grad_r + idx) = gr;
      *(double2*)(lam + idx) = l0;
      *(double2*)(lam + n + idx) = l1;
    }
  }
}

// ================================================================ column kernels
// Write the gradient multipliers i xi_c f_hat / n of one spectral value into
// the two gradient lines of the column block.
template <class C, typename T>
__device__ __forceinline__ void put_grad(cx<T>* buf, int c, int ky, int kx, const cx<T> v, const Geo& g) {
  constexpr int NY = C::NYv;
  const T sx = (T)(xi_col(kx, g.lx) * g.inv_n), sy = (T)(xi_tilde(ky, NY, g.ly) * g.inv_n);
  buf[c * C::LS + ky] = mk<T>(-sx * v.y, sx * v.x);
  buf[(C::C + c) * C::LS + ky] = mk<T>(-sy * v.y, sy * v.x);
}

// mixed -> spectral (null modes zeroed unless bit 1 of mode is set); with bit 0
// of mode also the gradient of the result back to mixed:
// Gx = F_y^-1(i xi_x f_hat / n), Gy likewise.
template <int NY>
__device__ __forceinline__ void col_fwd_body(Geo g, cd* in, cd* __restrict__ out, int mode, cd* Gx, cd* Gy) {
  using C = ColCfg<NY, 2>;
  __shared__ cd buf[C::NB * C::LS];
  const cd* tw = (const cd*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  cd tv[C::ET];
  colT_gload<C, 1>(tv, in, nullptr, kx0, g.h);
  colT_put<C, 1>(buf, tv);
  __syncthreads();
  lds_fft<double, -1, NY, C::C, C::LS, C::NT>(buf, tw, g.twn);
  cd v[C::EP];
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int c = p / NY, ky = p % NY;
    cd a = p < C::CN ? buf[c * C::LS + ky] : mk<double>(0.0, 0.0);
    if (!(mode & 2) && kx0 + c == 0 && (ky == 0 || 2 * ky == NY)) a = mk<double>(0.0, 0.0);
    v[i] = a;
    if (p < C::CN && kx0 + c < g.h) out[(size_t)(kx0 + c) * NY + ky] = a;
  }
  if (!(mode & 1)) return;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    if (p < C::CN) put_grad<C>(buf, p / NY, p % NY, kx0 + p / NY, v[i], g);
  }
  __syncthreads();
  lds_fft<double, +1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  colT_store<C, 2>(buf, Gx, Gy, kx0, g.h);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) k_col_fwd(Geo g, cd* in, cd* __restrict__ out, int mode, cd* Gx, cd* Gy) {
  col_fwd_body<NY>(g, in, out, mode, Gx, Gy);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) kb_col_fwd(const ColFwdArgs* __restrict__ A, int mode) {
  const ColFwdArgs& a = A[blockIdx.y];
  col_fwd_body<NY>(a.g, (cd*)a.in, (cd*)a.out, mode, (cd*)a.Gx, (cd*)a.Gy);
}

// spectral -> mixed: P = F_y^-1(x_hat / n)  (GRAD false)  or
//                    Gx, Gy as in k_col_fwd (GRAD true)
template <int NY, bool GRAD>
__device__ __forceinline__ void col_grad_body(Geo g, const cd* __restrict__ xh, cd* P, cd* Gx,
                                                               cd* Gy) {
  using C = ColCfg<NY, GRAD ? 2 : 1>;
  __shared__ cd buf[C::NB * C::LS];
  const cd* tw = (const cd*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  cd v[C::EP];
  colP_gload<C>(v, xh, kx0, g.h);
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    if (p < C::CN) {
      if (GRAD) put_grad<C>(buf, p / NY, p % NY, kx0 + p / NY, v[i], g);
      else buf[(p / NY) * C::LS + p % NY] = scl(v[i], g.inv_n);
    }
  }
  __syncthreads();
  lds_fft<double, +1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  if (GRAD) colT_store<C, 2>(buf, Gx, Gy, kx0, g.h);
  else colT_store<C, 1>(buf, P, nullptr, kx0, g.h);
}
template <int NY, bool GRAD>
__global__ void __launch_bounds__((ColCfg<NY, GRAD ? 2 : 1>::NT)) k_col_grad(Geo g, const cd* __restrict__ xh, cd* P, cd* Gx,
                                                               cd* Gy) {
  col_grad_body<NY, GRAD>(g, xh, P, Gx, Gy);
}
template <int NY, bool GRAD>
__global__ void __launch_bounds__((ColCfg<NY, GRAD ? 2 : 1>::NT)) kb_col_grad(const ColGradArgs* __restrict__ A) {
  const ColGradArgs& a = A[blockIdx.y];
  col_grad_body<NY, GRAD>(a.g, (const cd*)a.xh, (cd*)a.P, (cd*)a.Gx, (cd*)a.Gy);
}


// Operator end outside the loop: forward y transform of the fluxes, q_hat = -i xi . F_hat.
// INIT: r_hat = b_hat - q_hat (stored), partials <r,M^-1 r>, <r,r>, <b,b>;
//       also reduces the Kbar and compatibility partials of the row pass.
// else: q_hat stored (operator apply).
template <int NY, bool INIT>
__device__ __forceinline__ void col_div_body(Geo g, const cd* __restrict__ Fx, const cd* __restrict__ Fy,
                                             cd* __restrict__ qh, cd* rh, const cd* __restrict__ bh, int nwg_row) {
  using C = ColCfg<NY, 2>;
  if (INIT && g.st->outer_done != 0) return;
  __shared__ cd buf[C::NB * C::LS];
  __shared__ double red[4 * (C::NT / 64)];
  __shared__ double Ks[4];
  const cd* tw = (const cd*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  cd tv[C::ET];
  colT_gload<C, 2>(tv, Fx, Fy, kx0, g.h);
  if (INIT) {
    double kb[4], sc[2];
    sum_partials<C::NT, 4>(slot_ptr(g.part, SLOT_KBAR), nwg_row, MAX_WG, kb, red);
    sum_partials<C::NT, 2>(slot_ptr(g.part, SLOT_SCHK), nwg_row, MAX_WG, sc, red);
    if (threadIdx.x == 0) {
      Ks[0] = kb[0] * g.inv_n + kb[3] * g.inv_n;
      Ks[1] = kb[1] * g.inv_n;
      Ks[2] = kb[2] * g.inv_n + kb[3] * g.inv_n;
      Ks[3] = 0.0;
      if (blockIdx.x == 0) {
        for (int i = 0; i < 4; ++i) g.st->kbar[i] = Ks[i];
        if (fabs(sc[0]) > 1e-12 * sc[1]) atomicOr(&g.st->flags, (int)FLAG_INCOMPAT);
      }
    }
  }
  colT_put<C, 2>(buf, tv);
  __syncthreads();
  lds_fft<double, -1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  // b is loaded after the transform (fewer registers held across it)
  cd bv[C::EP];
  if (INIT) colP_gload<C>(bv, bh, kx0, g.h);
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int c = p / NY, ky = p % NY;
    const int kx = kx0 + c;
    if (p < C::CN && kx < g.h) {
      const cd fx = buf[c * C::LS + ky], fy = buf[(C::C + c) * C::LS + ky];
      const double xx = xi_col(kx, g.lx);
      const double yy = xi_tilde(ky, NY, g.ly);
      // q = -i (xx Fx + yy Fy)
      const double ax = xx * fx.x + yy * fy.x, ay = xx * fx.y + yy * fy.y;
      const cd q = mk<double>(ay, -ax);
      const size_t idx = (size_t)kx * NY + ky;
      if (INIT) {
        const double w = kx == 0 ? 1.0 : 2.0;
        const cd b = bv[i];
        const cd rn = sub(b, q);
        rh[idx] = rn;
        const double rr = rn.x * rn.x + rn.y * rn.y;
        s[0] += w * precond_symbol_inv(Ks, xx, yy) * rr;
        s[1] += w * rr;
        s[2] += w * (b.x * b.x + b.y * b.y);
      } else {
        qh[idx] = q;
      }
    }
  }
  if (INIT) {
    block_sum<C::NT, 3>(s, red);
    write_partials<C::NT>(slot_ptr(g.part, SLOT_P3INIT), s, 3);
  }
}
template <int NY, bool INIT>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) k_col_div(Geo g, const cd* __restrict__ Fx, const cd* __restrict__ Fy,
                                                 cd* __restrict__ qh, cd* rh, const cd* __restrict__ bh, int nwg_row) {
  col_div_body<NY, INIT>(g, Fx, Fy, qh, rh, bh, nwg_row);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) kb_col_div(const DivArgs* __restrict__ A, int nwg_row) {
  const DivArgs& a = A[blockIdx.y];
  col_div_body<NY, true>(a.g, (const cd*)a.Fx, (const cd*)a.Fy, nullptr, (cd*)a.rh, (const cd*)a.bh, nwg_row);
}

// Start of the FP64 loop: <r,M^-1 r>, ||r||^2 and ||b||^2 from the partials of the
// INIT pass, the stopping test on the initial residual, and the gradient of
// z = M^-1 r in the mixed buffers for the first row pass.
template <int NY>
__device__ __forceinline__ void col_start_body(Geo g, const cd* __restrict__ rh, cd* xh, cd* Gx, cd* Gy, int max_iter,
                                               double tol2, int nwg_col) {
  using C = ColCfg<NY, 2>;
  DevStatus* st = g.st;
  __shared__ cd buf[C::NB * C::LS];
  __shared__ double red[3 * (C::NT / 64)];
  const cd* tw = (const cd*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  double K[4];
  for (int i = 0; i < 4; ++i) K[i] = st->kbar[i];
  cd rv[C::EP];
  colP_gload<C>(rv, rh, kx0, g.h);
  double s[3];
  sum_partials<C::NT, 3>(slot_ptr(g.part, SLOT_P3INIT), nwg_col, MAX_WG, s, red);
  const double rho = s[0], rr = s[1], bb = s[2];
  const bool incompat = (st->flags & FLAG_INCOMPAT) != 0;
  bool zero_x = (bb == 0.0);
  const bool bad = !isfinite(rr) || !isfinite(bb);
  const bool conv = !bad && (incompat || zero_x || rr <= tol2 * bb);
  if (bad) zero_x = false;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    team_open(g);
    st->rho[0] = rho;
    st->rr[0] = zero_x ? 0.0 : rr;
    st->rr0 = rr;
    st->bb = bb;
    st->iters = 0;
    if (bad) st->flags |= FLAG_NONFINITE;
    if (conv || bad || max_iter <= 0) {
      st->conv_at = 0;
      st->converged = conv ? 1 : 0;
    }
  }
  if (zero_x) {
#pragma unroll
    for (int i = 0; i < C::EP; ++i) {
      const int p = threadIdx.x + i * C::NT;
      const int kx = kx0 + p / NY;
      if (p < C::CN && kx < g.h) xh[(size_t)kx * NY + p % NY] = vzero<cd>();
    }
  }
  if (conv || bad || max_iter <= 0) return;
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int c = p / NY, ky = p % NY;
    const int kx = kx0 + c;
    if (p < C::CN)
      put_grad<C>(buf, c, ky, kx, scl(rv[i], precond_symbol_inv(K, xi_col(kx, g.lx), xi_tilde(ky, NY, g.ly))), g);
  }
  __syncthreads();
  lds_fft<double, +1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  colT_store<C, 2>(buf, Gx, Gy, kx0, g.h);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) k_col_start(Geo g, const cd* __restrict__ rh, cd* xh, cd* Gx, cd* Gy,
                                                    int max_iter, double tol2, int nwg_col) {
  col_start_body<NY>(g, rh, xh, Gx, Gy, max_iter, tol2, nwg_col);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) kb_col_start(const IterArgs* __restrict__ A, int max_iter, double tol2, int nwg_col) {
  const IterArgs& a = A[blockIdx.y];
  col_start_body<NY>(a.g, (const cd*)a.rh, (cd*)a.xh, (cd*)a.M0, (cd*)a.M1, max_iter, tol2, nwg_col);
}

// Start of one correction of the mixed-precision solve (iterative refinement
// of A x = b: the inner solve A e = r runs in FP32, x and the residual
// r = b - A x in FP64).  Reads the FP64 residual partials <r,M^-1 r>, <r,r>,
// <b,b> left by the FP64 operator pass.  If ||r||^2 <= tol2 ||b||^2 (or b = 0,
// or S is incompatible, or the values are not finite) the solve is over: the
// status records the outcome and every later inner launch is a no-op.
// Otherwise the inner right-hand side is r / ||r|| in FP32, the inner
// iterate starts at 0, the gradient of M^-1 r goes to the FP32 mixed buffers
// for the first row pass, and the inner stopping threshold (a relative
// residual of tol_in on the unit right-hand side, kept in status.bb for the
// passes' test with tol2 = 1) asks for the reduction that reaches tol2 with a
// margin of 2, but no less than `floor_in`.  A residual no smaller than the
// previous correction's means the refinement has stalled: the solve ends
// unconverged, as it does when max_iter FP32 iterations have been spent.
// Instances that have finished repeat their final decision unchanged (their
// residual passes are skipped), so a batch can run until all have finished.
// Status fields read here are written only by other launches.
template <int NY>
__device__ __forceinline__ void col_refine_start_body(Geo g, const cd* __restrict__ r64, cd* x64,
                                                          cx<float>* x32, cx<float>* r32,
                                                          cx<float>* Gx, cx<float>* Gy, double tol2,
                                                          double floor_in, int max_iter, int nwg_col) {
  using C = ColCfg<NY, 2>;
  using V = cx<float>;
  DevStatus* st = g.st;
  __shared__ V buf[C::NB * C::LS];
  __shared__ double red[3 * (C::NT / 64)];
  const V* tw = (const V*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  const bool lead = (blockIdx.x == 0 && threadIdx.x == 0);
  double K[4];
  for (int i = 0; i < 4; ++i) K[i] = st->kbar[i];
  cd rv[C::EP];
  colP_gload<C>(rv, r64, kx0, g.h);
  double s[3];
  sum_partials<C::NT, 3>(slot_ptr(g.part, SLOT_P3INIT), nwg_col, MAX_WG, s, red);
  const double rho = s[0], rr = s[1], bb = s[2];
  const int budget = max_iter - st->itot;
  const double rr_cap = st->orr_prev;
  const bool incompat = (st->flags & FLAG_INCOMPAT) != 0;
  const bool bad = !isfinite(rr) || !isfinite(bb);
  const bool zero_b = !bad && bb == 0.0;
  const bool conv = !bad && (incompat || zero_b || rr <= tol2 * bb);
  if (conv || bad || budget <= 0 || rr >= rr_cap) {
    if (lead) {
      st->rr[0] = zero_b ? 0.0 : rr;
      st->bb = bb;
      st->orr = zero_b ? 0.0 : rr;
      st->obb = bb;
      if (bad) st->flags |= FLAG_NONFINITE;
      st->conv_at = 0;
      st->converged = conv ? 1 : 0;
      st->iters = 0;
      st->outer_done = 1;
      st->team = TEAM_NONE;
    }
    if (zero_b) {
#pragma unroll
      for (int i = 0; i < C::EP; ++i) {
        const int p = threadIdx.x + i * C::NT;
        const int kx = kx0 + p / NY;
        if (p < C::CN && kx < g.h) x64[(size_t)kx * NY + p % NY] = mk<double>(0.0, 0.0);
      }
    }
    return;
  }
  const double scale = 1.0 / sqrt(rr);
  double tin = 0.5 * sqrt(tol2 * bb / rr);
  tin = tin < floor_in ? floor_in : (tin > 0.5 ? 0.5 : tin);
  if (lead) {
    team_open(g);
    st->orr = rr;
    st->obb = bb;
    st->rscale = sqrt(rr);
    st->bb = tin * tin;
    st->rho[0] = rho * scale * scale;
    st->rr[0] = 1.0;
    st->rr0 = 1.0;
    st->iters = 0;
    st->budget = budget;
    st->converged = 0;
    st->conv_at = INT_MAX;
  }
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int c = p / NY, ky = p % NY;
    const int kx = kx0 + c;
    V d = vzero<V>();
    if (p < C::CN && kx < g.h) {
      const size_t idx = (size_t)kx * NY + ky;
      const double sig = precond_symbol_inv(K, xi_col(kx, g.lx), xi_tilde(ky, NY, g.ly));
      const double ux = rv[i].x * scale, uy = rv[i].y * scale;
      r32[idx] = mk<float>((float)ux, (float)uy);
      d = mk<float>((float)(sig * ux), (float)(sig * uy));
      x32[idx] = vzero<V>();
    }
    if (p < C::CN) put_grad<C>(buf, c, ky, kx, d, g);
  }
  __syncthreads();
  lds_fft<float, +1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  colT_store<C, 2>(buf, Gx, Gy, kx0, g.h);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) k_col_refine_start(Geo g, const cd* __restrict__ r64, cd* x64,
                                                          cx<float>* x32, cx<float>* r32,
                                                          cx<float>* Gx, cx<float>* Gy, double tol2,
                                                          double floor_in, int max_iter, int nwg_col) {
  col_refine_start_body<NY>(g, r64, x64, x32, r32, Gx, Gy, tol2, floor_in, max_iter, nwg_col);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) kb_col_refine_start(const RefStartArgs* __restrict__ A, double tol2, double floor_in, int max_iter, int nwg_col) {
  const RefStartArgs& a = A[blockIdx.y];
  col_refine_start_body<NY>(a.g, (const cd*)a.r64, (cd*)a.x64, (cx<float>*)a.x32, (cx<float>*)a.r32, (cx<float>*)a.Gx, (cx<float>*)a.Gy, tol2, floor_in, max_iter, nwg_col);
}

// End of one correction: x64 += ||r|| e32 (status.rscale), then the gradient
// of the new x64 into the FP64 mixed buffers for the next residual; the
// correction's FP32 iterations are added to the total.  No-op for a finished
// solve.
template <int NY>
__device__ __forceinline__ void col_refine_acc_body(Geo g, cd* x64, const cx<float>* __restrict__ x32,
                                                        cd* Gx, cd* Gy) {
  using C = ColCfg<NY, 2>;
  __shared__ cd buf[C::NB * C::LS];
  const cd* tw = (const cd*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  if (g.st->outer_done) return;
  const double sc = g.st->rscale;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    g.st->itot += g.st->iters;
    g.st->orr_prev = g.st->orr;
  }
  cd xv[C::EP];
  cx<float> ev[C::EP];
  colP_gload<C>(xv, x64, kx0, g.h);
  colP_gload<C>(ev, x32, kx0, g.h);
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int c = p / NY, ky = p % NY;
    const int kx = kx0 + c;
    cd x = mk<double>(0.0, 0.0);
    if (p < C::CN && kx < g.h) {
      x = mk<double>(fma(sc, (double)ev[i].x, xv[i].x), fma(sc, (double)ev[i].y, xv[i].y));
      x64[(size_t)kx * NY + ky] = x;
    }
    if (p < C::CN) put_grad<C>(buf, c, ky, kx, x, g);
  }
  __syncthreads();
  lds_fft<double, +1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  colT_store<C, 2>(buf, Gx, Gy, kx0, g.h);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) k_col_refine_acc(Geo g, cd* x64, const cx<float>* __restrict__ x32,
                                                        cd* Gx, cd* Gy) {
  col_refine_acc_body<NY>(g, x64, x32, Gx, Gy);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) kb_col_refine_acc(const RefAccArgs* __restrict__ A) {
  const RefAccArgs& a = A[blockIdx.y];
  col_refine_acc_body<NY>(a.g, (cd*)a.x64, (const cx<float>*)a.x32, (cd*)a.Gx, (cd*)a.Gy);
}

// Diffusion: forward y transform, multiply by exp(-D^2 |xi|^2 dt) / n (the
// packed column is unpacked into its kx = 0 and kx = Nx/2 halves for this),
// inverse y transform; both components batched.  Optional partial sum
// w |xi_tilde|^2 |m_hat_new|^2.
template <int NY>
__device__ __forceinline__ void col_heat_body(Geo g, cd* Mx, cd* My, double D2dt, double* eslot) {
  using C = ColCfg<NY, 2>;
  __shared__ cd buf[C::NB * C::LS];
  __shared__ double red[1 * (C::NT / 64)];
  const cd* tw = (const cd*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  const double xnyq = TWO_PI * (g.nx / 2) / g.lx;  // full wavenumber of the kx = Nx/2 column
  cd tv[C::ET];
  colT_gload<C, 2>(tv, Mx, My, kx0, g.h);
  colT_put<C, 2>(buf, tv);
  __syncthreads();
  lds_fft<double, -1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  double s[1] = {0.0};
  cd v[2][C::EP];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
#pragma unroll
    for (int i = 0; i < C::EP; ++i) {
      const int p = threadIdx.x + i * C::NT;
      const int c = p / NY, ky = p % NY;
      const int kx = kx0 + c;
      if (p >= C::CN) continue;
      const double yf = xi_full(ky, NY, g.ly);
      const cd* line = buf + (f * C::C + c) * C::LS;
      const cd a = line[ky];
      cd out;
      if (kx == 0) {
        const cd b = line[ky == 0 ? 0 : NY - ky];
        const double hA = exp(-D2dt * (yf * yf)) * g.inv_n;
        const double hB = exp(-D2dt * (xnyq * xnyq + yf * yf)) * g.inv_n;
        // P' = (hA+hB)/2 P(ky) + (hA-hB)/2 conj P(-ky)
        out = add(scl(a, 0.5 * (hA + hB)), scl(conj(b), 0.5 * (hA - hB)));
      } else {
        const double xx = TWO_PI * kx / g.lx;
        out = scl(a, exp(-D2dt * (xx * xx + yf * yf)) * g.inv_n);
      }
      v[f][i] = out;
      if (eslot && kx < g.h) {
        const double xt = xi_col(kx, g.lx), yt = xi_tilde(ky, NY, g.ly);
        const double w = kx == 0 ? 1.0 : 2.0;
        s[0] += w * (xt * xt + yt * yt) * (out.x * out.x + out.y * out.y);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < 2; ++f) {
#pragma unroll
    for (int i = 0; i < C::EP; ++i) {
      const int p = threadIdx.x + i * C::NT;
      if (p < C::CN) buf[(f * C::C + p / NY) * C::LS + p % NY] = v[f][i];
    }
  }
  __syncthreads();
  lds_fft<double, +1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  colT_store<C, 2>(buf, Mx, My, kx0, g.h);
  if (eslot) {
    block_sum<C::NT, 1>(s, red);
    write_partials<C::NT>(eslot, s, 1);
  }
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) k_col_heat(Geo g, cd* Mx, cd* My, double D2dt, double* eslot) {
  col_heat_body<NY>(g, Mx, My, D2dt, eslot);
}
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) kb_col_heat(const HeatArgs* __restrict__ A) {
  const HeatArgs& a = A[blockIdx.y];
  col_heat_body<NY>(a.g, (cd*)a.Mx, (cd*)a.My, a.D2dt, (double*)a.eslot);
}

// Adjoint right-hand side: b_hat = Pi F(G^T v) = -i xi_tilde . F(v) for the
// two mixed fields of v (null modes vanish since xi_tilde does).
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) k_col_divrhs(Geo g, const cd* __restrict__ V0, const cd* __restrict__ V1,
                                                        cd* __restrict__ bh) {
  using C = ColCfg<NY, 2>;
  __shared__ cd buf[C::NB * C::LS];
  const cd* tw = (const cd*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  cd tv[C::ET];
  colT_gload<C, 2>(tv, V0, V1, kx0, g.h);
  colT_put<C, 2>(buf, tv);
  __syncthreads();
  lds_fft<double, -1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  for (int p = threadIdx.x; p < C::CN; p += C::NT) {
    const int c = p / NY, ky = p % NY;
    const int kx = kx0 + c;
    if (kx < g.h) {
      const cd fx = buf[c * C::LS + ky], fy = buf[(C::C + c) * C::LS + ky];
      const double xx = xi_col(kx, g.lx), yy = xi_tilde(ky, NY, g.ly);
      const double ax = xx * fx.x + yy * fy.x, ay = xx * fx.y + yy * fy.y;
      bh[(size_t)kx * NY + ky] = mk<double>(ay, -ax);
    }
  }
}

__global__ void k_zero_d(double* p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

// Parseval sum w |xi_tilde|^2 |f_hat|^2 over two mixed fields (||grad m||^2 * n)
template <int NY>
__global__ void __launch_bounds__((ColCfg<NY, 2>::NT)) k_col_gradnorm(Geo g, const cd* __restrict__ Mx, const cd* __restrict__ My,
                                                      double* eslot) {
  using C = ColCfg<NY, 2>;
  __shared__ cd buf[C::NB * C::LS];
  __shared__ double red[1 * (C::NT / 64)];
  const cd* tw = (const cd*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  cd tv[C::ET];
  colT_gload<C, 2>(tv, Mx, My, kx0, g.h);
  colT_put<C, 2>(buf, tv);
  __syncthreads();
  lds_fft<double, -1, NY, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  double s[1] = {0.0};
  for (int e = threadIdx.x; e < 2 * C::CN; e += C::NT) {
    const int f = e / C::CN, ee = e % C::CN;
    const int c = ee / NY, ky = ee % NY;
    const int kx = kx0 + c;
    if (kx < g.h) {
      const cd a = buf[(f * C::C + c) * C::LS + ky];
      const double xt = xi_col(kx, g.lx), yt = xi_tilde(ky, NY, g.ly);
      const double w = kx == 0 ? 1.0 : 2.0;
      s[0] += w * (xt * xt + yt * yt) * (a.x * a.x + a.y * a.y);
    }
  }
  block_sum<C::NT, 1>(s, red);
  write_partials<C::NT>(eslot, s, 1);
}

static int row_threads(int nx, int nf) {
  const int t = row_tile(nx, nf) / 8 * nf;
  return t > 1024 ? 1024 : t;
}
static int row_nwg(const Geo& g, int nf) {
  const int R = tile_rows(g.nx / 2, row_tile(g.nx, nf));
  return (g.ny + R - 1) / R;
}
static int col_cols(int ny) {
  int c = TILE / ny;
  return c < 1 ? 1 : (c > 64 ? 64 : c);
}
// workgroups of the 2D row passes over one or two fields (the writers of row partials)
int row_nwg(const Geo& g) { return row_nwg(g, 2); }
int col_nwg(const Geo& g) {
  const int C = col_cols(g.ny);
  return (g.h + C - 1) / C;
}
int row_nwg_var(const Geo& g, int rv) {
  if (rv == VAR_DEFAULT) return row_nwg(g, 2);
  const int R = rv_rows(g.nx, rv);
  return (g.ny + R - 1) / R;
}
int col_nwg_var(const Geo& g, int cv) {
  if (cv == VAR_DEFAULT) return col_nwg(g);
  const int C = cv_cols(g.ny, cv);
  return (g.h + C - 1) / C;
}
bool flux_var_valid(const Geo& g, bool f32, int rv) {
  if (rv == VAR_DEFAULT) return true;
  const int es = f32 ? 8 : 16;
  if (rv >= RV_WIDE) return wide_row_ok(g.nx) && rv < NRV && rv_rows(g.nx, rv) >= 1 && g.nz == 1;
  if (rv >= RV_SEQ) return rv_seq_ok(g.nx, rv, es) && rv_rows(g.nx, rv) <= g.ny && g.nz == 1;
  if (rv >= RV_SMALL) return small_ok(rv_rows(g.nx, rv), g.nx / 2) && g.nz == 1;
  return var_size(g.nx) && g.nz == 1 && rv_ok(g.nx, g.ny, rv, es);
}
bool div_var_valid(const Geo& g, bool f32, int cv) {
  if (cv == VAR_DEFAULT) return true;
  if (cv >= CV_WIDE) return wide_col_ok(g.ny) && cv < NCV && cv_cols(g.ny, cv) >= 1 && g.nz == 1;
  if (cv >= CV_SEQ) return cv_seq_ok(g.ny, cv) && g.nz == 1;
  if (cv >= CV_SMALL) return small_ok(cv_cols(g.ny, cv), g.ny) && g.nz == 1;
  const int es = f32 ? 8 : 16;
  return var_size(g.ny) && g.nz == 1 && cv_ok(g.ny, g.h, cv, es);
}
__global__ void k_fill_d(double* p, size_t n, double v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
hipError_t launch_fill_doubles(double* p, size_t n, double v, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_d, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

// variant codes in use (a variant that cannot run on this grid falls back to the default)
int use_rv(const Geo& g, bool f32, int it) {
  const int rv = it < 0 ? VAR_DEFAULT : (g.wide == 2 ? (var_size(g.nx) ? 2 : VAR_DEFAULT) : (g.wide >= 0 ? RV_WIDE + g.wide : g.var_flux[f32 ? 1 : 0]));
  return flux_var_valid(g, f32, rv) ? rv : VAR_DEFAULT;
}
int use_cv(const Geo& g, bool f32) {
  const int cv = g.wide == 2 ? (int)VAR_DEFAULT : g.wide >= 0 ? CV_WIDE + g.wide : g.var_upd[f32 ? 1 : 0];
  return div_var_valid(g, f32, cv) ? cv : VAR_DEFAULT;
}
int rr_nwg(const Geo& g, bool f32) { return col_nwg_var(g, use_cv(g, f32)); }
int flux_var_rows(const Geo& g, int rv) {
  return rv == VAR_DEFAULT ? tile_rows(g.nx / 2, row_tile(g.nx, 2)) : rv_rows(g.nx, rv);
}
int flux_var_plan(int rv) { return rv >= RV_SMALL ? 0 : rv_plan(rv); }
int flux_var_threads(const Geo& g, int rv) {
  const int rt = rv == VAR_DEFAULT ? row_tile(g.nx, 2) : rv_rows(g.nx, rv) * (g.nx / 2);
  if (rv >= RV_WIDE) return wide_threads(rv - RV_WIDE);
  if (rv >= RV_SEQ) return rv_rows(g.nx, rv) * (g.nx / 2) / 8;
  if (rv >= RV_SMALL) return small_threads(rv_rows(g.nx, rv), g.nx / 2);
  const int nt = (rt / 8) * 2 > 1024 ? 1024 : (rt / 8) * 2;
  return nt / (rv == VAR_DEFAULT ? 1 : rv_td(rv));
}
int div_var_cols(const Geo& g, int cv) { return cv == VAR_DEFAULT ? col_cols(g.ny) : cv_cols(g.ny, cv); }
int div_var_threads(const Geo& g, int cv) {
  if (cv >= CV_SMALL) return cv_threads(g.ny, cv);
  return cv == VAR_DEFAULT ? col_threads(g.ny, 2) : 2 * TPF * cv_tm(cv);
}
bool tuned_length(int n) { return var_size(n); }
bool var_grid(const Geo& g) { return g.nz == 1 && (var_size(g.nx) || var_size(g.ny)); }

hipError_t launch_status_reset(const Geo& g, int full, hipStream_t s) {
  hipLaunchKernelGGL(k_status_reset, dim3(1), dim3(64), 0, s, g.st, full);
  return hipGetLastError();
}
hipError_t launch_zero_spec(const Geo& g, void* xh, hipStream_t s) {
  const size_t n = (size_t)g.h * g.ny;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (cd*)xh, n);
  return hipGetLastError();
}
hipError_t launch_sum_slot(const Geo& g, const double* slot, int K, int n, int o, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_slot, dim3(1), dim3(256), 0, s, slot, K, n, o, g.st);
  return hipGetLastError();
}

hipError_t launch_row_r2c(const Geo& g, const double* f, void* out, double* schk, hipStream_t s) {
  const dim3 grid(row_nwg(g, 1)), blk(row_threads(g.nx, 1));
#define L_(N) hipLaunchKernelGGL(k_row_r2c<N>, grid, blk, 0, s, g, f, (cd*)out, schk)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_row_c2r(const Geo& g, const void* in, double* f, hipStream_t s) {
  const dim3 grid(row_nwg(g, 1)), blk(row_threads(g.nx, 1));
#define L_(N) hipLaunchKernelGGL(k_row_c2r<N>, grid, blk, 0, s, g, (const cd*)in, f)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipGetLastError();
}
// Split update, pointwise part.  Where the three-field tile holds one row per
// workgroup (rows of 2048 and more), p is written by a one-field pass first and
// the activation and relaxation run in the two-field, two-row tile: the same
// bytes in runs of twice the length.
template <int NX>
static hipError_t split_go(const Geo& g, void* P, void* Gx, void* Gy, const double* m, double* p_out, double c2dt,
                           double gamma, double dt, double relax1, hipStream_t s) {
  if constexpr (split_separate_p<NX>()) {
    hipLaunchKernelGGL(k_row_c2r<NX>, dim3(row_nwg(g, 1)), dim3(row_threads(g.nx, 1)), 0, s, g, (const cd*)P, p_out);
    const int R = SplitCfg<NX>::R;
    hipLaunchKernelGGL((k_row_split<NX, false>), dim3((g.ny + R - 1) / R), dim3(SplitCfg<NX>::NT), 0, s, g, (cd*)P,
                       (cd*)Gx, (const cd*)Gy, m, p_out, c2dt, gamma, dt, relax1);
  } else {
    hipLaunchKernelGGL((k_row_split<NX, true>), dim3(row_nwg(g, 3)), dim3(row_threads(g.nx, 3)), 0, s, g, (cd*)P,
                       (cd*)Gx, (const cd*)Gy, m, p_out, c2dt, gamma, dt, relax1);
  }
  return hipGetLastError();
}
hipError_t launch_row_split(const Geo& g, void* P, void* Gx, void* Gy, const double* m, double* p_out,
                            double c2dt, double gamma, double dt, double relax1, hipStream_t s) {
#define L_(N) return split_go<N>(g, P, Gx, Gy, m, p_out, c2dt, gamma, dt, relax1, s)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipErrorInvalidValue;
}
hipError_t launch_row_final(const Geo& g, const void* Mx, const void* My, double* m, double* dslot,
                            hipStream_t s) {
  const dim3 grid(row_nwg(g, 2)), blk(row_threads(g.nx, 2));
#define L_(N) hipLaunchKernelGGL(k_row_final<N>, grid, blk, 0, s, g, (const cd*)Mx, (const cd*)My, m, dslot)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_row_energy(const Geo& g, const void* Gx, const void* Gy, const double* m, const double* r,
                             double gamma, double* slot, hipStream_t s) {
  const dim3 grid(row_nwg(g, 2)), blk(row_threads(g.nx, 2));
#define L_(N) \
  hipLaunchKernelGGL(k_row_energy<N>, grid, blk, 0, s, g, (const cd*)Gx, (const cd*)Gy, m, r, gamma, slot)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipGetLastError();
}

hipError_t launch_col_fwd(const Geo& g, void* in, void* out, int with_grad, void* Gx, void* Gy, hipStream_t s) {
  const dim3 grid(col_nwg(g)), blk(col_threads(g.ny, 2));
#define L_(N) hipLaunchKernelGGL(k_col_fwd<N>, grid, blk, 0, s, g, (cd*)in, (cd*)out, with_grad, (cd*)Gx, (cd*)Gy)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_col_grad(const Geo& g, const void* xh, void* P, void* Gx, void* Gy, hipStream_t s) {
  const dim3 grid(col_nwg(g));
  if (P) {
#define L_(N) hipLaunchKernelGGL((k_col_grad<N, false>), grid, dim3(col_threads(g.ny, 1)), 0, s, g, (const cd*)xh, (cd*)P, (cd*)Gx, (cd*)Gy)
    NF_DISPATCH(g.ny, L_)
#undef L_
  }
  if (Gx) {
#define L_(N) hipLaunchKernelGGL((k_col_grad<N, true>), grid, dim3(col_threads(g.ny, 2)), 0, s, g, (const cd*)xh, (cd*)P, (cd*)Gx, (cd*)Gy)
    NF_DISPATCH(g.ny, L_)
#undef L_
  }
  return hipGetLastError();
}
// The operator end outside the loop (default tile): the residual of the
// initial iterate (init) or the plain operator apply.
hipError_t launch_col_div(const Geo& g, int init, const void* Fx, const void* Fy, void* qh, void* rh, const void* bh,
                          int nwg_row, hipStream_t s) {
  const dim3 grid(col_nwg(g)), blk(col_threads(g.ny, 2));
  if (init) {
#define L_(N)                                                                                               \
  hipLaunchKernelGGL((k_col_div<N, true>), grid, blk, 0, s, g, (const cd*)Fx, (const cd*)Fy, (cd*)qh, (cd*)rh, \
                     (const cd*)bh, nwg_row)
    NF_DISPATCH(g.ny, L_)
#undef L_
  } else {
#define L_(N)                                                                                                \
  hipLaunchKernelGGL((k_col_div<N, false>), grid, blk, 0, s, g, (const cd*)Fx, (const cd*)Fy, (cd*)qh, (cd*)rh, \
                     (const cd*)bh, nwg_row)
    NF_DISPATCH(g.ny, L_)
#undef L_
  }
  return hipGetLastError();
}
hipError_t launch_col_start(const Geo& g, const void* rh, void* xh, void* Gx, void* Gy, int max_iter, double tol2,
                            hipStream_t s) {
  const dim3 grid(col_nwg(g)), blk(col_threads(g.ny, 2));
  const int nwg = col_nwg(g);
#define L_(N) \
  hipLaunchKernelGGL(k_col_start<N>, grid, blk, 0, s, g, (const cd*)rh, (cd*)xh, (cd*)Gx, (cd*)Gy, max_iter, tol2, nwg)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_col_refine_start(const Geo& g, const void* r64, void* x64, void* x32, void* r32,
                                   void* Gx, void* Gy, double tol2, double floor_in, int max_iter, hipStream_t s) {
  typedef cx<float> cf;
  const dim3 grid(col_nwg(g)), blk(col_threads(g.ny, 2));
  const int nwg = col_nwg(g);
#define L_(N)                                                                                                 \
  hipLaunchKernelGGL(k_col_refine_start<N>, grid, blk, 0, s, g, (const cd*)r64, (cd*)x64, (cf*)x32, (cf*)r32,  \
                     (cf*)Gx, (cf*)Gy, tol2, floor_in, max_iter, nwg)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_col_refine_acc(const Geo& g, void* x64, const void* x32, void* Gx, void* Gy, hipStream_t s) {
  const dim3 grid(col_nwg(g)), blk(col_threads(g.ny, 2));
#define L_(N)                                                                                                 \
  hipLaunchKernelGGL(k_col_refine_acc<N>, grid, blk, 0, s, g, (cd*)x64, (const cx<float>*)x32, (cd*)Gx, (cd*)Gy)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_col_heat(const Geo& g, void* Mx, void* My, double D2dt, double* eslot, hipStream_t s) {
  const dim3 grid(col_nwg(g)), blk(col_threads(g.ny, 2));
#define L_(N) hipLaunchKernelGGL(k_col_heat<N>, grid, blk, 0, s, g, (cd*)Mx, (cd*)My, D2dt, eslot)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_col_gradnorm(const Geo& g, const void* Mx, const void* My, double* eslot, hipStream_t s) {
  const dim3 grid(col_nwg(g)), blk(col_threads(g.ny, 2));
#define L_(N) hipLaunchKernelGGL(k_col_gradnorm<N>, grid, blk, 0, s, g, (const cd*)Mx, (const cd*)My, eslot)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}

// ---------------------------------------------------------------- batched launchers
hipError_t launchb_status_reset(DevStatus* st0, int count, int full, hipStream_t s) {
  hipLaunchKernelGGL(kb_status_reset, dim3(count), dim3(64), 0, s, st0, full);
  return hipGetLastError();
}
hipError_t launchb_sum_slot(const SumArgs* A, int count, int K, int n, int o, hipStream_t s) {
  hipLaunchKernelGGL(kb_sum_slot, dim3(1, count), dim3(256), 0, s, A, K, n, o);
  return hipGetLastError();
}
hipError_t launchb_row_r2c(const Geo& g, const RowR2cArgs* A, int count, hipStream_t s) {
  const dim3 grid(row_nwg(g, 1), count), blk(row_threads(g.nx, 1));
#define L_(N) hipLaunchKernelGGL(kb_row_r2c<N>, grid, blk, 0, s, A)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launchb_col_fwd(const Geo& g, const ColFwdArgs* A, int count, int mode, hipStream_t s) {
  const dim3 grid(col_nwg(g), count), blk(col_threads(g.ny, 2));
#define L_(N) hipLaunchKernelGGL(kb_col_fwd<N>, grid, blk, 0, s, A, mode)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launchb_col_grad(const Geo& g, const ColGradArgs* A, int count, bool grad, hipStream_t s) {
  const dim3 grid(col_nwg(g), count);
  if (grad) {
#define L_(N) hipLaunchKernelGGL((kb_col_grad<N, true>), grid, dim3(col_threads(g.ny, 2)), 0, s, A)
    NF_DISPATCH(g.ny, L_)
#undef L_
  } else {
#define L_(N) hipLaunchKernelGGL((kb_col_grad<N, false>), grid, dim3(col_threads(g.ny, 1)), 0, s, A)
    NF_DISPATCH(g.ny, L_)
#undef L_
  }
  return hipGetLastError();
}
hipError_t launchb_col_div_init(const Geo& g, const DivArgs* A, int count, hipStream_t s) {
  const dim3 grid(col_nwg(g), count), blk(col_threads(g.ny, 2));
  const int nwg_row = row_nwg(g);
#define L_(N) hipLaunchKernelGGL(kb_col_div<N>, grid, blk, 0, s, A, nwg_row)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launchb_col_start(const Geo& g, const IterArgs* A, int count, int max_iter, double tol2, hipStream_t s) {
  const dim3 grid(col_nwg(g), count), blk(col_threads(g.ny, 2));
  const int nwg = col_nwg(g);
#define L_(N) hipLaunchKernelGGL(kb_col_start<N>, grid, blk, 0, s, A, max_iter, tol2, nwg)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
template <int NX>
static hipError_t splitb_go(const Geo& g, const SplitArgs* A, int count, hipStream_t s) {
  if constexpr (split_separate_p<NX>()) {
    hipLaunchKernelGGL(kb_row_split_p<NX>, dim3(row_nwg(g, 1), count), dim3(row_threads(g.nx, 1)), 0, s, A);
    const int R = SplitCfg<NX>::R;
    hipLaunchKernelGGL((kb_row_split<NX, false>), dim3((g.ny + R - 1) / R, count), dim3(SplitCfg<NX>::NT), 0, s, A);
  } else {
    hipLaunchKernelGGL((kb_row_split<NX, true>), dim3(row_nwg(g, 3), count), dim3(row_threads(g.nx, 3)), 0, s, A);
  }
  return hipGetLastError();
}
hipError_t launchb_row_split(const Geo& g, const SplitArgs* A, int count, hipStream_t s) {
#define L_(N) return splitb_go<N>(g, A, count, s)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipErrorInvalidValue;
}
hipError_t launchb_col_heat(const Geo& g, const HeatArgs* A, int count, hipStream_t s) {
  const dim3 grid(col_nwg(g), count), blk(col_threads(g.ny, 2));
#define L_(N) hipLaunchKernelGGL(kb_col_heat<N>, grid, blk, 0, s, A)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launchb_row_final(const Geo& g, const FinalArgs* A, int count, hipStream_t s) {
  const dim3 grid(row_nwg(g, 2), count), blk(row_threads(g.nx, 2));
#define L_(N) hipLaunchKernelGGL(kb_row_final<N>, grid, blk, 0, s, A)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launchb_col_refine_start(const Geo& g, const RefStartArgs* A, int count, double tol2, double floor_in,
                                    int max_iter, hipStream_t s) {
  const dim3 grid(col_nwg(g), count), blk(col_threads(g.ny, 2));
  const int nwg = col_nwg(g);
#define L_(N) hipLaunchKernelGGL(kb_col_refine_start<N>, grid, blk, 0, s, A, tol2, floor_in, max_iter, nwg)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launchb_col_refine_acc(const Geo& g, const RefAccArgs* A, int count, hipStream_t s) {
  const dim3 grid(col_nwg(g), count), blk(col_threads(g.ny, 2));
#define L_(N) hipLaunchKernelGGL(kb_col_refine_acc<N>, grid, blk, 0, s, A)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}

}  // namespace nf

namespace nf {
hipError_t launch_row_adj1(const Geo& g, void* A0, void* A1, const void* G0, const void* G1, const double* m,
                           double* lam_out, double c2dt, double gamma, double dt, double relax1, hipStream_t s) {
  const dim3 grid(row_nwg(g, 4)), blk(row_threads(g.nx, 4));
#define L_(N)                                                                                                    \
  hipLaunchKernelGGL(k_row_adj1<N>, grid, blk, 0, s, g, (cd*)A0, (cd*)A1, (const cd*)G0, (const cd*)G1, m, lam_out, \
                     c2dt, gamma, dt, relax1)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_row_adj2(const Geo& g, const void* M1, const void* M2, const void* P1, const void* P2,
                           const double* m, const double* mu, double* lam, double* grad_r, double* grad_S,
                           hipStream_t s) {
  const dim3 grid(row_nwg(g, 4)), blk(row_threads(g.nx, 4));
#define L_(N)                                                                                                 \
  hipLaunchKernelGGL(k_row_adj2<N>, grid, blk, 0, s, g, (const cd*)M1, (const cd*)M2, (const cd*)P1,           \
                     (const cd*)P2, m, mu, lam, grad_r, grad_S)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_col_divrhs(const Geo& g, const void* V0, const void* V1, void* bh, hipStream_t s) {
  const dim3 grid(col_nwg(g)), blk(col_threads(g.ny, 2));
#define L_(N) hipLaunchKernelGGL(k_col_divrhs<N>, grid, blk, 0, s, g, (const cd*)V0, (const cd*)V1, (cd*)bh)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipGetLastError();
}
hipError_t launch_zero_doubles(double* p, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_d, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}
}  // namespace nf
