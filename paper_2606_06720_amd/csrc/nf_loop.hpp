// The two passes of a PCG iteration on 2D grids, shared by the FP64 and FP32
// instantiations (nf_loop_row*.hip, nf_loop_col*.hip).
//
// The loop is the single-reduction form of preconditioned CG (Chronopoulos and
// Gear 1989): with z = M^-1 r and w = A z,
//   gamma = <r, z>, delta = <z, w>, beta = gamma / gamma_prev,
//   alpha = gamma / (delta - beta gamma / alpha_prev),
//   d = z + beta d, s = w + beta s (= A d), x += alpha d, r -= alpha s.
// delta is the physical sum of grad z . K grad z, which the row pass has in
// hand, so every scalar of an iteration is known when its column pass starts:
// the operator end, the vector updates and the next gradient are one pass over
// the columns instead of two with a reduction between them.  Per grid point
// (FP64) a row pass moves 56 bytes (two gradient fields in, two flux fields
// out, m, r) and a column pass 96 (two fields in and out; x, r, d, s in and
// out); the textbook recurrence moved 168 in three passes.  The iterates are
// those of the textbook recurrence up to rounding.
//
// The FP32 loop (corrections of the refined solve) does not carry s = A d: the
// errors of the A z that s adds up, each relative to A z, stay in it, and where
// |A d| is much smaller they leave a gap between r and b - A x that costs the
// refinement more FP32 iterations (1024^2, m uniform in [-16, 16], r about 0.1,
// rtol 1e-10: 1069, with the textbook recurrence 921; log-normal r of sigma 1.5:
// 1098 and 930; the FP64 loop takes 838 and 807, textbook 839 and 802).  There
// the row pass keeps the physical gradient of the search direction instead,
// g_d = grad z + beta g_d, so that A d comes fresh from K g_d and delta =
// sum g_d . K g_d is the curvature of d: 925 and 945 iterations.  This moves 84
// instead of 76 bytes per point, which the loops in one launch, where g_d stays
// on chip, do not notice (1024^2 solve of mild data 2.79 -> 2.78 ms); as launches
// such a solve takes 60.3 instead of 55.8 ms at 4096^2 and 32.7 instead of 30.6 at
// 256 x 256 x 128 (three textbook passes: 62.2 and 36.7).
//
// Measured per iteration, one handle alone, three passes -> two (MI355X): 256^2 29.5
// -> 20.6 us, 1024^2 55 -> 43.7 us, 4096^2 FP64 880 -> 770 us.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

// Products are fused into sums within an expression only, not where the
// optimiser happens to find them: these passes and the kernel that runs them as
// one launch (nf_chip.hpp) have to round alike.
#pragma clang fp contract(on)

#include "nf_fft.hpp"
#include "nf_internal.h"
#include "nf_tiles.hpp"

namespace nf {

// ---------------------------------------------------------------- row pass
// Operator middle: gradient fields (mixed) -> physical g -> flux K g -> mixed,
// both components in one batched transform each way.  In place: G0/G1 hold
// grad_x/grad_y on entry and F_x/F_y on exit.  Optional partials: sum mx^2,
// mx my, my^2, r (the preconditioner's Kbar).  Optional lo: FP32 copies of
// m (2n values) followed by r (n values) for the single-precision inner solve.
// In the PCG loop (it >= 0) the pass leaves the partials of n sum g . K g =
// delta in SLOT_P3, and (it >= 1) first takes the stopping decision for the
// residual r_it left by the column pass: ||r_it||^2 (reduced from that pass's
// partials) <= tol2 * status.bb ends the solve at iteration it; its block 0
// also adds up gamma = <r, M^-1 r> into status.rho[it & 1].
// T is the arithmetic and storage type of the transforms and fields; the
// reductions are FP64 in both instantiations.
template <int NX, typename T, int RV>
__device__ __forceinline__ void row_flux_body(Geo g, cx<T>* G0, cx<T>* G1, const T* __restrict__ m,
                                              const T* __restrict__ r, int it, double* kslot, int nwg_col,
                                              double tol2, float* lo, T* gd) {
  using C = FluxCfg<NX, RV>;
  using V = cx<T>;
  using P = typename vec2<T>::type;
  constexpr int NW = C::NT / 64;
  // Short rows: the pass is a chain of latencies (a launch moves a few MB), so
  // m and r are requested with the gradient fields.  Long rows load them after
  // the first transform: held across it they would cost about 48 registers,
  // and a workgroup with fewer registers shares a compute unit more easily
  // with the passes of concurrent solves.
  constexpr bool EARLY = NX <= 512;
  constexpr bool GR = grad_rec<T>();
  if (it >= 0 ? g.st->conv_at <= it : g.st->outer_done != 0) return;
  tclk_start(g, 0, it);
  __shared__ V buf[C::NB * C::LS];
  __shared__ double red[4 * NW];
  __shared__ double redd[NW];
  const V* tw = (const V*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  const size_t n = (size_t)g.nx * g.ny;
  // Tiles of fewer than 1024 threads load the pairs (k, H - k) of each line, so
  // that the pre-processing of the inverse real transform happens on the way
  // into LDS; 1024-thread tiles (at most 128 registers per thread) load the
  // plain transposed image and pre-process in LDS, since the paired form
  // spills there.
  constexpr bool PAIRS = C::NT < 1024;
  constexpr int NA = PAIRS ? RowPairs<C>::ETP : C::ET, NBP = PAIRS ? RowPairs<C>::ETP : 1;
  V ta[NA], tb[NBP];
  if constexpr (PAIRS)
    rowTP_gload<C>(ta, tb, G0, G1, nullptr, g.ny, y0, nrow);
  else
    rowT_gload<C>(ta, G0, G1, nullptr, g.ny, y0, nrow);
  P mx[C::EP], my[C::EP], rv[C::EP];
  // points whose old gradient of d is in registers at a time
  constexpr int HE = C::EP > 8 ? 8 : C::EP;
  P dx[GR ? HE : 1], dy[GR ? HE : 1];
  auto load_grad = [&](int i0) {
    if constexpr (GR) {
      if (it >= 1) {
        rowP_gload_part<C>(dx, gd, i0, y0, nrow);
        rowP_gload_part<C>(dy, gd + n, i0, y0, nrow);
      }
    }
  };
  auto load_points = [&]() {
    rowP_gload<C>(mx, m, y0, nrow);
    rowP_gload<C>(my, m + n, y0, nrow);
    rowP_gload<C>(rv, r, y0, nrow);
    load_grad(0);
  };
  if constexpr (EARLY) load_points();
  T bt = 0;
  if (it >= 1) {
    const double* part = slot_ptr(g.part, SLOT_RR);
    double s[1] = {0.0};
    for (int i = threadIdx.x; i < nwg_col; i += C::NT) s[0] += part[i];
    wave_sums<1>(s, red);
    if (GR || blockIdx.x == 0) {
      double z[1] = {0.0};
      for (int i = threadIdx.x; i < nwg_col; i += C::NT) z[0] += part[MAX_WG + i];
      wave_sums<1>(z, red + NW);
    }
  }
  if constexpr (PAIRS)
    rowTP_put_pre<C>(buf, ta, tb, tw, g.twn);
  else
    rowT_put<C>(buf, ta);
  __syncthreads();
  if (it >= 1) {
    const double rr = waves_total<NW>(red);
    const bool bad = !isfinite(rr);
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    if (bad || rr <= tol2 * g.st->bb) {
      if (lead) {
        g.st->rr[0] = rr;
        g.st->converged = bad ? 0 : 1;
        if (bad) g.st->flags |= FLAG_NONFINITE;
        g.st->conv_at = it;
      }
      return;
    }
    if (lead) g.st->rho[it & 1] = waves_total<NW>(red + NW);
    if constexpr (GR) bt = (T)pcg_beta(waves_total<NW>(red + NW), g.st->rho[(it + 1) & 1], false);
  }
  if constexpr (!PAIRS) irfft_pre<T, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
  lds_fft<T, +1, C::H, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
  if constexpr (!EARLY) load_points();
  if (lo) {
#pragma unroll
    for (int i = 0; i < C::EP; ++i) {
      const int p = threadIdx.x + i * C::NT;
      const int rr = p / C::H, j = p % C::H;
      if (p < C::RH && rr < nrow) {
        const size_t o = (size_t)(y0 + rr) * NX + 2 * j;
        *(float2*)(lo + o) = make_float2((float)mx[i].x, (float)mx[i].y);
        *(float2*)(lo + n + o) = make_float2((float)my[i].x, (float)my[i].y);
        *(float2*)(lo + 2 * n + o) = make_float2((float)rv[i].x, (float)rv[i].y);
      }
    }
  }
  double ks[4] = {0.0, 0.0, 0.0, 0.0};
  double de[1] = {0.0};
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int rr = p / C::H, j = p % C::H;
    if (i > 0 && i % HE == 0) load_grad(i);
    if (p < C::RH && rr < nrow) {
      V* px = buf + rr * C::LS + j;
      V* py = buf + (C::R + rr) * C::LS + j;
      V gx = *px, gy = *py;
      if constexpr (GR) {
        if (it >= 1) {
          gx = add(gx, scl(mk<T>(dx[i % HE].x, dx[i % HE].y), bt));
          gy = add(gy, scl(mk<T>(dy[i % HE].x, dy[i % HE].y), bt));
        }
        const size_t o = (size_t)(y0 + rr) * NX + 2 * j;
        *(V*)(gd + o) = gx;
        *(V*)(gd + n + o) = gy;
      }
      // K g = (m.g) m + r g at the two grid points packed in this element
      const T a0 = mx[i].x * gx.x + my[i].x * gy.x;
      const T a1 = mx[i].y * gx.y + my[i].y * gy.y;
      const V fx = mk<T>(fma(a0, mx[i].x, rv[i].x * gx.x), fma(a1, mx[i].y, rv[i].y * gx.y));
      const V fy = mk<T>(fma(a0, my[i].x, rv[i].x * gy.x), fma(a1, my[i].y, rv[i].y * gy.y));
      *px = fx;
      *py = fy;
      de[0] += (double)gx.x * fx.x + (double)gx.y * fx.y + (double)gy.x * fy.x + (double)gy.y * fy.y;
      if (kslot) {
        ks[0] += (double)mx[i].x * mx[i].x + (double)mx[i].y * mx[i].y;
        ks[1] += (double)mx[i].x * my[i].x + (double)mx[i].y * my[i].y;
        ks[2] += (double)my[i].x * my[i].x + (double)my[i].y * my[i].y;
        ks[3] += (double)rv[i].x + (double)rv[i].y;
      }
    }
  }
  // wave sums of delta; the barriers of the transform order them before the total
  wave_sums<1>(de, redd);
  __syncthreads();
  lds_fft<T, -1, C::H, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
  if (it >= 0 && threadIdx.x == 0) slot_ptr(g.part, SLOT_P3)[blockIdx.x] = waves_total<NW>(redd) * (double)n;
  // post-processing of the forward real transform on the way out
  if constexpr (PAIRS) {
    rowTP_store_post<C, 2>(buf, G0, G1, nullptr, tw, g.twn, g.ny, y0, nrow);
  } else {
    rfft_post<T, C::H, C::NB, C::LS, C::NT>(buf, tw, g.twn);
    rowT_store<C, 2>(buf, G0, G1, nullptr, g.ny, y0, nrow);
  }
  if (kslot) {
    block_sum<C::NT, 4>(ks, red);
    write_partials<C::NT>(kslot, ks, 4);
  }
  tclk_end(g, 0, it);
}
// The loop's row pass with the two fields one after the other through one field's
// LDS (row variants from RV_SEQ to below RV_WIDE, rows of 2048 and more): grad_x waits in
// registers while grad_y is transformed, F_x while F_y is.  For the same rows
// the tile takes half the LDS and half the threads, so twice the workgroups
// share a compute unit and one's transforms overlap the others' memory phases
// (the two-field tile of 2048 keeps a compute unit's vector units 20%, its LDS
// 21% and HBM 50% busy, one phase after the other).
template <int NX, typename T, int RV>
__device__ __forceinline__ void row_flux_seq_body(Geo g, cx<T>* G0, cx<T>* G1, const T* __restrict__ m,
                                                  const T* __restrict__ r, int it, int nwg_col, double tol2, T* gd) {
  using C = FluxCfg<NX, RV>;
  using V = cx<T>;
  using P = typename vec2<T>::type;
  constexpr int NW = C::NT / 64;
  constexpr bool GR = grad_rec<T>();
  if (g.st->conv_at <= it) return;
  tclk_start(g, 0, it);
  __shared__ V buf[C::NB * C::LS];
  __shared__ double red[2 * NW];
  __shared__ double redd[NW];
  const V* tw = (const V*)g.tw;
  const int y0 = xcd_block() * C::R;
  const int nrow = min(C::R, g.ny - y0);
  const size_t n = (size_t)g.nx * g.ny;
  V ta[RowPairs<C>::ETP], tb[RowPairs<C>::ETP];
  rowTP_gload<C>(ta, tb, G0, nullptr, nullptr, g.ny, y0, nrow);
  T bt = 0;
  if (it >= 1) {
    const double* part = slot_ptr(g.part, SLOT_RR);
    double s[1] = {0.0};
    for (int i = threadIdx.x; i < nwg_col; i += C::NT) s[0] += part[i];
    wave_sums<1>(s, red);
    if (GR || blockIdx.x == 0) {
      double z[1] = {0.0};
      for (int i = threadIdx.x; i < nwg_col; i += C::NT) z[0] += part[MAX_WG + i];
      wave_sums<1>(z, red + NW);
    }
  }
  rowTP_put_pre<C>(buf, ta, tb, tw, g.twn);
  __syncthreads();
  if (it >= 1) {
    const double rr = waves_total<NW>(red);
    const bool bad = !isfinite(rr);
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    if (bad || rr <= tol2 * g.st->bb) {
      if (lead) {
        g.st->rr[0] = rr;
        g.st->converged = bad ? 0 : 1;
        if (bad) g.st->flags |= FLAG_NONFINITE;
        g.st->conv_at = it;
      }
      return;
    }
    if (lead) g.st->rho[it & 1] = waves_total<NW>(red + NW);
    if constexpr (GR) bt = (T)pcg_beta(waves_total<NW>(red + NW), g.st->rho[(it + 1) & 1], false);
  }
  rowTP_gload<C>(ta, tb, G1, nullptr, nullptr, g.ny, y0, nrow);
  lds_fft<T, +1, C::H, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
  V gx[C::EP];
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    if (p < C::RH) gx[i] = buf[(p / C::H) * C::LS + p % C::H];
  }
  __syncthreads();
  rowTP_put_pre<C>(buf, ta, tb, tw, g.twn);
  __syncthreads();
  lds_fft<T, +1, C::H, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
  double de[1] = {0.0};
  // half of the points at a time: the loads of m and r of one half are in
  // flight together
  constexpr int HE = C::EP > 4 ? 4 : C::EP;
#pragma unroll
  for (int i0 = 0; i0 < C::EP; i0 += HE) {
    P mx[HE], my[HE], rv[HE], dx[GR ? HE : 1], dy[GR ? HE : 1];
#pragma unroll
    for (int q = 0; q < HE; ++q) {
      const int p = threadIdx.x + (i0 + q) * C::NT;
      const int rr = p / C::H, j = p % C::H;
      const size_t o = (size_t)(y0 + rr) * NX + 2 * j;
      const bool ok = p < C::RH && rr < nrow;
      mx[q] = ok ? *(const P*)(m + o) : vzero<P>();
      my[q] = ok ? *(const P*)(m + n + o) : vzero<P>();
      rv[q] = ok ? *(const P*)(r + o) : vzero<P>();
      if constexpr (GR) {
        dx[q] = ok && it >= 1 ? *(const P*)(gd + o) : vzero<P>();
        dy[q] = ok && it >= 1 ? *(const P*)(gd + n + o) : vzero<P>();
      }
    }
#pragma unroll
    for (int q = 0; q < HE; ++q) {
      const int p = threadIdx.x + (i0 + q) * C::NT;
      if (p >= C::RH) continue;
      V* py = buf + (p / C::H) * C::LS + p % C::H;
      V gxv = gx[i0 + q], gyv = *py;
      if constexpr (GR) {
        if (it >= 1) {
          gxv = add(gxv, scl(mk<T>(dx[q].x, dx[q].y), bt));
          gyv = add(gyv, scl(mk<T>(dy[q].x, dy[q].y), bt));
        }
        const size_t o = (size_t)(y0 + p / C::H) * NX + 2 * (p % C::H);
        if (p / C::H < nrow) {
          *(V*)(gd + o) = gxv;
          *(V*)(gd + n + o) = gyv;
        }
      }
      const T a0 = mx[q].x * gxv.x + my[q].x * gyv.x;
      const T a1 = mx[q].y * gxv.y + my[q].y * gyv.y;
      const V fx = mk<T>(fma(a0, mx[q].x, rv[q].x * gxv.x), fma(a1, mx[q].y, rv[q].y * gxv.y));
      const V fy = mk<T>(fma(a0, my[q].x, rv[q].x * gyv.x), fma(a1, my[q].y, rv[q].y * gyv.y));
      gx[i0 + q] = fx;
      *py = fy;
      de[0] += (double)gxv.x * fx.x + (double)gxv.y * fx.y + (double)gyv.x * fy.x + (double)gyv.y * fy.y;
    }
  }
  wave_sums<1>(de, redd);
  __syncthreads();
  lds_fft<T, -1, C::H, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
  if (threadIdx.x == 0) slot_ptr(g.part, SLOT_P3)[blockIdx.x] = waves_total<NW>(redd) * (double)n;
  rowTP_store_post<C, 1>(buf, G1, nullptr, nullptr, tw, g.twn, g.ny, y0, nrow);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    if (p < C::RH) buf[(p / C::H) * C::LS + p % C::H] = gx[i];
  }
  __syncthreads();
  lds_fft<T, -1, C::H, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
  rowTP_store_post<C, 1>(buf, G0, nullptr, nullptr, tw, g.twn, g.ny, y0, nrow);
  tclk_end(g, 0, it);
}
template <int NX, typename T, int RV>
__global__ void __launch_bounds__((FluxCfg<NX, RV>::NT)) k_row_flux(Geo g, cx<T>* G0, cx<T>* G1, const T* __restrict__ m,
                                                  const T* __restrict__ r, int it, double* kslot, int nwg_col,
                                                  double tol2, float* lo, T* gd) {
  if constexpr (RV >= RV_SEQ && RV < RV_WIDE) row_flux_seq_body<NX, T, RV>(g, G0, G1, m, r, it, nwg_col, tol2, gd);
  else row_flux_body<NX, T, RV>(g, G0, G1, m, r, it, kslot, nwg_col, tol2, lo, gd);
}
template <int NX, typename T, int RV>
__global__ void __launch_bounds__((FluxCfg<NX, RV>::NT)) kb_row_flux(const FluxArgs* __restrict__ A, int it, int nwg_col, double tol2) {
  const FluxArgs& a = A[blockIdx.y];
  if constexpr (RV >= RV_SEQ && RV < RV_WIDE) row_flux_seq_body<NX, T, RV>(a.g, (cx<T>*)a.G0, (cx<T>*)a.G1, (const T*)a.m, (const T*)a.r, it, nwg_col, tol2, (T*)a.gd);
  else row_flux_body<NX, T, RV>(a.g, (cx<T>*)a.G0, (cx<T>*)a.G1, (const T*)a.m, (const T*)a.r, it, (double*)a.kslot, nwg_col, tol2, (float*)a.lo, (T*)a.gd);
}

// ---------------------------------------------------------------- column pass
// Iteration it of the loop on one block of columns: forward y transform of the
// fluxes, w = -i xi . F = A z; the scalars from the totals described above
// (gamma in status.rho, alpha of the last iteration in status.alpha, delta
// from the row pass's partials); the vector updates; z = M^-1 r of the new
// residual and its gradient back to the mixed buffers.  In place: M0/M1 hold
// F_x/F_y on entry and grad_x/grad_y on exit.  Partials ||r||^2 and
// <r, M^-1 r> of the new residual in SLOT_RR.  The scalars and reductions are
// FP64, the vector updates run in T.  The iteration that reaches max_iter (or
// the budget of a correction) updates x and r and ends the solve.
template <int NY, typename T, int CV>
__device__ __forceinline__ void col_iter_body(Geo g, cx<T>* M0, cx<T>* M1, cx<T>* __restrict__ xh,
                                              cx<T>* __restrict__ rh, cx<T>* __restrict__ dh, cx<T>* __restrict__ sh,
                                              int it, int max_iter, int nwg_row) {
  using C = DivCfg<NY, CV>;
  using V = cx<T>;
  constexpr int NW = C::NT / 64;
  // Short columns request the vectors together with the fluxes (the pass is a
  // chain of latencies); longer ones after the first transform, which saves
  // the registers they would hold across it.
  constexpr bool EARLY = NY <= 512;
  constexpr bool GR = grad_rec<T>();
  DevStatus* st = g.st;
  if (st->conv_at <= it) return;
  tclk_start(g, 2, it + 1);
  __shared__ V buf[C::NB * C::LS];
  __shared__ double red[NW];
  __shared__ double red2[2 * NW];
  const V* tw = (const V*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  const bool first = it == 0;
  V tv[C::ET];
  colT_gload<C, 2>(tv, M0, M1, kx0, g.h);
  V rv[C::EP], xv[C::EP], dv[C::EP], sv[GR ? 1 : C::EP];
  auto load_vectors = [&]() {
    colP_gload<C>(rv, rh, kx0, g.h);
    if (!first) {
      colP_gload<C>(dv, dh, kx0, g.h);
      if constexpr (!GR) colP_gload<C>(sv, sh, kx0, g.h);
    }
    colP_gload<C>(xv, xh, kx0, g.h);
  };
  if constexpr (EARLY) load_vectors();
  double K[4];
  for (int i = 0; i < 3; ++i) K[i] = st->kbar[i];
  const double ga = st->rho[it & 1], ga_prev = st->rho[(it + 1) & 1], al_prev = st->alpha[(it + 1) & 1];
  const int budget = st->budget;
  {
    const double* part = slot_ptr(g.part, SLOT_P3);
    double s[1] = {0.0};
    for (int i = threadIdx.x; i < nwg_row; i += C::NT) s[0] += part[i];
    wave_sums<1>(s, red);
  }
  colT_put<C, 2>(buf, tv);
  __syncthreads();
  lds_fft<T, -1, NY, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
  if constexpr (!EARLY) load_vectors();
  double beta = pcg_beta(ga, ga_prev, first);
  const double alpha = pcg_alpha<T>(ga, waves_total<NW>(red), al_prev, first, beta);
  const bool bad = !isfinite(ga) || !isfinite(alpha);
  const bool stop = bad || it + 1 >= max_iter || it + 1 >= budget;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->alpha[it & 1] = alpha;
    st->iters = it + 1;
    if (bad) st->flags |= FLAG_NONFINITE;
    if (stop) {
      st->conv_at = it + 1;
      st->converged = 0;
    }
  }
  const T a = (T)alpha, bt = (T)beta;
  double ps[2] = {0.0, 0.0};
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    const int c = p / NY, ky = p % NY;
    const int kx = kx0 + c;
    if (p >= C::CN) continue;
    V* px = buf + c * C::LS + ky;
    V* py = buf + (C::C + c) * C::LS + ky;
    V z = vzero<V>();
    const double xx = xi_col(kx, g.lx), yy = xi_tilde(ky, NY, g.ly);
    if (kx < g.h) {
      const V fx = *px, fy = *py;
      // w = -i (xx Fx + yy Fy)
      const T ax = (T)xx * fx.x + (T)yy * fy.x, ay = (T)xx * fx.y + (T)yy * fy.y;
      const V w = mk<T>(ay, -ax);
      const T sig = (T)precond_symbol_inv(K, xx, yy);
      V rn = rv[i];
      const V zo = scl(rn, sig);
      const V d = first ? zo : add(zo, scl(dv[i], bt));
      V s = w;
      if constexpr (!GR) {
        if (!first) s = add(w, scl(sv[i], bt));
      }
      const size_t idx = (size_t)kx * NY + ky;
      xh[idx] = add(xv[i], scl(d, a));
      rn = sub(rn, scl(s, a));
      rh[idx] = rn;
      dh[idx] = d;
      if constexpr (!GR) sh[idx] = s;
      const double wr = (kx == 0 ? 1.0 : 2.0) * ((double)rn.x * rn.x + (double)rn.y * rn.y);
      ps[0] += wr;
      ps[1] += (double)sig * wr;
      z = scl(rn, sig);
    }
    // the gradient of z takes the places of the flux values this thread read
    const T sx = (T)(xx * g.inv_n), sy = (T)(yy * g.inv_n);
    *px = mk<T>(-sx * z.y, sx * z.x);
    *py = mk<T>(-sy * z.y, sy * z.x);
  }
  wave_sums<2>(ps, red2);
  __syncthreads();
  if (!stop) {
    lds_fft<T, +1, NY, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
    colT_store<C, 2>(buf, M0, M1, kx0, g.h);
  }
  if (threadIdx.x < 2) slot_ptr(g.part, SLOT_RR)[threadIdx.x * MAX_WG + blockIdx.x] = waves_total<NW>(red2 + threadIdx.x * NW);
  tclk_end(g, 2, it + 1);
}
// The column pass with one field at a time through one field's LDS (column
// variants from CV_SEQ to below CV_WIDE): w is summed up in registers, grad_x leaves before
// grad_y is formed.  Half the LDS and, for the same elements per thread, half
// the threads per workgroup, so twice the workgroups share a compute unit.
template <int NY, typename T, int CV>
__device__ __forceinline__ void col_iter_seq_body(Geo g, cx<T>* M0, cx<T>* M1, cx<T>* __restrict__ xh,
                                                  cx<T>* __restrict__ rh, cx<T>* __restrict__ dh,
                                                  cx<T>* __restrict__ sh, int it, int max_iter, int nwg_row) {
  using C = DivCfg<NY, CV>;
  using V = cx<T>;
  constexpr int NW = C::NT / 64;
  constexpr bool GR = grad_rec<T>();
  DevStatus* st = g.st;
  if (st->conv_at <= it) return;
  tclk_start(g, 2, it + 1);
  __shared__ V buf[C::NB * C::LS];
  __shared__ double red[NW];
  __shared__ double red2[2 * NW];
  const V* tw = (const V*)g.tw;
  const int kx0 = blockIdx.x * C::C;
  const bool first = it == 0;
  V tv[C::EP], w[C::EP];
  colP_gload<C>(tv, M0, kx0, g.h);
  double K[4];
  for (int i = 0; i < 3; ++i) K[i] = st->kbar[i];
  const double ga = st->rho[it & 1], ga_prev = st->rho[(it + 1) & 1], al_prev = st->alpha[(it + 1) & 1];
  const int budget = st->budget;
  {
    const double* part = slot_ptr(g.part, SLOT_P3);
    double s[1] = {0.0};
    for (int i = threadIdx.x; i < nwg_row; i += C::NT) s[0] += part[i];
    wave_sums<1>(s, red);
  }
  auto put = [&]() {
#pragma unroll
    for (int i = 0; i < C::EP; ++i) {
      const int p = threadIdx.x + i * C::NT;
      if (p < C::CN) buf[(p / NY) * C::LS + p % NY] = tv[i];
    }
    __syncthreads();
  };
  put();
  colP_gload<C>(tv, M1, kx0, g.h);
  lds_fft<T, -1, NY, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
#pragma unroll
  for (int i = 0; i < C::EP; ++i) {
    const int p = threadIdx.x + i * C::NT;
    if (p >= C::CN) continue;
    const T xx = (T)xi_col(kx0 + p / NY, g.lx);
    const V f = buf[(p / NY) * C::LS + p % NY];
    w[i] = mk<T>(xx * f.y, -xx * f.x);
  }
  __syncthreads();
  put();
  lds_fft<T, -1, NY, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
  double beta = pcg_beta(ga, ga_prev, first);
  const double alpha = pcg_alpha<T>(ga, waves_total<NW>(red), al_prev, first, beta);
  const bool bad = !isfinite(ga) || !isfinite(alpha);
  const bool stop = bad || it + 1 >= max_iter || it + 1 >= budget;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->alpha[it & 1] = alpha;
    st->iters = it + 1;
    if (bad) st->flags |= FLAG_NONFINITE;
    if (stop) {
      st->conv_at = it + 1;
      st->converged = 0;
    }
  }
  const T a = (T)alpha, bt = (T)beta;
  double ps[2] = {0.0, 0.0};
  // w becomes z = M^-1 r of the new residual; a few elements at a time, their
  // vector loads in flight together
  constexpr int HE = C::EP > 4 ? 4 : C::EP;
#pragma unroll
  for (int i0 = 0; i0 < C::EP; i0 += HE) {
    V rv[HE], xv[HE], dv[HE], sv[GR ? 1 : HE];
#pragma unroll
    for (int q = 0; q < HE; ++q) {
      const int p = threadIdx.x + (i0 + q) * C::NT;
      const bool ok = p < C::CN && kx0 + p / NY < g.h;
      const size_t idx = (size_t)kx0 * NY + p;
      rv[q] = ok ? rh[idx] : vzero<V>();
      dv[q] = ok && !first ? dh[idx] : vzero<V>();
      if constexpr (!GR) sv[q] = ok && !first ? sh[idx] : vzero<V>();
      xv[q] = ok ? xh[idx] : vzero<V>();
    }
#pragma unroll
    for (int q = 0; q < HE; ++q) {
      const int p = threadIdx.x + (i0 + q) * C::NT;
      if (p >= C::CN) continue;
      const int kx = kx0 + p / NY, ky = p % NY;
      V z = vzero<V>();
      if (kx < g.h) {
        const double xx = xi_col(kx, g.lx), yy = xi_tilde(ky, NY, g.ly);
        const V fy = buf[(p / NY) * C::LS + ky];
        const V wv = mk<T>(w[i0 + q].x + (T)yy * fy.y, w[i0 + q].y - (T)yy * fy.x);
        const T sig = (T)precond_symbol_inv(K, xx, yy);
        V rn = rv[q];
        const V zo = scl(rn, sig);
        const V d = first ? zo : add(zo, scl(dv[q], bt));
        V s = wv;
        if constexpr (!GR) {
          if (!first) s = add(wv, scl(sv[q], bt));
        }
        const size_t idx = (size_t)kx0 * NY + p;
        xh[idx] = add(xv[q], scl(d, a));
        rn = sub(rn, scl(s, a));
        rh[idx] = rn;
        dh[idx] = d;
        if constexpr (!GR) sh[idx] = s;
        const double wr = (kx == 0 ? 1.0 : 2.0) * ((double)rn.x * rn.x + (double)rn.y * rn.y);
        ps[0] += wr;
        ps[1] += (double)sig * wr;
        z = scl(rn, sig);
      }
      w[i0 + q] = z;
    }
  }
  wave_sums<2>(ps, red2);
  if (!stop) {
#pragma unroll
    for (int f = 0; f < 2; ++f) {
#pragma unroll
      for (int i = 0; i < C::EP; ++i) {
        const int p = threadIdx.x + i * C::NT;
        if (p >= C::CN) continue;
        const int ky = p % NY;
        const T sc = (T)((f == 0 ? xi_col(kx0 + p / NY, g.lx) : xi_tilde(ky, NY, g.ly)) * g.inv_n);
        buf[(p / NY) * C::LS + ky] = mk<T>(-sc * w[i].y, sc * w[i].x);
      }
      __syncthreads();
      lds_fft<T, +1, NY, C::NB, C::LS, C::NT, C::PLAN>(buf, tw, g.twn);
      V* dst = f == 0 ? M0 : M1;
#pragma unroll
      for (int i = 0; i < C::EP; ++i) {
        const int p = threadIdx.x + i * C::NT;
        if (p < C::CN && kx0 + p / NY < g.h) dst[(size_t)kx0 * NY + p] = buf[(p / NY) * C::LS + p % NY];
      }
      if (f == 0) __syncthreads();
    }
  }
  __syncthreads();
  if (threadIdx.x < 2) slot_ptr(g.part, SLOT_RR)[threadIdx.x * MAX_WG + blockIdx.x] = waves_total<NW>(red2 + threadIdx.x * NW);
  tclk_end(g, 2, it + 1);
}
template <int NY, typename T, int CV>
__global__ void __launch_bounds__((DivCfg<NY, CV>::NT)) k_col_iter(Geo g, cx<T>* M0, cx<T>* M1, cx<T>* xh, cx<T>* rh,
                                                    cx<T>* dh, cx<T>* sh, int it, int max_iter, int nwg_row) {
  if constexpr (CV >= CV_SEQ && CV < CV_WIDE) col_iter_seq_body<NY, T, CV>(g, M0, M1, xh, rh, dh, sh, it, max_iter, nwg_row);
  else col_iter_body<NY, T, CV>(g, M0, M1, xh, rh, dh, sh, it, max_iter, nwg_row);
}
template <int NY, typename T, int CV>
__global__ void __launch_bounds__((DivCfg<NY, CV>::NT)) kb_col_iter(const IterArgs* __restrict__ A, int it, int max_iter, int nwg_row) {
  const IterArgs& a = A[blockIdx.y];
  if constexpr (CV >= CV_SEQ && CV < CV_WIDE) col_iter_seq_body<NY, T, CV>(a.g, (cx<T>*)a.M0, (cx<T>*)a.M1, (cx<T>*)a.xh, (cx<T>*)a.rh, (cx<T>*)a.dh, (cx<T>*)a.sh, it, max_iter, nwg_row);
  else col_iter_body<NY, T, CV>(a.g, (cx<T>*)a.M0, (cx<T>*)a.M1, (cx<T>*)a.xh, (cx<T>*)a.rh, (cx<T>*)a.dh, (cx<T>*)a.sh, it, max_iter, nwg_row);
}

// ---------------------------------------------------------------- dispatch
// A switch over the variant code that instantiates only the variants that exist
// for the size and real type.
#define NF_VARIANTS(V_) V_(0) V_(1) V_(2) V_(3) V_(4) V_(5) V_(6) V_(7) V_(8) V_(9) V_(10) V_(11) V_(12) V_(13) V_(14) V_(15) V_(16) V_(17) V_(18)

template <int NX, typename T, int RV>
static hipError_t flux_go(const Geo& g, cx<T>* G0, cx<T>* G1, const T* m, const T* r, int it, double* kslot,
                          int nwg_col, double tol2, float* lo, T* gd, hipStream_t s) {
  if constexpr (flux_var_exists<NX, RV, (int)sizeof(cx<T>)>()) {
    hipLaunchKernelGGL((k_row_flux<NX, T, RV>), dim3(row_nwg_var(g, RV)), dim3(FluxCfg<NX, RV>::NT), 0, s, g, G0, G1, m,
                       r, it, kslot, nwg_col, tol2, lo, gd);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}
template <int NX, typename T>
static hipError_t flux_var(int rv, const Geo& g, cx<T>* G0, cx<T>* G1, const T* m, const T* r, int it,
                           double* kslot, int nwg_col, double tol2, float* lo, T* gd, hipStream_t s) {
  switch (rv) {
#define V_(K) \
  case K: return flux_go<NX, T, K>(g, G0, G1, m, r, it, kslot, nwg_col, tol2, lo, gd, s);
    NF_VARIANTS(V_)
#undef V_
    default: return hipErrorInvalidValue;
  }
}
template <int NX, typename T, int RV>
static hipError_t fluxb_go(const Geo& g, const FluxArgs* A, int count, int it, int nwg_col, double tol2,
                           hipStream_t s) {
  if constexpr (flux_var_exists<NX, RV, (int)sizeof(cx<T>)>()) {
    hipLaunchKernelGGL((kb_row_flux<NX, T, RV>), dim3(row_nwg_var(g, RV), count), dim3(FluxCfg<NX, RV>::NT), 0, s, A, it,
                       nwg_col, tol2);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}
template <int NX, typename T>
static hipError_t fluxb_var(int rv, const Geo& g, const FluxArgs* A, int count, int it, int nwg_col, double tol2,
                            hipStream_t s) {
  switch (rv) {
#define V_(K) \
  case K: return fluxb_go<NX, T, K>(g, A, count, it, nwg_col, tol2, s);
    NF_VARIANTS(V_)
#undef V_
    default: return hipErrorInvalidValue;
  }
}
template <int NY, typename T, int CV>
static hipError_t iter_go(const Geo& g, cx<T>* M0, cx<T>* M1, cx<T>* xh, cx<T>* rh, cx<T>* dh, cx<T>* sh, int it,
                          int max_iter, int nwg_row, hipStream_t s) {
  if constexpr (div_var_exists<NY, CV, (int)sizeof(cx<T>)>()) {
    hipLaunchKernelGGL((k_col_iter<NY, T, CV>), dim3(col_nwg_var(g, CV)), dim3(DivCfg<NY, CV>::NT), 0, s, g, M0, M1, xh,
                       rh, dh, sh, it, max_iter, nwg_row);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}
template <int NY, typename T>
static hipError_t iter_var(int cv, const Geo& g, cx<T>* M0, cx<T>* M1, cx<T>* xh, cx<T>* rh, cx<T>* dh, cx<T>* sh,
                           int it, int max_iter, int nwg_row, hipStream_t s) {
  switch (cv) {
#define V_(K) \
  case K: return iter_go<NY, T, K>(g, M0, M1, xh, rh, dh, sh, it, max_iter, nwg_row, s);
    NF_VARIANTS(V_)
#undef V_
    default: return hipErrorInvalidValue;
  }
}
template <int NY, typename T, int CV>
static hipError_t iterb_go(const Geo& g, const IterArgs* A, int count, int it, int max_iter, int nwg_row,
                           hipStream_t s) {
  if constexpr (div_var_exists<NY, CV, (int)sizeof(cx<T>)>()) {
    hipLaunchKernelGGL((kb_col_iter<NY, T, CV>), dim3(col_nwg_var(g, CV), count), dim3(DivCfg<NY, CV>::NT), 0, s, A, it,
                       max_iter, nwg_row);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}
template <int NY, typename T>
static hipError_t iterb_var(int cv, const Geo& g, const IterArgs* A, int count, int it, int max_iter, int nwg_row,
                            hipStream_t s) {
  switch (cv) {
#define V_(K) \
  case K: return iterb_go<NY, T, K>(g, A, count, it, max_iter, nwg_row, s);
    NF_VARIANTS(V_)
#undef V_
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nf
