// The whole PCG loop of a mid-size 2D grid (65537 points to about a million) in one
// launch over the chip, one workgroup per compute unit.
//
// As two launches per iteration such a grid's loop costs two kernel boundaries, reads
// and writes x, r, d, s, m and r of every point, and forms the preconditioner anew.
// Here the tiles of the two passes of nf_loop.hpp stay with one workgroup for the
// whole loop: r, d, s of its columns (FP32: instead of s the gradient of d on its
// rows), symbols and twiddles in registers, x and m, r of its rows in LDS (tiles of
// 2048 elements leave x and r in the L2), and only the two mixed fields move between
// the passes, 64 instead of 152 bytes per point and iteration.  The L2s of the XCDs
// meet in the Infinity Cache, so the fields are stored and loaded with sc1 (past the
// L2); invalidating the L2s instead and loading through them measured 2 to 3 times
// slower.  A round of store, barrier and load over 256 workgroups takes 3.7 us for
// 512^2 and 6.3 us for 1024^2, the barrier alone 1.7.
// Measured per solve, launches -> team (same box): 400^2 2.27 -> 1.58 ms, 512^2 2.26 ->
// 1.41, 1024x512 3.44 -> 1.81, 800^2 4.17 -> 3.34, 1024^2 4.40 -> 3.44; FP32-refined
// 512x1024 3.01 -> 1.89, 1024^2 4.77 -> 2.94.  Of an iteration of 512^2 (32000 cycles)
// the two waits take 14000, the transforms 9000, loads and stores 6000: the loop is
// bound by the barrier's round trips and, on the larger tiles, by LDS traffic and the
// few registers that are left.
//
// A team takes all compute units, so a loop is one launch only if no other loop or
// ensemble is in progress on the device; concurrent loops overlap better as launches
// (three 512^2 handles: 1.21e9 grid-point steps per second with this rule, 1.16e9 with
// the tuned launches; three 1024^2 handles: 1.69e9 with teams, 2.1e9 as launches).
//
// Exchange layout: [row tile][kx][field][row] in the buffers of d and A d (FP32: the
// first half of that of the gradient), which the loop keeps in registers; kx below Nx/4 in the first, the others in the second, so
// that the two members of a real-transform pair come from one buffer each.  A row
// pass reads and writes one contiguous block per buffer, a column pass runs of 2 C
// rows.  Every pass writes where it has read: with a second layout for the
// gradient, contiguous for the column pass, the waits grew from 14000 to 19000
// cycles per iteration at 512^2 (presumably since the lines then are in another XCD's L2).
//
// A member does the work of one or two workgroups of the launched passes, and the
// totals are added up in the order in which those passes add them, so the results are
// bitwise those of the launches, which ensembles, timed and concurrent handles and
// handles whose team did not form run.  Tiles of 512 and 1024 elements are variants of
// their own (RV_WIDE, CV_WIDE: with 128 and 256 threads and radix 8 the 512^2 solve
// took 1.86 ms); tiles of 2048 elements are pairs of the launches' tuned tiles, since
// launches of 2048-element tiles cost three concurrent 1024^2 handles 14%.
//
// Formation is that of nf_team.hpp: all members draw tickets; the last one turns
// OPEN to GO, a member that waited CHIP_FORM_MS turns it to ABORT.  After GO all
// members are running, so every wait below ends; it is bounded all the same, and a
// member that gives one up records that the loop is lost.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

// see nf_loop.hpp: the launches and this kernel have to round alike
#pragma clang fp contract(on)

#include "nf_fft.hpp"
#include "nf_internal.h"
#include "nf_team.hpp"
#include "nf_tiles.hpp"

namespace nf {

constexpr double CHIP_FORM_MS = 5.0;
constexpr unsigned CHIP_POLLS = 1u << 22;  // polls (a second or more) before a member counts as lost

__device__ __forceinline__ void chip_store(__amdgpu_buffer_rsrc_t b, int i, cx<double> v) {
  union {
    u32x4 u;
    cx<double> c;
  } w;
  w.c = v;
  __builtin_amdgcn_raw_buffer_store_b128(w.u, b, i * 16, 0, TEAM_SC1);
}
__device__ __forceinline__ void chip_store(__amdgpu_buffer_rsrc_t b, int i, cx<float> v) {
  union {
    u32x2 u;
    cx<float> c;
  } w;
  w.c = v;
  __builtin_amdgcn_raw_buffer_store_b64(w.u, b, i * 8, 0, TEAM_SC1);
}

// A thread's twiddles of a length-L transform over B lines, all stages after
// the first, in stage order: the same in every iteration.  From the table they
// cost more than the butterflies (a wave's load gathers up to 24 cache lines; per
// iteration of 512^2 41500 cycles with the table, 33700 with these registers).
template <int L, int B, int NT>
constexpr int chip_per(int S) { return (B * (L / mplan_radix(L, S, wide_plan(L))) + NT - 1) / NT; }
template <int L, int B, int NT>
constexpr int chip_tw_off(int S) {
  int o = 0;
  for (int s = 1; s < S; ++s) o += chip_per<L, B, NT>(s) * (mplan_radix(L, s, wide_plan(L)) - 1);
  return o;
}
constexpr int CHIP_TW = 14;
// whether stage S's twiddles are held (the last ones of 2048-element tiles are not)
template <int L, int B, int NT>
constexpr bool chip_held(int S) {
  return chip_tw_off<L, B, NT>(S) + chip_per<L, B, NT>(S) * (mplan_radix(L, S, wide_plan(L)) - 1) <= CHIP_TW;
}
template <typename T, int L, int B, int NT, int S = 1>
__device__ __forceinline__ void chip_tw_load(cx<T> (&wt)[CHIP_TW], const cx<T>* __restrict__ tw, int twn, int tid) {
  if constexpr (S < mplan_nstages(L, wide_plan(L))) {
    constexpr int R = mplan_radix(L, S, wide_plan(L)), NS = mplan_ns(L, S, wide_plan(L)), O = chip_tw_off<L, B, NT>(S);
    if constexpr (chip_held<L, B, NT>(S)) {
      const int mult = twn / (NS * R);
#pragma unroll
      for (int b = 0; b < chip_per<L, B, NT>(S); ++b) {
        const int k = (tid + b * NT) % (L / R) % NS;
#pragma unroll
        for (int q = 1; q < R; ++q) wt[O + b * (R - 1) + q - 1] = tw[q * k * mult];
      }
    }
    chip_tw_load<T, L, B, NT, S + 1>(wt, tw, twn, tid);
  }
}
// The transform of lds_fft with the plan of the wide tiles and these twiddles.
template <typename T, int DIR, int L, int B, int LS, int NT, int S = 0>
__device__ __forceinline__ void chip_fft(cx<T>* buf, const cx<T> (&wt)[CHIP_TW], const cx<T>* __restrict__ tw, int twn,
                                         int tid) {
  if constexpr (S < mplan_nstages(L, wide_plan(L))) {
    constexpr int R = mplan_radix(L, S, wide_plan(L)), NS = mplan_ns(L, S, wide_plan(L)), Q = L / R, NBF = B * Q;
    constexpr int PER = chip_per<L, B, NT>(S), O = chip_tw_off<L, B, NT>(S > 0 ? S : 1);
    constexpr bool EXACT = PER * NT == NBF, WL = wave_local_ok<L, NT, wide_plan(L)>(), POW2 = (L & (L - 1)) == 0;
    constexpr bool PIN = S > 0, POUT = S + 1 < mplan_nstages(L, wide_plan(L)), HELD = S == 0 || chip_held<L, B, NT>(S);
    cx<T> v[PER][R], w[PER][R];
#pragma unroll
    for (int b = 0; b < PER; ++b) {
      const int f = tid + b * NT, j = f % Q;
      if (EXACT || f < NBF) {
        const cx<T>* src = buf + f / Q * LS;
#pragma unroll
        for (int q = 0; q < R; ++q) v[b][q] = src[PIN ? team_pad<POW2>(j, q * Q) : j + q * Q];
        if constexpr (!HELD) {
#pragma unroll
          for (int q = 1; q < R; ++q) w[b][q] = tw[q * (j % NS) * (twn / (NS * R))];
        }
      }
    }
    if constexpr (WL) wave_sync();
    else __syncthreads();
#pragma unroll
    for (int b = 0; b < PER; ++b) {
      const int f = tid + b * NT, j = f % Q, k = j % NS;
      if (EXACT || f < NBF) {
        if constexpr (S > 0) {
#pragma unroll
          for (int q = 1; q < R; ++q) {
            if constexpr (HELD) w[b][q] = wt[O + b * (R - 1) + q - 1];
            v[b][q] = mul(v[b][q], DIR > 0 ? conj(w[b][q]) : w[b][q]);
          }
        }
        dft<R, DIR>(v[b]);
        cx<T>* dst = buf + f / Q * LS;
        const int o = j / NS * NS * R + k;
#pragma unroll
        for (int q = 0; q < R; ++q) dst[POUT ? team_pad<POW2>(o, q * NS) : o + q * NS] = v[b][q];
      }
    }
    if constexpr (WL && POUT) wave_sync();
    else __syncthreads();
    chip_fft<T, DIR, L, B, LS, NT, S + 1>(buf, wt, tw, twn, tid);
  }
}

// The thread index as a value the compiler cannot follow: otherwise it hoists the
// addresses of all the lengths out of the loop, keeps the twiddles of a forward
// transform for the inverse one, and spills.
__device__ __forceinline__ void chip_opaque(int& t) { asm volatile("" : "+v"(t)); }

// The split of a grid.  A grid has a team over the chip if it has more than 65536
// points (below, the team of one XCD has the cheaper barrier) and tiles of the
// smallest class that holds it in at most 256 members, one per compute unit, divide
// it, so that the exchange layouts have no ragged blocks, and are covered by their
// threads; G is 0 otherwise.
__host__ __device__ constexpr ChipShape chip_split(int nx, int ny) {
  ChipShape cs{0, 0, 0, 0, 0, 0, 0};
  const int h = nx / 2;
  if ((long long)nx * ny <= 65536) return cs;
  for (int c = 0; c < 3; ++c) {
    if (!wide_row_ok(nx) || !wide_col_ok(ny) || wide_elems(c) < h || wide_elems(c) < ny) continue;
    if (c == 2 && (h == 256 || ny == 256)) continue;  // (their launches would have another plan)
    const int R = c < 2 ? wide_elems(c) / h : 2 * tile_rows(h, TILE), C = c < 2 ? wide_elems(c) / ny : 2 * cv_cols_default(ny);
    if (ny % R != 0 || h % 2 != 0 || h / 2 % C != 0) continue;
    const int nrow = ny / R, ncol = h / C, G = nrow > ncol ? nrow : ncol;
    const int step = wide_threads(c) / (2 * R * C);
    if (G > CHIP_MAX || step * 2 * wide_elems(c) < nrow * wide_threads(c)) continue;
    return ChipShape{G, c, R, C, nrow, ncol, step};
  }
  return cs;
}
// Launched tiles per member and pass, and the threads of those tiles: class 2 is two
// tiles of TILE elements (256 threads), except that the rows of tuned lengths are
// one tile of 512 threads, the tuner's choice there.
__host__ __device__ constexpr int chip_sr(int nx, int c) { return c < 2 || var_size(nx) ? 1 : 2; }
__host__ __device__ constexpr int chip_sc(int c) { return c < 2 ? 1 : 2; }
__host__ __device__ constexpr int chip_threads(int nx, int ny) {
  return chip_split(nx, ny).G > 0 ? wide_threads(chip_split(nx, ny).wide) : 64;
}

__host__ __device__ constexpr int chip_ep(int nx, int ny) {
  return wide_elems(chip_split(nx, ny).wide) / wide_threads(chip_split(nx, ny).wide);
}

// Line strides of the LDS tiles: the padded transform layout, on which the eight
// lanes of a 128-byte access of the exchange image (row, field, then line) fall
// on distinct bank groups.
__host__ __device__ constexpr int chip_ls(int len, int lines) {
  const int want = lines <= 1 ? 4 : (lines == 2 ? 2 : 1);
  return lpad_len(len) + ((want - lpad_len(len) % 8) + 8) % 8;
}
// complex elements of a tile's LDS, class c
constexpr int chip_lds(int c) { return 2 * wide_elems(c) + wide_elems(c) / 4 + 100; }
// the largest class keeps in global memory (in the L2) what no longer fits
constexpr bool chip_big(int c) { return wide_elems(c) > 1024; }

// Element i of a thread in the pointwise phases: that of the launched tiles, SUB of
// which share the N elements of the member; at least N if there is none.
template <int NT, int SUB, int N>
__host__ __device__ constexpr int chip_elem(int tid, int i) {
  constexpr int NS = NT / SUB, M = N / SUB;
  const int p = tid % NS + i * NS;
  return SUB == 1 ? p : (p < M ? tid / NS * M + p : N);
}
// Task t of a row tile at element `base` (its first row times Nx/2) covers the entries k
// and pair_mirror(k) of one line; the first is element base + t of the lower exchange
// buffer, this is the other one's place in the upper.
template <int H, int R>
__host__ __device__ constexpr int chip_hi(int base, int t) {
  return base + ((pair_mirror(t / (2 * R), H) - H / 2) * 2 + (t / R & 1)) * R + t % R;
}
// Exchange image of a column tile: the 2 C R elements of a row tile are
// consecutive lanes (row, field, column), as many row tiles at a time as fit the
// threads; later ones follow at a fixed stride.  Of thread tid: the row tile of its
// first element (beyond all if it has none), that element's place in the exchange
// buffer of the tile's half and in LDS.
struct ChipPlace {
  int t, go, li;
};
template <int NX, int NY>
__host__ __device__ constexpr ChipPlace chip_place(int kx0, int tid) {
  constexpr int NT = wide_threads(chip_split(NX, NY).wide), R = chip_split(NX, NY).R, NC = chip_split(NX, NY).C;
  constexpr int H = NX / 2, LS = chip_ls(NY, NC), w = 2 * NC * R, h2 = H / 2;
  const int rr = tid % R, f = tid / R & 1, c = tid % w / (2 * R);
  const int k0 = kx0 >= h2 ? kx0 - h2 : kx0;
  return ChipPlace{tid < NT / w * w && kx0 < H ? tid / w : INT_MAX / 2, tid / w * R * H + ((k0 + c) * 2 + f) * R + rr,
                   (f * NC + c) * LS + tid / w * R + rr};
}
// What a thread keeps for the whole loop (EP elements of a field): the vectors
// and symbols of its spectral elements; in FP32 the gradient of d at its grid-point
// pairs instead of s (see grad_rec).  (x and, for its grid-point pairs, m and r
// stay in LDS: in registers they made the members of 512 FP64 threads spill.)
template <typename T, int EP>
struct ChipState {
  cx<T> r[EP], d[EP], s[grad_rec<T>() ? 1 : EP];
  cx<T> gx[grad_rec<T>() ? EP : 1], gy[grad_rec<T>() ? EP : 1];
  T sig[EP];
  cx<T> wr[CHIP_TW], wc[CHIP_TW], wp[EP];  // twiddles of its row and column transforms and pairs
  ChipPlace at;  // of its first element of the exchange image
};

template <typename T, int NX, int CL, int R>
__device__ __forceinline__ void chip_row_setup(ChipState<T, wide_elems(CL) / wide_threads(CL)>& st, cx<T>* ms, const Geo& g,
                                               const T* __restrict__ m, const T* __restrict__ r, int y0, int tid) {
  constexpr int NT = wide_threads(CL), E = wide_elems(CL), H = NX / 2, RH = R * H;
  const int ny = g.ny;
  const size_t n = (size_t)NX * ny;
  const cx<T>* tw = (const cx<T>*)g.tw;
  chip_tw_load<T, H, 2 * R, NT>(st.wr, tw, g.twn, tid);
#pragma unroll
  for (int i = 0; i < E / NT; ++i) {
    const int p = tid + i * NT;
    if (!chip_big(CL)) st.wp[i] = tw[p < RH ? p / (2 * R) * (g.twn / NX) : 0];
    const size_t o = (size_t)(y0 + p / H) * NX + 2 * (p % H);
    const bool ok = p < RH && y0 < ny;
    ms[p] = ok ? *(const cx<T>*)(m + o) : vzero<cx<T>>();
    ms[E + p] = ok ? *(const cx<T>*)(m + n + o) : vzero<cx<T>>();
    if (!chip_big(CL)) ms[2 * E + p] = ok ? *(const cx<T>*)(r + o) : vzero<cx<T>>();
  }
}
template <typename T, int NX, int NY>
__device__ __forceinline__ void chip_col_setup(ChipState<T, chip_ep(NX, NY)>& st, const Geo& g, const double* K, int kx0, int tid) {
  constexpr int CL = chip_split(NX, NY).wide, NT = wide_threads(CL), NC = chip_split(NX, NY).C;
#pragma unroll
  for (int i = 0; i < chip_ep(NX, NY); ++i) {
    const int p = chip_elem<NT, chip_sc(CL), NC * NY>(tid, i);
    st.sig[i] = (T)precond_symbol_inv(K, xi_col(kx0 + p / NY, g.lx), xi_tilde(p % NY, NY, g.ly));
  }
  chip_tw_load<T, NY, 2 * NC, NT>(st.wc, (const cx<T>*)g.tw, g.twn, tid);
  st.at = chip_place<NX, NY>(kx0, tid);
}

// The gradient of d at a thread's grid-point pairs (FP32), from and to its buffer
// between launches, in units of pairs [2][Ny][Nx/2].
template <typename T, int NX, int NY, bool STORE>
__device__ __forceinline__ void chip_grad(ChipState<T, chip_ep(NX, NY)>& st, cx<T>* gd, int y0, int tid) {
  if constexpr (grad_rec<T>()) {
    constexpr int CL = chip_split(NX, NY).wide, H = NX / 2, RH = chip_split(NX, NY).R * H;
#pragma unroll
    for (int i = 0; i < chip_ep(NX, NY); ++i) {
      const int p = chip_elem<wide_threads(CL), chip_sr(NX, CL), RH>(tid, i);
      const bool ok = p < RH && y0 < NY;
      const size_t o = (size_t)y0 * H + p, n2 = (size_t)H * NY;
      if (STORE) {
        if (ok) {
          gd[o] = st.gx[i];
          gd[n2 + o] = st.gy[i];
        }
      } else {
        st.gx[i] = ok ? gd[o] : vzero<cx<T>>();
        st.gy[i] = ok ? gd[n2 + o] : vzero<cx<T>>();
      }
    }
  }
}

// Row pass of the tile at row y0 (see row_flux_body; bt: beta of the iteration, used
// in FP32 beyond the first one, it0 of the loop): this thread's part of sum g . K g.  lo, hi: the exchange buffers; G0, G1: the mixed fields in
// their usual layout, which the first pass after a launch reads.
template <typename T, int NX, int NY>
__device__ __forceinline__ double chip_row(ChipState<T, chip_ep(NX, NY)>& st, cx<T>* buf, const cx<T>* ms,
                                           const T* __restrict__ rg, const Geo& g, const cx<T>* G0,
                                           const cx<T>* G1, __amdgpu_buffer_rsrc_t lo, __amdgpu_buffer_rsrc_t hi, int y0,
                                           bool first, T bt, bool start, int tid) {
  constexpr int CL = chip_split(NX, NY).wide, NT = wide_threads(CL), E = wide_elems(CL), ny = NY;
  using V = cx<T>;
  constexpr int H = NX / 2, R = chip_split(NX, NY).R, EP = chip_ep(NX, NY), NTK = R * H, LS = chip_ls(H, R), ETP = (NTK + NT - 1) / NT;
  static_assert(2 * R * LS <= chip_lds(CL), "tile exceeds its LDS");
  const V* tw = (const V*)g.tw;
  const int base = y0 * H, mult = g.twn / NX;
  const bool on = NY / R == chip_split(NX, NY).G || y0 < ny;
  V a[ETP], b[ETP];
#pragma unroll
  for (int i = 0; i < ETP; ++i) {
    const int t = tid + i * NT;
    const int rr = t % R, f = t / R & 1, k = t / (2 * R);
    a[i] = b[i] = vzero<V>();
    if (t < NTK && on) {
      if (first) {
        const V* src = (f ? G1 : G0) + y0 + rr;
        a[i] = src[(size_t)k * ny];
        b[i] = src[(size_t)pair_mirror(k, H) * ny];
      } else {
        a[i] = team_load(lo, base + t, (V*)nullptr);
        b[i] = team_load(hi, chip_hi<H, R>(base, t), (V*)nullptr);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < ETP; ++i) {
    const int t = tid + i * NT;
    if (t >= NTK) continue;
    const int rr = t % R, f = t / R & 1, k = t / (2 * R);
    V* l = buf + (f * R + rr) * LS;
    if (k == 0) {
      const V p = a[i], xh = b[i];
      l[0] = mk<T>(p.x + p.y, p.x - p.y);
      l[H / 2] = mk<T>(xh.x + xh.x, -(xh.y + xh.y));
    } else {
      const V xk = a[i], xm = b[i];
      const V w = chip_big(CL) ? tw[k * mult] : st.wp[i];
      const V e1 = add(xk, conj(xm)), o1 = sub(xk, conj(xm));
      const V e2 = add(xm, conj(xk)), o2 = sub(xm, conj(xk));
      l[k] = add(e1, mul_i<+1>(mul(conj(w), o1)));
      l[H - k] = add(e2, mul_i<-1>(mul(w, o2)));
    }
  }
  __syncthreads();
  chip_opaque(tid);
  chip_fft<T, +1, H, 2 * R, LS, NT>(buf, st.wr, tw, g.twn, tid);
  chip_opaque(tid);
  double de = 0.0;
#pragma unroll
  for (int i = 0; i < EP; ++i) {
    const int p = chip_elem<NT, chip_sr(NX, CL), R * H>(tid, i);
    if (p < R * H && on) {
      V* px = buf + p / H * LS + p % H;
      V* py = px + R * LS;
      V gx = *px, gy = *py;
      if constexpr (grad_rec<T>()) {
        if (!start) {
          gx = add(gx, scl(st.gx[i], bt));
          gy = add(gy, scl(st.gy[i], bt));
        }
        st.gx[i] = gx;
        st.gy[i] = gy;
      }
      const V mx = ms[p], my = ms[E + p];
      const V rv = chip_big(CL) ? *(const V*)(rg + (size_t)(y0 + p / H) * NX + 2 * (p % H)) : ms[2 * E + p];
      const T a0 = mx.x * gx.x + my.x * gy.x;
      const T a1 = mx.y * gx.y + my.y * gy.y;
      const V fx = mk<T>(fma(a0, mx.x, rv.x * gx.x), fma(a1, mx.y, rv.y * gx.y));
      const V fy = mk<T>(fma(a0, my.x, rv.x * gy.x), fma(a1, my.y, rv.y * gy.y));
      *px = fx;
      *py = fy;
      de += (double)gx.x * fx.x + (double)gx.y * fx.y + (double)gy.x * fy.x + (double)gy.y * fy.y;
    }
  }
  __syncthreads();
  chip_opaque(tid);
  chip_fft<T, -1, H, 2 * R, LS, NT>(buf, st.wr, tw, g.twn, tid);
  chip_opaque(tid);
#pragma unroll
  for (int i = 0; i < ETP; ++i) {
    const int t = tid + i * NT;
    if (t >= NTK || !on) continue;
    const int rr = t % R, f = t / R & 1, k = t / (2 * R);
    const V* l = buf + (f * R + rr) * LS;
    const int oh = chip_hi<H, R>(base, t);
    if (k == 0) {
      const V z0 = l[0];
      chip_store(lo, base + t, mk<T>(z0.x + z0.y, z0.x - z0.y));
      chip_store(hi, oh, conj(l[H / 2]));
    } else {
      const V zk = l[k], zm = l[H - k];
      const V w = chip_big(CL) ? tw[k * mult] : st.wp[i];
      const V e1 = add(zk, conj(zm)), o1 = sub(zk, conj(zm));
      const V e2 = add(zm, conj(zk)), o2 = sub(zm, conj(zk));
      const V t1 = mul_i<-1>(mul(w, o1));
      const V t2 = mul_i<+1>(mul(conj(w), o2));
      chip_store(lo, base + t, scl(add(e1, t1), (T)0.5));
      chip_store(hi, oh, scl(add(e2, t2), (T)0.5));
    }
  }
  return de;
}

// Column pass of the tile at column kx0 (see col_iter_body) through its half's
// exchange buffer; ps: this thread's parts of ||r||^2 and <r, M^-1 r>.  The
// gradient stays in buf as well.
template <typename T, int NX, int NY>
__device__ __forceinline__ void chip_col(ChipState<T, chip_ep(NX, NY)>& st, cx<T>* buf, cx<T>* xs,
                                         cx<T>* xh, const Geo& g, __amdgpu_buffer_rsrc_t ex, int kx0,
                                         T a, T bt, bool first, bool last, double (&ps)[2], int tid) {
  constexpr ChipShape cs = chip_split(NX, NY);
  constexpr int CL = cs.wide, NT = wide_threads(CL), EP = chip_ep(NX, NY), H = NX / 2;
  constexpr int NC = cs.C, CN = NC * NY;
  using V = cx<T>;
  constexpr int LS = chip_ls(NY, NC);
  static_assert(2 * NC * LS <= chip_lds(CL), "tile exceeds its LDS");
  const V* tw = (const V*)g.tw;
  const bool on = cs.ncol == cs.G || kx0 < H;
  constexpr int dt = cs.step, dg = dt * cs.R * H, dl = dt * cs.R;
  V f[2 * EP];
#pragma unroll
  for (int i = 0; i < 2 * EP; ++i)
    if (st.at.t + i * dt < cs.nrow) f[i] = team_load(ex, st.at.go + i * dg, (V*)nullptr);
#pragma unroll
  for (int i = 0; i < 2 * EP; ++i)
    if (st.at.t + i * dt < cs.nrow) buf[st.at.li + i * dl] = f[i];
  __syncthreads();
  chip_fft<T, -1, NY, 2 * NC, LS, NT>(buf, st.wc, tw, g.twn, tid);
  ps[0] = ps[1] = 0.0;
#pragma unroll
  for (int i = 0; i < EP; ++i) {
    const int p = chip_elem<NT, chip_sc(CL), CN>(tid, i);
    if (p < CN && on) {
      V* px = buf + p / NY * LS + p % NY;
      V* py = px + NC * LS;
      const double xx = xi_col(kx0 + p / NY, g.lx), yy = xi_tilde(p % NY, NY, g.ly);
      const V fx = *px, fy = *py;
      // w = -i (xx Fx + yy Fy)
      const T ax = (T)xx * fx.x + (T)yy * fy.x, ay = (T)xx * fx.y + (T)yy * fy.y;
      const V w = mk<T>(ay, -ax);
      const T sig = st.sig[i];
      V rn = st.r[i];
      const V zo = scl(rn, sig);
      const V d = first ? zo : add(zo, scl(st.d[i], bt));
      V s = w;
      if constexpr (!grad_rec<T>()) {
        if (!first) s = add(w, scl(st.s[i], bt));
        st.s[i] = s;
      }
      if (!chip_big(CL)) xs[p] = add(xs[p], scl(d, a));
      rn = sub(rn, scl(s, a));
      st.r[i] = rn;
      st.d[i] = d;
      const double wr = (kx0 + p / NY == 0 ? 1.0 : 2.0) * ((double)rn.x * rn.x + (double)rn.y * rn.y);
      ps[0] += wr;
      ps[1] += (double)sig * wr;
      const V z = scl(rn, sig);
      const T sx = (T)(xx * g.inv_n), sy = (T)(yy * g.inv_n);
      *px = mk<T>(-sx * z.y, sx * z.x);
      *py = mk<T>(-sy * z.y, sy * z.x);
    }
  }
  __syncthreads();
  auto update_x = [&]() {
    if constexpr (chip_big(CL)) {
      cx<T>* xg = xh + (size_t)kx0 * NY;
      V xv[EP];
#pragma unroll
      for (int i = 0; i < EP; ++i) {
        const int p = chip_elem<NT, chip_sc(CL), CN>(tid, i);
        if (p < CN && on) xv[i] = xg[p];
      }
#pragma unroll
      for (int i = 0; i < EP; ++i) {
        const int p = chip_elem<NT, chip_sc(CL), CN>(tid, i);
        if (p < CN && on) xg[p] = add(xv[i], scl(st.d[i], a));
      }
    }
  };
  if (last) {
    update_x();
    return;
  }
  chip_opaque(tid);
  chip_fft<T, +1, NY, 2 * NC, LS, NT>(buf, st.wc, tw, g.twn, tid);
#pragma unroll
  for (int i = 0; i < 2 * EP; ++i)
    if (st.at.t + i * dt < cs.nrow) chip_store(ex, st.at.go + i * dg, buf[st.at.li + i * dl]);
  update_x();
}
template <typename T, int NY, int NC, int NT>
__device__ __forceinline__ void chip_col_out(const cx<T>* buf, cx<T>* M0, cx<T>* M1, int kx0, int h, int tid) {
  constexpr int LS = chip_ls(NY, NC), CN = NC * NY;
  if (kx0 >= h) return;
  for (int e = tid; e < 2 * CN; e += NT) {
    const int f = e / CN, c = e % CN / NY, ky = e % NY;
    (f ? M1 : M0)[(size_t)(kx0 + c) * NY + ky] = buf[(f * NC + c) * LS + ky];
  }
}

// The barrier of the team with K partial sums per tile.  Every tile leaves its sums
// in its slot of the set of the epoch's parity; member 0 waits for all of them,
// adds them up and publishes the totals in eight lines, which the others wait
// for (all members reading all slots: 2.2 us instead of 1.7 us over 256 members,
// 3.3 instead of 2.1 over 512).  A tile's slot of a set is rewritten only after
// the barrier in between.
// own: sum k of the tile in its thread k; scale multiplies them.
// Polls stay three deep in flight: a single one sees a value half a round trip
// late on average.  sh: chip_red(NT) doubles, which alternate between two halves.
__host__ __device__ constexpr int chip_red(int nt) { return 2 * (4 * (nt / 64) + 2); }
union ChipSlot {
  u32x4 u;
  double d[2];
};
// Wait until the entry at byte offset o carries the epoch in every active lane.
__device__ __forceinline__ bool chip_wait(__amdgpu_buffer_rsrc_t slots, int o, unsigned epoch, ChipSlot& w) {
  auto poll = [&]() {
    asm volatile("" ::: "memory");
    return __builtin_amdgcn_raw_buffer_load_b128(slots, o, 0, TEAM_SC1);
  };
  u32x4 a = poll(), b = poll(), c = poll();
  for (unsigned q = 0; q < CHIP_POLLS; ++q) {
    w.u = a;
    if (__all(w.u.z == epoch)) return true;
    a = b;
    b = c;
    c = poll();
  }
  return false;
}
// Q launched tiles per member, NTL threads of the launched pass that adds the sums up,
// XCD whether the tiles' places are those of xcd_block, quit whether a member but the
// first leaves without the totals.
template <int NT, int K, int Q, int NTL, bool XCD>
__device__ __forceinline__ bool chip_meet(__amdgpu_buffer_rsrc_t slots, int member, int ntiles, unsigned epoch,
                                          const double (&v)[K], double scale, double* sh, double& own, double (&tot)[K],
                                          bool quit = false) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63;
  sh += (epoch & 1) * (chip_red(NT) / 2);
  double* all = sh + K * NW;
  wave_sums<K>(v, sh);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const int set = (int)(epoch & 1) * (CHIP_TILES * 2), pub = 2 * CHIP_TILES * 2 + (int)(epoch & 1) * 64;
  ChipSlot w;
  if (threadIdx.x < Q * K) {
    const int q = threadIdx.x / K, k = threadIdx.x % K, t = member * Q + q;
    const int slot = XCD && ntiles % 8 == 0 ? t % (ntiles / 8) * 8 + t / (ntiles / 8) : t;
    own = waves_total<NW / Q>(sh + k * NW + q * (NW / Q)) * scale;
    w.d[0] = own;
    w.u.z = epoch;
    w.u.w = 0;
    if (t < ntiles) __builtin_amdgcn_raw_buffer_store_b128(w.u, slots, (set + slot * 2 + k) * 16, 0, TEAM_SC1);
  }
  double* okp = sh + 4 * NW;
  if (member == 0) {
    double s[K];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = 0.0;
    if (threadIdx.x < NTL) {
#pragma unroll
      for (int i = 0; i < (Q * CHIP_MAX + NTL - 1) / NTL; ++i) {
        const int t = threadIdx.x + i * NTL;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          ok = chip_wait(slots, (set + (t < ntiles ? t : 0) * 2 + k) * 16, epoch, w) && ok;
          if (t < ntiles) s[k] += w.d[0];
        }
      }
    }
    wave_sums<K>(s, all);
    if (!__syncthreads_and(ok)) return false;
#pragma unroll
    for (int k = 0; k < K; ++k) tot[k] = waves_total<NTL / 64>(all + k * NW);
    if (threadIdx.x < 8 * K) {
      w.d[0] = K == 2 && threadIdx.x % K == 1 ? tot[K - 1] : tot[0];
      w.u.z = epoch;
      w.u.w = 0;
      __builtin_amdgcn_raw_buffer_store_b128(w.u, slots, (pub + threadIdx.x / K * 8 + threadIdx.x % K) * 16, 0, TEAM_SC1);
    }
    return true;
  }
  if (threadIdx.x < 64) {
    const bool ok = !quit && chip_wait(slots, (pub + (member & 7) * 8 + lane % K) * 16, epoch, w);
    if (lane < K) all[lane] = w.d[0];
    if (lane == 0) okp[0] = ok ? 1.0 : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) tot[k] = all[k];
  return okp[0] != 0.0;
}

// Iterations it0 .. it0 + nk - 1 of the loop (fewer if it stops).  On entry the
// mixed buffers hold the gradient of z and status.rho the scalar gamma of
// iteration it0 (it0 > 0: status.alpha, d and s of the iteration before; sh holds s
// or, in FP32, the gradient of d, of which the exchange uses the first half).  On exit x, r (and, if iterations are left, d, s, the gradient and the partial sums) are
// written back and the status records the outcome as the launches of nf_loop.hpp
// do; status.team tells whether the team formed.
// A kernel per grid shape: one that switches between the lengths inside the loop
// keeps address and wavenumber terms of all of them and spills at 512 threads.
template <typename T, int NX, int NY>
__global__ void __launch_bounds__(chip_threads(NX, NY)) k_chip(Geo g, unsigned epoch, int lose, cx<T>* M0, cx<T>* M1,
                                                               const T* __restrict__ m, const T* __restrict__ r,
                                                               cx<T>* xh, cx<T>* rh, cx<T>* dh, cx<T>* sh, int it0,
                                                               int nk, int max_iter, double tol2) {
  using V = cx<T>;
  constexpr ChipShape cs = chip_split(NX, NY);
  constexpr int CL = cs.wide, NT = wide_threads(CL), E = wide_elems(CL), EP = E / NT;
  constexpr int SR = chip_sr(NX, CL), SC = chip_sc(CL), CN = cs.C * NY;
  DevStatus* st = g.st;
  TeamCtl* ctl = (TeamCtl*)g.team;
  if (st->conv_at <= it0) return;
  __shared__ V buf[chip_lds(CL)];
  __shared__ V ms[(chip_big(CL) ? 2 : 3) * E];  // pairs of m_x, m_y, r of the tile's rows
  __shared__ V xs[chip_big(CL) ? 1 : E];        // x of its columns
  __shared__ double red[chip_red(NT)];
  __shared__ int role_s, go_s;
  constexpr int G = cs.G;
  if (threadIdx.x == 0) {
    const int ticket = (int)__hip_atomic_fetch_add(&ctl->tickets, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    role_s = ticket;
    int state = TEAM_ABORT;
    if (ticket < G) {
      unsigned expect = TEAM_OPEN;
      if (ticket == G - 1)
        __hip_atomic_compare_exchange_strong(&ctl->state, &expect, (unsigned)TEAM_GO, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
      const unsigned long long t0 = wall_clock64();
      for (;;) {
        state = (int)__hip_atomic_load(&ctl->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (state != TEAM_OPEN) break;
        if (wall_clock64() - t0 > (unsigned long long)(CHIP_FORM_MS * 1e5)) {
          unsigned e2 = TEAM_OPEN;
          __hip_atomic_compare_exchange_strong(&ctl->state, &e2, (unsigned)TEAM_ABORT, __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    go_s = state;
  }
  __syncthreads();
  const int member = __builtin_amdgcn_readfirstlane(role_s);
  if (member >= G || go_s != TEAM_GO) return;

  const int tid = threadIdx.x;
  constexpr int h = NX / 2, ny = NY, nx = NX;
  const int bytes = h * ny * (int)sizeof(V);
  const __amdgpu_buffer_rsrc_t lo = team_rsrc(dh, bytes), hi = team_rsrc(sh, bytes);
  const __amdgpu_buffer_rsrc_t slots = team_rsrc(slot_ptr(g.part, SLOT_P3) + MAX_WG, CHIP_SLOTS * 16);
  const int kx0 = member * cs.C, y0 = member * cs.R;
  const bool upper = kx0 >= h / 2;
  ChipState<T, EP> S;
  {
    const size_t base = (size_t)kx0 * ny;
#pragma unroll
    for (int i = 0; i < EP; ++i) {
      const int p = chip_elem<NT, SC, CN>(tid, i);
      const bool ok = p < CN && kx0 < h;
      if (!chip_big(CL)) xs[p] = ok ? xh[base + p] : vzero<V>();
      S.r[i] = ok ? rh[base + p] : vzero<V>();
      S.d[i] = ok && it0 > 0 ? dh[base + p] : vzero<V>();
      if constexpr (!grad_rec<T>()) S.s[i] = ok && it0 > 0 ? sh[base + p] : vzero<V>();
    }
    if (it0 > 0) chip_grad<T, NX, NY, false>(S, sh, y0, tid);
  }
  const double K[4] = {st->kbar[0], st->kbar[1], st->kbar[2], 0.0};
  chip_row_setup<T, NX, CL, cs.R>(S, ms, g, m, r, y0, tid);
  chip_col_setup<T, NX, NY>(S, g, K, kx0, tid);
  const double bb = st->bb;
  const int budget = st->budget;
  double ga = st->rho[it0 & 1], ga_prev = st->rho[(it0 + 1) & 1], al_prev = st->alpha[(it0 + 1) & 1];
  const double npts = (double)((size_t)nx * ny);
  int it = it0;
  int outcome = TEAM_MORE;
  double rr = 0.0;
  double own = 0.0, od;
  bool bad = false;
  if (it0 > 0) {
    // d and s (or the gradient of d) are in registers everywhere before the first exchange store
    const double v0[1] = {0.0};
    double t0[1];
    if (!chip_meet<NT, 1, SC, NT / SC, false>(slots, member, cs.ncol * SC, ++epoch, v0, 1.0, red, od, t0)) outcome = TEAM_LOST;
    ++epoch;
  }
  for (; outcome == TEAM_MORE && it < it0 + nk; ++it) {
    int t = tid;
    chip_opaque(t);
    double de[1] = {0.0}, det[1];
    const T bt = grad_rec<T>() ? (T)pcg_beta(ga, ga_prev, it == 0) : (T)0;
    de[0] = chip_row<T, NX, NY>(S, buf, ms, r, g, M0, M1, lo, hi, y0, it == it0, bt, it == 0, t);
    if (!chip_meet<NT, 1, SR, NT / SC, true>(slots, member, cs.nrow * SR, ++epoch, de, npts, red, od, det)) {
      outcome = TEAM_LOST;
      break;
    }
    const TeamStep q = team_step<T>(ga, ga_prev, al_prev, det[0], it, max_iter, budget);
    bad = q.bad;
    double ps[2] = {0.0, 0.0}, pt[2];
    chip_col<T, NX, NY>(S, buf, xs, xh, g, upper ? hi : lo, kx0, (T)q.alpha, (T)q.beta, it == 0, q.stop,
                        ps, t);
    if (!chip_meet<NT, 2, SC, NT / SR, false>(slots, member, cs.ncol * SC, ++epoch, ps, 1.0, red, own, pt,
                                                   it + 1 == lose)) {
      outcome = TEAM_LOST;
      break;
    }
    rr = pt[0];
    al_prev = q.alpha;
    ga_prev = ga;
    ga = pt[1];
    if (q.stop) outcome = TEAM_STOP;
    else if (!isfinite(rr) || rr <= tol2 * bb) {
      bad = !isfinite(rr);
      outcome = TEAM_CONV;
    }
  }
  if (outcome != TEAM_LOST) {
    const size_t base = (size_t)kx0 * ny;
#pragma unroll
    for (int i = 0; i < EP; ++i) {
      const int p = chip_elem<NT, SC, CN>(tid, i);
      if (p < CN && kx0 < h) {
        if (!chip_big(CL)) xh[base + p] = xs[p];
        rh[base + p] = S.r[i];
        if (outcome == TEAM_MORE) {
          dh[base + p] = S.d[i];
          if constexpr (!grad_rec<T>()) sh[base + p] = S.s[i];
        }
      }
    }
    if (outcome == TEAM_MORE) {
      chip_grad<T, NX, NY, true>(S, sh, y0, tid);
      chip_col_out<T, NY, cs.C, NT>(buf, M0, M1, kx0, h, tid);
      if (tid < 2 * SC && member < cs.ncol) slot_ptr(g.part, SLOT_RR)[tid % 2 * MAX_WG + member * SC + tid / 2] = own;
    }
  }
  if (outcome == TEAM_LOST && threadIdx.x == 0) st->lost = 1;
  if (member == 0 && threadIdx.x == 0) {
    st->iters = it;
    st->rr[0] = rr;
    if (bad) st->flags |= FLAG_NONFINITE;
    if (outcome == TEAM_MORE) {
      st->rho[it & 1] = ga;
      st->rho[(it + 1) & 1] = ga_prev;
      st->alpha[(it + 1) & 1] = al_prev;
    } else if (outcome != TEAM_LOST) {
      st->converged = !bad && rr <= tol2 * bb ? 1 : 0;
      st->conv_at = it;
    }
    st->team = outcome;
  }
}

template <typename T, int NX, int NY>
static hipError_t chip_pair(const TeamGo& go, hipStream_t s) {
  if constexpr (chip_split(NX, NY).G > 0) {
    typedef cx<T> V;
    const FluxArgs& f = go.f;
    const IterArgs& a = go.a;
    hipLaunchKernelGGL((k_chip<T, NX, NY>), dim3(chip_split(NX, NY).G - (go.miss ? 1 : 0)), dim3(chip_threads(NX, NY)), 0, s, a.g, go.ts.epoch, go.ts.lose,
                       (V*)a.M0, (V*)a.M1, (const T*)f.m, (const T*)f.r, (V*)a.xh, (V*)a.rh, (V*)a.dh, (V*)a.sh, go.it,
                       go.nk, go.max_iter, go.tol2);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}
template <typename T, int NX>
static hipError_t chip_launch(const TeamGo& go, hipStream_t s) {
  switch (go.a.g.ny) {
    case 64: return chip_pair<T, NX, 64>(go, s);
    case 128: return chip_pair<T, NX, 128>(go, s);
    case 256: return chip_pair<T, NX, 256>(go, s);
    case 512: return chip_pair<T, NX, 512>(go, s);
    case 1024: return chip_pair<T, NX, 1024>(go, s);
    case 100: return chip_pair<T, NX, 100>(go, s);
    case 200: return chip_pair<T, NX, 200>(go, s);
    case 400: return chip_pair<T, NX, 400>(go, s);
    case 800: return chip_pair<T, NX, 800>(go, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nf
