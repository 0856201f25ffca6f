// The whole PCG loop of a small 2D grid in one launch (FP64 and FP32
// instantiations in nf_team64*.hip and nf_team32*.hip).
//
// On grids of up to 65536 points a loop pass is a chain of latencies: a launch,
// the status and partial sums of the pass before, a tile of a few KB through a
// handful of LDS stages.  Here a team of at most 32 workgroups on ONE XCD, a
// workgroup per compute unit, runs the iterations of nf_loop.hpp with x, r, d,
// s (FP32: the gradient of d), m and r of its columns and rows on chip.  Only the
// two mixed fields move between the passes, through that XCD's L2, and the passes
// meet at a barrier that carries the partial sums.  A store-barrier-load round of 32
// workgroups takes 0.84 us on one XCD (1.8 us over all XCDs, whose L2s meet in
// the Infinity Cache); two kernel boundaries with their reloads cost most of the
// 12 us of a 64^2 iteration.  Measured per iteration, launches -> team: 64^2 12
// -> 5.6 us, 128^2 12 -> 8 us, 200^2 20 -> 13 us, 256^2 15.2 -> 14 us (there the
// 1024 elements per field of each member fill a compute unit: larger grids
// use compute units of all XCDs, nf_chip.hpp).
//
// Visibility inside the team: stores go through the vector L1 to the L2 that
// the team shares; every wave waits for its stores (vmcnt 0) before the
// workgroup announces its arrival, and the other workgroups read with sc1
// loads, which miss the L1.
//
// Team formation.  The grid has workgroups for every XCD; those of the chosen
// one draw tickets, the first G form the team.  The member with the last ticket
// turns the team's state from OPEN to GO; a member that has waited
// TEAM_FORM_MS turns it from OPEN to ABORT.  Both are compare-and-swaps, so all
// members see the same outcome.  After ABORT (workgroups of other kernels kept
// members from becoming resident) nothing has been written.  After GO every
// member is resident and runs the same control flow, so every later wait ends;
// a wait of TEAM_WAIT_S seconds would end the kernel with an error all the same (any
// member records it: the others may have passed the last barrier).
//
// The same passes also exist as launches of their own (team_row_phase,
// team_col_phase, G workgroups per instance), which ensembles and handles whose
// team did not form use: the members' work and the order of every sum are those
// of the team, so the results agree bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

// Products are fused into sums within an expression only, not where the
// optimiser happens to find them: the team and the launches inline the same
// passes into different kernels and have to round alike.
#pragma clang fp contract(on)

#include "nf_fft.hpp"
#include "nf_internal.h"
#include "nf_tiles.hpp"

namespace nf {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int TEAM_SC1 = 16;       // cache policy of the exchange loads (agent scope: miss the vector L1)
constexpr int TEAM_EP = 2;         // spectral elements and grid-point pairs per thread
constexpr double TEAM_FORM_MS = 5.0, TEAM_WAIT_S = 2.0;

// A complex value of the exchange buffers, index i.
__device__ __forceinline__ cx<double> team_load(__amdgpu_buffer_rsrc_t b, int i, cx<double>*) {
  union {
    u32x4 u;
    cx<double> c;
  } v;
  v.u = __builtin_amdgcn_raw_buffer_load_b128(b, i * 16, 0, TEAM_SC1);
  return v.c;
}
__device__ __forceinline__ cx<float> team_load(__amdgpu_buffer_rsrc_t b, int i, cx<float>*) {
  union {
    u32x2 u;
    cx<float> c;
  } v;
  v.u = __builtin_amdgcn_raw_buffer_load_b64(b, i * 8, 0, TEAM_SC1);
  return v.c;
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t team_rsrc(void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x00027000);
}

// Radix plan of the team's transforms: 5s, then 4s, then a 2.  A member works on
// 2 * TEAM_EP elements per thread over its two fields, one radix-4 butterfly:
// radix 8 would leave half of the threads idle in stages that a single
// workgroup per compute unit spends on instruction latency.
constexpr int team_nstages(int n) {
  const int p = ilog2(n / pow5(f5(n)));
  return f5(n) + p / 2 + p % 2;
}
constexpr int team_radix(int n, int s) {
  const int p = ilog2(n / pow5(f5(n)));
  return s < f5(n) ? 5 : (s - f5(n) < p / 2 ? 4 : 2);
}
constexpr int team_ns(int n, int s) { return s == 0 ? 1 : team_ns(n, s - 1) * team_radix(n, s - 1); }
// Butterflies per thread of a radix-R stage.
__host__ __device__ constexpr int team_per(int R) { return R == 2 ? 2 : 1; }
// A thread's twiddles of a length-L transform, all stages after the first, in
// stage order: the same in every iteration, so the first TEAM_TW stay in
// registers (lengths up to 256 need no more); a later stage reads the table.
constexpr int TEAM_TW = 9;
template <int L>
constexpr int team_tw_off(int S) {
  int o = 0;
  for (int s = 1; s < S; ++s) o += team_per(team_radix(L, s)) * (team_radix(L, s) - 1);
  return o;
}
template <int L>
constexpr bool team_tw_held(int S) {
  return team_tw_off<L>(S) + team_per(team_radix(L, S)) * (team_radix(L, S) - 1) <= TEAM_TW;
}
// Padded index of element i + d of a line (see lpad), d known at compile time.
// Where the low three bits of i and d never carry (powers of two: the elements
// of a butterfly), it is lpad(i) plus a constant, which the LDS instructions
// take as their offset.
template <bool POW2>
__device__ __forceinline__ int team_pad(int i, int d) {
  return POW2 ? lpad(i) + lpad(d) : lpad(i + d);
}
template <typename T, int L, int NT, int S = 1>
__device__ __forceinline__ void team_tw_load(cx<T> (&wt)[TEAM_TW], const cx<T>* __restrict__ tw, int twn, int tid) {
  if constexpr (S < team_nstages(L)) {
    if constexpr (team_tw_held<L>(S)) {
      constexpr int R = team_radix(L, S), NS = team_ns(L, S), PER = team_per(R), O = team_tw_off<L>(S);
      const int mult = twn / (NS * R);
#pragma unroll
      for (int b = 0; b < PER; ++b) {
        const int k = (tid + b * NT) % (L / R) % NS;
#pragma unroll
        for (int q = 1; q < R; ++q) wt[O + b * (R - 1) + q - 1] = tw[q * k * mult];
      }
    }
    team_tw_load<T, L, NT, S + 1>(wt, tw, twn, tid);
  }
}

// One Stockham stage over nl lines of length L (see fft_stage of nf_fft.hpp) with
// the line count known at run time.
template <typename T, int DIR, int L, int LS, int NT, int S>
__device__ __forceinline__ void team_stage(cx<T>* buf, const cx<T> (&wt)[TEAM_TW], const cx<T>* __restrict__ tw, int twn,
                                           int nl, int tid) {
  constexpr int R = team_radix(L, S), NS = team_ns(L, S), Q = L / R, PER = team_per(R);
  constexpr bool HELD = S > 0 && team_tw_held<L>(S);
  constexpr int O = HELD ? team_tw_off<L>(S) : 0;
  constexpr bool PIN = S > 0, POUT = S + 1 < team_nstages(L), POW2 = (L & (L - 1)) == 0;
  const int nbf = nl * Q;
  cx<T> v[PER][R], w[PER][R];
#pragma unroll
  for (int b = 0; b < PER; ++b) {
    const int f = tid + b * NT;
    if (f < nbf) {
      const int j = f % Q;
      if constexpr (NS > 1) {
        const int k = j % NS, mult = twn / (NS * R);
#pragma unroll
        for (int q = 1; q < R; ++q) w[b][q] = HELD ? wt[O + b * (R - 1) + q - 1] : tw[q * k * mult];
      }
      const cx<T>* src = buf + (f / Q) * LS;
#pragma unroll
      for (int q = 0; q < R; ++q) v[b][q] = src[PIN ? team_pad<POW2>(j, q * Q) : j + q * Q];
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < PER; ++b) {
    const int f = tid + b * NT;
    if (f < nbf) {
      const int j = f % Q;
      if constexpr (NS > 1) {
#pragma unroll
        for (int q = 1; q < R; ++q) v[b][q] = mul(v[b][q], DIR > 0 ? conj(w[b][q]) : w[b][q]);
      }
      dft<R, DIR>(v[b]);
      cx<T>* dst = buf + (f / Q) * LS;
      const int o = (j / NS) * NS * R + j % NS;
#pragma unroll
      for (int q = 0; q < R; ++q) dst[POUT ? team_pad<POW2>(o, q * NS) : o + q * NS] = v[b][q];
    }
  }
  __syncthreads();
}
template <typename T, int DIR, int L, int LS, int NT, int S = 0>
__device__ __forceinline__ void team_fft(cx<T>* buf, const cx<T> (&wt)[TEAM_TW], const cx<T>* __restrict__ tw, int twn,
                                         int nl, int tid) {
  if constexpr (S < team_nstages(L)) {
    team_stage<T, DIR, L, LS, NT, S>(buf, wt, tw, twn, nl, tid);
    team_fft<T, DIR, L, LS, NT, S + 1>(buf, wt, tw, twn, nl, tid);
  }
}

// Line stride: the padded layout of a transform, odd multiples that spread the
// rows of a transposed access over the banks.
__host__ __device__ constexpr int team_ls(int L) { return (lpad_len(L) + 7) / 8 * 8 + 1; }

// What a thread keeps of its workgroup's columns and rows for the whole loop: the
// vectors, wavenumbers and inverse preconditioner symbol of its spectral
// elements, in FP32 the gradient of d at its grid-point pairs (see grad_rec), and
// the twiddles of its butterflies and real-transform pairs.  (m
// and r of its grid points stay in LDS: in registers they made 512-thread
// members spill.)
template <typename T>
struct TeamState {
  cx<T> x[TEAM_EP], r[TEAM_EP], d[TEAM_EP], s[grad_rec<T>() ? 1 : TEAM_EP];
  cx<T> gx[grad_rec<T>() ? TEAM_EP : 1], gy[grad_rec<T>() ? TEAM_EP : 1];
  double xx[TEAM_EP], yy[TEAM_EP], sig[TEAM_EP];
  cx<T> wc[TEAM_TW], wr[TEAM_TW], wp[TEAM_EP];
};

template <typename T, int NT, int NX>
__device__ __forceinline__ void team_row_setup(TeamState<T>& st, const Geo& g, int lr, int tid) {
  constexpr int H = NX / 2, NP = (H + 1) / 2;
  const cx<T>* tw = (const cx<T>*)g.tw;
  const int R = 1 << lr, mult = g.twn / NX;
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int t = tid + i * NT, u = t >= R * NP ? t - R * NP : t;
    st.wp[i] = t < 2 * R * NP ? tw[(u >> lr) * mult] : vzero<cx<T>>();
  }
  team_tw_load<T, H, NT>(st.wr, tw, g.twn, tid);
}
template <typename T, int NT, int NY>
__device__ __forceinline__ void team_col_setup(TeamState<T>& st, const Geo& g, const double* K, int kx0, int tid) {
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = tid + i * NT;
    st.xx[i] = xi_col(kx0 + p / NY, g.lx);
    st.yy[i] = xi_tilde(p % NY, NY, g.ly);
    st.sig[i] = precond_symbol_inv(K, st.xx[i], st.yy[i]);
  }
  team_tw_load<T, NY, NT>(st.wc, (const cx<T>*)g.tw, g.twn, tid);
}

// Row pass on the R = 1 << lr rows from y0 (see row_flux_body; bt: beta of the
// iteration, used in FP32 beyond the first): the return value is this thread's part
// of sum g . K g.
template <typename T, int NT, int NX>
__device__ __forceinline__ double team_row(TeamState<T>& st, cx<T>* buf, const cx<T>* mr, const Geo& g, cx<T>* M0, cx<T>* M1,
                                           __amdgpu_buffer_rsrc_t b0, __amdgpu_buffer_rsrc_t b1, int y0, int lr,
                                           T bt, bool first, int tid) {
  using V = cx<T>;
  constexpr int H = NX / 2, NP = (H + 1) / 2, LS = team_ls(H);
  const int R = 1 << lr, ntk = 2 * R * NP, ny = g.ny;
  V a[TEAM_EP], b[TEAM_EP];
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int t = tid + i * NT;
    a[i] = b[i] = vzero<V>();
    if (t < ntk) {
      const int f = t >= R * NP ? 1 : 0, u = t - f * R * NP;
      const int y = y0 + (u & (R - 1)), k = u >> lr;
      const __amdgpu_buffer_rsrc_t src = f ? b1 : b0;
      if (y < ny) {
        a[i] = team_load(src, k * ny + y, (V*)nullptr);
        if (k != 0 || H % 2 == 0) b[i] = team_load(src, pair_mirror(k, H) * ny + y, (V*)nullptr);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int t = tid + i * NT;
    if (t < ntk) {
      const int f = t >= R * NP ? 1 : 0, u = t - f * R * NP;
      const int k = u >> lr;
      V* l = buf + (f * R + (u & (R - 1))) * LS;
      if (k == 0) {
        l[0] = mk<T>(a[i].x + a[i].y, a[i].x - a[i].y);
        if (H % 2 == 0) l[H / 2] = mk<T>(b[i].x + b[i].x, -(b[i].y + b[i].y));
      } else {
        const V w = st.wp[i];
        const V e1 = add(a[i], conj(b[i])), o1 = sub(a[i], conj(b[i]));
        const V e2 = add(b[i], conj(a[i])), o2 = sub(b[i], conj(a[i]));
        l[k] = add(e1, mul_i<+1>(mul(conj(w), o1)));
        l[H - k] = add(e2, mul_i<-1>(mul(w, o2)));
      }
    }
  }
  __syncthreads();
  team_fft<T, +1, H, LS, NT>(buf, st.wr, (const V*)g.tw, g.twn, 2 * R, tid);
  double de = 0.0;
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = tid + i * NT;
    if (p < R * H) {
      V* px = buf + (p / H) * LS + p % H;
      V* py = px + R * LS;
      V gx = *px, gy = *py;
      if constexpr (grad_rec<T>()) {
        if (!first) {
          gx = add(gx, scl(st.gx[i], bt));
          gy = add(gy, scl(st.gy[i], bt));
        }
        st.gx[i] = gx;
        st.gy[i] = gy;
      }
      const V m0 = mr[p], m1 = mr[NT * TEAM_EP + p], rr = mr[2 * NT * TEAM_EP + p];
      const T a0 = m0.x * gx.x + m1.x * gy.x;
      const T a1 = m0.y * gx.y + m1.y * gy.y;
      const V fx = mk<T>(fma(a0, m0.x, rr.x * gx.x), fma(a1, m0.y, rr.y * gx.y));
      const V fy = mk<T>(fma(a0, m1.x, rr.x * gy.x), fma(a1, m1.y, rr.y * gy.y));
      *px = fx;
      *py = fy;
      de += (double)gx.x * fx.x + (double)gx.y * fx.y + (double)gy.x * fy.x + (double)gy.y * fy.y;
    }
  }
  __syncthreads();
  team_fft<T, -1, H, LS, NT>(buf, st.wr, (const V*)g.tw, g.twn, 2 * R, tid);
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int t = tid + i * NT;
    if (t < ntk) {
      const int f = t >= R * NP ? 1 : 0, u = t - f * R * NP;
      const int rr = u & (R - 1), k = u >> lr;
      if (y0 + rr < ny) {
        const V* l = buf + (f * R + rr) * LS;
        V* dst = (f ? M1 : M0) + y0 + rr;
        if (k == 0) {
          const V z0 = l[0];
          dst[0] = mk<T>(z0.x + z0.y, z0.x - z0.y);
          if (H % 2 == 0) dst[(H / 2) * ny] = conj(l[H / 2]);
        } else {
          const V zk = l[k], zm = l[H - k];
          const V w = st.wp[i];
          const V e1 = add(zk, conj(zm)), o1 = sub(zk, conj(zm));
          const V e2 = add(zm, conj(zk)), o2 = sub(zm, conj(zk));
          dst[k * ny] = scl(add(e1, mul_i<-1>(mul(w, o1))), (T)0.5);
          dst[(H - k) * ny] = scl(add(e2, mul_i<+1>(mul(conj(w), o2))), (T)0.5);
        }
      }
    }
  }
  return de;
}

// Column pass on nc columns from kx0 (see col_iter_body); ps receives this
// thread's parts of ||r||^2 and <r, M^-1 r>.
template <typename T, int NT, int NY>
__device__ __forceinline__ void team_col(TeamState<T>& st, cx<T>* buf, const Geo& g, cx<T>* M0, cx<T>* M1,
                                          __amdgpu_buffer_rsrc_t b0, __amdgpu_buffer_rsrc_t b1, int kx0,
                                         int nc, T a, T bt, bool first, bool last, double (&ps)[2], int tid) {
  using V = cx<T>;
  constexpr int LS = team_ls(NY);
  const int cn = nc * NY, base = kx0 * NY;
  V f0[TEAM_EP], f1[TEAM_EP];
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = tid + i * NT;
    if (p < cn) {
      f0[i] = team_load(b0, base + p, (V*)nullptr);
      f1[i] = team_load(b1, base + p, (V*)nullptr);
    }
  }
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = tid + i * NT;
    if (p < cn) {
      V* l = buf + (p / NY) * LS + p % NY;
      l[0] = f0[i];
      l[nc * LS] = f1[i];
    }
  }
  __syncthreads();
  team_fft<T, -1, NY, LS, NT>(buf, st.wc, (const V*)g.tw, g.twn, 2 * nc, tid);
  ps[0] = ps[1] = 0.0;
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = tid + i * NT;
    if (p < cn) {
      const int kx = kx0 + p / NY, ky = p % NY;
      V* px = buf + (p / NY) * LS + ky;
      V* py = px + nc * LS;
      const double xx = st.xx[i], yy = st.yy[i];
      const V fx = *px, fy = *py;
      // w = -i (xx Fx + yy Fy)
      const T ax = (T)xx * fx.x + (T)yy * fy.x, ay = (T)xx * fx.y + (T)yy * fy.y;
      const V w = mk<T>(ay, -ax);
      const T sig = (T)st.sig[i];
      const V zo = scl(st.r[i], sig);
      st.d[i] = first ? zo : add(zo, scl(st.d[i], bt));
      st.x[i] = add(st.x[i], scl(st.d[i], a));
      V s = w;
      if constexpr (!grad_rec<T>()) {
        if (!first) s = add(w, scl(st.s[i], bt));
        st.s[i] = s;
      }
      const V rn = sub(st.r[i], scl(s, a));
      st.r[i] = rn;
      const double wr = (kx == 0 ? 1.0 : 2.0) * ((double)rn.x * rn.x + (double)rn.y * rn.y);
      ps[0] += wr;
      ps[1] += (double)sig * wr;
      const V z = scl(rn, sig);
      const T sx = (T)(xx * g.inv_n), sy = (T)(yy * g.inv_n);
      *px = mk<T>(-sx * z.y, sx * z.x);
      *py = mk<T>(-sy * z.y, sy * z.x);
    }
  }
  __syncthreads();
  if (last) return;
  team_fft<T, +1, NY, LS, NT>(buf, st.wc, (const V*)g.tw, g.twn, 2 * nc, tid);
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = tid + i * NT;
    if (p < cn) {
      const V* l = buf + (p / NY) * LS + p % NY;
      M0[base + p] = l[0];
      M1[base + p] = l[nc * LS];
    }
  }
}

// Barrier of the team with K partial sums (per-thread parts in v): every member
// gets the totals, added in the same order, so their decisions agree.  Slots
// alternate between two sets: a member overwrites a set only after the barrier
// in between, which the slowest reader of that set has then passed.  quit: announce
// the arrival, but do not wait.
template <int NT, int K>
__device__ __forceinline__ bool team_barrier(__amdgpu_buffer_rsrc_t slots, int role, int G, unsigned epoch,
                                             const double (&v)[K], double* sh, double (&tot)[K], bool quit = false) {
  constexpr int NW = NT / 64;
  wave_sums<K>(v, sh);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const int set = (epoch & 1) * TEAM_MAX * 2;
  double t[K];
#pragma unroll
  for (int k = 0; k < K; ++k) t[k] = waves_total<NW>(sh + k * NW);
  if (NW > 1) __syncthreads();
  if (threadIdx.x < K) {
    union {
      u32x4 u;
      double d[2];
    } w;
    w.d[0] = K == 2 && threadIdx.x == 1 ? t[K - 1] : t[0];
    w.u.z = epoch;
    w.u.w = 0;
    __builtin_amdgcn_raw_buffer_store_b128(w.u, slots, (set + role * 2 + threadIdx.x) * 16, 0, 0);
  }
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const unsigned long long t0 = wall_clock64();
    bool ok = false;
    double got[K] = {};
    const unsigned want = quit ? ~epoch : epoch;
    for (unsigned q = 0;; ++q) {
      asm volatile("" ::: "memory");
      bool mine = true;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        union {
          u32x4 u;
          double d[2];
        } w;
        w.u = __builtin_amdgcn_raw_buffer_load_b128(slots, (set + (lane < G ? lane : 0) * 2 + k) * 16, 0, TEAM_SC1);
        got[k] = lane < G ? w.d[0] : 0.0;
        mine = mine && w.u.z == want;
      }
      if (__all(mine)) {
        ok = true;
        break;
      }
      if ((q & 255) == 255 && (quit || wall_clock64() - t0 > (unsigned long long)(TEAM_WAIT_S * 1e8))) break;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) got[k] = wave_sum(got[k]);
    if (NW == 1) {
#pragma unroll
      for (int k = 0; k < K; ++k) tot[k] = got[k];
      return ok;
    }
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) sh[k] = got[k];
      sh[K] = ok ? 1.0 : 0.0;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) tot[k] = sh[k];
  const bool ok = sh[K] != 0.0;
  __syncthreads();
  return ok;
}

#define NF_TEAM_NX(N, M_)                                                                                         \
  switch (N) {                                                                                                    \
    case 8: M_(8); break;                                                                                         \
    case 16: M_(16); break;                                                                                       \
    case 32: M_(32); break;                                                                                       \
    case 64: M_(64); break;                                                                                       \
    case 128: M_(128); break;                                                                                     \
    case 256: M_(256); break;                                                                                     \
    case 512: M_(512); break;                                                                                     \
    case 1024: M_(1024); break;                                                                                   \
    case 2048: M_(2048); break;                                                                                   \
    case 50: M_(50); break;                                                                                       \
    case 100: M_(100); break;                                                                                     \
    case 200: M_(200); break;                                                                                     \
    case 400: M_(400); break;                                                                                     \
    case 800: M_(800); break;                                                                                     \
    default: M_(1600); break;                                                                                     \
  }
#define NF_TEAM_NY(N, M_)                                                                                         \
  switch (N) {                                                                                                    \
    case 8: M_(8); break;                                                                                         \
    case 16: M_(16); break;                                                                                       \
    case 32: M_(32); break;                                                                                       \
    case 64: M_(64); break;                                                                                       \
    case 128: M_(128); break;                                                                                     \
    case 256: M_(256); break;                                                                                     \
    case 512: M_(512); break;                                                                                     \
    case 1024: M_(1024); break;                                                                                   \
    case 50: M_(50); break;                                                                                       \
    case 100: M_(100); break;                                                                                     \
    case 200: M_(200); break;                                                                                     \
    case 400: M_(400); break;                                                                                     \
    default: M_(800); break;                                                                                      \
  }

// The sums of a set of slots as team_barrier forms them, for the passes as
// launches; the sets are those of the team's barriers (epochs start even), so
// that the passes can go on where a team has ended.
enum { TEAM_SET_COL = 0, TEAM_SET_ROW = 1 };
template <int NT, int K>
__device__ __forceinline__ void team_totals(const TeamCtl* ctl, int set, int G, double* sh, double (&tot)[K]) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double v = lane < G ? ctl->slots[2 * ((set * TEAM_MAX + lane) * 2 + k)] : 0.0;
      tot[k] = wave_sum(v);
      if (NT > 64 && lane == 0) sh[k] = tot[k];
    }
  }
  if constexpr (NT > 64) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) tot[k] = sh[k];
    __syncthreads();
  }
}
// A member's partial sums into its slot.
template <int NT, int K>
__device__ __forceinline__ void team_leave(TeamCtl* ctl, int set, int role, const double (&v)[K], double* sh) {
  constexpr int NW = NT / 64;
  wave_sums<K>(v, sh);
  __syncthreads();
  if (threadIdx.x < K) ctl->slots[2 * ((set * TEAM_MAX + role) * 2 + threadIdx.x)] = waves_total<NW>(sh + threadIdx.x * NW);
}
// m and r of the pairs of a member's rows
template <int NT, typename T>
__device__ __forceinline__ void team_load_mr(cx<T>* mr, const T* __restrict__ m, const T* __restrict__ r, int nx, int ny,
                                             int y0, int R) {
  typedef cx<T> V;
  const size_t n = (size_t)nx * ny;
  const int h = nx / 2;
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = threadIdx.x + i * NT;
    const int rr = p / h, j = p - rr * h;
    const bool ok = rr < R && y0 + rr < ny;
    const size_t o = (size_t)(y0 + rr) * nx + 2 * j;
    mr[p] = ok ? *(const V*)(m + o) : vzero<V>();
    mr[NT * TEAM_EP + p] = ok ? *(const V*)(m + n + o) : vzero<V>();
    mr[2 * NT * TEAM_EP + p] = ok ? *(const V*)(r + o) : vzero<V>();
  }
}
// The gradient of d at a member's grid-point pairs (FP32), from and to its buffer
// between launches: gd in units of pairs, [2][Ny][Nx/2].
template <int NT, bool STORE, typename T>
__device__ __forceinline__ void team_grad(TeamState<T>& st, cx<T>* gd, int h, int ny, int y0, int R) {
  if constexpr (grad_rec<T>()) {
#pragma unroll
    for (int i = 0; i < TEAM_EP; ++i) {
      const int p = threadIdx.x + i * NT;
      const bool ok = p < R * h && y0 + p / h < ny;
      const size_t o = (size_t)y0 * h + p, n2 = (size_t)h * ny;
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
// The scalars of an iteration (see nf_loop.hpp).
struct TeamStep {
  double alpha, beta;
  bool bad, stop;
};
template <typename T>
__device__ __forceinline__ TeamStep team_step(double ga, double ga_prev, double al_prev, double de, int it, int max_iter,
                                              int budget) {
  TeamStep q;
  const bool first = it == 0;
  q.beta = pcg_beta(ga, ga_prev, first);
  q.alpha = pcg_alpha<T>(ga, de, al_prev, first, q.beta);
  q.bad = !isfinite(ga) || !isfinite(q.alpha);
  q.stop = q.bad || it + 1 >= max_iter || it + 1 >= budget;
  return q;
}

// Row pass of iteration it as a launch: for it >= 1 also the stopping test on
// the residual the last column pass left.
template <typename T, int NT>
__device__ __forceinline__ void team_row_phase(const Geo& g, const TeamShape& ts, cx<T>* M0, cx<T>* M1,
                                               const T* __restrict__ m, const T* __restrict__ r, cx<T>* gd, int it,
                                               double tol2) {
  using V = cx<T>;
  DevStatus* st = g.st;
  TeamCtl* ctl = (TeamCtl*)g.team;
  if (st->conv_at <= it) return;
  tclk_start(g, 0, it);
  __shared__ V buf[team_lds(NT)];
  __shared__ V mr[3 * NT * TEAM_EP];
  __shared__ double red[2 * (NT / 64) + 4];
  const int role = blockIdx.x, y0 = role << ts.lr;
  const bool lead = role == 0 && threadIdx.x == 0;
  T bt = 0;
  if (it >= 1) {
    double t[2];
    team_totals<NT, 2>(ctl, TEAM_SET_COL, ts.G, red, t);
    const bool bad = !isfinite(t[0]);
    if (bad || t[0] <= tol2 * st->bb) {
      if (lead) {
        st->rr[0] = t[0];
        st->converged = bad ? 0 : 1;
        if (bad) st->flags |= FLAG_NONFINITE;
        st->conv_at = it;
      }
      return;
    }
    if (lead) st->rho[it & 1] = t[1];
    if constexpr (grad_rec<T>()) bt = (T)pcg_beta(t[1], st->rho[(it + 1) & 1], false);
  }
  double de[1] = {0.0};
  if (y0 < g.ny) {
    const int bytes = g.h * g.ny * (int)sizeof(V);
    const __amdgpu_buffer_rsrc_t b0 = team_rsrc(M0, bytes), b1 = team_rsrc(M1, bytes);
    TeamState<T> S;
    team_load_mr<NT>(mr, m, r, g.nx, g.ny, y0, 1 << ts.lr);
    if (it >= 1) team_grad<NT, false>(S, gd, g.h, g.ny, y0, 1 << ts.lr);
#define M_(N)                                            \
  team_row_setup<T, NT, N>(S, g, ts.lr, threadIdx.x);    \
  de[0] = team_row<T, NT, N>(S, buf, mr, g, M0, M1, b0, b1, y0, ts.lr, bt, it == 0, threadIdx.x)
    NF_TEAM_NX(g.nx, M_)
#undef M_
    team_grad<NT, true>(S, gd, g.h, g.ny, y0, 1 << ts.lr);
  }
  de[0] *= (double)g.nx * g.ny;
  team_leave<NT, 1>(ctl, TEAM_SET_ROW, role, de, red);
  tclk_end(g, 0, it);
}

// Column pass of iteration it as a launch.
template <typename T, int NT>
__device__ __forceinline__ void team_col_phase(const Geo& g, const TeamShape& ts, cx<T>* M0, cx<T>* M1, cx<T>* xh,
                                               cx<T>* rh, cx<T>* dh, cx<T>* sh, int it, int max_iter) {
  using V = cx<T>;
  DevStatus* st = g.st;
  TeamCtl* ctl = (TeamCtl*)g.team;
  if (st->conv_at <= it) return;
  tclk_start(g, 2, it + 1);
  __shared__ V buf[team_lds(NT)];
  __shared__ double red[2 * (NT / 64) + 4];
  const int role = blockIdx.x, kx0 = role * ts.C, nc = kx0 < g.h ? min(ts.C, g.h - kx0) : 0;
  const int cn = nc * g.ny;
  const size_t base = (size_t)kx0 * g.ny;
  const bool first = it == 0;
  TeamState<T> S;
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = threadIdx.x + i * NT;
    const bool ok = p < cn;
    S.x[i] = ok ? xh[base + p] : vzero<V>();
    S.r[i] = ok ? rh[base + p] : vzero<V>();
    S.d[i] = ok && !first ? dh[base + p] : vzero<V>();
    if constexpr (!grad_rec<T>()) S.s[i] = ok && !first ? sh[base + p] : vzero<V>();
  }
  const double K[4] = {st->kbar[0], st->kbar[1], st->kbar[2], 0.0};
  double det[1];
  team_totals<NT, 1>(ctl, TEAM_SET_ROW, ts.G, red, det);
  const TeamStep q = team_step<T>(st->rho[it & 1], st->rho[(it + 1) & 1], st->alpha[(it + 1) & 1], det[0], it, max_iter,
                                  st->budget);
  if (role == 0 && threadIdx.x == 0) {
    st->alpha[it & 1] = q.alpha;
    st->iters = it + 1;
    if (q.bad) st->flags |= FLAG_NONFINITE;
    if (q.stop) {
      st->conv_at = it + 1;
      st->converged = 0;
    }
  }
  double ps[2] = {0.0, 0.0};
  if (nc > 0) {
    const int bytes = g.h * g.ny * (int)sizeof(V);
    const __amdgpu_buffer_rsrc_t b0 = team_rsrc(M0, bytes), b1 = team_rsrc(M1, bytes);
#define M_(N)                                                   \
  team_col_setup<T, NT, N>(S, g, K, kx0, threadIdx.x);          \
  team_col<T, NT, N>(S, buf, g, M0, M1, b0, b1, kx0, nc, (T)q.alpha, (T)q.beta, first, q.stop, ps, threadIdx.x)
    NF_TEAM_NY(g.ny, M_)
#undef M_
  }
#pragma unroll
  for (int i = 0; i < TEAM_EP; ++i) {
    const int p = threadIdx.x + i * NT;
    if (p < cn) {
      xh[base + p] = S.x[i];
      rh[base + p] = S.r[i];
      dh[base + p] = S.d[i];
      if constexpr (!grad_rec<T>()) sh[base + p] = S.s[i];
    }
  }
  team_leave<NT, 2>(ctl, TEAM_SET_COL, role, ps, red);
  tclk_end(g, 2, it + 1);
}
template <typename T, int NT>
__global__ void __launch_bounds__(NT) k_team_row(FluxArgs a, TeamShape ts, int it, double tol2) {
  team_row_phase<T, NT>(a.g, ts, (cx<T>*)a.G0, (cx<T>*)a.G1, (const T*)a.m, (const T*)a.r, (cx<T>*)a.gd, it, tol2);
}
template <typename T, int NT>
__global__ void __launch_bounds__(NT) kb_team_row(const FluxArgs* __restrict__ A, TeamShape ts, int it, double tol2) {
  const FluxArgs& a = A[blockIdx.y];
  team_row_phase<T, NT>(a.g, ts, (cx<T>*)a.G0, (cx<T>*)a.G1, (const T*)a.m, (const T*)a.r, (cx<T>*)a.gd, it, tol2);
}
template <typename T, int NT>
__global__ void __launch_bounds__(NT) k_team_col(IterArgs a, TeamShape ts, int it, int max_iter) {
  team_col_phase<T, NT>(a.g, ts, (cx<T>*)a.M0, (cx<T>*)a.M1, (cx<T>*)a.xh, (cx<T>*)a.rh, (cx<T>*)a.dh, (cx<T>*)a.sh, it,
                        max_iter);
}
template <typename T, int NT>
__global__ void __launch_bounds__(NT) kb_team_col(const IterArgs* __restrict__ A, TeamShape ts, int it, int max_iter) {
  const IterArgs& a = A[blockIdx.y];
  team_col_phase<T, NT>(a.g, ts, (cx<T>*)a.M0, (cx<T>*)a.M1, (cx<T>*)a.xh, (cx<T>*)a.rh, (cx<T>*)a.dh, (cx<T>*)a.sh, it,
                        max_iter);
}

// Iterations it0 .. it0 + nk - 1 of the loop (fewer if it stops).  On entry the
// mixed buffers hold the gradient of z and status.rho the scalar gamma of
// iteration it0 (it0 > 0: status.alpha, d and s of the iteration before; sh holds
// s or, in FP32, the gradient of d).  On exit x, r (and, if iterations are left, d, s)
// are written back and the status records the outcome as the launches of
// nf_loop.hpp do; status.team tells whether the team formed.
template <typename T, int NT>
__global__ void __launch_bounds__(NT) k_team(Geo g, TeamShape ts, cx<T>* M0, cx<T>* M1, const T* __restrict__ m,
                                             const T* __restrict__ r, cx<T>* xh, cx<T>* rh, cx<T>* dh, cx<T>* sh,
                                             int it0, int nk, int max_iter, double tol2) {
  using V = cx<T>;
  DevStatus* st = g.st;
  TeamCtl* ctl = (TeamCtl*)g.team;
  if (__builtin_amdgcn_s_getreg(20 /* XCC_ID */ | (3 << 11)) != (unsigned)ts.xcc) return;
  if (st->conv_at <= it0) return;
  __shared__ V buf[team_lds(NT)];
  __shared__ V mr[3 * NT * TEAM_EP];  // pairs of m_x, m_y, r of this member's rows
  __shared__ double red[2 * (NT / 64) + 4];
  __shared__ int role_s, go_s;
  const int tid = threadIdx.x, G = ts.G;
  if (tid == 0) {
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
        if (wall_clock64() - t0 > (unsigned long long)(TEAM_FORM_MS * 1e5)) {
          unsigned e2 = TEAM_OPEN;
          __hip_atomic_compare_exchange_strong(&ctl->state, &e2, (unsigned)TEAM_ABORT, __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    go_s = state;
  }
  __syncthreads();
  const int role = role_s;
  if (role >= G || go_s != TEAM_GO) return;

  const int h = g.h, ny = g.ny, nx = g.nx;
  const int bytes = h * ny * (int)sizeof(V);
  const __amdgpu_buffer_rsrc_t b0 = team_rsrc(M0, bytes), b1 = team_rsrc(M1, bytes);
  const __amdgpu_buffer_rsrc_t slots = team_rsrc(ctl->slots, 2 * TEAM_MAX * 2 * 16);
  const int kx0 = role * ts.C, nc = kx0 < h ? min(ts.C, h - kx0) : 0;
  const int y0 = role << ts.lr, R = 1 << ts.lr;
  const bool has_rows = y0 < ny;
  TeamState<T> S;
  {
    const int cn = nc * ny;
    const size_t base = (size_t)kx0 * ny;
#pragma unroll
    for (int i = 0; i < TEAM_EP; ++i) {
      const int p = tid + i * NT;
      const bool ok = p < cn;
      S.x[i] = ok ? xh[base + p] : vzero<V>();
      S.r[i] = ok ? rh[base + p] : vzero<V>();
      S.d[i] = ok && it0 > 0 ? dh[base + p] : vzero<V>();
      if constexpr (!grad_rec<T>()) S.s[i] = ok && it0 > 0 ? sh[base + p] : vzero<V>();
    }
    if (it0 > 0) team_grad<NT, false>(S, sh, h, ny, y0, R);
    team_load_mr<NT>(mr, m, r, nx, ny, y0, R);
  }
  const double K[4] = {st->kbar[0], st->kbar[1], st->kbar[2], 0.0};
#define M_(N) team_row_setup<T, NT, N>(S, g, ts.lr, tid)
  NF_TEAM_NX(nx, M_)
#undef M_
#define M_(N) team_col_setup<T, NT, N>(S, g, K, kx0, tid)
  NF_TEAM_NY(ny, M_)
#undef M_
  const double bb = st->bb;
  const int budget = st->budget;
  double ga = st->rho[it0 & 1], ga_prev = st->rho[(it0 + 1) & 1], al_prev = st->alpha[(it0 + 1) & 1];
  const double npts = (double)nx * ny;
  unsigned epoch = ts.epoch;
  int it = it0;
  int outcome = TEAM_MORE;
  double rr = 0.0;
  bool bad = false;
  for (; it < it0 + nk; ++it) {
    // The thread index as a value the compiler cannot follow: otherwise it
    // hoists the addresses, twiddles and multipliers of all the lengths below
    // out of the loop and spills them.
    int t = tid;
    asm volatile("" : "+v"(t));
    double de[1] = {0.0}, det[1];
    const T bt = grad_rec<T>() ? (T)pcg_beta(ga, ga_prev, it == 0) : (T)0;
    if (has_rows) {
#define M_(N) de[0] = team_row<T, NT, N>(S, buf, mr, g, M0, M1, b0, b1, y0, ts.lr, bt, it == 0, t)
      NF_TEAM_NX(nx, M_)
#undef M_
    }
    de[0] *= npts;
    if (!team_barrier<NT, 1>(slots, role, G, ++epoch, de, red, det)) {
      outcome = TEAM_LOST;
      break;
    }
    const TeamStep q = team_step<T>(ga, ga_prev, al_prev, det[0], it, max_iter, budget);
    bad = q.bad;
    double ps[2] = {0.0, 0.0}, pt[2];
    if (nc > 0) {
#define M_(N) team_col<T, NT, N>(S, buf, g, M0, M1, b0, b1, kx0, nc, (T)q.alpha, (T)q.beta, it == 0, q.stop, ps, t)
      NF_TEAM_NY(ny, M_)
#undef M_
    }
    if (!team_barrier<NT, 2>(slots, role, G, ++epoch, ps, red, pt, it + 1 == ts.lose && role != 0)) {
      outcome = TEAM_LOST;
      break;
    }
    rr = pt[0];
    al_prev = q.alpha;
    ga_prev = ga;
    ga = pt[1];
    if (q.stop) {
      outcome = TEAM_STOP;
      ++it;
      break;
    }
    if (!isfinite(rr) || rr <= tol2 * bb) {
      bad = !isfinite(rr);
      outcome = TEAM_CONV;
      ++it;
      break;
    }
  }
  if (outcome != TEAM_LOST) {
    const int cn = nc * ny;
    const size_t base = (size_t)kx0 * ny;
#pragma unroll
    for (int i = 0; i < TEAM_EP; ++i) {
      const int p = tid + i * NT;
      if (p < cn) {
        xh[base + p] = S.x[i];
        rh[base + p] = S.r[i];
        if (outcome == TEAM_MORE) {
          dh[base + p] = S.d[i];
          if constexpr (!grad_rec<T>()) sh[base + p] = S.s[i];
        }
      }
    }
    if (outcome == TEAM_MORE) team_grad<NT, true>(S, sh, h, ny, y0, R);
  }
  if (outcome == TEAM_LOST && tid == 0) st->lost = 1;
  if (role == 0 && tid == 0) {
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

// Launch of what `go` names: the team (G members per XCD are enough: workgroups
// are dealt round-robin over the 8 XCDs), or one pass for one or `count` instances.
template <typename T, int NT>
static hipError_t team_launch(const TeamGo& go, hipStream_t s) {
  typedef cx<T> V;
  const TeamShape& ts = go.ts;
  const FluxArgs& f = go.f;
  const IterArgs& a = go.a;
  switch (go.what) {
    case TeamGo::LOOP:
      hipLaunchKernelGGL((k_team<T, NT>), dim3(go.miss ? ts.G - 1 : 8 * (ts.G + 4)), dim3(NT), 0, s, a.g, ts, (V*)a.M0, (V*)a.M1,
                         (const T*)f.m, (const T*)f.r, (V*)a.xh, (V*)a.rh, (V*)a.dh, (V*)a.sh, go.it, go.nk, go.max_iter,
                         go.tol2);
      break;
    case TeamGo::ROW: hipLaunchKernelGGL((k_team_row<T, NT>), dim3(ts.G), dim3(NT), 0, s, f, ts, go.it, go.tol2); break;
    case TeamGo::COL: hipLaunchKernelGGL((k_team_col<T, NT>), dim3(ts.G), dim3(NT), 0, s, a, ts, go.it, go.max_iter); break;
    case TeamGo::ROWS:
      hipLaunchKernelGGL((kb_team_row<T, NT>), dim3(ts.G, go.count), dim3(NT), 0, s, go.fb, ts, go.it, go.tol2);
      break;
    case TeamGo::COLS:
      hipLaunchKernelGGL((kb_team_col<T, NT>), dim3(ts.G, go.count), dim3(NT), 0, s, go.ab, ts, go.it, go.max_iter);
      break;
  }
  return hipGetLastError();
}

}  // namespace nf
