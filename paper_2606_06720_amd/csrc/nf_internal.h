// Structures shared by the host driver and the kernels (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nf {

// Device-resident solver status.  Written by exactly one workgroup (block 0)
// of the kernel that owns each field; read by later launches and copied to the
// host for convergence checks.
struct DevStatus {
  double kbar[8];   // grid mean of K = m m^T + r I: 2D Kxx, Kxy, Kyy; 3D Kxx, Kxy, Kxz, Kyy, Kyz, Kzz
  double bb;        // weighted ||b_hat||^2 of the projected right-hand side
  double rho[2];    // <r, M^-1 r> by iteration parity
  double alpha[2];  // step length by iteration parity (follows rho: the tuner fills both)
  double rr[2];     // rr[0]: ||r||^2 of the residual at which the solve stopped
  double rr0;       // initial ||r||^2
  double orr, obb;  // mixed-precision solve: FP64 ||r||^2 and ||b||^2 at the last correction start
  double rscale;    // mixed-precision solve: ||r|| scaling the FP32 correction
  double orr_prev;  // mixed-precision solve: ||r||^2 at the previous correction start (+inf before the first)
  double out[16];   // results of the final reductions (energy terms, dm, ...)
  int conv_at;      // iteration at which PCG stopped (converged or max_iter); INT_MAX while running
  int converged;    // 1 if the stop was convergence
  int iters;        // PCG iterations done
  int flags;        // FLAG_* bits of the current PCG solve
  int sticky;       // FLAG_* bits raised since the last full reset (split update)
  int outer_done;   // mixed-precision solve: 1 once the FP64 residual test has ended it
  int itot;         // mixed-precision solve: FP32 iterations of the finished corrections
  int budget;       // iteration limit of the current (inner) PCG run, INT_MAX when unused
  int team;         // outcome of the last team launch (TEAM_*) at its first member, TEAM_NONE if no team ran
  int lost;         // 1 if any member of it stopped waiting at a barrier: its part of x is then missing,
                    // whatever the others found
};
// what a team launch left (DevStatus::team): more iterations to do, stopped by
// max_iter, stopped by the residual test, a wait given up
enum { TEAM_NONE = 0, TEAM_MORE = 1, TEAM_STOP = 2, TEAM_CONV = 3, TEAM_LOST = 4 };
// formation of a team (TeamCtl::state)
enum { TEAM_OPEN = 0, TEAM_GO = 1, TEAM_ABORT = 2 };
enum {
  TEAM_MAX = 32,      // members at most: the compute units of an XCD
  TEAM_CHUNK = 4096,  // iterations per team launch at most
  // Loops as launches after two misses in a row: a miss costs 5 ms, a team saves
  // about a millisecond per loop, so that tries that keep failing cost a few
  // per cent at first and next to nothing later
  TEAM_PAUSE_MIN = 64,
  TEAM_PAUSE_MAX = 4096,
};
// Device memory of a handle's team: formation and the barrier's slots, two sets
// of two 16-byte entries (partial sum, epoch) per member.
struct TeamCtl {
  unsigned tickets, state;
  unsigned pad[14];
  double slots[2 * TEAM_MAX * 2 * 2];
};
// Split of a grid over a team: members, columns and 2^lr rows per member,
// threads per member, the XCD it runs on, and the epoch its barriers count from.
// complex elements of a member's transform buffer: two fields of at most 2 nt
// elements in padded lines, with room for short lines
constexpr int team_lds(int nt) { return nt == 64 ? 672 : (nt == 128 ? 1120 : (nt == 256 ? 1664 : 2688)); }
struct TeamShape {
  int G, C, lr, nt, xcc;
  unsigned epoch;
  int lose;  // iteration + 1 in which the members but the first stop waiting (tests; 0: none)
};
// The team over the chip (nf_chip.hpp): members at most, launched tiles at most; its barrier's
// 16-byte entries (two sets of two per tile, two sets of eight published lines), which
// lie in the arrays of SLOT_P3 that the 2D passes leave unused; the split of a grid:
// members, the tiles' class (Geo::wide) with rows and columns per tile, row and
// column tiles, row tiles whose elements a column tile's threads take at a time.
enum { CHIP_MAX = 256, CHIP_TILES = 2 * CHIP_MAX, CHIP_SLOTS = 2 * CHIP_TILES * 2 + 2 * 64 };
struct ChipShape {
  int G, wide, R, C, nrow, ncol, step;
};

enum { FLAG_NONFINITE = 1, FLAG_INCOMPAT = 2 };

// Slots of the partial-sum area; each slot holds up to SLOT_K arrays of
// MAX_WG doubles.
enum {
  SLOT_P3 = 0,      // delta of the PCG loop (nf_loop.hpp); 2D: also CHIP_SLOTS, from its second array on
  SLOT_P3INIT = 1,  // <r,M^-1 r>, <r,r>, <b,b>
  SLOT_KBAR = 2,    // sum mx^2, mx my, my^2, r
  SLOT_SCHK = 3,    // sum S, sum |S|
  SLOT_DM = 4,      // sum (m_new - m_old)^2, sum m_old^2
  SLOT_EPT = 5,     // sum r|g|^2, sum (m.g)^2, sum |m|^{2 gamma}
  SLOT_EGM = 6,     // sum w |xi|^2 |m_hat|^2 (both components)
  SLOT_RR = 7,      // ||r||^2 and <r, M^-1 r> of the residual that the last iteration of the loop left
  NSLOTS = 8,
  SLOT_K = 8,
  MAX_WG = 4096,
};

// Geometry and workspace pointers passed by value to every kernel.
struct Geo {
  int nx, ny, h, twn;
  double lx, ly;
  double inv_n;       // 1 / (number of grid points)
  const void* tw;     // cx<double>[twn] (cx<float> for the FP32 passes), tw[u] = exp(-2 pi i u / twn);
                      // twn is a common multiple of every transform length
  DevStatus* st;
  double* part;       // 2D: NSLOTS * SLOT_K * MAX_WG doubles; 3D: NSLOTS * SLOT_K * pstride doubles
  // 3D only (nz = 1 in 2D)
  int nz;
  double lz;
  int pstride;        // stride of the partial-sum arrays of one slot
  double* tot;        // NSLOTS * SLOT_K totals of the 3D partials (formed by a one-workgroup pass)
  // optional execution-span timing of one PCG-loop pass (nullptr = off): for
  // iteration it, the workgroups of kind tkind fold their start and end stamps
  // (device wall clock) into TCLK_W (min, max) pairs at
  // tclk[2 (it TCLK_W + (block mod TCLK_W))]; the host reduces them
  unsigned long long* tclk;
  int tkind;
  void* team;         // TeamCtl of the handle (2D)
  // tile variants of the PCG-loop passes chosen by the tuner (index 0: FP64
  // passes, 1: FP32 passes; VAR_DEFAULT = 1 is the untuned tile): row pass (row
  // variant), column pass (column variant var_upd; var_div keeps the code a
  // caller set for the operator end, which is part of that pass).  Read by the
  // launchers only.
  int var_flux[2], var_div[2], var_upd[2];
  // grids with a team over the chip: the loop's passes take that team's tiles instead,
  // row variant RV_WIDE + wide and column variant CV_WIDE + wide for wide = 0 and 1, row
  // variant 2 (tuned lengths) or 1 and column variant 1 for wide = 2 (-1: no team)
  int wide;
};

enum { TCLK_CAP = 2048, TCLK_W = 64 };  // timed iterations per PCG loop, stamp slots per iteration
// tile variants of the PCG-loop passes (see nf_tiles.hpp; the tuner times codes below NVAR);
// VAR_DEFAULT is the untuned tile
enum { VAR_DEFAULT = 1, RV_SMALL = 9, RV_SEQ = 12, RV_WIDE = 15, NRV = 17, CV_SMALL = 12, CV_SEQ = 15, CV_WIDE = 17,
       NCV = 19, NVAR = 17 };

__host__ __device__ inline double* slot_ptr(double* part, int slot) {
  return part + (size_t)slot * SLOT_K * MAX_WG;
}

// ---- per-instance arguments of the batched passes --------------------------------
// A batched launch covers `count` instances of one grid shape: blockIdx.y picks
// the instance, whose pointers and parameters are read from a device array of
// these structs (same names and meaning as the single-instance launchers'
// arguments; void* fields hold complex double, complex float or double data
// as the pass expects).
struct RowR2cArgs {
  Geo g;
  const double* f;
  void* out;
  double* schk;
};
struct ColFwdArgs {
  Geo g;
  void* in;
  void* out;
  void* Gx;
  void* Gy;
};
struct ColGradArgs {
  Geo g;
  const void* xh;
  void* P;
  void* Gx;
  void* Gy;
};
struct FluxArgs {
  Geo g;
  void* G0;
  void* G1;
  const void* m;
  const void* r;
  double* kslot;
  float* lo;
  void* gd;  // FP32 loop: gradient of the search direction on the grid, [d][..][Ny][Nx]
};
struct DivArgs {
  Geo g;
  const void* Fx;
  const void* Fy;
  void* rh;
  const void* bh;
};
struct IterArgs {
  Geo g;
  void* M0;
  void* M1;
  void* xh;
  void* rh;
  void* dh;
  void* sh;  // A d (FP64); in the FP32 loop the gradient of d on the grid (FluxArgs::gd)
};
struct SplitArgs {
  Geo g;
  void* P;
  void* Gx;
  const void* Gy;
  const double* m;
  double* p_out;
  double c2dt, gamma, dt, relax1;
};
struct HeatArgs {
  Geo g;
  void* Mx;
  void* My;
  double D2dt;
  double* eslot;
};
struct FinalArgs {
  Geo g;
  const void* Mx;
  const void* My;
  double* m;
  double* dslot;
};
struct RefStartArgs {
  Geo g;
  const void* r64;
  void* x64;
  void* x32;
  void* r32;
  void* Gx;
  void* Gy;
};
struct RefAccArgs {
  Geo g;
  void* x64;
  const void* x32;
  void* Gx;
  void* Gy;
};
struct SumArgs {
  const double* slot;
  DevStatus* st;
};

// ---- fixed workspace of the allocation-free solve (nf_noalloc.hip) ------------------
// Size of the per-GPU device array and the largest grid it serves: 2D FP64,
// Nx * Ny <= NOALLOC_MAX_POINTS (8 complex half-spectrum fields of 8 bytes per
// grid point, the partial-sum slots, the status block and a twiddle table of
// at most 4096 entries).
enum : size_t { NOALLOC_SCRATCH_BYTES = 8u << 20 };
enum { NOALLOC_MAX_POINTS = 65536, NOALLOC_MAX_TWIDDLES = 4096, NOALLOC_MAX_DEVICES = 64 };
// Device address of the current GPU's copy of the array (looked up on the
// first call for that GPU and kept).
hipError_t noalloc_scratch(void** out);

// ---- host-callable launchers (defined in nf_kernels.hip) --------------------------
// All take the stream last and return hipError_t of the launch.
struct Bufs;

hipError_t launch_status_reset(const Geo& g, int full, hipStream_t s);

// ---- 3D passes (nf_kernels3d.hip).  g: the 3D geometry (ny = Ny, nz = Nz);
// row passes take the same geometry and treat the Ny*Nz lines (z, y) as rows.
// Mixed buffers hold [kx][z][y] (after x) or, in place, [kx][z][ky] (after
// x and y); spectral buffers hold [kx][ky][kz].
int nwg3_row(const Geo& g);
int nwg3_z(const Geo& g);
int nwg3_flux(const Geo& g, bool f32);   // operator middle
int nwg3_ziter(const Geo& g, bool f32);  // z pass of the PCG loop
hipError_t launch3_row_r2c(const Geo& g, const double* f, void* out, int schk, hipStream_t s);
hipError_t launch3_row_c2r(const Geo& g, const void* in, double* f, hipStream_t s);
// lo: FP32 copies of m (3n) then r (n), written when non-null; kbar: write the Kbar partials;
// tol2: stopping test of the loop (it >= 1)
// gd: gradient of the search direction on the grid (FP32 loop)
hipError_t launch3_row_flux(const Geo& g, bool f32, void* G0, void* G1, void* G2, const void* m, const void* r, int it,
                            int kbar, float* lo, void* gd, double tol2, hipStream_t s);
hipError_t launch3_row_split(const Geo& g, void* P, void* G0, void* G1, void* G2, const double* m, double* p_out,
                             double c2dt, double gamma, double dt, double relax1, double D2dt, hipStream_t s);
hipError_t launch3_row_final(const Geo& g, const void* M0, const void* M1, const void* M2, double* m, hipStream_t s);
// y passes over nf fields (1..4) in place; dir -1 forward, +1 inverse; nsum > 0: also add up the
// nsum partials of the pass before (PCG loop, 3 fields); heat_D2dt >= 0: multiply by exp(-D2dt xi_y^2)
hipError_t launch3_ypass(const Geo& g, bool f32, int nf, int dir, void* F0, void* F1, void* F2, void* F3, int it,
                         int nsum, double heat_D2dt, hipStream_t s);
// z passes
hipError_t launch3_zfwd(const Geo& g, const void* in, void* out, int project, hipStream_t s);
// mode 1: P = x/n; 2: gradient (G0..G2); 3: both
hipError_t launch3_zinv(const Geo& g, int mode, const void* xh, void* P, void* G0, void* G1, void* G2, hipStream_t s);
hipError_t launch3_zdiv(const Geo& g, int init, const void* F0, const void* F1, const void* F2, void* qh, void* rh,
                        const void* bh, hipStream_t s);
hipError_t launch3_zstart(const Geo& g, const void* rh, void* xh, void* G0, void* G1, void* G2, int max_iter,
                          double tol2, hipStream_t s);
hipError_t launch3_ziter(const Geo& g, bool f32, void* M0, void* M1, void* M2, void* xh, void* rh, void* dh, void* sh,
                         int it, int max_iter, hipStream_t s);
hipError_t launch3_zheat(const Geo& g, void* M0, void* M1, void* M2, double D2dt, hipStream_t s);
hipError_t launch3_zrefine_start(const Geo& g32, const void* r64, void* x64, void* x32, void* r32,
                                 void* G0, void* G1, void* G2, double tol2, double floor_in, int max_iter,
                                 hipStream_t s);
hipError_t launch3_zrefine_acc(const Geo& g, void* x64, const void* x32, void* G0, void* G1, void* G2,
                               hipStream_t s);
// reduced totals of a slot into st->out[o..o+K)
hipError_t launch3_copy_tot(const Geo& g, int slot, int K, int o, hipStream_t s);
// energy terms (Sec. 2.5) in 3D: totals of sum r|g|^2, sum (m.g)^2, sum |m|^{2 gamma}
// into the SLOT_EPT totals (g = grad p as three physical fields), and of the
// Parseval sum of the three spectra of m into the SLOT_EGM total
hipError_t launch3_energy_pt(const Geo& g, const double* m, const double* r, const double* gx, const double* gy,
                             const double* gz, double gamma, hipStream_t s);
hipError_t launch3_spec_gradnorm(const Geo& g, const void* F0, const void* F1, const void* F2, hipStream_t s);
// adjoint of one 3D step (grid-stride passes): reverse of activation and
// relaxation (lam in: after diffusion, out: lam_m; G in: grad p, out: lam_g),
// the right-hand side -i xi_tilde . F(v) of the adjoint pressure from three
// spectra, and the final gradient terms (U = grad mu, P = grad p)
hipError_t launch3_adj1(const Geo& g, const double* m, double* lam, double* G0, double* G1, double* G2, double c2dt,
                        double gamma, double dt, double relax1, hipStream_t s);
hipError_t launch3_spec_divrhs(const Geo& g, const void* F0, const void* F1, const void* F2, void* bh, hipStream_t s);
hipError_t launch3_adj2(const Geo& g, const double* m, const double* mu, const double* U0, const double* U1,
                        const double* U2, const double* P0, const double* P1, const double* P2, double* lam,
                        double* grad_r, double* grad_S, hipStream_t s);
// g.tot of a slot from the n partials the passes of the PCG loop store (one
// workgroup; K = 1, 2, 3 or 7 arrays)
hipError_t launch3_sum_tot(const Geo& g, int slot, int K, int n, hipStream_t s);
hipError_t launch_zero_spec(const Geo& g, void* xh, hipStream_t s);
// row passes (physical <-> mixed)
int row_nwg(const Geo& g);
int col_nwg(const Geo& g);
// workgroups of the row variant rv of the row pass / column variant cv of the
// column pass
int row_nwg_var(const Geo& g, int rv);
int col_nwg_var(const Geo& g, int cv);
// whether a variant exists for the grid of g and the real type (f32) and can run
bool flux_var_valid(const Geo& g, bool f32, int rv);
bool div_var_valid(const Geo& g, bool f32, int cv);
// workgroups of the column pass of the loop (the partials of ||r||^2 and <r, M^-1 r>)
int rr_nwg(const Geo& g, bool f32);
// rows per workgroup of row variant rv, columns per workgroup of column variant cv
int flux_var_rows(const Geo& g, int rv);
int flux_var_threads(const Geo& g, int rv);
int flux_var_plan(int rv);
int div_var_cols(const Geo& g, int cv);
int div_var_threads(const Geo& g, int cv);
// variants in use by the loop (it >= 0), the column pass
int use_rv(const Geo& g, bool f32, int it);
int use_cv(const Geo& g, bool f32);
// the small-grid team (nf_team.hpp): the split of a grid if it has one; reset of its
// formation before a launch that no loop start precedes; what to launch
bool team_shape(const Geo& g, TeamShape* ts);
hipError_t launch_team_reset(const Geo& g, hipStream_t s);
struct TeamGo {
  enum { LOOP, ROW, COL, ROWS, COLS } what;  // the team; a pass as a launch, for one or `count` instances
  bool miss;                                 // LOOP: with too few workgroups to form (tests)
  TeamShape ts;
  int it, nk, max_iter;
  double tol2;
  FluxArgs f;          // LOOP, ROW
  IterArgs a;          // LOOP, COL
  const FluxArgs* fb;  // ROWS
  const IterArgs* ab;  // COLS
  int count;
};
hipError_t launch_team(bool f32, const TeamGo& go, hipStream_t s);
hipError_t launch_team_rr(const Geo& g, const TeamShape& ts, hipStream_t s);
// the team over the chip (nf_chip.hpp): the split of a grid, if it has one; the launch
// (go.a, go.f, go.ts.epoch)
bool chip_shape(const Geo& g, ChipShape* cs);
hipError_t launch_chip(bool f32, const TeamGo& go, hipStream_t s);
// whether an axis length has tuned variants; whether the grid has any
bool tuned_length(int n);
bool var_grid(const Geo& g);
// fill n doubles with a value (a kernel, so that no memset node is recorded)
hipError_t launch_fill_doubles(double* p, size_t n, double v, hipStream_t s);
hipError_t launch_row_r2c(const Geo& g, const double* f, void* out_mixed, double* schk_slot, hipStream_t s);
hipError_t launch_row_c2r(const Geo& g, const void* in_mixed, double* f, hipStream_t s);
// lo: optional FP32 copies of m then r (3n floats), written when non-null
hipError_t launch_row_flux(const Geo& g, void* G0, void* G1, const double* m, const double* r, int it,
                           double* kbar_slot, double tol2, hipStream_t s, float* lo = nullptr);
hipError_t launch_row_split(const Geo& g, void* P, void* Gx, void* Gy, const double* m, double* p_out,
                            double c2dt, double gamma, double dt, double relax_gamma1, hipStream_t s);
hipError_t launch_row_final(const Geo& g, const void* Mx, const void* My, double* m, double* dm_slot,
                            hipStream_t s);
hipError_t launch_row_energy(const Geo& g, const void* Gx, const void* Gy, const double* m, const double* r,
                             double gamma, double* slot, hipStream_t s);
// column passes (mixed <-> spectral)
hipError_t launch_col_fwd(const Geo& g, void* in_mixed, void* out_spec, int with_grad, void* Gx, void* Gy,
                          hipStream_t s);
hipError_t launch_col_grad(const Geo& g, const void* xh, void* P, void* Gx, void* Gy, hipStream_t s);
hipError_t launch_col_div(const Geo& g, int init, const void* Fx, const void* Fy, void* qh, void* rh, const void* bh,
                          int nwg_row, hipStream_t s);
hipError_t launch_col_start(const Geo& g, const void* rh, void* xh, void* Gx, void* Gy, int max_iter, double tol2,
                            hipStream_t s);
// column pass of the PCG loop (M0, M1: fluxes in, gradient out; sh: A d, FP64 only)
hipError_t launch_col_iter64(const Geo& g, void* M0, void* M1, void* xh, void* rh, void* dh, void* sh, int it,
                             int max_iter, hipStream_t s);
// FP32 instantiations of the PCG-loop passes (g.tw points at the FP32 table;
// m32/r32 are the FP32 copies written by launch_row_flux, gd the gradient of the
// search direction on the grid)
hipError_t launch_row_flux32(const Geo& g, void* G0, void* G1, const float* m32, const float* r32, float* gd, int it,
                             double tol2, hipStream_t s);
hipError_t launch_col_iter32(const Geo& g, void* M0, void* M1, void* xh, void* rh, void* dh, int it, int max_iter,
                             hipStream_t s);
// mixed-precision correction start / accumulation (g32: FP32 twiddles)
hipError_t launch_col_refine_start(const Geo& g32, const void* r64, void* x64, void* x32, void* r32,
                                   void* Gx32, void* Gy32, double tol2, double floor_in, int max_iter, hipStream_t s);
hipError_t launch_col_refine_acc(const Geo& g, void* x64, const void* x32, void* Gx, void* Gy, hipStream_t s);
hipError_t launch_col_heat(const Geo& g, void* Mx, void* My, double D2dt, double* egm_slot, hipStream_t s);
hipError_t launch_col_gradnorm(const Geo& g, const void* Mx, const void* My, double* egm_slot, hipStream_t s);
// adjoint passes
hipError_t launch_row_adj1(const Geo& g, void* A0, void* A1, const void* G0, const void* G1, const double* m,
                           double* lam_out, double c2dt, double gamma, double dt, double relax1, hipStream_t s);
hipError_t launch_row_adj2(const Geo& g, const void* M1, const void* M2, const void* P1, const void* P2,
                           const double* m, const double* mu, double* lam, double* grad_r, double* grad_S,
                           hipStream_t s);
hipError_t launch_col_divrhs(const Geo& g, const void* V0, const void* V1, void* bh, hipStream_t s);
hipError_t launch_zero_doubles(double* p, size_t n, hipStream_t s);
// set the TCLK_CAP * TCLK_W stamp pairs to (max, 0)
hipError_t launch_tclk_reset(unsigned long long* t, hipStream_t s);
// reduce K arrays of n partials of a slot into st->out[o..o+K)
hipError_t launch_sum_slot(const Geo& g, const double* slot, int K, int n, int o, hipStream_t s);

// Batched launchers: `shape` gives the grid shape shared by the instances
// (sizes only), A points at `count` device-resident argument structs; the
// remaining arguments are common to the batch.  st0: `count` contiguous statuses.
hipError_t launchb_status_reset(DevStatus* st0, int count, int full, hipStream_t s);
hipError_t launchb_sum_slot(const SumArgs* A, int count, int K, int n, int o, hipStream_t s);
hipError_t launchb_row_r2c(const Geo& shape, const RowR2cArgs* A, int count, hipStream_t s);
hipError_t launchb_col_fwd(const Geo& shape, const ColFwdArgs* A, int count, int mode, hipStream_t s);
hipError_t launchb_col_grad(const Geo& shape, const ColGradArgs* A, int count, bool grad, hipStream_t s);
hipError_t launchb_row_flux64(const Geo& shape, const FluxArgs* A, int count, int it, double tol2, hipStream_t s);
hipError_t launchb_row_flux32(const Geo& shape, const FluxArgs* A, int count, int it, double tol2, hipStream_t s);
hipError_t launchb_col_div_init(const Geo& shape, const DivArgs* A, int count, hipStream_t s);
hipError_t launchb_col_start(const Geo& shape, const IterArgs* A, int count, int max_iter, double tol2,
                             hipStream_t s);
hipError_t launchb_col_iter64(const Geo& shape, const IterArgs* A, int count, int it, int max_iter, hipStream_t s);
hipError_t launchb_col_iter32(const Geo& shape, const IterArgs* A, int count, int it, int max_iter, hipStream_t s);
hipError_t launchb_row_split(const Geo& shape, const SplitArgs* A, int count, hipStream_t s);
hipError_t launchb_col_heat(const Geo& shape, const HeatArgs* A, int count, hipStream_t s);
hipError_t launchb_row_final(const Geo& shape, const FinalArgs* A, int count, hipStream_t s);
hipError_t launchb_col_refine_start(const Geo& shape, const RefStartArgs* A, int count, double tol2,
                                    double floor_in, int max_iter, hipStream_t s);
hipError_t launchb_col_refine_acc(const Geo& shape, const RefAccArgs* A, int count, hipStream_t s);

}  // namespace nf
