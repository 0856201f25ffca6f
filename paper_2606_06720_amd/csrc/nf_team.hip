// The small-grid team: shapes, formation reset and the choice of its kernel (nf_team.hpp).
#include "nf_team.hpp"

namespace nf {

hipError_t team_go64_64(const TeamGo& go, hipStream_t s);
hipError_t team_go64_128(const TeamGo& go, hipStream_t s);
hipError_t team_go64_256(const TeamGo& go, hipStream_t s);
hipError_t team_go64_512(const TeamGo& go, hipStream_t s);
hipError_t team_go32_64(const TeamGo& go, hipStream_t s);
hipError_t team_go32_128(const TeamGo& go, hipStream_t s);
hipError_t team_go32_256(const TeamGo& go, hipStream_t s);
hipError_t team_go32_512(const TeamGo& go, hipStream_t s);

// The team of a grid, if it has one: 2D, at most 65536 points, columns of up to
// 1024 and rows of up to 2048; 32 workgroups (one per compute unit of an XCD)
// or as many as there are columns or rows, with the fewest threads that leave
// each at most TEAM_EP elements of a field.
bool team_shape(const Geo& g, TeamShape* ts) {
  if (g.nz != 1 || (long long)g.nx * g.ny > 65536) return false;
  if (g.ny > 1024 || g.nx > 2048) return false;
  ts->C = (g.h + TEAM_MAX - 1) / TEAM_MAX;
  ts->lr = 0;
  while ((TEAM_MAX << ts->lr) < g.ny) ++ts->lr;
  const int R = 1 << ts->lr;
  const int gc = (g.h + ts->C - 1) / ts->C, gr = (g.ny + R - 1) / R;
  ts->G = gc > gr ? gc : gr;
  const int cn = ts->C * g.ny, pairs = 2 * R * ((g.h + 1) / 2);  // pairs >= R * h
  const int e = cn > pairs ? cn : pairs;
  const int lc = 2 * ts->C * team_ls(g.ny), lrow = 2 * R * team_ls(g.h);
  const int lds = lc > lrow ? lc : lrow;
  for (int nt = 64; nt <= 512; nt *= 2) {
    ts->nt = nt;
    if (e <= nt * TEAM_EP && lds <= team_lds(nt)) return true;
  }
  return false;
}

__global__ void k_team_reset(DevStatus* st, TeamCtl* ctl) {
  if (threadIdx.x == 0) {
    st->team = TEAM_NONE;
    st->lost = 0;
    ctl->tickets = 0;
    ctl->state = TEAM_OPEN;
  }
}
hipError_t launch_team_reset(const Geo& g, hipStream_t s) {
  hipLaunchKernelGGL(k_team_reset, dim3(1), dim3(64), 0, s, g.st, (TeamCtl*)g.team);
  return hipGetLastError();
}

hipError_t launch_team(bool f32, const TeamGo& go, hipStream_t s) {
  switch (go.ts.nt) {
    case 64: return f32 ? team_go32_64(go, s) : team_go64_64(go, s);
    case 128: return f32 ? team_go32_128(go, s) : team_go64_128(go, s);
    case 256: return f32 ? team_go32_256(go, s) : team_go64_256(go, s);
    default: return f32 ? team_go32_512(go, s) : team_go64_512(go, s);
  }
}

// ||r||^2 of the last column pass as a launch into status.out[11] (solves that
// max_iter stopped)
__global__ void k_team_rr(DevStatus* st, const TeamCtl* ctl, int G) {
  double t[2];
  team_totals<64, 2>(ctl, TEAM_SET_COL, G, nullptr, t);
  if (threadIdx.x == 0) st->out[11] = t[0];
}
hipError_t launch_team_rr(const Geo& g, const TeamShape& ts, hipStream_t s) {
  hipLaunchKernelGGL(k_team_rr, dim3(1), dim3(64), 0, s, g.st, (const TeamCtl*)g.team, ts.G);
  return hipGetLastError();
}

}  // namespace nf
