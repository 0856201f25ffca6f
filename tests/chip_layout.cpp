// Replays on the host the indices of the loop over the chip (nf_chip.hpp) for every
// grid it is built for: every access has to lie in its buffer or LDS array, the row
// and the column tiles have to agree on the place of every element of the exchange,
// and every element has to have one owner.  Exit status 0 if all of it holds.
#include <cstdio>
#include <vector>

#include "nf_chip.hpp"

using namespace nf;

static int bad = 0;
static void expect(bool ok, const char* what, int nx, int ny) {
  if (!ok && bad++ < 20) std::printf("%d x %d: %s\n", nx, ny, what);
}
#define EXPECT(X) expect((X), #X, NX, NY)

template <int NX, int NY>
static int check() {
  if constexpr (chip_split(NX, NY).G == 0) {
    return 0;
  } else {
    constexpr ChipShape cs = chip_split(NX, NY);
    constexpr int CL = cs.wide, NT = wide_threads(CL), E = wide_elems(CL), EP = chip_ep(NX, NY), H = NX / 2, R = cs.R, NC = cs.C;
    constexpr int SR = chip_sr(NX, CL), SC = chip_sc(CL), NTK = R * H, CN = NC * NY, ETP = (NTK + NT - 1) / NT;
    constexpr int LSR = chip_ls(H, R), LSC = chip_ls(NY, NC), n = H * NY;
    EXPECT(cs.G <= CHIP_MAX && cs.nrow * R == NY && cs.ncol * NC == H && (H / 2) % NC == 0 && cs.G >= cs.nrow && cs.G >= cs.ncol);
    EXPECT(LSR >= lpad_len(H) && LSC >= lpad_len(NY) && 2 * R * LSR <= chip_lds(CL) && 2 * NC * LSC <= chip_lds(CL));
    EXPECT(NTK <= E && CN <= E && EP * NT == E && R * H <= SR * (E / SR) && NT % SR == 0 && NT % SC == 0);
    EXPECT(cs.nrow * SR <= CHIP_TILES && cs.ncol * SC <= CHIP_TILES && cs.ncol * SC <= MAX_WG);
    EXPECT(2 * CHIP_TILES * 2 + 64 + 7 * 8 + 2 <= CHIP_SLOTS && CHIP_SLOTS * 2 <= (SLOT_K - 1) * MAX_WG);
    // row side: which (k, field, y) each exchange element holds, -1: none
    std::vector<int> where[2] = {std::vector<int>(n, -1), std::vector<int>(n, -1)};
    for (int member = 0; member < cs.G; ++member) {
      const int y0 = member * R;
      if (y0 >= NY) continue;
      std::vector<int> pts(R * H, 0);
      for (int tid = 0; tid < NT; ++tid) {
        for (int i = 0; i < ETP; ++i) {
          const int t = tid + i * NT;
          if (t >= NTK) continue;
          const int rr = t % R, f = t / R & 1, k = t / (2 * R), base = y0 * H;
          EXPECT(k >= 0 && k < H / 2 && pair_mirror(k, H) >= H / 2 && pair_mirror(k, H) < H);
          EXPECT((f * R + rr) * LSR + H - (k ? k : 1) < 2 * R * LSR);
          for (int s = 0; s < 2; ++s) {
            const int o = s ? chip_hi<H, R>(base, t) : base + t;
            const bool in = o >= 0 && o < n;
            EXPECT(in);
            if (!in) continue;
            EXPECT(where[s][o] == -1);
            where[s][o] = ((s ? pair_mirror(k, H) : k) * 2 + f) * NY + y0 + rr;
          }
        }
        for (int i = 0; i < EP; ++i) {
          EXPECT(tid + i * NT < E);
          const int p = chip_elem<NT, SR, R * H>(tid, i);
          if (p >= R * H) continue;
          EXPECT(p >= 0 && p / H * LSR + p % H + R * LSR < 2 * R * LSR && (size_t)(y0 + p / H) * NX + 2 * (p % H) + 1 < (size_t)NX * NY);
          if (p >= 0) ++pts[p];
        }
      }
      for (int p = 0; p < R * H; ++p) EXPECT(pts[p] == 1);
    }
    for (int s = 0; s < 2; ++s)
      for (int o = 0; o < n; ++o) EXPECT(where[s][o] >= 0);
    // column side
    for (int member = 0; member < cs.G; ++member) {
      const int kx0 = member * NC, s = kx0 >= H / 2;
      std::vector<int> lds(2 * NC * LSC, 0), els(CN, 0);
      for (int tid = 0; tid < NT; ++tid) {
        const ChipPlace at = chip_place<NX, NY>(kx0, tid);
        for (int i = 0; i < 2 * EP; ++i) {
          if (at.t + i * cs.step >= cs.nrow) continue;
          const int o = at.go + i * cs.step * R * H, l = at.li + i * cs.step * R;
          const bool in = kx0 < H && o >= 0 && o < n && l >= 0 && l < 2 * NC * LSC;
          EXPECT(in);
          if (!in) continue;
          ++lds[l];
          const int line = l / LSC, y = l % LSC;
          EXPECT(y < NY && where[s][o] == ((kx0 + line % NC) * 2 + line / NC) * NY + y);
        }
        for (int i = 0; i < EP; ++i) {
          const int p = chip_elem<NT, SC, CN>(tid, i);
          if (p >= CN || kx0 >= H) continue;
          EXPECT(p >= 0 && p / NY * LSC + p % NY + NC * LSC < 2 * NC * LSC && (size_t)kx0 * NY + p < (size_t)n);
          if (p >= 0) ++els[p];
        }
      }
      if (kx0 >= H) continue;
      for (int c = 0; c < 2 * NC; ++c)
        for (int y = 0; y < NY; ++y) EXPECT(lds[c * LSC + y] == 1);
      for (int p = 0; p < CN; ++p) EXPECT(els[p] == 1);
    }
    return 1;
  }
}
template <int NX>
static int rows() {
  return check<NX, 64>() + check<NX, 128>() + check<NX, 256>() + check<NX, 512>() + check<NX, 1024>() + check<NX, 100>() +
         check<NX, 200>() + check<NX, 400>() + check<NX, 800>();
}
int main() {
  const int shapes = rows<128>() + rows<256>() + rows<512>() + rows<1024>() + rows<2048>() + rows<200>() + rows<400>() +
                     rows<800>() + rows<1600>();
  std::printf("%d grids, %d faults\n", shapes, bad);
  return bad || shapes < 19 ? 1 : 0;
}
