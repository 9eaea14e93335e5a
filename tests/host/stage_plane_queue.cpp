// Host check of the 2D stage kernel (k_stage_plane, csrc/kernels.hip): its
// source runs on the CPU (cpu/hip/hip_runtime.h) on a forest with coarse-fine
// faces, and every schedule, with waves in several orders, has to give the
// result of one workgroup per leaf bit for bit, each leaf once.  The
// device-timed step's beginning and end inside the kernel, too.
// Prints "checked N wrong M"; exit status 0 iff M == 0.
#define AMRV_STAGE_UNIT 0
#include "kernels.hip"
#include "forest.hpp"

#include <array>

using namespace amrv;

namespace {

long long checked = 0, wrong = 0;

struct Problem {
  amrv_config c{};
  Tables t;
  Geo g{};
  std::vector<double> U, G, FF, pp;

  explicit Problem(int physics) {
    c.ndim = 2;
    c.block_nx[0] = c.block_nx[1] = 16;
    c.block_nx[2] = 1;
    c.nghost = 2;
    c.base_blocks[0] = 3;
    c.base_blocks[1] = 2;
    c.base_blocks[2] = 1;
    c.max_level = 2;
    c.physics = physics;
    c.flux = AMRV_HLL;
    c.limiter = AMRV_VANLEER;
    c.rk_stages = 2;
    c.bc[1][0] = c.bc[1][1] = AMRV_BC_ZERO_GRADIENT;
    for (int d = 0; d < 2; d++) c.xmax[d] = 1.0;
    c.gamma = 1.4;
    c.cfl = 0.4;
    c.glm_cr = 0.18;
    c.cad = 0.5;
    std::vector<int32_t> lev, ijk;  // level 1, its middle block refined
    for (int j = 0; j < 2; j++)
      for (int i = 0; i < 3; i++) {
        const bool fine = i == 1 && j == 0;
        for (int q = 0; q < (fine ? 4 : 1); q++) {
          lev.push_back(fine ? 2 : 1);
          for (int x : {fine ? 2 * i + (q & 1) : i, fine ? 2 * j + (q >> 1) : j, 0}) ijk.push_back(x);
        }
      }
    if (build_tables(c, (int64_t)lev.size(), lev.data(), ijk.data(), t)) {
      printf("%s\n", t.err.c_str());
      exit(2);
    }
    std::mt19937_64 rng(7);
    std::uniform_real_distribution<double> u01(0.0, 1.0);
    auto state = [&](std::vector<double>& v, size_t blocks, size_t cells) {  // [block or var][var][cells]
      v.resize(blocks * t.nvar * cells);
      for (double& x : v) x = 0.2 * u01(rng);
    };
    state(U, (size_t)t.n, (size_t)t.ncell);
    state(G, (size_t)t.nslot, 2 * (size_t)t.T);
    state(FF, (size_t)t.nslot, (size_t)t.T);
    const size_t vs = (size_t)t.n * t.ncell;
    for (size_t i = 0; i < vs; i++) U[i] += 1.0;  // density, energy
    if (physics != AMRV_POLYTROPE)
      for (size_t i = 0; i < vs; i++) U[3 * vs + i] += 2.0;
    for (int s = 0; s < t.nslot; s++)
      for (int i = 0; i < 2 * t.T; i++) {
        G[(size_t)s * t.nvar * 2 * t.T + i] += 1.0;
        if (physics != AMRV_POLYTROPE) G[((size_t)s * t.nvar + 3) * 2 * t.T + i] += 2.0;
      }
    pp.assign(PP_COUNT, 0.0);
    pp[PP_GAMMA] = c.gamma;
    pp[PP_GM1] = c.gamma - 1.0;
    pp[PP_IGM1] = 1.0 / (c.gamma - 1.0);
    pp[PP_CH] = 2.5;
    pp[PP_CAD] = c.cad;
    pp[PP_GCAD] = c.gamma * c.cad;
    pp[PP_DT] = 1e-3;
    pp[PP_DAMP] = 0.97;
    g.n = (int)t.n;
    g.ndim = 2;
    g.nx = t.nx;
    g.ncell = t.ncell;
    g.T = t.T;
    g.nslot = t.nslot;
    g.nvar = t.nvar;
    g.lvl = t.lvl.data();
    g.ijk = t.ijk.data();
    g.nbr = t.nbr.data();
    g.kind = t.kind.data();
    g.slot = t.slot.data();
    g.fslot = t.fslot.data();
    g.sleaf = t.sleaf.data();
    g.sface = t.sface.data();
    g.G = G.data();
    g.FF = FF.data();
    for (int l = 1; l <= 2; l++)
      for (int d = 0; d < 2; d++) g.rdx[l][d] = (double)((c.base_blocks[d] << (l - 1)) * 16);
  }
};

struct Result {
  std::vector<double> U, pp;
  std::vector<unsigned long long> red;
  std::vector<unsigned> cnt;
  bool operator==(const Result& o) const {
    return U.size() == o.U.size() && !memcmp(U.data(), o.U.data(), 8 * U.size()) &&
           !memcmp(pp.data(), o.pp.data(), 8 * pp.size()) && red == o.red && cnt == o.cnt;
  }
};

// one launch of stage `stage`; clock: as part of a device-timed step
template <int PH, int FLUX, int LIM>
Result run(const Problem& p, int stage, bool clock, int mode, int xcd, int grid, emu::Order order) {
  Result r;
  r.U.assign(p.U.size(), -1.0);
  r.pp = p.pp;
  r.red.assign(RED_WORDS, 0);
  r.cnt.assign(CNT_COUNT, 0);
  const double speed = 60.0, ch = 2.0;
  memcpy(&r.red[5 * RED_STRIDE], &speed, 8);
  memcpy(&r.red[9 * RED_STRIDE + 1], &ch, 8);
  StageArgs a{};
  a.Uin = p.U.data();
  a.Un = p.U.data();
  a.Uout = r.U.data();
  a.stage = stage;
  a.rk = 2;
  if (clock) {
    a.begin = stage == 1;
    a.end = stage == 2;
    a.cflred = stage == 2 ? r.red.data() : nullptr;
    a.clk = {r.red.data(), r.cnt.data(), r.pp.data(), 0.4, 10.0, 0.18, PH == PH_MHD};
    r.cnt[CNT_STEP1] = 1;
    r.pp[PP_T1] = 0.25;
  }
  std::vector<unsigned> queue(8, 0);
  Sched s{};
  s.mode = mode;
  s.xcd_remap = xcd;
  s.per_xcd = (p.g.n + 7) / 8;
  s.counter = queue.data();
  emu::launch((unsigned)grid, WGS2, order, [&] { k_stage_plane<PH, FLUX, LIM, 0>(p.g, a, r.pp.data(), s); });
  return r;
}

template <int PH, int FLUX, int LIM>
void check(const char* name) {
  const Problem p(PH);
  const int n = p.g.n;
  for (int stage = 1; stage <= 2; stage++)
    for (int clock = 0; clock < 2; clock++) {
      const Result ref = run<PH, FLUX, LIM>(p, stage, clock, 1, 0, n, emu::ASCENDING);
      for (double x : ref.U)
        if (!(x == x) || x == -1.0) wrong++;
      for (emu::Order order : {emu::ASCENDING, emu::DESCENDING, emu::RANDOM})
        for (const auto& s : {std::array<int, 3>{1, 0, n}, {1, 0, 1}, {1, 0, 4}, {1, 1, 8}, {1, 1, 16}, {2, 0, 1}, {2, 0, 3},
                              {2, 1, 1}, {2, 1, 9}}) {
          checked++;
          if (run<PH, FLUX, LIM>(p, stage, clock, s[0], s[1], s[2], order) == ref) continue;
          wrong++;
          printf("%s stage %d clock %d: mode %d xcd %d, %d workgroups, order %d differ\n", name, stage, clock, s[0], s[1],
                 s[2], (int)order);
        }
    }
}

}  // namespace

int main() {
  check<PH_EULER, FLX_HLL, LIM_VANLEER>("Euler, van Leer");
  check<PH_EULER, FLX_HLLC, LIM_KOREN>("Euler, Koren");
  check<PH_MHD, FLX_HLL, LIM_MC>("MHD, MC");
  check<PH_POLY, FLX_TVDLF, LIM_MINMOD>("polytrope, minmod");
  printf("checked %lld wrong %lld\n", checked, wrong);
  return wrong != 0;
}
