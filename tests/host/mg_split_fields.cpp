// Host check of the 3D multigrid's kernels that read and write a caller's fields
// in pairs of cells (csrc/multigrid.hip, run on the CPU by cpu/hip/hip_runtime.h):
// fields need no more alignment than a double's.  Built with -fsanitize=alignment,
// on fields that start 8 bytes past a 16-byte boundary; results bit for bit those
// on aligned ones.
// Prints "wrong N"; exit status 0 iff N == 0.
#include "multigrid.hip"

int amrv::set_error(int code, const char*) { return code; }

namespace {

int wrong = 0;

struct Field {  // n doubles, 8 bytes past a 16-byte boundary (odd) or on one
  std::vector<double> store;
  double* at;
  Field(size_t n, bool odd) : store(n + 2) {
    at = store.data() + ((reinterpret_cast<uintptr_t>(store.data()) & 15) != 0);
    if (odd) at++;
  }
};

void fill(double* p, size_t n, unsigned seed) {
  std::mt19937_64 rng(seed);
  std::uniform_real_distribution<double> u(0.5, 1.5);
  for (size_t i = 0; i < n; i++) p[i] = u(rng);
}

void same(const double* a, const double* b, size_t n, const char* what) {
  if (!memcmp(a, b, 8 * n)) return;
  wrong++;
  printf("%s differs\n", what);
}

}  // namespace

int main() {
  const int lg = 3, n = 1 << lg, half = n * n * n / 2;
  const size_t cells = 2 * (size_t)half;
  Field nat(cells, false), split(cells, false), from(cells, true), back(cells, true);
  fill(nat.at, cells, 1);
  memcpy(from.at, nat.at, 8 * cells);
  auto reorder = [&](const double* src, double* dst, int to_split) {
    emu::launch((unsigned)((half + 255) / 256), 256, emu::ASCENDING, [&] { k_mg3_reorder(lg, src, dst, to_split); });
  };
  reorder(from.at, split.at, 1);
  for (int z = 0, i = 0; z < n; z++)
    for (int y = 0; y < n; y++)
      for (int x = 0; x < n; x++, i++) wrong += split.at[split_idx<3>(x, y, z, lg)] != nat.at[i];
  reorder(split.at, back.at, 0);
  same(back.at, nat.at, cells, "reorder");

  MgDev g{};
  g.nd = 3;
  g.bc = AMRV_MG_NEUMANN;
  g.nf = 2;
  g.n[0] = n;
  g.lg[0] = lg;
  g.cells[0] = (int)cells;
  std::vector<double> par(PAR_COUNT, 1.0), phi0(cells), phi1(cells);
  fill(phi0.data(), cells, 2);
  fill(phi1.data(), cells, 3);
  g.par = par.data();
  g.phi[0][0] = phi0.data();
  g.phi[1][0] = phi1.data();
  RdK k{};
  k.model = AMRV_RD_SCHNAKENBERG;
  k.Du = 0.3;
  k.Dv = 0.2;
  k.p1 = 1.1;
  k.p2 = 0.2;
  k.p3 = 0.9;
  Field Eu(cells, false), Ev(cells, false);
  fill(Eu.at, cells, 4);
  fill(Ev.at, cells, 5);
  std::vector<double> got[2];
  for (int odd = 0; odd < 2; odd++) {
    Field u(cells, odd), v(cells, odd);
    fill(u.at, cells, 6);
    fill(v.at, cells, 7);
    emu::launch((unsigned)((half + 255) / 256), 256, emu::ASCENDING,
                [&] { k_rd3_imex_final(g, k, u.at, v.at, Eu.at, Ev.at, 1e-2); });
    got[odd].assign(u.at, u.at + cells);
    got[odd].insert(got[odd].end(), v.at, v.at + cells);
  }
  same(got[0].data(), got[1].data(), 2 * cells, "imex");
  printf("wrong %d\n", wrong);
  return wrong != 0;
}
