// Host check of the multigrid's kernels with barriers (csrc/multigrid.hip, run on
// the CPU by cpu/hip/hip_runtime.h): the coarse tail in each of its forms, with its
// coarse matrix, and the tiled 2D level launches.  Each wave, and within it each
// lane, runs to its next wait before the others, in several orders of the waves;
// LDS starts as NaN.  Bar: the same bits in every order, and no NaN.
// Prints "checked N wrong M"; exit status 0 iff M == 0.
#include "multigrid.hip"

int amrv::set_error(int code, const char*) { return code; }

namespace {

thread_local double lds[160 * 1024 / 8];  // the tail's dynamic LDS

int checked = 0, wrong = 0;

template <int ND>
std::vector<double> cycle(int n, int bc, bool tiles, int pre, int post, emu::Order order) {
  std::mt19937_64 rng(5);
  std::uniform_real_distribution<double> u(-1.0, 1.0);
  std::vector<std::vector<double>> arrays;
  arrays.reserve(3 * MG_MAXL);
  auto array = [&](size_t cells) {
    arrays.emplace_back(cells);
    for (double& x : arrays.back()) x = u(rng);
    return arrays.back().data();
  };
  std::vector<double> par(PAR_COUNT), matrix(COARSE_CELLS * COARSE_CELLS, NAN);
  std::vector<unsigned long long> norms(2 * NFMAX * 16);
  MgDev g{};
  g.nd = ND;
  g.bc = bc;
  g.nf = 1;
  par[PAR_LAM] = 3.0;
  for (int m = n; m >= 2; m >>= 1, g.nlev++) {
    const int l = g.nlev;
    g.n[l] = m;
    while (1 << g.lg[l] < m) g.lg[l]++;
    g.cells[l] = ND == 2 ? m * m : m * m * m;
    g.phi[0][l] = array(g.cells[l]);
    g.f[0][l] = array(g.cells[l]);
    g.phi2[0][l] = array(g.cells[l]);
    par[PAR_IH2 + l] = (double)m * m;
    par[PAR_IDIAG + l] = 1.0 / (2.0 * ND * m * m + 3.0);
  }
  g.par = par.data();
  g.cmat[0] = g.cells[0] >= TAIL_CELLS ? matrix.data() : nullptr;
  g.hpart = norms.data();
  g.maxb = 16;
  std::fill(std::begin(lds), std::end(lds), NAN);
  int top = 0, coarse = 0;
  while (g.cells[top] > TAIL_CELLS) top++;
  while (g.cells[coarse] > COARSE_CELLS) coarse++;
  if (tiles) {
    if constexpr (ND == 2) {
      const unsigned nt = (unsigned)(n / TS);
      emu::launch(dim3(nt * nt), TT, order, [&] { k_mg_down2d(g, 0, pre); });
      emu::launch(dim3(nt * nt), TT, order, [&] { k_mg_up2d(g, 0, post, 1); });
    }
  } else if (g.cells[0] <= COARSE_CELLS) {
    emu::launch(dim3(1), 64, order, [&] { k_mg_small<ND>(g, pre, post); });
  } else {
    const unsigned threads = tail_threads<ND>();
    if (g.cmat[0]) {
      emu::launch(dim3(COARSE_CELLS), 64, order, [&] { k_mg_coarse_matrix<ND>(g, coarse, pre, post); });
      emu::launch(dim3(1), threads, order, [&] { k_mg_tail<ND, true>(g, top, pre, post, top > 0); });
    } else {
      emu::launch(dim3(1), threads, order, [&] { k_mg_tail<ND, false>(g, top, pre, post, top > 0); });
    }
  }
  std::vector<double> out;
  for (const auto& a : arrays) out.insert(out.end(), a.begin(), a.end());
  for (unsigned long long v : norms) out.push_back(bits_to_double(v));
  return out;
}

template <int ND>
void check(int n, bool tiles) {
  for (int bc : {AMRV_MG_PERIODIC, AMRV_MG_NEUMANN})
    for (int pre : {1, 2}) {
      const std::vector<double> ref = cycle<ND>(n, bc, tiles, pre, 3 - pre, emu::ASCENDING);
      for (emu::Order order : {emu::ASCENDING, emu::DESCENDING, emu::RANDOM}) {
        const std::vector<double> got = cycle<ND>(n, bc, tiles, pre, 3 - pre, order);
        checked++;
        if (!memcmp(got.data(), ref.data(), 8 * ref.size()) && std::none_of(got.begin(), got.end(), [](double x) { return x != x; }))
          continue;
        wrong++;
        printf("%dD n %d %s boundary %d pre %d order %d: differs or NaN\n", ND, n, tiles ? "tiles" : "tail", bc, pre,
               (int)order);
      }
    }
}

}  // namespace

int main() {
  for (int n : {4, 8, 16, 32, 64, 128}) check<2>(n, false);
  for (int n : {4, 8, 16, 32}) check<3>(n, false);
  check<2>(128, true);
  printf("checked %d wrong %d\n", checked, wrong);
  return wrong != 0;
}
