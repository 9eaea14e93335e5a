// Host check of the forest multigrid's kernels (csrc/fmg.hip): their source runs
// on the CPU (cpu/hip/hip_runtime.h) on a forest read from argv[1], one V-cycle's
// launches in order, each against the per-cell functions (stencil, apply_cell,
// across) bit for bit: the coarse-fine ghosts kept in a leaf's residual array and
// every sum that reads them, in the batch sizes the kernels use, with one and
// several workgroups per block.  Arrays start as NaN where nothing may read them.
// Input: "nleaves base max_level bc ndim", then "level i j k" per leaf.
// Prints "checked N mismatches M"; exit status 0 iff M == 0.
#include "fmg.hip"

#include <fstream>

int amrv::set_error(int code, const char* msg) {
  printf("%s\n", msg);
  return code;
}
int amrv::mg_correction_grids(amrv_mg*, double**, double**, bool*) { return -1; }
int amrv::mg_enqueue_correction(amrv_mg*, const double*, double*, double, int, bool) { return -1; }
size_t amrv_mg_workspace_bytes(const amrv_mg_config*) { return 0; }
int amrv_mg_create(const amrv_mg_config*, void*, size_t, void*, amrv_mg**) { return -1; }
int amrv_mg_destroy(amrv_mg*) { return 0; }

namespace {

long long checked = 0, bad = 0;

void same(double a, double b, const char* what, int block) {
  checked++;
  if (!memcmp(&a, &b, 8)) return;
  if (bad++ < 10) printf("%s: block %d: %.17g instead of %.17g\n", what, block, b, a);
}

template <int ND>
struct Check {
  static constexpr int NCB = ncb<ND>(), NF = nface<ND>();
  const Tree& T;
  const amrv_fmg_config& c;
  std::vector<double> u, f, fu, r, uo;
  FmgDev g{};

  Check(const Tree& t, const amrv_fmg_config& cfg) : T(t), c(cfg) {
    std::mt19937_64 rng(5);
    std::uniform_real_distribution<double> U(-1.0, 1.0);
    const size_t n = (size_t)T.nblk * NCB;
    for (auto* v : {&u, &f, &fu, &r, &uo}) {
      v->resize(n);
      for (double& x : *v) x = v == &r || v == &uo ? NAN : U(rng);
    }
    for (int b = 0; b < T.nblk; b++)  // a leaf's right-hand side is the problem's, as loading it leaves it
      if (T.chi[CS * b] < 0) std::copy_n(&fu[(size_t)b * NCB], NCB, &f[(size_t)b * NCB]);
    g.lvl = T.lvl.data();
    g.ij = T.ij.data();
    g.nbr = T.nbr.data();
    g.chi = T.chi.data();
    g.cnb = T.cnb.data();
    g.par = T.par.data();
    g.u = u.data();
    g.f = f.data();
    g.fu = fu.data();
    g.r = r.data();
    g.uo = uo.data();
    g.lam = 7.0;
    for (int l = 1; l <= FMG_MAXL; l++) {
      const double q = (double)((long long)c.base * NB << (l - 1)) / c.length;
      g.ih2[l] = q * q;
      g.rh[l] = q;
    }
  }

  bool leaf(int b) const { return T.chi[CS * b] < 0; }
  template <class Fn>
  void cells(Fn fn) {
    for (int t = 0; t < NCB; t++) {
      int x[3];
      ncell(t, x);
      fn(x);
    }
  }
  template <class Fn>
  void level(int l, Fn fn) {
    for (int b = T.lstart[l]; b < T.lstart[l + 1]; b++) cells([&](const int* x) { fn(b, x, (size_t)b * NCB + cidx(x)); });
  }
  unsigned blocks(int l) const { return (unsigned)(T.lstart[l + 1] - T.lstart[l]); }
  template <class K>
  void launch(dim3 grid, unsigned threads, K kernel) {
    emu::launch(grid, threads, emu::RANDOM, kernel);
  }

  void ghosts(int l, const char* what) {  // of every leaf (l = 0) or of one level's
    for (int b = l ? T.lstart[l] : 0; b < (l ? T.lstart[l + 1] : T.nblk); b++)
      for (int face = 0; face < 2 * ND && leaf(b); face++)
        for (int t = 0; t < NF && T.nbr[FS * b + face] == NBR_NONE; t++) {
          int x[3];
          face_coord<ND>(face, t, x);
          same(across<ND>(g, b, false, x, face).cv, r[(size_t)b * NCB + face * NF + t], what, b);
        }
  }

  void sweep(int l, int colour, unsigned parts) {
    std::vector<double> want = u;
    level(l, [&](int b, const int* x, size_t i) {
      if (((x[0] + x[1] + x[2]) & 1) != colour) return;
      double sc, sw;
      stencil<ND>(g, b, false, x, sc, sw);
      const double ih2 = g.ih2[l];
      want[i] = (f[i] - ih2 * sc) / (ih2 * (sw - 2.0 * ND) - g.lam);
    });
    launch(dim3(blocks(l), ND == 3 ? parts : 1), ND == 3 ? WG : WG / 2, [&] { k_fmg_smooth<ND>(g, T.lstart[l], colour); });
    for (size_t i = 0; i < u.size(); i++) same(want[i], u[i], "sweep", (int)(i / NCB));
  }

  void restriction(int l, unsigned parts) {
    std::vector<double> wu = u, wo = uo, wr = r;
    for (int b = T.lstart[l]; b < T.lstart[l + 1]; b++)
      for (int t = 0; t < NCB >> ND; t++) {
        const int y[3] = {t & 7, (t >> 3) & 7, t >> 6};
        double s[8], d[8];
        for (int k = 0; k < 1 << ND; k++) {
          const int x[3] = {2 * y[0] + (k & 1), 2 * y[1] + ((k >> 1) & 1), ND == 3 ? 2 * y[2] + (k >> 2) : 0};
          const size_t i = (size_t)b * NCB + cidx(x);
          s[k] = u[i];
          d[k] = f[i] - apply_cell<ND>(g, b, false, x);
        }
        auto mean = [](const double* v) {
          const double lo = (v[0] + v[1]) + (v[2] + v[3]);
          return ND == 2 ? 0.25 * lo : 0.125 * (lo + ((v[4] + v[5]) + (v[6] + v[7])));
        };
        int p[3];
        for (int e = 0; e < 3; e++) p[e] = (e < ND ? 8 * (T.ij[TS * b + e] & 1) : 0) + y[e];
        const size_t i = (size_t)T.par[b] * NCB + cidx(p);
        wu[i] = wo[i] = mean(s);
        wr[i] = mean(d);
      }
    launch(dim3(blocks(l), ND == 3 ? parts : 1), ND == 3 ? WG : 64, [&] { k_fmg_resid_restrict<ND>(g, T.lstart[l]); });
    for (size_t i = 0; i < u.size(); i++) {
      same(wu[i], u[i], "restricted state", (int)(i / NCB));
      same(wo[i], uo[i], "kept restricted state", (int)(i / NCB));
      same(wr[i], r[i], "restricted residual", (int)(i / NCB));
    }
  }

  void fas(int l, unsigned parts) {
    std::vector<double> want = f;
    level(l, [&](int b, const int* x, size_t i) {
      const double lp = apply_cell<ND>(g, b, false, x);
      if (!leaf(b)) {
        want[i] = lp + r[i];
        return;
      }
      bool along = false;
      for (int face = 0; face < 2 * ND; face++) {
        const int nb = T.nbr[FS * b + face];
        along = along || (nb >= 0 && !leaf(nb) && x[face >> 1] == ((face & 1) ? NB - 1 : 0));
      }
      const double lc = apply_cell<ND>(g, b, true, x);
      if (along) want[i] = lp == lc ? fu[i] : lp + (fu[i] - lc);
    });
    launch(dim3(blocks(l), ND == 3 ? parts : 1), WG, [&] { k_fmg_fas<ND>(g, T.lstart[l]); });
    for (size_t i = 0; i < f.size(); i++) same(want[i], f[i], "coarse right-hand side", (int)(i / NCB));
  }

  // level 1 to the n^ND grid and its correction back
  void grid(unsigned parts, bool split) {
    const int n = c.base * NB;
    size_t cellsn = 1;
    for (int e = 0; e < ND; e++) cellsn *= (size_t)n;
    std::vector<double> fg(cellsn, NAN), vg(cellsn, NAN);
    launch(dim3(blocks(1), ND == 3 ? parts : 1), WG,
           [&] { k_fmg_resid_grid<ND>(g, T.lstart[1], n, split, fg.data(), vg.data()); });
    auto at = [&](int b, const int* x) {
      int q[3] = {0, 0, 0}, lg = 0;
      for (int e = 0; e < ND; e++) q[e] = T.ij[TS * b + e] * NB + x[e];
      while (1 << lg < n) lg++;
      return split ? (size_t)amrv::split_idx<ND>(q[0], q[1], q[2], lg) : ((size_t)q[2] * n + q[1]) * n + q[0];
    };
    level(1, [&](int b, const int* x, size_t i) {
      same(f[i] - apply_cell<ND>(g, b, false, x), fg[at(b, x)], "level-1 residual", b);
      same(0.0, vg[at(b, x)], "level-1 correction", b);
      vg[at(b, x)] = 0.01 * u[i];
    });
    std::vector<double> want = u;
    level(1, [&](int b, const int* x, size_t i) {
      if ((x[0] + x[1] + x[2]) & 1) want[i] += vg[at(b, x)];
    });
    launch(dim3(blocks(1)), ND == 3 ? WG : WG / 2, [&] { k_fmg_from_grid<ND>(g, T.lstart[1], n, split, vg.data()); });
    for (size_t i = 0; i < u.size(); i++) same(want[i], u[i], "level-1 update", (int)(i / NCB));
  }

  void prolong(int l) {
    std::vector<double> want = u;
    level(l, [&](int b, const int* x, size_t i) {
      if (!((x[0] + x[1] + x[2]) & 1)) return;
      int I[3] = {0, 0, 0}, J[3] = {0, 0, 0};  // the parent's cell and its neighbour toward x, within the parent
      for (int e = 0; e < ND; e++) {
        I[e] = 8 * (T.ij[TS * b + e] & 1) + (x[e] >> 1);
        J[e] = std::min(std::max(I[e] + ((x[e] & 1) ? 1 : -1), 0), NB - 1);
      }
      auto e = [&](int p, int q, int s) {
        const int k[3] = {p ? J[0] : I[0], q ? J[1] : I[1], s ? J[2] : I[2]};
        const size_t j = (size_t)T.par[b] * NCB + cidx(k);
        return u[j] - uo[j];
      };
      const double d = ND == 2 ? (9.0 * e(0, 0, 0) + 3.0 * e(1, 0, 0) + 3.0 * e(0, 1, 0) + e(1, 1, 0)) * (1.0 / 16.0)
                               : (27.0 * e(0, 0, 0) + 9.0 * (e(1, 0, 0) + e(0, 1, 0) + e(0, 0, 1)) +
                                  3.0 * (e(1, 1, 0) + e(1, 0, 1) + e(0, 1, 1)) + e(1, 1, 1)) *
                                     (1.0 / 64.0);
      want[i] += d;
    });
    launch(dim3(blocks(l), ND == 3 ? 3 : 2), ND == 3 ? WG : WG / 2, [&] { k_fmg_prolong<ND>(g, T.lstart[l]); });
    for (size_t i = 0; i < u.size(); i++) same(want[i], u[i], "prolonged state", (int)(i / NCB));
    ghosts(l, "ghosts of a prolonged level");
  }

  void norms(unsigned parts) {
    const int n = (int)T.leafblk.size();
    double mr = 0.0, mf = 0.0, host[2] = {-1.0, -1.0};
    for (int b : T.leafblk)
      cells([&](const int* x) {
        const double q = fu[(size_t)b * NCB + cidx(x)];
        mr = std::max(mr, std::fabs(q - apply_cell<ND>(g, b, true, x)));
        mf = std::max(mf, std::fabs(q));
      });
    launch(dim3((unsigned)n, parts), WG, [&] { k_fmg_resmax<ND>(g, T.leafblk.data(), 1); });
    launch(dim3(1), 1024, [&] { k_fmg_resmax_all<ND>(g, T.leafblk.data(), n, (int)parts, 1, host); });
    same(mr, host[0], "max |r|", -1);
    same(mf, host[1], "max |f|", -1);
  }

  // a leaf field loaded (from 8 bytes past a 16-byte boundary), its Laplacian
  void field() {
    const int n = (int)T.leafblk.size();
    const size_t off = (reinterpret_cast<uintptr_t>(fu.data()) & 15) ? 0 : 1;
    std::vector<double> w((size_t)n * NCB + 1), out((size_t)n * NCB, NAN), keep = u;
    for (size_t i = 0; i < w.size(); i++) w[i] = std::sin(0.37 * (double)i);
    FmgDev h = g;
    h.lam = 0.0;
    launch(dim3((unsigned)n), WG, [&] { k_fmg_load<ND>(h, T.leafblk.data(), w.data() + off); });
    std::vector<double> want = keep;
    for (int k = 0; k < n; k++)
      for (int t = 0; t < NCB; t++) {
        int x[3];
        ncell(t, x);
        want[(size_t)T.leafblk[k] * NCB + cidx(x)] = w[off + (size_t)k * NCB + t];
      }
    for (size_t i = 0; i < u.size(); i++) same(want[i], u[i], "loaded field", (int)(i / NCB));
    if (ND == 3) launch(dim3((unsigned)n, 2), WG, [&] { k_fmg_ghosts<ND>(h, T.leafblk.data()); });
    launch(dim3((unsigned)n), WG, [&] { k_fmg_lap<ND>(h, T.leafblk.data(), 0.7, out.data()); });
    for (int k = 0; k < n; k++)
      cells([&](const int* x) {
        same(0.7 * apply_cell<ND>(h, T.leafblk[k], true, x), out[(size_t)k * NCB + nidx(x)], "Laplacian", T.leafblk[k]);
      });
    u = keep;
    g.u = u.data();
  }

  void run() {
    const int L = T.nlev;
    field();
    launch(dim3((unsigned)T.leafblk.size(), ND == 3 ? 2 : 1), WG, [&] { k_fmg_ghosts<ND>(g, T.leafblk.data()); });
    ghosts(0, "ghosts");
    norms(ND == 3 ? 2 : 1);
    for (int l = L; l >= 2; l--) {
      sweep(l, 0, 1);
      sweep(l, 1, 2);
      restriction(l, l == L ? 2 : 1);
      fas(l - 1, l == L ? 4 : 1);
    }
    sweep(1, 0, 2);
    sweep(1, 1, 1);
    grid(4, false);
    if (ND == 3) grid(1, true);
    sweep(1, 0, 1);
    for (int l = 2; l <= L; l++) {
      prolong(l);
      sweep(l, 0, 2);
      sweep(l, 1, 1);
    }
    norms(ND == 3 ? 2 : 1);
  }
};

}  // namespace

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  std::ifstream in(argv[1]);
  amrv_fmg_config c{};
  long long n;
  in >> n >> c.base >> c.max_level >> c.bc >> c.ndim;
  if (!in || (c.ndim != 2 && c.ndim != 3)) return 2;
  c.nleaves = n;
  c.pre_sweeps = c.post_sweeps = 2;
  c.length = 1.0;
  std::vector<int32_t> lev(n), ijk(3 * n);
  for (long long k = 0; k < n; k++) in >> lev[k] >> ijk[3 * k] >> ijk[3 * k + 1] >> ijk[3 * k + 2];
  Tree T;
  if (build_tree(&c, lev.data(), ijk.data(), T)) return 1;
  if (c.ndim == 3)
    Check<3>(T, c).run();
  else
    Check<2>(T, c).run();
  printf("blocks %d levels %d checked %lld mismatches %lld\n", T.nblk, T.nlev, checked, bad);
  return bad != 0;
}
