// Host-side check of the direct solver's elimination plan: runs the plan's tasks in their
// order on the CPU, each reading only what the tables name, and checks that every task
// comes after those it waits for.
#include <cmath>
#include <vector>

#include "direct.h"

using namespace phisft;

// A: [maxnz][9][nv] symmetric positive definite; x receives the solution of A x = b
// ([3][nv] both). Returns 0, or the number of the check that failed.
extern "C" int direct_check(int nv, int maxnz, const int* ell_col, int nsheets, const int* voff,
                            const int* sheet_nv, const double* xr, const double* A,
                            const double* b, double* x, int* out_counts) {
  DsPlan P;
  build_direct_plan(nv, maxnz, std::vector<int>(ell_col, ell_col + (size_t)maxnz * nv),
                    std::vector<int>(voff, voff + nsheets),
                    std::vector<int>(sheet_nv, sheet_nv + nsheets),
                    std::vector<double>(xr, xr + 3 * (size_t)nv), P);
  if (!P.ok) return 1;
  out_counts[0] = (int)P.fronts.size();
  out_counts[1] = P.levels();
  out_counts[2] = P.max_np;
  out_counts[3] = P.max_nb;
  std::vector<double> fac(P.factor_doubles, 0.0), ws(P.work_doubles, 0.0);
  std::vector<int> count(P.counters, 0), owner(nv, 0);
  auto rows_of = [&](const DsFront& F) { return (F.nb + kDsRowTile - 1) / kDsRowTile; };
  constexpr int per = kDsSchurTile / kDsRowTile;
  for (const DsTask& k : P.factor_tasks) {
    const DsFront& F = P.fronts[k.front];
    double* X = fac.data() + F.xo;
    double* W = fac.data() + F.wo;
    double* S = ws.data() + F.so;
    double* B = ws.data() + F.bo;
    if (k.kind == kDsPivot) {
      std::vector<double> M((size_t)F.np * F.np, 0.0);
      for (int i = 3 * F.p; i < F.np; ++i) M[(size_t)i * F.np + i] = 1.0;
      for (int e = 0; e < F.nalist; ++e) {
        const int at = P.tab[F.alist + 2 * e], l = P.tab[F.alist + 2 * e + 1] >> 16,
                  i = P.tab[F.alist + 2 * e + 1] & 0xffff;
        for (int q = 0; q < 9; ++q) {
          const double v = A[at + (size_t)q * nv];
          M[(size_t)(3 * l + q % 3) * F.np + 3 * i + q / 3] = v;
          M[(size_t)(3 * i + q / 3) * F.np + 3 * l + q % 3] = v;
        }
      }
      for (int i = 0; i < F.p; ++i) ++owner[P.tab[F.verts + i]];
      for (int c = F.c0; c < F.c0 + F.nc; ++c) {
        const DsChild& K = P.kids[c];
        if (count[K.cnt + kDsHeadDone] < K.nhead) return 2;
        // the parent's pivots are inside the child's first two tile rows
        if (3 * K.q > 2 * kDsSchurTile) return 3;
        for (int u = 0; u < 3 * K.q; ++u)
          for (int v = 0; v <= u; ++v) {
            const int r = 3 * P.tab[K.map + u / 3] + u % 3, s = 3 * P.tab[K.map + v / 3] + v % 3;
            M[(size_t)r * F.np + s] += ws[K.so + (long long)u * K.nb + v];
            if (r != s) M[(size_t)s * F.np + r] += ws[K.so + (long long)u * K.nb + v];
          }
      }
      for (int d = 0; d < F.np; ++d) {   // in-place Gauss-Jordan inverse
        const double piv = 1.0 / M[(size_t)d * F.np + d];
        if (!(piv > 0.0)) return 4;
        M[(size_t)d * F.np + d] = 1.0;
        for (int j = 0; j < F.np; ++j) M[(size_t)d * F.np + j] *= piv;
        for (int i = 0; i < F.np; ++i) {
          if (i == d) continue;
          const double f = M[(size_t)i * F.np + d];
          M[(size_t)i * F.np + d] = 0.0;
          for (int j = 0; j < F.np; ++j) M[(size_t)i * F.np + j] -= f * M[(size_t)d * F.np + j];
        }
      }
      std::copy(M.begin(), M.end(), X);
      ++count[F.cnt + kDsPivotDone];
    } else if (k.kind == kDsBorder) {
      if (count[F.cnt + kDsPivotDone] < 1) return 5;
      const int r0 = k.a * kDsRowTile, r1 = std::min(F.nb, r0 + kDsRowTile);
      for (int e = P.tab[F.blist + k.a]; e < P.tab[F.blist + k.a + 1]; e += 2) {
        const int at = P.tab[e], l = P.tab[e + 1] >> 16, i = P.tab[e + 1] & 0xffff;
        for (int q = 0; q < 9; ++q) {
          const int r = 3 * (l - F.p) + q % 3;
          if (r >= r0 && r < r1) B[(size_t)r * F.np + 3 * i + q / 3] += A[at + (size_t)q * nv];
        }
      }
      for (int c = F.c0; c < F.c0 + F.nc; ++c) {
        const DsChild& K = P.kids[c];
        if (count[K.cnt + kDsSchurDone] < K.nschur) return 6;
        for (int r = r0; r < std::min(r1, 3 * F.b); ++r) {
          const int u = P.tab[K.inv + F.p + r / 3];
          for (int s = 0; u >= 0 && s < 3 * F.p; ++s) {
            const int v = P.tab[K.inv + s / 3];
            if (v >= 0) B[(size_t)r * F.np + s] += ws[K.so + (long long)(3 * u + r % 3) * K.nb + 3 * v + s % 3];
          }
        }
      }
      for (int r = r0; r < r1; ++r)
        for (int c = 0; c < F.np; ++c) {
          double w = 0.0;
          for (int d = 0; d < F.np; ++d) w += B[(size_t)r * F.np + d] * X[(size_t)d * F.np + c];
          W[(size_t)r * F.np + c] = w;
        }
      ++count[F.cnt + kDsRowsDone + k.a / per];
    } else if (k.kind == kDsSchur) {
      const int I = k.a >> 16, J = k.a & 0xffff;
      for (int g : {I, J})
        if (count[F.cnt + kDsRowsDone + g] < std::min(per, rows_of(F) - per * g)) return 7;
      for (int r = I * kDsSchurTile; r < std::min(F.nb, (I + 1) * kDsSchurTile); ++r)
        for (int c = J * kDsSchurTile; c <= std::min(r, (J + 1) * kDsSchurTile - 1); ++c) {
          double s = 0.0;
          for (int d = 0; d < F.np; ++d) s -= W[(size_t)r * F.np + d] * B[(size_t)c * F.np + d];
          for (int h = F.c0; h < F.c0 + F.nc && r < 3 * F.b; ++h) {
            const DsChild& K = P.kids[h];
            if (count[K.cnt + kDsSchurDone] < K.nschur) return 8;
            const int u = P.tab[K.inv + F.p + r / 3], v = P.tab[K.inv + F.p + c / 3];
            if (u >= 0 && v >= 0)
              s += ws[K.so + (long long)(3 * u + r % 3) * K.nb + 3 * v + c % 3];
          }
          S[(size_t)r * F.nb + c] = s;
        }
      if (I < 2) ++count[F.cnt + kDsHeadDone];
      ++count[F.cnt + kDsSchurDone];
    } else if (k.kind == kDsForward) {
      if (count[F.cnt + kDsPivotDone] < 1) return 9;
      std::vector<double> v(3 * (F.p + F.b), 0.0);
      for (int i = 0; i < 3 * F.p; ++i) v[i] = b[(size_t)(i % 3) * nv + P.tab[F.verts + i / 3]];
      for (int h = 0; h < F.nc; ++h) {
        const DsChild& K = P.kids[F.c0 + h];
        if (count[K.cnt + kDsForwardDone] < K.nfwd) return 10;
        for (int i = 0; i < 3 * (F.p + F.b); ++i) {
          const int at = P.tab[F.gsrc + h * (F.p + F.b) + i / 3];
          if (at >= 0) v[i] += ws[at + i % 3];
        }
      }
      for (int g = 0; g * kDsSchurTile < F.nb; ++g)
        if (count[F.cnt + kDsRowsDone + g] < std::min(per, rows_of(F) - per * g)) return 11;
      if (k.a == 0)
        for (int i = 0; i < 3 * F.p; ++i) ws[F.t + i] = v[i];
      for (int r = k.a * kDsFwdRows; r < std::min(3 * F.b, (k.a + 1) * kDsFwdRows); ++r) {
        double g = v[3 * F.p + r];
        for (int d = 0; d < 3 * F.p; ++d) g -= W[(size_t)r * F.np + d] * v[d];
        ws[F.g + r] = g;
      }
      ++count[F.cnt + kDsForwardDone];
    } else {
      if (count[F.cnt + kDsForwardDone] < F.nfwd) return 12;
      if (F.pcnt >= 0 && count[F.pcnt + kDsBackwardDone] < F.pbwd) return 13;
      for (int c = k.a * kDsBwdCols; c < std::min(3 * F.p, (k.a + 1) * kDsBwdCols); ++c) {
        double s = 0.0;
        for (int d = 0; d < 3 * F.p; ++d) s += X[(size_t)c * F.np + d] * ws[F.t + d];
        for (int r = 0; r < 3 * F.b; ++r)
          s -= W[(size_t)r * F.np + c] * ws[P.tab[F.xsrc + r / 3] + r % 3];
        ws[F.x + c] = s;
        x[(size_t)(c % 3) * nv + P.tab[F.verts + c / 3]] = s;
      }
      ++count[F.cnt + kDsBackwardDone];
    }
  }
  for (int v = 0; v < nv; ++v)
    if (owner[v] != 1) return 14;
  // the two passes alone: a subsequence of the same tasks in the same order
  size_t at = 0;
  for (const DsTask& k : P.factor_tasks)
    if (k.kind >= kDsForward) {
      if (at >= P.solve_tasks.size()) return 15;
      const DsTask& q = P.solve_tasks[at++];
      if (q.kind != k.kind || q.front != k.front || q.a != k.a) return 16;
    }
  return at == P.solve_tasks.size() ? 0 : 17;
}
