// direct_prep.cpp -- elimination plan of the direct solver: nested dissection of every
// sheet's vertex graph by its rest shape, the fronts of its elimination tree and the
// maps by which a front gathers its children's updates.
//
// A piece of the sheet is cut across its longest extent; the vertices on one side of the
// cut that couple to the other side are its separator (two grid lines of a grid sheet,
// whose rows reach two vertices far). Both halves are eliminated first, then the
// separator, in chunks of at most kDsMaxPiv vertices: a chunk's pivot block then fits one
// workgroup.

#include "direct.h"

#include <algorithm>
#include <cstdint>
#include <utility>

namespace phisft {
namespace {

struct Builder {
  int nv, maxnz;
  const std::vector<int>& col;
  const std::vector<double>& xr;
  std::vector<std::vector<int>> chunks;   // pivots of each front, elimination order
  std::vector<int> mark;
  int leaf = 0;

  int neighbour(int i, int k) const { return col[(size_t)k * nv + i]; }

  void emit(std::vector<int> s) {
    if (s.empty()) return;
    const int n = (int)s.size(), parts = (n + kDsMaxPiv - 1) / kDsMaxPiv;
    int at = 0;
    for (int c = 0; c < parts; ++c) {
      const int end = (int)((long long)n * (c + 1) / parts);
      chunks.emplace_back(s.begin() + at, s.begin() + end);
      at = end;
    }
  }

  // Cuts s: `low` and `high` keep no coupling, `sep` separates them.
  void cut(std::vector<int>& s, std::vector<int>& low, std::vector<int>& high,
           std::vector<int>& sep) {
    const int n = (int)s.size();
    double lo[3], hi[3];
    for (int c = 0; c < 3; ++c) lo[c] = hi[c] = xr[3 * (size_t)s[0] + c];
    for (int v : s)
      for (int c = 0; c < 3; ++c) {
        lo[c] = std::min(lo[c], xr[3 * (size_t)v + c]);
        hi[c] = std::max(hi[c], xr[3 * (size_t)v + c]);
      }
    int ax = 0;
    for (int c = 1; c < 3; ++c)
      if (hi[c] - lo[c] > (hi[ax] - lo[ax]) * (1.0 + 1e-9)) ax = c;
    const double eps = 1e-7 * (hi[ax] - lo[ax]);
    std::sort(s.begin(), s.end(), [&](int a, int b) {
      const double xa = xr[3 * (size_t)a + ax], xb = xr[3 * (size_t)b + ax];
      return xa != xb ? xa < xb : a < b;
    });
    // candidate cuts: where the coordinate jumps, the nearest ones around the middle
    std::vector<int> cand;
    int below = 0, above = 0;
    for (int d = 0; d < n && (below < 3 || above < 3); ++d)
      for (int side = 0; side < 2; ++side) {
        const int i = side == 0 ? n / 2 + d : n / 2 - 1 - d;
        int& cnt = side == 0 ? above : below;
        if (i < 1 || i >= n || cnt >= 3) continue;
        if (xr[3 * (size_t)s[i] + ax] - xr[3 * (size_t)s[i - 1] + ax] > eps) {
          cand.push_back(i);
          ++cnt;
        }
      }
    if (cand.empty()) cand.push_back(n / 2);
    long long best = -1;
    int best_i = cand[0], best_side = 0;
    auto separator = [&](int i, int side, std::vector<int>* out) {
      // side 0: the low vertices that couple to a high one; side 1: the reverse
      for (int q = 0; q < n; ++q) mark[s[q]] = q < i ? 1 : 2;
      int cnt = 0;
      const int from = side == 0 ? 0 : i, to = side == 0 ? i : n, other = side == 0 ? 2 : 1;
      for (int q = from; q < to; ++q)
        for (int k = 0; k < maxnz; ++k) {
          const int j = neighbour(s[q], k);
          if (j >= 0 && mark[j] == other) {
            ++cnt;
            if (out) out->push_back(s[q]);
            break;
          }
        }
      for (int q = 0; q < n; ++q) mark[s[q]] = 0;
      return cnt;
    };
    for (int i : cand)
      for (int side = 0; side < 2; ++side) {
        const int m = separator(i, side, nullptr);
        const int a = side == 0 ? i - m : i, b = side == 0 ? n - i : n - i - m;
        const long long cost = 4LL * m * m + (long long)std::max(a, b) * std::max(a, b) / 4;
        if (best < 0 || cost < best) {
          best = cost;
          best_i = i;
          best_side = side;
        }
      }
    separator(best_i, best_side, &sep);
    for (int v : sep) mark[v] = 3;
    for (int q = 0; q < n; ++q)
      if (mark[s[q]] != 3) (q < best_i ? low : high).push_back(s[q]);
    for (int v : sep) mark[v] = 0;
  }

  void dissect(std::vector<int> s) {
    if ((int)s.size() <= leaf) {
      emit(std::move(s));
      return;
    }
    std::vector<int> low, high, sep;
    cut(s, low, high, sep);
    if (low.empty() || high.empty()) {   // no cut separates it: dense
      emit(std::move(s));
      return;
    }
    s.clear();
    s.shrink_to_fit();
    dissect(std::move(low));
    dissect(std::move(high));
    emit(std::move(sep));
  }
};

int up16(int n) { return (n + kDsTile - 1) / kDsTile * kDsTile; }

}  // namespace

void build_direct_plan(int nv, int maxnz, const std::vector<int>& ell_col,
                       const std::vector<int>& inst_voff, const std::vector<int>& inst_nv,
                       const std::vector<double>& xr, DsPlan& P, double max_doubles) {
  P = DsPlan{};
  const int ninst = (int)inst_voff.size();
  Builder B{nv, maxnz, ell_col, xr, {}, std::vector<int>(nv, 0)};
  for (int b = 0; b < ninst; ++b) {
    std::vector<int> s(inst_nv[b]);
    for (int q = 0; q < inst_nv[b]; ++q) s[q] = inst_voff[b] + q;
    B.leaf = inst_nv[b] <= kDsSmallSheet ? kDsLeafSmall : kDsLeaf;
    B.dissect(std::move(s));
  }
  const int nf = (int)B.chunks.size();
  std::vector<int> epos(nv, -1), owner(nv, -1), first(nf);
  int at = 0;
  for (int f = 0; f < nf; ++f) {
    first[f] = at;
    for (int v : B.chunks[f]) {
      epos[v] = at++;
      owner[v] = f;
    }
  }
  // borders, bottom up (elimination order is a postorder of the tree)
  std::vector<std::vector<int>> border(nf), kids(nf);
  std::vector<int> parent(nf, -1), level(nf, 0);
  std::vector<int> stamp(nv, -1);
  for (int f = 0; f < nf; ++f) {
    const int last = first[f] + (int)B.chunks[f].size() - 1;
    auto add = [&](int v) {
      if (epos[v] > last && stamp[v] != f) {
        stamp[v] = f;
        border[f].push_back(v);
      }
    };
    for (int v : B.chunks[f])
      for (int k = 0; k < maxnz; ++k) {
        const int j = ell_col[(size_t)k * nv + v];
        if (j >= 0) add(j);
      }
    for (int c : kids[f]) {
      for (int v : border[c]) add(v);
      level[f] = std::max(level[f], level[c] + 1);
    }
    std::sort(border[f].begin(), border[f].end(), [&](int a, int b) { return epos[a] < epos[b]; });
    if (!border[f].empty()) {
      parent[f] = owner[border[f][0]];
      kids[parent[f]].push_back(f);
    }
    if (3 * (int)border[f].size() > kDsMaxBorder - kDsTile) return;
  }
  // fronts by level
  std::vector<int> order(nf), id(nf);
  for (int f = 0; f < nf; ++f) order[f] = f;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return level[a] < level[b]; });
  for (int q = 0; q < nf; ++q) id[order[q]] = q;
  const int nlev = nf ? level[order[nf - 1]] + 1 : 0;
  P.fronts.resize(nf);
  P.level0.assign(nlev + 1, 0);
  for (int f = 0; f < nf; ++f) P.level0[level[f] + 1]++;
  for (int l = 0; l < nlev; ++l) P.level0[l + 1] += P.level0[l];
  // sizes and places of the fronts' arrays
  auto tiles = [](int n, int t) { return (n + t - 1) / t; };
  auto heads = [&](const DsFront& F) {
    const int st = std::min(2, tiles(F.nb, kDsSchurTile));
    return st * (st + 1) / 2;
  };
  auto schurs = [&](const DsFront& F) {
    const int st = tiles(F.nb, kDsSchurTile);
    return st * (st + 1) / 2;
  };
  for (int q = 0; q < nf; ++q) {
    const int f = order[q];
    DsFront& F = P.fronts[q];
    F.p = (int)B.chunks[f].size();
    F.b = (int)border[f].size();
    F.np = up16(3 * F.p);
    F.nb = up16(3 * F.b);
    F.nfwd = std::max(1, tiles(F.nb, kDsFwdRows));
    F.t = (int)P.work_doubles;
    F.x = F.t + F.np;
    F.g = F.x + F.np;
    P.work_doubles += 2LL * F.np + F.nb;
    F.cnt = P.counters;
    P.counters += (kDsRowsDone + tiles(F.nb, kDsSchurTile) + 7) / 8 * 8;
    F.xo = P.factor_doubles;
    F.wo = F.xo + (long long)F.np * F.np;
    P.factor_doubles = F.wo + (long long)F.nb * F.np;
    P.max_np = std::max(P.max_np, F.np);
    P.max_nb = std::max(P.max_nb, F.nb);
  }
  for (DsFront& F : P.fronts) {
    F.so = P.work_doubles;
    F.bo = F.so + (long long)F.nb * F.nb;
    P.work_doubles = F.bo + (long long)F.nb * F.np;
  }
  if (max_doubles > 0.0 && (double)P.factor_doubles + (double)P.work_doubles > max_doubles) return;
  // index tables
  std::vector<int> local(nv, -1);
  std::vector<std::vector<std::pair<int, int>>> rows;
  for (int q = 0; q < nf; ++q) {
    const int f = order[q];
    DsFront& F = P.fronts[q];
    F.verts = (int)P.tab.size();
    P.tab.insert(P.tab.end(), B.chunks[f].begin(), B.chunks[f].end());
    P.tab.insert(P.tab.end(), border[f].begin(), border[f].end());
    for (int l = 0; l < F.p + F.b; ++l) local[P.tab[F.verts + l]] = l;
    F.pcnt = -1;
    F.pbwd = 0;
    if (parent[f] >= 0) {
      const DsFront& O = P.fronts[id[parent[f]]];
      F.pcnt = O.cnt;
      F.pbwd = tiles(O.np, kDsBwdCols);
    }
    // entries of A: the pivots' rows, columns not eliminated before
    std::vector<std::pair<int, int>> piv;
    rows.assign(tiles(F.nb, kDsRowTile), {});
    for (int i = 0; i < F.p; ++i) {
      const int v = B.chunks[f][i];
      for (int k = 0; k < maxnz; ++k) {
        const int j = ell_col[(size_t)k * nv + v];
        if (j < 0 || epos[j] < first[f]) continue;
        const int l = local[j];
        const std::pair<int, int> e(k * 9 * nv + v, l << 16 | i);
        if (l < F.p) {
          if (l >= i) piv.push_back(e);
        } else {
          const int r = 3 * (l - F.p);
          rows[r / kDsRowTile].push_back(e);
          if ((r + 2) / kDsRowTile != r / kDsRowTile) rows[(r + 2) / kDsRowTile].push_back(e);
        }
      }
    }
    P.tab.resize((P.tab.size() + 1) / 2 * 2);   // pairs are read as int2
    F.alist = (int)P.tab.size();
    F.nalist = (int)piv.size();
    for (auto& e : piv) {
      P.tab.push_back(e.first);
      P.tab.push_back(e.second);
    }
    std::vector<int> at;
    for (auto& r : rows) {
      at.push_back((int)P.tab.size());
      for (auto& e : r) {
        P.tab.push_back(e.first);
        P.tab.push_back(e.second);
      }
    }
    at.push_back((int)P.tab.size());
    F.blist = (int)P.tab.size();
    P.tab.insert(P.tab.end(), at.begin(), at.end());
    F.xsrc = (int)P.tab.size();
    for (int v : border[f]) {
      const DsFront& O = P.fronts[id[owner[v]]];
      P.tab.push_back(O.x + 3 * (epos[v] - first[owner[v]]));
    }
    F.c0 = (int)P.kids.size();
    F.nc = (int)kids[f].size();
    F.gsrc = (int)P.tab.size();
    P.tab.resize(P.tab.size() + (size_t)F.nc * (F.p + F.b), -1);
    for (int k = 0; k < 2; ++k) F.kcnt[k] = F.khead[k] = F.kschur[k] = F.kfwd[k] = 0;
    for (int k = 0; k < F.nc; ++k) {
      const int c = kids[f][k];
      const DsFront& O = P.fronts[id[c]];
      DsChild C;
      C.cnt = O.cnt;
      C.nhead = heads(O);
      C.nschur = schurs(O);
      C.nfwd = O.nfwd;
      C.nb = O.nb;
      C.g = O.g;
      C.so = O.so;
      C.q = 0;
      C.inv = (int)P.tab.size();
      P.tab.resize(P.tab.size() + F.p + F.b, -1);
      C.map = (int)P.tab.size();
      for (int u = 0; u < (int)border[c].size(); ++u) {
        const int l = local[border[c][u]];
        P.tab.push_back(l);
        P.tab[C.inv + l] = u;
        P.tab[F.gsrc + k * (F.p + F.b) + l] = O.g + 3 * u;
        if (l < F.p) ++C.q;
      }
      if (k < 2) {
        F.kcnt[k] = C.cnt;
        F.khead[k] = C.nhead;
        F.kschur[k] = C.nschur;
        F.kfwd[k] = C.nfwd;
      }
      P.kids.push_back(C);
    }
    for (int l = 0; l < F.p + F.b; ++l) local[P.tab[F.verts + l]] = -1;
  }
  // Homes: whole subtrees of at most a sixteenth of all work each (of a batch of equal
  // sheets: whole sheets), the largest first to the queue with the least; the tasks of the
  // fronts above them are dealt by rows. On eight 64x64 sheets this takes the reads that
  // miss the dies' caches from 2.9 to 2.0 GB a factorisation, and that from 64.4 to 62.3 ms
  // a forward and adjoint of 16 steps (200x200: 215 to 213, 64x64: 49.8 to 49.3). Small
  // plans, whose tasks are fewer than the workgroups, keep one queue: nothing is shared
  // often enough, and seven eighths of the workgroups would search for work.
  std::vector<double> work(nf);
  double total = 0.0;
  std::vector<int> up(nf, -1);
  for (int q = 0; q < nf; ++q) {
    const DsFront& F = P.fronts[q];
    if (parent[order[q]] >= 0) up[q] = id[parent[order[q]]];
    const double nbt = F.nb + kDsSchurTile, npt = F.np + 16;
    work[q] += npt * npt * npt + nbt * nbt * npt;   // children come first
    total += npt * npt * npt + nbt * nbt * npt;
    if (up[q] >= 0) work[up[q]] += work[q];
  }
  std::vector<int> home(nf, -1), cut;
  for (int q = 0; q < nf; ++q)
    if (up[q] < 0) cut.push_back(q);
  auto less = [&](int x, int y) { return work[x] != work[y] ? work[x] < work[y] : x < y; };
  const double share = cut.size() >= (size_t)kDsQueues ? 1.1 / kDsQueues : 0.5 / kDsQueues;
  std::make_heap(cut.begin(), cut.end(), less);
  while (!cut.empty() && work[cut[0]] > share * total && cut.size() < 64) {
    std::pop_heap(cut.begin(), cut.end(), less);
    const int q = cut.back();
    cut.pop_back();
    for (int k : kids[order[q]]) {
      cut.push_back(id[k]);
      std::push_heap(cut.begin(), cut.end(), less);
    }
  }
  std::sort(cut.begin(), cut.end(), [&](int x, int y) { return less(y, x); });
  double load[kDsQueues] = {};
  for (int q : cut) {
    const int h = (int)(std::min_element(load, load + kDsQueues) - load);
    home[q] = h;
    load[h] += work[q];
  }
  for (int q = nf - 1; q >= 0; --q)
    if (home[q] < 0 && up[q] >= 0) home[q] = home[up[q]];
  size_t ntasks = 0;
  for (const DsFront& F : P.fronts) ntasks += 1 + tiles(F.nb, kDsRowTile) + schurs(F);
  auto queue_of = [&](int kind, int q, int a) {
    if (ntasks < kDsOneQueue) return 0;
    if (home[q] >= 0) return home[q];
    int row = a;                                   // forward, backward
    if (kind == kDsPivot) row = q;
    if (kind == kDsBorder) row = a * kDsRowTile / kDsSchurTile;
    if (kind == kDsSchur) row = a >> 16;
    return row % kDsQueues;
  };
  // Tasks, level by level. A level's pivot blocks need only the head tiles of the level
  // below, so they come right after those: the pivot sweeps, the longest links of the
  // chain, then run beside the bulk of the Schur tiles.
  constexpr int HR = 2 * kDsSchurTile / kDsRowTile;   // row tiles of the head
  auto record = [&](std::vector<DsTask>& list, int kind, int q, int a) {
    list.emplace_back();
    DsTask& t = list.back();
    const DsFront& F = P.fronts[q];
    t = DsTask{};
    t.kind = kind;
    t.front = q;
    t.a = a;
    t.f = F;
    for (int k = 0; k < std::min(F.nc, 2); ++k) {
      const DsChild& C = P.kids[F.c0 + k];
      t.kid[k] = C;
      if (kind == kDsBackward) continue;
      const int* inv = P.tab.data() + C.inv;
      // the vertices of border rows [r0, r0 + n)
      auto rows_of = [&](short* out, int r0, int n) {
        const int v0 = r0 / 3, v1 = std::min(F.b, (r0 + n + 2) / 3);
        for (int v = v0; v < v0 + 24; ++v) out[v - v0] = v < v1 ? (short)inv[F.p + v] : -1;
      };
      if (kind == kDsBorder) rows_of(t.row[k], a * kDsRowTile, kDsRowTile);
      if (kind == kDsForward) rows_of(t.row[k], a * kDsFwdRows, kDsFwdRows);
      if (kind == kDsSchur) {
        rows_of(t.row[k], (a >> 16) * kDsSchurTile, kDsSchurTile);
        rows_of(t.col[k], (a & 0xffff) * kDsSchurTile, kDsSchurTile);
      }
      if (kind == kDsForward)
        for (int l = 0; l < F.p; ++l) t.col[k][l] = (short)inv[l];
      if (kind == kDsPivot || kind == kDsBorder)
        for (int u = 0; u < C.q; ++u) t.col[k][u] = (short)P.tab[C.map + u];
    }
    if (kind == kDsBorder) {
      t.lo = P.tab[F.blist + a] / 2;
      t.hi = P.tab[F.blist + a + 1] / 2;
    }
  };
  size_t nfac = 0, nsol = 0;
  for (const DsFront& F : P.fronts) {
    nsol += F.nfwd + tiles(F.np, kDsBwdCols);
    nfac += 1 + tiles(F.nb, kDsRowTile) + schurs(F);
  }
  P.solve_tasks.reserve(nsol);
  P.factor_tasks.reserve(nsol + nfac);
  auto push = [&](int kind, int q, int a) {
    record(P.factor_tasks, kind, q, a);
    P.factor_queue.push_back((unsigned char)queue_of(kind, q, a));
  };
  auto pivots = [&](int l) {
    for (int q = P.level0[l]; q < P.level0[l + 1]; ++q) push(kDsPivot, q, 0);
  };
  if (nlev > 0) pivots(0);
  for (int l = 0; l < nlev; ++l) {
    const int q0 = P.level0[l], q1 = P.level0[l + 1];
    for (int q = q0; q < q1; ++q)
      for (int r = 0; r < std::min(HR, tiles(P.fronts[q].nb, kDsRowTile)); ++r) push(kDsBorder, q, r);
    for (int q = q0; q < q1; ++q)
      for (int i = 0; i < std::min(2, tiles(P.fronts[q].nb, kDsSchurTile)); ++i)
        for (int j = 0; j <= i; ++j) push(kDsSchur, q, i << 16 | j);
    if (l + 1 < nlev) pivots(l + 1);
    for (int q = q0; q < q1; ++q)
      for (int r = HR; r < tiles(P.fronts[q].nb, kDsRowTile); ++r) push(kDsBorder, q, r);
    for (int q = q0; q < q1; ++q)
      for (int i = 2; i < tiles(P.fronts[q].nb, kDsSchurTile); ++i)
        for (int j = 0; j <= i; ++j) push(kDsSchur, q, i << 16 | j);
    for (int q = q0; q < q1; ++q)
      for (int r = 0; r < P.fronts[q].nfwd; ++r) {
        push(kDsForward, q, r);
        record(P.solve_tasks, kDsForward, q, r);
        P.solve_queue.push_back(P.factor_queue.back());
      }
  }
  for (int q = nf - 1; q >= 0; --q)
    for (int c = 0; c < tiles(P.fronts[q].np, kDsBwdCols); ++c) {
      push(kDsBackward, q, c);
      record(P.solve_tasks, kDsBackward, q, c);
      P.solve_queue.push_back(P.factor_queue.back());
    }
  P.res0.assign(1, 0);
  for (int b = 0; b < ninst; ++b) {
    for (int r = 0; r < inst_nv[b]; r += kDsResRows) P.res_tasks.push_back({b, inst_voff[b] + r});
    P.res0.push_back((int)P.res_tasks.size());
  }
  P.ok = P.tab.size() < (size_t)1 << 31 && P.work_doubles < 1LL << 40 &&
         9LL * maxnz * nv < 1LL << 31;
}

}  // namespace phisft
