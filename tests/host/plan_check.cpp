// Shape of the direct solver's elimination tree.
#include <cstddef>

#include "direct.h"

using namespace phisft;

// Largest number of children of a front, and the number of fronts with more than two.
extern "C" int plan_children(int nv, int maxnz, const int* ell_col, const double* xr, int* more) {
  DsPlan P;
  build_direct_plan(nv, maxnz, std::vector<int>(ell_col, ell_col + (size_t)maxnz * nv), {0}, {nv},
                    std::vector<double>(xr, xr + 3 * (size_t)nv), P);
  int most = P.ok ? 0 : -1;
  *more = 0;
  for (const DsFront& F : P.fronts) {
    most = F.nc > most ? F.nc : most;
    *more += F.nc > 2;
  }
  return most;
}
