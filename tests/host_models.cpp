// The cell models of a target with SIP, made on the host from the same
// templates as the device's.
#include "cell_model.hpp"
#include "plan.hpp"

using namespace dfr;

// any != 0: the instance of any order, else the one for orders up to 5.
extern "C" int host_cell_model(const dfr_wcs *sw, const dfr_wcs *tw, int any, int cx, int cy,
                               double mx[10], double my[10], int base[2], double range[2],
                               double *bound, double *tie) {
  FramePlan P;
  build_plan(nullptr, 0, 0, 0, *sw, *tw, (cy + 1) * kCell, (cx + 1) * kCell, nullptr, nullptr, P);
  const SipCoefs C{P.sA, P.sB, P.tA, P.tB};
  CellModel M;
  if (any)
    cell_model<-1, kMaxOrder>(P, C, cx, cy, M);
  else
    cell_model<5, 5>(P, C, cx, cy, M);
  for (int k = 0; k < 10; ++k) {
    mx[k] = M.mx[k];
    my[k] = M.my[k];
  }
  base[0] = M.bx;
  base[1] = M.by;
  range[0] = M.ex;
  range[1] = M.ey;
  *bound = M.err;
  *tie = M.tie;
  return M.certified;
}
