// Coils per workgroup of the fused plane kernels (host code without HIP).
//
// The time of a launch is about its rounds over the compute units (one workgroup each: the
// kernels' LDS takes all of a unit's) times the coils of a group, plus half a coil's worth of
// set-up per workgroup.  Halving from 16 until every compute unit had a workgroup took 2 coils in
// 2 rounds where 3 fit one (64 planes, 12 coils).  The adjoint's groups each write a gx partial: no
// more of them than the halving rule gives, and the fewest at equal cost.
#pragma once

#include <algorithm>
#include <cstdint>

namespace mx {

struct PlaneGroups {
  int fwd, adj;
};

inline PlaneGroups plane_groups(int64_t planes, int J, int cus) {
  auto groups = [&](int G) { return (J + G - 1) / G; };
  int halved = 16;
  while (halved > 1 && planes * groups(halved) < cus) halved /= 2;
  auto pick = [&](int max_groups) {
    int best = halved;
    double cost = 0.0;
    for (int G = std::min(16, J); G >= 1; --G) {
      if (groups(G) > max_groups || groups(G) * (int64_t)G - J >= G) continue;
      const double c = (double)((planes * groups(G) + cus - 1) / cus) * (G + 0.5);
      if (cost == 0.0 || c < cost) {
        cost = c;
        best = G;
      }
    }
    return best;
  };
  return {pick(J), pick(groups(halved))};
}

}  // namespace mx
