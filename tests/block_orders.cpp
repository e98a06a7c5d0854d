// Enumerates the block orders of csrc/schedule.h over even extents and prints
// "x y z t mode H what" for every launch whose blocks do not do what the
// operator kernels assume, then the number of launches looked at and of faults:
//   cover   a half site computed by no block, by two, or one that does not exist
//   rows    a row of partial sums written by no block or by two, or out of range
//   plane   (forms that stage rows in LDS) a block that starts within an x row,
//           is not whole, or reaches into another (z, t) plane
#include <algorithm>
#include <cstdio>
#include <utility>
#include <vector>

#include "schedule.h"

using namespace qcd;

int main() {
  const int t_extents[] = {2, 8};
  const int max_lxh = 64;  // the longest x rows of any LDS form
  long looked = 0, faults = 0;
  std::vector<std::pair<int, int>> seen;
  std::vector<int> rows;
  for (int x = 2; x <= 48; x += 2)
    for (int y = 2; y <= 48; y += 2)
      for (int z = 2; z <= 48; z += 2)
        for (int t : t_extents)
          for (int eo = 0; eo < 2; eo++)
            for (int mode = 0; mode <= 4; mode++) {
              const int lxh = x / 2, plane = lxh * y;
              for (int T : {1, 4}) {
                if (T > 1 && t > 2) continue;
                const int n = z % 4 ? T : 2 * T;  // one tile of right-hand sides, or two
                const DslashSched sc = make_sched(lxh, y, z, t, mode, T, n, eo);
                const bool lds = T == 1 && n == 1 && lds_rows_apply(lxh, y, sc.H, max_lxh);
                bool cover = true, row = true, flat = true;
                for (int tile = 0; tile < sc.ntiles; tile++) {
                  seen.clear();
                  rows.assign(sc.nsb, 0);
                  for (int b = 0; b < sc.grid; b++) {
                    const BlockPos p = block_pos(sc, b);
                    if (p.tile < 0 || p.tile >= sc.ntiles) row = false;
                    if (p.tile != tile || p.cnt < 0) continue;
                    if (p.sb < 0 || p.sb >= sc.nsb) row = false;
                    else rows[p.sb]++;
                    if (p.cnt > sc.H) cover = false;
                    if (p.cnt == 0) continue;
                    seen.push_back({p.h0, p.cnt});
                    if (p.cnt != sc.H || p.h0 % lxh || p.h0 % plane + sc.H > plane) flat = false;
                  }
                  std::sort(seen.begin(), seen.end());
                  int next = 0;
                  for (auto& s : seen) {
                    if (s.first != next) cover = false;
                    next = s.first + s.second;
                  }
                  if (next != sc.Vh || sc.Vh != plane * z * t) cover = false;
                  for (int r : rows)
                    if (r != 1) row = false;
                }
                looked++;
                const char* what = !cover ? "cover" : (!row ? "rows" : (lds && !flat ? "plane" : nullptr));
                if (what && faults++ < 40) std::printf("%d %d %d %d %d %d %s\n", x, y, z, t, mode, sc.H, what);
              }
            }
  std::printf("%ld launches, %ld faults\n", looked, faults);
  return faults != 0;
}
