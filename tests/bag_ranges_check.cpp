// Host check of the range arithmetic behind the bags of the positions (csrc/sfc_device.h), as the kernel
// uses it: 64 bags at a time; where none of them is malformed, all positions between the first start and
// the last end at once, else bag by bag.  Input: n, n_bags, n_bags + 1 offsets, repeated.  Prints for each case the
// violations counted and, where every position that the plain 64-bit loop writes was written and no
// other, "ok".
#include <cstdio>
#include <vector>
#include "../paper_2104_08542_amd/csrc/sfc_device.h"

int main() {
  int n, nb;
  while (scanf("%d %d", &n, &nb) == 2) {
    std::vector<long long> off(nb + 1);
    for (long long& x : off) if (scanf("%lld", &x) != 1) return 1;
    std::vector<char> want(n, 0), got(n, 0);
    for (int b = 0; b < nb; ++b)
      for (long long q = off[b] < 0 ? 0 : off[b]; q < off[b + 1] && q < n; ++q) want[q] = 1;
    int bad = 0;
    bool inside = true;
    for (int b0 = 0; b0 < nb; b0 += sfc::kWave) {
      const int last = nb - b0 < sfc::kWave ? nb - b0 - 1 : sfc::kWave - 1;
      int here = 0;
      for (int l = 0; l <= last; ++l) here += sfc::bag_malformed(off[b0 + l], off[b0 + l + 1], b0 + l, nb, n);
      bad += here;
      for (int l = 0; l <= last; ++l) {
        const sfc::BagRange r = here ? sfc::bag_range(off[b0 + l], off[b0 + l + 1], n)
                                     : sfc::BagRange{sfc::bag_range(off[b0], off[b0 + 1], n).lo,
                                                     sfc::bag_range(off[b0 + last], off[b0 + last + 1], n).hi};
        if (r.lo < 0 || r.lo > n || r.hi < 0 || r.hi > n) { inside = false; break; }
        for (int q = r.lo; q < r.hi; ++q) got[q] = 1;
      }
    }
    printf("%d %s\n", bad, !inside ? "outside" : got == want ? "ok" : "differs");
  }
  return 0;
}
