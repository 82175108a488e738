// The tile plan of the resident time loop.
#include "emm_resident_plan.h"

#include <algorithm>

namespace emm {

ResidentPlan resident_plan(int r, int n1, int n2, int n3, int cus) {
    ResidentPlan best;
    const int L = 2 * r, nx = n1 - L, ny = n2 - L, nz = n3 - L;
    if (r > 3 || nx <= 0 || ny <= 0 || nz <= 0) return best;
    double cost = -1;
    for (int gz = 1; gz <= std::min(nz, cus); ++gz) {
        const int tz = (nz + gz - 1) / gz;
        if (gz > 1 && nz / gz < r) break;
        for (int gy = 1; gy * gz <= cus && gy <= ny; ++gy) {
            const int ty = (ny + gy - 1) / gy;
            if (gy > 1 && ny / gy < r) break;
            if (tz > kResTall || (tz + L - 1) * (ty + L - 1) * n1 > kResSlot) continue;
            const int waves = (nx * ty + 63) / 64;
            for (int planes = 1; planes <= kResPlanes; ++planes) {
                const int groups = (tz + planes - 1) / planes;
                if (64 * waves * groups > resident_threads(planes)) continue;
                const int words = (2 * (L - 1) * (ty + tz) * nx + 64 * waves * groups - 1) / (64 * waves * groups);
                if (words > resident_words(planes)) continue;
                // clocks of a half step beyond some 3800 that every plan
                // takes (measured: 6300 with 12 wavefronts of one plane and
                // 2100 words, 9100 with 8 of three and 4020; five planes
                // spill a little)
                const double c = 0.6 * (2 * (L - 1) * (ty + tz) * nx) + (planes == 5 ? 170.0 : 130.0) * planes * waves * groups;
                if (cost >= 0 && c >= cost) continue;
                ResidentPlan p;
                p.gy = gy;
                p.gz = gz;
                p.ty = ty;
                p.tz = tz;
                p.planes = planes;
                p.groups = groups;
                p.threads = 64 * waves * groups;
                if (resident_reach(r, n1, p) >= 6l * kResSlot) continue;
                cost = c;
                best = p;
            }
        }
    }
    return best;
}

}  // namespace emm
