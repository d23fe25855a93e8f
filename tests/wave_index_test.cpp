// Host test of the index of the one-cell-per-wave kernels into the pressure-dependent
// records (rkc_wave_index.h): for every lane and round of every compiled form, and
// mechanisms whose unit counts sit at, just below and just past the rounds of the
// lane-group plan, no lane reads outside the records, every pressure-dependent unit
// finds its own, and no other unit's.  Prints "OK" and exits 0 on success.
#include <algorithm>
#include <cstdio>

#include "rkc_wave_index.h"

struct Form { int SG, RUC, NW; };
static const Form forms[] = {{16, 1, 1}, {32, 5, 1}, {64, 4, 4}};

int main() {
    long lanes = 0;
    for (const Form &f : forms) {
        const int LANES = 64 * f.NW;
        for (int nU = 1; nU <= f.RUC * LANES; ++nU) {
            const int RU = (nU + f.SG - 1) / f.SG;
            for (int n_plain : {0, 1, nU / 3, nU / 2, nU - 1, nU - f.SG, RU * f.SG - f.SG}) {
                if (n_plain < 0 || n_plain >= nU) continue;
                const int RUp = n_plain / f.SG, NPR = RU - RUp;
                const int pd0 = RUp * f.SG, RUpw = n_plain / LANES;
                for (int r = 0; r < f.RUC; ++r)
                    for (int l = 0; l < LANES; ++l, ++lanes) {
                        const int unit = r * LANES + l;
                        const int place =
                            r >= RUpw ? rkcdev::pdep_place(unit, pd0, nU - pd0) : -1;
                        const bool pd = unit >= n_plain && unit < nU;
                        bool ok = !pd || place == unit - pd0;
                        if (place >= 0)
                            for (int q = 0; q < 6; ++q) {
                                const int at = rkcdev::pdep_piece(place, q, f.SG);
                                ok = ok && at >= 0 && at < NPR * f.SG * 6;
                            }
                        ok = ok && (place < 0 || unit < nU);
                        if (!ok) {
                            std::printf("FAIL %d lanes, %d units (%d plain), unit slot %d: record "
                                        "%d of %d\n", f.SG, nU, n_plain, unit, place, NPR * f.SG);
                            return 1;
                        }
                    }
            }
        }
    }
    std::printf("%ld lanes\nOK\n", lanes);
    return 0;
}
