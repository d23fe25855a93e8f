// One-cell-per-wave kernel forms (rkc_wave.h), with plain reactions (RKC_WAVE)
// or pressure-dependent ones (RKC_WAVE_PD) of the variants that the automatic
// choice gives those mechanisms.
#include "rkc_internal.h"
#include "rkc_wave.h"

#define RKC_WAVE_K(K_, PD_, ...)                                                                     \
    reinterpret_cast<const void *>(&rkcdev::K_##_wave_kernel<__VA_ARGS__, PD_>)

#define RKC_WAVE(FILL_, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_)                         \
    rkchost::WaveDesc {                                                                              \
        SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, OCC_, false, FILL_,                           \
            RKC_WAVE_K(rkc, false, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_),             \
            RKC_WAVE_K(rkck, false, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_)             \
    }
#define RKC_WAVE_PD(FILL_, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_)                      \
    rkchost::WaveDesc {                                                                              \
        SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, OCC_, true, FILL_,                            \
            RKC_WAVE_K(rkc, true, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_),              \
            RKC_WAVE_K(rkck, true, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_)              \
    }

namespace rkchost {

// In order of preference: the first that fits the mechanism and the cell count
// runs.  fill: the most cells per resident one (0: any number).
static const WaveDesc kTable[] = {
    RKC_WAVE(2.0, 3, 16, 1, 1, rkcdev::UNITS_REG, 1, 1, 8, 4, 2),
    RKC_WAVE(2.0, 3, 16, 1, 1, rkcdev::UNITS_REG, 1, 1, 8, 4, 4),
    RKC_WAVE_PD(2.0, 3, 16, 1, 1, rkcdev::UNITS_REG, 1, 1, 8, 4, 4),
    RKC_WAVE(1.125, 2, 64, 1, 3, rkcdev::UNITS_REG, 2, 2, 6, 8, 4),
    RKC_WAVE(0.0, 2, 64, 1, 5, rkcdev::UNITS_REG, 1, 4, 6, 8, 4),
    RKC_WAVE(0.0, 2, 64, 1, 5, rkcdev::UNITS_REG, 1, 3, 10, 8, 4),
    RKC_WAVE_PD(4.0, 2, 32, 2, 5, rkcdev::UNITS_LDS, 1, 3, 12, 6, 2),
    RKC_WAVE(1.0, 2, 64, 2, 2, rkcdev::UNITS_GLOBAL, 8, 1, 10, 6, 4),
    RKC_WAVE(16.0, 2, 64, 2, 4, rkcdev::UNITS_REG, 4, 2, 10, 6, 4),
    RKC_WAVE_PD(8.0, 2, 64, 2, 4, rkcdev::UNITS_GLOBAL, 4, 2, 10, 6, 4),
};

const WaveDesc *wave_variants(int *n) {
    *n = (int)(sizeof(kTable) / sizeof(kTable[0]));
    return kTable;
}

}  // namespace rkchost
