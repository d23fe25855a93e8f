// One-cell-per-wave kernel forms (rkc_wave.h), with plain reactions (RKC_WAVE)
// or pressure-dependent ones (RKC_WAVE_PD) of the variants that the automatic
// choice gives those mechanisms.
#include "rkc_internal.h"
#include "rkc_wave.h"

// A form's lanes per cell of the plan, once its LDS fits whatever the mechanism: all
// its unit rounds pressure-dependent, with the most efficiency sets.  So no mechanism
// that the host gives to a form is refused for LDS (the largest, 111 species with
// falloff, takes 155,840 of 163,840 bytes).
template <int SG, int NSL, int RUC, int UL, int NW, int MS, bool PD>
constexpr int fits_lds() {
    constexpr rkcdev::WaveShape sh{SG * NSL, 64 * NW, RUC, MS, PD ? RUC * 64 * NW / SG : 0,
                                   PD ? rkcdev::MAX_EFFSETS : 0, SG, UL};
    static_assert(rkcdev::wave_lds_bytes(sh, 1) <= 160 * 1024, "a form's workgroup exceeds LDS");
    return SG;
}

#define RKC_WAVE_K(K_, ...)                                                                          \
    reinterpret_cast<const void *>(&rkcdev::K_##_wave_kernel<__VA_ARGS__>)

#define RKC_WAVE(FILL_, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_)                         \
    rkchost::WaveDesc {                                                                              \
        fits_lds<SG_, NSL_, RUC_, UL_, NW_, MS_, false>(), NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, \
            OCC_, false, FILL_,                                                                      \
            RKC_WAVE_K(rkc, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, false),             \
            RKC_WAVE_K(rkck, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, false),            \
            nullptr, nullptr                                                                         \
    }
#define RKC_WAVE_PD(FILL_, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_)                      \
    rkchost::WaveDesc {                                                                              \
        fits_lds<SG_, NSL_, RUC_, UL_, NW_, MS_, true>(), NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_,  \
            OCC_, true, FILL_,                                                                       \
            RKC_WAVE_K(rkc, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, true),              \
            RKC_WAVE_K(rkck, OCC_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, true),             \
            nullptr, nullptr                                                                         \
    }
// also with the kernels that finish the cells handed over by 16-lane groups
#define RKC_WAVE_T(FILL_, PD_, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_)                        \
    rkchost::WaveDesc {                                                                              \
        fits_lds<SG_, NSL_, RUC_, UL_, NW_, MS_, PD_>(), NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_,   \
            3, PD_, FILL_,                                                                           \
            RKC_WAVE_K(rkc, 3, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, PD_),                  \
            RKC_WAVE_K(rkck, 3, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, PD_),                 \
            RKC_WAVE_K(rkc, 3, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, PD_, true),            \
            RKC_WAVE_K(rkck, 3, SG_, NSL_, RUC_, UL_, NW_, MS_, SL_, LP_, LN_, PD_, true)            \
    }

namespace rkchost {

// In order of preference: the first that fits the mechanism and the cell count
// runs.  fill: the most cells per resident one (0: any number).
static const WaveDesc kTable[] = {
    RKC_WAVE_T(4.0, false, 16, 1, 1, rkcdev::UNITS_REG, 1, 1, 8, 4, 2),
    RKC_WAVE_T(4.0, false, 16, 1, 1, rkcdev::UNITS_REG, 1, 1, 8, 4, 4),
    RKC_WAVE_T(4.0, true, 16, 1, 1, rkcdev::UNITS_REG, 1, 1, 8, 4, 4),
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
