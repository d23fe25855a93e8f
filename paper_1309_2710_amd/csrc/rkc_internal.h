// Internal declarations shared by the host runtime and the kernel variants.
#pragma once

#include <hip/hip_runtime.h>

#include "rkc.h"
#include "rkc_device.h"

namespace rkchost {

// One compiled kernel variant: G lanes per cell, NSL state elements per lane,
// RUC reaction units per lane held in registers (0: parameters read from LDS,
// -1: from global memory, any number of units).
struct VariantDesc {
    int G, NSL, RUC;
    int max_threads;
    const void *k_rkc;
    const void *k_rkck;
    const void *k_rhs;
    // the same kernels with the third-body/falloff rounds (null: not built)
    const void *k_rkc_pd;
    const void *k_rkck_pd;
    const void *k_rhs_pd;
    // the source term by a grid that walks over the cells, and the one that classes
    // them by cost (null: one lane per cell)
    const void *k_walk, *k_class;
    const void *k_walk_pd, *k_class_pd;
};

const VariantDesc *variants_g64(int *n);
const VariantDesc *variants_g32(int *n);
const VariantDesc *variants_g16(int *n);
const VariantDesc *variants_g8(int *n);
// one lane per cell (G = 1, NSL = the state capacity NMAX of the kernel)
const VariantDesc *variants_lane(int *n);

// One compiled one-cell-per-wave form (rkc_wave.h) of the variant with SG lanes
// per cell and NSL state elements per lane: NW waves per cell, at most RUC unit
// rounds of 64 NW lanes with their parameters placed as UL says, MS gather
// segments of at most SL terms, LP positive and LN negative pieces per state
// slot, occ waves per SIMD; for plain or pressure-dependent mechanisms; used for
// up to `fill` cells per resident one (0: any number).
struct WaveDesc {
    int SG, NSL, RUC, UL, NW, MS, SL, LP, LN, occ;
    bool pd;
    double fill;
    const void *k_rkc, *k_rkck;
    const void *k_rkc_tail, *k_rkck_tail;   // for cells handed over by lane groups, or null
};
const WaveDesc *wave_variants(int *n);

// 8-byte words of a launch's aggregate counters.
constexpr int AGG_N = rkcdev::AGG_USED * rkcdev::AGG_STRIDE;

// What one integrator launch ran (for rkc_stats).
struct LaunchInfo {
    int G = 0, RUC = 0, blocks = 0, threads = 0;
    bool persistent = false;
    size_t lds = 0;
};

}  // namespace rkchost


namespace rkchost {

// Validate the scalar arguments and options of an integration.
int check_integrate_args(double dt, double rtol, double atol, const rkc_opts &o);

// Scratch of a cost-ordered work queue: 6 bytes per cell and 16 KB, grown to
// the largest launch (at most 2^22 cells are ordered) and kept by its owner;
// and the records of cells handed over to the wave form (512 bytes per resident
// wave, 1.5 MB).
struct OrderScratch {
    int *order = nullptr;
    uint16_t *key = nullptr;
    unsigned *hist = nullptr;
    size_t cap = 0;
    double *tail = nullptr;
    size_t tail_cap = 0;
};
void free_order(OrderScratch *s);
bool reserve_tail(OrderScratch *s, size_t cells, bool may_build);
// Room for n cells; false if there is none and none may be or could be allocated.
bool reserve_order(OrderScratch *s, size_t n, bool may_build);

// Enqueue one integration of n cells whose arrays are device pointers on the
// mechanism's device, with the launch's own scratch (aggregate counters
// [AGG_N], work-queue head): launches that use distinct scratch may run
// concurrently on different streams.  Not thread-safe for one mechanism
// (its per-shape table cache is filled on first use).  With may_build false
// nothing is allocated: RKC_ENOTSUP if the tables of the selected variant
// have not been built by an earlier call.  With `ord` the queue is ordered by
// expected cost (not shared by launches that run concurrently).
int enqueue_integrate(rkc_mech *m, size_t n, double *Td, const double *Pd, double *Yd, double dt,
                      double rtol, double atol, const rkc_opts &o, int32_t *sd, int32_t *cd,
                      unsigned long long *agg_d, int *queue_d, hipStream_t st, LaunchInfo *li,
                      bool may_build = true, OrderScratch *ord = nullptr);

// Select the variant and build the device tables a later enqueue_integrate
// with these options will use (so that concurrent launches only read them);
// with n_cells > 0 also fix the launch attributes of that launch's kernels and,
// with `ord`, reserve the scratch it uses.
int prepare(rkc_mech *m, const rkc_opts &o, size_t n_cells, double atol = 0.0,
            OrderScratch *ord = nullptr);
int mech_species(const rkc_mech *m);
int mech_device(const rkc_mech *m);

// Statistics of one launch from its aggregate counters ([AGG_N], see the kernels).
void fill_stats(const unsigned long long *agg, const LaunchInfo &li, rkc_stats *stats);

}  // namespace rkchost

#define RKC_FN(...) reinterpret_cast<const void *>(&rkcdev::__VA_ARGS__)

// A variant with plain-reaction kernels only (register-resident parameters).
#define RKC_VARIANT(G_, NSL_, RUC_)                                                            \
    rkchost::VariantDesc {                                                                     \
        G_, NSL_, RUC_, (rkcdev::Occ<RUC_, NSL_>::threads),                                    \
            RKC_FN(rkc_kernel<G_, NSL_, RUC_, false>),                                         \
            RKC_FN(rkck_kernel<G_, NSL_, RUC_, false>),                                        \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, false, rkcdev::RHS_ONCE>),                       \
            nullptr, nullptr, nullptr,                                                         \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, false, rkcdev::RHS_WALK>),                       \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, false, rkcdev::RHS_CLASS>),                      \
            nullptr, nullptr                                                                   \
    }

// Plain and pressure-dependent kernels.
#define RKC_VARIANT_BOTH(G_, NSL_, RUC_)                                                       \
    rkchost::VariantDesc {                                                                     \
        G_, NSL_, RUC_, (rkcdev::Occ<RUC_, NSL_>::threads),                                    \
            RKC_FN(rkc_kernel<G_, NSL_, RUC_, false>),                                         \
            RKC_FN(rkck_kernel<G_, NSL_, RUC_, false>),                                        \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, false, rkcdev::RHS_ONCE>),                       \
            RKC_FN(rkc_kernel<G_, NSL_, RUC_, true>),                                          \
            RKC_FN(rkck_kernel<G_, NSL_, RUC_, true>),                                         \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, true, rkcdev::RHS_ONCE>),                        \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, false, rkcdev::RHS_WALK>),                       \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, false, rkcdev::RHS_CLASS>),                      \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, true, rkcdev::RHS_WALK>),                        \
            RKC_FN(rhs_kernel<G_, NSL_, RUC_, true, rkcdev::RHS_CLASS>)                        \
    }
// ... with the parameters in LDS, and with them and the species table in global memory.
#define RKC_VARIANT_PD(G_, NSL_) RKC_VARIANT_BOTH(G_, NSL_, 0)
#define RKC_VARIANT_PD_GLOBAL(G_, NSL_) RKC_VARIANT_BOTH(G_, NSL_, -1)
