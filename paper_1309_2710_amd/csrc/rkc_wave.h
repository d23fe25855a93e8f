// One cell per wave (or per workgroup of NW waves): the integrators for launches
// with too few cells to fill the chip, where a call lasts as long as its longest
// cell's chain of source-term evaluations.
//
// The arithmetic is that of the lane-group kernels (rkc_integrate.h) for G = SG
// lanes and NSL state slots per lane, operation by operation, so a cell's
// result does not depend on which of the two forms ran.  What differs is where
// the work is done and what is kept where:
//   - state element k = s SG + g is held by every lane with lane % SG = g, so
//     the group reductions are those of the lane-group kernel;
//   - reaction unit p is evaluated by lane p % (64 NW) of the cell's lanes and
//     gather chunk c is summed by lane c % (64 NW): fewer rounds than SG lanes
//     need, the same values in the same Q and piece slots;
//   - a lane's share of the mechanism (reaction parameters, LDS addresses of
//     reactant slots and gather terms, molar masses) stays in registers;
//   - the control state is wave-uniform, so phases are scalar branches and
//     scalars are not kept in LDS; the next stage's coefficients are loaded one
//     evaluation ahead.
// With NW > 1 every wave of the workgroup holds the whole state and takes the
// same decisions from the same values; the waves exchange only net rates and
// gather pieces, through LDS, with three barriers per evaluation.
//
// What bounds it.  A wave issues one instruction in about 5 cycles whatever its
// kind, and dependent FP64 FMAs issue back to back, so a lone cell's time is
// its instruction count plus the waits for LDS (64 cycles and up, five exchanges
// an evaluation).  Hence addresses, constants and table entries in registers,
// one exchange for two sums, loads issued under the exponentials, and scalar
// branches.  Per evaluation of the longest cell, alone on its SIMD, against the
// lane-group kernels: 9 species 0.83 us against 3.3 (239 vector instructions),
// 13 species 0.88 / 2.3, 53 species 1.5 / 4.1 (two waves a cell 1.3), 111 species
// 1.8 / 5.1 (four waves a cell).  At two waves per SIMD (255 registers, 460
// vector instructions per evaluation against 561) 131,072 cells of the
// 53-species set take 127 ms against 143 with four waves of the lane-group
// kernel: fewer instructions outweigh the lower occupancy.  There the FP64 pipe
// is 73 % busy and LDS about as much; parameters in LDS and three waves
// (168 registers) spilled, 38 ms against 33 for 32,768 cells.
#pragma once

#include "rkc_integrate.h"
#include "rkc_wave_index.h"

namespace rkcdev {

typedef __attribute__((address_space(3))) double lds_double;

__device__ __forceinline__ uint32_t lds_addr(const void *p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
// An address as a register of its own: otherwise the compiler keeps base and
// offset apart and adds them at every read, 69 of the 427 vector instructions of
// an evaluation of 53 species.
__device__ __forceinline__ uint32_t opaque_vu(uint32_t a) {
    asm("" : "+v"(a));
    return a;
}
__device__ __forceinline__ double lds_at(uint32_t a) { return *(const lds_double *)(uintptr_t)a; }

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ bool any(bool c) { return __builtin_amdgcn_ballot_w64(c) != 0ull; }
__device__ __forceinline__ bool rare(bool c) { return __builtin_expect(c, 0); }

// Sums over the state lanes, the additions of gsum<SG> and gsum2<SG>.  Every
// lane receives the result: with SG = 16 the rows hold copies of the state and
// each row's four exchanges end with the sum in all its lanes.
template <int SG>
__device__ __forceinline__ double usum(double x) {
    x += dpp_f64<DPP_XOR1>(x);
    x += dpp_f64<DPP_XOR2>(x);
    x += dpp_f64<DPP_HALF_MIRROR>(x);
    if constexpr (SG >= 16) x += dpp_f64<DPP_MIRROR>(x);
    if constexpr (SG >= 32) x += dpp_f64<DPP_BCAST15>(x);
    if constexpr (SG == 64) x += dpp_f64<DPP_BCAST31>(x);
    if constexpr (SG >= 32) x = readlane_f64(x, SG - 1);
    return x;
}

// Maximum over the state lanes (exact in any order).
template <int SG>
__device__ __forceinline__ double umax(double x) {
    x = fmax(x, dpp_f64<DPP_XOR1>(x));
    x = fmax(x, dpp_f64<DPP_XOR2>(x));
    x = fmax(x, dpp_f64<DPP_HALF_MIRROR>(x));
    if constexpr (SG >= 16) x = fmax(x, dpp_f64<DPP_MIRROR>(x));
    if constexpr (SG >= 32) x = fmax(x, dpp_f64<DPP_BCAST15>(x));
    if constexpr (SG == 64) x = fmax(x, dpp_f64<DPP_BCAST31>(x));
    if constexpr (SG >= 32) x = readlane_f64(x, SG - 1);
    return x;
}

// Two sums: the copies of the state in the upper half of the wave form the
// second while the lower half forms the first.
template <int SG>
__device__ __forceinline__ void usum2(double &a, double &b) {
    if constexpr (SG == 64) {
        gsum2<64>(a, b);
    } else {
        double x = (__lane_id() < 32) ? a : b;
        x += dpp_f64<DPP_XOR1>(x);
        x += dpp_f64<DPP_XOR2>(x);
        x += dpp_f64<DPP_HALF_MIRROR>(x);
        if constexpr (SG >= 16) x += dpp_f64<DPP_MIRROR>(x);
        if constexpr (SG >= 32) x += dpp_f64<DPP_BCAST15>(x);
        a = readlane_f64(x, 31);
        b = readlane_f64(x, 63);
    }
}

// Waits of the LDS exchange between the cell's lanes.
template <int NW>
__device__ __forceinline__ void cell_sync() {
    if constexpr (NW == 1) wave_sync();
    else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
}

// Where a wave's reaction parameters are kept.
enum { UNITS_REG = 0, UNITS_LDS = 1, UNITS_GLOBAL = 2 };

// A lane's share of the mechanism.  RUC unit rounds, MS gather segments of SL
// terms, LP positive and LN negative pieces per state slot.
template <int NSL, int RUC, int UL, int MS, int SL, int LP, int LN>
struct WaveTab {
    static constexpr int RP = UL != UNITS_REG ? 1 : RUC;
    double l2Af[RP], bf[RP], tf[RP], l2Ar[RP], br[RP], tr[RP];
    uint32_t sf[RUC][3], sr[RUC][3];     // LDS addresses of the reactant slots
    uint32_t gt[MS][SL];                 // of the gather terms
    uint32_t gp[NSL][LP], gn[NSL][LN];   // of the pieces
    uint32_t qst, pst;                   // where the lane stores its first rate and piece
    uint32_t cst[NSL];                   // its concentrations (lanes without one: a spare slot)
    double W[NSL], invW[NSL], tmid[NSL];
    double invTmax;
};

// What a wave keeps in LDS between its cells: their totals, and the Chebyshev
// recurrences of a step whose stage count is not tabulated.
struct WaveState {
    double w0, w1, Tm1, Tm2, Tpm1, Tpm2, Tppm1, Tppm2, bm1, ibm1, ibm2;
    double t, sigma, h_prev, rprev, t_end, h_min, rtol, atol, invN;
    Agg agg;
    int slot;
};

// LDS of one workgroup: per cell C [NK] and a spare slot, Q [RUC lanes + 2], piece [MS
// lanes + 2], [M] of the efficiency sets; then the tables shared by its cells: species
// records, mu~_1 of the tabulated stage counts, pressure-dependent records and
// efficiency sets in the lane-group layout.
struct WaveShape {
    int NK, lanes, RUC, MS, NPR, NMS, SG;
    int UL;
};
constexpr int MUT_N = 130;
constexpr int WAVE_STATE = 32;   // doubles of a wave's WaveState
static_assert(sizeof(WaveState) <= 8 * WAVE_STATE, "wave state exceeds its LDS slot");
__host__ __device__ inline int wave_segments(int NSEG, int SG, int lanes) {
    return (NSEG * SG + lanes - 1) / lanes;
}
__host__ __device__ constexpr size_t wave_cell_doubles(const WaveShape &s) {
    return (size_t)s.NK + 2 + (size_t)s.RUC * s.lanes + 2 + (size_t)s.MS * s.lanes + 2 +
           (size_t)((s.NMS + 1) & ~1) + (size_t)WAVE_STATE * (s.lanes / 64);
}
__host__ __device__ constexpr size_t wave_lds_bytes(const WaveShape &s, int cells) {
    return 8 * ((size_t)cells * wave_cell_doubles(s) + (size_t)NFIELD * s.NK + MUT_N +
                (size_t)s.NPR * s.SG * PDEP_DOUBLES + (size_t)s.NMS * s.NK +
                (s.UL == UNITS_LDS ? (size_t)6 * s.RUC * s.lanes : 0));
}

struct WaveLds {
    const double *spec, *mut1, *pdep, *eff;
    const double2 *units;   // UL: the lane's first record, [round][3][lanes]
    double *C, *Q, *piece, *Mv;
    WaveState *state, *state0;   // the wave's own; the one of the cell's first wave
};

template <int SG, int NSL, int RUC, int UL, int NW, int MS, int SL, int LP, int LN>
__device__ __forceinline__ void wave_setup(const Params &p, unsigned char *lds_raw, WaveLds &L,
                                           WaveTab<NSL, RUC, UL, MS, SL, LP, LN> &w) {
    constexpr int LANES = 64 * NW, NK = SG * NSL;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int cells = nt / LANES, cib = tid / LANES, l = tid % LANES, g = tid % SG;
    const WaveShape sh{NK, LANES, RUC, MS, p.NPR, p.NMS, SG, UL};
    double *base = reinterpret_cast<double *>(lds_raw);
    double *c0 = base + (size_t)cib * wave_cell_doubles(sh);
    L.C = c0;
    L.Q = L.C + NK + 2;
    L.piece = L.Q + RUC * LANES + 2;
    L.Mv = L.piece + MS * LANES + 2;
    L.state0 = reinterpret_cast<WaveState *>(L.Mv + ((p.NMS + 1) & ~1));
    L.state = reinterpret_cast<WaveState *>(L.Mv + ((p.NMS + 1) & ~1) + WAVE_STATE * (l / 64));
    if (l == 0) L.state->agg = Agg{0, 0, 0, 0, 0, 0, 0, 0};
    double *spec = base + (size_t)cells * wave_cell_doubles(sh);
    double *mut = spec + NFIELD * NK;
    double *ul = mut + MUT_N;
    double *pd = ul + (UL == UNITS_LDS ? 6 * RUC * LANES : 0);
    double *ef = pd + (size_t)p.NPR * SG * PDEP_DOUBLES;
    L.spec = spec; L.mut1 = mut; L.pdep = pd; L.eff = ef;
    if constexpr (UL == UNITS_GLOBAL)
        // the 64-lane records, whose round 64 NW / 64 r + l / 64 is round r here
        L.units = reinterpret_cast<const double2 *>(p.tab.units_il) + (l / 64) * 256 + l % 64;
    else
        L.units = reinterpret_cast<const double2 *>(ul) + l;
    for (int i = tid; i < NFIELD * NK; i += nt) spec[i] = p.tab.spec[i];
    for (int s = tid; s < MUT_N; s += nt)
        mut[s] = (s >= 2 && s <= p.coef_smax) ? p.coef[4 * coef_offset(s)] : 0.0;
    for (int i = tid; i < p.NPR * SG * PDEP_DOUBLES; i += nt) pd[i] = p.tab.pdep[i];
    for (int i = tid; i < p.NMS * NK; i += nt) ef[i] = p.tab.eff[i];
    for (int k = l; k < NK; k += LANES) L.C[k] = (k == p.nS) ? 1.0 : 0.0;
    if (l < 2) { L.Q[RUC * LANES + l] = 0.0; L.piece[MS * LANES + l] = 0.0; }

    const uint32_t Ca = lds_addr(L.C), Qa = lds_addr(L.Q), Pa = lds_addr(L.piece);
    // every load is unconditional (clamped index), so that they are in flight together
#pragma unroll
    for (int r = 0; r < RUC; ++r) {
        // a lane past the last unit evaluates the empty record, without pressure
        // dependence: 1 - 1 = 0, not gathered
        const int u = r * LANES + l;
        const bool used = u < p.nU;
        const double *rec = p.tab.units + (size_t)min(u, p.nU_pad - 1) * UNIT_DOUBLES;
        const uint64_t f = __double_as_longlong(rec[6]), v = __double_as_longlong(rec[7]);
        if constexpr (UL == UNITS_LDS) {
            if (cib == 0)
                for (int q = 0; q < 6; ++q)
                    ul[2 * ((r * 3 + q / 2) * LANES + l) + q % 2] = used ? rec[q] : 0.0;
        } else if constexpr (UL == UNITS_REG) {
            const double x0 = rec[0], x1 = rec[1], x2 = rec[2], x3 = rec[3], x4 = rec[4], x5 = rec[5];
            w.l2Af[r] = used ? x0 : 0.0; w.bf[r] = used ? x1 : 0.0; w.tf[r] = used ? x2 : 0.0;
            w.l2Ar[r] = used ? x3 : 0.0; w.br[r] = used ? x4 : 0.0; w.tr[r] = used ? x5 : 0.0;
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            w.sf[r][s] = opaque_vu(Ca + (used ? (uint32_t)((f >> (16 * s)) & 0xffffu) : 8u * p.nS));
            w.sr[r][s] = opaque_vu(Ca + (used ? (uint32_t)((v >> (16 * s)) & 0xffffu) : 8u * p.nS));
        }
    }
    // the gather tables of the SG-lane plan, chunk c = segment * SG + lane;
    // segments shorter than SL end with zero terms (adding 0.0 changes no sum)
    const int H = p.SEGL / 2;
    const uint32_t zt = (uint32_t)(p.RU * SG * 8), zp = (uint32_t)(p.NSEG * SG * 8);
    const uint32_t zt_w = (uint32_t)(RUC * LANES * 8), zp_w = (uint32_t)(MS * LANES * 8);
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        const int c = m * LANES + l;
        const bool used = c < p.NSEG * SG;
        const uint32_t *t = p.tab.gather + (used ? (size_t)(c / SG) * H * SG + c % SG : 0);
        uint32_t x[(SL + 1) / 2];
#pragma unroll
        for (int e = 0; e < SL; e += 2) x[e / 2] = t[(e < p.SEGL ? e / 2 : 0) * SG];
#pragma unroll
        for (int e = 0; e < SL; ++e) {
            const uint32_t y = (e & 1) ? (x[e / 2] >> 16) : (x[e / 2] & 0xffffu);
            w.gt[m][e] = opaque_vu(Qa + (used && e < p.SEGL && y != zt ? y : zt_w));
        }
    }
    const int H2 = (p.L2P + p.L2N) / 2;
    auto piece_of = [&](int s, int i, bool used) {
        const uint32_t x = p.tab.gather2[(s * H2 + (used ? i / 2 : 0)) * SG + g];
        const uint32_t y = (i & 1) ? (x >> 16) : (x & 0xffffu);
        return opaque_vu(Pa + (used && y != zp ? y : zp_w));
    };
#pragma unroll
    for (int s = 0; s < NSL; ++s) {
#pragma unroll
        for (int i = 0; i < LP; ++i) w.gp[s][i] = piece_of(s, i, i < p.L2P);
#pragma unroll
        for (int i = 0; i < LN; ++i) w.gn[s][i] = piece_of(s, p.L2P + i, i < p.L2N);
        const int k = s * SG + g;
        w.W[s] = p.tab.spec[F_W * NK + k];
        w.invW[s] = p.tab.spec[F_INVW * NK + k];
        w.tmid[s] = p.tab.spec[F_TMID * NK + k];
        w.cst[s] = opaque_vu(Ca + 8u * (uint32_t)((k >= 1 && k < p.N && l < SG) ? k - 1 : NK));
    }
    w.qst = opaque_vu(Qa + 8u * l);
    w.pst = opaque_vu(Pa + 8u * l);
    w.invTmax = opaque_vd(p.invTmax);
    __syncthreads();
}

__device__ __forceinline__ void lds_put(uint32_t a, double v) { *(lds_double *)(uintptr_t)a = v; }

template <int N>
__device__ __forceinline__ double lds_sum(const uint32_t (&a)[N]) {
    double v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = lds_at(a[i]);
    double acc = v[0];
#pragma unroll
    for (int i = 1; i < N; ++i) acc += v[i];
    return acc;
}

// The source term of rhs_eval (rkc_device.h) for the wave's cell.  Lanes
// without a state element have zeros in every table row, so nothing is masked.
template <int SG, int NSL, int RUC, int UL, int NW, int MS, int SL, int LP, int LN, bool PD>
__device__ __forceinline__ void rhs_wave(const double (&z)[NSL], double P10, double invP10,
                                         double (&fz)[NSL], const WaveLds &L,
                                         const WaveTab<NSL, RUC, UL, MS, SL, LP, LN> &w, const ExpK &K,
                                         int g, int l, int N, int RUpw, int NMS, int pd0,
                                         int npd) {
    constexpr int NK = NSL * SG, LANES = 64 * NW;
    const double T = readlane_f64(z[0], 0);

    double2 ga{0.0, 0.0}, gb{0.0, 0.0}, gc{0.0, 0.0};
    if constexpr (UL == UNITS_GLOBAL) { ga = L.units[0]; gb = L.units[64]; gc = L.units[128]; }
    // the coefficients' loads run under the logarithm (with one slot per lane;
    // with two they would hold 44 registers meanwhile)
    double ca[NSL][5], cb[NSL][6];
#pragma unroll
    for (int s = 0; s < NSL; ++s) {
        const double *a = L.spec + s * SG + g + (T >= w.tmid[s] ? F_CPHI * NK : F_CPLO * NK);
#pragma unroll
        for (int q = 0; q < 5; ++q) ca[s][q] = a[q * NK];
#pragma unroll
        for (int q = 0; q < 6; ++q) cb[s][q] = a[(F_HLO - F_CPLO + q) * NK];
    }
    if constexpr (NSL == 1) __builtin_amdgcn_sched_barrier(0);
    const double invT = rcp_nr(T);
    const double l2T = log2_pos(T, K);
    const double invTa = fmin(invT, w.invTmax);
    if constexpr (NSL == 1) __builtin_amdgcn_sched_barrier(0);

    double sYW = 0.0, sYcp = 0.0;
    double hRT[NSL];
#pragma unroll
    for (int s = 0; s < NSL; ++s) {
        const double *a = ca[s], *b = cb[s];
        const double cpR = a[0] + T * (a[1] + T * (a[2] + T * (a[3] + T * a[4])));
        hRT[s] = b[0] + T * (b[1] + T * (b[2] + T * (b[3] + T * b[4]))) + b[5] * invT;
        const double YW = z[s] * w.invW[s];
        if (s == 0) {
            sYW = YW;
            sYcp = YW * cpR;
        } else {
            sYW += YW;
            sYcp += YW * cpR;
        }
    }
    usum2<SG>(sYW, sYcp);
    const double RTW = R_ERG * T * sYW;
    const double rho = P10 * rcp_nr(RTW);
    const double inv_rho = RTW * invP10;

    double Ck[NSL];
#pragma unroll
    for (int s = 0; s < NSL; ++s) {
        Ck[s] = rho * z[s] * w.invW[s];
        lds_put(w.cst[s], Ck[s]);
    }
    if constexpr (PD)
    for (int q = 0; q < NMS; q += 2) {
        double p0 = 0.0, p1 = 0.0;
        const bool two = q + 1 < NMS;
#pragma unroll
        for (int s = 0; s < NSL; ++s) {
            const int k = s * SG + g;
            const double Cs = (k >= 1 && k < N) ? Ck[s] : 0.0;
            p0 += L.eff[q * NK + k] * Cs;
            if (two) p1 += L.eff[(q + 1) * NK + k] * Cs;
        }
        if (two) usum2<SG>(p0, p1);
        else p0 = usum<SG>(p0);
        if (l % 64 == 0) {
            L.Mv[q] = p0;
            if (two) L.Mv[q + 1] = p1;
        }
    }
    cell_sync<NW>();

    // (a round's parameters too when they come from global memory; the first
    // round's were loaded at the start)
    // a round's concentrations load under the exponentials of the round before
    double xf[3], xr[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) { xf[s] = lds_at(w.sf[0][s]); xr[s] = lds_at(w.sr[0][s]); }
#pragma unroll
    for (int r = 0; r < RUC; ++r) {
        double nf[3], nr[3];
#pragma unroll
        for (int s = 0; s < 3 && r + 1 < RUC; ++s) {
            nf[s] = lds_at(w.sf[r + 1][s]);
            nr[s] = lds_at(w.sr[r + 1][s]);
        }
        double kf, kr;
        if constexpr (UL != UNITS_REG) {
            double2 a, b, c;
            if constexpr (UL == UNITS_LDS) {
                a = L.units[(3 * r) * LANES];
                b = L.units[(3 * r + 1) * LANES];
                c = L.units[(3 * r + 2) * LANES];
            } else {
                a = ga; b = gb; c = gc;
                if (r + 1 < RUC) {
                    ga = L.units[(r + 1) * 4 * LANES];
                    gb = L.units[(r + 1) * 4 * LANES + 64];
                    gc = L.units[(r + 1) * 4 * LANES + 128];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            kf = exp2_b31(arrhenius_arg(a.x, a.y, b.x, l2T, invTa), K);
            kr = exp2_b31(arrhenius_arg(b.y, c.x, c.y, l2T, invTa), K);
        } else {
            __builtin_amdgcn_sched_barrier(0);
            kf = exp2_b31(arrhenius_arg(w.l2Af[r], w.bf[r], w.tf[r], l2T, invTa), K);
            kr = exp2_b31(arrhenius_arg(w.l2Ar[r], w.br[r], w.tr[r], l2T, invTa), K);
        }
        if constexpr (PD) {
            // the lanes past the last unit have no record
            const int u = pdep_place(r * LANES + l, pd0, npd);
            if (r >= RUpw && u >= 0) {
                const double2 *pd = reinterpret_cast<const double2 *>(L.pdep) + pdep_piece(u, 0, SG);
                const double2 d0 = pd[0];
                const uint64_t tag = __double_as_longlong(d0.x);
                const int kind = (int)(tag & 0xffu);
                if (kind != 0) {
                    const double M = L.Mv[(tag >> 8) & 0xffu];
                    if (kind == 1) {
                        kf *= M;
                        kr *= M;
                    } else {
                        const double2 d1 = pd[SG], d2 = pd[2 * SG], d3 = pd[3 * SG];
                        const double k0f = exp2_b31(arrhenius_arg(d0.y, d1.x, d1.y, l2T, invTa), K);
                        const double k0r = exp2_b31(arrhenius_arg(d2.x, d2.y, d3.x, l2T, invTa), K);
                        double lFc = 0.0;
                        if (kind == 3) {
                            const double2 d4 = pd[4 * SG], d5 = pd[5 * SG];
                            const double Fc = (1.0 - d4.x) * exp2_sat(-T * d4.y, K) +
                                              d4.x * exp2_sat(-T * d5.x, K) +
                                              (d5.y > 0.0 ? exp2_sat(-d5.y * invT, K) : 0.0);
                            lFc = log2_pos(Fc, K) * LOG10_2;
                        }
                        kf = falloff_rate(kf, k0f * M, lFc, kind == 3, K);
                        kr = falloff_rate(kr, k0r * M, lFc, kind == 3, K);
                    }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        const double cf = xf[0] * xf[1] * xf[2];
        const double cr = xr[0] * xr[1] * xr[2];
        lds_put(w.qst + (uint32_t)(r * LANES * 8), net_rate(kf, cf, kr, cr));
#pragma unroll
        for (int s = 0; s < 3 && r + 1 < RUC; ++s) { xf[s] = nf[s]; xr[s] = nr[s]; }
    }
    cell_sync<NW>();

#pragma unroll
    for (int m = 0; m < MS; ++m) lds_put(w.pst + (uint32_t)(m * LANES * 8), lds_sum<SL>(w.gt[m]));
    cell_sync<NW>();
    double wn[NSL];
#pragma unroll
    for (int s = 0; s < NSL; ++s) wn[s] = lds_sum<LP>(w.gp[s]) - lds_sum<LN>(w.gn[s]);
    double hs = 0.0;
#pragma unroll
    for (int s = 0; s < NSL; ++s) {
        fz[s] = w.W[s] * wn[s] * inv_rho;
        if (s == 0) hs = hRT[s] * wn[s];
        else hs += hRT[s] * wn[s];
    }
    hs = usum<SG>(hs);
    const double fT = opaque_vd(-T * hs * inv_rho * rcp_nr(sYcp));
    fz[0] = (g == 0) ? fT : fz[0];
}

// Weighted RMS norm as rms_norm2, whose scaling of weights below 2^-900 has no
// effect here: these kernels run with atol >= ATOL_WAVE only.
constexpr double ATOL_WAVE = 0x1p-900;
template <int SG, int NSL>
__device__ __forceinline__ double wave_rms2(const double (&d)[NSL], const double (&ya)[NSL],
                                            const double (&yb)[NSL], double rtol, double atol,
                                            int g, int N, double invN) {
    double s2 = 0.0;
#pragma unroll
    for (int s = 0; s < NSL; ++s) {
        const double m = fmax(fabs(ya[s]), fabs(yb[s]));
        const double w = atol + rtol * m;
        const double q = opaque_vd(d[s] * rcp_nr(w));
        const double q0 = (s * SG + g < N) ? q : 0.0;
        if (s == 0) s2 = q0 * q0;
        else s2 += q0 * q0;
    }
    return usum<SG>(s2) * invN;
}

// floor(sqrt(x)) of the correctly rounded root, for x >= 1.  The integer k
// nearest to an approximate root decides it by the sign of k^2 - x, which one
// FMA gives exactly, unless x is within rounding of k^2.
__device__ __forceinline__ double floor_sqrt(double x) {
    const double k = __builtin_rint(x * __builtin_amdgcn_rsq(x));
    const double d = __builtin_fma(k, k, -x);
    if (rare(any(!(fabs(d) > 0x1p-50 * x)))) return floor(sqrt(x));
    return d > 0.0 ? k - 1.0 : k;
}

// The cell that follows in the queue, the same in every wave of the cell.
template <int NW>
__device__ __forceinline__ int wave_next(const Params &p, Claim<64, NW> &claim, WaveState &S0, int l) {
    if (!p.persistent) return -1;
    if constexpr (NW == 1) {
        return uni(cell_at(p, claim.next(p, l)));
    } else {
        __syncthreads();
        if (l < 64) {
            const int pos = claim.next(p, l);
            if (l == 0) S0.slot = pos;
        }
        __syncthreads();
        return uni(cell_at(p, S0.slot));
    }
}

template <int SG, int NSL>
__device__ __forceinline__ bool wave_load(const Params &p, int cell, int g, double (&y)[NSL],
                                          double &P10) {
    bool bad = false;
#pragma unroll
    for (int s = 0; s < NSL; ++s) {
        const int k = s * SG + g;
        double v = 0.0;
        if (k == 0) {
            v = p.T[cell];
            bad |= !(v > 0.0) || !isfinite(v);
        } else if (k < p.N) {
            v = p.Y[(long long)cell * p.ycs + (long long)(k - 1) * p.yss];
            bad |= !isfinite(v);
        }
        y[s] = v;
    }
    const double P = opaque_vd(p.P[cell]);
    bad |= !(P > 0.0) || !isfinite(P);
    P10 = opaque_vd(P * 10.0);
    return !any(bad);
}

// Coefficients of the next stage of a step past the table, by the recurrences.
__device__ __forceinline__ double4 wave_recurrence(WaveState &S) {
    const double w0 = S.w0, Tm1 = S.Tm1, Tpm1 = S.Tpm1, Tppm1 = S.Tppm1, bm1 = S.bm1;
    const double ibm1 = S.ibm1;
    const double Tj = 2.0 * w0 * Tm1 - S.Tm2;
    const double Tpj = 2.0 * w0 * Tpm1 - S.Tpm2 + 2.0 * Tm1;
    const double Tppj = 2.0 * w0 * Tppm1 - S.Tppm2 + 4.0 * Tpm1;
    const double bj = Tppj / (Tpj * Tpj);
    double4 c;
    c.x = 2.0 * bj * w0 * ibm1;
    c.y = -bj * S.ibm2;
    c.z = 2.0 * bj * S.w1 * ibm1;
    c.w = -(1.0 - bm1 * Tm1) * c.z;
    S.Tm2 = Tm1; S.Tm1 = Tj; S.Tpm2 = Tpm1; S.Tpm1 = Tpj; S.Tppm2 = Tppm1; S.Tppm1 = Tppj;
    S.bm1 = bj; S.ibm2 = ibm1; S.ibm1 = 1.0 / bj;
    return c;
}

#define RKC_WAVE_PROLOGUE                                                                    \
    extern __shared__ __align__(16) unsigned char lds_raw[];                                 \
    constexpr int LANES = 64 * NW;                                                           \
    const int wave = uni((int)(threadIdx.x / 64));                                           \
    /* TAIL: the cells that the lane groups handed over, instead of a queue */               \
    int n_tail = 0, at = (int)(threadIdx.x / LANES * gridDim.x + blockIdx.x);                \
    if constexpr (TAIL) {                                                                    \
        n_tail = min(p.queue[QUEUE_TAIL], p.tail_cap);                                       \
        if ((int)blockIdx.x >= n_tail) return;                                               \
    }                                                                                        \
    unsigned long long done = 0;   /* evaluations of these cells before */                   \
    const TailCell *rec = nullptr;                                                           \
    auto tail_cell = [&]() {                                                                 \
        if (at >= n_tail) return -1;                                                         \
        rec = reinterpret_cast<const TailCell *>(p.tail + (long long)at * TAIL_DOUBLES);     \
        at += (int)(blockDim.x / LANES * gridDim.x);                                         \
        return uni(rec->cell);                                                               \
    };                                                                                       \
    auto first_cell = [&]() {                                                                \
        if constexpr (TAIL) return tail_cell();                                              \
        else return uni(cell_at(p, first_position<64>(p, blockDim.x / LANES, threadIdx.x / LANES))); \
    };                                                                                       \
    WaveLds L;                                                                               \
    WaveTab<NSL, RUC, UL, MS, SL, LP, LN> w;                                                     \
    wave_setup<SG, NSL, RUC, UL, NW, MS, SL, LP, LN>(p, lds_raw, L, w);                          \
    WaveState &S = *L.state;                                                                 \
    const int l = threadIdx.x % LANES, g = threadIdx.x % SG;                                 \
    const int N = p.N, RUpw = p.n_plain / LANES, NMS = p.NMS, pd0 = p.RUp * SG;              \
    const int npd = p.nU - pd0;   /* units with a record */                                 \
    const double u_round = 0x1p-53;                                                          \
    /* scalars that only the step control reads: in registers, or in LDS where the        */ \
    /* lane's share of a large mechanism needs the registers                              */ \
    constexpr bool PARK = RUC * NSL >= 3;                                                    \
    double sc_[9] = {0.0, 0.0, 0.0, 0.0, opaque_vd(p.dt), 0.0, opaque_vd(p.rtol),            \
                     opaque_vd(p.atol), opaque_vd(p.invN)};                                  \
    sc_[5] = 10.0 * u_round * sc_[4];                                                        \
    if constexpr (PARK) {                                                                    \
        S.t_end = sc_[4]; S.h_min = sc_[5]; S.rtol = sc_[6]; S.atol = sc_[7]; S.invN = sc_[8]; \
    }                                                                                        \
    const double &t_end = PARK ? S.t_end : sc_[4], &h_min = PARK ? S.h_min : sc_[5],         \
                 &rtol = PARK ? S.rtol : sc_[6], &atol = PARK ? S.atol : sc_[7],             \
                 &invN = PARK ? S.invN : sc_[8];                                             \
    double &t = PARK ? S.t : sc_[0], &sigma = PARK ? S.sigma : sc_[1],                       \
           &h_prev = PARK ? S.h_prev : sc_[2], &rprev = PARK ? S.rprev : sc_[3];             \
    const ExpK K = exp_k_local();                                                            \
    auto rhs = [&](const double (&x)[NSL], double P10, double invP10, double (&f)[NSL]) {    \
        rhs_wave<SG, NSL, RUC, UL, NW, MS, SL, LP, LN, PD>(x, P10, invP10, f, L, w, K, g, l, N,  \
                                                       RUpw, NMS, pd0, npd);                 \
    };

#define RKC_WAVE_TEMPLATE                                                                    \
    template <int OCC, int SG, int NSL, int RUC, int UL, int NW, int MS, int SL, int LP, int LN, bool PD, bool TAIL = false>

#define RKC_WAVE_BOUNDS __launch_bounds__((NW > 1 ? 64 * NW : 256 * OCC), OCC)

// Totals of the cells of the workgroup; every evaluation a wave issued, all but
// `before` of theirs, advanced one.
template <int NW>
__device__ __forceinline__ void flush_wave(const Params &p, const Agg &a, unsigned long long before,
                                           unsigned char *lds, int wave) {
    unsigned long long v[AGG_USED] = {a.rhs, a.steps, a.rej, a.sig, a.piter,
                                      (unsigned long long)a.smax, (unsigned long long)a.failed,
                                      (unsigned long long)a.worst, a.rhs - before};
    if (wave % NW != 0)   // the cell's first wave counts it
#pragma unroll
        for (int k = 0; k < AGG_USED; ++k) v[k] = 0;
    flush_block(p, v, lds, wave);
}

RKC_WAVE_TEMPLATE
__global__ RKC_WAVE_BOUNDS void rkc_wave_kernel(Params p) {
    RKC_WAVE_PROLOGUE
    const double sqrt_u = sqrt(u_round);
    const int coef_smax = p.coef_smax;
    Claim<64, NW> claim;
    claim.init();
    auto next_cell = [&]() {
        if constexpr (TAIL) return tail_cell();
        else return wave_next<NW>(p, claim, *L.state0, l);
    };
    for (int cell = first_cell(); cell >= 0; cell = next_cell()) {
        double y[NSL], f0[NSL], z[NSL], fz[NSL], v[NSL];
        Counts c{0, 0, 0, 0, 0, 0, 0};
        double P10;
        if constexpr (TAIL) {
            y[0] = reinterpret_cast<const double *>(rec)[16 + g];
            c = rec->c;
            done += (unsigned)c.n_rhs;
            P10 = opaque_vd(p.P[cell] * 10.0);
        } else if (!wave_load<SG, NSL>(p, cell, g, y, P10)) {
            if (l == 0) { store_counts(p, cell, 0, c, ST_BADINPUT); agg_cell(S.agg, c, ST_BADINPUT); }
            continue;
        }
        const double invP10 = opaque_vd(1.0 / P10);
        double h = 0.0;
        t = 0.0; sigma = 0.0; h_prev = 0.0; rprev = 0.0;
        int need_sigma = 1, since_sigma = 0, fin = ST_OK;
        bool initial = true, predictive = false;
#pragma unroll
        for (int i = 0; i < NSL; ++i) z[i] = y[i];
        if constexpr (TAIL) {
            f0[0] = reinterpret_cast<const double *>(rec)[32 + g];
            v[0] = reinterpret_cast<const double *>(rec)[48 + g];
            h = opaque_vd(rec->h); t = opaque_vd(rec->t); sigma = opaque_vd(rec->sigma);
            h_prev = opaque_vd(rec->h_prev); rprev = opaque_vd(rec->rprev);
            need_sigma = uni(rec->need_sigma);
            since_sigma = uni(rec->since_sigma);
            predictive = uni(rec->flag) != 0;
            initial = false;
        }
        for (;;) {
            if (rare(need_sigma)) {
                // spectral radius by the nonlinear power method; before the
                // first step f(y0) comes first and the initial step follows
                double delta = 0.0, sigma_prev = 0.0, ht = 0.0;
                int k_pow = 0, mode = initial ? PH_F0 : PH_POWER;
                bool done = false;
                for (;;) {
                    if (mode == PH_POWER && k_pow == 0) {
                        double ny2 = 0.0, nv2 = 0.0;
#pragma unroll
                        for (int i = 0; i < NSL; ++i) { ny2 += y[i] * y[i]; nv2 += v[i] * v[i]; }
                        usum2<SG>(ny2, nv2);
                        const double ny = sqrt(ny2);
                        delta = (ny > 0.0) ? sqrt_u * ny : sqrt_u;
                        double nv = sqrt(nv2);
                        if (!any(nv > 0.0)) {
                            double o2 = 0.0;
#pragma unroll
                            for (int i = 0; i < NSL; ++i) {
                                v[i] = (i * SG + g < N) ? 1.0 : 0.0;
                                o2 += v[i] * v[i];
                            }
                            nv = sqrt(usum<SG>(o2));
                        }
                        const double q = delta / nv;
#pragma unroll
                        for (int i = 0; i < NSL; ++i) z[i] = y[i] + q * v[i];
                        k_pow = 1;
                        sigma_prev = 0.0;
                    }
                    rhs(z, P10, invP10, fz);
                    c.n_rhs += 1;
                    if (mode == PH_POWER) {
                        c.n_piter += 1;
                        double gv[NSL];
                        double ng2 = 0.0, dz2 = 0.0;
#pragma unroll
                        for (int i = 0; i < NSL; ++i) {
                            gv[i] = fz[i] - f0[i];
                            const double dd = z[i] - y[i];
                            ng2 += gv[i] * gv[i];
                            dz2 += dd * dd;
                        }
                        usum2<SG>(ng2, dz2);
                        const double ng = sqrt(ng2);
                        double sig = ng / sqrt(dz2);
                        bool stop = false;
                        if (k_pow >= 2 && any(fabs(sig - sigma_prev) <= 0.01 * sig)) stop = true;
                        else if (any(ng == 0.0)) { sig = 0.0; stop = true; }
                        else if (k_pow == 50) stop = true;
                        if (!stop) {
                            const double q = delta / ng;
#pragma unroll
                            for (int i = 0; i < NSL; ++i) z[i] = y[i] + q * gv[i];
                            sigma_prev = sig;
                            k_pow = k_pow + 1;
                            continue;
                        }
#pragma unroll
                        for (int i = 0; i < NSL; ++i) v[i] = z[i] - y[i];
                        c.n_sigma += 1;
                        sigma = 1.2 * sig;
                        if (!any(isfinite(sigma))) { done = true; fin = ST_NONFINITE; break; }
                        if (!initial) break;
                        ht = (sigma > 0.0) ? 1.0 / sigma : t_end;
                        if (ht > t_end) ht = t_end;
#pragma unroll
                        for (int i = 0; i < NSL; ++i) z[i] = y[i] + ht * f0[i];
                        mode = PH_INIT;
                    } else if (mode == PH_F0) {
                        int bad = 0;
#pragma unroll
                        for (int i = 0; i < NSL; ++i) {
                            f0[i] = fz[i];
                            v[i] = fz[i];
                            bad |= (i * SG + g < N) && !isfinite(fz[i]);
                        }
                        if (any(bad)) { done = true; fin = ST_NONFINITE; break; }
                        mode = PH_POWER;
                    } else {
                        double d[NSL];
#pragma unroll
                        for (int i = 0; i < NSL; ++i) d[i] = ht * (fz[i] - f0[i]);
                        const double e0 = sqrt(wave_rms2<SG, NSL>(d, y, y, rtol, atol, g, N, invN));
                        if (!any(isfinite(e0))) { done = true; fin = ST_NONFINITE; break; }
                        h = (e0 > 0.0) ? 0.1 * ht / sqrt(e0) : ht;
                        if (h < h_min) h = h_min;
                        if (h > t_end) h = t_end;
                        initial = false;
                        break;
                    }
                }
                if (done) break;
                need_sigma = 0;
                since_sigma = 0;
            }

            // stage count from the spectral radius, then the first stage (E:rkc1)
            const double left = t_end - t;
            bool last = any(h >= left);
            h = (h >= left) ? left : h;
            const int sv = cvt_sat_i32(floor_sqrt(1.0 + 1.54 * h * sigma));
            int s = uni(sv);
            const int st_u = s + 1;   // the stage count unless it is capped
            // both reads use the per-lane copy of s + 1, which is ready first
            const int st = min(sv, MUT_N - 2) + 1;
            double mu_t1 = L.mut1[st];
            double4 cf;   // mu, nu, mu~, gamma~ of the stage that follows the next evaluation
            if (rare(s >= p.s_max)) {
                s = p.s_max;
                h = ((double)(p.s_max - 1) * (double)(p.s_max - 1) - 1.0) / (1.54 * sigma);
                last = false;
            } else {
                s = 1 + s;
            }
            c.s_hash = (int)((unsigned)c.s_hash * 31u + (unsigned)s);
            c.s_max_used = max(c.s_max_used, s);
            const bool tab = s <= coef_smax;
            const double *cs = p.coef + 4 * (coef_offset(s) + 1);
            if (!rare(!tab)) {
                if (rare(s != st_u)) mu_t1 = L.mut1[s];
                cf = *reinterpret_cast<const double4 *>(cs);
            } else {
                const double w0 = 1.0 + KAPPA / ((double)s * (double)s);
                double T0 = 1.0, T1 = w0, P0 = 0.0, P1 = 1.0, Q0 = 0.0, Q1 = 0.0;
                double P2 = 0.0, Q2 = 0.0;
                for (int jj = 2; jj <= s; ++jj) {
                    const double Tn = 2.0 * w0 * T1 - T0;
                    const double Pn = 2.0 * w0 * P1 - P0 + 2.0 * T1;
                    const double Qn = 2.0 * w0 * Q1 - Q0 + 4.0 * P1;
                    if (jj == 2) { P2 = Pn; Q2 = Qn; }
                    T0 = T1; T1 = Tn; P0 = P1; P1 = Pn; Q0 = Q1; Q1 = Qn;
                }
                const double w1 = P1 / Q1;
                const double b1 = 1.0 / w0;
                const double b2 = Q2 / (P2 * P2);
                S.w0 = w0; S.w1 = w1;
                S.Tm1 = w0; S.Tm2 = 1.0; S.Tpm1 = 1.0; S.Tpm2 = 0.0; S.Tppm1 = 0.0; S.Tppm2 = 0.0;
                S.bm1 = b1; S.ibm1 = w0; S.ibm2 = 1.0 / b2;
                mu_t1 = b1 * w1;
                cf = wave_recurrence(S);
            }
            double wm1[NSL], wm2[NSL];
#pragma unroll
            for (int i = 0; i < NSL; ++i) {
                wm2[i] = y[i];
                wm1[i] = y[i] + mu_t1 * h * f0[i];
            }
            for (int j = 2;; ++j) {
                rhs(wm1, P10, invP10, fz);
                if (j > s) break;
                const double c0 = 1.0 - cf.x - cf.y, ch1 = cf.z * h, ch2 = cf.w * h;
#pragma unroll
                for (int i = 0; i < NSL; ++i) {
                    const double wj = c0 * y[i] + cf.x * wm1[i] + cf.y * wm2[i] + ch1 * fz[i] +
                                      ch2 * f0[i];
                    wm2[i] = wm1[i];
                    wm1[i] = opaque_vd(wj);
                }
                // after the last use of this stage's, so that the load lands
                // in the same registers while the next evaluation runs
                asm volatile("" ::: "memory");
                if (!rare(!tab)) {
                    cs += 4;
                    cf = *reinterpret_cast<const double4 *>(cs);
                } else {
                    cf = wave_recurrence(S);
                }
            }
            c.n_rhs += s;

            // error estimate, weighted RMS norm (E:rmsE) and step control
            double d[NSL];
#pragma unroll
            for (int i = 0; i < NSL; ++i)
                d[i] = 0.8 * (y[i] - wm1[i]) + 0.4 * h * (f0[i] + fz[i]);
            const double e2 = wave_rms2<SG, NSL>(d, y, wm1, rtol, atol, g, N, invN);
            if (rare(!any(e2 <= NORM2_ACCEPT))) {
                c.n_reject += 1;
                double fac = any(isfinite(e2)) ? 0.8 * rsixth_pos(e2) : 0.1;
                if (fac < 0.1) fac = 0.1;
                h = h * fac;
                need_sigma = 1;
                predictive = false;
            } else {
                c.n_steps += 1;
#pragma unroll
                for (int i = 0; i < NSL; ++i) { y[i] = wm1[i]; f0[i] = fz[i]; }
                if (rare(last)) break;
                t = t + h;
                since_sigma = since_sigma + 1;
                need_sigma = (since_sigma >= 25);
                double r = rsixth_pos(e2);
                const double fp = 0.8 * h * r * r * rcp_nr(h_prev * rprev);
                double fac = predictive ? fp : 0.8 * r;
                if (rare(any(!(fac == fac)))) {
                    // an error estimate of 0, now or (kept as r = 0) before
                    const bool zero = any(e2 == 0.0);
                    fac = zero ? 10.0 : 0.0;
                    if (zero) r = 0.0;
                }
                fac = fmax(fmin(fac, 10.0), 0.1);
                h_prev = h;
                rprev = r;
                predictive = true;
                h = h * fac;
            }
            if (rare(any(h < h_min))) { fin = ST_UNDERFLOW; break; }
            if (rare(c.n_steps + c.n_reject >= p.max_steps)) { fin = ST_MAXSTEPS; break; }
        }
        if (l < SG) store_state<SG, NSL>(p, cell, g, y);
        if (l == 0) { store_counts(p, cell, 0, c, fin); agg_cell(S.agg, c, fin); }
    }
    flush_wave<NW>(p, S.agg, done, lds_raw, wave);
}

RKC_WAVE_TEMPLATE
__global__ RKC_WAVE_BOUNDS void rkck_wave_kernel(Params p) {
    RKC_WAVE_PROLOGUE
    Claim<64, NW> claim;
    claim.init();
    auto next_cell = [&]() {
        if constexpr (TAIL) return tail_cell();
        else return wave_next<NW>(p, claim, *L.state0, l);
    };
    for (int cell = first_cell(); cell >= 0; cell = next_cell()) {
        double y[NSL];
        Counts c{0, 0, 0, 0, 0, 0, 0};
        double P10;
        if constexpr (TAIL) {
            y[0] = reinterpret_cast<const double *>(rec)[16 + g];
            c = rec->c;
            done += (unsigned)c.n_rhs;
            P10 = opaque_vd(p.P[cell] * 10.0);
        } else if (!wave_load<SG, NSL>(p, cell, g, y, P10)) {
            if (l == 0) { store_counts(p, cell, 0, c, ST_BADINPUT); agg_cell(S.agg, c, ST_BADINPUT); }
            continue;
        }
        const double invP10 = opaque_vd(1.0 / P10);
        // first trial step is the whole interval; the last step lands on dt
        double h = t_end;
        t = 0.0;
        bool last = true;
        int fin;
        if constexpr (TAIL) {
            h = opaque_vd(rec->h);
            t = opaque_vd(rec->t);
            last = uni(rec->flag) != 0;
        }
        for (;;) {
            double k1[NSL], k2[NSL], k3[NSL], k4[NSL], k5[NSL], z[NSL], fz[NSL];
            rhs(y, P10, invP10, fz);
#pragma unroll
            for (int i = 0; i < NSL; ++i) { k1[i] = h * fz[i]; z[i] = y[i] + CK_B21 * k1[i]; }
            rhs(z, P10, invP10, fz);
#pragma unroll
            for (int i = 0; i < NSL; ++i) {
                k2[i] = h * fz[i];
                z[i] = y[i] + CK_B31 * k1[i] + CK_B32 * k2[i];
            }
            rhs(z, P10, invP10, fz);
#pragma unroll
            for (int i = 0; i < NSL; ++i) {
                k3[i] = h * fz[i];
                z[i] = y[i] + CK_B41 * k1[i] + CK_B42 * k2[i] + CK_B43 * k3[i];
            }
            rhs(z, P10, invP10, fz);
#pragma unroll
            for (int i = 0; i < NSL; ++i) {
                k4[i] = h * fz[i];
                z[i] = y[i] + CK_B51 * k1[i] + CK_B52 * k2[i] + CK_B53 * k3[i] + CK_B54 * k4[i];
            }
            rhs(z, P10, invP10, fz);
#pragma unroll
            for (int i = 0; i < NSL; ++i) {
                k5[i] = h * fz[i];
                z[i] = y[i] + CK_B61 * k1[i] + CK_B62 * k2[i] + CK_B63 * k3[i]
                     + CK_B64 * k4[i] + CK_B65 * k5[i];
            }
            rhs(z, P10, invP10, fz);
            c.n_rhs += 6;

            // embedded error estimate and step control (E:hnew)
            double y5[NSL];
            double emax = 0.0;
            int bad = 0;
#pragma unroll
            for (int i = 0; i < NSL; ++i) {
                const double k6 = h * fz[i];
                y5[i] = y[i] + CK_C1 * k1[i] + CK_C3 * k3[i] + CK_C4 * k4[i] + CK_C6 * k6;
                const double del = CK_D1 * k1[i] + 0.0 * k2[i] + CK_D3 * k3[i] + CK_D4 * k4[i]
                                 + CK_D5 * k5[i] + CK_D6 * k6;
                const double d0 = rtol * (fabs(y[i]) + fabs(k1[i]) + 1e-30);
                const double r = (i * SG + g < N) ? fabs(del / d0) : 0.0;
                bad |= !isfinite(r);
                emax = fmax(emax, isfinite(r) ? r : 0.0);
            }
            const double errmax = any(bad) ? __builtin_inf() : umax<SG>(emax);
            double hn = h;
            if (any(errmax <= 1.0)) {
                c.n_steps += 1;
#pragma unroll
                for (int i = 0; i < NSL; ++i) y[i] = y5[i];
                if (last) { fin = ST_OK; break; }
                t = t + h;
                double fac = any(errmax == 0.0) ? 5.0 : 0.9 * exp2_sat(-0.2 * log2_pos(errmax, K), K);
                if (fac > 5.0) fac = 5.0;
                hn = h * fac;
            } else {
                c.n_reject += 1;
                double fac = any(isfinite(errmax)) ? 0.9 * exp2_sat(-0.25 * log2_pos(errmax, K), K) : 0.1;
                if (fac < 0.1) fac = 0.1;
                hn = h * fac;
            }
            if (rare(any(hn < h_min))) { fin = ST_UNDERFLOW; break; }
            if (rare(c.n_steps + c.n_reject >= p.max_steps)) { fin = ST_MAXSTEPS; break; }
            const double left = t_end - t;
            last = any(hn >= left);
            h = (hn >= left) ? left : hn;
        }
        if (l < SG) store_state<SG, NSL>(p, cell, g, y);
        if (l == 0) { store_counts(p, cell, 0, c, fin); agg_cell(S.agg, c, fin); }
    }
    flush_wave<NW>(p, S.agg, done, lds_raw, wave);
}

}  // namespace rkcdev
