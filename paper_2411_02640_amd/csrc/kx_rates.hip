// kx_rates.hip -- species net production rates on gfx950.
//
// Three kernels.  Mechanisms of up to kWideMaxSpecies species: one lane per point,
// every species and reaction wave-uniform (kx_wide.h, rates_wide_tile below), or for
// calls of few points one point per workgroup with the same arithmetic (kx_few.h,
// rates_few_point).  Larger ones, whose species rows for 64 points exceed the LDS:
// lanes over species and (reaction, point) pairs (rates_tile).
//
// All evaluate, per point,
//  1. species: C_k, the Gibbs energy g_k = G_k/RT of eq:Ck (range by T_mid),
//     a_k = (p_atm/RT) exp(-g_k) and b_k = C_k / a_k into LDS.  With these,
//     prod_k C_k^nu' = A' B' and prod_k C_k^nu'' / K_c = A' B''
//     (A' = prod_reac a^nu', B' = prod_reac b^nu', B'' = prod_prod b^nu''), since
//     K_c = prod_k a_k^(nu''-nu') by eq:K_p and K_c = K_p (p_atm/RT)^(sum nu).
//     So K_c needs one exponential per species instead of one per reaction and
//     the rate of progress needs no division:
//         R_i = c_i k_f A' (B' - B'')                   (eq:r_i, eq:c_i)
//     and B' - B'' is the near-equilibrium difference, formed in FP64;
//  2. reactions: k_f (eq:arrhenius, with the beta = E_R = 0 shortcut of eq:k_f),
//     [X]_i, the Lindemann / Troe factor (eq:blend) and R_i into LDS, one chunk
//     of reactions at a time, heaviest type first;
//  3. species: wdot_k = sum_i nu_ki R_i gathered from species-major lists of R
//     slots (a net |nu| of 2 or 3 is listed that many times).  The summation
//     order is fixed, so results are deterministic; the mixed path adds its
//     groups' sums with Neumaier-compensated steps.
//
// What bounds the one-lane-per-point kernel (53 species, FP64, 2^20 points;
// measured 1.02 ms, 1.57 ms by the lanes-over-reactions form it replaced; 9
// species 0.083 against 0.64 ms, 100 species at 2^18 points 0.77 against 0.94):
// it issues about 400 vector and 310 scalar instructions per point (657 vector
// ones before: the record decoding, the padded gather lists and the idle lanes
// are gone), 65 % of the time the vector units could take at best; the rest
// is the latency of the scalar loads that miss the 16 KB scalar cache (the
// tables stream through it once per tile: their size and the number of waves
// decide, see DevWide and wide_shape) and the chunk barriers.
#include <float.h>

#include <type_traits>

#include "kx_few.h"
#include "kx_internal.h"
#include "kx_math.h"
#include "kx_wide.h"

namespace kx {
namespace {


__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The falloff data of a reaction: k_0's Arrhenius parameters and the blend
// parameters (loaded with the third-body data, for the same reason).
struct Falloff {
    double lnA0, beta0, ER0;
    double fp[5];
    int has_T2;
};

__device__ __forceinline__ Falloff load_falloff(const DevAux &ax)
{
    Falloff f;
    f.lnA0 = ax.lnA0;
    f.beta0 = ax.beta0;
    f.ER0 = ax.ER0;
#pragma unroll
    for (int e = 0; e < 5; ++e) f.fp[e] = ax.fp[e];
    f.has_T2 = ax.has_T2;
    return f;
}

// Falloff blending factor F (eq:blend), Troe and SRI in one code path (so a
// wave mixing the two runs it once):
//   Troe  log10 F = log10 F_cent / (1 + f1^2), f1 = (l + c) / (n - 0.14 (l + c)),
//         F_cent = (1 - alpha) e^(-T/T***) + alpha e^(-T/T*) [+ e^(-T**/T)],
//         c = -0.4 - 0.67 log10 F_cent, n = 0.75 - 1.27 log10 F_cent;
//   SRI   F = d T^e B^X, B = a e^(-b/T) + e^(-T/c), X = 1 / (1 + l^2),
// with l = log10 P_r.  Both are ln F = ln B / (1 + w^2) + extra, where B is
// F_cent or the SRI bracket, w = f1 or l, and extra = 0 or ln d + e ln T.  The
// base-10 logarithms are formed from natural ones.
__device__ __forceinline__ double blend_F64(const Falloff &ax, bool sri, double T, double lnT,
                                            double invT, double lnPr)
{
    constexpr double kInvLn10 = 0.43429448190325182765;
    const double a0 = ax.fp[0], a1 = ax.fp[1], a2 = ax.fp[2], a3 = ax.fp[3], a4 = ax.fp[4];
    double B = (sri ? a0 : 1.0 - a0) * kexp(-a1 * (sri ? invT : T)) +
               (sri ? 1.0 : a0) * kexp(-T * a2);
    if (!sri && ax.has_T2) B += kexp(-a3 * invT);
    const double lnB = kln(fmax(B, DBL_MIN));
    const double lB = lnB * kInvLn10;
    const double x = fma(lnPr, kInvLn10, sri ? 0.0 : fma(-0.67, lB, -0.4));
    const double nn = sri ? 1.0 : fma(-1.27, lB, 0.75);
    const double w = x * krcp(fma(sri ? 0.0 : -0.14, x, nn));
    return kexp(fma(lnB, krcp(fma(w, w, 1.0)), sri ? fma(a4, lnT, a3) : 0.0));
}

// The same in FP32 from l = log10 P_r (computed by the caller without overflow).
__device__ __forceinline__ float blend_F32(const Falloff &ax, bool sri, float T, float lnT,
                                           float invT, float lPr)
{
    const float a0 = (float)ax.fp[0], a1 = (float)ax.fp[1], a2 = (float)ax.fp[2];
    const float a3 = (float)ax.fp[3], a4 = (float)ax.fp[4];
    float B = (sri ? a0 : 1.0f - a0) * __expf(-a1 * (sri ? invT : T)) +
              (sri ? 1.0f : a0) * __expf(-T * a2);
    if (!sri && ax.has_T2) B += __expf(-a3 * invT);
    const float lnB = __logf(fmaxf(B, FLT_MIN));
    const float lB = lnB * 0.43429448190325182765f;
    const float x = lPr + (sri ? 0.0f : -0.4f - 0.67f * lB);
    const float nn = sri ? 1.0f : 0.75f - 1.27f * lB;
    const float w = x / (nn - (sri ? 0.0f : 0.14f) * x);
    return __expf(lnB / (1.0f + w * w) + (sri ? a4 * lnT + a3 : 0.0f));
}

// Exponent ln k_f of a pressure-table reaction at ln p: linear in ln p between
// the neighbouring reference pressures, the nearest end point's value outside
// them (App. A.2, pressure-dependent reactions).
__device__ __forceinline__ double plog_exponent(const DevPlog *pl, int cnt, double lnT,
                                                double invT, double lnp)
{
    int j = 0;
    while (j + 1 < cnt && pl[j + 1].lnp <= lnp) ++j;
    const DevPlog &a = pl[j];
    const double x1 = fma(a.beta, lnT, fma(-a.ER, invT, a.lnA));
    if (j + 1 >= cnt || lnp <= a.lnp) return x1;
    const DevPlog &b = pl[j + 1];
    const double x2 = fma(b.beta, lnT, fma(-b.ER, invT, b.lnA));
    return fma(x2 - x1, (lnp - a.lnp) * a.inv_dlnp, x1);
}

// Per-point factors of one species in LDS: {a_k, b_k}, 16 bytes, aligned so
// that one 16-byte LDS read fetches a pair (as two 8-byte halves it costs the
// LDS about twice the cycles).
struct alignas(16) Pair {
    double a, b;
};

__device__ __forceinline__ Pair load_pair(const char *pb, int off)
{
    return *reinterpret_cast<const Pair *>(pb + off);
}

__device__ __forceinline__ double load_b(const char *pb, int off)
{
    return *reinterpret_cast<const double *>(pb + off + 8);
}

// One reaction record held in registers: the three 16-byte words of DevRxn.
struct RxnWords {
    uint4 w0, w1, w2;
};

__device__ __forceinline__ double as_double(unsigned lo, unsigned hi)
{
    return __hiloint2double((int)hi, (int)lo);
}

// The third-body data of a reaction: the default efficiency, the inline
// efficiencies (alpha - default) and their LDS offsets, and the count of
// further ones.  Loaded as one batch as soon as the reaction record is decoded,
// so that its memory latency overlaps the Arrhenius exponentials (loaded where
// the sum is formed, each of its dependent batches stalls the wave).
struct ThirdBody {
    double def;
    double dalpha[kInlineEff];
    unsigned eoff2[kInlineEff / 2];  // two 16-bit offsets per word (unpacked where used)
    int ext_off, ext_cnt;
};

__device__ __forceinline__ ThirdBody load_third_body(const DevAux &ax)
{
    ThirdBody t;
    t.def = ax.eff_default;
#pragma unroll
    for (int e = 0; e < kInlineEff; ++e) t.dalpha[e] = ax.dalpha[e];
    const unsigned *eo = reinterpret_cast<const unsigned *>(ax.eoff);
#pragma unroll
    for (int e = 0; e < kInlineEff / 2; ++e) t.eoff2[e] = eo[e];
    t.ext_off = ax.ext_off;
    t.ext_cnt = ax.ext_cnt;
    return t;
}

// [X]_i = default [M] + sum over listed species of (alpha - default) C_k.
__device__ __forceinline__ double third_body(const MechDev &m, const ThirdBody &tb,
                                             const char *__restrict__ pb, double Mconc)
{
    double X = tb.def * Mconc;
    // the reads are issued four at a time (left to itself the scheduler waits
    // for each read in turn; eight in flight would cost registers)
#pragma unroll
    for (int e0 = 0; e0 < kInlineEff; e0 += 4) {
        Pair s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int ee = e0 + e;
            s[e] = load_pair(pb, (tb.eoff2[ee / 2] >> (16 * (ee & 1))) & 0xFFFFu);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) X = fma(tb.dalpha[e0 + e], s[e].a * s[e].b, X);
    }
    for (int e = 0; e < tb.ext_cnt; ++e) {
        const DevEff f = m.eff[tb.ext_off + e];
        const Pair s = load_pair(pb, 16 * f.sp);
        X = fma(f.dalpha, s.a * s.b, X);
    }
    return X;
}

// The per-point values phase 2 needs.
struct PtVals {
    double T, lnT, invT, M, lnp;
};

// Rate of progress R_i = c_i k_f A' (B' - B'') of one reaction at the point of
// this lane.  The LDS reads are issued before the first exponential.
template <bool MIXED>
__device__ __forceinline__ double rate_of_progress(const MechDev &m, const RxnWords &w,
                                                   const char *pb, const PtVals &q)
{
    const double lnA = as_double(w.w0.x, w.w0.y);
    const double beta = as_double(w.w0.z, w.w0.w);
    const double ER = as_double(w.w1.x, w.w1.y);
    const double A = as_double(w.w1.z, w.w1.w);
    const unsigned type = w.w2.w & 0xFFu;
    const unsigned flags = (w.w2.w >> 8) & 0xFFu;
    const unsigned aux = w.w2.w >> 16;
    const unsigned o0 = w.w2.x & 0xFFFFu, o1 = w.w2.x >> 16;
    const unsigned o3 = w.w2.y >> 16, o4 = w.w2.z & 0xFFFFu;

    const bool has_tb = type != KX_RXN_ELEMENTARY && type != KX_RXN_PLOG;
    const bool has_fo = has_tb && type != KX_RXN_THREEBODY;
    ThirdBody tb;
    Falloff fo;
    if (has_tb) tb = load_third_body(m.aux[aux]);

    // exponent of k_f (eq:k_f); k_f = A without an exponential when beta = E_R = 0
    // (such reactions are sorted together, so the branch is mostly wave-uniform),
    // or interpolated in ln p for a pressure-table reaction
    const bool kconst = (flags & kFlagKfConst) != 0;
    double xf = kconst ? lnA : fma(beta, q.lnT, fma(-ER, q.invT, lnA));
    if (type == KX_RXN_PLOG) {
        const DevAux &ax = m.aux[aux];
        xf = plog_exponent(m.plog + ax.plog_off, ax.plog_cnt, q.lnT, q.invT, q.lnp);
    }
    // the LDS reads go before the exponentials so that their latency hides behind them
    const Pair r0 = load_pair(pb, o0), r1 = load_pair(pb, o1);
    const double bp0 = load_b(pb, o3), bp1 = load_b(pb, o4);
    double kf = A;
    if (!kconst) kf = MIXED ? exp_mixed(xf) : kexp(xf);
    double Ap = r0.a * r1.a, Bp = r0.b * r1.b, Bpp = bp0 * bp1;
    // third molecule slots: skipped by the whole wave when none of its
    // reactions has three molecules on a side (the dummy species gives 1)
    const unsigned o2 = w.w2.y & 0xFFFFu, o5 = w.w2.z >> 16;
    const unsigned dummy = 16u * (unsigned)m.ns;
    if (__builtin_amdgcn_ballot_w64(o2 != dummy || o5 != dummy) != 0) {
        const Pair r2 = load_pair(pb, o2);
        Ap *= r2.a;
        Bp *= r2.b;
        Bpp *= load_b(pb, o5);
    }
    if (flags & kFlagOrders) {
        // explicit forward orders (irreversible): prod_k C_k^o_k, C_k = a_k b_k
        const DevAux &ax = m.aux[aux];
        double s = 0.0;
        bool zero = false;
#pragma unroll
        for (int e = 0; e < kMaxOrd; ++e) {
            const double o = ax.oval[e];
            if (o != 0.0) {
                const Pair qq = load_pair(pb, ax.ooff[e]);
                const double C = qq.a * qq.b;
                zero = zero || !(C > 0.0);
                s = fma(o, kln(fmax(C, DBL_MIN)), s);
            }
        }
        Ap = zero ? 0.0 : kexp(s);
        Bp = 1.0;
        Bpp = 0.0;
    }
    double c = 1.0;
    if (has_tb) {
        // FP64: the falloff data is read before the third-body sums, whose LDS
        // reads and products then cover its memory latency (the mixed path
        // reads it where it is used: the earlier read measured slower there)
        if (!MIXED && has_fo) fo = load_falloff(m.aux[aux]);
        const double X = third_body(m, tb, pb, q.M);
        c = X;
        if (has_fo) {
            if (MIXED) fo = load_falloff(m.aux[aux]);
            // P_r = k_0 [X] / k_inf = e0 [X] with e0 = exp(x_0 - x_inf) (no division)
            const double d0 = fma(fo.beta0, q.lnT, fma(-fo.ER0, q.invT, fo.lnA0)) - xf;
            const double e0 = MIXED ? exp_mixed(d0) : kexp(d0);
            const double Pr = e0 * X;
            double F = 1.0;
            if (type == KX_RXN_TROE || type == KX_RXN_SRI) {
                const bool sri = type == KX_RXN_SRI;
                if (MIXED) {
                    F = (double)blend_F32(fo, sri, (float)q.T, (float)q.lnT, (float)q.invT,
                                          log10_wide(Pr));
                } else {
                    // ln max(P_r, DBL_MIN) without forming the logarithm of P_r
                    const double lnPr = fmax(d0 + kln(fmax(X, DBL_MIN)), -708.39641853226410622);
                    F = blend_F64(fo, sri, q.T, q.lnT, q.invT, lnPr);
                }
            }
            // eq:c_i: P_r/(1+P_r) F; chemically activated: F/(1+P_r) with k_0 =
            // e0 k_inf in r_i, i.e. c k_inf = e0 F/(1+P_r) k_inf
            const double g = krcp(1.0 + Pr) * F;
            c = (flags & kFlagChemAct) ? e0 * g : Pr * g;
        }
    }
    const double rev = (flags & kFlagReversible) ? 1.0 : 0.0;
    return c * kf * Ap * fma(-rev, Bpp, Bp);
}

// Gibbs energy g = G/RT of one species at one temperature (eq:Ck with the
// coefficients pre-scaled: g = c0 (1 - ln T) + c1 T + ... + c4 T^4 + c5 / T + c6).
__device__ __forceinline__ double gibbs(const double (&g)[7], double T, double lnT, double invT)
{
    const double poly = T * fma(T, fma(T, fma(T, g[4], g[3]), g[2]), g[1]);
    return fma(g[0], 1.0 - lnT, poly) + fma(g[5], invT, g[6]);
}

// The lanes-over-reactions kernel: points per tile, and species per lane in the
// species phases (mechanisms above 128 species).
constexpr int kPts = 2;
constexpr int kSpl = 4;

// Two groups' partial sums ga, gb per trip of a gather loop: FP64 adds each to
// the running sum as it is formed (first_of_pair, then second_of_pair); the
// mixed path adds their sum with one compensated step (the two groups' plain
// sum carries FP64 rounding, far below the mixed path's error).
template <bool MIXED>
__device__ __forceinline__ void first_of_pair(double (&acc)[kPts], const double (&ga)[kPts])
{
    if (!MIXED) {
#pragma unroll
        for (int j = 0; j < kPts; ++j) acc[j] += ga[j];
    }
}

template <bool MIXED>
__device__ __forceinline__ void second_of_pair(double (&acc)[kPts], double (&cmp)[kPts],
                                               const double (&ga)[kPts], const double (&gb)[kPts])
{
#pragma unroll
    for (int j = 0; j < kPts; ++j) {
        if (MIXED)
            accumulate<true>(acc[j], cmp[j], ga[j] + gb[j]);
        else
            acc[j] += gb[j];
    }
}

// Per-point constants of a tile, computed once per point (lane = point).
struct PointConst {
    double T, lnT, invT, M;  // temperature, ln T, 1/T, [M] = p / RT
    double P0, cf;           // p_atm / RT; C_k = Y_k / W_k * cf with cf = [M] W-bar
    double lnp, pad;         // ln p (pressure-table reactions)
};

// LDS layout of one workgroup (one wave):
//   sq    [chunk + 1][2]    rates of progress of the current chunk, the two points
//         side by side; slot `chunk` is zero and absorbs the gather padding; at byte
//         0 so that the gather offsets are LDS addresses
//   pairs [2][ns + 1]       {a, b} per point (entry ns is the dummy species, {1, 1})
//   pc    [2]               PointConst of the tile's points
//   Yt    [ns][3]           Y tile in, wdot tile out (coalesced row loads/stores)
// One tile of `npts` (<= 2) points starting at point i0 of arrays whose species
// rows have stride ld:
//   phase 1 -- lane = species, both points;
//   phase 2 -- lane = (reaction, point): lane 2r + j takes reaction r at point j, so
//              a group of 32 falloff reactions fills a whole 64-lane iteration;
//   phase 3 -- lane = species: one 16-byte LDS read per list entry returns the
//              rate of progress of the reaction at both points.
// Two other forms were measured against this one for 200 species (1500 reactions,
// 100003 points, 1.13 ms): one lane per point as below with 40 points per tile (what
// the LDS holds, so 24 lanes idle and four waves per SIMD) 1.27 ms, also with the
// tables read ahead by vector loads (1.29); half a wave per species and reaction
// with 32 points per tile 1.31 ms.
// A 16-byte LDS read at a byte address (the gather lists hold addresses
// relative to the dynamic LDS, which starts at 0 when the kernel has no static
// LDS; rates_tile<..., true> is only entered after checking that).
__device__ __forceinline__ double2 lds_read16(unsigned addr)
{
    typedef double v2d __attribute__((ext_vector_type(2)));
    const v2d v = *(const __attribute__((address_space(3))) v2d *)(size_t)addr;
    return make_double2(v.x, v.y);
}

__device__ __forceinline__ unsigned lds_base()
{
    extern __shared__ double lds[];
    return (unsigned)(size_t)(__attribute__((address_space(3))) double *)lds;
}

// ---- phase 3: wdot_k = sum_i nu_ki R_i for both points, one chunk of reactions.
// Lane = species (kSpl per lane); a group is eight list entries, summed plainly per
// point (the mixed path compensates the running sum once per two groups).  All reads
// of a group are issued before the first sum (left to itself the scheduler waits for
// each read in turn), and two groups are handled per trip with alternating offset
// registers (the next group's offsets in flight).
//
// gather_split: a +q list and a -q list per species, each padded to whole
// groups (the group's sum is negated for the -q groups).
template <bool MIXED, bool DIRECT>
__device__ __forceinline__ void gather_split(const MechDev &m, int c, int gw, int lane,
                                             const char *qb, double (&acc)[kSpl][kPts],
                                             double (&cmp)[kSpl][kPts])
{
    const int npos = m.gpos[c], ngrp = npos + m.gneg[c];
    const uint4 *ge = m.gent + ((size_t)m.goff[c] * gw + lane) * 2;
#pragma unroll
    for (int s = 0; s < kSpl; ++s) {
        const uint4 *g = ge + 2 * kWave * s;
        auto group = [&](const uint4 &v0, const uint4 &v1, int it, double (&gs)[kPts]) {
            const unsigned off[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
            double2 q2[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                q2[u] = DIRECT ? lds_read16(off[u])
                               : *reinterpret_cast<const double2 *>(qb + off[u]);
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);  // DS reads
            __builtin_amdgcn_sched_group_barrier(0x002, 16, 0);  // VALU
            double g0 = q2[0].x, g1 = q2[0].y;
#pragma unroll
            for (int u = 1; u < 8; ++u) {
                g0 += q2[u].x;
                g1 += q2[u].y;
            }
            if (it >= npos) {
                g0 = -g0;
                g1 = -g1;
            }
            gs[0] = g0;
            gs[1] = g1;
        };
        uint4 a0 = make_uint4(0, 0, 0, 0), a1 = a0, b0 = a0, b1 = a0;
        if (ngrp > 0) {
            a0 = g[0];
            a1 = g[1];
        }
        int it = 0;
        for (; it + 1 < ngrp; it += 2) {
            b0 = g[(size_t)(it + 1) * 2 * gw];
            b1 = g[(size_t)(it + 1) * 2 * gw + 1];
            double ga[kPts], gb[kPts];
            group(a0, a1, it, ga);
            first_of_pair<MIXED>(acc[s], ga);
            if (it + 2 < ngrp) {
                a0 = g[(size_t)(it + 2) * 2 * gw];
                a1 = g[(size_t)(it + 2) * 2 * gw + 1];
            }
            group(b0, b1, it + 1, gb);
            second_of_pair<MIXED>(acc[s], cmp[s], ga, gb);
        }
        if (it < ngrp) {
            double ga[kPts];
            group(a0, a1, it, ga);
#pragma unroll
            for (int j = 0; j < kPts; ++j) accumulate<MIXED>(acc[s][j], cmp[s][j], ga[j]);
        }
    }
}

// `lane` is threadIdx.x; the batch kernel passes it through an opaque move in
// each trip of its tile loop, so that the tile's lane-dependent addresses are
// not hoisted out of the loop (kept live across tiles they cost registers).
template <bool MIXED, bool DIRECT>
__device__ __forceinline__ void rates_tile(int lane, const MechDev &m, int64_t ld, int64_t i0,
                                           int npts, const double *__restrict__ T,
                                           const double *__restrict__ P,
                                           const double *__restrict__ Y,
                                           double *__restrict__ wdot)
{
    extern __shared__ double lds[];
    constexpr int NGW = kWave / kPts;  // species groups of the W-bar pass
    const int ns = m.ns;
    const int ys = kPts + 1;
    double *sq = lds;
    double *pairs = sq + (2 * (m.chunk + 1));
    PointConst *pc = reinterpret_cast<PointConst *>(pairs + 2 * kPts * (ns + 1));
    double *Yt = reinterpret_cast<double *>(pc + kPts);
    const char *qb = reinterpret_cast<const char *>(sq);

    // the temperature and pressure of the tile's points are read first, so
    // that their memory latency overlaps the Y tile's
    double Tl = 0.0, Pl = 0.0;
    if (lane < kPts) {
        const int64_t i = i0 + min(lane, npts - 1);
        Tl = T[i];
        Pl = P[i];
    }
    // the tile's Y, eight row loads per lane in flight before the first LDS
    // store (a loop of load-wait-store would pay one memory latency per row)
    constexpr int kLd = 8;
    for (int e0 = lane; e0 < ns * kPts; e0 += kLd * kWave) {
        double v[kLd];
#pragma unroll
        for (int u = 0; u < kLd; ++u) {
            const int e = e0 + u * kWave, k = e / kPts, c = e % kPts;
            v[u] = (e < ns * kPts && c < npts) ? Y[(int64_t)k * ld + i0 + c] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kLd; ++u) {
            const int e = e0 + u * kWave;
            if (e < ns * kPts) Yt[(e / kPts) * ys + e % kPts] = v[u];
        }
    }
    __syncthreads();
    {
        // sum_k Y_k / W_k = 1 / W-bar: lane = (point, species group); the
        // group partials meet in the (still unused) rate-of-progress array.
        // The 1/W_k of eight species are loaded before they are used.
        const int c = lane % kPts, g = lane / kPts;
        const int cc = min(c, npts - 1);  // padding points repeat the last one
        double part = 0.0;
        for (int k0 = g; k0 < ns; k0 += kLd * NGW) {
            double iw[kLd];
#pragma unroll
            for (int u = 0; u < kLd; ++u) {
                const int k = k0 + u * NGW;
                iw[u] = k < ns ? m.gsoa[((size_t)(k / kWave) * 16 + 15) * kWave + k % kWave] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kLd; ++u) {
                const int k = k0 + u * NGW;
                if (k < ns) part = fma(Yt[k * ys + cc], iw[u], part);
            }
        }
        sq[g * kPts + c] = part;
    }
    __syncthreads();
    if (lane < kPts) {
        double wsum = 0.0;
#pragma unroll
        for (int g = 0; g < NGW; ++g) wsum += sq[g * kPts + lane];
        PointConst q;
        q.T = Tl;
        q.lnT = kln(q.T);
        q.invT = krcp(q.T);
        const double invRT = krcp(kRu * q.T);
        q.M = Pl * invRT;
        q.P0 = kPatm * invRT;
        q.cf = q.M * krcp(wsum);
        q.lnp = kln(Pl);
        q.pad = 0.0;
        pc[lane] = q;
    }
    __syncthreads();
    if (lane < kPts) {
        pairs[2 * ns + 2 * (ns + 1) * lane] = 1.0;
        pairs[2 * ns + 2 * (ns + 1) * lane + 1] = 1.0;
    }
    if (lane < 2) {
        sq[2 * m.chunk + lane] = 0.0;
    }

    const int jl = lane & 1;   // point of this lane in phase 2
    const int rl = lane >> 1;  // reaction slot of this lane in phase 2
    const char *pbl = reinterpret_cast<const char *>(pairs + 2 * (ns + 1) * jl);
    const int gw = kWave * m.gpass;
    // ---- phase 1: species (both points per lane)
    PointConst ps[kPts];
#pragma unroll
    for (int j = 0; j < kPts; ++j) ps[j] = pc[j];
#pragma unroll
    for (int s = 0; s < kSpl; ++s) {
        const int k = lane + kWave * s;
        if (k < ns) {
            // both temperature ranges' coefficients are read once per tile
            // and selected per point (one read per point would cost the
            // vector-memory unit four times as many loads), from the
            // by-field table (a wave's read is one contiguous row)
            const double *gs = m.gsoa + (size_t)s * 16 * kWave + lane;
            // the same rows every step: read them per step (kept in
            // registers across the steps they would cost spills)
            asm volatile("" : "+v"(gs));
            double glo[7], ghi[7];
#pragma unroll
            for (int e = 0; e < 7; ++e) {
                glo[e] = gs[e * kWave];
                ghi[e] = gs[(7 + e) * kWave];
            }
            const double tmid = gs[14 * kWave], iw = gs[15 * kWave];
#pragma unroll
            for (int j = 0; j < kPts; ++j) {
                const PointConst &q = ps[j];
                double g[7];
                const bool lo = q.T < tmid;
#pragma unroll
                for (int e = 0; e < 7; ++e) g[e] = lo ? glo[e] : ghi[e];
                const double ak = q.P0 * kexp(-gibbs(g, q.T, q.lnT, q.invT));
                const double Ck = Yt[k * ys + j] * iw * q.cf;
                double *pr = pairs + 2 * (ns + 1) * j + 2 * k;
                pr[0] = ak;
                pr[1] = Ck * krcp(ak);
            }
        }
    }
    wave_sync();
    // the point of this lane in phase 2
    const PointConst &ql = pc[jl];  // LDS (a lane-dependent index)
    const PtVals qv{ql.T, ql.lnT, ql.invT, ql.M, ql.lnp};

    // ---- phases 2 and 3, one chunk of reactions at a time
    double acc[kSpl][kPts], cmp[kSpl][kPts];
#pragma unroll
    for (int s = 0; s < kSpl; ++s)
#pragma unroll
        for (int j = 0; j < kPts; ++j) acc[s][j] = cmp[s][j] = 0.0;
    for (int c = 0; c < m.nchunks; ++c) {
        const int base = c * m.chunk;
        const int cnt = min(m.chunk, m.nr - base);
        // 48-byte reaction records as three 16-byte loads, the next
        // iteration's record in flight while this one is evaluated
        const uint4 *rsrc = reinterpret_cast<const uint4 *>(m.rxn + base);
        RxnWords w;
        w.w0 = w.w1 = w.w2 = make_uint4(0, 0, 0, 0);
        if (rl < cnt) {
            w.w0 = rsrc[3 * rl];
            w.w1 = rsrc[3 * rl + 1];
            w.w2 = rsrc[3 * rl + 2];
        }
        for (int r = rl; r < cnt; r += kWave / 2) {
            const RxnWords cur = w;
            const int rn = r + kWave / 2;
            if (rn < cnt) {
                w.w0 = rsrc[3 * rn];
                w.w1 = rsrc[3 * rn + 1];
                w.w2 = rsrc[3 * rn + 2];
            }
            sq[2 * r + jl] = rate_of_progress<MIXED>(m, cur, pbl, qv);
        }
        wave_sync();
        gather_split<MIXED, DIRECT>(m, c, gw, lane, qb, acc, cmp);
        wave_sync();
    }
#pragma unroll
    for (int s = 0; s < kSpl; ++s) {
        const int k = lane + kWave * s;
        if (k < ns) {
#pragma unroll
            for (int j = 0; j < kPts; ++j)
                Yt[k * ys + j] = MIXED ? acc[s][j] + cmp[s][j] : acc[s][j];
        }
    }
    __syncthreads();
    for (int e = lane; e < ns * kPts; e += kWave) {
        const int k = e / kPts, c = e % kPts;
        if (c < npts) wdot[(int64_t)k * ld + i0 + c] = Yt[k * ys + c];
    }
    __syncthreads();  // the LDS tile may be reused by the next tile
}

// Workgroups are dispatched to the eight XCDs round-robin (workgroup b runs on
// XCD b mod 8).  This bijection gives each XCD one contiguous range of tiles,
// so neighbouring tiles -- which share cache lines of Y and wdot -- meet in the
// same L2.
__device__ __forceinline__ unsigned xcd_tile(unsigned b, unsigned nblk)
{
    constexpr unsigned kXcd = 8;
    const unsigned x = b % kXcd, q = nblk / kXcd, r = nblk % kXcd;
    return x * q + min(x, r) + b / kXcd;
}

// DIRECT: the gather lists' offsets are LDS addresses, which holds when the
// kernel has no static LDS (its dynamic LDS then starts at address 0); the
// host checks the kernel's static LDS size and launches the DIRECT = false
// instance otherwise.
template <bool MIXED, bool DIRECT>
__global__ __launch_bounds__(kWave, 2) void rates_kernel(MechDev m, int64_t n,
                                                      const double *__restrict__ T,
                                                      const double *__restrict__ P,
                                                      const double *__restrict__ Y,
                                                      double *__restrict__ wdot)
{
    const int64_t i0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * kPts;
    const int np = (int)min((int64_t)kPts, n - i0);
    rates_tile<MIXED, DIRECT>(threadIdx.x, m, n, i0, np, T, P, Y, wdot);
}

// Batched requests.  The batch's tiles are split into kXcds contiguous ranges,
// one per XCD (workgroup b runs on XCD b mod kXcds); a workgroup takes tiles
// of its own XCD's range from that range's counter (kTicketTiles consecutive
// tiles per ticket), so neighbouring tiles --
// which share cache lines of Y and wdot -- meet in the same L2 as in a direct
// launch, and then helps with the other ranges in turn.  Every workgroup
// exits after the last range is exhausted.  Tile t belongs to the last item
// whose first tile is <= t.
//
// Tiles per ticket: a ticket's atomic returns after the wave's next memory
// wait (the wait counter is in order), so each ticket costs the wave about one
// atomic round trip; four tiles per ticket spread it.
constexpr int kTicketTiles = 4;

template <bool MIXED, bool DIRECT>
__global__ __launch_bounds__(kWave, 2) void rates_batch_kernel(MechDev m,
                                                            const WorkList *__restrict__ wl,
                                                            int *__restrict__ counter)
{
    const int ntiles = wl->ntiles[0];
    const int x0 = (int)(blockIdx.x % kXcds);
    int r = 0;  // item of the previous tile
    for (int step = 0; step < kXcds; ++step) {
        const int x = (x0 + step) % kXcds;
        const int lo = (int)((int64_t)ntiles * x / kXcds);
        const int hi = (int)((int64_t)ntiles * (x + 1) / kXcds);
        int tn = 0;
        if (threadIdx.x == 0) tn = atomicAdd(counter + x, 1);
        int t0 = 0, k = kTicketTiles;  // tiles t0 .. t0 + kTicketTiles - 1 of a ticket
        for (;;) {
            if (k == kTicketTiles) {
                t0 = lo + kTicketTiles * __builtin_amdgcn_readfirstlane(tn);  // lane 0's ticket
                k = 0;
                // the next ticket is taken now, so its round trip overlaps these tiles
                if (t0 < hi && threadIdx.x == 0) tn = atomicAdd(counter + x, 1);
            }
            const int t = t0 + k++;
            if (t >= hi) break;
            r = work_item_of(wl, 0, t, r);
            const WorkItem it = wl->items[r];
            const int64_t i0 = (int64_t)(t - wl->start[0][r]) * kPts;
            const int np = (int)min((int64_t)kPts, it.n - i0);
            int lane;
            asm volatile("v_mov_b32 %0, %1" : "=v"(lane) : "v"((int)threadIdx.x));
            rates_tile<MIXED, DIRECT>(lane, m, it.n, i0, np, it.T, it.p, it.Y, it.wdot);
        }
    }
}

// Batched requests, one tile per workgroup (grid = the batch's tiles, mapped
// to XCDs as in a direct launch; the item of tile t by work_item_ballot).
// Persistent workgroups that take tickets measured about a tenth slower per
// tile than this one-tile form.
template <bool MIXED, bool DIRECT>
__global__ __launch_bounds__(kWave, 2) void rates_items_kernel(
    MechDev m, const WorkList *__restrict__ wl)
{
    const int ntiles = wl->ntiles[0];
    const int t = (int)xcd_tile(blockIdx.x, gridDim.x);
    if (t >= ntiles) return;
    const int r = work_item_ballot(wl, 0, t);
    const WorkItem it = wl->items[r];
    const int64_t i0 = (int64_t)(t - wl->start[0][r]) * kPts;
    const int np = (int)min((int64_t)kPts, it.n - i0);
    rates_tile<MIXED, DIRECT>(threadIdx.x, m, it.n, i0, np, it.T, it.p, it.Y, it.wdot);
}

// ---------------------------------------------------------------------------
// One lane per point (mechanisms of up to kWideMaxSpecies species, see
// kx_wide.h): one tile of 64 points by NW waves.
template <bool MIXED, int NW>
__device__ __forceinline__ void rates_wide_tile(const MechDev &m, int64_t ld, int64_t i0, int npts,
                                                const double *__restrict__ T,
                                                const double *__restrict__ P,
                                                const double *__restrict__ Y,
                                                double *__restrict__ wdot)
{
    extern __shared__ double lds[];
    const WideTile<NW> t(m, m.wmaps[NW == 16 ? (MIXED ? 1 : 2) : 0], i0, npts);
    const Exp2 ex;
    const WidePoint q = species_rows<MIXED, NW, false>(ex, m, t, ld, T, P, Y, lds);
    rates_of_rows<MIXED, NW, false>(ex, m, t, q, ld, lds, wdot);
}

template <bool MIXED, int NW>
__global__ __launch_bounds__(NW *kWave, wide_waves(NW)) void rates_wide_kernel(
    MechDev m, int64_t n, const double *__restrict__ T, const double *__restrict__ P,
    const double *__restrict__ Y, double *__restrict__ wdot)
{
    const int64_t i0 = (int64_t)blockIdx.x * kRow;
    rates_wide_tile<MIXED, NW>(m, n, i0, (int)min((int64_t)kRow, n - i0), T, P, Y, wdot);
}

// Batched requests, one tile per workgroup.  YX: more tiles than one grid dimension
// takes, kYX in each row of a two-dimensional grid (an instance of its own, see
// launch_tiles).
constexpr int kYX = 1 << 21;
template <bool MIXED, int NW, bool YX>
__global__ __launch_bounds__(NW *kWave, wide_waves(NW)) void rates_wide_items_kernel(
    MechDev m, const WorkList *__restrict__ wl)
{
    const int t = (int)(YX ? blockIdx.y * kYX + blockIdx.x : blockIdx.x);
    if (t >= wl->ntiles[0]) return;
    const int r = work_item_ballot(wl, 0, t);
    const WorkItem it = wl->items[r];
    const int64_t i0 = (int64_t)(t - wl->start[0][r]) * kRow;
    rates_wide_tile<MIXED, NW>(m, it.n, i0, (int)min((int64_t)kRow, it.n - i0), it.T, it.p,
                                it.Y, it.wdot);
}

// Batched requests, persistent workgroups taking one tile at a time from one
// counter (a tile is 64 points by NW waves, so its ticket costs little).
template <bool MIXED, int NW>
__global__ __launch_bounds__(NW *kWave, wide_waves(NW)) void rates_wide_batch_kernel(
    MechDev m, const WorkList *__restrict__ wl, int *__restrict__ counter)
{
    __shared__ int tile;
    const int ntiles = wl->ntiles[0];
    int r = 0;  // item of the previous tile
    for (;;) {
        __syncthreads();  // the previous tile's LDS reads are done
        if (threadIdx.x == 0) tile = atomicAdd(counter, 1);
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(tile);
        if (t >= ntiles) break;
        r = work_item_of(wl, 0, t, r);
        const WorkItem it = wl->items[r];
        const int64_t i0 = (int64_t)(t - wl->start[0][r]) * kRow;
        rates_wide_tile<MIXED, NW>(m, it.n, i0, (int)min((int64_t)kRow, it.n - i0), it.T,
                                    it.p, it.Y, it.wdot);
    }
}

size_t wide_lds_bytes(const MechDev &m, int precision, int nw)
{
    const WideMap &wm = m.wmaps[nw == 16 ? (precision == KX_MIXED ? 1 : 2) : 0];
    return sizeof(double) * kRow * (2 * (size_t)(m.ns + 2) + (size_t)wm.chunk + 1);
}

// Waves per workgroup for a launch of `tiles` tiles: all 16 a workgroup can have
// when every tile gets a CU of its own (the tile's latency is then all that
// counts), else the number the mechanism's LDS share was laid out for.  A point's
// results do not depend on it.
int wide_launch_waves(const MechDev &m, int64_t tiles) { return tiles <= 256 ? 16 : m.wnw; }

// The instance of a wide kernel for a precision and number of waves.  FORM 0:
// direct launch, 1: work-stealing batch, 2: one tile per workgroup, 3: the same over
// two grid dimensions.
template <int FORM, bool MIXED, int NW> const void *wide_instance()
{
    if (FORM == 1) return (const void *)rates_wide_batch_kernel<MIXED, NW>;
    if (FORM >= 2) return (const void *)rates_wide_items_kernel<MIXED, NW, FORM == 3>;
    return (const void *)rates_wide_kernel<MIXED, NW>;
}

template <int FORM> const void *wide_kernel(int precision, int nw)
{
    auto pick = [&](auto mixed) {
        constexpr bool M = decltype(mixed)::value;
        return nw == 4    ? wide_instance<FORM, M, 4>()
               : nw == 8  ? wide_instance<FORM, M, 8>()
               : nw == 12 ? wide_instance<FORM, M, 12>()
                          : wide_instance<FORM, M, 16>();
    };
    return precision == KX_MIXED ? pick(std::true_type{}) : pick(std::false_type{});
}

template <int FORM>
kx_status launch_wide(const MechDev &m, int precision, int nw, int64_t grid, void **args,
                      hipStream_t s, const char *what)
{
    const void *kern = wide_kernel<FORM>(precision, nw);
    const size_t lds = wide_lds_bytes(m, precision, nw);
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute (rates)");
    const dim3 g = FORM == 3 ? dim3(kYX, (unsigned)((grid + kYX - 1) / kYX)) : dim3((unsigned)grid);
    e = hipLaunchKernel(kern, g, dim3(nw * kWave), args, lds, s);
    if (e != hipSuccess) return hip_fail(e, what);
    return ok();
}

// ---------------------------------------------------------------------------
// One point per workgroup (kx_few.h), for calls of few points.
size_t few_lds_bytes(const MechDev &m)
{
    return sizeof(AB) * ((size_t)m.ns + 2) + sizeof(double) * ((size_t)m.nr + 1 + 4);
}

#pragma float_control(push)
#pragma clang fp contract(off)
template <bool MIXED, int NT>
__device__ __forceinline__ void rates_few_point(const MechDev &m, const FewDev &f, int64_t i,
                                                int64_t ld,
                                                const double *__restrict__ T,
                                                const double *__restrict__ P,
                                                const double *__restrict__ Y,
                                                double *__restrict__ wdot)
{
    extern __shared__ double lds[];
    const int ns = m.ns, nr = m.nr, tid = threadIdx.x;
    AB *sp = reinterpret_cast<AB *>(lds);
    double *R = reinterpret_cast<double *>(sp + ns + 2);  // [nr + 1]
    const Exp2 ex;
    const WidePoint q = few_species<MIXED, false, NT>(ex, m, i, ld, T, P, Y, sp, R + nr + 1);
    KX_CONST DevWide *rx = const_table(MIXED ? m.wrx32 : m.wrx);
    for (int r = tid; r < nr; r += NT) {
        const WideTerms t = reaction_wide<MIXED>(ex, m, rx + r, PointPairs{sp}, q);
        R[r] = t.ckf * t.A * (t.Bf - t.Br);
    }
    if (tid == 0) R[nr] = 0.0;
    __syncthreads();
    for (int k = tid; k < ns; k += NT)
        wdot[(int64_t)k * ld + i] = few_gather<MIXED>(f.ent, f.ptr[k], f.ptr[k + 1], R);
}
#pragma float_control(pop)

template <bool MIXED, int NT>
__global__ __launch_bounds__(NT, 4) void rates_few_kernel(MechDev m, FewDev f, int64_t ld,
                                                          const double *__restrict__ T,
                                                          const double *__restrict__ P,
                                                          const double *__restrict__ Y,
                                                          double *__restrict__ wdot)
{
    rates_few_point<MIXED, NT>(m, f, blockIdx.x, ld, T, P, Y, wdot);
}

// Batched requests of few points together: a tile is a point.
template <bool MIXED, int NT>
__global__ __launch_bounds__(NT, 4) void rates_few_items_kernel(MechDev m, FewDev f,
                                                                const WorkList *__restrict__ wl)
{
    const int t = (int)blockIdx.x;
    if (t >= wl->ntiles[0]) return;
    const int r = work_item_ballot(wl, 0, t);
    const WorkItem it = wl->items[r];
    rates_few_point<MIXED, NT>(m, f, t - wl->start[0][r], it.n, it.T, it.p, it.Y, it.wdot);
}

template <bool ITEMS, bool MIXED, int NT> const void *few_instance()
{
    return ITEMS ? (const void *)rates_few_items_kernel<MIXED, NT>
                 : (const void *)rates_few_kernel<MIXED, NT>;
}

template <bool ITEMS>
kx_status launch_few(const MechDev &m, int precision, int nt, int64_t points, void **args,
                     hipStream_t s)
{
    auto pick = [&](auto mixed) {
        constexpr bool M = decltype(mixed)::value;
        return nt == 64    ? few_instance<ITEMS, M, 64>()
               : nt == 128 ? few_instance<ITEMS, M, 128>()
               : nt == 256 ? few_instance<ITEMS, M, 256>()
                           : few_instance<ITEMS, M, 512>();
    };
    const void *kern = precision == KX_MIXED ? pick(std::true_type{}) : pick(std::false_type{});
    const size_t lds = few_lds_bytes(m);
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute (rates)");
    e = hipLaunchKernel(kern, dim3((unsigned)points), dim3(nt), args, lds, s);
    if (e != hipSuccess) return hip_fail(e, "rates kernel launch");
    return ok();
}

// Threads per point of a call of `points` points, 0: tiles of 64 points.  A tile's
// chain grows with the number of reactions, a point's hardly does, so the line
// depends on it (FP64, us a call, one point per workgroup / tiles): 9 species (21
// reactions) 7.0 / 6.6 at any size; 17 (119) 8.1 / 10.1 at 2000 points, 11.2 / 10.1
// at 4096; 53 (371) 6.6 / 22.7 at 1 point, 9.0 / 23.1 at 1000, 18.9 / 23.2 at 4096,
// 25.6 / 23.3 at 5000; 128 (896) 8.1 / 64.6 at 1 point, 37 / 66 at 4096.  Above 120
// species a tile has so few rate rows that points past what the CUs hold at once pay:
// 128 (896), 5000 points 53 / 66, 6000 55 / 66 (mixed 62 / 68), 7000 60 / 66 (69 / 68);
// 128 (1231), 6144 points 73 / 87 (86 / 90); 128 (2500), 5000 points 138 / 166 (162 /
// 172), 6144 173 / 166; not 100 (700), 6000 points 45 / 45 (52 / 45).  Nor do up to 4096
// have to be resident at once where the reactions' LDS leaves fewer places: 128 (1231),
// 4096 points 60 / 87 (68 / 89), 53 (2000) 74 / 101 (96 / 119).
int rates_few_threads(const MechDev &m, int64_t points)
{
    const size_t lds = few_lds_bytes(m);
    if (m.wnw == 0 || m.nr <= 64 || lds > 160 * 1024) return 0;
    const int64_t most = m.nr <= 160 ? 2048 : m.ns <= 120 ? 4096 : m.nr <= 1280 ? 6144 : 5120;
    if (points > most) return 0;
    const int nt = few_threads(points, lds);
    return nt ? nt : kWave;
}

// Points at the end of a call of n points that go one to a workgroup, after tiles
// on every CU: a few tiles more than CUs cost a second round (one workgroup per CU)
// or take the CUs' shared shape, which is slower per tile.  FP64, us a call with /
// without: 57 species, 16500 points 33.7 / 49.8; 128 species
// 77 / 131; 53 species 31 / 40 (17 species 16.9 / 14.6, hence the number of reactions).
int64_t rates_tail(const MechDev &m, int64_t n)
{
    const int64_t tail = n - 256 * kRow;
    const int64_t most = m.wnw == 16 ? 4096 : (m.nr > 300 ? 2048 : 0);
    return tail > 0 && tail <= most && rates_few_threads(m, tail) ? tail : 0;
}

size_t rates_lds_bytes(const MechDev &m)
{
    return sizeof(double) * (2 * (size_t)(m.chunk + 1) + 2 * (size_t)kPts * (m.ns + 1) +
                             8 * kPts + (size_t)m.ns * (kPts + 1));
}

}  // namespace

int rates_tile_points(const MechDev &m)
{
    return m.wnw ? kRow : kPts;
}

int rates_items_tile_points(const MechDev &m, int64_t points)
{
    return rates_few_threads(m, points) ? 1 : rates_tile_points(m);
}

namespace {
template <class K>
kx_status set_lds(K kern, size_t lds)
{
    hipError_t e = hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute (rates)");
    return KX_OK;
}

// The instance to launch: the DIRECT one when it has no static LDS.
template <class K>
K pick_direct(K direct, K indirect)
{
    hipFuncAttributes a;
    if (hipFuncGetAttributes(&a, (const void *)direct) == hipSuccess && a.sharedSizeBytes == 0)
        return direct;
    return indirect;
}

}  // namespace

kx_status launch_rates(const kx_mech *mech, int64_t n, const double *T, const double *p,
                       const double *Y, double *wdot, int precision, hipStream_t s)
{
    const MechDev &m = mech->dev;
    if (m.wnw) {
        const int64_t tail = rates_few_threads(m, n) ? n : rates_tail(m, n), body = n - tail;
        const int64_t nblk = (body + kRow - 1) / kRow;
        if (nblk > 0x7fffffff) return fail(KX_EINVAL, "production rates: n too large");
        if (body) {  // whole tiles if there is a tail
            const int nw = wide_launch_waves(m, nblk);
            kx_status st = launch_tiles(body, kRow, nw * kWave, [&](int64_t i, int64_t groups) {
                const double *Ti = T + i, *pi = p + i, *Yi = Y + i;
                double *wi = wdot + i;
                void *args[] = {(void *)&m, (void *)&n, (void *)&Ti, (void *)&pi, (void *)&Yi, (void *)&wi};
                return launch_wide<0>(m, precision, nw, groups, args, s, "rates kernel launch");
            });
            if (st != KX_OK || !tail) return st;
        }
        T += body, p += body, Y += body, wdot += body;
        void *args[] = {(void *)&m, (void *)&mech->few, (void *)&n,   (void *)&T,
                        (void *)&p, (void *)&Y,         (void *)&wdot};
        return launch_few<false>(m, precision, rates_few_threads(m, tail), tail, args, s);
    }
    const size_t lds = rates_lds_bytes(m);
    if (lds > 160 * 1024)
        return fail(KX_EUNSUPPORTED, "production rates: mechanism too large for LDS");
    const int64_t nblk = (n + kPts - 1) / kPts;
    if (nblk > 0x7fffffff) return fail(KX_EINVAL, "production rates: n too large");
    auto pick = [&](auto mixed) {
        constexpr bool M = decltype(mixed)::value;
        return pick_direct(rates_kernel<M, true>, rates_kernel<M, false>);
    };
    auto kern = precision == KX_MIXED ? pick(std::true_type{}) : pick(std::false_type{});
    kx_status st = set_lds(kern, lds);
    if (st != KX_OK) return st;
    return launch_tiles(n, kPts, kWave, [&](int64_t i, int64_t groups) {
        hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(kWave), lds, s, m, n, T + i, p + i,
                           Y + i, wdot + i);
        hipError_t e = hipGetLastError();
        return e != hipSuccess ? hip_fail(e, "rates kernel launch") : KX_OK;
    });
}

namespace {
auto pick_batch(int precision)
{
    auto pick = [&](auto mixed) {
        constexpr bool M = decltype(mixed)::value;
        return pick_direct(rates_batch_kernel<M, true>, rates_batch_kernel<M, false>);
    };
    return precision == KX_MIXED ? pick(std::true_type{}) : pick(std::false_type{});
}
auto pick_items(int precision)
{
    auto pick = [&](auto mixed) {
        constexpr bool M = decltype(mixed)::value;
        return pick_direct(rates_items_kernel<M, true>, rates_items_kernel<M, false>);
    };
    return precision == KX_MIXED ? pick(std::true_type{}) : pick(std::false_type{});
}
}  // namespace

kx_status launch_rates_items(const MechDev &m, const FewDev *few, const WorkList *wl,
                             int64_t ntiles, int precision, hipStream_t s)
{
    if (ntiles <= 0) return ok();
    if (ntiles > 0x7fffffff) return fail(KX_EINVAL, "production rates: too many tiles");
    if (few) {
        void *args[] = {(void *)&m, (void *)few, (void *)&wl};
        return launch_few<true>(m, precision, rates_few_threads(m, ntiles), ntiles, args, s);
    }
    if (m.wnw) {
        void *args[] = {(void *)&m, (void *)&wl};
        const int nw = wide_launch_waves(m, ntiles);
        return ntiles <= max_workgroups(nw * kWave)
                   ? launch_wide<2>(m, precision, nw, ntiles, args, s, "rates items kernel launch")
                   : launch_wide<3>(m, precision, nw, ntiles, args, s, "rates items kernel launch");
    }
    if (ntiles > max_workgroups(kWave))
        return fail(KX_EINVAL, "production rates: too many tiles");
    const size_t lds = rates_lds_bytes(m);
    if (lds > 160 * 1024)
        return fail(KX_EUNSUPPORTED, "production rates: mechanism too large for LDS");
    auto kern = pick_items(precision);
    kx_status st = set_lds(kern, lds);
    if (st != KX_OK) return st;
    hipLaunchKernelGGL(kern, dim3((unsigned)ntiles), dim3(kWave), lds, s, m, wl);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "rates items kernel launch");
    return ok();
}

kx_status prepare_rates_batch(const MechDev &m, int precision)
{
    if (m.wnw) {
        hipError_t e = hipFuncSetAttribute(wide_kernel<1>(precision, m.wnw),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)wide_lds_bytes(m, precision, m.wnw));
        if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute (rates)");
        return KX_OK;
    }
    const size_t lds = rates_lds_bytes(m);
    if (lds > 160 * 1024)
        return fail(KX_EUNSUPPORTED, "production rates: mechanism too large for LDS");
    return set_lds(pick_batch(precision), lds);
}

kx_status launch_rates_batch(const MechDev &m, const WorkList *wl, int *counter, int precision,
                             int grid, hipStream_t s)
{
    if (m.wnw) {
        void *args[] = {(void *)&m, (void *)&wl, (void *)&counter};
        // as many workgroups as the CUs hold: one of 16 waves, or 24 waves (53 species,
        // 65536 points 121 -> 103 us against 16 waves a CU, 100000 points 176 -> 147; 24
        // species 60000 points 51 -> 47); of the smallest mechanisms' groups of four
        // waves, whose tiles are over soonest, 16 (9 species, 100000 points 37 us, with
        // 24 waves 40)
        const int groups = 256 * (m.wnw == 16 ? 1 : (m.wnw == 4 ? 4 : 24 / m.wnw));
        hipError_t e = hipLaunchKernel(wide_kernel<1>(precision, m.wnw), dim3(groups),
                                       dim3(m.wnw * kWave), args, wide_lds_bytes(m, precision, m.wnw), s);
        if (e != hipSuccess) return hip_fail(e, "rates batch kernel launch");
        return ok();
    }
    const size_t lds = rates_lds_bytes(m);
    hipLaunchKernelGGL(pick_batch(precision), dim3(grid), dim3(kWave), lds, s, m, wl,
                       counter);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "rates batch kernel launch");
    return ok();
}

}  // namespace kx
