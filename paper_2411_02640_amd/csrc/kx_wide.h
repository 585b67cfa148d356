// kx_wide.h -- the one-lane-per-point evaluation of the rates of progress,
// shared by the kernels for mechanisms of up to kWideMaxSpecies species.
//
// A workgroup of several waves owns 64 points; lane = point in every phase, and
// the waves divide the species and the reactions among themselves.  Every
// species and every reaction is therefore wave-uniform: its constants come
// through the scalar cache as instruction operands, its type is a scalar branch
// (no lane idles because a neighbour's reaction has another type), LDS rows
// are 64 consecutive doubles (no bank conflicts) and Y and wdot rows are read
// and written as 512-byte segments without staging.
//
// LDS of a workgroup (rows of 64 doubles, lane = point):
//   species rows, two per species k = 0 .. ns + 1: a_k, then b_k (see
//     kx_rates.hip); species ns is the dummy of unused molecule slots
//     (a = b = 1), species ns + 1 the products of irreversible reactions
//     (a = 1, b = 0);
//   rate rows, WideMap::chunk + 1: R of the current chunk's reactions and one row of
//     zeros that absorbs the padding of the gather lists.
#pragma once

#include <float.h>

#include "kx_internal.h"
#include "kx_math.h"

namespace kx {

// exp(x) for the mixed path: the argument stays in FP64, is reduced by n ln 2
// in FP64 and only exp(r), |r| <= ln2/2, is evaluated in FP32.
__device__ __forceinline__ double exp_mixed(double x)
{
    const double nd = rint(x * 1.4426950408889634);
    const double r = fma(-nd, 6.93147180559945286e-01, x);
    const float er = __expf((float)r);
    return ldexp((double)er, (int)nd);
}

// log10 of a positive double over its whole range, in FP32 arithmetic.
__device__ __forceinline__ float log10_wide(double v)
{
    int ex;
    const double mant = frexp(fmax(v, DBL_MIN), &ex);
    return (__log2f((float)mant) + (float)ex) * 0.30102999566398120f;
}

template <bool MIXED>
__device__ __forceinline__ void accumulate(double &acc, double &cmp, double t)
{
    if (MIXED) {
        const double sum = acc + t;
        cmp += (fabs(acc) >= fabs(t)) ? (acc - sum) + t : (t - sum) + acc;
        acc = sum;
    } else {
        acc += t;
    }
}

// the FP64 steps round the same way in every instance (number of waves, batch
// or direct launch): fused multiply-adds only where written
#pragma float_control(push)
#pragma clang fp contract(off)

constexpr int kRow = 64;           // doubles per LDS row and point of a lane
// Waves per SIMD the kernels are compiled for (16 waves: one workgroup per CU).
constexpr int wide_waves(int nw) { return nw == 16 ? 4 : 6; }
// Species per wave of a workgroup of nw waves, at most.
constexpr int wide_species(int nw) { return nw == 16 ? 8 : (nw == 12 ? 5 : 4); }

// This lane's value in row `row` of the rows that start at `lds` (the sign bit of
// a gather entry leaves with the shift).
__device__ __forceinline__ double row_val(const double *lds, unsigned row, unsigned lane8)
{
    return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(lds) +
                                             ((row << 9) + lane8));
}
// a and b of a species.
struct alignas(16) AB {
    double a, b;
};
// Where a lane reads them: the species rows (lane = point, one ds_read2st64_b64
// per pair), or one point's pairs side by side (kx_few.h).
struct RowPairs {
    const double *lds;
    unsigned lane8;
    __device__ __forceinline__ AB pair(unsigned k) const
    {
        const char *p = reinterpret_cast<const char *>(lds) + ((k << 10) + lane8);
        return AB{*reinterpret_cast<const double *>(p), *reinterpret_cast<const double *>(p + 512)};
    }
    __device__ __forceinline__ double b(unsigned k) const
    {
        return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(lds) +
                                                 ((k << 10) + lane8) + 512);
    }
};

// What a lane knows about a point of its own.  L is log2 T on the FP64 path and
// ln T on the mixed path, whose FP32 exponential cores take natural arguments.
struct WidePoint {
    double T, L, invT, M, lnp;
};

// Falloff blending factor F (eq:blend), Troe and SRI:
//   Troe  log10 F = log10 F_cent / (1 + f1^2), f1 = (l + c) / (n - 0.14 (l + c)),
//         F_cent = (1 - alpha) e^(-T/T***) + alpha e^(-T/T*) [+ e^(-T**/T)],
//         c = -0.4 - 0.67 log10 F_cent, n = 0.75 - 1.27 log10 F_cent;
//   SRI   F = d T^e B^X, B = a e^(-b/T) + e^(-T/c), X = 1 / (1 + l^2),
// with l = log10 P_r, in base 2 (the table's parameters of the exponentials
// carry the factor log2 e, see DevAux of the FP64 path).
__device__ __forceinline__ double blend_base2(const Exp2 &ex, KX_CONST DevAux *ax, bool sri, const WidePoint &q,
                                              double log2Pr)
{
    constexpr double kLog10of2 = 0.30102999566398119521;
    double x, w, B;
    if (sri) {
        B = ax->fp[0] * ex(-ax->fp[1] * q.invT) + ex(-q.T * ax->fp[2]);
    } else {
        const double al = ax->fp[0];
        B = (1.0 - al) * ex(-ax->fp[1] * q.T) + al * ex(-q.T * ax->fp[2]);
        if (ax->has_T2) B += ex(-ax->fp[3] * q.invT);
    }
    const double l2B = kl2(fmax(B, DBL_MIN));
    double extra = 0.0;
    if (sri) {
        w = log2Pr * kLog10of2;
        extra = fma(ax->fp[4], q.L, ax->fp[3]);
    } else {
        const double lB = l2B * kLog10of2;
        x = fma(log2Pr, kLog10of2, fma(-0.67, lB, -0.4));
        w = x * krcp(fma(-0.14, x, fma(-1.27, lB, 0.75)));
    }
    return ex(fma(l2B, krcp(fma(w, w, 1.0)), extra));
}

// The same in FP32 from l = log10 P_r (natural parameters).
__device__ __forceinline__ float blend_F32(KX_CONST DevAux *ax, bool sri, float T, float lnT,
                                           float invT, float lPr)
{
#pragma clang fp contract(fast)
    const float a0 = (float)ax->fp[0], a1 = (float)ax->fp[1], a2 = (float)ax->fp[2];
    const float a3 = (float)ax->fp[3], a4 = (float)ax->fp[4];
    float B = (sri ? a0 : 1.0f - a0) * __expf(-a1 * (sri ? invT : T)) +
              (sri ? 1.0f : a0) * __expf(-T * a2);
    if (!sri && ax->has_T2) B += __expf(-a3 * invT);
    const float lnB = __logf(fmaxf(B, FLT_MIN));
    const float lB = lnB * 0.43429448190325182765f;
    const float x = lPr + (sri ? 0.0f : -0.4f - 0.67f * lB);
    const float nn = sri ? 1.0f : 0.75f - 1.27f * lB;
    const float w = x / (nn - (sri ? 0.0f : 0.14f) * x);
    return __expf(lnB / (1.0f + w * w) + (sri ? a4 * lnT + a3 : 0.0f));
}

// Exponent of k_f of a pressure-table reaction at ln p: linear in ln p between
// the neighbouring reference pressures, the nearest end point's value outside
// them (App. A.2, pressure-dependent reactions).  Every interval is evaluated
// and the point's one kept: the table is wave-uniform, the pressure is not.
__device__ __forceinline__ double plog_exponent_wide(KX_CONST DevPlog *pl, int cnt,
                                                     const WidePoint &q)
{
    auto at = [&](int j) { return fma(pl[j].beta, q.L, fma(-pl[j].ER, q.invT, pl[j].lnA)); };
    double xj = at(0), x = xj;
    for (int j = 0; j + 1 < cnt; ++j) {
        const double xn = at(j + 1);
        const double d = q.lnp - pl[j].lnp;
        if (d > 0.0) x = fma(xn - xj, d * pl[j].inv_dlnp, xj);
        xj = xn;
    }
    if (cnt > 1 && q.lnp >= pl[cnt - 1].lnp) x = xj;
    return x;
}

// Two 16-bit offsets of a uniform table in one word (a 16-bit load would not go
// through the scalar cache).
__device__ __forceinline__ unsigned offsets16(KX_CONST uint16_t *o, int pair)
{
    return ((KX_CONST uint32_t *)o)[pair];
}

// [X]_i = default [M] + sum over listed species of (alpha - default) C_k.
template <class Pairs>
__device__ __forceinline__ double third_body_wide(const MechDev &m, KX_CONST DevAux *ax,
                                                  const Pairs &sp, double M)
{
    double X = ax->eff_default * M;
    auto add = [&](double d, unsigned k) {
        const AB s = sp.pair(k);
        X = fma(d, s.a * s.b, X);
    };
#pragma unroll
    for (int e = 0; e < kInlineEff; e += 2) {
        if (e >= ax->eff_cnt) break;
        const unsigned o = offsets16(ax->eoff, e / 2);
        add(ax->dalpha[e], (o & 0xFFFFu) / 16u);
        add(ax->dalpha[e + 1], o >> 20);
    }
    KX_CONST DevEff *f = const_table(m.eff) + ax->ext_off;
    for (int e = 0; e < ax->ext_cnt; ++e) add(f[e].dalpha, f[e].sp);
    return X;
}

// The pieces of one reaction at this lane's point: R = ckf A' (B' - B'') with
// A' = prod_reac a, B' = prod_reac b, B'' = prod_prod b and ckf = c_i k_f.
struct WideTerms {
    double ckf, A, Bf, Br;
};

template <bool MIXED, class Pairs>
__device__ __forceinline__ WideTerms reaction_wide(const Exp2 &ex, const MechDev &m,
                                                   KX_CONST DevWide *r, const Pairs &sp,
                                                   const WidePoint &q)
{
    const unsigned meta = r->meta;
    const unsigned r01 = r->r01, p01 = r->p01;
    // the LDS reads are issued first; the exponential covers their latency
    const AB r0 = sp.pair(r01 & 0xFFFFu);
    const AB r1 = sp.pair(r01 >> 16);
    const double p0 = sp.b(p01 & 0xFFFFu);
    const double p1 = sp.b(p01 >> 16);
    KX_CONST DevAux *ax = const_table(MIXED ? m.aux : m.waux) + (meta >> 16);
    WideTerms t;
    double x;
    if (meta & kWideConst) {
        x = r->lA;
        t.ckf = r->beta;
    } else {
        if (meta & kWidePlog)
            x = plog_exponent_wide(const_table(MIXED ? m.plog : m.wplog) + ax->plog_off,
                                   ax->plog_cnt, q);
        else
            x = fma(r->beta, q.L, fma(-r->ER, q.invT, r->lA));
        t.ckf = MIXED ? exp_mixed(x) : ex(x);
    }
    t.A = r0.a * r1.a;
    t.Bf = r0.b * r1.b;
    t.Br = p0 * p1;
    if (meta & kWideThird) {
        const unsigned rp2 = r->rp2;
        const AB r2 = sp.pair(rp2 & 0xFFFFu);
        t.A *= r2.a;
        t.Bf *= r2.b;
        t.Br *= sp.b(rp2 >> 16);
    }
    if (meta & kWideOrders) {
        // explicit forward orders (irreversible): prod_k C_k^o_k, C_k = a_k b_k
        double s = 0.0;
        bool zero = false;
#pragma unroll
        for (int e = 0; e < kMaxOrd; ++e) {
            const double o = ax->oval[e];
            if (o != 0.0) {
                const unsigned w = offsets16(ax->ooff, e / 2) >> 16 * (e & 1);
                const AB c = sp.pair((w & 0xFFFFu) / 16u);
                const double C = c.a * c.b;
                zero = zero || !(C > 0.0);
                s = fma(o, kl2(fmax(C, DBL_MIN)), s);
            }
        }
        t.A = zero ? 0.0 : ex(s);
        t.Bf = 1.0;
        t.Br = 0.0;
    }
    if (meta & kWideThirdBody) {
        const double X = third_body_wide(m, ax, sp, q.M);
        double c = X;
        if (meta & kWideFalloff) {
            // P_r = k_0 [X] / k_inf = e0 [X] with e0 from the difference of the exponents
            const double d0 = fma(ax->beta0, q.L, fma(-ax->ER0, q.invT, ax->lnA0)) - x;
            const double e0 = MIXED ? exp_mixed(d0) : ex(d0);
            const double Pr = e0 * X;
            double F = 1.0;
            if (meta & (kWideTroe | kWideSri)) {
                const bool sri = (meta & kWideSri) != 0;
                if (MIXED)
                    F = (double)blend_F32(ax, sri, (float)q.T, (float)q.L, (float)q.invT,
                                          log10_wide(Pr));
                else  // log2 max(P_r, DBL_MIN) without forming the logarithm of P_r
                    F = blend_base2(ex, ax, sri, q, fmax(d0 + kl2(fmax(X, DBL_MIN)), -1022.0));
            }
            // eq:c_i: P_r/(1+P_r) F; chemically activated: F/(1+P_r) with k_0 =
            // e0 k_inf in r_i, i.e. c k_inf = e0 F/(1+P_r) k_inf
            const double g = krcp(1.0 + Pr) * F;
            c = (meta & kWideChemAct) ? e0 * g : Pr * g;
        }
        t.ckf *= c;
    }
    return t;
}

// B' - B'' of a reaction alone, as reaction_wide forms the two products.
template <class Pairs>
__device__ __forceinline__ double bracket_wide(KX_CONST DevWide *r, const Pairs &sp)
{
    const unsigned meta = r->meta, r01 = r->r01, p01 = r->p01;
    double f = sp.b(r01 & 0xFFFFu) * sp.b(r01 >> 16);
    double b = sp.b(p01 & 0xFFFFu) * sp.b(p01 >> 16);
    if (meta & kWideThird) {
        const unsigned rp2 = r->rp2;
        f *= sp.b(rp2 & 0xFFFFu);
        b *= sp.b(rp2 >> 16);
    }
    return (meta & kWideOrders) ? 1.0 : f - b;
}

// A workgroup's tile of 64 points: this lane's point (points past npts repeat
// the last one and are not stored), this wave's species, and the LDS rows.
template <int NW> struct WideTile {
    static constexpr int NS = wide_species(NW);
    const WideMap &wm;
    int lane, w;
    int64_t i;
    bool store;
    int ks[NS];  // species of this wave (-1: none)
    __device__ __forceinline__ WideTile(const MechDev &m, const WideMap &map, int64_t i0, int npts)
        : wm(map)
    {
        lane = threadIdx.x & (kWave - 1);
        w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
        i = i0 + min(lane, npts - 1);
        store = lane < npts;
#pragma unroll
        for (int s = 0; s < NS; ++s) ks[s] = const_table(wm.species)[8 * w + s];
    }
    // the rate rows
    __device__ __forceinline__ double *rates(const MechDev &m, double *lds) const
    {
        return lds + 2 * (m.ns + 2) * kRow;
    }
};

// Phase 1 of a tile: the point constants (returned) and the species rows.  Four
// of the rate rows (not yet in use) carry partial sums of Y_k / W_k: the sums are
// the same whatever the number of waves, so a point's results are too.  QSS: the
// mechanism has QSS species; their 1/W in wsp is 0 (the mixture is that of the
// transported species) and C = 1 in their rows.
template <bool MIXED, int NW, bool QSS>
__device__ __forceinline__ WidePoint species_rows(const Exp2 &ex, const MechDev &m,
                                                  const WideTile<NW> &tile, int64_t ld,
                                                  const double *__restrict__ T,
                                                  const double *__restrict__ P,
                                                  const double *__restrict__ Y, double *lds)
{
    constexpr int NS = wide_species(NW);
    const int ns = m.ns, w = tile.w, lane = tile.lane;
    const int64_t i = tile.i;
    const int(&ks)[NS] = tile.ks;
    double *part = tile.rates(m, lds);
    KX_CONST double *sp = const_table(m.wsp);
    WidePoint q;
    q.T = T[i];
    const double p = P[i];
    double y[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) y[s] = ks[s] >= 0 ? Y[(int64_t)ks[s] * ld + i] : 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (ks[s] >= 0) {
            const double iw = sp[16 * ks[s] + 15];
            y[s] = QSS && iw == 0.0 ? 0.0 : y[s] * iw;  // a QSS entry of Y does not enter
            lds[2 * ks[s] * kRow + lane] = y[s];
        }
    }
    const double l2T = kl2(q.T);
    q.L = MIXED ? kln(q.T) : l2T;
    q.invT = krcp(q.T);
    const double invRT = krcp(kRu * q.T);
    q.M = p * invRT;
    q.lnp = m.nplog ? kln(p) : 0.0;
    const double P0 = kPatm * invRT;
    __syncthreads();
    if (w < 4) {
        double sum = 0.0;
        for (int k = w; k < ns; k += 4) sum += lds[2 * k * kRow + lane];
        part[w * kRow + lane] = sum;
    }
    // log2 (a_k / P0) = -G_k / (RT ln 2) from both ranges' coefficients:
    // selecting the value costs less than selecting seven coefficients
    double a[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (ks[s] >= 0) {
            KX_CONST double *g = sp + 16 * ks[s];
            const double t = q.T;
            double e[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double poly = fma(t, fma(t, fma(t, g[7 * h + 4], g[7 * h + 3]), g[7 * h + 2]),
                                        g[7 * h + 1]);
                e[h] = fma(t, poly, fma(g[7 * h + 5], q.invT, fma(g[7 * h], l2T, g[7 * h + 6])));
            }
            a[s] = P0 * ex(t < g[14] ? e[0] : e[1]);
        }
    }
    __syncthreads();
    const double wsum = (part[lane] + part[kRow + lane]) +
                        (part[2 * kRow + lane] + part[3 * kRow + lane]);
    const double cf = q.M * krcp(wsum);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (ks[s] >= 0) {
            double C = y[s] * cf;
            if (QSS && sp[16 * ks[s] + 15] == 0.0) C = 1.0;
            double *row = lds + 2 * ks[s] * kRow + lane;
            row[0] = a[s];
            row[kRow] = C * krcp(a[s]);
        }
    }
    if (w == NW - 1) {  // the dummy species
        double *row = lds + 2 * ns * kRow + lane;
        row[0] = row[kRow] = row[2 * kRow] = 1.0;
        row[3 * kRow] = 0.0;
    }
    __syncthreads();
    return q;
}

// One chunk's part of a wave's sums: acc[s] += sum of +-1 times the rate rows
// that the stream at g lists for accumulator s; h0, h1: its header's counts.
template <bool MIXED, int NS>
__device__ __forceinline__ KX_CONST uint32_t *gather_stream(KX_CONST uint32_t *g, uint32_t h0,
                                                            uint32_t h1, const double *sq,
                                                            unsigned lane8, double (&acc)[NS],
                                                            double (&cmp)[NS])
{
    g += 4;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma clang loop unroll(disable)
        for (int n = ((s < 4 ? h0 : h1) >> 8 * (s & 3)) & 255u; n > 0; --n, g += 4) {
            double v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = row_val(sq, g[e], lane8);
            auto nu = [&](int e) { return (int)g[e] < 0 ? -1.0 : 1.0; };
            if (MIXED) {
                double t = v[0] * nu(0);
#pragma unroll
                for (int e = 1; e < 4; ++e) t = fma(v[e], nu(e), t);
                accumulate<true>(acc[s], cmp[s], t);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[s] = fma(v[e], nu(e), acc[s]);
            }
        }
    }
    return g;
}

// Phases 2 and 3: the rates of progress of every reaction from the species rows,
// chunk by chunk, and wdot.  QSS: the QSS rows of wdot are written as 0.
template <bool MIXED, int NW, bool QSS>
__device__ __forceinline__ void rates_of_rows(const Exp2 &ex, const MechDev &m,
                                              const WideTile<NW> &t, const WidePoint &q, int64_t ld,
                                              double *lds, double *__restrict__ wdot)
{
    constexpr int NS = wide_species(NW);
    const int nr = m.nr, chunk = t.wm.chunk;
    double *sq = t.rates(m, lds);
    if (t.w == 0) sq[chunk * kRow + t.lane] = 0.0;
    KX_CONST DevWide *rx = const_table(MIXED ? m.wrx32 : m.wrx);
    KX_CONST uint32_t *g =
        (KX_CONST uint32_t *)(const_table(t.wm.gather) + const_table(t.wm.start)[t.w]);
    const unsigned lane8 = 8u * (unsigned)t.lane;
    const RowPairs sp{lds, lane8};
    double acc[NS], cmp[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[s] = cmp[s] = 0.0;
    for (int c = 0; c < t.wm.nchunks; ++c) {
        const int base = c * chunk, cnt = min(chunk, nr - base);
        const uint32_t h0 = g[0], h1 = g[1];  // groups of each species
        for (int r = t.w; r < cnt; r += NW) {
            const WideTerms x = reaction_wide<MIXED>(ex, m, rx + base + r, sp, q);
            sq[r * kRow + t.lane] = x.ckf * x.A * (x.Bf - x.Br);
        }
        __syncthreads();
        g = gather_stream<MIXED>(g, h0, h1, sq, lane8, acc, cmp);
        if (c + 1 < t.wm.nchunks) __syncthreads();
    }
    if (t.store) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (t.ks[s] >= 0) {
                double x = MIXED ? acc[s] + cmp[s] : acc[s];
                if (QSS && const_table(m.qidx)[t.ks[s]] >= 0) x = 0.0;
                wdot[(int64_t)t.ks[s] * ld + t.i] = x;
            }
    }
}

#pragma float_control(pop)
}  // namespace kx
