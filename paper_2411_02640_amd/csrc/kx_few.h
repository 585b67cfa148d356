// kx_few.h -- one point per workgroup: the evaluation of kx_wide.h with the lanes
// over the species, then over the reactions, then over the species' lists of
// rates, for calls of few points.
//
// Every value of a point comes from the same operations in the same order as in
// the one-lane-per-point kernels (the functions are shared, the sums run over the
// same terms one after another), so a point's results do not depend on the form
// that the number of points selects.
//
// A tile of 64 points is one chain of nr / 16 reactions per wave, however few of
// its lanes are in use; here a point's chain is nr / NT reactions and the longest
// list, and a call of n points has n workgroups.  The tables come through the
// vector cache, once per point instead of once per 64.
//
// The rule (few_threads): as many threads per point as leave every wave of the call
// resident at once -- 16 per CU, what the kernels' 128 registers allow, fewer where
// the LDS does.  Measured, 53 species with 6 QSS species, us a call by 512 / 256 /
// 128 / 64 threads: 1 point 9.4 / 10.1 / 10.7 / 13.4; 1000 points 20.4 / 12.4 /
// 12.9 / 15.0; 4096 points 77 / 44 / 31 / 25 (one lane per point: 34 at all three).
#pragma once

#include <algorithm>

#include "kx_wide.h"

namespace kx {

// Threads per point for a call of n points whose workgroups take `lds` bytes; 0: too
// many points for one wave each to be resident at once.
inline int few_threads(int64_t n, size_t lds)
{
    for (int nt = 512; nt >= kWave; nt /= 2)
        if (n <= 256 * (int64_t)std::min<size_t>(16 * kWave / nt, 160 * 1024 / lds)) return nt;
    return 0;
}

#pragma float_control(push)
#pragma clang fp contract(off)

// {a, b} of one point, ns + 2 pairs (kx_wide.h's dummy species included).
struct PointPairs {
    const AB *sp;
    __device__ __forceinline__ AB pair(unsigned k) const { return sp[k]; }
    __device__ __forceinline__ double b(unsigned k) const { return sp[k].b; }
};

// Point constants and pairs of point i (species_rows of kx_wide.h); `part` holds
// four doubles.
template <bool MIXED, bool QSS, int NT>
__device__ __forceinline__ WidePoint few_species(const Exp2 &ex, const MechDev &m, int64_t i,
                                                 int64_t ld, const double *__restrict__ T,
                                                 const double *__restrict__ P,
                                                 const double *__restrict__ Y, AB *sp, double *part)
{
    const int ns = m.ns, tid = threadIdx.x;
    WidePoint q;
    q.T = T[i];
    const double p = P[i];
    const double l2T = kl2(q.T);
    q.L = MIXED ? kln(q.T) : l2T;
    q.invT = krcp(q.T);
    const double invRT = krcp(kRu * q.T);
    q.M = p * invRT;
    q.lnp = m.nplog ? kln(p) : 0.0;
    const double P0 = kPatm * invRT;
    for (int k = tid; k < ns; k += NT) {
        KX_CONST double *g = const_table(m.wsp) + 16 * k;
        const double iw = g[15], y = Y[(int64_t)k * ld + i];
        const double t = q.T;
        KX_CONST double *c = t < g[14] ? g : g + 7;
        const double poly = fma(t, fma(t, fma(t, c[4], c[3]), c[2]), c[1]);
        const double e = fma(t, poly, fma(c[5], q.invT, fma(c[0], l2T, c[6])));
        sp[k] = AB{QSS && iw == 0.0 ? 0.0 : y * iw, P0 * ex(e)};
    }
    __syncthreads();
    if (tid < 4) {
        double sum = 0.0;
        for (int k = tid; k < ns; k += 4) sum += sp[k].a;
        part[tid] = sum;
    }
    __syncthreads();
    const double cf = q.M * krcp((part[0] + part[1]) + (part[2] + part[3]));
    for (int k = tid; k < ns; k += NT) {
        const AB v = sp[k];  // {Y / W, a}
        double C = v.a * cf;
        if (QSS && const_table(m.wsp)[16 * k + 15] == 0.0) C = 1.0;
        sp[k] = AB{v.b, C * krcp(v.b)};
    }
    if (tid == 0) {
        sp[ns] = AB{1.0, 1.0};
        sp[ns + 1] = AB{1.0, 0.0};
    }
    __syncthreads();
    return q;
}

// The sum of +-1 times the values that a list of words [w0, w1) names, in list
// order (the mixed path: compensated at every entry that ends a group of
// gather_stream's).
template <bool MIXED>
__device__ __forceinline__ double few_gather(const uint4 *__restrict__ list, int w0, int w1,
                                             const double *R)
{
    double acc = 0.0, cmp = 0.0, t = 0.0;
    const uint4 none = make_uint4(0, 0, 0, 0);
    uint4 c0 = w0 < w1 ? list[w0] : none, c1 = w0 + 1 < w1 ? list[w0 + 1] : none;
    for (int w = w0; w < w1; ++w) {
        const uint32_t e[4] = {c0.x, c0.y, c0.z, c0.w};
        c0 = c1;
        if (w + 2 < w1) c1 = list[w + 2];
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = R[e[u] & kFewIndex];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double nu = (e[u] & kFewMinus) ? -1.0 : 1.0;
            if (MIXED) {
                t = fma(v[u], nu, t);
                if (e[u] & kFewLast) {
                    accumulate<true>(acc, cmp, t);
                    t = 0.0;
                }
            } else {
                acc = fma(v[u], nu, acc);
            }
        }
    }
    return MIXED ? acc + cmp : acc;
}

#pragma float_control(pop)
}  // namespace kx
