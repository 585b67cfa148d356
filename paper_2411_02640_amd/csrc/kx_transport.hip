// kx_transport.hip -- mixture-averaged transport and mixture thermo on gfx950.
//
// Three evaluations of the same sums (App. A.3):
//  * the matrix-core kernel (tables holding fits of 1/D_kj and at least 24
//    species): the pair sums as products of fixed matrices with per-point
//    stacks on 16x16x4 MFMAs, described where it is defined below;
//  * the vector-ALU kernel (tables of D_kj fits, or fewer species): lane = point,
//    the waves of a workgroup divide the species k, whose sums they hold in
//    registers while j streams over all species; X_j and rho_j come from LDS rows,
//    every mechanism constant from scalar loads, as an instruction operand; in calls
//    of very many points one thread takes two points and all species in turn, with
//    the same sums (transport_lanes_tile);
//  * the symmetric evaluation of D_kj fits (KX_DKJ_SYMMETRIC, §2.2.2 / §2.3.2),
//    described where it is defined below.
// Common to them:
//  * pure species (App. A.3 "Polynomial fits"): eta_k, lambda_k, D_kj as
//    polynomials in u = (ln T - L0)/h (Horner), D_kj divided by p/p_atm;
//  * Wilke / Bird viscosity with phi_kj = c1_kj (1 + sigma_k rho_j)^2, where
//    c1_kj = (8 (1 + W_k/W_j))^(-1/2), sigma_k = sqrt(eta_k) / W_k^(1/4) and
//    rho_j = W_j^(1/4) / sqrt(eta_j): (W_j/W_k)^(1/4) separates into
//    per-species factors, so each pair reads one coefficient;
//  * Mathur conductivity; eq:mix_diff for D_km, the reciprocals of the
//    positive sums by v_rcp_f64 and one Newton step (about 2^-48 relative).
#include <float.h>

#include <type_traits>

#include "kx_internal.h"
#include "kx_math.h"

namespace kx {
namespace {

constexpr int kBlock = 256;

// Horner evaluation of a wave-uniform polynomial (coefficients in scalar
// registers, constant term first) at a per-lane point.
__device__ __forceinline__ double fma_u(double a, double b, double c) { return fma_s(a, b, c); }
__device__ __forceinline__ float fma_u(float a, float b, float c) { return fmaf_s(a, b, c); }

template <int ORDER, class F>
__device__ __forceinline__ F horner(const F *__restrict__ c, F u, int order)
{
    if (ORDER > 1) {
        F r = u * c[ORDER - 1] + c[ORDER - 2];
#pragma unroll
        for (int o = ORDER - 3; o >= 0; --o) r = fma_u(r, u, c[o]);
        return r;
    }
    if (ORDER == 1) return c[0];
    F r = c[order - 1];
    for (int o = order - 2; o >= 0; --o) r = fma_u(r, u, c[o]);
    return r;
}

// The same with per-lane coefficients (vector registers).
template <int ORDER, class F>
__device__ __forceinline__ F horner_v(const F *__restrict__ c, F u, int order)
{
    const int o = ORDER > 0 ? ORDER : order;
    F r = c[o - 1];
    for (int q = o - 2; q >= 0; --q) r = fma(r, u, c[q]);
    return r;
}

// Reciprocals and square roots by arithmetic type: double on the FP64 path, float
// on the mixed path.
template <class F> __device__ __forceinline__ F rcp_fast(F x);
template <> __device__ __forceinline__ double rcp_fast<double>(double x) { return krcp1(x); }
template <> __device__ __forceinline__ float rcp_fast<float>(float x)
{
    return __builtin_amdgcn_rcpf(x);
}
template <class F> __device__ __forceinline__ F rsqrt_acc(F x);
template <> __device__ __forceinline__ double rsqrt_acc<double>(double x) { return krsqrt(x); }
template <> __device__ __forceinline__ float rsqrt_acc<float>(float x) { return rsqrtf(x); }
template <class F> __device__ __forceinline__ F rcp_acc(F x);
template <> __device__ __forceinline__ double rcp_acc<double>(double x) { return krcp(x); }
template <> __device__ __forceinline__ float rcp_acc<float>(float x) { return 1.0f / x; }
// Reciprocals in the matrix-core kernel, where each result is a term of a sum
// of positive terms or a factor of one output: FP64 from v_rcp_f64 with one
// Newton step (about 2^-48 relative; FP64 vector instructions also cost the
// matrix pipe, so the second step is left out), FP32 from v_rcp_f32 with one
// Newton step (about 1 ulp, without the IEEE division's scaling and fix-up
// steps).
template <class F> __device__ __forceinline__ F rcp_mfma(F x);
template <> __device__ __forceinline__ double rcp_mfma<double>(double x) { return krcp1(x); }
template <> __device__ __forceinline__ float rcp_mfma<float>(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}

template <class F> struct Tabs;
template <> struct Tabs<double> {
    static __device__ const double *visc(const MechDev &m) { return m.visc; }
    static __device__ const double *cond(const MechDev &m) { return m.cond; }
    static __device__ const double *wq(const MechDev &m) { return m.wq; }
    static __device__ const double *wilke(const MechDev &m) { return m.wilke; }
    static __device__ const double *dfit(const MechDev &m) { return m.dfit; }
    static __device__ const double *ddiag(const MechDev &m) { return m.ddiag; }
};
template <> struct Tabs<float> {
    static __device__ const float *visc(const MechDev &m) { return m.visc32; }
    static __device__ const float *cond(const MechDev &m) { return m.cond32; }
    static __device__ const float *wq(const MechDev &m) { return m.wq32; }
    static __device__ const float *wilke(const MechDev &m) { return m.wilke32; }
    static __device__ const float *dfit(const MechDev &m) { return m.dfit32; }
    static __device__ const float *ddiag(const MechDev &m) { return m.ddiag32; }
};

// Horner with the coefficients read through the constant address space.
template <int ORDER, class F>
__device__ __forceinline__ F horner_c(KX_CONST F *c, F u, int order)
{
    const int o = ORDER > 0 ? ORDER : order;
    if (o == 1) return c[0];
    F r = fma(u, c[o - 1], c[o - 2]);
#pragma unroll
    for (int q = ORDER - 3; q >= 0; --q) r = fma_u(r, u, c[q]);
    if (ORDER == 0)
        for (int q = o - 3; q >= 0; --q) r = fma_u(r, u, c[q]);
    return r;
}

// Vector-ALU kernel: one tile of 64 points (lane = point) starting at point
// `base` of arrays with n points, by ceil(ns / RW) waves; wave w owns the species
// k = RW w .. RW w + RW - 1.  Per chunk of kRowsChunk species j the waves put X_j
// and rho_j of every j into LDS rows (each wave its share), then every wave adds
// the chunk to the Wilke and D_km sums of its species.  F is the arithmetic type
// of the fits and mixing sums (double: FP64 path; float: mixed path); KIND is the
// diffusion fit kind (0: D_kj, 1: 1/D_kj).
//
// It is bound by vector issue (about 11 FP64 operations and half a reciprocal per
// pair for kind 0: two neighbouring j share one, X1/f1 + X2/f2 = (X1 f2 + X2 f1) /
// (f1 f2)) and by the scalar stream of coefficients (48 bytes per pair and 64
// points).  The form before it (one thread per four points, all k in turn) ran a
// chain of ns^2 pairs per wave and recomputed X_j and rho_j per four species k:
// 53 species, 1000 points 803 -> 38 us, 300007 points 1240 -> 745 us.
constexpr int kRowsChunk = 32;

// Kind 0: a wave copies the coefficients of its species, kStage species j and four
// species k at a time, from the tables into LDS of its own and reads them there
// (one address per wave: a broadcast).  Through the scalar cache each pair's 48
// bytes (24 mixed) were a load the wave waited for: 200 species, 2^20 points 56 -> 39
// ms, mixed 39 -> 22; 53 species mixed 2.16 -> 1.89.  FP64 with four species per wave
// keeps the scalar loads: there the stages' LDS leaves one workgroup per CU (53
// species, 2^20 points: 2.41 ms scalar, 3.16 staged).  Calls of very many points take
// transport_lanes_tile where it is the faster form (lanes_form).
constexpr int kStage = 8;
static_assert(kRowsChunk % kStage == 0 && kStage % 2 == 0, "whole stages of pairs");

// Waves per SIMD: two workgroups of 14 waves (53 species) where the registers allow.
template <class F> constexpr int rows_min_waves(int kind, int rw)
{
    return kind == 0 && rw == 4 && sizeof(F) == 4 ? 7 : 4;
}
template <class F> __host__ __device__ constexpr bool rows_staged(int kind, int rw)
{
    return kind == 0 && (rw > 4 || sizeof(F) == 4);
}
// elements of a wave's stage: the fits [j][kStageK][order], then the Wilke factors
constexpr int kStageK = 4;
static_assert(kKB % kStageK == 0, "a stage lies in one block of the tables");
__host__ __device__ constexpr int stage_size(int order) { return kStage * kStageK * (order + 1); }

template <class F>
__host__ __device__ constexpr size_t rows_lds_bytes(int ns, int nw)  // without the stages
{
    // the waves' partial sums; X, rho (and for the mixed path lambda_j,
    // 1 / lambda_j) rows of a chunk, which later hold, with further rows, the
    // factors X_k eta_k and 1 / den_k of the mixed path's viscosity terms
    const size_t rows = (size_t)(ns < kRowsChunk ? ns : kRowsChunk) * (sizeof(F) == 8 ? 2 : 4);
    return (size_t)nw * (sizeof(F) == 8 ? 4 : 1) * kWave * sizeof(double) +
           (sizeof(F) == 8 || rows > 2 * (size_t)ns ? rows : 2 * (size_t)ns) * kWave * sizeof(F);
}

template <class F, int ORDER, int KIND, int RW>
__device__ __forceinline__ void transport_rows_tile(const MechDev &m, int64_t n, int64_t base,
                                                    const double *__restrict__ T,
                                                    const double *__restrict__ Pp,
                                                    const double *__restrict__ Y,
                                                    double *__restrict__ mu,
                                                    double *__restrict__ lam,
                                                    double *__restrict__ Dmix)
{
    using Tb = Tabs<F>;
    constexpr bool F64 = std::is_same<F, double>::value;
    constexpr int NROW = F64 ? 2 : 4;  // LDS rows per species of a chunk
    extern __shared__ double smem_d[];
    const int ns = m.ns, order = m.fit_order;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int nw = (ns + RW - 1) / RW;
    constexpr int NPART = F64 ? 4 : 1;
    double *part = smem_d + lane;
    F *rows = reinterpret_cast<F *>(smem_d + (size_t)nw * NPART * kWave) + lane;
    KX_CONST DevSpecies *sp = const_table(m.sp);
    KX_CONST double *Wt = const_table(m.W);
    KX_CONST F *visc_t = const_table(Tb::visc(m)), *cond_t = const_table(Tb::cond(m));
    KX_CONST F *wq_t = const_table(Tb::wq(m));

    const bool act = base + lane < n;
    const int64_t i = act ? base + lane : n - 1;
    const F u = (F)((kln(T[i]) - m.fit_L0) * m.inv_fit_h);
    const double pr = Pp[i] * (1.0 / kPatm);
    auto Yat = [&](int k) { return Y[(int64_t)k * n + i]; };
    {
        double s = 0.0;
        for (int k = w; k < ns; k += nw) s = fma(Yat(k), sp[k].inv_W, s);
        part[w * kWave] = s;
    }
    __syncthreads();
    double sYW = 0.0;
    for (int q = 0; q < nw; ++q) sYW += part[q * kWave];
    const double xf = krcp(sYW);

    F sig[RW], den[RW], acc[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int k = w * RW + r, kc = min(k, ns - 1);
        const F ek = horner_c<ORDER>(visc_t + kc * order, u, order);
        // sigma_k = sqrt(eta_k) / W_k^(1/4)
        sig[r] = k < ns ? ek * rsqrt_acc(ek) * rcp_acc((F)wq_t[kc]) : (F)0;
        den[r] = acc[r] = (F)0;
    }
    // FP64: this wave's shares of W-bar and Mathur's sums; mixed: Mathur's FP32 sums
    // in species order by wave 0
    double wb = 0.0;
    F s1 = (F)0, s2 = (F)0;
    for (int j0 = 0; j0 < ns; j0 += kRowsChunk) {
        const int j1 = min(j0 + kRowsChunk, ns);
        __syncthreads();  // the previous chunk's rows (and `part`) are read
        for (int j = j0 + w; j < j1; j += nw) {
            F *row = rows + (j - j0) * NROW * kWave;
            const double X = Yat(j) * sp[j].inv_W * xf;
            row[0] = (F)X;
            // rho_j = W_j^(1/4) / sqrt(eta_j)
            row[kWave] = (F)wq_t[j] * rsqrt_acc(horner_c<ORDER>(visc_t + j * order, u, order));
            const F lk = horner_c<ORDER>(cond_t + j * order, u, order);
            if constexpr (F64) {
                s1 = fma(X, lk, s1);
                s2 = fma(X, rcp_acc(lk), s2);
            } else {
                row[2 * kWave] = lk;
                row[3 * kWave] = rcp_acc(lk);
            }
            wb = fma(X, Wt[j], wb);
        }
        __syncthreads();
        if (!F64 && w == 0) {
            for (int j = 0; j < j1 - j0; ++j) {
                const F *row = rows + j * NROW * kWave;
                s1 = fma(row[0], row[2 * kWave], s1);
                s2 = fma(row[0], row[3 * kWave], s2);
            }
        }
        auto c1_of = [&](int j, int r) {
            const int k = w * RW + r;
            return const_table(Tb::wilke(m))[((size_t)(k / kKB) * ns + j) * kKB + k % kKB];
        };
        auto fit_of = [&](int j, int r) {
            const int k = w * RW + r;
            return horner_c<ORDER>(const_table(Tb::dfit(m)) +
                                       (((size_t)(k / kKB) * ns + j) * kKB + k % kKB) * order,
                                   u, order);
        };
        auto wilke = [&](int j, int r, F X, F rho) {
            // X_j phi_kj = c1 X_j (1 + sigma_k rho_j)^2
            const F t = fma(sig[r], rho, (F)1);
            const F xt = X * t;
            den[r] = fma(c1_of(j, r), xt * t, den[r]);
        };
        if constexpr (rows_staged<F>(KIND, RW)) {
            const int o = ORDER > 0 ? ORDER : order;
            const int nfit = kStageK * o;  // coefficients of one j
            F *stage = reinterpret_cast<F *>(reinterpret_cast<char *>(smem_d) +
                                             rows_lds_bytes<F>(ns, nw)) +
                       w * stage_size(o);
            F *wstage = stage + kStage * nfit;
            for (int js = j0; js < j1; js += kStage) {
                const int nj = min(kStage, j1 - js);
#pragma unroll
                for (int b = 0; b < RW / kStageK; ++b) {
                    const int k0 = w * RW + b * kStageK;
                    if (RW > kStageK && k0 >= ns) break;
                    // j and coefficient of element e: the tables hold kKB species per j
                    const size_t at = ((size_t)(k0 / kKB) * ns + js) * kKB + k0 % kKB;
                    const F *fsrc = Tb::dfit(m) + at * o;
                    const F *wsrc = Tb::wilke(m) + at;
                    auto src = [&](int e) { return e / nfit * kKB * o + e % nfit; };
                    const F wv = lane < nj * kStageK
                                     ? wsrc[lane / kStageK * kKB + lane % kStageK] : (F)0;
                    if constexpr (ORDER > 0) {
                        constexpr int NL = (kStage * kStageK * ORDER + kWave - 1) / kWave;
                        F v[NL];
#pragma unroll
                        for (int e = 0; e < NL; ++e)
                            v[e] = e * kWave + lane < nj * nfit ? fsrc[src(e * kWave + lane)] : (F)0;
#pragma unroll
                        for (int e = 0; e < NL; ++e)
                            if (e * kWave + lane < kStage * nfit) stage[e * kWave + lane] = v[e];
                    } else {
                        for (int e = lane; e < nj * nfit; e += kWave) stage[e] = fsrc[src(e)];
                    }
                    if (lane < kStage * kStageK) wstage[lane] = wv;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    auto staged_wilke = [&](int jj, int r, F X, F rho) {
                        // X_j phi_kj = c1 X_j (1 + sigma_k rho_j)^2
                        const F t = fma(sig[b * kStageK + r], rho, (F)1);
                        const F xt = X * t;
                        den[b * kStageK + r] = fma(wstage[jj * kStageK + r], xt * t, den[b * kStageK + r]);
                    };
                    auto staged_fit = [&](int jj, int r) {
                        const F *c = stage + jj * nfit + r * o;
                        F f = c[o - 1];
#pragma unroll
                        for (int q = ORDER - 2; q >= 0; --q) f = fma(f, u, c[q]);
                        if (ORDER == 0)
                            for (int q = o - 2; q >= 0; --q) f = fma(f, u, c[q]);
                        return f;
                    };
                    int jj = 0;
                    if constexpr (F64) {
#pragma clang loop unroll(disable)
                        for (; jj + 1 < nj; jj += 2) {
                            const int j = js + jj;
                            const F *row = rows + (j - j0) * NROW * kWave;
                            const F Xa = row[0], ra = row[kWave];
                            const F Xb = row[2 * kWave], rb = row[3 * kWave];
#pragma unroll
                            for (int r = 0; r < kStageK; ++r) {
                                const int k = k0 + r, q = b * kStageK + r;
                                staged_wilke(jj, r, Xa, ra);
                                staged_wilke(jj + 1, r, Xb, rb);
                                // X_j / D_kj (j != k) of both
                                const F fa = staged_fit(jj, r), fb = staged_fit(jj + 1, r);
                                const F xa = k == j ? (F)0 : Xa, xb = k == j + 1 ? (F)0 : Xb;
                                acc[q] = fma(fma(xa, fb, xb * fa), rcp_fast(fa * fb), acc[q]);
                            }
                        }
                    }
#pragma clang loop unroll(disable)
                    for (; jj < nj; ++jj) {
                        const int j = js + jj;
                        const F *row = rows + (j - j0) * NROW * kWave;
                        const F X = row[0], rho = row[kWave];
#pragma unroll
                        for (int r = 0; r < kStageK; ++r) {
                            const int k = k0 + r, q = b * kStageK + r;
                            staged_wilke(jj, r, X, rho);
                            acc[q] = fma(k == j ? (F)0 : X, rcp_fast(staged_fit(jj, r)), acc[q]);
                        }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();  // the stage is read
                }
            }
        } else {
            int j = j0;
            if constexpr (F64 && KIND == 0) {
                for (; j + 1 < j1; j += 2) {
                    const F *row = rows + (j - j0) * NROW * kWave;
                    const F Xa = row[0], ra = row[kWave], Xb = row[2 * kWave], rb = row[3 * kWave];
#pragma unroll
                    for (int r = 0; r < RW; ++r) {
                        const int k = w * RW + r;
                        wilke(j, r, Xa, ra);
                        wilke(j + 1, r, Xb, rb);
                        // X_j / D_kj (j != k) of both
                        const F fa = fit_of(j, r), fb = fit_of(j + 1, r);
                        const F xa = k == j ? (F)0 : Xa, xb = k == j + 1 ? (F)0 : Xb;
                        acc[r] = fma(fma(xa, fb, xb * fa), rcp_fast(fa * fb), acc[r]);
                    }
                }
            }
            for (; j < j1; ++j) {
                const F *row = rows + (j - j0) * NROW * kWave;
                const F X = row[0], rho = row[kWave];
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    wilke(j, r, X, rho);
                    const F f = fit_of(j, r);
                    acc[r] = fma(w * RW + r == j ? (F)0 : X, KIND == 0 ? rcp_fast(f) : f, acc[r]);
                }
            }
        }
    }
    __syncthreads();  // `part` and the chunk's rows are free
    part[w * NPART * kWave] = wb;
    if constexpr (F64) {
        part[(w * 4 + 1) * kWave] = s1;
        part[(w * 4 + 2) * kWave] = s2;
    }
    __syncthreads();
    double wbar = 0.0;
    for (int q = 0; q < nw; ++q) wbar += part[q * NPART * kWave];
    double visc = 0.0;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int k = w * RW + r;
        if (k < ns) {
            const double Xk = Yat(k) * sp[k].inv_W * xf;
            const F ek = horner_c<ORDER>(visc_t + k * order, u, order);
            if constexpr (F64) {
                visc = fma(Xk * ek, rcp_acc(den[r]), visc);
            } else {
                rows[2 * k * kWave] = (F)Xk * ek;
                rows[(2 * k + 1) * kWave] = rcp_acc(den[r]);
            }
            double D;
            if (acc[r] == (F)0) {
                const F f = horner_c<ORDER>(const_table(Tb::ddiag(m)) + k * order, u, order);
                D = (KIND == 0) ? (double)f / pr : 1.0 / ((double)f * pr);
            } else {
                // sum_{j!=k} X_j / D_kj = (p/p_atm) acc for either fit kind; the
                // numerator (W-bar - X_k W_k)/W-bar is formed in FP64
                D = fma(-Xk, Wt[k], wbar) * krcp(wbar * (double)acc[r] * pr);
            }
            if (act) Dmix[(int64_t)k * n + i] = D;
        }
    }
    if (F64) part[(w * 4 + 3) * kWave] = visc;
    __syncthreads();
    if (w == 0 && act) {
        if constexpr (F64) {
            double a1 = 0.0, a2 = 0.0, v = 0.0;
            for (int q = 0; q < nw; ++q) {
                a1 += part[(q * 4 + 1) * kWave];
                a2 += part[(q * 4 + 2) * kWave];
                v += part[(q * 4 + 3) * kWave];
            }
            lam[i] = 0.5 * (a1 + rcp_acc(a2));
            mu[i] = v;
        } else {
            lam[i] = (double)((F)0.5 * (s1 + rcp_acc(s2)));
            F v = (F)0;
            for (int k = 0; k < ns; ++k)
                v = fma(rows[2 * k * kWave], rows[(2 * k + 1) * kWave], v);
            mu[i] = (double)v;
        }
    }
}

// The same results by one thread per P points (a wave per 64 P), for calls of very
// many points: species k in blocks of KB, j streaming over all species with X_j and
// rho_j formed again per block, so that a coefficient serves 64 P points and nothing
// waits at a barrier.  Every sum runs over the same terms in the same order as in
// transport_rows_tile (the shares of its waves of rw species one after another), so a
// point's bits are the same.
template <class F, int ORDER, int KIND, int P, int KB>
__device__ __forceinline__ void transport_lanes_tile(const MechDev &m, int rw, int64_t n,
                                                     int64_t base, const double *__restrict__ T,
                                                     const double *__restrict__ Pp,
                                                     const double *__restrict__ Y,
                                                     double *__restrict__ mu,
                                                     double *__restrict__ lam,
                                                     double *__restrict__ Dmix)
{
    using Tb = Tabs<F>;
    constexpr bool F64 = std::is_same<F, double>::value;
    static_assert(kKB % KB == 0 && KB % 2 == 0, "blocks of the tables");
    const int ns = m.ns, order = ORDER > 0 ? ORDER : m.fit_order, nw = (ns + rw - 1) / rw;
    KX_CONST DevSpecies *sp = const_table(m.sp);
    KX_CONST double *Wt = const_table(m.W);
    KX_CONST F *visc_t = const_table(Tb::visc(m)), *cond_t = const_table(Tb::cond(m));
    KX_CONST F *wq_t = const_table(Tb::wq(m));

    int64_t idx[P];
    bool act[P];
    F u[P];
    double pr[P], xf[P], wbar[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const int64_t i = base + threadIdx.x + kWave * q;
        act[q] = i < n;
        idx[q] = act[q] ? i : n - 1;
        u[q] = (F)((kln(T[idx[q]]) - m.fit_L0) * m.inv_fit_h);
        pr[q] = Pp[idx[q]] * (1.0 / kPatm);
    }
    auto Yat = [&](int k, int q) { return Y[(int64_t)k * n + idx[q]]; };
    {
        double sYW[P];
#pragma unroll
        for (int q = 0; q < P; ++q) sYW[q] = 0.0;
        for (int w = 0; w < nw; ++w) {
            double s[P];
#pragma unroll
            for (int q = 0; q < P; ++q) s[q] = 0.0;
            for (int k = w; k < ns; k += nw) {
                const double iw = sp[k].inv_W;
#pragma unroll
                for (int q = 0; q < P; ++q) s[q] = fma(Yat(k, q), iw, s[q]);
            }
#pragma unroll
            for (int q = 0; q < P; ++q) sYW[q] += s[q];
        }
#pragma unroll
        for (int q = 0; q < P; ++q) xf[q] = krcp(sYW[q]);
    }
    // W-bar and Mathur's sums: FP64 by the waves' shares, mixed Mathur's in species
    // order
    {
        double a1[P], a2[P];
        F s1[P], s2[P];
#pragma unroll
        for (int q = 0; q < P; ++q) {
            wbar[q] = a1[q] = a2[q] = 0.0;
            s1[q] = s2[q] = (F)0;
        }
        for (int w = 0; w < nw; ++w) {
            double wb[P];
#pragma unroll
            for (int q = 0; q < P; ++q) {
                wb[q] = 0.0;
                if (F64) s1[q] = s2[q] = (F)0;
            }
            for (int j0 = 0; j0 < ns; j0 += kRowsChunk)
                for (int j = j0 + w; j < min(j0 + kRowsChunk, ns); j += nw) {
                    const double iw = sp[j].inv_W, W = Wt[j];
#pragma unroll
                    for (int q = 0; q < P; ++q) {
                        const double X = Yat(j, q) * iw * xf[q];
                        if constexpr (F64) {
                            const F lk = horner_c<ORDER>(cond_t + j * order, u[q], order);
                            s1[q] = fma(X, lk, s1[q]);
                            s2[q] = fma(X, rcp_acc(lk), s2[q]);
                        }
                        wb[q] = fma(X, W, wb[q]);
                    }
                }
#pragma unroll
            for (int q = 0; q < P; ++q) {
                wbar[q] += wb[q];
                if constexpr (F64) {
                    a1[q] += s1[q];
                    a2[q] += s2[q];
                }
            }
        }
        if constexpr (!F64) {
            for (int j = 0; j < ns; ++j) {
                const double iw = sp[j].inv_W;
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    const double X = Yat(j, q) * iw * xf[q];
                    const F lk = horner_c<ORDER>(cond_t + j * order, u[q], order);
                    s1[q] = fma((F)X, lk, s1[q]);
                    s2[q] = fma((F)X, rcp_acc(lk), s2[q]);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < P; ++q)
            if (act[q]) {
                if constexpr (F64)
                    lam[idx[q]] = 0.5 * (a1[q] + rcp_acc(a2[q]));
                else
                    lam[idx[q]] = (double)((F)0.5 * (s1[q] + rcp_acc(s2[q])));
            }
    }

    double v[P], vp[P];  // FP64: mu and the current share's part of it
    F v32[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
        v[q] = vp[q] = 0.0;
        v32[q] = (F)0;
    }
    for (int k0 = 0; k0 < ns; k0 += KB) {
        if (F64 && k0 > 0 && k0 % rw == 0) {
#pragma unroll
            for (int q = 0; q < P; ++q) {
                v[q] += vp[q];
                vp[q] = 0.0;
            }
        }
        F sig[P][KB], den[P][KB], acc[P][KB];
#pragma unroll
        for (int r = 0; r < KB; ++r) {
            const int k = k0 + r, kc = min(k, ns - 1);
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const F ek = horner_c<ORDER>(visc_t + kc * order, u[q], order);
                sig[q][r] = k < ns ? ek * rsqrt_acc(ek) * rcp_acc((F)wq_t[kc]) : (F)0;
                den[q][r] = acc[q][r] = (F)0;
            }
        }
        KX_CONST F *c1b = const_table(Tb::wilke(m)) + (size_t)(k0 / kKB) * ns * kKB + k0 % kKB;
        KX_CONST F *dfb = const_table(Tb::dfit(m)) +
                          ((size_t)(k0 / kKB) * ns * kKB + k0 % kKB) * order;
        auto point = [&](int j, F (&X)[P], F (&rho)[P]) {
            const double iw = sp[j].inv_W;
            const F wj = (F)wq_t[j];
#pragma unroll
            for (int q = 0; q < P; ++q) {
                X[q] = (F)(Yat(j, q) * iw * xf[q]);
                rho[q] = wj * rsqrt_acc(horner_c<ORDER>(visc_t + j * order, u[q], order));
            }
        };
        auto wilke = [&](F c1, int q, int r, F X, F rho) {
            const F t = fma(sig[q][r], rho, (F)1);
            const F xt = X * t;
            den[q][r] = fma(c1, xt * t, den[q][r]);
        };
        constexpr bool PAIRS = F64 && KIND == 0;
        // species j0 .. j1 - 1; diag: they hold species of the block
        auto steps = [&](int j0, int j1, bool diag) {
            int j = j0;
            if constexpr (PAIRS) {
#pragma clang loop unroll(disable)
                for (; j + 1 < j1; j += 2) {
                    F Xa[P], ra[P], Xb[P], rb[P];
                    point(j, Xa, ra);
                    point(j + 1, Xb, rb);
                    KX_CONST F *ca = c1b + (size_t)j * kKB, *da = dfb + (size_t)j * kKB * order;
#pragma unroll
                    for (int r = 0; r < KB; ++r) {
                        const bool sa = diag && k0 + r == j, sb = diag && k0 + r == j + 1;
#pragma unroll
                        for (int q = 0; q < P; ++q) {
                            wilke(ca[r], q, r, Xa[q], ra[q]);
                            wilke(ca[kKB + r], q, r, Xb[q], rb[q]);
                            const F fa = horner_c<ORDER>(da + r * order, u[q], order);
                            const F fb = horner_c<ORDER>(da + (kKB + r) * order, u[q], order);
                            const F xa = sa ? (F)0 : Xa[q], xb = sb ? (F)0 : Xb[q];
                            acc[q][r] = fma(fma(xa, fb, xb * fa), rcp_fast(fa * fb), acc[q][r]);
                        }
                        // two species' coefficients in scalar registers at a time (all
                        // four spill: 200 species, 2^20 points 38.6 against 33.9 ms)
                        if (r % 2) __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
#pragma clang loop unroll(disable)
            for (; j < j1; ++j) {
                F X[P], rho[P];
                point(j, X, rho);
                KX_CONST F *c1 = c1b + (size_t)j * kKB, *df = dfb + (size_t)j * kKB * order;
#pragma unroll
                for (int r = 0; r < KB; ++r) {
                    const bool self = diag && k0 + r == j;
#pragma unroll
                    for (int q = 0; q < P; ++q) {
                        wilke(c1[r], q, r, X[q], rho[q]);
                        const F f = horner_c<ORDER>(df + r * order, u[q], order);
                        acc[q][r] = fma(self ? (F)0 : X[q], KIND == 0 ? rcp_fast(f) : f, acc[q][r]);
                    }
                }
            }
        };
        const int k1 = min(k0 + KB, ns);
        steps(0, k0, false);
        steps(k0, k1, true);
        steps(k1, ns, false);
#pragma unroll
        for (int r = 0; r < KB; ++r) {
            const int k = k0 + r;
            if (k < ns) {
                const double iw = sp[k].inv_W, Wk = Wt[k];
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    const double Xk = Yat(k, q) * iw * xf[q];
                    const F ek = horner_c<ORDER>(visc_t + k * order, u[q], order);
                    if constexpr (F64)
                        vp[q] = fma(Xk * ek, rcp_acc(den[q][r]), vp[q]);
                    else
                        v32[q] = fma((F)Xk * ek, rcp_acc(den[q][r]), v32[q]);
                    double D;
                    if (acc[q][r] == (F)0) {
                        const F f = horner_c<ORDER>(const_table(Tb::ddiag(m)) + k * order, u[q], order);
                        D = (KIND == 0) ? (double)f / pr[q] : 1.0 / ((double)f * pr[q]);
                    } else {
                        D = fma(-Xk, Wk, wbar[q]) * krcp(wbar[q] * (double)acc[q][r] * pr[q]);
                    }
                    if (act[q]) Dmix[(int64_t)k * n + idx[q]] = D;
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < P; ++q)
        if (act[q]) mu[idx[q]] = F64 ? v[q] + vp[q] : (double)v32[q];
}

// ---------------------------------------------------------------------------
// Symmetric evaluation of the D_kj fits (§2.2.2, §2.3.2: D_kj = D_jk, so half
// of the polynomial evaluations can be skipped).  With tables of D_kj fits
// (kind 0) every pair costs a polynomial and a reciprocal; here each unordered
// pair {k, j} is evaluated once and its 1/D_kj enters both sums
// S_k = sum_{j != k} X_j / D_kj and S_j.  One wave per workgroup, one point per
// lane (64 points).  S_j of a pair belongs to a species whose row is finished
// later, so the sums of every species are kept per lane in LDS (ns x 64
// values; each lane its own column).  The k rows are taken KB at a time with
// S_k in registers: pairs (k, j) with j before the block were added to S_k's
// LDS entry when j's block ran, pairs inside the block update the block's
// registers, and pairs with j after the block add X_k / D_kj to S_j's entry.
// The Wilke sums take the ordered pairs (phi_kj != phi_jk) as the full kernel.
template <class F, int ORDER, int KB>
__global__ __launch_bounds__(kWave) void transport_sym_kernel(MechDev m, int64_t n,
                                                              const double *__restrict__ T,
                                                              const double *__restrict__ Pp,
                                                              const double *__restrict__ Y,
                                                              double *__restrict__ mu,
                                                              double *__restrict__ lam,
                                                              double *__restrict__ Dmix)
{
    using Tb = Tabs<F>;
    extern __shared__ double smem_d[];
    F *sj = reinterpret_cast<F *>(smem_d);  // [ns][kWave]: S_j of this lane's point
    const int lane = threadIdx.x;
    const int ns = m.ns, order = m.fit_order;
    const int64_t ir = (int64_t)blockIdx.x * kWave + lane;
    const bool act = ir < n;
    const int64_t i = act ? ir : n - 1;
    const double Ti = T[i];
    const F u = (F)((kln(Ti) - m.fit_L0) * m.inv_fit_h);
    const double pr = Pp[i] / kPatm;
    auto Yat = [&](int k) { return Y[(int64_t)k * n + i]; };

    // X_k = (Y_k / W_k) xf; W-bar = sum_k X_k W_k; Mathur conductivity
    double xf, wbar = 0.0;
    {
        double sYW = 0.0;
        for (int k = 0; k < ns; ++k) sYW = fma(Yat(k), m.sp[k].inv_W, sYW);
        xf = 1.0 / sYW;
        F s1 = (F)0, s2 = (F)0;
        for (int k = 0; k < ns; ++k) {
            const double X = Yat(k) * m.sp[k].inv_W * xf;
            const F lk = horner<ORDER>(Tb::cond(m) + k * order, u, order);
            s1 = fma((F)X, lk, s1);
            s2 = fma((F)X, rcp_acc(lk), s2);
            wbar = fma(X, m.W[k], wbar);
            sj[k * kWave + lane] = (F)0;
        }
        if (act) lam[i] = (double)((F)0.5 * (s1 + rcp_acc(s2)));
    }

    F visc = (F)0;
    const int nkb = (ns + KB - 1) / KB;
    for (int kb = 0; kb < nkb; ++kb) {
        const int k0 = kb * KB, k1 = min(k0 + KB, ns);
        const int tb = k0 / kKB, toff = k0 % kKB;
        F sig[KB], den[KB], acc[KB], xk[KB];
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
            const int k = k0 + kk;
            const bool valid = k < ns;
            const int kc = valid ? k : 0;
            const F ek = horner<ORDER>(Tb::visc(m) + kc * order, u, order);
            sig[kk] = valid ? ek * rsqrt_acc(ek) * rcp_acc(Tb::wq(m)[kc]) : (F)0;
            den[kk] = (F)0;
            acc[kk] = valid ? sj[kc * kWave + lane] : (F)0;
            xk[kk] = valid ? (F)(Yat(kc) * m.sp[kc].inv_W * xf) : (F)0;
        }
        const F *c1b = Tb::wilke(m) + (size_t)tb * ns * kKB + toff;
        const F *dfb = Tb::dfit(m) + ((size_t)tb * ns * kKB + toff) * order;
        // pairs inside the block: (k0 + a, k0 + b), a < b
#pragma unroll
        for (int a = 0; a < KB; ++a)
#pragma unroll
            for (int b = a + 1; b < KB; ++b)
                if (k0 + b < ns) {
                    const F f = horner<ORDER>(dfb + ((size_t)(k0 + b) * kKB + a) * order, u,
                                              order);
                    const F g = rcp_fast(f);
                    acc[a] = fma(xk[b], g, acc[a]);
                    acc[b] = fma(xk[a], g, acc[b]);
                }
        for (int j = 0; j < ns; ++j) {
            const F wj = Tb::wq(m)[j];
            const F Xj = (F)(Yat(j) * m.sp[j].inv_W * xf);
            const F rho = wj * rsqrt_acc(horner<ORDER>(Tb::visc(m) + j * order, u, order));
            const F *c1 = c1b + (size_t)j * kKB;
#pragma unroll
            for (int kk = 0; kk < KB; ++kk) {
                // Wilke: X_j phi_kj = c1 X_j (1 + sigma_k rho_j)^2, every ordered pair
                const F t = fma(sig[kk], rho, (F)1);
                den[kk] = fma(c1[kk], Xj * t * t, den[kk]);
            }
            if (j >= k1) {
                const F *df = dfb + (size_t)j * kKB * order;
                F s = (F)0;
#pragma unroll
                for (int kk = 0; kk < KB; ++kk) {
                    const F g = rcp_fast(horner<ORDER>(df + kk * order, u, order));
                    acc[kk] = fma(Xj, g, acc[kk]);
                    s = fma(xk[kk], g, s);  // xk = 0 past the last species
                }
                sj[j * kWave + lane] += s;
            }
        }
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
            const int k = k0 + kk;
            if (k < ns) {
                const double Xk = Yat(k) * m.sp[k].inv_W * xf;
                const F ek = horner<ORDER>(Tb::visc(m) + k * order, u, order);
                visc = fma((F)Xk * ek, rcp_acc(den[kk]), visc);
                double D;
                if (acc[kk] == (F)0) {
                    const F f = horner<ORDER>(Tb::ddiag(m) + k * order, u, order);
                    D = (double)f / pr;
                } else {
                    D = (wbar - Xk * m.W[k]) / (wbar * (double)acc[kk] * pr);
                }
                if (act) Dmix[(int64_t)k * n + i] = D;
            }
        }
    }
    if (act) mu[i] = (double)visc;
}

// ---------------------------------------------------------------------------
// Matrix-core form (tables holding fits of 1/D_kj, the form the paper's
// generated code evaluates).  With g_kj(u) = 1/D_kj(1 atm) = sum_n d_kjn u^n,
//     S_k = sum_{j != k} X_j g_kj = sum_n sum_j d_kjn (u^n X_j),
// a product of the fixed matrix [G_0 | ... | G_{N-1}] (G_n[k][j] = d_kjn, zero
// diagonal) with the per-point stack (u^n X_j).  The Wilke denominator, with
// t_kj = 1 + sigma_k rho_j and sigma_k = 1 / rho_k,
//     sum_j c1_kj X_j t_kj^2 = A_k + 2 sigma_k B_k + sigma_k^2 C_k,
// needs the products of the fixed matrix c1 with X, X rho and X rho^2 (all
// terms positive, so the expansion loses nothing).  A workgroup of four waves
// takes NP points: X and rho go to LDS, each wave runs 16x16x4 MFMAs for its
// blocks of 16 species k, and the epilogue forms mu, D_km per (k, point).

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <class F> struct Mfma;
template <> struct Mfma<double> {
    using V = v4d;
    static __device__ __forceinline__ V op(double a, double b, V c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // row of the 16x16 result held by lane l in element r
    static __device__ __forceinline__ int row(int l, int r) { return (l >> 4) + 4 * r; }
    static __device__ const double *gfrag(const MechDev &m) { return m.gfrag; }
    static __device__ const double *c1frag(const MechDev &m) { return m.c1frag; }
};
template <> struct Mfma<float> {
    using V = v4f;
    static __device__ __forceinline__ V op(float a, float b, V c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int l, int r) { return 4 * (l >> 4) + r; }
    static __device__ const float *gfrag(const MechDev &m) { return m.gfrag32; }
    static __device__ const float *c1frag(const MechDev &m) { return m.c1frag32; }
};

constexpr int kMfmaPad = 2;  // LDS row padding of the X / rho tiles (elements)

// Per-point values shared by the phases of a tile.
struct MfmaPoint {
    double u, xf, wbar, pr;
};

// A tile's shape: points, threads, and how its sums over species are cut into
// partial sums -- the prologue's by j mod PG, mu's by row block mod MC -- which with
// their order fix the bits.  A thread of a shape with fewer groups (or row blocks in
// flight) keeps several partial sums, so that two shapes of a mechanism give the same.
template <int NP_, int NT_, int PG_ = NT_ / NP_, int MC_ = 0> struct MfmaShape {
    static constexpr int NP = NP_, NT = NT_, PG = PG_;
    // a wave takes NB of the 16-point column blocks, WC waves share a row block, WR
    // row blocks are in flight
    static constexpr int WC = NT == 512 && NP == 64 ? 2 : 1, NB = NP / 16 / WC;
    static constexpr int WR = NT / kWave / WC, MC = MC_ ? MC_ : WR;
    static constexpr int NG = NT / NP;  // species groups of the prologue
    static_assert((PG == NG || PG == 2 * NG) && MC % WR == 0 && MC <= PG, "partial sums");
};

template <class F, class S> constexpr size_t mfma_lds_bytes(int kstep)
{
    // X and rho tiles, point table, partial sums (per (class, point) in the
    // prologue: 3 sums, and the normalisation sum in a slot of its own; 4 MC per
    // point for mu)
    return 2 * (size_t)(4 * kstep) * (S::NP + kMfmaPad) * sizeof(F) + S::NP * sizeof(MfmaPoint) +
           (size_t)4 * S::PG * S::NP * sizeof(double);
}

// `tid` is threadIdx.x; the batch kernel passes it through an opaque move in
// each trip of its tile loop, so that the tile's lane-dependent addresses are
// not hoisted out of the loop (kept live across tiles they cost the kernel
// its occupancy).  LOOP: the workgroup takes another tile after this one (its
// LDS is then reused).
template <class F, class Sh, int ORDER, bool LOOP>
__device__ __forceinline__ void transport_mfma_tile(int tid, const MechDev &m, int64_t n,
                                                    int64_t base,
                                                    const double *__restrict__ T,
                                                    const double *__restrict__ Pp,
                                                    const double *__restrict__ Y,
                                                    double *__restrict__ mu,
                                                    double *__restrict__ lam,
                                                    double *__restrict__ Dmix)
{
    using Tb = Tabs<F>;
    using MF = Mfma<F>;
    using V = typename MF::V;
    constexpr int NP = Sh::NP, NT = Sh::NT, NG = Sh::NG, NB = Sh::NB, WC = Sh::WC, WR = Sh::WR;
    constexpr int PH = Sh::PG / NG, MH = Sh::MC / WR;  // partial sums per thread
    constexpr int LD = NP + kMfmaPad;    // LDS row stride of the tiles
    const int ns = m.ns, order = ORDER > 0 ? ORDER : m.fit_order;
    const int KS = m.kstep, MB = m.mblk, Kp = 4 * KS;
    const int t = tid, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);

    extern __shared__ double smem_d[];
    F *Xs = reinterpret_cast<F *>(smem_d);
    F *Rs = Xs + (size_t)Kp * LD;
    MfmaPoint *pt = reinterpret_cast<MfmaPoint *>(Rs + (size_t)Kp * LD);
    double *part = reinterpret_cast<double *>(pt + NP);  // [PG][3][NP], then mu's [4 MC][NP]
    double *part1 = part + 3 * Sh::PG * NP;              // [PG][NP]: sum of Y_j / W_j

    // ---- prologue: thread = (point p, species group g)
    const int p = t % NP;
    // with 64-point tiles the species group is the wave: uniform, so the
    // per-species coefficients below come from scalar loads
    const int g = NP == 64 ? __builtin_amdgcn_readfirstlane(t / NP) : t / NP;
    const int64_t ip = min(base + p, n - 1);  // points past n repeat the last one
    const double Tp = T[ip];
    const double up = (kln(Tp) - m.fit_L0) * m.inv_fit_h;
    // every Y load of this thread is issued before the first is used (a
    // thread covers at most kJmax species: ns <= kJmax NG for the chosen tile)
    constexpr int kJmax = NT == 512 && NP == 64 ? 8 : 16;
    double yw[kJmax];
#pragma unroll
    for (int q = 0; q < kJmax; ++q) {
        const int j = g + NG * q;
        yw[q] = j < ns ? Y[(int64_t)j * n + ip] : 0.0;
    }
    // the partial sums in scalars: as arrays they change the code of the prologue
    // also where there is one (200 species FP64 1.3 % slower)
    double s = 0.0, sB = 0.0;
#pragma unroll
    for (int q = 0; q < kJmax; ++q) {
        const int j = g + NG * q;
        if (j < ns) {
            yw[q] *= m.sp[j].inv_W;  // Y_j / W_j
            if (PH > 1 && q % 2)
                sB += yw[q];
            else
                s += yw[q];
        }
    }
    part1[g * NP + p] = s;
    if (PH > 1) part1[(g + NG) * NP + p] = sB;
    __syncthreads();
    double sYW = 0.0;
#pragma unroll
    for (int q = 0; q < Sh::PG; ++q) sYW += part1[q * NP + p];
    const double xf = krcp(sYW);
    if (t < NP) {
        MfmaPoint P;
        P.u = up;
        P.xf = xf;
        P.wbar = 0.0;  // the epilogue adds the group partials
        P.pr = Pp[ip] * (1.0 / kPatm);
        pt[p] = P;
    }
    double wb = 0.0, s1 = 0.0, s2 = 0.0, wbB = 0.0, s1B = 0.0, s2B = 0.0;
#pragma unroll
    for (int q = 0; q < kJmax; ++q) {
        const int j = g + NG * q;
        if (j >= Kp) break;
        if (j < ns) {
            const double X = yw[q] * xf;  // FP64 X_j for W-bar and the Mathur sums
            if (PH > 1 && q % 2)
                wbB = fma(X, m.W[j], wbB);
            else
                wb = fma(X, m.W[j], wb);
            const F lj = NP == 64 ? horner<ORDER>(Tb::cond(m) + j * order, (F)up, order)
                                  : horner_v<ORDER>(Tb::cond(m) + j * order, (F)up, order);
            if (PH > 1 && q % 2) {
                s1B = fma(X, (double)lj, s1B);
                s2B = fma(X, (double)rcp_mfma(lj), s2B);
            } else {
                s1 = fma(X, (double)lj, s1);
                s2 = fma(X, (double)rcp_mfma(lj), s2);
            }
            const F ej = NP == 64 ? horner<ORDER>(Tb::visc(m) + j * order, (F)up, order)
                                  : horner_v<ORDER>(Tb::visc(m) + j * order, (F)up, order);
            Xs[(size_t)j * LD + p] = (F)X;
            Rs[(size_t)j * LD + p] = Tb::wq(m)[j] * rsqrt_acc(ej);  // rho_j
        } else {
            Xs[(size_t)j * LD + p] = (F)0;
            Rs[(size_t)j * LD + p] = (F)1;
        }
    }
    part[(g * 3 + 0) * NP + p] = wb;
    part[(g * 3 + 1) * NP + p] = s1;
    part[(g * 3 + 2) * NP + p] = s2;
    if (PH > 1) {
        double *pg = part + (g + NG) * 3 * NP + p;
        pg[0] = wbB;
        pg[NP] = s1B;
        pg[2 * NP] = s2B;
    }
    __syncthreads();
    if (t < NP && base + p < n) {
        double a1 = 0.0, a2 = 0.0;
#pragma unroll
        for (int q = 0; q < Sh::PG; ++q) {
            a1 += part[(q * 3 + 1) * NP + p];
            a2 += part[(q * 3 + 2) * NP + p];
        }
        lam[base + p] = 0.5 * (a1 + krcp(a2));  // Mathur
    }

    // ---- products on the matrix cores: wave w takes row blocks wr, wr + WR, ...
    // and the points from c0
    const int wr = w / WC, c0 = (w % WC) * 16 * NB;
    const int col = c0 + (lane & 15), jr = lane >> 4;
    F uc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) uc[nb] = (F)pt[16 * nb + col].u;
    double mup[MH][NB] = {};
    const F *gf = MF::gfrag(m), *cf = MF::c1frag(m);
    constexpr int MO = ORDER > 0 ? ORDER : kMaxFitOrder;  // A fragments per K-step
    const size_t ostride = (size_t)MB * KS * 64;           // between fit orders
    for (int mb = wr; mb < MB; mb += WR) {
        V S[NB], A[NB], B[NB], C[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) S[nb] = A[nb] = B[nb] = C[nb] = V{0, 0, 0, 0};
        // A fragments of the next K-step are in flight during this one
        const F *cfb = cf + (size_t)mb * KS * 64 + lane;
        const F *gfb = gf + (size_t)mb * KS * 64 + lane;
        F a1n = cfb[0], ggn[MO];
#pragma unroll
        for (int o = 0; o < MO; ++o)
            if (o < order) ggn[o] = gfb[o * ostride];
        for (int ks = 0; ks < KS; ++ks) {
            const F a1 = a1n;
            F gg[MO];
#pragma unroll
            for (int o = 0; o < MO; ++o) gg[o] = ggn[o];
            if (ks + 1 < KS) {
                a1n = cfb[(ks + 1) * 64];
#pragma unroll
                for (int o = 0; o < MO; ++o)
                    if (o < order) ggn[o] = gfb[o * ostride + (ks + 1) * 64];
            }
            const int j = 4 * ks + jr;
            F x[NB], r[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                x[nb] = Xs[(size_t)j * LD + 16 * nb + col];
                r[nb] = Rs[(size_t)j * LD + 16 * nb + col];
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const F xr = x[nb] * r[nb];
                A[nb] = MF::op(a1, x[nb], A[nb]);
                B[nb] = MF::op(a1, xr, B[nb]);
                C[nb] = MF::op(a1, xr * r[nb], C[nb]);
            }
            F bb[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) bb[nb] = x[nb];
#pragma unroll
            for (int o = 0; o < MO; ++o) {
                if (o < order) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        S[nb] = MF::op(gg[o], bb[nb], S[nb]);
                        bb[nb] *= uc[nb];
                    }
                }
            }
        }
        // ---- epilogue of this row block: element e of lane l is (k, point).
        // The Wilke denominator with sigma_k = 1/rho_k is
        //   A + sigma (2B + sigma C) = (A rho^2 + 2 B rho + C) / rho^2,
        // and the viscosity term X_k eta_k / den with eta_k = (W_k^(1/4) / rho_k)^2
        // becomes X_k W_k^(1/2) / (A rho^2 + 2 B rho + C): one reciprocal per
        // element, of a sum of positive terms.  In FP64, Z_k = X_k from the tile
        // and the row factor is W_k^(1/2); the mixed path (FP32 tile) forms
        // Z_k = Y_k W-bar' = X_k W_k in FP64 from the input, so its row factor
        // is W_k^(-1/2) and the D_km numerator W-bar - X_k W_k is W-bar - Z_k.
        constexpr bool F64 = std::is_same<F, double>::value;
        int krow[4];
        F rf[4];
        double wk[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            krow[e] = 16 * mb + MF::row(lane, e);
            const int kc = min(krow[e], ns - 1);
            const F q = Tb::wq(m)[kc];
            rf[e] = F64 ? q * q : (F)1 / (q * q);
            wk[e] = F64 ? m.W[kc] : 1.0;
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int pp = 16 * nb + col;
            const int64_t i = base + pp;
            const MfmaPoint P = pt[pp];
            double wbar = 0.0;
#pragma unroll
            for (int q = 0; q < Sh::PG; ++q) wbar += part[(q * 3 + 0) * NP + pp];
            double own = 0.0;  // this row block's class of mu (several per thread)
            if constexpr (MH > 1) {
#pragma unroll
                for (int h = 0; h < MH; ++h)
                    if (mb / WR % MH == h) own = mup[h][nb];
            }
            double &mue = MH > 1 ? own : mup[0][nb];
            double yk[4];
            if (!F64) {
                const int64_t ic = min(i, n - 1);
#pragma unroll
                for (int e = 0; e < 4; ++e) yk[e] = Y[(int64_t)min(krow[e], ns - 1) * n + ic];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = krow[e];
                if (k >= ns) continue;
                const F rho = Rs[(size_t)k * LD + pp];
                const F den = fma(fma(A[nb][e], rho, (F)2 * B[nb][e]), rho, C[nb][e]);
                const double Zk = F64 ? (double)Xs[(size_t)k * LD + pp] : yk[e] * P.xf;
                mue = fma(Zk, (double)(rf[e] * rcp_mfma(den)), mue);
                double D;
                if (S[nb][e] == (F)0) {
                    // no other species present: D_km -> D_kk
                    const F gk = horner_v<ORDER>(Tb::ddiag(m) + k * order, (F)P.u, order);
                    D = 1.0 / ((double)gk * P.pr);
                } else {
                    D = (wbar - Zk * wk[e]) * krcp1(wbar * (double)S[nb][e] * P.pr);
                }
                if (i < n) Dmix[(int64_t)k * n + i] = D;
            }
            if constexpr (MH > 1) {
#pragma unroll
                for (int h = 0; h < MH; ++h)
                    if (mb / WR % MH == h) mup[h][nb] = own;
            }
        }
    }
    // mu: 4 MC partial sums per point (row block classes x 4 row groups), fixed order
    __syncthreads();
#pragma unroll
    for (int h = 0; h < MH; ++h)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            part[((wr + WR * h) * 4 + jr) * NP + 16 * nb + col] = mup[h][nb];
    __syncthreads();
    if (t < NP && base + t < n) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < 4 * Sh::MC; ++q) v += part[q * NP + t];
        mu[base + t] = v;
    }
    if (LOOP) __syncthreads();  // LDS reused by the next tile
}

// Waves per SIMD: four for 512-thread workgroups of which two share a CU, else two.
template <class F> constexpr int mfma_waves(int nt, int np)
{
    return nt == 512 && (np == 64 || sizeof(F) == 4) ? 4 : 2;
}

template <class F, class S, int ORDER>
__global__ __launch_bounds__(S::NT, mfma_waves<F>(S::NT, S::NP)) void transport_mfma_kernel(MechDev m, int64_t n,
                                                                const double *__restrict__ T,
                                                                const double *__restrict__ Pp,
                                                                const double *__restrict__ Y,
                                                                double *__restrict__ mu,
                                                                double *__restrict__ lam,
                                                                double *__restrict__ Dmix)
{
    transport_mfma_tile<F, S, ORDER, false>(threadIdx.x, m, n, (int64_t)blockIdx.x * S::NP, T, Pp, Y,
                                             mu, lam, Dmix);
}

// At most 256 VGPRs (two waves per SIMD): the FP64 form for fits of any order
// would otherwise take 258 and run one wave per SIMD.
template <class F, class S, int ORDER>
__global__ __launch_bounds__(S::NT, mfma_waves<F>(S::NT, S::NP)) void transport_mfma_batch_kernel(
    MechDev m, const WorkList *__restrict__ wl, int *__restrict__ counter)
{
    __shared__ int tile;
    const int ntiles = wl->ntiles[1];
    int r = 0;  // item of the previous tile
    for (;;) {
        if (threadIdx.x == 0) tile = atomicAdd(counter, 1);
        __syncthreads();
        // wave-uniform (the compiler then keeps the item's pointers in scalar
        // registers; read as a per-lane value they cost the tile its occupancy)
        const int t = __builtin_amdgcn_readfirstlane(tile);
        __syncthreads();
        if (t >= ntiles) break;
        r = work_item_of(wl, 1, t, r);
        const WorkItem it = wl->items[r];
        int tid;
        asm volatile("v_mov_b32 %0, %1" : "=v"(tid) : "v"((int)threadIdx.x));
        transport_mfma_tile<F, S, ORDER, true>(tid, m, it.n, (int64_t)(t - wl->start[1][r]) * S::NP, it.T,
                                          it.p, it.Y, it.mu, it.lam, it.Dmix);
    }
}

// Batched requests, one tile per workgroup (grid = the batch's transport
// tiles).  Uniform per workgroup, so a workgroup past the last tile returns
// before any barrier.
template <class F, class S, int ORDER>
__global__ __launch_bounds__(S::NT, mfma_waves<F>(S::NT, S::NP)) void transport_mfma_items_kernel(
    MechDev m, const WorkList *__restrict__ wl)
{
    const int t = (int)blockIdx.x;
    if (t >= wl->ntiles[1]) return;
    const int r = work_item_ballot(wl, 1, t);
    const WorkItem it = wl->items[r];
    transport_mfma_tile<F, S, ORDER, false>(threadIdx.x, m, it.n, (int64_t)(t - wl->start[1][r]) * S::NP,
                                      it.T, it.p, it.Y, it.mu, it.lam, it.Dmix);
}

template <class F, int ORDER, int KIND, int RW>
__global__ __launch_bounds__(1024, rows_min_waves<F>(KIND, RW)) void transport_rows_kernel(MechDev m, int64_t n,
                                                              const double *__restrict__ T,
                                                              const double *__restrict__ Pp,
                                                              const double *__restrict__ Y,
                                                              double *__restrict__ mu,
                                                              double *__restrict__ lam,
                                                              double *__restrict__ Dmix)
{
    transport_rows_tile<F, ORDER, KIND, RW>(m, n, (int64_t)blockIdx.x * kWave, T, Pp, Y, mu, lam,
                                            Dmix);
}

// Points of a thread and species of a block of transport_lanes_tile.  Four points by
// four species in FP64 (219 registers, two waves per SIMD) took 3.45 ms for 53
// species and 2^20 points, three by four (169) 3.03, two by eight 2.73, two by four
// (119, four waves) 2.57; mixed four by four 2.40 ms, four by eight 2.27, two by four
// 1.63, two by eight (96 registers) 1.50.
constexpr int kLanePoints = 2, kLaneTile = kLanePoints * kWave;
template <class F> constexpr int lane_species() { return sizeof(F) == 8 ? 4 : 8; }

template <class F, int KIND>
__global__ __launch_bounds__(kWave, 2) void transport_lanes_kernel(
    MechDev m, int rw, int64_t n, const double *__restrict__ T, const double *__restrict__ Pp,
    const double *__restrict__ Y, double *__restrict__ mu, double *__restrict__ lam,
    double *__restrict__ Dmix)
{
    transport_lanes_tile<F, 5, KIND, kLanePoints, lane_species<F>()>(
        m, rw, n, (int64_t)blockIdx.x * kLaneTile, T, Pp, Y, mu, lam, Dmix);
}

// Batched requests of very many points together.
template <class F, int KIND>
__global__ __launch_bounds__(kWave, 2) void transport_lanes_items_kernel(
    MechDev m, int rw, const WorkList *__restrict__ wl)
{
    const int t = (int)blockIdx.x;
    if (t >= wl->ntiles[1]) return;
    const int r = work_item_ballot(wl, 1, t);
    const WorkItem it = wl->items[r];
    transport_lanes_tile<F, 5, KIND, kLanePoints, lane_species<F>()>(
        m, rw, it.n, (int64_t)(t - wl->start[1][r]) * kLaneTile, it.T, it.p, it.Y, it.mu, it.lam,
        it.Dmix);
}

// Batched requests: persistent workgroups taking tiles from a counter.
template <class F, int ORDER, int KIND, int RW>
__global__ __launch_bounds__(1024, rows_min_waves<F>(KIND, RW)) void transport_rows_batch_kernel(MechDev m,
                                                                    const WorkList *__restrict__ wl,
                                                                    int *__restrict__ counter)
{
    __shared__ int tile;
    const int ntiles = wl->ntiles[1];
    int r = 0;  // item of the previous tile
    for (;;) {
        __syncthreads();  // the previous tile's LDS reads are done
        if (threadIdx.x == 0) tile = atomicAdd(counter, 1);
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(tile);  // wave-uniform
        if (t >= ntiles) break;
        r = work_item_of(wl, 1, t, r);
        const WorkItem it = wl->items[r];
        transport_rows_tile<F, ORDER, KIND, RW>(m, it.n, (int64_t)(t - wl->start[1][r]) * kWave,
                                                it.T, it.p, it.Y, it.mu, it.lam, it.Dmix);
    }
}

template <class F, int ORDER, int KIND, int RW>
__global__ __launch_bounds__(1024, rows_min_waves<F>(KIND, RW)) void transport_rows_items_kernel(MechDev m,
                                                                    const WorkList *__restrict__ wl)
{
    const int t = (int)blockIdx.x;
    if (t >= wl->ntiles[1]) return;
    const int r = work_item_ballot(wl, 1, t);
    const WorkItem it = wl->items[r];
    transport_rows_tile<F, ORDER, KIND, RW>(m, it.n, (int64_t)(t - wl->start[1][r]) * kWave, it.T,
                                            it.p, it.Y, it.mu, it.lam, it.Dmix);
}

__global__ void zero_kernel(int *p, int count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0;
}

// Mixture thermo (App. A.1): cp_k = Cp_k/W_k, h_k = H_k/W_k, cp = sum Y_k cp_k.
// Bound by memory (one row read and two written per species).  The four waves of
// a workgroup take every fourth species of its 64 points, four Y rows of a wave in
// flight: a call of few points has four times the waves at a quarter of the chain
// (53 species, 1000 points 27 -> 12 us), a large one more loads in flight (2^20
// points 327 -> 281 us, 4.8 TB/s; 200 species, 100003 points 273 -> 147 us).  The
// outputs are not read again here: non-temporal stores (131072 points 35 -> 29 us).
__global__ __launch_bounds__(kBlock) void thermo_kernel(MechDev m, int64_t n,
                                                        const double *__restrict__ T,
                                                        const double *__restrict__ Y,
                                                        double *__restrict__ cpk,
                                                        double *__restrict__ hk,
                                                        double *__restrict__ cpmix)
{
    constexpr int NW = kBlock / kWave;
    __shared__ double part[NW][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t i = (int64_t)blockIdx.x * kWave + lane;
    const int64_t ic = min(i, n - 1);  // lanes past the end repeat the last point
    const bool act = i < n;
    const double t = T[ic], invT = 1.0 / t;
    double cp = 0.0;
    constexpr int U = 4;  // species per trip
    for (int k0 = w; k0 < m.ns; k0 += U * NW) {
        double y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) y[u] = Y[(int64_t)min(k0 + u * NW, m.ns - 1) * n + ic];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * NW;
            if (k >= m.ns) break;
            KX_CONST DevSpecies &S = const_table(m.sp)[k];
            const bool lo = t < S.t_mid;
            // both ranges' values, one kept: cheaper than selecting coefficients (the
            // asm keeps the compiler from selecting the table's address instead, and
            // reading the coefficients per lane)
            auto pick = [&](double a, double b) {
                asm("" : "+v"(a), "+v"(b));
                return lo ? a : b;
            };
            auto cpr = [&](KX_CONST double *a) {
                return fma(t, fma(t, fma(t, fma(t, a[4], a[3]), a[2]), a[1]), a[0]);
            };
            const double c = pick(cpr(S.nasa_lo), cpr(S.nasa_hi)) * kRu * S.inv_W;
            cp = fma(y[u], c, cp);
            if (cpk && act) __builtin_nontemporal_store(c, cpk + (int64_t)k * n + i);
            if (hk) {
                auto hrt = [&](KX_CONST double *a) {
                    return fma(t, fma(t, fma(t, fma(t, a[4] * 0.2, a[3] * 0.25), a[2] * (1.0 / 3.0)),
                                      a[1] * 0.5),
                               a[0]) +
                           a[5] * invT;
                };
                const double h = pick(hrt(S.nasa_lo), hrt(S.nasa_hi)) * kRu * t * S.inv_W;
                if (act) __builtin_nontemporal_store(h, hk + (int64_t)k * n + i);
            }
        }
    }
    if (cpmix) {
        part[w][lane] = cp;
        __syncthreads();
        if (w == 0 && act)
            cpmix[i] = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
    }
}

// Species per wave of the vector-ALU kernel: the fewest that keep it within 16
// waves (a wave with fewer species has a shorter chain and fewer registers; 9
// species, 2^20 points: 117 us with 4 species a wave, 146 with 8, 159 with 16).
int rows_per_wave(const MechDev &m) { return m.ns <= 64 ? 4 : (m.ns <= 128 ? 8 : 16); }
int rows_waves(const MechDev &m) { return (m.ns + rows_per_wave(m) - 1) / rows_per_wave(m); }

template <class F> size_t rows_lds(const MechDev &m)
{
    const int nw = rows_waves(m);
    const size_t stages = rows_staged<F>(m.diff_kind, rows_per_wave(m)) ? nw * stage_size(m.fit_order) * sizeof(F) : 0;
    return rows_lds_bytes<F>(m.ns, nw) + stages;
}

// FORM 0: direct launch, 1: work-stealing batch, 2: one tile per workgroup
template <class F, int FORM, int KIND, int RW> const void *rows_instance(bool o5)
{
    if (FORM == 1)
        return o5 ? (const void *)transport_rows_batch_kernel<F, 5, KIND, RW>
                  : (const void *)transport_rows_batch_kernel<F, 0, KIND, RW>;
    if (FORM == 2)
        return o5 ? (const void *)transport_rows_items_kernel<F, 5, KIND, RW>
                  : (const void *)transport_rows_items_kernel<F, 0, KIND, RW>;
    return o5 ? (const void *)transport_rows_kernel<F, 5, KIND, RW>
              : (const void *)transport_rows_kernel<F, 0, KIND, RW>;
}

// The kernel of a mechanism (fits of 1/D_kj come here below kMfmaMinSpecies only).
template <class F, int FORM> const void *rows_kernel(const MechDev &m)
{
    const bool o5 = m.fit_order == 5;
    const int rw = rows_per_wave(m);
    if (m.diff_kind == 1) return rows_instance<F, FORM, 1, 4>(o5);
    return rw == 4   ? rows_instance<F, FORM, 0, 4>(o5)
           : rw == 8 ? rows_instance<F, FORM, 0, 8>(o5)
                     : rows_instance<F, FORM, 0, 16>(o5);
}

// Whether a call of `points` points takes one thread per two points.  That form has
// no barriers and reads a coefficient once per 128 points, but a wave is a chain of
// ns^2 pairs, and of waves it has rounds of 4 per SIMD, 524288 points (mixed 5, 655360),
// so it is for calls of much of one whose last round is not nearly empty.  There it
// gains where the waves of transport_rows_tile leave much of a CU unused (FP64: 9 to 12
// waves, of which one workgroup fits) and, mixed, where its chains are short.  us, rows
// / lanes, D_kj fits.  FP64: 33 species (9 waves), 350000 points 466 / 388, 2^20 1425 /
// 950; 129 species, 2^20 20956 / 14430; 40 species (10), 300000 points 458 / 502, 450000
// 701 / 660; 48 species (12), 700000 points 1251 / 1339, 2^20 faster; 17 species, 450000
// points 165 / 147, 24 species 400000 points 218 / 240; not with 53 species (14), 600000
// points 1392 / 1679, 2^20 2400 / 2329, but 2^21 with the rates call before it 6900 /
// 7070; 200 species (13), 450000 points 16999 / 17392, 524288 20009 / 18298, 2^20 40095 /
// 33910; not with 128 species (13838 / 15787).  Mixed: 33 species, 450000 points 359 /
// 347, 2^20 849 / 679; 53 species, 2^20 1883 / 1497; 129 species 13488 / 8792; 200
// species, 450000 points 9706 / 10167, 2^20 22215 / 20231; 44 species, 786432 points 833
// / 933, 900000 points equal; 24 species, 700000 points 258 / 281, 2^20 387 / 349; not
// with 48 (1127 / 1188) or 100 species.  Fits of 1/D_kj (below 24 species), 2^20 points:
// 17 species FP64 322 / 302, mixed 278 / 228.
template <class F> bool lanes_form(const MechDev &m, int64_t points)
{
    constexpr bool F64 = sizeof(F) == 8;
    constexpr int64_t round = (F64 ? 4096 : 5120) * (int64_t)kLaneTile;
    const int nw = rows_waves(m), ns = m.ns;
    const int64_t rest = points > round && points % round ? points % round : round;
    if (m.fit_order != 5 || ns < 17 || points < 250000) return false;
    if (F64) {
        if (m.diff_kind == 1) return points > round && rest > round * 9 / 10;
        if (nw == 9) return points >= 300000;
        if (nw <= 11 && nw != 7 && nw != 8) return points >= 420000 && rest >= round / 5;
        if (nw == 12 && points >= 750000) return true;
        return (ns > 64 && (nw == 12 || nw == 13) && points >= 500000 && points <= round) ||
               (ns > 64 && (nw == 13 || nw == 14) && points >= 900000 && rest >= round * 9 / 20);
    }
    if (ns > 128 && nw == 9) return true;
    if (rest < round / 4) return false;
    if (m.diff_kind == 1 || (ns > 32 && ns <= 40) || (ns > 48 && ns <= 56) ||
        (ns > 64 && (nw == 9 || nw == 10)))
        return points >= 450000;
    return (ns <= 44 || (ns > 48 && ns <= 64) || ns > 160) && points >= 900000;
}
template <class F> const void *lanes_kernel(const MechDev &m, bool items)
{
    if (items)
        return m.diff_kind == 0 ? (const void *)transport_lanes_items_kernel<F, 0>
                                : (const void *)transport_lanes_items_kernel<F, 1>;
    return m.diff_kind == 0 ? (const void *)transport_lanes_kernel<F, 0>
                            : (const void *)transport_lanes_kernel<F, 1>;
}

template <class F, int FORM> kx_status rows_prepare(const MechDev &m)
{
    hipError_t e = hipFuncSetAttribute(rows_kernel<F, FORM>(m),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)rows_lds<F>(m));
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute (transport)");
    return KX_OK;
}

template <class F, int FORM>
kx_status rows_launch(const MechDev &m, int64_t grid, void **args, hipStream_t s, const char *what)
{
    hipError_t e = hipLaunchKernel(rows_kernel<F, FORM>(m), dim3((unsigned)grid),
                                   dim3(rows_waves(m) * kWave), args, rows_lds<F>(m), s);
    if (e != hipSuccess) return hip_fail(e, what);
    return ok();
}

// Shape of the matrix-core tile: points and threads.  The prologue gives each
// thread at most 16 species (8 in a 64-point tile of 512 threads).
//  * up to 64 species: 64 points; 512 threads below four row blocks (48 species),
//    where four waves would leave one or two without a block (30 species, 500000
//    points 0.38 -> 0.24 ms, mixed 0.22 -> 0.18); with four blocks four waves
//    already keep the FP64 datapath busy that the products and the vector work
//    share (53 species, 2^20 points: 1.22 ms with 256 threads, 1.24 with 512, mixed
//    0.71 and 0.74);
//  * up to 128: 32 points, 256 threads, two workgroups per CU;
//  * above, FP64: 16 points, 256 threads (32 points leave one workgroup per CU:
//    1.68 against 1.58 ms);
//  * above, mixed: 32 points, 512 threads, two workgroups per CU, or 16 points and
//    256 threads.  us by 32 / 16 points: 200 species, 1000 points 73 / 62 and 4096
//    points 74 / 63 (a tile is a shorter chain, and each has a CU of its own), 8192
//    points 79 / 88, 10000 points 122 / 111 (the first CU with two 32-point tiles),
//    16384 points 125 / 142, 100003 points 746 / 794; with nine row blocks, which eight
//    waves take in two turns (144 species), 32768 points 140 / 145, 100003 points 441 /
//    410; where two 32-point groups do not share a CU's LDS (256 species) 100003 points
//    1289 / 1212, 16384 points 199 / 224.
// Three row blocks, mixed: from 160000 points on the 256-thread groups are the faster
// ones after all (48 species, 131072 points 88 us by 512 threads, 91 by 256; 200000
// points 134 and 134, 524288 points 326 and 312).
// A shape's bits are its partial sums (MfmaShape), so what a mechanism and precision
// use has the same ones throughout; where two shapes do, the number of points decides.
enum MfmaId { k64x512, k64x256, k64x256of8, k32x256, k32x512, k16x256, k16x256of8 };
template <class F> MfmaId mfma_shape(const MechDev &m, int64_t points)
{
    const int kp = 4 * m.kstep;
    constexpr bool F64 = sizeof(F) == 8;
    if (kp <= 64) {
        if (m.mblk >= 4) return k64x256;
        return !F64 && m.mblk == 3 && points >= 160000 ? k64x256of8 : k64x512;
    }
    if (kp <= 128) return k32x256;
    if (F64) return k16x256;
    const bool alone = mfma_lds_bytes<F, MfmaShape<32, 512>>(m.kstep) > 80 * 1024;
    const bool small = points >= 0 && (points <= 4096 || (points > 8192 && points <= 10240));
    const bool large = (m.mblk == 9 && points > 49152) || (alone && points > 16384);
    return small || large ? k16x256of8 : k32x512;
}
constexpr int64_t kAnyPoints = -1;  // the shape of the batch kernels

// f(MfmaShape) of the shape.  The batch kernels' shapes do not depend on the points.
template <class F, int FORM, class Fn> auto with_mfma_shape(MfmaId id, Fn f)
{
    if (id == k64x512) return f(MfmaShape<64, 512>{});
    if constexpr (sizeof(F) == 4) {
        if constexpr (FORM != 1) {
            if (id == k64x256of8) return f(MfmaShape<64, 256, 8>{});
            if (id == k16x256of8) return f(MfmaShape<16, 256, 16, 8>{});
        }
        if (id == k32x512) return f(MfmaShape<32, 512>{});
    } else {
        if (id == k16x256) return f(MfmaShape<16, 256>{});
    }
    if (id == k32x256) return f(MfmaShape<32, 256>{});
    return f(MfmaShape<64, 256>{});
}
template <class F> int mfma_np(const MechDev &m, int64_t points)
{
    return with_mfma_shape<F, 0>(mfma_shape<F>(m, points), [](auto s) { return decltype(s)::NP; });
}
template <class F> int mfma_nt(const MechDev &m, int64_t points)
{
    return with_mfma_shape<F, 0>(mfma_shape<F>(m, points), [](auto s) { return decltype(s)::NT; });
}
template <class F> size_t mfma_lds(const MechDev &m, int64_t points)
{
    return with_mfma_shape<F, 0>(mfma_shape<F>(m, points), [&](auto s) {
        return mfma_lds_bytes<F, decltype(s)>(m.kstep);
    });
}

bool use_mfma(const MechDev &m)
{
    return m.diff_kind == 1 && m.gfrag != nullptr && m.ns >= kMfmaMinSpecies;
}

// FORM 0: direct launch, 1: work-stealing batch, 2: one tile per workgroup
template <class F, int FORM, class S> const void *mfma_instance(bool o5)
{
    if (FORM == 1)
        return o5 ? (const void *)transport_mfma_batch_kernel<F, S, 5>
                  : (const void *)transport_mfma_batch_kernel<F, S, 0>;
    if (FORM == 2)
        return o5 ? (const void *)transport_mfma_items_kernel<F, S, 5>
                  : (const void *)transport_mfma_items_kernel<F, S, 0>;
    return o5 ? (const void *)transport_mfma_kernel<F, S, 5>
              : (const void *)transport_mfma_kernel<F, S, 0>;
}
template <class F, int FORM> const void *mfma_kernel(const MechDev &m, int64_t points)
{
    const bool o5 = m.fit_order == 5;
    return with_mfma_shape<F, FORM>(mfma_shape<F>(m, points), [&](auto s) {
        return mfma_instance<F, FORM, decltype(s)>(o5);
    });
}

template <class F, int FORM> kx_status mfma_prepare(const MechDev &m, int64_t points, size_t *lds)
{
    *lds = mfma_lds<F>(m, points);
    if (*lds > 160 * 1024)
        return fail(KX_EUNSUPPORTED, "transport: mechanism too large for the LDS tiles");
    hipError_t e = hipFuncSetAttribute(mfma_kernel<F, FORM>(m, points),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)*lds);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute (transport)");
    return KX_OK;
}

}  // namespace

int transport_items_tile_points(const MechDev &m, int precision, int64_t points)
{
    if (use_mfma(m))
        return precision == KX_MIXED ? mfma_np<float>(m, points) : mfma_np<double>(m, points);
    if (precision == KX_MIXED ? lanes_form<float>(m, points) : lanes_form<double>(m, points))
        return kLaneTile;
    return kWave;
}

int transport_tile_points(const MechDev &m, int precision)
{
    return transport_items_tile_points(m, precision, kAnyPoints);
}

kx_status prepare_transport_batch(const MechDev &m, int precision)
{
    if (!use_mfma(m))
        return precision == KX_MIXED ? rows_prepare<float, 1>(m) : rows_prepare<double, 1>(m);
    size_t lds = 0;
    return precision == KX_MIXED ? mfma_prepare<float, 1>(m, kAnyPoints, &lds)
                                 : mfma_prepare<double, 1>(m, kAnyPoints, &lds);
}

namespace {
// The arrays of one launch (kernel arguments).
struct TransportPtrs {
    const double *T, *p, *Y;
    double *mu, *lam, *Dmix;
};

template <class F>
kx_status go_transport(const MechDev &m, int64_t n, const double *T, const double *p,
                       const double *Y, double *mu, double *lam, double *Dmix, bool sym,
                       hipStream_t s)
{
    if (sym && m.diff_kind == 0) {
        // one wave per 64 points, the per-lane sums of every species in LDS
        const size_t lds = (size_t)m.ns * kWave * sizeof(F);
        if (lds > 160 * 1024) return fail(KX_EUNSUPPORTED, "transport: symmetric D_kj sums "
                                                           "of this many species exceed the LDS");
        constexpr int KB = 8;
        auto k = m.fit_order == 5 ? transport_sym_kernel<F, 5, KB> : transport_sym_kernel<F, 0, KB>;
        hipError_t e = hipFuncSetAttribute((const void *)k,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute (symmetric transport)");
        const int64_t nblk = (n + kWave - 1) / kWave;
        if (nblk > 0x7fffffff) return fail(KX_EINVAL, "transport: n too large");
        hipLaunchKernelGGL(k, dim3((unsigned)nblk), dim3(kWave), lds, s, m, n, T, p, Y, mu, lam,
                           Dmix);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "symmetric transport kernel launch");
        return ok();
    }
    if (use_mfma(m)) {
        size_t lds = 0;
        kx_status st = mfma_prepare<F, 0>(m, n, &lds);
        if (st != KX_OK) return st;
        const int np = mfma_np<F>(m, n);
        const int64_t nblk = (n + np - 1) / np;
        if (nblk > 0x7fffffff) return fail(KX_EINVAL, "transport: n too large");
        return launch_tiles(n, np, mfma_nt<F>(m, n), [&](int64_t i, int64_t groups) {
            TransportPtrs a{T + i, p + i, Y + i, mu + i, lam + i, Dmix + i};
            void *args[] = {(void *)&m, (void *)&n, &a.T, &a.p, &a.Y, &a.mu, &a.lam, &a.Dmix};
            hipError_t e = hipLaunchKernel(mfma_kernel<F, 0>(m, n), dim3((unsigned)groups),
                                           dim3(mfma_nt<F>(m, n)), args, lds, s);
            return e != hipSuccess ? hip_fail(e, "transport kernel launch") : KX_OK;
        });
    }
    const int64_t nblk = (n + kWave - 1) / kWave;
    if (nblk > 0x7fffffff) return fail(KX_EINVAL, "transport: n too large");
    if (lanes_form<F>(m, n)) {
        int rw = rows_per_wave(m);
        return launch_tiles(n, kLaneTile, kWave, [&](int64_t i, int64_t groups) {
            TransportPtrs a{T + i, p + i, Y + i, mu + i, lam + i, Dmix + i};
            void *args[] = {(void *)&m, &rw, (void *)&n, &a.T, &a.p, &a.Y, &a.mu, &a.lam, &a.Dmix};
            hipError_t e = hipLaunchKernel(lanes_kernel<F>(m, false), dim3((unsigned)groups),
                                           dim3(kWave), args, 0, s);
            return e != hipSuccess ? hip_fail(e, "transport kernel launch") : KX_OK;
        });
    }
    kx_status st = rows_prepare<F, 0>(m);
    if (st != KX_OK) return st;
    return launch_tiles(n, kWave, rows_waves(m) * kWave, [&](int64_t i, int64_t groups) {
        TransportPtrs a{T + i, p + i, Y + i, mu + i, lam + i, Dmix + i};
        void *args[] = {(void *)&m, (void *)&n, &a.T, &a.p, &a.Y, &a.mu, &a.lam, &a.Dmix};
        return rows_launch<F, 0>(m, groups, args, s, "transport kernel launch");
    });
}

template <class F>
kx_status go_transport_batch(const MechDev &m, const WorkList *wl, int *counter, int grid,
                             hipStream_t s)
{
    if (use_mfma(m)) {
        const size_t lds = mfma_lds<F>(m, kAnyPoints);
        void *args[] = {(void *)&m, (void *)&wl, (void *)&counter};
        hipError_t e = hipLaunchKernel(mfma_kernel<F, 1>(m, kAnyPoints), dim3(grid),
                                       dim3(mfma_nt<F>(m, kAnyPoints)), args, lds, s);
        if (e != hipSuccess) return hip_fail(e, "transport batch kernel launch");
        return ok();
    }
    void *args[] = {(void *)&m, (void *)&wl, (void *)&counter};
    return rows_launch<F, 1>(m, grid, args, s, "transport batch kernel launch");
}
template <class F>
kx_status go_transport_items(const MechDev &m, const WorkList *wl, int64_t ntiles, int64_t points,
                             hipStream_t s)
{
    if (ntiles <= 0) return ok();
    if (ntiles > max_workgroups(use_mfma(m) ? mfma_nt<F>(m, points) : rows_waves(m) * kWave))
        return fail(KX_EINVAL, "transport: too many tiles");
    if (use_mfma(m)) {
        size_t lds = 0;
        kx_status st = mfma_prepare<F, 2>(m, points, &lds);
        if (st != KX_OK) return st;
        void *args[] = {(void *)&m, (void *)&wl};
        hipError_t e = hipLaunchKernel(mfma_kernel<F, 2>(m, points), dim3((unsigned)ntiles),
                                       dim3(mfma_nt<F>(m, points)), args, lds, s);
        if (e != hipSuccess) return hip_fail(e, "transport items kernel launch");
        return ok();
    }
    if (lanes_form<F>(m, points)) {
        int rw = rows_per_wave(m);
        void *args[] = {(void *)&m, &rw, (void *)&wl};
        hipError_t e = hipLaunchKernel(lanes_kernel<F>(m, true), dim3((unsigned)ntiles), dim3(kWave),
                                       args, 0, s);
        if (e != hipSuccess) return hip_fail(e, "transport items kernel launch");
        return ok();
    }
    kx_status st = rows_prepare<F, 2>(m);
    if (st != KX_OK) return st;
    void *args[] = {(void *)&m, (void *)&wl};
    return rows_launch<F, 2>(m, ntiles, args, s, "transport items kernel launch");
}
}  // namespace

kx_status launch_transport_items(const MechDev &m, const WorkList *wl, int64_t ntiles,
                                 int64_t points, int precision, hipStream_t s)
{
    if (precision == KX_MIXED) return go_transport_items<float>(m, wl, ntiles, points, s);
    return go_transport_items<double>(m, wl, ntiles, points, s);
}

kx_status launch_transport(const kx_mech *mech, int64_t n, const double *T, const double *p,
                           const double *Y, double *mu, double *lam, double *Dmix,
                           int precision, hipStream_t s)
{
    const bool sym = (precision & KX_DKJ_SYMMETRIC) != 0;
    if ((precision & ~KX_DKJ_SYMMETRIC) == KX_MIXED)
        return go_transport<float>(mech->dev, n, T, p, Y, mu, lam, Dmix, sym, s);
    return go_transport<double>(mech->dev, n, T, p, Y, mu, lam, Dmix, sym, s);
}

kx_status launch_transport_batch(const MechDev &m, const WorkList *wl, int *counter,
                                 int precision, int grid, hipStream_t s)
{
    if (precision == KX_MIXED) return go_transport_batch<float>(m, wl, counter, grid, s);
    return go_transport_batch<double>(m, wl, counter, grid, s);
}

kx_status launch_zero(int *p, int count, hipStream_t s)
{
    hipLaunchKernelGGL(zero_kernel, dim3((count + 63) / 64), dim3(64), 0, s, p, count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "zero kernel launch");
    return ok();
}

kx_status launch_thermo(const kx_mech *mech, int64_t n, const double *T, const double *Y,
                        double *cpk, double *hk, double *cpmix, hipStream_t s)
{
    const int64_t nblk = (n + kWave - 1) / kWave;
    if (nblk > 0x7fffffff) return fail(KX_EINVAL, "thermo: n too large");
    return launch_tiles(n, kWave, kBlock, [&](int64_t i, int64_t groups) {
        hipLaunchKernelGGL(thermo_kernel, dim3((unsigned)groups), dim3(kBlock), 0, s, mech->dev, n,
                           T + i, Y + i, cpk ? cpk + i : cpk, hk ? hk + i : hk,
                           cpmix ? cpmix + i : cpmix);
        hipError_t e = hipGetLastError();
        return e != hipSuccess ? hip_fail(e, "thermo kernel launch") : KX_OK;
    });
}

}  // namespace kx
