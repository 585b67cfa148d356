// kx_mech.cpp -- host-side mechanism table builder (kx_mech_create).
//
// Validates a kx_mech_desc, derives every table the gfx950 kernels read and
// uploads them to the device in one allocation:
//  * reactions re-ordered heaviest type first (Troe, Lindemann, three-body,
//    elementary; constant-k_f reactions last inside each type) so that the
//    falloff code runs in as few 64-lane iterations as possible and a partial
//    last iteration holds the cheapest reactions;
//  * each reaction side as a list of LDS byte offsets, one per molecule, padded
//    with a dummy species whose per-point factors are 1;
//  * ln A, E_R = E_a / R and the beta = E_R = 0 shortcut of eq:k_f;
//  * third-body efficiencies as (alpha - default) lists, falloff k_0 and Troe
//    parameters (inverse temperatures);
//  * the gather lists of wdot_k = sum_i nu_ki R_i: one stream per wave and chunk for
//    the one-lane-per-point kernels, lists of pairs of rate rows for the calls of few
//    points, and where neither runs one list per species and chunk, padded to one trip
//    count and interleaved for coalesced loads (each laid out only for a mechanism
//    whose kernels read it);
//  * Gibbs coefficients of eq:Ck pre-scaled per range, raw NASA-7 for cp / h;
//  * Wilke constants c1_kj = (8 (1 + W_k/W_j))^(-1/2) and W_k^(1/4) (so that
//    (W_j/W_k)^(1/4) separates into per-species factors), and the ln T fit
//    tables in the k-blocked order of the transport kernel, in FP64 and FP32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "kx_internal.h"

namespace kx {
namespace {

struct Blob {
    std::vector<uint8_t> host;
    size_t add(const void *src, size_t bytes)
    {
        size_t off = (host.size() + 255) & ~size_t(255);
        host.resize(off + bytes);
        if (bytes) std::memcpy(host.data() + off, src, bytes);
        return off;
    }
};

template <class T> size_t add_vec(Blob &b, const std::vector<T> &v)
{
    return b.add(v.data(), v.size() * sizeof(T));
}

// Shape of the one-lane-per-point kernels: waves per workgroup and reactions per
// chunk.  The rate rows fill what the species rows leave of a workgroup's share
// of the 160 KB of LDS: as many workgroups per CU as 24 waves allow with at
// least 24 rows each (above 56 species the species rows take more than half of
// the LDS, so one workgroup of 16 waves).  Measured on 2^20 points, 53 species:
// two workgroups of 12 waves 1.00 ms, two of 8 waves 1.28, one of 16 waves with
// 192 rows 1.36.
struct WideShape {
    int nw = 0, chunk = 0, nchunks = 0;
};
WideShape wide_shape(int ns, int nr)
{
    WideShape s;
    if (ns > kWideMaxSpecies) return s;
    s.nw = ns <= 16 ? 4 : (ns <= 32 ? 8 : (ns <= 56 ? 12 : 16));
    const int need = std::min(24, nr);
    int groups = (s.nw == 16 ? 16 : 24) / s.nw, rows = 0;
    for (; groups >= 1; --groups) {
        rows = (160 * 1024 / groups - 256) / 512 - (2 * (ns + 2) + 1);
        if (rows >= need) break;
    }
    s.chunk = std::max(s.nw, std::min({rows, kChunkMax, nr + s.nw - 1}) / s.nw * s.nw);
    s.nchunks = (nr + s.chunk - 1) / s.chunk;
    return s;
}

// The shape for calls of few tiles: every tile has a CU to itself, so 16 waves
// and all of the LDS (53 species, 2000 points: 2 chunks instead of 7, 23 against
// 26 us a call).
WideShape wide_shape_alone(int ns, int nr)
{
    WideShape s;
    s.nw = 16;
    const int rows = (160 * 1024 - 256) / 512 - (2 * (ns + 2) + 1);
    s.chunk = std::max(s.nw, std::min({rows, kChunkMax, nr + s.nw - 1}) / s.nw * s.nw);
    s.nchunks = (nr + s.chunk - 1) / s.chunk;
    return s;
}

// Net stoichiometric coefficient nu''_ki - nu'_ki of species k in reaction i.
int net_nu(const kx_mech_desc *d, int i, int k)
{
    int nu = 0;
    for (int e = d->reac_ptr[i]; e < d->reac_ptr[i + 1]; ++e)
        if (d->reac_sp[e] == k) nu -= d->reac_nu[e];
    for (int e = d->prod_ptr[i]; e < d->prod_ptr[i + 1]; ++e)
        if (d->prod_sp[e] == k) nu += d->prod_nu[e];
    return nu;
}

// (reaction in kernel order, net nu) of every species, one species after another:
// those of species k are row[first[k]] .. row[first[k + 1]] (exclusive).
struct SpeciesRows {
    std::vector<std::pair<int, int>> row;
    std::vector<int> first;
};
SpeciesRows species_rows(const kx_mech_desc *d, const std::vector<int> &perm)
{
    const int ns = d->n_species, nr = d->n_reactions;
    struct Item {
        int k, s, nu;
    };
    std::vector<Item> items;
    items.reserve((size_t)6 * nr);
    SpeciesRows r;
    r.first.assign(ns + 1, 0);
    for (int s = 0; s < nr; ++s) {
        const int i = perm[s];
        const size_t own = items.size();
        for (int side = 0; side < 2; ++side) {
            const int32_t *ptr = side ? d->prod_ptr : d->reac_ptr;
            const int32_t *sp = side ? d->prod_sp : d->reac_sp;
            const int32_t *nu = side ? d->prod_nu : d->reac_nu;
            for (int e = ptr[i]; e < ptr[i + 1]; ++e) {
                const int v = side ? nu[e] : -nu[e];
                size_t q = own;
                while (q < items.size() && items[q].k != sp[e]) ++q;
                if (q < items.size()) {
                    items[q].nu += v;
                } else {
                    items.push_back({sp[e], s, v});
                    ++r.first[sp[e] + 1];
                }
            }
        }
    }
    for (int k = 0; k < ns; ++k) r.first[k + 1] += r.first[k];
    r.row.resize(items.size());
    std::vector<int> at(r.first.begin(), r.first.end() - 1);
    for (const Item &i : items) r.row[at[i.k]++] = {i.s, i.nu};
    return r;
}

// The species of each wave of a shape and the waves' gather streams (WideMap).
void wide_gather(const SpeciesRows &rows, const WideShape &ws, std::vector<int32_t> &species,
                 std::vector<uint32_t> &start, std::vector<uint32_t> &gather)
{
    const int ns = (int)rows.first.size() - 1, nw = ws.nw;
    // longest list first, to the wave with the shortest total so far that has a
    // slot free (a list costs about four entries more than it holds)
    std::vector<int> len(ns, 0), order(ns), load(nw, 0), used(nw, 0);
    for (int k = 0; k < ns; ++k)
        for (int e = rows.first[k]; e < rows.first[k + 1]; ++e) len[k] += std::abs(rows.row[e].second);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return len[a] > len[b]; });
    species.assign((size_t)nw * 8, -1);
    const int cap = (ns + nw - 1) / nw;
    for (int k : order) {
        int best = -1;
        for (int w = 0; w < nw; ++w)
            if (used[w] < cap && (best < 0 || load[w] < load[best])) best = w;
        species[best * 8 + used[best]++] = k;
        load[best] += len[k] + 4;
    }
    for (int w = 0; w < nw; ++w) {
        start.push_back((uint32_t)(gather.size() / 4));
        int at[8] = {};  // next entry of each species' list
        for (int q = 0; q < 8; ++q)
            if (species[w * 8 + q] >= 0) at[q] = rows.first[species[w * 8 + q]];
        for (int c = 0; c < ws.nchunks; ++c) {
            const size_t head = gather.size();
            gather.resize(head + 4, 0);
            for (int q = 0; q < 8; ++q) {
                const int k = species[w * 8 + q];
                if (k < 0) continue;
                const size_t first = gather.size();
                for (; at[q] < rows.first[k + 1] && rows.row[at[q]].first < (c + 1) * ws.chunk;
                     ++at[q]) {
                    const auto &e = rows.row[at[q]];
                    for (int u = 0; u < std::abs(e.second); ++u)
                        gather.push_back((uint32_t)(e.first - c * ws.chunk) |
                                         (e.second < 0 ? 0x80000000u : 0u));
                }
                while (gather.size() % 4) gather.push_back((uint32_t)ws.chunk);
                gather[head + q / 4] |= (uint32_t)((gather.size() - first) / 4) << (8 * (q % 4));
            }
        }
    }
}

// The species' lists of the one-point-per-workgroup kernels; an entry is the last
// of its group where the streams of wide_gather end one: after four entries of a
// chunk, or at the chunk's end.
void few_lists(const SpeciesRows &rows, int nr, int chunk, std::vector<int32_t> &ptr,
               std::vector<uint32_t> &ent)
{
    const int ns = (int)rows.first.size() - 1;
    for (int k = 0; k < ns; ++k) {
        ptr.push_back((int32_t)(ent.size() / 4));
        int group = 0;  // entries of the current group
        for (int e = rows.first[k]; e < rows.first[k + 1]; ++e) {
            const int s = rows.row[e].first, nu = rows.row[e].second;
            for (int u = 0; u < std::abs(nu); ++u) {
                ent.push_back((uint32_t)s | (nu < 0 ? kFewMinus : 0u));
                if (++group == 4) {
                    ent.back() |= kFewLast;
                    group = 0;
                }
            }
            if (group && (e + 1 == rows.first[k + 1] || rows.row[e + 1].first / chunk != s / chunk)) {
                ent.back() |= kFewLast;
                group = 0;
            }
        }
        while (ent.size() % 4) ent.push_back((uint32_t)nr);
    }
    ptr.push_back((int32_t)(ent.size() / 4));
}

// QSS species of one side of reaction i (the first one) and their molecule count.
int qss_side(const kx_mech_desc *d, int i, bool prod, int *count)
{
    const int32_t *ptr = prod ? d->prod_ptr : d->reac_ptr;
    const int32_t *sp = prod ? d->prod_sp : d->reac_sp;
    const int32_t *nu = prod ? d->prod_nu : d->reac_nu;
    int first = -1, c = 0;
    for (int e = ptr[i]; e < ptr[i + 1]; ++e)
        if (d->qss[sp[e]]) {
            if (first < 0) first = sp[e];
            c += nu[e];
        }
    *count = c;
    return first;
}

// The linearised QSSA needs every rate of progress affine in the QSS
// concentrations and every QSS balance to hold a sink.
kx_status validate_qss(const kx_mech_desc *d)
{
    const int ns = d->n_species, nr = d->n_reactions;
    int nq = 0;
    for (int k = 0; k < ns; ++k) {
        if (d->qss[k] != 0 && d->qss[k] != 1)
            return fail(KX_EINVAL, "kx_mech_create: qss flags must be 0 or 1");
        nq += d->qss[k];
    }
    if (nq > kMaxQss)
        return fail(KX_EUNSUPPORTED, "kx_mech_create: at most 64 QSS species are supported");
    if (nq == ns) return fail(KX_EINVAL, "kx_mech_create: every species is QSS");
    std::vector<char> consumed(ns, 0);
    for (int i = 0; i < nr; ++i) {
        const std::string ri = " (reaction " + std::to_string(i) + ")";
        int cr = 0, cp = 0;
        qss_side(d, i, false, &cr);
        qss_side(d, i, true, &cp);
        if (cr > 1 || cp > 1)
            return fail(KX_EUNSUPPORTED, "kx_mech_create: two QSS molecules on one side of a "
                                         "reaction" + ri);
        const int t = d->rxn_type[i];
        if (t != KX_RXN_ELEMENTARY && t != KX_RXN_PLOG)
            for (int e = d->eff_ptr[i]; e < d->eff_ptr[i + 1]; ++e)
                if (d->qss[d->eff_sp[e]])
                    return fail(KX_EUNSUPPORTED, "kx_mech_create: QSS species in an "
                                                 "efficiency list" + ri);
        if (d->ord_ptr && d->ord_ptr[i + 1] > d->ord_ptr[i]) {
            bool any = cr > 0 || cp > 0;
            for (int e = d->ord_ptr[i]; e < d->ord_ptr[i + 1]; ++e) any |= d->qss[d->ord_sp[e]] != 0;
            if (any)
                return fail(KX_EUNSUPPORTED, "kx_mech_create: QSS species in a reaction with "
                                             "explicit orders" + ri);
        }
        for (int k = 0; k < ns; ++k) {
            if (!d->qss[k]) continue;
            const int nu = net_nu(d, i, k);
            if (nu < 0 || (nu > 0 && d->reversible[i])) consumed[k] = 1;
        }
    }
    for (int k = 0; k < ns; ++k)
        if (d->qss[k] && !consumed[k])
            return fail(KX_EINVAL, "kx_mech_create: QSS species " + std::to_string(k) +
                                       " is consumed by no reaction");
    return KX_OK;
}

kx_status validate(const kx_mech_desc *d, std::vector<double> &W)
{
    if (!d) return fail(KX_EINVAL, "kx_mech_create: desc is NULL");
    const int ns = d->n_species, nr = d->n_reactions, ne = d->n_elements;
    if (ns <= 0 || nr < 0 || ne <= 0)
        return fail(KX_EINVAL, "kx_mech_create: n_species and n_elements must be > 0, "
                               "n_reactions >= 0");
    if (ns > kMaxSpecies)
        return fail(KX_EUNSUPPORTED, "kx_mech_create: at most 256 species are supported");
    if (!d->elem_mass || !d->composition || !d->nasa_lo || !d->nasa_hi || !d->t_mid ||
        !d->visc_fit || !d->cond_fit || !d->diff_fit)
        return fail(KX_EINVAL, "kx_mech_create: NULL species array");
    if (nr > 0 && (!d->rxn_type || !d->reversible || !d->reac_ptr || !d->reac_sp ||
                   !d->reac_nu || !d->prod_ptr || !d->prod_sp || !d->prod_nu || !d->A ||
                   !d->beta || !d->Ea || !d->A0 || !d->beta0 || !d->Ea0 || !d->troe ||
                   !d->eff_ptr || !d->eff_default))
        return fail(KX_EINVAL, "kx_mech_create: NULL reaction array");
    if (d->fit_order < 1 || d->fit_order > kMaxFitOrder)
        return fail(KX_EINVAL, "kx_mech_create: fit_order must be in 1..8");
    if (!(d->fit_h != 0.0) || !std::isfinite(d->fit_h) || !std::isfinite(d->fit_L0))
        return fail(KX_EINVAL, "kx_mech_create: fit_h must be finite and non-zero");
    if (d->diff_fit_kind != 0 && d->diff_fit_kind != 1)
        return fail(KX_EINVAL, "kx_mech_create: diff_fit_kind must be 0 or 1");
    W.assign(ns, 0.0);
    for (int k = 0; k < ns; ++k) {
        for (int e = 0; e < ne; ++e) {
            if (d->composition[k * ne + e] < 0)
                return fail(KX_EINVAL, "kx_mech_create: negative atom count");
            W[k] += d->composition[k * ne + e] * d->elem_mass[e];
        }
        if (!(W[k] > 0.0))
            return fail(KX_EINVAL, "kx_mech_create: species " + std::to_string(k) +
                                       " has non-positive molecular weight");
    }
    const int order = d->fit_order;
    for (int k = 0; k < ns; ++k)
        for (int j = 0; j < ns; ++j)
            for (int o = 0; o < order; ++o)
                if (d->diff_fit[((size_t)k * ns + j) * order + o] !=
                    d->diff_fit[((size_t)j * ns + k) * order + o])
                    return fail(KX_EINVAL, "kx_mech_create: diff_fit is not symmetric");
    for (int i = 0; i < nr; ++i) {
        const std::string ri = " (reaction " + std::to_string(i) + ")";
        const int t = d->rxn_type[i];
        if (t < KX_RXN_ELEMENTARY || t > KX_RXN_PLOG)
            return fail(KX_EINVAL, "kx_mech_create: unknown reaction type" + ri);
        const bool falloff = t == KX_RXN_LINDEMANN || t == KX_RXN_TROE || t == KX_RXN_SRI;
        if (t == KX_RXN_PLOG) {
            if (!d->plog_ptr || !d->plog_p || !d->plog_A || !d->plog_beta || !d->plog_Ea)
                return fail(KX_EINVAL, "kx_mech_create: NULL PLOG array" + ri);
            const int b = d->plog_ptr[i], e = d->plog_ptr[i + 1];
            if (b < 0 || e <= b)
                return fail(KX_EINVAL, "kx_mech_create: PLOG reaction without pressures" + ri);
            for (int j = b; j < e; ++j) {
                if (!(d->plog_p[j] > 0.0) || !std::isfinite(d->plog_p[j]) ||
                    (j > b && !(d->plog_p[j] > d->plog_p[j - 1])))
                    return fail(KX_EINVAL, "kx_mech_create: PLOG pressures must be positive "
                                           "and strictly increasing" + ri);
                if (!(d->plog_A[j] > 0.0) || !std::isfinite(d->plog_A[j]) ||
                    !std::isfinite(d->plog_beta[j]) || !std::isfinite(d->plog_Ea[j]))
                    return fail(KX_EINVAL, "kx_mech_create: PLOG A must be > 0, beta and "
                                           "Ea finite" + ri);
            }
        } else if (!(d->A[i] > 0.0) || !std::isfinite(d->A[i]) || !std::isfinite(d->beta[i]) ||
                   !std::isfinite(d->Ea[i])) {
            return fail(KX_EINVAL, "kx_mech_create: A must be > 0, beta and Ea finite" + ri);
        }
        if (d->ord_ptr && d->ord_ptr[i + 1] > d->ord_ptr[i]) {
            if (!d->ord_sp || !d->ord_val || d->ord_ptr[i] < 0)
                return fail(KX_EINVAL, "kx_mech_create: bad order arrays" + ri);
            if (d->reversible[i])
                return fail(KX_EINVAL, "kx_mech_create: explicit orders need an "
                                       "irreversible reaction" + ri);
            for (int e = d->ord_ptr[i]; e < d->ord_ptr[i + 1]; ++e) {
                if (d->ord_sp[e] < 0 || d->ord_sp[e] >= ns)
                    return fail(KX_EINVAL, "kx_mech_create: order species out of range" + ri);
                if (!(d->ord_val[e] >= 0.0) || !std::isfinite(d->ord_val[e]))
                    return fail(KX_EINVAL, "kx_mech_create: orders must be finite and >= 0" +
                                               ri);
                for (int f = d->ord_ptr[i]; f < e; ++f)
                    if (d->ord_sp[f] == d->ord_sp[e])
                        return fail(KX_EINVAL, "kx_mech_create: order listed twice" + ri);
            }
        }
        if (d->chem_act && d->chem_act[i] && !falloff)
            return fail(KX_EINVAL, "kx_mech_create: chem_act on a reaction that is not a "
                                   "falloff reaction" + ri);
        if (t == KX_RXN_SRI) {
            if (!d->sri) return fail(KX_EINVAL, "kx_mech_create: NULL sri array" + ri);
            const double *q = d->sri + 5 * i;
            for (int j = 0; j < 5; ++j)
                if (!std::isfinite(q[j]))
                    return fail(KX_EINVAL, "kx_mech_create: SRI parameters must be finite" + ri);
            if (!(q[0] >= 0.0) || !(q[2] != 0.0) || !(q[3] > 0.0))
                return fail(KX_EINVAL, "kx_mech_create: SRI needs a >= 0, c != 0, d > 0" + ri);
        }
        if (falloff &&
            (!(d->A0[i] > 0.0) || !std::isfinite(d->beta0[i]) || !std::isfinite(d->Ea0[i])))
            return fail(KX_EINVAL, "kx_mech_create: falloff A0 must be > 0" + ri);
        if (t == KX_RXN_TROE && (!(d->troe[4 * i + 1] != 0.0) || !(d->troe[4 * i + 2] != 0.0)))
            return fail(KX_EINVAL, "kx_mech_create: Troe T*** and T* must be non-zero" + ri);
        std::vector<long> bal(ne, 0);
        for (int side = 0; side < 2; ++side) {
            const int32_t *ptr = side ? d->prod_ptr : d->reac_ptr;
            const int32_t *sp = side ? d->prod_sp : d->reac_sp;
            const int32_t *nu = side ? d->prod_nu : d->reac_nu;
            if (ptr[i] < 0 || ptr[i + 1] < ptr[i])
                return fail(KX_EINVAL, "kx_mech_create: bad CSR pointer" + ri);
            long molecules = 0;
            for (int e = ptr[i]; e < ptr[i + 1]; ++e) molecules += nu[e] > 0 ? nu[e] : 0;
            if (molecules > kMaxSide)
                return fail(KX_EUNSUPPORTED,
                            "kx_mech_create: more than 3 molecules on one side" + ri);
            for (int e = ptr[i]; e < ptr[i + 1]; ++e) {
                if (sp[e] < 0 || sp[e] >= ns)
                    return fail(KX_EINVAL, "kx_mech_create: species index out of range" + ri);
                if (nu[e] <= 0 || nu[e] > 255)
                    return fail(KX_EINVAL, "kx_mech_create: nu must be in 1..255" + ri);
                for (int f = ptr[i]; f < e; ++f)
                    if (sp[f] == sp[e])
                        return fail(KX_EINVAL,
                                    "kx_mech_create: species listed twice on one side" + ri);
                for (int el = 0; el < ne; ++el)
                    bal[el] += (side ? 1 : -1) * (long)nu[e] * d->composition[sp[e] * ne + el];
            }
        }
        for (int el = 0; el < ne; ++el)
            if (bal[el] != 0)
                return fail(KX_EINVAL, "kx_mech_create: reaction is not element-balanced" + ri);
        if (t != KX_RXN_ELEMENTARY && t != KX_RXN_PLOG) {
            if (d->eff_ptr[i] < 0 || d->eff_ptr[i + 1] < d->eff_ptr[i])
                return fail(KX_EINVAL, "kx_mech_create: bad efficiency CSR" + ri);
            for (int e = d->eff_ptr[i]; e < d->eff_ptr[i + 1]; ++e)
                if (!d->eff_sp || !d->eff_val || d->eff_sp[e] < 0 || d->eff_sp[e] >= ns)
                    return fail(KX_EINVAL, "kx_mech_create: efficiency species out of range" + ri);
        }
    }
    if (d->qss) return validate_qss(d);
    return KX_OK;
}

// Tables of the Jacobian in row blocks: which slot derivatives of which reactions
// add up to each element.  A reaction's slot derivatives, in this order: its
// reactant molecules (or the species of explicit orders), its product molecules
// if reversible, its listed colliders, and the part that is the same for every
// column.
struct JacTables {
    int nv = 0, rows = 0, nblk = 0, pts = 2;
    std::vector<uint32_t> val;
    std::vector<int32_t> ptr;
    std::vector<uint2> list, ent;
    std::vector<uint16_t> tgt;
};

void jac_tables(const kx_mech_desc *d, const std::vector<int> &perm, const std::vector<DevRxn> &rx,
                const std::vector<DevAux> &aux, const std::vector<DevEff> &eff, JacTables &t)
{
    const int ns = d->n_species, nr = d->n_reactions;
    if (ns > kJacBlockSpecies || nr == 0) return;
    if (d->qss && std::any_of(d->qss, d->qss + ns, [](int32_t q) { return q != 0; })) return;
    const int dense = ns;  // pseudo column
    // contributions to (row, column), |nu| times: slot derivative and sign
    struct Item {
        uint32_t el;
        uint16_t val;
    };
    std::vector<Item> items;
    items.reserve((size_t)32 * nr);
    std::vector<uint32_t> first((size_t)ns * (ns + 1) + 1, 0);  // of an element's list
    t.val.reserve(nr);
    std::vector<std::pair<int, int>> net;
    for (int s = 0; s < nr; ++s) {
        const DevRxn &r = rx[s];
        const int i = perm[s];
        net.clear();
        for (int side = 0; side < 2; ++side) {
            const int32_t *ptr = side ? d->prod_ptr : d->reac_ptr;
            for (int e = ptr[i]; e < ptr[i + 1]; ++e) {
                const int k = (side ? d->prod_sp : d->reac_sp)[e];
                const int v = side ? d->prod_nu[e] : -d->reac_nu[e];
                bool found = false;
                for (auto &q : net)
                    if (q.first == k) q.second += v, found = true;
                if (!found) net.push_back({k, v});
            }
        }
        t.val.push_back((uint32_t)t.nv);
        auto add = [&](int column) {
            if (t.nv >= 0x7FFF) {
                t.nv = 0x8000;
                return;
            }
            for (auto &q : net)
                for (int u = 0; u < std::abs(q.second); ++u) {
                    const uint32_t e = (uint32_t)(q.first * (ns + 1) + column);
                    items.push_back({e, (uint16_t)(t.nv | (q.second < 0 ? 0x8000 : 0))});
                    ++first[e + 1];
                }
            ++t.nv;
        };
        const DevAux *ax = r.aux == 0xFFFF ? nullptr : &aux[r.aux];
        if (r.flags & kFlagOrders) {
            for (int e = 0; e < kMaxOrd; ++e)
                if (ax->oval[e] != 0.0) add(ax->ooff[e] / 16);
        } else {
            for (int q = 0; q < kMaxSide; ++q)
                if (r.roff[q] != 16 * ns) add(r.roff[q] / 16);
        }
        if (r.flags & kFlagReversible)
            for (int q = 0; q < kMaxSide; ++q)
                if (r.poff[q] != 16 * ns) add(r.poff[q] / 16);
        if (r.type != KX_RXN_ELEMENTARY && r.type != KX_RXN_PLOG) {
            for (int e = 0; e < ax->eff_cnt; ++e) add(ax->eoff[e] / 16);
            for (int e = 0; e < ax->ext_cnt; ++e) add(eff[ax->ext_off + e].sp);
        }
        if (r.type != KX_RXN_ELEMENTARY) add(dense);
        if (t.nv > 0x7FFF) break;
    }
    // points per workgroup and rows per block: the most points with which four
    // workgroups share a CU's LDS, each with at least eight rows; two points and
    // fewer workgroups if there is no such number
    int rows = 0;
    const int need = std::min(8, ns);
    auto fit = [&](int pts, int groups) {
        const size_t share = 160 * 1024 / groups;
        const size_t fixed = 8 * (size_t)pts * ((size_t)t.nv + 1 + 2 * (ns + 1) + 4) + 16;
        return share > fixed ? (int)std::min<size_t>((share - fixed) / (8 * pts * (ns + 1)), ns) : 0;
    };
    for (t.pts = 8; t.pts > 2 && (rows = fit(t.pts, 4)) < need;) t.pts /= 2;
    if (t.pts == 2)
        for (int groups = 4; groups >= 1 && (rows = fit(2, groups)) < need;) --groups;
    if (t.nv > 0x7FFF || rows == 0) {
        t = JacTables();
        return;
    }
    // the lists one after another
    for (size_t e = 1; e < first.size(); ++e) first[e] += first[e - 1];
    std::vector<uint16_t> el(items.size() + 1);
    {
        std::vector<uint32_t> at(first.begin(), first.end() - 1);
        for (const Item &i : items) el[at[i.el]++] = i.val;
    }
    auto length = [&](int e) { return first[e + 1] - first[e]; };
    t.nblk = (ns + rows - 1) / rows;
    t.rows = (ns + t.nblk - 1) / t.nblk;
    t.ptr.push_back(0);
    std::vector<int> order;
    std::vector<uint32_t> bucket;
    for (int b = 0; b < t.nblk; ++b) {
        // the elements of the block, longest list first, 64 to a lane block
        const int r0 = b * t.rows, r1 = std::min(ns, r0 + t.rows);
        const int e0 = r0 * (ns + 1), e1 = r1 * (ns + 1);
        uint32_t longest = 0;
        for (int e = e0; e < e1; ++e) longest = std::max(longest, length(e));
        bucket.assign(longest + 2, 0);
        for (int e = e0; e < e1; ++e) ++bucket[longest - length(e) + 1];
        for (uint32_t l = 1; l <= longest; ++l) bucket[l] += bucket[l - 1];
        order.resize(e1 - e0);
        for (int e = e0; e < e1; ++e) order[bucket[longest - length(e)]++] = e;
        for (size_t o = 0; o < order.size(); o += 64) {
            const size_t len = length(order[o]), words = (len + 3) / 4, at = t.ent.size();
            t.list.push_back(uint2{(uint32_t)(at / 64), (uint32_t)len});
            const uint32_t zero = (uint32_t)t.nv | (uint32_t)t.nv << 16;
            t.ent.resize(at + 64 * words, uint2{zero, zero});
            t.tgt.resize(t.tgt.size() + 64, 0xFFFF);
            uint16_t *tgt = t.tgt.data() + t.tgt.size() - 64;
            for (size_t l = 0; l < std::min<size_t>(64, order.size() - o); ++l) {
                const int e = order[o + l], k = e / (ns + 1), j = e % (ns + 1);
                tgt[l] = (uint16_t)(j < ns ? (k - r0) * ns + j : t.rows * ns + k - r0);
                for (uint32_t u = 0; u < length(e); ++u) {
                    uint2 &w = t.ent[at + 64 * (u / 4) + l];
                    uint32_t &half = u & 2 ? w.y : w.x;
                    const uint32_t v = el[first[e] + u];
                    half = u & 1 ? (half & 0xFFFFu) | v << 16 : (half & 0xFFFF0000u) | v;
                }
            }
        }
        t.ptr.push_back((int32_t)t.list.size());
    }
    t.ent.resize(t.ent.size() + 64);  // an empty list's first word is read, not used
}

}  // namespace

namespace {
std::atomic<uint64_t> next_uid{0};
}  // namespace

kx_status build_mech(const kx_mech_desc *d, int device, bool host_only, kx_mech **out)
{
    if (!out) return fail(KX_EINVAL, "kx_mech_create: out is NULL");
    *out = nullptr;
    std::vector<double> W;
    kx_status st = validate(d, W);
    if (st != KX_OK) return st;
    const int ns = d->n_species, nr = d->n_reactions, order = d->fit_order;

    // ---- reaction order: heaviest type first, constant-k_f last within a type
    std::vector<int> perm(nr);
    std::iota(perm.begin(), perm.end(), 0);
    auto kfconst = [&](int i) {
        return d->rxn_type[i] != KX_RXN_PLOG && d->beta[i] == 0.0 && d->Ea[i] == 0.0;
    };
    std::stable_sort(perm.begin(), perm.end(), [&](int a, int b) {
        if (d->rxn_type[a] != d->rxn_type[b]) return d->rxn_type[a] > d->rxn_type[b];
        return !kfconst(a) && kfconst(b);
    });

    std::vector<DevRxn> rx(nr);
    std::vector<DevAux> aux;
    std::vector<DevEff> eff;
    std::vector<DevPlog> plog;
    for (int s = 0; s < nr; ++s) {
        const int i = perm[s];
        DevRxn r;
        std::memset(&r, 0, sizeof r);
        r.lnA = std::log(d->A[i]);
        r.beta = d->beta[i];
        r.ER = d->Ea[i] / kRcal;
        r.A = d->A[i];
        const uint16_t dummy = (uint16_t)(16 * ns);
        for (int q = 0; q < kMaxSide; ++q) r.roff[q] = r.poff[q] = dummy;
        int c = 0;
        for (int e = d->reac_ptr[i]; e < d->reac_ptr[i + 1]; ++e)
            for (int v = 0; v < d->reac_nu[e]; ++v) r.roff[c++] = (uint16_t)(16 * d->reac_sp[e]);
        c = 0;
        for (int e = d->prod_ptr[i]; e < d->prod_ptr[i + 1]; ++e)
            for (int v = 0; v < d->prod_nu[e]; ++v) r.poff[c++] = (uint16_t)(16 * d->prod_sp[e]);
        r.type = (uint8_t)d->rxn_type[i];
        r.flags = (d->reversible[i] ? kFlagReversible : 0) | (kfconst(i) ? kFlagKfConst : 0) |
                  (d->chem_act && d->chem_act[i] ? kFlagChemAct : 0);
        if (r.type == KX_RXN_PLOG) {  // k_f comes from the pressure table
            r.lnA = 0.0;
            r.beta = r.ER = 0.0;
            r.A = 1.0;
        }
        // forward orders: reactants at nu' unless listed, listed species at
        // their order; zero orders dropped
        std::vector<std::pair<int, double>> ord;
        const bool has_ord = d->ord_ptr && d->ord_ptr[i + 1] > d->ord_ptr[i];
        if (has_ord) {
            for (int e = d->reac_ptr[i]; e < d->reac_ptr[i + 1]; ++e)
                ord.push_back({d->reac_sp[e], (double)d->reac_nu[e]});
            for (int e = d->ord_ptr[i]; e < d->ord_ptr[i + 1]; ++e) {
                bool found = false;
                for (auto &o : ord)
                    if (o.first == d->ord_sp[e]) {
                        o.second = d->ord_val[e];
                        found = true;
                    }
                if (!found) ord.push_back({d->ord_sp[e], d->ord_val[e]});
            }
            ord.erase(std::remove_if(ord.begin(), ord.end(),
                                     [](const std::pair<int, double> &o) { return o.second == 0.0; }),
                      ord.end());
            if ((int)ord.size() > kMaxOrd)
                return fail(KX_EUNSUPPORTED, "kx_mech_create: more than 4 species with "
                                             "explicit orders (reaction " + std::to_string(i) + ")");
            r.flags |= kFlagOrders;
        }
        r.aux = 0xFFFF;
        if (r.type != KX_RXN_ELEMENTARY || has_ord) {
            if (aux.size() >= 0xFFFF)
                return fail(KX_EUNSUPPORTED, "kx_mech_create: too many non-elementary reactions");
            DevAux a;
            std::memset(&a, 0, sizeof a);
            const bool collider = r.type != KX_RXN_PLOG && r.type != KX_RXN_ELEMENTARY;
            a.eff_default = collider ? d->eff_default[i] : 0.0;
            for (int q = 0; q < kInlineEff; ++q) {
                a.eoff[q] = (uint16_t)(16 * ns);  // dummy species, alpha - default = 0
                a.dalpha[q] = 0.0;
            }
            int q = 0;
            a.ext_off = (int32_t)eff.size();
            const int e0 = collider ? d->eff_ptr[i] : 0, e1 = collider ? d->eff_ptr[i + 1] : 0;
            for (int e = e0; e < e1; ++e) {
                const double da = d->eff_val[e] - d->eff_default[i];
                if (q < kInlineEff) {
                    a.eoff[q] = (uint16_t)(16 * d->eff_sp[e]);
                    a.dalpha[q] = da;
                    ++q;
                } else {
                    DevEff f;
                    std::memset(&f, 0, sizeof f);
                    f.sp = d->eff_sp[e];
                    f.dalpha = da;
                    eff.push_back(f);
                }
            }
            a.eff_cnt = q;
            a.ext_cnt = (int32_t)eff.size() - a.ext_off;
            if (r.type == KX_RXN_LINDEMANN || r.type == KX_RXN_TROE || r.type == KX_RXN_SRI) {
                a.lnA0 = std::log(d->A0[i]);
                a.beta0 = d->beta0[i];
                a.ER0 = d->Ea0[i] / kRcal;
            }
            if (r.type == KX_RXN_TROE) {
                a.fp[0] = d->troe[4 * i + 0];
                a.fp[1] = 1.0 / d->troe[4 * i + 1];
                a.fp[2] = 1.0 / d->troe[4 * i + 2];
                a.has_T2 = std::isnan(d->troe[4 * i + 3]) ? 0 : 1;
                a.fp[3] = a.has_T2 ? d->troe[4 * i + 3] : 0.0;
            }
            if (r.type == KX_RXN_SRI) {
                const double *q = d->sri + 5 * i;
                a.fp[0] = q[0];
                a.fp[1] = q[1];
                a.fp[2] = 1.0 / q[2];
                a.fp[3] = std::log(q[3]);
                a.fp[4] = q[4];
            }
            for (int q = 0; q < kMaxOrd; ++q) {
                a.ooff[q] = (uint16_t)(16 * ns);
                a.oval[q] = 0.0;
            }
            for (size_t q = 0; q < ord.size(); ++q) {
                a.ooff[q] = (uint16_t)(16 * ord[q].first);
                a.oval[q] = ord[q].second;
            }
            if (r.type == KX_RXN_PLOG) {
                a.plog_off = (int32_t)plog.size();
                a.plog_cnt = d->plog_ptr[i + 1] - d->plog_ptr[i];
                for (int j = d->plog_ptr[i]; j < d->plog_ptr[i + 1]; ++j) {
                    DevPlog e;
                    std::memset(&e, 0, sizeof e);
                    e.lnp = std::log(d->plog_p[j]);
                    e.lnA = std::log(d->plog_A[j]);
                    e.beta = d->plog_beta[j];
                    e.ER = d->plog_Ea[j] / kRcal;
                    e.inv_dlnp = j + 1 < d->plog_ptr[i + 1]
                                     ? 1.0 / (std::log(d->plog_p[j + 1]) - e.lnp) : 0.0;
                    plog.push_back(e);
                }
            }
            r.aux = (uint16_t)aux.size();
            aux.push_back(a);
        }
        rx[s] = r;
    }
    if (eff.empty()) eff.resize(1);
    if (aux.empty()) aux.resize(1);
    if (plog.empty()) plog.resize(1);

    // ---- chunks of the species-major gather lists (below)
    const int chunk = std::max(kWave, std::min(kChunkMax, (nr + kWave - 1) / kWave * kWave));
    const int nchunks = std::max(1, (nr + chunk - 1) / chunk);
    // species per lane of the species phases: 1, 2 or 4, so lists are laid out for
    // 64 * gpass lanes
    const int gpass = ns <= kWave ? 1 : (ns <= 2 * kWave ? 2 : 4);
    const int gw = kWave * gpass;

    // ---- QSS species: index per species, per reaction (kernel order) the QSS
    // species of either side, and per QSS species the reactions of its balance
    int nq = 0;
    std::vector<int32_t> qidx(ns, -1);
    if (d->qss)
        for (int k = 0; k < ns; ++k)
            if (d->qss[k]) qidx[k] = nq++;
    std::vector<int2> qrx(std::max(nr, 1), int2{-1, -1});
    std::vector<int32_t> qrow_ptr(nq + 1, 0);
    std::vector<int4> qrow_ent;
    if (nq > 0) {
        for (int s = 0; s < nr; ++s) {
            int c = 0;
            const int a = qss_side(d, perm[s], false, &c), b = qss_side(d, perm[s], true, &c);
            qrx[s] = int2{a >= 0 ? qidx[a] : -1, b >= 0 ? qidx[b] : -1};
        }
        for (int k = 0; k < ns; ++k) {
            if (qidx[k] < 0) continue;
            for (int s = 0; s < nr; ++s) {
                const int nu = net_nu(d, perm[s], k);
                // x: the reaction's LDS slot in the QSS kernel (a zero slot
                // follows each chunk, so reaction s sits at s + s / chunk)
                if (nu != 0) qrow_ent.push_back(int4{s + s / chunk, nu, qrx[s].x, qrx[s].y});
            }
            qrow_ptr[qidx[k] + 1] = (int32_t)qrow_ent.size();
        }
    }
    if (qrow_ent.empty()) qrow_ent.push_back(int4{0, 0, -1, -1});
    // the balances of the one-lane-per-point kernel: the reactions that enter
    // them, and per balance row the streams of its columns (rate rows 2 r and
    // 2 r + 1 hold the forward and reverse terms of reaction r of a chunk)
    std::vector<int32_t> qsp, qlist;
    std::vector<uint32_t> qstart, qgather, qfent;
    std::vector<int32_t> qfptr, qinfo;
    int qchunk = 0;
    {
        const WideShape q = wide_shape(ns, nr);
        if (nq > 0 && nq <= std::min(kWideQss, q.nw)) {
            std::vector<int> seen(nr, -1);
            for (int k = 0; k < ns; ++k)
                if (qidx[k] >= 0) qsp.push_back(k);
            for (int s = 0; s < nr; ++s)
                for (int k : qsp)
                    if (seen[s] < 0 && net_nu(d, perm[s], k) != 0) {
                        seen[s] = (int)qlist.size();
                        qlist.push_back(s);
                    }
            qchunk = std::max(1, q.chunk / 2);
            const int nqr = (int)qlist.size();
            for (int j = 0; j < nq; ++j) {
                qstart.push_back((uint32_t)(qgather.size() / 4));
                for (int c0 = 0; c0 < nqr; c0 += qchunk) {
                    const size_t head = qgather.size();
                    qgather.resize(head + 4, 0);
                    for (int col = 0; col <= nq; ++col) {
                        const size_t first = qgather.size();
                        for (int r = c0; r < std::min(nqr, c0 + qchunk); ++r) {
                            const int s = qlist[r], nu = net_nu(d, perm[s], qsp[j]);
                            for (int side = 0; side < 2; ++side) {
                                const int at = side ? qrx[s].y : qrx[s].x;
                                if ((at >= 0 ? at : nq) != col) continue;
                                for (int u = 0; u < std::abs(nu); ++u)
                                    qgather.push_back((uint32_t)(2 * (r - c0) + side) |
                                                      ((nu < 0) != (side == 1) ? 0x80000000u : 0u));
                            }
                        }
                        while (qgather.size() % 4) qgather.push_back((uint32_t)(2 * qchunk));
                        qgather[head + col / 4] |= (uint32_t)((qgather.size() - first) / 4)
                                                   << (8 * (col % 4));
                    }
                }
            }
            // one point per workgroup: the same entries, a list per (row, column)
            qinfo.assign(nr, -1);
            for (int s = 0; s < nr; ++s)
                if (qrx[s].x >= 0 || qrx[s].y >= 0) qinfo[s] = seen[s] < 0 ? -2 : seen[s];
            for (int j = 0; j < nq; ++j)
                for (int col = 0; col <= nq; ++col) {
                    qfptr.push_back((int32_t)(qfent.size() / 4));
                    for (int r = 0; r < nqr; ++r) {
                        const int s = qlist[r], nu = net_nu(d, perm[s], qsp[j]);
                        for (int side = 0; nu != 0 && side < 2; ++side) {
                            const int at = side ? qrx[s].y : qrx[s].x;
                            if ((at >= 0 ? at : nq) != col) continue;
                            for (int u = 0; u < std::abs(nu); ++u)
                                qfent.push_back((uint32_t)(2 * r + side) |
                                                ((nu < 0) != (side == 1) ? kFewMinus : 0u));
                        }
                    }
                    while (qfent.size() % 4) qfent.push_back((uint32_t)(2 * nqr));
                }
            qfptr.push_back((int32_t)(qfent.size() / 4));
        }
    }

    // ---- species thermo
    std::vector<DevSpecies> spv(ns);
    for (int k = 0; k < ns; ++k) {
        DevSpecies s;
        std::memset(&s, 0, sizeof s);
        for (int r = 0; r < 2; ++r) {
            const double *a = (r ? d->nasa_hi : d->nasa_lo) + 7 * k;
            double *g = r ? s.g_hi : s.g_lo;
            g[0] = a[0];
            g[1] = -a[1] / 2.0;
            g[2] = -a[2] / 6.0;
            g[3] = -a[3] / 12.0;
            g[4] = -a[4] / 20.0;
            g[5] = a[5];
            g[6] = -a[6];
            std::memcpy(r ? s.nasa_hi : s.nasa_lo, a, 7 * sizeof(double));
        }
        s.t_mid = d->t_mid[k];
        s.inv_W = 1.0 / W[k];
        spv[k] = s;
    }
    std::vector<double> gsoa(ns > kWideMaxSpecies ? (size_t)((ns + kWave - 1) / kWave) * 16 * kWave
                                                  : 0);
    for (int k = 0; k < ns && !gsoa.empty(); ++k) {
        double *g = gsoa.data() + (size_t)(k / kWave) * 16 * kWave + k % kWave;
        for (int e = 0; e < 7; ++e) {
            g[e * kWave] = spv[k].g_lo[e];
            g[(7 + e) * kWave] = spv[k].g_hi[e];
        }
        g[14 * kWave] = spv[k].t_mid;
        g[15 * kWave] = spv[k].inv_W;
    }

    // ---- tables of the one-lane-per-point kernels (kx_wide.h)
    const WideShape ws = wide_shape(ns, nr);
    const long double kLog2e = 1.44269504088896340735992468100189214L;
    std::vector<DevWide> wrx, wrx32;
    std::vector<DevAux> waux;
    std::vector<DevPlog> wplog;
    std::vector<double> wsp;
    WideShape wsh[3];
    std::vector<int32_t> wmap[3];
    std::vector<uint32_t> wstart[3], wgat[3];
    int wsame[3] = {0, 1, 2};
    std::vector<int32_t> fptr;
    std::vector<uint32_t> fent;
    int nplog = 0;
    if (ws.nw > 0) {
        for (int s = 0; s < nr; ++s) {
            const DevRxn &r = rx[s];
            const int i = perm[s];
            DevWide v;
            const uint32_t dummy = (uint32_t)ns;
            uint32_t o[2 * kMaxSide];
            for (int q = 0; q < kMaxSide; ++q) {
                o[q] = r.roff[q] / 16u;
                o[kMaxSide + q] = r.poff[q] / 16u;
            }
            // an irreversible reaction's products: the species with b = 0
            if (!(r.flags & kFlagReversible)) o[kMaxSide] = (uint32_t)ns + 1;
            v.r01 = o[0] | o[1] << 16;
            v.p01 = o[3] | o[4] << 16;
            v.rp2 = o[2] | o[5] << 16;
            const bool kconst = r.flags & kFlagKfConst;
            v.lA = r.lnA;
            v.beta = kconst ? r.A : r.beta;
            v.ER = r.ER;
            const bool fall = r.type == KX_RXN_LINDEMANN || r.type == KX_RXN_TROE ||
                              r.type == KX_RXN_SRI;
            v.meta = (r.flags & kFlagKfConst ? kWideConst : 0u) |
                     (r.type == KX_RXN_PLOG ? kWidePlog : 0u) |
                     (o[2] != dummy || o[5] != dummy ? kWideThird : 0u) |
                     (r.flags & kFlagOrders ? kWideOrders : 0u) |
                     (fall || r.type == KX_RXN_THREEBODY ? kWideThirdBody : 0u) |
                     (fall ? kWideFalloff : 0u) | (r.type == KX_RXN_TROE ? kWideTroe : 0u) |
                     (r.type == KX_RXN_SRI ? kWideSri : 0u) |
                     (r.flags & kFlagChemAct ? kWideChemAct : 0u) |
                     ((r.aux == 0xFFFF ? 0u : (uint32_t)r.aux) << 16);
            nplog += r.type == KX_RXN_PLOG;
            wrx32.push_back(v);
            if (r.type != KX_RXN_PLOG) {
                v.lA = (double)std::log2((long double)d->A[i]);
                v.ER = (double)((long double)d->Ea[i] / kRcal * kLog2e);
            }
            wrx.push_back(v);
        }
        auto l2 = [&](double x) { return (double)((long double)x * kLog2e); };
        waux = aux;
        for (int s = 0; s < nr; ++s) {
            if (rx[s].aux == 0xFFFF) continue;
            DevAux &a = waux[rx[s].aux];
            const int i = perm[s], t = rx[s].type;
            if (t == KX_RXN_LINDEMANN || t == KX_RXN_TROE || t == KX_RXN_SRI) {
                a.lnA0 = (double)std::log2((long double)d->A0[i]);
                a.ER0 = (double)((long double)d->Ea0[i] / kRcal * kLog2e);
                for (int q = 1; q < 4; ++q) a.fp[q] = l2(a.fp[q]);
            }
        }
        wplog = plog;
        for (DevPlog &e : wplog) {
            e.lnA = l2(e.lnA);
            e.ER = l2(e.ER);
        }
        wsp.assign((size_t)16 * ns, 0.0);
        for (int k = 0; k < ns; ++k) {
            for (int r = 0; r < 2; ++r) {
                const double *g = r ? spv[k].g_hi : spv[k].g_lo;
                double *o = &wsp[(size_t)16 * k + 7 * r];
                o[0] = g[0];  // c0 (1 - ln T) = c0 - c0 ln 2 log2 T
                for (int e = 1; e < 6; ++e) o[e] = -l2(g[e]);
                o[6] = -(double)(((long double)g[0] + g[6]) * kLog2e);
            }
            wsp[(size_t)16 * k + 14] = spv[k].t_mid;
            wsp[(size_t)16 * k + 15] = d->qss && d->qss[k] ? 0.0 : spv[k].inv_W;
        }
        wsh[0] = wsh[1] = ws;
        wsh[1].nw = 16;
        wsh[2] = wide_shape_alone(ns, nr);
        const SpeciesRows rows = species_rows(d, perm);
        for (int v = 0; v < 3; ++v) {
            for (wsame[v] = 0; wsame[v] < v; ++wsame[v])  // an equal shape's tables serve both
                if (wsh[wsame[v]].nw == wsh[v].nw && wsh[wsame[v]].chunk == wsh[v].chunk) break;
            if (wsame[v] == v) wide_gather(rows, wsh[v], wmap[v], wstart[v], wgat[v]);
        }
        few_lists(rows, nr, ws.chunk, fptr, fent);
    }
    if (wrx.empty()) wrx.resize(1), wrx32.resize(1);
    if (waux.empty()) waux.resize(1);
    if (wplog.empty()) wplog.resize(1);
    if (wsp.empty()) wsp.resize(16);

    JacTables jt;
    jac_tables(d, perm, rx, aux, eff, jt);

    // ---- species-major gather lists per reaction chunk, where a kernel reads them:
    // rates above kWideMaxSpecies, QSS rates by one wave per point, the Jacobian by one
    // row per thread.  Each species lists the chunk slots of the reactions that
    // produce it (+q, once per unit of net nu) and of those that consume it (-q); both
    // lists are padded to a whole number of eight-entry groups common to all lanes,
    // and a group is eight 32-bit LDS offsets (32 bytes per lane, so lane k reads it
    // with a pair of coalesced 16-byte loads).  The rates of progress of two points
    // sit side by side in LDS, so one offset addresses both.
    std::vector<int32_t> gpos(nchunks), gneg(nchunks), goff(nchunks);
    std::vector<uint32_t> gent;  // 8 per (group, lane)
    size_t ngroups = 0;
    const bool lists = ns > kWideMaxSpecies || (nq > 0 ? qlist.empty() : jt.rows == 0);
    for (int c = 0; c < nchunks && lists; ++c) {
        std::vector<std::vector<uint32_t>> pos(gw), neg(gw);
        for (int s = c * chunk; s < std::min(nr, (c + 1) * chunk); ++s) {
            const int i = perm[s];
            std::vector<std::pair<int, int>> net;  // (species, nu'' - nu')
            auto addnu = [&](int k, int v) {
                for (auto &pr : net)
                    if (pr.first == k) { pr.second += v; return; }
                net.push_back({k, v});
            };
            for (int e = d->reac_ptr[i]; e < d->reac_ptr[i + 1]; ++e)
                addnu(d->reac_sp[e], -d->reac_nu[e]);
            for (int e = d->prod_ptr[i]; e < d->prod_ptr[i + 1]; ++e)
                addnu(d->prod_sp[e], d->prod_nu[e]);
            const uint32_t slot = (uint32_t)(16 * (s - c * chunk));
            for (auto &pr : net)
                for (int u = 0; u < std::abs(pr.second); ++u)
                    (pr.second > 0 ? pos : neg)[pr.first].push_back(slot);
        }
        size_t lp = 0, ln = 0;
        for (int k = 0; k < gw; ++k) {
            lp = std::max(lp, pos[k].size());
            ln = std::max(ln, neg[k].size());
        }
        gpos[c] = (int32_t)((lp + 7) / 8);
        gneg[c] = (int32_t)((ln + 7) / 8);
        goff[c] = (int32_t)ngroups;
        const uint32_t pad = (uint32_t)(16 * chunk);  // the zero slot
        for (int side = 0; side < 2; ++side) {
            const auto &lists = side ? neg : pos;
            const int groups = side ? gneg[c] : gpos[c];
            for (int g = 0; g < groups; ++g)
                for (int k = 0; k < gw; ++k)
                    for (int u = 0; u < 8; ++u) {
                        const size_t e = (size_t)g * 8 + u;
                        gent.push_back(e < lists[k].size() ? lists[k][e] : pad);
                    }
            ngroups += groups;
        }
    }
    if (gent.empty()) gent.resize(8, 0);

    // ---- transport tables
    const int nkb = (ns + kKB - 1) / kKB;
    std::vector<double> visc((size_t)ns * order), cond((size_t)ns * order);
    std::memcpy(visc.data(), d->visc_fit, visc.size() * sizeof(double));
    std::memcpy(cond.data(), d->cond_fit, cond.size() * sizeof(double));
    // the matrix-core kernel reads fragments of the pair tables (below), the others
    // the pair tables themselves
    const bool mfma = d->diff_fit_kind == 1 && ns >= kMfmaMinSpecies;
    std::vector<double> wilke(mfma ? 1 : (size_t)nkb * ns * kKB, 0.0), wq(ns);
    for (int k = 0; k < ns; ++k) wq[k] = std::pow(W[k], 0.25);
    std::vector<double> dfit(mfma ? 1 : (size_t)nkb * ns * kKB * order, 0.0);
    std::vector<double> ddiag((size_t)ns * order);
    for (int kb = 0; kb < nkb && !mfma; ++kb)
        for (int j = 0; j < ns; ++j)
            for (int kk = 0; kk < kKB; ++kk) {
                const int k = kb * kKB + kk;
                if (k >= ns) {
                    // padding rows of the last block: a fit identically 1 keeps
                    // the branch-free pair loop finite (their sums are unused)
                    dfit[(((size_t)kb * ns + j) * kKB + kk) * order] = 1.0;
                    continue;
                }
                // phi_kj = c1_kj (1 + sigma_k rho_j)^2 with c2_kj = (W_j/W_k)^(1/4)
                // = wq_j / wq_k folded into the per-species factors
                wilke[((size_t)kb * ns + j) * kKB + kk] = 1.0 / std::sqrt(8.0 * (1.0 + W[k] / W[j]));
                std::memcpy(&dfit[(((size_t)kb * ns + j) * kKB + kk) * order],
                            d->diff_fit + ((size_t)k * ns + j) * order, order * sizeof(double));
            }
    for (int k = 0; k < ns; ++k)
        std::memcpy(&ddiag[(size_t)k * order], d->diff_fit + ((size_t)k * ns + k) * order,
                    order * sizeof(double));
    auto to32 = [](const std::vector<double> &v) {
        return std::vector<float>(v.begin(), v.end());
    };

    // ---- MFMA fragments of the quadratic sums (fits of 1/D_kj only)
    const int mblk = (ns + 15) / 16, kstep = (ns + 3) / 4;
    std::vector<double> gfrag, c1frag;
    if (mfma) {
        gfrag.assign((size_t)order * mblk * kstep * 64, 0.0);
        c1frag.assign((size_t)mblk * kstep * 64, 0.0);
        for (int mb = 0; mb < mblk; ++mb)
            for (int ks = 0; ks < kstep; ++ks)
                for (int l = 0; l < 64; ++l) {
                    const int k = 16 * mb + l % 16, j = 4 * ks + l / 16;
                    if (k >= ns || j >= ns) continue;
                    c1frag[((size_t)mb * kstep + ks) * 64 + l] =
                        1.0 / std::sqrt(8.0 * (1.0 + W[k] / W[j]));
                    if (j == k) continue;
                    for (int o = 0; o < order; ++o)
                        gfrag[(((size_t)o * mblk + mb) * kstep + ks) * 64 + l] =
                            d->diff_fit[((size_t)k * ns + j) * order + o];
                }
    } else {
        gfrag.resize(1);
        c1frag.resize(1);
    }

    Blob b;
    const size_t o_rxn = add_vec(b, rx), o_aux = add_vec(b, aux), o_eff = add_vec(b, eff);
    const size_t o_plog = add_vec(b, plog);
    const size_t o_sp = add_vec(b, spv), o_gpos = add_vec(b, gpos), o_gneg = add_vec(b, gneg);
    const size_t o_gsoa = add_vec(b, gsoa);
    const size_t o_goff = add_vec(b, goff);
    const size_t o_gent = add_vec(b, gent);
    const size_t o_wrx = add_vec(b, wrx), o_wrx32 = add_vec(b, wrx32), o_waux = add_vec(b, waux);
    const size_t o_wplog = add_vec(b, wplog), o_wsp = add_vec(b, wsp);
    const size_t o_qsp = add_vec(b, qsp), o_qlist = add_vec(b, qlist);
    const size_t o_qstart = add_vec(b, qstart), o_qgather = add_vec(b, qgather);
    const size_t o_jval = add_vec(b, jt.val), o_jptr = add_vec(b, jt.ptr);
    const size_t o_jlist = add_vec(b, jt.list), o_jent = add_vec(b, jt.ent);
    const size_t o_jtgt = add_vec(b, jt.tgt);
    size_t o_wmap[3], o_wstart[3], o_wgat[3];
    for (int v = 0; v < 3; ++v) {
        o_wmap[v] = add_vec(b, wmap[v]);
        o_wstart[v] = add_vec(b, wstart[v]);
        o_wgat[v] = add_vec(b, wgat[v]);
        o_wmap[v] = o_wmap[wsame[v]], o_wstart[v] = o_wstart[wsame[v]], o_wgat[v] = o_wgat[wsame[v]];
    }
    const size_t o_W = add_vec(b, W), o_visc = add_vec(b, visc), o_cond = add_vec(b, cond);
    const size_t o_wil = add_vec(b, wilke), o_df = add_vec(b, dfit), o_dd = add_vec(b, ddiag);
    const size_t o_wq = add_vec(b, wq), o_wq32 = add_vec(b, to32(wq));
    const size_t o_visc32 = add_vec(b, to32(visc)), o_cond32 = add_vec(b, to32(cond));
    const size_t o_wil32 = add_vec(b, to32(wilke)), o_df32 = add_vec(b, to32(dfit));
    const size_t o_dd32 = add_vec(b, to32(ddiag));
    const size_t o_gf = add_vec(b, gfrag), o_c1f = add_vec(b, c1frag);
    const size_t o_gf32 = add_vec(b, to32(gfrag)), o_c1f32 = add_vec(b, to32(c1frag));
    const size_t o_qidx = add_vec(b, qidx), o_qrx = add_vec(b, qrx);
    const size_t o_qptr = add_vec(b, qrow_ptr), o_qent = add_vec(b, qrow_ent);
    const size_t o_fptr = add_vec(b, fptr), o_fent = add_vec(b, fent);
    const size_t o_qfptr = add_vec(b, qfptr), o_qfent = add_vec(b, qfent);
    const size_t o_qinfo = add_vec(b, qinfo);

    void *blob = nullptr;
    if (!host_only) {
        int prev = 0;
        hipError_t e = hipGetDevice(&prev);
        if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
        e = hipSetDevice(device);
        if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
        e = hipMalloc(&blob, b.host.size());
        if (e != hipSuccess) {
            hipSetDevice(prev);
            return fail(KX_ENOMEM, "kx_mech_create: hipMalloc of " +
                                       std::to_string(b.host.size()) + " bytes failed");
        }
        e = hipMemcpy(blob, b.host.data(), b.host.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            hipFree(blob);
            hipSetDevice(prev);
            return hip_fail(e, "hipMemcpy (mechanism upload)");
        }
        hipSetDevice(prev);
    }

    kx_mech *m = new kx_mech;
    m->device = host_only ? -1 : device;
    m->blob = blob;
    m->bytes = (int64_t)b.host.size();
    m->n_species = ns;
    m->uid = next_uid.fetch_add(1) + 1;
    m->n_reactions = nr;
    MechDev &v = m->dev;
    // device addresses of the tables (null for a host-only handle)
    auto at = [&](size_t off) {
        return blob ? (const void *)((const uint8_t *)blob + off) : (const void *)nullptr;
    };
    v.ns = ns;
    v.nr = nr;
    v.chunk = chunk;
    v.nchunks = nchunks;
    v.gpass = gpass;
    v.fit_order = order;
    v.diff_kind = d->diff_fit_kind;
    v.fit_L0 = d->fit_L0;
    v.inv_fit_h = 1.0 / d->fit_h;
    v.rxn = (const DevRxn *)at(o_rxn);
    v.aux = (const DevAux *)at(o_aux);
    v.eff = (const DevEff *)at(o_eff);
    v.plog = (const DevPlog *)at(o_plog);
    v.sp = (const DevSpecies *)at(o_sp);
    v.gsoa = (const double *)at(o_gsoa);
    v.gpos = (const int32_t *)at(o_gpos);
    v.gneg = (const int32_t *)at(o_gneg);
    v.goff = (const int32_t *)at(o_goff);
    v.gent = (const uint4 *)at(o_gent);
    v.jnv = jt.nv;
    v.jrows = jt.rows;
    v.jnblk = jt.nblk;
    v.jpts = jt.pts;
    v.jval = (const uint32_t *)at(o_jval);
    v.jptr = (const int32_t *)at(o_jptr);
    v.jlist = (const uint2 *)at(o_jlist);
    v.jent = (const uint2 *)at(o_jent);
    v.jtgt = (const uint16_t *)at(o_jtgt);
    v.wnw = ws.nw;
    v.nplog = nplog;
    v.wrx = (const DevWide *)at(o_wrx);
    v.wrx32 = (const DevWide *)at(o_wrx32);
    v.waux = (const DevAux *)at(o_waux);
    v.wplog = (const DevPlog *)at(o_wplog);
    v.wsp = (const double *)at(o_wsp);
    for (int q = 0; q < 3; ++q) {
        v.wmaps[q].chunk = wsh[q].chunk;
        v.wmaps[q].nchunks = wsh[q].nchunks;
        v.wmaps[q].species = (const int32_t *)at(o_wmap[q]);
        v.wmaps[q].start = (const uint32_t *)at(o_wstart[q]);
        v.wmaps[q].gather = (const uint4 *)at(o_wgat[q]);
    }
    v.W = (const double *)at(o_W);
    v.visc = (const double *)at(o_visc);
    v.cond = (const double *)at(o_cond);
    v.wilke = (const double *)at(o_wil);
    v.wq = (const double *)at(o_wq);
    v.wq32 = (const float *)at(o_wq32);
    v.dfit = (const double *)at(o_df);
    v.ddiag = (const double *)at(o_dd);
    v.visc32 = (const float *)at(o_visc32);
    v.cond32 = (const float *)at(o_cond32);
    v.wilke32 = (const float *)at(o_wil32);
    v.dfit32 = (const float *)at(o_df32);
    v.ddiag32 = (const float *)at(o_dd32);
    v.mblk = mblk;
    v.kstep = kstep;
    v.gfrag = mfma ? (const double *)at(o_gf) : nullptr;
    v.c1frag = mfma ? (const double *)at(o_c1f) : nullptr;
    v.gfrag32 = mfma ? (const float *)at(o_gf32) : nullptr;
    v.c1frag32 = mfma ? (const float *)at(o_c1f32) : nullptr;
    v.nq = nq;
    v.nqent = nq > 0 ? qrow_ptr[nq] : 0;
    v.qidx = (const int32_t *)at(o_qidx);
    v.wnqr = (int32_t)qlist.size();
    v.qchunk = qchunk;
    v.qsp = (const int32_t *)at(o_qsp);
    v.qlist = (const int32_t *)at(o_qlist);
    v.qstart = (const uint32_t *)at(o_qstart);
    v.qgather = (const uint4 *)at(o_qgather);
    v.qrx = (const int2 *)at(o_qrx);
    v.qrow_ptr = (const int32_t *)at(o_qptr);
    v.qrow_ent = (const int4 *)at(o_qent);
    m->few.ptr = (const int32_t *)at(o_fptr);
    m->few.ent = (const uint4 *)at(o_fent);
    m->few.qptr = (const int32_t *)at(o_qfptr);
    m->few.qent = (const uint4 *)at(o_qfent);
    m->few.qinfo = (const int32_t *)at(o_qinfo);
    *out = m;
    return ok();
}

bool rebase_tables(const kx_mech *m, const void *base, MechDev *out)
{
    MechDev v = m->dev;
    const char *old = static_cast<const char *>(m->blob);
    const char *nb = static_cast<const char *>(base);
#define KX_REBASE(f) \
    v.f = m->dev.f ? reinterpret_cast<decltype(v.f)>(nb + (reinterpret_cast<const char *>(m->dev.f) - old)) \
                   : nullptr
    KX_REBASE(rxn); KX_REBASE(aux); KX_REBASE(eff); KX_REBASE(plog); KX_REBASE(sp);
    KX_REBASE(gsoa);
    KX_REBASE(gpos); KX_REBASE(gneg); KX_REBASE(goff); KX_REBASE(gent);
    KX_REBASE(wrx); KX_REBASE(wrx32); KX_REBASE(waux); KX_REBASE(wplog); KX_REBASE(wsp);
    KX_REBASE(jval); KX_REBASE(jptr); KX_REBASE(jlist); KX_REBASE(jent); KX_REBASE(jtgt);
    for (int q = 0; q < 3; ++q) {
        KX_REBASE(wmaps[q].species); KX_REBASE(wmaps[q].start); KX_REBASE(wmaps[q].gather);
    }
    KX_REBASE(W); KX_REBASE(visc); KX_REBASE(cond); KX_REBASE(wq); KX_REBASE(wilke);
    KX_REBASE(dfit); KX_REBASE(ddiag);
    KX_REBASE(visc32); KX_REBASE(cond32); KX_REBASE(wq32); KX_REBASE(wilke32);
    KX_REBASE(dfit32); KX_REBASE(ddiag32);
    KX_REBASE(gfrag); KX_REBASE(c1frag); KX_REBASE(gfrag32); KX_REBASE(c1frag32);
    KX_REBASE(qsp); KX_REBASE(qlist); KX_REBASE(qstart); KX_REBASE(qgather);
    KX_REBASE(qidx); KX_REBASE(qrow_ptr); KX_REBASE(qrow_ent); KX_REBASE(qrx);
#undef KX_REBASE
    // every table pointer must have moved: no 8-byte word of the result may
    // still address the original tables
    uintptr_t words[sizeof(MechDev) / sizeof(uintptr_t)];
    std::memcpy(words, &v, sizeof words);
    const uintptr_t lo = reinterpret_cast<uintptr_t>(old), hi = lo + (uintptr_t)m->bytes;
    for (uintptr_t w : words)
        if (w >= lo && w < hi) return false;
    *out = v;
    return true;
}

}  // namespace kx
