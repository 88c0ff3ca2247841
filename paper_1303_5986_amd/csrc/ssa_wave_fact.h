// ssa_wave_fact.h -- the wave-per-walker event loop with every table it
// reads in LDS: reaction descriptors, the factored dependency graph (an
// 8-byte change header per reaction, a start/count word per species and the
// species -> reaction incidence lists, see fact_code in we_common.h) and the
// walker's counts.  No global memory is touched between the first and the
// last event of an interval.
//
// Per event (one 64-wide wave, Sec. II.A's direct method):
//  1. a0 and the chunk holding u2*a0: inclusive scan of the 64 chunk sums
//     (lane c holds the sum of reactions 64c .. 64c+63) and a ballot;
//  2. the reaction inside the chunk: the chunk's 64 propensities from the
//     counts, a second scan and a ballot; each lane also loads its
//     reaction's change header, so the chosen one is two readlanes away;
//     lanes 0-3 then read the changed species' incidence words and counts;
//  3. the dependents: the incidence lists of the changed species, laid end
//     to end over the lanes (one or two rounds of 64); a reaction listed
//     under two changed species counts under the first only.  The firing is
//     one LDS store per changed species (the wave's LDS accesses complete in
//     order).  Networks of reactions of at most two molecules: a lane's entry
//     names the reaction and its other reactant, so its rate constant and that
//     count are one LDS read away, and h' - h is a few small-integer
//     operations (one run of the 354/3680 network 234 -> 211 us per launch
//     against descriptor, counts, firing and counts again: two LDS round trips
//     fewer in the chain of an event, which is what bounds the launch).  Others: each lane reads its reaction's descriptor and
//     counts before the firing and its counts again after it;
//  4. each dependent's change of propensity is added to its chunk's sum,
//     held per wave in LDS, by an LDS atomic (ds_add_f64); the chunk lanes
//     then reload their sums.  The LDS unit applies the lanes of one atomic
//     instruction that hit the same address in a fixed order, so a run
//     still repeats bit for bit.
// A reaction whose dependents exceed two rounds rebuilds every chunk sum.
// Every 16 events the wave's issue priority follows its walker's expected
// remaining events (chain_priority), so the longest chains issue first.
#pragma once
#include "ssa_wave_body.h"

#define FACT_DEP_ROUNDS 2

namespace {

template <class D>
union DescBits {
    D d;
    uint4 u;
};

template <class D>
__device__ __forceinline__ D desc_of(const uint4 &u) {
    DescBits<D> b;
    b.u = u;
    return b.d;
}

}  // namespace

struct FactTables {
    const uint4 *d;        // LDS [R] descriptors
    const uint2 *h;        // LDS [R] change headers
    const uint32_t *tab;   // LDS [S] incidence start | count << 16
    const uint16_t *inc;   // LDS [n_inc] incidence lists (general form)
    const uint32_t *inc2;  // LDS [n_inc] incidence lists as fact_pair_entry words (pair form)
};

// One walker through one interval on the calling wave; lchunk (64 doubles,
// the chunk sums) and lx (S + 1 ints: the counts, and the 1 an absent reactant
// reads) are this wave's LDS slices.  D: the descriptors' form.
template <class D>
__device__ inline void wave_walker_fact(const SimArgs &a, const FactTables &tab, int32_t *__restrict__ xs,
                                        int32_t run, int32_t k, uint32_t iter, double *lchunk, int32_t *lx) {
    constexpr bool PAIR = std::is_same<D, RxnDesc2>::value;
    const int lane = threadIdx.x & 63;
    const int32_t S = a.S, R = a.R;
    int32_t *xw = xs + ((size_t)run * a.cap + k) * S;
    for (int s = lane; s < S; s += 64) lx[s] = xw[s];
    if (PAIR && lane == 0) lx[S] = 1;
    __builtin_amdgcn_wave_barrier();

    // chunk sums from scratch
    auto rebuild = [&]() {
        return chunk_sums(R, lane, [&](int32_t r) {
            const D d = desc_of<D>(tab.d[r]);
            return propensity_from(d, (uint32_t)lx[d.s1], (uint32_t)lx[d.s2]);
        });
    };
    double csum = rebuild();
    lchunk[lane] = csum;

    const uint64_t seed = a.seeds[run];
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const double tau = a.tau;
    double t = 0.0;
    uint32_t e = 0, fired = 0;
    bool bad = false;
    double rexp = 0.0, ru2 = 0.0;   // random numbers of 64 events, one per lane

    for (;;) {
        const double P = scan_incl(csum);
        const double a0 = lane_value(P, 63);
        if (!(a0 > 0.0)) break;
        if ((e & 63u) == 0u) {
            const U4 rnd = philox4x32_10(e + (uint32_t)lane, (uint32_t)k, iter, 0u, k0, k1);
            rexp = -log(1.0 - uniform53(rnd.x, rnd.y));
            ru2 = uniform53(rnd.z, rnd.w);
        }
        const double ex = lane_value(rexp, (int)(e & 63u));
        const double u2 = lane_value(ru2, (int)(e & 63u));
        e += 1;
        const double dt = ex * recip(a0);
        if (!(t + dt <= tau)) break;   // recip(a0) below 2^-1024: not a number
        t = t + dt;
        if ((e & 15u) == 1u) chain_priority((tau - t) * a0);
        const double target = u2 * a0;

        // chunk holding the target
        const unsigned long long m1 = __ballot(P > target);
        int cs = m1 ? (__ffsll((long long)m1) - 1) : last_set(__ballot(csum > 0.0));
        if (cs < 0) cs = 0;
        cs = __builtin_amdgcn_readfirstlane(cs);
        const double base = lane_value(P - csum, cs);
        const double target2 = target - base;
        // reaction inside the chunk, with every lane's descriptor and header
        const int rsel = cs * 64 + lane;
        double v = 0.0;
        uint4 dsel{0u, 0u, 0u, 0u};
        uint2 hsel{0u, 0u};
        if (rsel < R) {
            dsel = tab.d[rsel];
            hsel = tab.h[rsel];
            const D d = desc_of<D>(dsel);
            v = propensity_from(d, (uint32_t)lx[d.s1], (uint32_t)lx[d.s2]);
        }
        const double Q = scan_incl(v);
        const unsigned long long m2 = __ballot(Q > target2);
        const int ls = m2 ? (__ffsll((long long)m2) - 1) : last_set(__ballot(v > 0.0));
        if (ls < 0) {              // chunk sum drifted above an all-zero chunk
            if (lane == 0) atomicOr(a.err, WE_DERR_SELECT);
            break;
        }
        // the fired reaction's changes (wave-uniform)
        const int32_t nchg = (int32_t)((__builtin_amdgcn_readlane((int)dsel.w, ls) >> 16) & 0xFF);
        const uint32_t hlo = (uint32_t)__builtin_amdgcn_readlane((int)hsel.x, ls);
        const uint32_t hhi = (uint32_t)__builtin_amdgcn_readlane((int)hsel.y, ls);
        // lanes 0..nchg-1: the changed species' old counts and incidence words
        const uint32_t code = (uint32_t)((((uint64_t)hhi << 32) | hlo) >> (16 * (lane & 3)));
        const int32_t spl = fact_species(code), dll = fact_delta(code);
        int32_t xold = 0;
        uint32_t iw = 0u;
        if (lane < nchg) {
            xold = lx[spl];
            iw = tab.tab[spl];
        }
        // wave-uniform, in scalars: the four changes (absent ones: species -1) and
        // the four incidence lists laid end to end, list k from lane off_k on, its
        // entries at at_k + lane
        const uint32_t iw0 = (uint32_t)__builtin_amdgcn_readlane((int)iw, 0);
        const uint32_t iw1 = (uint32_t)__builtin_amdgcn_readlane((int)iw, 1);
        const uint32_t iw2 = (uint32_t)__builtin_amdgcn_readlane((int)iw, 2);
        const uint32_t iw3 = (uint32_t)__builtin_amdgcn_readlane((int)iw, 3);
        const int32_t sp0 = nchg > 0 ? fact_species(hlo) : -1, sp1 = nchg > 1 ? fact_species(hlo >> 16) : -1;
        const int32_t sp2 = nchg > 2 ? fact_species(hhi) : -1, sp3 = nchg > 3 ? fact_species(hhi >> 16) : -1;
        const int32_t dl0 = fact_delta(hlo), dl1 = fact_delta(hlo >> 16), dl2 = fact_delta(hhi), dl3 = fact_delta(hhi >> 16);
        const int32_t off1 = (int32_t)(iw0 >> 16), off2 = off1 + (int32_t)(iw1 >> 16);
        const int32_t off3 = off2 + (int32_t)(iw2 >> 16), nd = off3 + (int32_t)(iw3 >> 16);
        const int32_t at0 = (int32_t)(iw0 & 0xFFFFu), at1 = (int32_t)(iw1 & 0xFFFFu) - off1;
        const int32_t at2 = (int32_t)(iw2 & 0xFFFFu) - off2, at3 = (int32_t)(iw3 & 0xFFFFu) - off3;
        // v_k of the list k that dependent idx comes from.  Scalars: with arrays
        // the compiler kept them in scratch and selected the address.
        auto pick = [&](int32_t idx, int32_t v0, int32_t v1, int32_t v2, int32_t v3) {
            int32_t r = idx >= off1 ? v1 : v0;
            r = idx >= off2 ? v2 : r;
            return idx >= off3 ? v3 : r;
        };

        const bool fits = nd <= 64 * FACT_DEP_ROUNDS;
        uint32_t eq[FACT_DEP_ROUNDS];           // pair form: the dependents' entries
        double cq[FACT_DEP_ROUNDS];             //   and rate constants
        int32_t xd[FACT_DEP_ROUNDS];            //   and their list's species' old count | change + 8 << 17
        uint4 dq[FACT_DEP_ROUNDS];              // general form: descriptors
        int32_t x1q[FACT_DEP_ROUNDS], x2q[FACT_DEP_ROUNDS], chk[FACT_DEP_ROUNDS];   // counts before the firing, chunk
        const int32_t xd0 = __builtin_amdgcn_readlane(xold, 0) | ((dl0 + 8) << 17);
        const int32_t xd1 = __builtin_amdgcn_readlane(xold, 1) | ((dl1 + 8) << 17);
        const int32_t xd2 = __builtin_amdgcn_readlane(xold, 2) | ((dl2 + 8) << 17);
        const int32_t xd3 = __builtin_amdgcn_readlane(xold, 3) | ((dl3 + 8) << 17);
#pragma unroll
        for (int q = 0; q < FACT_DEP_ROUNDS; ++q) {
            chk[q] = -1;
            const int32_t idx = q * 64 + lane;
            if (q > 0 && nd <= 64 * q) continue;   // uniform: no lane has a dependent here
            if (fits && idx < nd) {
                if constexpr (PAIR) {
                    eq[q] = tab.inc2[pick(idx, at0, at1, at2, at3) + idx];
                    xd[q] = pick(idx, xd0, xd1, xd2, xd3);
                    const int32_t r = (int32_t)(eq[q] & 0xFFFu);
                    chk[q] = r >> 6;
                    cq[q] = *reinterpret_cast<const double *>(&tab.d[r]);
                } else {
                    const int32_t r = tab.inc[pick(idx, at0, at1, at2, at3) + idx];
                    dq[q] = tab.d[r];
                    const D d = desc_of<D>(dq[q]);
                    x1q[q] = lx[d.s1];
                    x2q[q] = lx[d.s2];
                    chk[q] = r >> 6;
                }
            }
        }
        // fire j (the dependents' old counts were read above)
        bool lbad = false;
        if (lane < nchg) {
            const int32_t nv = xold + dll;
            lx[spl] = nv;
            lbad = (nv < 0) || (nv > WE_COUNT_MAX_DEV);
        }
        fired += 1;
        if (__ballot(lbad)) { bad = true; break; }

        __builtin_amdgcn_wave_barrier();
        if (!fits) {
            csum = rebuild();
            lchunk[lane] = csum;
            continue;
        }
#pragma unroll
        for (int q = 0; q < FACT_DEP_ROUNDS; ++q) {
            if (q * 64 >= nd) break;
            if (chk[q] >= 0) {
                const int32_t idx = q * 64 + lane;
                const bool b1 = idx >= off1, b2 = idx >= off2, b3 = idx >= off3;
                if constexpr (PAIR) {
                    // h' - h with the list's species going from xs to xs + dk and
                    // the other reactant by dother to xo:
                    // (xs + dk)(xo - hom) - xs (xo - dother - hom), small integers
                    const int32_t other = (int32_t)((eq[q] >> 12) & 0x3FFu), hom = (int32_t)(eq[q] >> 22);
                    const int32_t xo = lx[other] - hom;
                    const bool m0 = other == sp0, m1 = other == sp1, m2 = other == sp2, m3 = other == sp3;
                    int32_t dother = m0 ? dl0 : 0;
                    dother = m1 ? dl1 : dother;
                    dother = m2 ? dl2 : dother;
                    dother = m3 ? dl3 : dother;
                    // listed under an earlier changed species too: counted there
                    const bool dup = (b1 & m0) | (b2 & m1) | (b3 & m2);
                    const int32_t dh = __mul24((xd[q] >> 17) - 8, xo) + __mul24(xd[q] & 0x1FFFF, dother);
                    if (!dup) lds_add_f64(&lchunk[chk[q]], cq[q] * (double)dh);
                } else {
                    const D d = desc_of<D>(dq[q]);
                    // listed under an earlier changed species too: counted there
                    // (its other reactant is one of sp0 .. sp[k-1])
                    const int32_t spk = pick(idx, sp0, sp1, sp2, sp3);
                    const int32_t other = d.s1 == spk ? (int32_t)d.s2 : (int32_t)d.s1;
                    const bool dup = d.nu2 > 0 && ((b1 && other == sp0) || (b2 && other == sp1) ||
                                                   (b3 && other == sp2));
                    if (!dup) {
                        const double before = propensity_from(d, (uint32_t)x1q[q], (uint32_t)x2q[q]);
                        const double after = propensity_from(d, (uint32_t)lx[d.s1], (uint32_t)lx[d.s2]);
                        lds_add_f64(&lchunk[chk[q]], after - before);
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        csum = lchunk[lane];
    }
    if (bad && lane == 0) atomicOr(a.err, WE_DERR_OVERFLOW);
    __builtin_amdgcn_wave_barrier();
    for (int s = lane; s < S; s += 64) xw[s] = lx[s];
    if (lane == 0) a.ev_walker[(size_t)run * a.cap + k] = fired;
}
