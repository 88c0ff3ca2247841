// ssa_group_body.h -- Gillespie direct-method SSA with L lanes per walker,
// 64 / L walkers per wave (gfx950); shared by ssa_group.hip and batch.hip.
//
// The middle ground between the lane kernels (one lane per walker, tables in
// registers, up to 64 reactions) and the wave kernels (one wave per walker):
// a group of L consecutive lanes (L = 2 ... 32) carries one walker, and lane
// g of the group owns the block of reactions [g B, (g + 1) B), B = ceil(R/L).
// Per event (Sec. II.A):
//   1. each lane sums its block's propensities, recomputed from the walker's
//      counts in LDS (descriptors and changes from the network tables: an
//      LDS copy in ssa_group_kernel when they fit, else through the cache);
//   2. an inclusive scan over the group's L partial sums (log2 L DPP
//      steps) gives a0 and, with a ballot, the lane whose block holds u2 a0;
//      the random numbers of L events are drawn at once, one event per lane
//      of the group, and read by the event that uses them;
//   3. that lane walks its block again to find j;
//   4. the group applies j's changes to the counts, one change per lane.
// The blocks follow the reactions' own order, so j is the reaction the
// sequential direct method picks; u1, u2 come from Philox4x32-10 at (event,
// slot, iteration, 0) with the run's seed as key, as in the oracle, and
// dt = -log(1 - u1) / a0 with the overshoot past tau discarded.  Only the
// summation order differs from the oracle's (partial sums, then a scan), so
// a0 and the running sums may differ in the last bits: an event changes only
// when u2 a0 or t + dt falls within a few ulps of a boundary.
//
// The groups of a wave run their walkers' event loops in lockstep: the loop
// ends when every group's walker has reached tau; a group that is done
// idles.  All cross-lane steps are executed by the whole wave.
#pragma once

#include "queue_first.h"
#include "we_common.h"

#include <algorithm>

// Ints of a group's slice of counts.
__host__ __device__ inline int32_t group_slice(int32_t S) { return S + 1; }

// Largest group walker table: counts of 64 / L walkers per wave in LDS.
#define GROUP_LDS_INTS_PER_WAVE 4096

__host__ __device__ inline bool group_lanes_valid(int32_t lanes) {
    return lanes == 2 || lanes == 4 || lanes == 8 || lanes == 16 || lanes == 32;
}

// Whether L lanes per walker fit: the counts of 64 / L walkers per wave,
// GROUP_LDS_INTS_PER_WAVE ints, and 16-bit species ids.
__host__ __device__ inline bool group_kernel_fits(int32_t S, int32_t R, int32_t lanes) {
    return group_lanes_valid(lanes) && R >= 1 && R <= 65535 && S >= 1 && (64 / lanes) * S <= GROUP_LDS_INTS_PER_WAVE;
}

union GroupF64 {
    double d;
    int32_t w[2];
};

// Row-shift DPP move of a double (source outside the 16-lane row: 0).
template <int CTRL, int ROW_MASK, bool BOUND>
__device__ __forceinline__ double group_dpp(double v) {
    GroupF64 in, out;
    in.d = v;
    out.w[0] = __builtin_amdgcn_update_dpp(0, in.w[0], CTRL, ROW_MASK, 0xF, BOUND);
    out.w[1] = __builtin_amdgcn_update_dpp(0, in.w[1], CTRL, ROW_MASK, 0xF, BOUND);
    return out.d;
}

// Inclusive scan within groups of L lanes by DPP row shifts (groups of up
// to 16 lie inside a row); a group of 32 adds the first row's total to its
// second row by a row broadcast.  A step adds its source only from the same
// group, so the sums follow a fixed order.
template <int L>
__device__ __forceinline__ double group_scan_incl(double v) {
    const int gl = (int)threadIdx.x & (L - 1);
    double u;
    if (L > 1) { u = group_dpp<0x111, 0xF, true>(v); if (gl >= 1) v += u; }    // row_shr:1
    if (L > 2) { u = group_dpp<0x112, 0xF, true>(v); if (gl >= 2) v += u; }    // row_shr:2
    if (L > 4) { u = group_dpp<0x114, 0xF, true>(v); if (gl >= 4) v += u; }    // row_shr:4
    if (L > 8) { u = group_dpp<0x118, 0xF, true>(v); if (gl >= 8) v += u; }    // row_shr:8
    if (L > 16) { u = group_dpp<0x142, 0xA, false>(v); if (gl >= 16) v += u; } // row_bcast:15, rows 1, 3
    return v;
}

// The value of a group's last lane on all its lanes: row broadcasts (two banks of
// four lanes each for groups of 8), a quad permutation, or lane reads.
template <int CTRL, int BANKS>
__device__ __forceinline__ double group_bcast(double old, double v) {
    GroupF64 in, was, out;
    in.d = v;
    was.d = old;
    out.w[0] = __builtin_amdgcn_update_dpp(was.w[0], in.w[0], CTRL, 0xF, BANKS, false);
    out.w[1] = __builtin_amdgcn_update_dpp(was.w[1], in.w[1], CTRL, 0xF, BANKS, false);
    return out.d;
}
template <int L>
__device__ __forceinline__ double group_last(double v) {
    if constexpr (L == 2) return group_bcast<0xF5, 0xF>(v, v);                              // quad_perm [1,1,3,3]
    else if constexpr (L == 4) return group_bcast<0xFF, 0xF>(v, v);                         // quad_perm [3,3,3,3]
    else if constexpr (L == 8) return group_bcast<0x15F, 0xC>(group_bcast<0x157, 0x3>(v, v), v);   // row_newbcast:7, 15
    else if constexpr (L == 16) return group_bcast<0x15F, 0xF>(v, v);                       // row_newbcast:15
    else {
        GroupF64 in, lo, hi;
        in.d = v;
        for (int i = 0; i < 2; ++i) {
            lo.w[i] = __builtin_amdgcn_readlane(in.w[i], 31);
            hi.w[i] = __builtin_amdgcn_readlane(in.w[i], 63);
        }
        return (threadIdx.x & 32) ? hi.d : lo.d;
    }
}

// The network tables a group walker reads: a.desc, a.chg_ptr and a.chg, or
// a block's LDS copy of them.
template <class D>
struct GroupTables {
    const D *desc;
    const int32_t *chg_ptr;
    const int32_t *chg;
};

// LDS copy of the network tables (descriptors, change offsets, changes),
// 16-byte aligned.
__host__ __device__ inline size_t group_tables_bytes(int32_t R, int32_t n_chg) {
    return (16 * (size_t)R + 4 * ((size_t)R + 1 + (size_t)n_chg) + 15) & ~(size_t)15;
}

// The block's LDS copy of the tables at `lds`; copies them there first when
// `stage` is set (every thread of the block calls it; uniform).
template <class D>
__device__ __forceinline__ GroupTables<D> group_stage(const SimArgs &a, const D *gdesc, unsigned char *lds, bool stage) {
    const int32_t R = a.R;
    uint4 *ld = reinterpret_cast<uint4 *>(lds);
    int32_t *lcp = reinterpret_cast<int32_t *>(lds + 16 * (size_t)R);
    int32_t *lcg = lcp + R + 1;
    if (stage) {
        const uint4 *gd = reinterpret_cast<const uint4 *>(gdesc);
        for (int32_t i = threadIdx.x; i < R; i += blockDim.x) ld[i] = gd[i];
        for (int32_t i = threadIdx.x; i <= R; i += blockDim.x) lcp[i] = a.chg_ptr[i];
        for (int32_t i = threadIdx.x; i < a.n_chg; i += blockDim.x) lcg[i] = a.chg[i];
        __syncthreads();
    }
    return GroupTables<D>{reinterpret_cast<const D *>(ld), lcp, lcg};
}

// The walkers in slots k of run `run` for the groups with live set (k may
// differ per group); lx is this group's slice of S + 1 ints in LDS (the counts,
// and the 1 that an absent reactant of a RxnDesc2 reads).  Every lane of the
// wave must call it.  D: the descriptors' form; a lane evaluates its whole block
// every event, so the general form's two binomials per reaction were most of
// an event's instructions.  The event is free of branches but for the draw and
// the change, so that the waiting time's division runs beside the selection, and
// a0 comes by row broadcasts, not through LDS.  What bounds it is an event's chain
// through LDS and the scan.  Toggle, 16 runs on 8 walkers per wave: 46.2 us per
// launch with binomials, 42.4 with branches, 39.3, and 37.9 with no idle slots.  BR > 0 (blocks of at most BR reactions): each
// lane keeps its block's descriptors in registers for the whole interval and
// its block's propensities from step 1 for step 3, instead of reading the
// descriptors again every event.
template <int L, int BR, class D>
__device__ inline void group_walker(const SimArgs &a, const GroupTables<D> &tb, int32_t *__restrict__ xs, int32_t run,
                                    int32_t k, bool live, uint32_t iter, int32_t *lx) {
    const int lane = threadIdx.x & 63;
    const int gl = lane & (L - 1);
    const int gbase = lane - gl;
    const uint64_t gmask = (L == 64) ? ~0ull : (((1ull << L) - 1ull) << gbase);
    const int32_t S = a.S, R = a.R;
    const int32_t B = (R + L - 1) / L;
    const int32_t r_lo = std::min(R, gl * B), r_hi = std::min(R, r_lo + B);
    int32_t *xw = live ? xs + ((size_t)run * a.cap + k) * S : nullptr;
    if (live)
        for (int32_t s = gl; s < S; s += L) lx[s] = xw[s];
    if (std::is_same<D, RxnDesc2>::value && gl == 0) lx[S] = 1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    uint32_t k0 = 0, k1 = 0;
    if (live) {
        const uint64_t seed = a.seeds[run];
        k0 = (uint32_t)seed;
        k1 = (uint32_t)(seed >> 32);
    }
    const double tau = a.tau;
    double t = 0.0;
    uint32_t e = 0, fired = 0;
    bool go = live, bad = false, nosel = false;
    // random numbers of L events at a time: lane gl of a group holds
    // -log(1 - u1) and u2 of the group's event (e & ~(L - 1)) + gl
    double rexp = 0.0, ru2 = 0.0;
    constexpr int NR = BR > 0 ? BR : 1;
    D dr[NR];
    double pr[NR];
    if constexpr (BR > 0) {
#pragma unroll
        for (int b = 0; b < NR; ++b) {
            dr[b] = D{};
            pr[b] = 0.0;
            if (r_lo + b < r_hi) dr[b] = tb.desc[r_lo + b];
        }
    }
    while (__ballot(go)) {
        // 1. this lane's partial sum over its block (0 past its end)
        double part = 0.0;
        if constexpr (BR > 0) {
#pragma unroll
            for (int b = 0; b < NR; ++b) {
                const double p = propensity_from(dr[b], (uint32_t)lx[dr[b].s1], (uint32_t)lx[dr[b].s2]);
                pr[b] = r_lo + b < r_hi ? p : 0.0;
                part += pr[b];
            }
        } else if (go) {
            for (int32_t r = r_lo; r < r_hi; ++r) {
                const D d = tb.desc[r];
                part += propensity_from(d, (uint32_t)lx[d.s1], (uint32_t)lx[d.s2]);
            }
        }
        // 2. group scan, a0, waiting time (e is the same on a group's lanes)
        if (go && (e & (L - 1)) == 0u) {
            const U4 rnd = philox4x32_10(e + (uint32_t)gl, (uint32_t)k, iter, 0u, k0, k1);
            rexp = -log(1.0 - uniform53(rnd.x, rnd.y));
            ru2 = uniform53(rnd.z, rnd.w);
        }
        const int src = gbase + (int)(e & (L - 1));
        const double ex = __shfl(rexp, src, 64);
        const double uu = __shfl(ru2, src, 64);
        const double incl = group_scan_incl<L>(part);
        const double a0 = group_last<L>(incl);
        const double target = uu * a0;
        const double dt = ex / a0;
        // 3. the lane holding the target (rounding past the last block: the last
        // lane with a positive sum) and the reaction inside its block
        const uint64_t over = __ballot(incl > target) & gmask;
        const uint64_t pos = __ballot(part > 0.0) & gmask;
        const int chosen = over ? (__ffsll((long long)over) - 1)
                                : (pos ? 63 - __builtin_clzll(pos) : gbase + L - 1);
        go = go && a0 > 0.0;
        e += go ? 1u : 0u;
        go = go && !(t + dt > tau);
        t = go ? t + dt : t;
        int32_t j = -1;
        if constexpr (BR > 0) {
            // the propensities of step 1, in the same order
            const double t2 = target - (incl - part);
            double run_s = 0.0;
            bool found = false;
#pragma unroll
            for (int b = 0; b < NR; ++b) {
                const bool on = !found && pr[b] > 0.0;
                run_s = on ? run_s + pr[b] : run_s;
                j = on ? r_lo + b : j;
                found = found || (on && run_s > t2);
            }
        } else if (go && lane == chosen) {
            const double t2 = target - (incl - part);
            double run_s = 0.0;
            for (int32_t r = r_lo; r < r_hi; ++r) {
                const D d = tb.desc[r];
                const double ar = propensity_from(d, (uint32_t)lx[d.s1], (uint32_t)lx[d.s2]);
                if (ar > 0.0) {
                    j = r;
                    run_s += ar;
                    if (run_s > t2) break;
                }
            }
        }
        j = __shfl(j, chosen, 64);
        if (go && j < 0) {
            nosel = true;
            go = false;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // 4. state update, one change per lane
        bool lbad = false;
        if (go) {
            const int32_t c0 = tb.chg_ptr[j], c1 = tb.chg_ptr[j + 1];
            for (int32_t c = c0 + gl; c < c1; c += L) {
                const int32_t p = tb.chg[c];
                const int32_t sp = change_species(p);
                const int32_t nv = lx[sp] + change_delta(p);
                lx[sp] = nv;
                lbad = lbad || nv < 0 || nv > WE_COUNT_MAX_DEV;
            }
            fired += 1;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (__ballot(lbad) & gmask) {
            bad = true;
            go = false;
        }
    }
    if (live && gl == 0) {
        if (bad) atomicOr(a.err, WE_DERR_OVERFLOW);
        if (nosel) atomicOr(a.err, WE_DERR_SELECT);
    }
    if (live)
        for (int32_t s = gl; s < S; s += L) xw[s] = lx[s];
    if (live && gl == 0) a.ev_walker[(size_t)run * a.cap + k] = fired;
}
