// ssa_wave_body.h -- the wave-per-walker event loop, shared by the per-sim
// kernel and the batched persistent kernel.
//
// Cross-lane work uses the CDNA data-parallel primitives directly:
//  * inclusive prefix sums of FP64 values: four DPP row shifts (1, 2, 4, 8)
//    build scans inside each 16-lane row, then the row_bcast:15 and
//    row_bcast:31 broadcasts carry row totals across the wave -- six steps
//    of two 32-bit DPP moves and one add, no LDS round trip;
//  * broadcasts of one lane: v_readlane;
//  * the dependents' propensity changes go into the per-wave chunk sums in
//    LDS by ds_add_f64, one instruction per round of 64 dependents.
// Per event the dependent loads from global memory are: the chosen chunk's
// reaction headers (unless they are in LDS), then the fired reaction's
// dependency ids together with its changes.
#pragma once
#include <type_traits>

#include "queue_first.h"
#include "we_common.h"

#define WAVE_DEP_ROUNDS 2

namespace {

template <class D>
__device__ __forceinline__ double prop_lds(const D &d, const int32_t *lx) {
    return propensity_from(d, (uint32_t)lx[d.s1], (uint32_t)lx[d.s2]);
}

union F64Bits {
    double d;
    int32_t w[2];
};

template <int CTRL, int ROW_MASK, bool BOUND>
__device__ __forceinline__ double dpp_f64(double v) {
    F64Bits in, out;
    in.d = v;
    out.w[0] = __builtin_amdgcn_update_dpp(0, in.w[0], CTRL, ROW_MASK, 0xF, BOUND);
    out.w[1] = __builtin_amdgcn_update_dpp(0, in.w[1], CTRL, ROW_MASK, 0xF, BOUND);
    return out.d;
}

// Inclusive prefix sum over the 64 lanes (fixed order, reproducible).
__device__ __forceinline__ double scan_incl(double v) {
    v = v + dpp_f64<0x111, 0xF, true>(v);    // row_shr:1
    v = v + dpp_f64<0x112, 0xF, true>(v);    // row_shr:2
    v = v + dpp_f64<0x114, 0xF, true>(v);    // row_shr:4
    v = v + dpp_f64<0x118, 0xF, true>(v);    // row_shr:8
    v = v + dpp_f64<0x142, 0xA, false>(v);   // row_bcast:15 into rows 1 and 3
    v = v + dpp_f64<0x143, 0xC, false>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    F64Bits in, out;
    in.d = v;
    out.w[0] = __builtin_amdgcn_readlane(in.w[0], lane);
    out.w[1] = __builtin_amdgcn_readlane(in.w[1], lane);
    return out.d;
}

__device__ __forceinline__ int32_t last_set(unsigned long long m) {
    return m ? 63 - __clzll((long long)m) : -1;
}

// Issue priority of the calling wave from its walker's expected remaining
// events in the interval, (tau - t) * a0: longest remaining chain first.  A
// launch lasts as long as its longest walker chain, and waves sharing a SIMD
// compete for issue; the wave with more left to do then issues first and the
// others fill its dependency stalls.  Four levels (s_setprio 0..3), at 16,
// 48 and 96 remaining events.  Scheduling only: no result depends on it.
__device__ __forceinline__ void chain_priority(double rem) {
    if (rem > 96.0)
        __builtin_amdgcn_s_setprio(3);
    else if (rem > 48.0)
        __builtin_amdgcn_s_setprio(2);
    else if (rem > 16.0)
        __builtin_amdgcn_s_setprio(1);
    else
        __builtin_amdgcn_s_setprio(0);
}

// a + b with the upper half of a exchanged for the lower half of b: lanes 0-31
// hold the sums over lane pairs (l, l + 32) of a, lanes 32-63 those of b.
__device__ __forceinline__ double fold_halves(double a, double b) {
    F64Bits x, y;
    x.d = a;
    y.d = b;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)x.w[w], (uint32_t)y.w[w], false, false);
        x.w[w] = (int32_t)r[0];
        y.w[w] = (int32_t)r[1];
    }
    return x.d + y.d;
}

// The same between neighbouring 16-lane rows: even rows hold a's sums over the
// two rows of each half, odd rows b's.
__device__ __forceinline__ double fold_rows(double a, double b) {
    F64Bits x, y;
    x.d = a;
    y.d = b;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)x.w[w], (uint32_t)y.w[w], false, false);
        x.w[w] = (int32_t)r[0];
        y.w[w] = (int32_t)r[1];
    }
    return x.d + y.d;
}

// All chunk sums from scratch, chunk c's in lane c; prop(r) is this lane's
// propensity of reaction r.  Every walker starts each interval with this, so
// where an interval holds few events it is most of the work.  Four chunks at a
// time (c, c + 16, c + 32, c + 48) are folded into one register by lane-half
// and row swaps, row i then holding chunk c + 16 i, and summed over the rows
// together: 23 instructions of summation for four chunks where a scan of
// each took 26 apiece.
template <class P>
__device__ __forceinline__ double chunk_sums(int32_t R, int lane, P &&prop) {
    double cs = 0.0;
    const int32_t K = (R + 63) >> 6;
    for (int32_t c = 0; c < min(K, 16); ++c) {
        double v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int32_t r = (c + 16 * i) * 64 + lane;
            v[i] = 0.0;
            if (r < R) v[i] = prop(r);
        }
        // halves first: v[0], v[2] go to the lower and upper half, then v[1],
        // v[3] take the odd row of each
        double s = fold_rows(fold_halves(v[0], v[2]), fold_halves(v[1], v[3]));
        s = s + dpp_f64<0xB1, 0xF, true>(s);    // quad_perm [1,0,3,2]
        s = s + dpp_f64<0x4E, 0xF, true>(s);    // quad_perm [2,3,0,1]
        s = s + dpp_f64<0x141, 0xF, true>(s);   // row_half_mirror
        s = s + dpp_f64<0x140, 0xF, true>(s);   // row_mirror
        cs = (lane & 15) == c ? s : cs;
    }
    return cs;
}

// Add v to a double in LDS with one ds_add_f64 (no return value).  The LDS
// unit applies the lanes of one such instruction that hit the same address
// in a fixed order, so a sum built this way repeats bit for bit.
__device__ __forceinline__ void lds_add_f64(double *p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Add each lane's propensity change dv of dependent reaction rr (rr < 0 for
// idle lanes) to its chunk's sum.
__device__ __forceinline__ void add_chunk_deltas(double *lchunk, int rr, double dv) {
    if (rr >= 0) lds_add_f64(&lchunk[rr >> 6], dv);
}

}  // namespace

// Where the wave reads the network from.
//  LdsTables: descriptors from the block's LDS copy, headers from LDS or
//    global memory, the dependency lists (16-bit reaction ids) from global
//    memory and the dependents' descriptors from LDS.
// D: the descriptors' form (RxnDesc2 where the network has it).
template <class D>
struct LdsTables {
    struct Dep : D {
        uint16_t r;
    };
    static constexpr bool PAIR = std::is_same<D, RxnDesc2>::value;
    const D *d;                        // LDS
    const RxnInfo *h;                  // LDS or global
    const uint16_t *__restrict__ ids;  // global
    __device__ __forceinline__ D desc(int r) const { return d[r]; }
    __device__ __forceinline__ RxnInfo info(int j) const { return h[j]; }
    __device__ __forceinline__ Dep dep(int i) const {
        const int r = ids[i];
        Dep o;
        static_cast<D &>(o) = d[r];
        o.r = (uint16_t)r;
        return o;
    }
};

// One walker through one interval on the calling wave; lchunk (64 doubles)
// and lx (S + 1 ints: the counts, and the 1 an absent reactant reads) are this
// wave's LDS slices.
template <class T>
__device__ inline void wave_walker_t(const SimArgs &a, const T &tab, int32_t *__restrict__ xs, int32_t run,
                                     int32_t k, uint32_t iter, double *lchunk, int32_t *lx) {
    const int lane = threadIdx.x & 63;
    const int32_t S = a.S, R = a.R;
    int32_t *xw = xs + ((size_t)run * a.cap + k) * S;
    for (int s = lane; s < S; s += 64) lx[s] = xw[s];
    if (T::PAIR && lane == 0) lx[S] = 1;
    __builtin_amdgcn_wave_barrier();

    // chunk sums from scratch
    auto rebuild = [&]() {
        return chunk_sums(R, lane, [&](int32_t r) { return prop_lds(tab.desc(r), lx); });
    };
    double csum = rebuild();
    lchunk[lane] = csum;

    const uint64_t seed = a.seeds[run];
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const double tau = a.tau;
    double t = 0.0;
    uint32_t e = 0, fired = 0;
    bool bad = false;
    // random numbers of 64 events at a time, one event per lane: lane l holds
    // -log(1 - u1) and u2 of event (e & ~63) + l.  The general-purpose log is
    // kept here: it runs once per 64 events, and the lane kernels' shorter one
    // would hold its coefficients in registers across the whole event loop
    // (132 VGPRs instead of 124, one block per CU instead of two).
    double rexp = 0.0, ru2 = 0.0;

    for (;;) {
        const double P = scan_incl(csum);
        const double a0 = lane_value(P, 63);
        if ((e & 63u) == 0u) {
            const U4 rnd = philox4x32_10(e + (uint32_t)lane, (uint32_t)k, iter, 0u, k0, k1);
            rexp = -log(1.0 - uniform53(rnd.x, rnd.y));
            ru2 = uniform53(rnd.z, rnd.w);
        }
        const double ex = lane_value(rexp, (int)(e & 63u));
        const double u2 = lane_value(ru2, (int)(e & 63u));
        e += 1;
        const double dt = ex / a0;
        const double target = u2 * a0;

        // chunk holding the target
        const unsigned long long m1 = __ballot(P > target);
        int cs = m1 ? (__ffsll((long long)m1) - 1) : last_set(__ballot(csum > 0.0));
        if (cs < 0) cs = 0;
        cs = __builtin_amdgcn_readfirstlane(cs);
        const double base = lane_value(P - csum, cs);
        const double target2 = target - base;
        // reaction inside the chunk; each lane also fetches its reaction's
        // header, so the chosen one is a readlane away once j is known
        const int rsel = cs * 64 + lane;
        double v = 0.0;
        RxnInfo hinfo{0, 0, 0, 0};
        if (rsel < R) {
            hinfo = tab.info(rsel);
            v = prop_lds(tab.desc(rsel), lx);
        }
        // the interval's end, tested here so that the division's chain runs beside the
        // choice of the chunk and its loads (eight runs of 354 species x 4096 walkers
        // 938 -> 926 us per interval)
        if (!(a0 > 0.0) || t + dt > tau) break;
        t = t + dt;
        if ((e & 15u) == 1u) chain_priority((tau - t) * a0);
        const double Q = scan_incl(v);
        const unsigned long long m2 = __ballot(Q > target2);
        const int ls = m2 ? (__ffsll((long long)m2) - 1) : last_set(__ballot(v > 0.0));
        if (ls < 0) {              // chunk sum drifted above an all-zero chunk
            if (lane == 0) atomicOr(a.err, WE_DERR_SELECT);
            break;
        }
        // header of j; its dependents (with descriptors) and changes
        RxnInfo info;
        info.dep_begin = __builtin_amdgcn_readlane(hinfo.dep_begin, ls);
        info.dep_count = __builtin_amdgcn_readlane(hinfo.dep_count, ls);
        info.chg_begin = __builtin_amdgcn_readlane(hinfo.chg_begin, ls);
        info.chg_count = __builtin_amdgcn_readlane(hinfo.chg_count, ls);
        const int32_t nd = info.dep_count;
        const int nround = (nd + 63) >> 6;
        int32_t pc = 0;
        if (lane < info.chg_count) pc = a.chg[info.chg_begin + lane];
        int rr[WAVE_DEP_ROUNDS];
        double old[WAVE_DEP_ROUNDS];
        typename T::Dep de[WAVE_DEP_ROUNDS];
        if (nround <= WAVE_DEP_ROUNDS) {
#pragma unroll
            for (int q = 0; q < WAVE_DEP_ROUNDS; ++q) {
                rr[q] = -1;
                old[q] = 0.0;
                if (q < nround) {
                    const int idx = q * 64 + lane;
                    if (idx < nd) {
                        de[q] = tab.dep(info.dep_begin + idx);
                        rr[q] = de[q].r;
                        old[q] = prop_lds(de[q], lx);
                    }
                }
            }
        }
        // fire j
        __builtin_amdgcn_wave_barrier();
        bool lbad = false;
        if (lane < info.chg_count) {
            const int32_t s = change_species(pc);
            const int32_t nv = lx[s] + change_delta(pc);
            lx[s] = nv;
            lbad = (nv < 0) || (nv > WE_COUNT_MAX_DEV);
        }
        __builtin_amdgcn_wave_barrier();
        fired += 1;
        if (__ballot(lbad)) { bad = true; break; }

        // fold the dependents' changes into the chunk sums
        if (nround <= WAVE_DEP_ROUNDS) {
#pragma unroll
            for (int q = 0; q < WAVE_DEP_ROUNDS; ++q) {
                if (q < nround) {
                    double dv = 0.0;
                    if (rr[q] >= 0) dv = prop_lds(de[q], lx) - old[q];
                    add_chunk_deltas(lchunk, rr[q], dv);
                    __builtin_amdgcn_wave_barrier();
                }
            }
            csum = lchunk[lane];
        } else {
            // very long dependency list: rebuild every chunk sum
            csum = rebuild();
            lchunk[lane] = csum;
        }
    }
    if (bad && lane == 0) atomicOr(a.err, WE_DERR_OVERFLOW);
    __builtin_amdgcn_wave_barrier();
    for (int s = lane; s < S; s += 64) xw[s] = lx[s];
    if (lane == 0) a.ev_walker[(size_t)run * a.cap + k] = fired;
}
