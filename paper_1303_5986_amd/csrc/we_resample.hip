// we_resample.hip -- the WE bookkeeping between two propagation steps:
// recycling, binning, per-bin split/merge, the state gather and the
// observables (gfx950).  Per iteration, after the SSA kernel:
//
//   recycle_bin (one lane per walker, whole grid)
//      recycling (Sec. II.B.2): a walker whose state lies in
//      B = { x : sum_s coef_s x_s >= thr } is flagged and restarts from the
//      state A, keeping its weight; checked once, at the end of the interval
//      (the paper checks walkers only every tau);
//      bin of every walker on the progress coordinate, or on a grid over two
//      coordinates, bin = b1 + n1 * b2 (or, with learned bins, the bin is
//      written afterwards by the committor kernel);
//   resample (one workgroup per run)
//      stable placement of the walkers by bin: per-wave cursor rows let
//      several waves place their own runs of slots at once;
//      the run's recycled weight (summed in slot order) and reactions fired;
//      per-bin split/merge (Sec. II.B), one wave per bin:
//        n == M: unchanged;
//        n <  M: replicate to M copies; one more copy is given, repeatedly,
//                to the parent with the largest per-copy weight w/c (ties:
//                lowest slot); each copy carries w/c, so the bin's weight is
//                conserved (a lone walker gets the paper's w/M exactly); the
//                wave finds the largest share with DPP max steps;
//        n >  M: merge the two lowest-weight walkers (ties: lowest slot): the
//                first survives with probability w_i/(w_i+w_j), else the
//                second, and the survivor carries w_i + w_j; repeat.
//        With the weight-equalizing rule (rs_rule 1), whatever n: W is the
//        bin's weight summed in slot order and w* = W/M; the two lowest are
//        merged as above while their sum is <= w* or the bin has no room to
//        split its heavy walkers (sum_k max(1, ceil(w_k/(2w*))) > M, which
//        includes n > M); the survivors are then replicated up to M as above.
//        Up to 256 walkers a bin is held in registers, up to four walkers per
//        lane, and each merge takes two DPP wave minima.  Larger bins are sorted once
//        by (weight, slot); merged walkers queue up in the order they are
//        made, which is also non-decreasing in weight, so each merge only
//        compares the heads of the two queues (ties of equal sums ordered by
//        a small heap): the same pairs as a full search, in O(n log n)
//        instead of O(n^2);
//        where one wave per bin has the LDS for it, many such merges at a time
//        (merge_bin_rounds);
//      output order: bins ascending, parents by ascending slot, copies of a
//      parent consecutive -- neighbouring lanes then hold walkers of similar
//      state for the next SSA step;
//      per-walker bin, weight and list arrays are staged in LDS;
//   gather_rows (one lane per count, whole grid): new state rows copied
//      from their parents;
//   observe: P(x_s = k, t) accumulated per run with FP64 atomics.
// All weight arithmetic is sequential per bin, so weights are reproducible
// bit for bit.
#include "we_common.h"
#include "we_internal.h"

#include <algorithm>

#define RESAMPLE_LDS_CAP 8192
#define RESAMPLE_LDS_MAX (150 * 1024)
// Cursor rows for placing walkers in parallel: one row of n_bins per wave, as
// long as the rows hold at most this many counters.
#define RESAMPLE_PLACE_INTS 8192   // 16 rows of 512 bins
// With more bins than this (up to 8192) the tables, 20 bytes a bin beside the 8 KB
// of event totals, would pass a CU's 160 KB (from 7782 bins on).  The events per bin
// then lie where the output offsets are written once they are read; 16 bytes a bin.
#define RESAMPLE_EVB_BINS 7600
// Bin-parallel resampling: runs fewer than this, bins at least this many.
#define RESAMPLE_BIN_PARALLEL_RUNS 256
#define RESAMPLE_BIN_PARALLEL_BINS 32
#define RESAMPLE_BIG_M 128
// Recycling and binning in the run's workgroup: rows of at most this many counts.
#define RESAMPLE_ROW_MAX 4
// Threads per run: up to 16 waves, so up to 16 bins are split/merged at
// once.  With many runs the grid fills the chip anyway and smaller blocks
// cost less to start, so launches with at least RESAMPLE_MANY_RUNS blocks use
// 4 waves per run.
#define RESAMPLE_THREADS 1024
#define RESAMPLE_MANY_RUNS 512
__host__ inline unsigned resample_threads(int64_t blocks) {
    return blocks >= RESAMPLE_MANY_RUNS ? 256u : (unsigned)RESAMPLE_THREADS;
}

// sum_s coef_s x_s in ascending species order over the nonzero
// coefficients only: a zero coefficient adds +0 or -0, which leaves a sum
// that started at +0 unchanged, so the result is the full sum bit for bit.
__device__ __forceinline__ double coord_of(const double *__restrict__ coef, const int32_t *__restrict__ nz,
                                           int32_t n_nz, const int32_t *__restrict__ xr) {
    double q = 0.0;
    for (int32_t i = 0; i < n_nz; ++i) {
        const int32_t s = nz[i];
        q = q + coef[s] * (double)xr[s];
    }
    return q;
}

__device__ __forceinline__ void recycle_bin_one(const SimArgs &a, int32_t *__restrict__ x_cur, int32_t grid_bins,
                                                int64_t gid) {
    const int32_t run = (int32_t)(gid / a.cap);
    const int32_t k = (int32_t)(gid - (int64_t)run * a.cap);
    if (run >= a.n_runs) return;
    if (k >= a.n_walk[run]) return;
    const int32_t S = a.S;
    const size_t idx = (size_t)run * a.cap + k;
    int32_t *row = x_cur + idx * S;
    int32_t rec = 0;
    if (a.recycle && coord_of(a.tgt_coef, a.tgt_nz, a.n_tgt_nz, row) >= a.tgt_thr) {
        rec = 1;
        for (int32_t s = 0; s < S; ++s) row[s] = a.x_rec[s];
    }
    a.s_rec[idx] = rec;
    if (grid_bins) {
        int32_t b = bin_index(a.edges, a.n_bins1, coord_of(a.bin_coef, a.bin_nz, a.n_bin_nz, row));
        if (a.n_bins2 > 1)
            b += a.n_bins1 * bin_index(a.edges2, a.n_bins2, coord_of(a.bin_coef2, a.bin_nz2, a.n_bin_nz2, row));
        a.s_bin[idx] = b;
    }
}

__global__ __launch_bounds__(256) void we_recycle_bin_kernel(SimArgs a, int32_t *__restrict__ x_cur,
                                                             int32_t grid_bins) {
    recycle_bin_one(a, x_cur, grid_bins, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Per-walker working arrays of one run (LDS when the run fits, else global);
// Idx is the type of an index inside one bin (uint16 in LDS, int32 in global).
template <class Idx>
struct RunWork {
    double *w;          // weights in bin-major order (-1 marks a merged-away walker)
    int32_t *list;      // slots in bin-major order
    uint16_t *tag;      // per slot: bin | 0x8000 if recycled (until placement)
    Idx *aux;           // per position: split copy counts, or the merge sort order
    Idx *qa;            // per position: queue of merged walkers (aliases tag)
};

namespace {

union RsBits {
    double d;
    int32_t w[2];
};

template <int CTRL>
__device__ __forceinline__ double rs_dpp(double v) {
    RsBits in, out;
    in.d = v;
    out.w[0] = __builtin_amdgcn_update_dpp(0, in.w[0], CTRL, 0xF, 0xF, false);
    out.w[1] = __builtin_amdgcn_update_dpp(0, in.w[1], CTRL, 0xF, 0xF, false);
    return out.d;
}

__device__ __forceinline__ double rs_readlane(double v, int l) {
    RsBits in, out;
    in.d = v;
    out.w[0] = __builtin_amdgcn_readlane(in.w[0], l);
    out.w[1] = __builtin_amdgcn_readlane(in.w[1], l);
    return out.d;
}

// Largest value over the 64 lanes (every lane gets it): quad swaps, half-row
// and row mirrors give each 16-lane row its maximum; four readlanes finish.
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, rs_dpp<0xB1>(v));    // quad_perm [1,0,3,2]
    v = fmax(v, rs_dpp<0x4E>(v));    // quad_perm [2,3,0,1]
    v = fmax(v, rs_dpp<0x141>(v));   // row_half_mirror
    v = fmax(v, rs_dpp<0x140>(v));   // row_mirror
    return fmax(fmax(rs_readlane(v, 0), rs_readlane(v, 16)), fmax(rs_readlane(v, 32), rs_readlane(v, 48)));
}

// Smallest value over the 64 lanes, by the same steps as wave_max.
__device__ __forceinline__ double wave_min(double v) {
    v = fmin(v, rs_dpp<0xB1>(v));
    v = fmin(v, rs_dpp<0x4E>(v));
    v = fmin(v, rs_dpp<0x141>(v));
    v = fmin(v, rs_dpp<0x140>(v));
    return fmin(fmin(rs_readlane(v, 0), rs_readlane(v, 16)), fmin(rs_readlane(v, 32), rs_readlane(v, 48)));
}

// Integer sum, minimum and exclusive prefix sum over the 64 lanes by DPP moves
// (a shuffle per step is an LDS round trip of over a hundred cycles).
template <int CTRL, int ROW_MASK, bool BOUND>
__device__ __forceinline__ int32_t rs_dpp_i32(int32_t v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xF, BOUND);
}
__device__ __forceinline__ int32_t wave_sum_i32(int32_t v) {
    v += rs_dpp_i32<0xB1, 0xF, false>(v);
    v += rs_dpp_i32<0x4E, 0xF, false>(v);
    v += rs_dpp_i32<0x141, 0xF, false>(v);
    v += rs_dpp_i32<0x140, 0xF, false>(v);
    return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
           (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
__device__ __forceinline__ int32_t wave_excl_scan(int32_t v, int32_t *total) {
    int32_t x = v;
    x += rs_dpp_i32<0x111, 0xF, true>(x);    // row_shr:1, 2, 4, 8
    x += rs_dpp_i32<0x112, 0xF, true>(x);
    x += rs_dpp_i32<0x114, 0xF, true>(x);
    x += rs_dpp_i32<0x118, 0xF, true>(x);
    x += rs_dpp_i32<0x142, 0xA, false>(x);   // row_bcast:15 into rows 1 and 3
    x += rs_dpp_i32<0x143, 0xC, false>(x);   // row_bcast:31 into rows 2 and 3
    *total = __builtin_amdgcn_readlane(x, 63);
    return x - v;
}

// Sum over the 64 lanes (every lane gets it), by the steps of wave_max.
__device__ __forceinline__ double wave_sum_f64(double v) {
    v += rs_dpp<0xB1>(v);
    v += rs_dpp<0x4E>(v);
    v += rs_dpp<0x141>(v);
    v += rs_dpp<0x140>(v);
    return (rs_readlane(v, 0) + rs_readlane(v, 16)) + (rs_readlane(v, 32) + rs_readlane(v, 48));
}

// Orders the LDS/global accesses of the lanes of one wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lanes whose v has the same low `bits` bits, among the valid ones; and
// how many of them come before this lane.
__device__ __forceinline__ unsigned long long match_lanes(int32_t v, bool valid, int bits) {
    unsigned long long m = __ballot(valid);
    for (int i = 0; i < bits; ++i) {
        const bool one = (v >> i) & 1;
        const unsigned long long o = __ballot(one);
        m &= one ? o : ~o;
    }
    return m;
}
__device__ __forceinline__ int32_t lanes_below(unsigned long long m) {
    return (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// sum[b] += v over the lanes with b >= 0.  Lanes of one 16-lane row are folded
// pairwise where they hold the same b first: LDS atomics of 64 lanes on one
// address take their turns, and walkers sit by their previous bin.
template <int CTRL>
__device__ __forceinline__ int32_t rs_dpp(int32_t v, int32_t none) {
    return __builtin_amdgcn_update_dpp(none, v, CTRL, 0xF, 0xF, false);
}
template <int FROM_HIGH, int FROM_LOW, int BIT>
__device__ __forceinline__ void fold_same(int32_t &b, float &v, int lane) {
    const int32_t hi_b = rs_dpp<FROM_HIGH>(b, -2), lo_b = rs_dpp<FROM_LOW>(b, -2);
    const float hi_v = __int_as_float(rs_dpp<FROM_HIGH>(__float_as_int(v), 0));
    const bool high = (lane & BIT) != 0;
    v = !high && hi_b == b ? v + hi_v : v;
    b = high && lo_b == b ? -1 : b;
}
__device__ __forceinline__ void add_by_bin(float *sum, int32_t b, float v, int lane) {
    fold_same<0x101, 0x111, 1>(b, v, lane);   // row_shl, row_shr by 1, 2, 4, 8
    fold_same<0x102, 0x112, 2>(b, v, lane);
    fold_same<0x104, 0x114, 4>(b, v, lane);
    fold_same<0x108, 0x118, 8>(b, v, lane);
    if (b >= 0) atomicAdd(&sum[b], v);
}

__device__ __forceinline__ int32_t uni(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Copies a walker of weight v needs so that none carries more than twice the
// bin's ideal weight (at least one: every walker holds a place).
__device__ __forceinline__ int32_t need_copies(double v, double two_ideal) {
    const double q = ceil(v / two_ideal);
    return q < 1.0 ? 1 : (int32_t)q;
}

struct BinOut {
    int32_t *orig;
    double *wn;
    int32_t *obin;
};

// n < M: M - n extra copies handed out one at a time to the parent with the
// largest per-copy weight w/c, ties to the lowest slot.  Lane L owns the
// contiguous parents [L*kq, (L+1)*kq), so the lowest lane holding the wave's
// largest share holds the lowest tied slot.
template <class Idx>
__device__ void split_bin(const RunWork<Idx> &wk, int32_t p0, int32_t nb, int32_t M, int32_t b, int32_t o0,
                          const BinOut &out, int lane) {
    const int32_t kq = (nb + 63) >> 6;
    const int32_t q_lo = min(lane * kq, nb), q_hi = min(q_lo + kq, nb);
    const double *w = wk.w + p0;
    Idx *c = wk.aux + p0;
    double bs = -1.0;
    int32_t bq = -1;
    for (int32_t q = q_lo; q < q_hi; ++q) {
        c[q] = 1;
        const double s = w[q] / 1.0;
        if (s > bs) { bs = s; bq = q; }
    }
    for (int32_t e = nb; e < M; ++e) {
        const double mx = wave_max(bs);
        const unsigned long long win = __ballot(bs == mx);
        const int wl = __ffsll((long long)win) - 1;
        if (lane == wl) {
            c[bq] = (Idx)(c[bq] + 1);
            bs = -1.0;
            bq = -1;
            for (int32_t q = q_lo; q < q_hi; ++q) {
                const double s = w[q] / (double)c[q];
                if (s > bs) { bs = s; bq = q; }
            }
        }
    }
    int32_t cl = 0;
    for (int32_t q = q_lo; q < q_hi; ++q) cl += (int32_t)c[q];
    int32_t tot;
    int32_t o = o0 + wave_excl_scan(cl, &tot);
    for (int32_t q = q_lo; q < q_hi; ++q) {
        const int32_t cc = (int32_t)c[q];
        const double share = w[q] / (double)cc;
        const int32_t k = wk.list[p0 + q];
        for (int32_t r = 0; r < cc; ++r) {
            out.orig[o] = k;
            out.wn[o] = share;
            out.obin[o] = b;
            ++o;
        }
    }
}

// Steady-state reweighting's flux matrix (Sec. II.B.2): row `Frow` (end bin
// b) gains, walker by walker in slot order, the weight of each of the bin's
// walkers in the column of its start bin (held in aux; bits: bits of a bin's
// number).  The row is this wave's alone.  64 walkers at a time: the first lane
// of each start bin fetches the column, adds its lanes' weights in lane order
// and writes it back, the start bins side by side.  One column after another
// (a fetch each, and a wave minimum to find the next) the split/merge of 64 runs
// of 465 bins x 16 walkers took 92 us, this way 53.6; 32 runs of 80 x 32 44 and 33.8.
template <class Idx>
__device__ void rw_flux_bin(double *__restrict__ Frow, const RunWork<Idx> &wk, int32_t p0, int32_t nb, int bits,
                            int lane) {
    for (int32_t c0 = 0; c0 < nb; c0 += 64) {
        const int32_t q = c0 + lane;
        const bool valid = q < nb;
        const int32_t j = valid ? (int32_t)wk.aux[p0 + q] : 0;
        const double wv = valid ? wk.w[p0 + q] : 0.0;
        const unsigned long long grp = match_lanes(j, valid, bits);
        const bool first = valid && lanes_below(grp) == 0;
        unsigned long long left = first ? grp : 0ull;   // lanes still to add
        double acc = first ? Frow[j] : 0.0;
        while (__ballot(left != 0ull)) {
            const double v = __shfl(wv, left ? __ffsll((long long)left) - 1 : 0, 64);
            acc = left ? acc + v : acc;
            left &= left - 1ull;
        }
        if (first) Frow[j] = acc;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        wave_sync();
    }
}

// The lowest slot whose entry of v equals w, given that there is one: walker
// q of a bin held in registers lives in lane q % 64, register q / 64.
template <int K>
__device__ __forceinline__ int32_t lowest_slot(const double (&v)[K], double w) {
    int32_t q = -1;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
        const unsigned long long m = __ballot(v[k] == w);
        if (m) q = 64 * k + __ffsll((long long)m) - 1;
    }
    return q;
}

// The n walkers of a bin with live[k] set, weights wv, replicated up to M
// copies and written out: one copy each, then one more at a time to the largest
// share w/c, ties to the lowest slot.  One at a time each copy is a chain of a
// wave maximum, ballots and a division, so two things are done at once:
//  - what is certain.  The copies given are the M - n largest of all shares w/1,
//    w/2, ... in that order, so for any lambda with at most M - n shares of
//    lambda or more, every share above it is given: a walker has at least
//    ceil(w / lambda) copies.  lambda is bisected, from W / (M - n) down (W the
//    sum of the weights), until at most RESAMPLE_FEW copies are left.  Counts are
//    taken at 1 -+ 2^-36 times w / lambda, which covers every rounding here and
//    of the shares (weights of 1e-280 and more; subnormal shares round by more);
//  - ties.  Walkers of the same largest share get their copy together, the
//    lowest slots first if there are more of them than copies left.
#define RESAMPLE_FEW 3
template <int K, class Idx>
__device__ __forceinline__ void hand_out(const RunWork<Idx> &wk, int32_t p0, int32_t M, int32_t b, int32_t o0,
                                         const BinOut &out, const double (&wv)[K], const bool (&live)[K], int32_t n,
                                         int lane) {
    int32_t c[K];
    double sh[K];                         // per-copy shares; -1: not live
#pragma unroll
    for (int k = 0; k < K; ++k) {
        c[k] = live[k] ? 1 : 0;
        sh[k] = live[k] ? wv[k] : -1.0;
    }
    int32_t have = n;
    if (M - n > 2 * RESAMPLE_FEW) {
        double wl = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) wl += live[k] ? wv[k] : 0.0;
        const double W = wave_sum_f64(wl);
        if (W >= 1e-280) {
            // 1 / lambda: at f_lo few enough shares, at f_hi (perhaps) too many
            double f_lo = (double)(M - n) / W * (1.0 - 0x1.0p-35), f_hi = (double)M / W, f = f_lo;
            for (int32_t it = 0; it < 12; ++it) {
                int32_t up = 0, dn = 0;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (live[k]) {
                        const double x = wv[k] * f;
                        up += max(1, (int32_t)ceil(x * (1.0 + 0x1.0p-36)));
                        dn += max(1, (int32_t)ceil(x * (1.0 - 0x1.0p-36)));
                    }
                if (wave_sum_i32(up) <= M) {
                    f_lo = f;
                    have = wave_sum_i32(dn);
                    if (M - have <= RESAMPLE_FEW) break;
                } else {
                    f_hi = f;
                }
                f = 0.5 * (f_lo + f_hi);
            }
            if (have > n) {
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (live[k]) {
                        c[k] = max(1, (int32_t)ceil(wv[k] * f_lo * (1.0 - 0x1.0p-36)));
                        sh[k] = wv[k] / (double)c[k];
                    }
            }
        }
    }
    while (have < M) {
        double lm = sh[0];
#pragma unroll
        for (int k = 1; k < K; ++k) lm = fmax(lm, sh[k]);
        const double mx = wave_max(lm);
        // a share that another copy may not make smaller (0, or subnormal): the
        // lowest slot alone, which then stays in front
        const int32_t room = mx >= 1e-280 ? M - have : 1;
        int32_t before = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool tied = sh[k] == mx;
            const unsigned long long m = __ballot(tied);
            if (tied && before + (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0)) < room) {
                c[k] += 1;
                sh[k] = wv[k] / (double)c[k];
            }
            before += (int32_t)__popcll(m);
        }
        have += min(before, room);
    }
    int32_t o = o0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int32_t tot;
        int32_t ok = o + wave_excl_scan(c[k], &tot);
        if (c[k] > 0) {
            const int32_t kk = wk.list[p0 + 64 * k + lane];
            for (int32_t r = 0; r < c[k]; ++r) {
                out.orig[ok] = kk;
                out.wn[ok] = sh[k];
                out.obin[ok] = b;
                ++ok;
            }
        }
        o += tot;
    }
}

// n < M with at most 64 K parents, in registers.
template <int K, class Idx>
__device__ void split_bin_lanes(const RunWork<Idx> &wk, int32_t p0, int32_t nb, int32_t M, int32_t b, int32_t o0,
                                const BinOut &out, int lane) {
    double wv[K];
    bool live[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        live[k] = 64 * k + lane < nb;
        wv[k] = live[k] ? wk.w[p0 + 64 * k + lane] : 0.0;
    }
    hand_out<K>(wk, p0, M, b, o0, out, wv, live, nb, lane);
}

// The merge queues of one bin.  Q1: the bin's walkers sorted by (weight,
// slot).  Q2: merged walkers in the order they were made; their weights never
// decrease (each merge takes the two lightest, so every later pair sums to at
// least as much), so only equal-weight runs of Q2 need ordering by slot: the
// run at the front of Q2 is kept as a min-heap on the slot in A[hs, he);
// A[he, re) are spent entries and A[re, t) is the rest of Q2 in order.
// Every lane runs the same steps; lane 0 does the stores.
template <class Idx>
struct MergeQueues {
    const Idx *perm;
    Idx *A;
    double *W;
    int32_t nb, h1, q1;
    double w1;
    int32_t hs, he, re, t;
    double hw;
    int lane;

    __device__ void put(int32_t i, int32_t v) {
        if (lane == 0) A[i] = (Idx)v;
        wave_sync();
    }

    __device__ void sift_down(int32_t pos, int32_t size, int32_t x) {
        for (;;) {
            int32_t ch = 2 * pos + 1;
            if (ch >= size) break;
            int32_t cv = uni((int32_t)A[hs + ch]);
            if (ch + 1 < size) {
                const int32_t cv2 = uni((int32_t)A[hs + ch + 1]);
                if (cv2 < cv) { ch += 1; cv = cv2; }
            }
            if (cv >= x) break;
            put(hs + pos, cv);
            pos = ch;
        }
        put(hs + pos, x);
    }

    __device__ void refill() {
        hs = re;
        hw = W[uni((int32_t)A[re])];
        int32_t e = re + 1;
        while (e < t && W[uni((int32_t)A[e])] == hw) ++e;
        he = e;
        re = e;
        for (int32_t i = (e - hs) / 2 - 1; i >= 0; --i) sift_down(i, e - hs, uni((int32_t)A[hs + i]));
    }

    // remove and return the lightest walker (ties: lowest slot)
    __device__ void pop(double *wo, int32_t *qo) {
        if (he == hs && re < t) refill();
        const bool has1 = h1 < nb, has2 = he > hs;
        int32_t q2 = has2 ? uni((int32_t)A[hs]) : 0;
        const bool take1 = has1 && (!has2 || w1 < hw || (w1 == hw && q1 < q2));
        if (take1) {
            *wo = w1;
            *qo = q1;
            ++h1;
            if (h1 < nb) {
                q1 = uni((int32_t)perm[h1]);
                w1 = W[q1];
            }
        } else {
            *wo = hw;
            *qo = q2;
            --he;
            if (he > hs) sift_down(0, he - hs, uni((int32_t)A[he]));
        }
    }

    __device__ void push(double s, int32_t q) {
        if (he > hs && re == t && s == hw) {
            int32_t pos = he - hs;
            if (he == t) { ++t; ++re; }
            ++he;
            while (pos > 0) {
                const int32_t par = (pos - 1) >> 1;
                const int32_t pv = uni((int32_t)A[hs + par]);
                if (pv <= q) break;
                put(hs + pos, pv);
                pos = par;
            }
            put(hs + pos, q);
        } else {
            put(t, q);
            ++t;
        }
    }
};

// n > M with at most 64 K walkers: walker q lives in lane q % 64, register
// q / 64.  Each merge finds the lightest live walker by a wave minimum (ties:
// the lowest register, then the lowest lane, i.e. the lowest slot), then the
// lightest of the rest; the merged-away walker holds +inf from then on.  The
// same pairs, draws and sums as merge_bin, without its sort of the bin.
template <int K, class Idx>
__device__ void merge_bin_lanes(const RunWork<Idx> &wk, int32_t p0, int32_t nb, int32_t M, int32_t b, int32_t o0,
                                const BinOut &out, uint32_t iter, uint32_t k0, uint32_t k1, int lane) {
    const double inf = __builtin_huge_val();
    double wv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) wv[k] = 64 * k + lane < nb ? wk.w[p0 + 64 * k + lane] : inf;
    double ul = 0.0;
    for (int32_t m = 0; m < nb - M; ++m) {
        if ((m & 63) == 0) {   // the next 64 merge draws, one per lane
            const U4 rr = philox4x32_10((uint32_t)(m + lane), (uint32_t)b, iter, 1u, k0, k1);
            ul = uniform53(rr.x, rr.y);
        }
        double lm = wv[0];
#pragma unroll
        for (int k = 1; k < K; ++k) lm = fmin(lm, wv[k]);
        const double wi = wave_min(lm);
        const int32_t qi = lowest_slot(wv, wi);
        double wr[K];
#pragma unroll
        for (int k = 0; k < K; ++k) wr[k] = (64 * k + lane == qi) ? inf : wv[k];
        double lr = wr[0];
#pragma unroll
        for (int k = 1; k < K; ++k) lr = fmin(lr, wr[k]);
        const double wj = wave_min(lr);
        const int32_t qj = lowest_slot(wr, wj);
        const double u = rs_readlane(ul, m & 63);
        const double sum = wi + wj;
        const double p_i = wi / sum;
        const int32_t keep = (u < p_i) ? qi : qj;
        const int32_t drop = (keep == qi) ? qj : qi;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (64 * k + lane == keep) wv[k] = sum;
            if (64 * k + lane == drop) wv[k] = inf;
        }
    }
    int32_t o = o0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool live = 64 * k + lane < nb && wv[k] != inf;
        int32_t tot;
        const int32_t ok = o + wave_excl_scan(live ? 1 : 0, &tot);
        if (live) {
            out.orig[ok] = wk.list[p0 + 64 * k + lane];
            out.wn[ok] = wv[k];
            out.obin[ok] = b;
        }
        o += tot;
    }
}

// After merging with the weight-equalizing rule: the n_live survivors of a
// bin (positions whose weight is >= 0; merged-away ones hold -1) replicated
// up to M copies as in split_bin, the counts in aux.
template <class Idx>
__device__ void split_survivors(const RunWork<Idx> &wk, int32_t p0, int32_t nb, int32_t n_live, int32_t M,
                                int32_t b, int32_t o0, const BinOut &out, int lane) {
    const int32_t kq = (nb + 63) >> 6;
    const int32_t q_lo = min(lane * kq, nb), q_hi = min(q_lo + kq, nb);
    const double *w = wk.w + p0;
    Idx *c = wk.aux + p0;
    double bs = -1.0;
    int32_t bq = -1;
    for (int32_t q = q_lo; q < q_hi; ++q) {
        const bool live = w[q] >= 0.0;
        c[q] = (Idx)(live ? 1 : 0);
        if (live) {
            const double sh = w[q] / 1.0;
            if (sh > bs) { bs = sh; bq = q; }
        }
    }
    for (int32_t e = n_live; e < M; ++e) {
        const double mx = wave_max(bs);
        const int wl = __ffsll((long long)__ballot(bs == mx)) - 1;
        if (lane == wl) {
            c[bq] = (Idx)(c[bq] + 1);
            bs = -1.0;
            bq = -1;
            for (int32_t q = q_lo; q < q_hi; ++q) {
                if (!(w[q] >= 0.0)) continue;
                const double sh = w[q] / (double)c[q];
                if (sh > bs) { bs = sh; bq = q; }
            }
        }
    }
    int32_t cl = 0;
    for (int32_t q = q_lo; q < q_hi; ++q) cl += (int32_t)c[q];
    int32_t tot;
    int32_t o = o0 + wave_excl_scan(cl, &tot);
    for (int32_t q = q_lo; q < q_hi; ++q) {
        const int32_t cc = (int32_t)c[q];
        if (cc == 0) continue;
        const double share = w[q] / (double)cc;
        const int32_t k = wk.list[p0 + q];
        for (int32_t r = 0; r < cc; ++r) {
            out.orig[o] = k;
            out.wn[o] = share;
            out.obin[o] = b;
            ++o;
        }
    }
}

// Weight-equalizing rule with at most 64 K walkers: walker q lives in lane
// q % 64, register q / 64.  The merges are merge_bin_lanes' (same pairs, draws
// and sums) under the rule's condition; the survivors are then replicated by
// the same hand-out as split_bin (the largest share, ties to the lowest slot:
// the lowest register, then the lowest lane), merged-away ones holding +inf
// and getting no copy.  Every step of a bin is a chain of wave reductions, so
// what bounds it is their latency: in registers a merge takes two wave minima
// (about a thousand cycles) where merge_bin's queues wait on several dependent
// loads of the bin's arrays.  Ten futile-cycle runs of 101 bins x 100 walkers:
// 428 -> 252 us per interval with bins of 65 to 256 walkers on this path, which
// the bin-parallel launch now merges in rounds.
template <int K, class Idx>
__device__ void equalize_bin_lanes(const RunWork<Idx> &wk, int32_t p0, int32_t nb, int32_t M, int32_t b,
                                   int32_t o0, const BinOut &out, uint32_t iter, uint32_t k0, uint32_t k1,
                                   int lane) {
    const double inf = __builtin_huge_val();
    double wv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) wv[k] = 64 * k + lane < nb ? wk.w[p0 + 64 * k + lane] : inf;
    double Wb = 0.0;                      // the bin's weight, in slot order
#pragma unroll
    for (int k = 0; k < K; ++k)
        for (int32_t l = 0; l < min(nb - 64 * k, 64); ++l) Wb = Wb + rs_readlane(wv[k], l);
    const bool eq = Wb > 0.0;
    const double ideal = Wb / (double)M;
    const double two_ideal = ideal + ideal;
    int32_t nl = 0;
    if (eq) {
#pragma unroll
        for (int k = 0; k < K; ++k) nl += 64 * k + lane < nb ? need_copies(wv[k], two_ideal) : 0;
    }
    int32_t need = wave_sum_i32(nl);
    int32_t n = nb;
    double ul = 0.0;
    for (int32_t m = 0; n > 1; ++m) {
        double lm = wv[0];
#pragma unroll
        for (int k = 1; k < K; ++k) lm = fmin(lm, wv[k]);
        const double wi = wave_min(lm);
        const int32_t qi = lowest_slot(wv, wi);
        double wr[K];
#pragma unroll
        for (int k = 0; k < K; ++k) wr[k] = 64 * k + lane == qi ? inf : wv[k];
        double lr = wr[0];
#pragma unroll
        for (int k = 1; k < K; ++k) lr = fmin(lr, wr[k]);
        const double wj = wave_min(lr);
        const double sum = wi + wj;
        const bool go = eq ? (sum <= ideal || need > M) : (n > M);
        if (!go) break;
        const int32_t qj = lowest_slot(wr, wj);
        if ((m & 63) == 0) {   // the next 64 merge draws, one per lane
            const U4 rr = philox4x32_10((uint32_t)(m + lane), (uint32_t)b, iter, 1u, k0, k1);
            ul = uniform53(rr.x, rr.y);
        }
        const double u = rs_readlane(ul, m & 63);
        const double p_i = wi / sum;
        const int32_t keep = (u < p_i) ? qi : qj;
        const int32_t drop = (keep == qi) ? qj : qi;
        if (eq) need = need - need_copies(wi, two_ideal) - need_copies(wj, two_ideal) + need_copies(sum, two_ideal);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (64 * k + lane == keep) wv[k] = sum;
            if (64 * k + lane == drop) wv[k] = inf;
        }
        n -= 1;
    }
    bool live[K];
#pragma unroll
    for (int k = 0; k < K; ++k) live[k] = 64 * k + lane < nb && wv[k] != inf;
    hand_out<K>(wk, p0, M, b, o0, out, wv, live, n, lane);
}

// n > M: merge the two lightest walkers (ties: lowest slot) until M remain.
// EQ: the weight-equalizing rule's merges, then the survivors' split.
template <class Idx, bool EQ>
__device__ void merge_bin(const RunWork<Idx> &wk, int32_t p0, int32_t nb, int32_t M, int32_t b, int32_t o0,
                          const BinOut &out, uint32_t iter, uint32_t k0, uint32_t k1, int lane) {
    double *W = wk.w + p0;
    Idx *perm = wk.aux + p0;
    bool eq = false;
    double ideal = 0.0, two_ideal = 0.0;
    int32_t need = 0;
    if (EQ) {
        double Wb = 0.0;                  // the bin's weight, in slot order
        for (int32_t q = 0; q < nb; ++q) Wb = Wb + W[q];
        eq = Wb > 0.0;
        ideal = Wb / (double)M;
        two_ideal = ideal + ideal;
        if (eq) {
            int32_t nl = 0;
            for (int32_t q = lane; q < nb; q += 64) nl += need_copies(W[q], two_ideal);
            need = wave_sum_i32(nl);
        }
        wave_sync();
    }
    // sort order of the bin by (weight, slot): bitonic network whose first
    // step of every merge compares mirrored pairs, so positions past nb act as
    // +inf and never move
    for (int32_t q = lane; q < nb; q += 64) perm[q] = (Idx)q;
    wave_sync();
    int32_t P = 1;
    while (P < nb) P <<= 1;
    for (int32_t size = 2; size <= P; size <<= 1) {
        for (int32_t d = size >> 1; d > 0; d >>= 1) {
            const bool mirror = d == (size >> 1);
            for (int32_t cidx = lane; cidx < (P >> 1); cidx += 64) {
                const int32_t blk = cidx / d, r = cidx - blk * d;
                int32_t i, j;
                if (mirror) {
                    i = blk * size + r;
                    j = blk * size + size - 1 - r;
                } else {
                    i = blk * 2 * d + r;
                    j = i + d;
                }
                if (j < nb) {
                    const int32_t qi = (int32_t)perm[i], qj = (int32_t)perm[j];
                    const double wi = W[qi], wj = W[qj];
                    if (wj < wi || (wj == wi && qj < qi)) {
                        perm[i] = (Idx)qj;
                        perm[j] = (Idx)qi;
                    }
                }
            }
            wave_sync();
        }
    }

    MergeQueues<Idx> Q;
    Q.perm = perm;
    Q.A = wk.qa + p0;
    Q.W = W;
    Q.nb = nb;
    Q.h1 = 0;
    Q.q1 = uni((int32_t)perm[0]);
    Q.w1 = W[Q.q1];
    Q.hs = Q.he = Q.re = Q.t = 0;
    Q.hw = 0.0;
    Q.lane = lane;
    double ul = 0.0;
    int32_t n = nb;
    for (int32_t m = 0; EQ ? (n > 1) : (m < nb - M); ++m) {
        double wi, wj;
        int32_t qi, qj;
        Q.pop(&wi, &qi);
        Q.pop(&wj, &qj);
        const double sum = wi + wj;
        if (EQ) {
            // the two just taken stay live (their weights are untouched)
            const bool go = eq ? (sum <= ideal || need > M) : (n > M);
            if (!go) break;
            if (eq)
                need = need - need_copies(wi, two_ideal) - need_copies(wj, two_ideal) +
                       need_copies(sum, two_ideal);
        }
        if ((m & 63) == 0) {   // the next 64 merge draws, one per lane
            const U4 rr = philox4x32_10((uint32_t)(m + lane), (uint32_t)b, iter, 1u, k0, k1);
            ul = uniform53(rr.x, rr.y);
        }
        const double u = rs_readlane(ul, m & 63);
        const double p_i = wi / sum;
        const int32_t keep = (u < p_i) ? qi : qj;
        const int32_t drop = (keep == qi) ? qj : qi;
        if (lane == 0) {
            W[keep] = sum;
            W[drop] = -1.0;
        }
        wave_sync();
        Q.push(sum, keep);
        n -= 1;
    }
    wave_sync();
    if (EQ) {
        split_survivors(wk, p0, nb, n, M, b, o0, out, lane);
        return;
    }

    const int32_t kq = (nb + 63) >> 6;
    const int32_t q_lo = min(lane * kq, nb), q_hi = min(q_lo + kq, nb);
    int32_t cl = 0;
    for (int32_t q = q_lo; q < q_hi; ++q) cl += (W[q] >= 0.0) ? 1 : 0;
    int32_t tot;
    int32_t o = o0 + wave_excl_scan(cl, &tot);
    for (int32_t q = q_lo; q < q_hi; ++q) {
        const double wq = W[q];
        if (!(wq >= 0.0)) continue;
        out.orig[o] = wk.list[p0 + q];
        out.wn[o] = wq;
        out.obin[o] = b;
        ++o;
    }
}

// n > M for larger bins: the same merges, many at a time.  A is the bin sorted
// by (weight, slot), B the merged walkers in the order they are made, sorted
// the same way (their weights never decrease).  With s the sum of the two
// lightest walkers, every merge made from here on weighs at least s, so all
// walkers lighter than s are merged in pairs in their order before any of the
// new ones: a round takes up to 64 from the front of A and of B, ranks them
// together, and merges pairs side by side, one per lane, each with its own
// Philox draw (merge number m0 + pair).  A round of one pair (always valid)
// is the serial step.  Serial merging is a chain of wave minima or dependent
// loads per merge: the 64-network batch's resample, which waits for its bins of
// 512 walkers, 392 us that way and 158 in rounds (placement included).  A round
// costs about two serial merges, and where weights span many decades it may hold
// one pair, so the count-only rule takes rounds past 256 walkers only (16 toggle
// runs of 64 bins x 16: 10.2 us serial, 16.4 in rounds from 12 merges on); the
// weight-equalizing rule, which merges on while two weights are far below the
// ideal, from 65 (see equalize_bin_rounds).
// CAP: the most walkers the wave's LDS holds (0: none), a multiple of 8.
#define MERGE_ROUNDS_MAX 2048
struct MergeLds {
    double *aw, *bw, *cw;      // [n] sorted weights, [n] merged weights, [128] a round's walkers
    uint16_t *aq, *bq, *cq;    // their slots in the bin
};
template <int CAP>
__host__ __device__ constexpr size_t merge_lds_bytes() {
    return CAP ? (size_t)CAP * 2 * (sizeof(double) + sizeof(uint16_t)) + 128 * (sizeof(double) + sizeof(uint16_t)) : 0;
}
template <int CAP>
__device__ __forceinline__ MergeLds merge_lds(unsigned char *p) {
    MergeLds l;
    l.aw = reinterpret_cast<double *>(p);
    l.bw = l.aw + CAP;
    l.cw = l.bw + CAP;
    l.aq = reinterpret_cast<uint16_t *>(l.cw + 128);
    l.bq = l.aq + CAP;
    l.cq = l.bq + CAP;
    return l;
}

__device__ __forceinline__ bool lighter(double w0, int32_t q0, double w1, int32_t q1) {
    return w0 < w1 || (w0 == w1 && q0 < q1);
}

// B[t0, t) was appended to B[h, t0): puts every run of equal weights that has
// an appended walker into slot order.  Odd-even transposition, as long as
// something moves: runs are short unless many weights are equal.
__device__ __forceinline__ void sort_ties(const MergeLds &l, int32_t h, int32_t t0, int32_t t, int lane) {
    int32_t lo = t0;                          // the run that reaches back starts here
    const double w0 = l.bw[t0];
    while (lo > h && l.bw[lo - 1] == w0) --lo;
    for (int32_t still = 0, odd = 0; still < 2; odd ^= 1) {
        bool moved = false;
        for (int32_t c0 = lo + odd; c0 + 1 < t; c0 += 128) {
            const int32_t i = c0 + 2 * lane;
            if (i + 1 < t) {
                const int32_t q0 = l.bq[i], q1 = l.bq[i + 1];
                if (l.bw[i] == l.bw[i + 1] && q1 < q0) {
                    l.bq[i] = (uint16_t)q1;
                    l.bq[i + 1] = (uint16_t)q0;
                    moved = true;
                }
            }
        }
        still = __ballot(moved) ? 0 : still + 1;
        wave_sync();
    }
}

// EQ: the weight-equalizing rule's merges (equalize_bin_lanes' condition; how many
// of a round's pairs it lets through is a scan over what each changes `need` by).
// W ends with the survivors' weights, merged-away walkers -1; -> survivors.
template <bool EQ, int CAP>
__device__ __forceinline__ int32_t merge_rounds(double *W, int32_t nb, int32_t M, int32_t b, uint32_t iter, uint32_t k0, uint32_t k1,
                                const MergeLds &l, int lane) {
    for (int32_t q = lane; q < nb; q += 64) {
        l.aw[q] = W[q];
        l.aq[q] = (uint16_t)q;
    }
    wave_sync();
    bool eq = false;
    double ideal = 0.0, two_ideal = 0.0;
    int32_t need = 0;
    if constexpr (EQ) {
        double Wb = 0.0;                  // the bin's weight, in slot order
#pragma unroll 8
        for (int32_t q = 0; q < nb; ++q) Wb = Wb + l.aw[q];
        eq = Wb > 0.0;
        ideal = Wb / (double)M;
        two_ideal = ideal + ideal;
        if (eq)
            for (int32_t q = lane; q < nb; q += 64) need += need_copies(l.aw[q], two_ideal);
        need = wave_sum_i32(need);
    }
    int32_t n = nb;
    // bitonic network; mirrored first steps make positions past nb act as +inf.
    // AHEAD pairs of a lane are read before the first is written: the largest bins
    // of a 64-network batch (700 walkers) 123 -> 111 us, ten futile-cycle runs of
    // 101 bins x 100 38 -> 35.6.  A wave alone on its SIMD, it is bound by issue now.
    constexpr int AHEAD = CAP >= 1024 ? 8 : CAP >= 512 ? 4 : 2;
    int32_t P = 1;
    while (P < nb) P <<= 1;
    for (int32_t size = 2; size <= P; size <<= 1)
        for (int32_t d = size >> 1; d > 0; d >>= 1) {
            const bool mirror = d == (size >> 1);
            for (int32_t c0 = 0; c0 < (P >> 1); c0 += 64 * AHEAD) {
                double wi[AHEAD], wj[AHEAD];
                int32_t qi[AHEAD], qj[AHEAD], at[AHEAD], to[AHEAD];
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    const int32_t c = c0 + 64 * u + lane;
                    const int32_t r = c & (d - 1), base = (c - r) << 1;
                    at[u] = base + r;
                    to[u] = mirror ? base + 2 * d - 1 - r : base + r + d;
                    if (to[u] >= nb) at[u] = to[u] = nb - 1;   // nothing to exchange with
                    wi[u] = l.aw[at[u]];
                    wj[u] = l.aw[to[u]];
                    qi[u] = l.aq[at[u]];
                    qj[u] = l.aq[to[u]];
                }
#pragma unroll
                for (int u = 0; u < AHEAD; ++u)
                    if (lighter(wj[u], qj[u], wi[u], qi[u])) {
                        l.aw[at[u]] = wj[u];
                        l.aw[to[u]] = wi[u];
                        l.aq[at[u]] = (uint16_t)qj[u];
                        l.aq[to[u]] = (uint16_t)qi[u];
                    }
            }
            wave_sync();
        }
    const double inf = __builtin_huge_val();
    int32_t ha = 0, hb = 0, t = 0;          // fronts of A and B, end of B
    int32_t m0 = 0;                          // merges made
    while (EQ ? n > 1 : n > M) {
        // up to 64 walkers from the front of each
        const int32_t ia = ha + lane, ib = hb + lane;
        const double wa = ia < nb ? l.aw[ia] : inf, wb = ib < t ? l.bw[ib] : inf;
        const int32_t qa = ia < nb ? (int32_t)l.aq[ia] : 0, qb = ib < t ? (int32_t)l.bq[ib] : 0;
        // the two lightest: among the first two of each, as sums of sorted heads
        const double a0 = rs_readlane(wa, 0), a1 = rs_readlane(wa, 1), b0 = rs_readlane(wb, 0), b1 = rs_readlane(wb, 1);
        const double s = fmin(fmin(a0 + a1, b0 + b1), a0 + b0);
        int32_t na = (int32_t)__popcll(__ballot(wa < s)), nbm = (int32_t)__popcll(__ballot(wb < s));
        if (na + nbm < 2) {                  // zero weights, or a pair that rounds to its heavier walker
            na = min(2, nb - ha);
            nbm = min(2, t - hb);
        }
        // rank each walker among the na + nbm taken: walk the shorter list
        int32_t ra = lane, rb = lane;
        if (na <= nbm) {
            for (int32_t j = 0; j < na; ++j) {
                const bool less = lane < nbm && lighter(wb, qb, rs_readlane(wa, j), __builtin_amdgcn_readlane(qa, j));
                const int32_t r = (int32_t)__popcll(__ballot(less));
                if (lane == j) ra += r;
                if (!less) rb += 1;
            }
        } else {
            for (int32_t j = 0; j < nbm; ++j) {
                const bool less = lane < na && lighter(wa, qa, rs_readlane(wb, j), __builtin_amdgcn_readlane(qb, j));
                const int32_t r = (int32_t)__popcll(__ballot(less));
                if (lane == j) rb += r;
                if (!less) ra += 1;
            }
        }
        if (lane < na) {
            l.cw[ra] = wa;
            l.cq[ra] = (uint16_t)qa;
        }
        if (lane < nbm) {
            l.cw[rb] = wb;
            l.cq[rb] = (uint16_t)qb;
        }
        wave_sync();
        // all below s: as many pairs as there are; else (the first two of each
        // list, ranked) only the first pair is certain
        const bool all = __ballot((lane < na && !(wa < s)) || (lane < nbm && !(wb < s))) == 0ull;
        // and none past the last one of a full window: further ones of that list
        // may come before those of the other
        int32_t sure = na + nbm;
        if (na == 64 && ha + 64 < nb) sure = min(sure, __builtin_amdgcn_readlane(ra, 63) + 1);
        if (nbm == 64 && hb + 64 < t) sure = min(sure, __builtin_amdgcn_readlane(rb, 63) + 1);
        int32_t pairs = min(all ? sure >> 1 : 1, EQ ? n - 1 : n - M);
        const int32_t offered = pairs;
        double wi = 0.0, wj = 0.0, sum = 0.0;
        if (lane < offered) {
            wi = l.cw[2 * lane];
            wj = l.cw[2 * lane + 1];
            sum = wi + wj;
        }
        if constexpr (EQ) {
            int32_t more = 0, tot;        // what the lane's merge adds to need
            if (eq && lane < offered)
                more = need_copies(sum, two_ideal) - need_copies(wi, two_ideal) - need_copies(wj, two_ideal);
            const int32_t at = need + wave_excl_scan(more, &tot);
            const bool go = eq ? (sum <= ideal || at > M) : (n - lane > M);
            const unsigned long long stop = __ballot(lane < offered && !go);
            if (stop) pairs = __ffsll((long long)stop) - 1;
            need = pairs < offered ? __builtin_amdgcn_readlane(at, pairs) : need + tot;
        }
        int32_t keep = 0;
        if (lane < pairs) {
            const int32_t qi = l.cq[2 * lane], qj = l.cq[2 * lane + 1];
            const U4 rr = philox4x32_10((uint32_t)(m0 + lane), (uint32_t)b, iter, 1u, k0, k1);
            const double u = uniform53(rr.x, rr.y);
            const double p_i = wi / sum;
            keep = (u < p_i) ? qi : qj;
            W[keep] = sum;
            W[keep == qi ? qj : qi] = -1.0;
        }
        n -= pairs;
        if (EQ && pairs < offered) break;
        // consumed: the walkers of rank below 2 pairs
        ha += (int32_t)__popcll(__ballot(lane < na && ra < 2 * pairs));
        hb += (int32_t)__popcll(__ballot(lane < nbm && rb < 2 * pairs));
        // the new walkers behind B, sorted by weight; runs of equal weights
        // (which may reach back into B) are put into slot order
        if (lane < pairs) {
            l.bw[t + lane] = sum;
            l.bq[t + lane] = (uint16_t)keep;
        }
        wave_sync();
        const int32_t t0 = t;
        t += pairs;
        const bool tie = lane < pairs && t0 + lane > hb && l.bw[t0 + lane - 1] == sum;
        if (__ballot(tie)) sort_ties(l, hb, t0, t, lane);
        m0 += pairs;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    wave_sync();
    return n;
}

template <int CAP>
__device__ __forceinline__ void merge_bin_rounds(const RunWork<int32_t> &wk, int32_t p0, int32_t nb, int32_t M, int32_t b, int32_t o0,
                                 const BinOut &out, uint32_t iter, uint32_t k0, uint32_t k1, unsigned char *lds,
                                 int lane) {
    const double *W = wk.w + p0;
    merge_rounds<false, CAP>(wk.w + p0, nb, M, b, iter, k0, k1, merge_lds<CAP>(lds), lane);
    // survivors in slot order
    int32_t o = o0;
    for (int32_t c0 = 0; c0 < nb; c0 += 64) {
        const int32_t q = c0 + lane;
        const double wq = q < nb ? W[q] : -1.0;
        const bool live = wq >= 0.0;
        int32_t tot;
        const int32_t ok = o + wave_excl_scan(live ? 1 : 0, &tot);
        if (live) {
            out.orig[ok] = wk.list[p0 + q];
            out.wn[ok] = wq;
            out.obin[ok] = b;
        }
        o += tot;
    }
}

// equalize_bin_lanes with its merges in rounds.  Ten futile-cycle runs of 101 bins
// x 100 walkers wait for one bin of 190 walkers and 138 merges: 85 us merged one
// by one, 35.6 in rounds.
template <int K, int CAP>
__device__ __forceinline__ void equalize_bin_rounds(const RunWork<int32_t> &wk, int32_t p0, int32_t nb, int32_t M,
                                                    int32_t b, int32_t o0, const BinOut &out, uint32_t iter,
                                                    uint32_t k0, uint32_t k1, unsigned char *lds, int lane) {
    const int32_t n = merge_rounds<true, CAP>(wk.w + p0, nb, M, b, iter, k0, k1, merge_lds<CAP>(lds), lane);
    double wv[K];
    bool live[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        wv[k] = 64 * k + lane < nb ? wk.w[p0 + 64 * k + lane] : -1.0;
        live[k] = wv[k] >= 0.0;
    }
    hand_out<K>(wk, p0, M, b, o0, out, wv, live, n, lane);
}

}  // namespace

// One bin's split/merge (and its row of the reweighting flux matrix) on the
// calling wave: the walkers at positions [p0, p0 + nb) of wk, the output at
// slots [o0, o0 + M).  RULE: the sim's rs_rule (-1: read from a).  CAP: walkers
// the wave's LDS lds holds for merges in rounds (bins_cap).  With 512 or more the
// bins to split or equalize in registers reach 512 walkers, eight per lane (more
// than a 1024-thread workgroup has room for; else 128 and 256).
template <class Idx, int RULE, int CAP>
__device__ void resample_bin(const SimArgs &a, const RunWork<Idx> &wk, const BinOut &out, int32_t run, int32_t b,
                             int32_t nb, int32_t p0, int32_t o0, uint32_t iter, uint32_t k0, uint32_t k1,
                             bool rw_acc, int lane, unsigned char *lds = nullptr) {
    constexpr bool BIG = CAP >= 512;
    const int32_t NB = a.n_bins, M = a.m_targ;
    if (rw_acc) rw_flux_bin(a.rw_F + ((size_t)run * NB + b) * NB, wk, p0, nb, NB > 1 ? 32 - __clz(NB - 1) : 0, lane);
    if (RULE < 0 ? a.rs_rule == 1 : RULE == 1) {
        if (nb <= 64) equalize_bin_lanes<1>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
        else if constexpr (CAP > 0) {
            if (nb <= 128) equalize_bin_rounds<2, CAP>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lds, lane);
            else if (nb <= 256) equalize_bin_rounds<4, CAP>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lds, lane);
            else if (BIG && nb <= 512) equalize_bin_rounds<8, CAP>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lds, lane);
            else merge_bin<Idx, true>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
        }
        else if (nb <= 128) equalize_bin_lanes<2>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
        else if (nb <= 256) equalize_bin_lanes<4>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
        else merge_bin<Idx, true>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
    } else if (nb == M) {
        for (int32_t q = lane; q < nb; q += 64) {
            out.orig[o0 + q] = wk.list[p0 + q];
            out.wn[o0 + q] = wk.w[p0 + q];
            out.obin[o0 + q] = b;
        }
    } else if (nb < M) {
        if (nb <= 64) split_bin_lanes<1>(wk, p0, nb, M, b, o0, out, lane);
        else if (nb <= 128) split_bin_lanes<2>(wk, p0, nb, M, b, o0, out, lane);
        else if (BIG && nb <= 256) split_bin_lanes<4>(wk, p0, nb, M, b, o0, out, lane);
        else if (BIG && nb <= 512) split_bin_lanes<8>(wk, p0, nb, M, b, o0, out, lane);
        else split_bin(wk, p0, nb, M, b, o0, out, lane);
    } else {
        if (nb <= 64) merge_bin_lanes<1>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
        else if (nb <= 128) merge_bin_lanes<2>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
        else if (nb <= 256) merge_bin_lanes<4>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
        else if (BIG && nb <= CAP) {
            if constexpr (BIG) merge_bin_rounds<CAP>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lds, lane);
        }
        else merge_bin<Idx, false>(wk, p0, nb, M, b, o0, out, iter, k0, k1, lane);
    }
}

// The run's working arrays in device memory (see resample_run_t).
__device__ __forceinline__ RunWork<int32_t> global_work(const SimArgs &a, size_t base) {
    RunWork<int32_t> wk;
    wk.w = a.s_w + base;
    wk.list = a.s_list + base;
    wk.tag = reinterpret_cast<uint16_t *>(a.s_cnt + base);
    wk.qa = a.s_bin + base;
    wk.aux = a.s_cnt + base;
    return wk;
}

// LDS: the run's working arrays in LDS (Idx uint16), else in device memory
// (Idx int32).  PLACE (device arrays only): stop after placement and staging,
// and leave each bin's count, first position and first output slot in
// binfo[run][3][n_bins] for we_resample_bins_kernel.
// x_cur (LDS, at most one walker per thread; null: already done): recycle and bin
// the run's walkers first.
template <class Idx, bool LDS, int RULE, bool PLACE>
__device__ void resample_run_t(const SimArgs &a, int32_t *__restrict__ x_cur, const double *__restrict__ w_cur,
                               double *__restrict__ w_nxt, int32_t run, unsigned char *lds,
                               int32_t *__restrict__ binfo) {
    const int32_t tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, n_waves = nthr >> 6;
    const int32_t NB = a.n_bins, M = a.m_targ, cap = a.cap;
    __shared__ int64_t ev_part[RESAMPLE_THREADS];
    // once the event totals are read: recycled weights to add, then the
    // recycled walkers per cursor row
    double *next_w = reinterpret_cast<double *>(ev_part);
    int32_t *rec_row = reinterpret_cast<int32_t *>(ev_part + RESAMPLE_THREADS / 2);
    int32_t *cnt = reinterpret_cast<int32_t *>(lds);   // [NB]
    int32_t *start = cnt + NB;                          // [NB+1]
    int32_t *ostart = start + NB + 1;                   // [NB+1]
    // walkers are placed by P waves at once, wave r over its own contiguous
    // run of 64-slot chunks; row r of the cursor table first counts, per bin,
    // the walkers of those chunks, then holds where the next one goes
    const int32_t P = max(1, min(n_waves, a.place_rows));
    int32_t *cursor = ostart + NB + 1;                  // [a.place_rows][NB]
    int32_t *after = cursor + (size_t)max(1, a.place_rows) * NB;
    const bool evb_shared = !LDS && NB > RESAMPLE_EVB_BINS;
    float *evb = reinterpret_cast<float *>(evb_shared ? ostart : after);   // [NB] events per bin
    unsigned char *tail = reinterpret_cast<unsigned char *>(after + NB);    // LDS: the working arrays
    tail += (16 - ((uintptr_t)tail & 15)) & 15;

    const uint32_t iter = *a.iter_dev;
    const int32_t rec_slot = (int32_t)iter;
    const int32_t n = a.n_walk[run];
    const size_t base = (size_t)run * cap;
    const double *wr = w_cur + base;
    double *rec_w = w_nxt + base;   // until the new weights are written: each row's recycled weights, side by side
    const int32_t *sbin = a.s_bin + base;
    const int32_t *srec = a.s_rec + base;
    RunWork<Idx> wk;
    if constexpr (LDS) {
        wk.w = reinterpret_cast<double *>(tail);
        wk.list = reinterpret_cast<int32_t *>(wk.w + cap);
        wk.tag = reinterpret_cast<uint16_t *>(wk.list + cap);
        wk.qa = reinterpret_cast<Idx *>(wk.tag);
        wk.aux = reinterpret_cast<Idx *>(wk.tag + cap);
    } else {
        // global: the tag array in the first half of the s_cnt rows, the
        // queue over s_bin (read only before the first barrier), the aux
        // array over s_cnt once placement is done
        const RunWork<int32_t> g = global_work(a, base);
        wk.w = g.w;
        wk.list = g.list;
        wk.tag = g.tag;
        wk.qa = reinterpret_cast<Idx *>(g.qa);
        wk.aux = reinterpret_cast<Idx *>(g.aux);
    }

    const int32_t n_chunks = (n + 63) >> 6;
    const int32_t per_row = max(1, (n_chunks + P - 1) / P) * 64;   // slots per row
    for (int32_t b = tid; b < NB; b += nthr) {
        cnt[b] = 0;
        evb[b] = 0.0f;
    }
    for (int32_t i = tid; i < P * NB; i += nthr) cursor[i] = 0;
    if constexpr (LDS)
        if (x_cur && tid < n) recycle_bin_one(a, x_cur, 1, (int64_t)run * cap + tid);   // counted by this thread below
    __syncthreads();
    // counts per bin and per cursor row: each wave takes 64 consecutive slots
    // (one cursor row: per_row is a multiple of 64), four such chunks' loads at a
    // time, and one lane of each bin adds the bin's lanes
    const int bits = NB > 1 ? 32 - __clz(NB - 1) : 0;
    int64_t my_ev = 0;
    for (int32_t c4 = wave * 64; c4 < n; c4 += 4 * nthr) {
        int32_t bs[4], rs[4];
        uint32_t evs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c4 + u * nthr < n) {
                const int32_t k = min(c4 + u * nthr + lane, n - 1);
                bs[u] = sbin[k];
                evs[u] = a.ev_walker[base + k];
                rs[u] = srec[k];
            }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t c0 = c4 + u * nthr, k = c0 + lane, b = bs[u];
            if (c0 >= n) break;
            const bool valid = k < n, rc = valid && rs[u] != 0;
            const unsigned long long grp = match_lanes(b, valid, bits);
            if (valid) {
                wk.tag[k] = (uint16_t)(b | (rc ? 0x8000 : 0));
                my_ev += evs[u];
                if (lanes_below(grp) == 0) {
                    atomicAdd(&cnt[b], (int32_t)__popcll(grp));
                    atomicAdd(&cursor[c0 / per_row * NB + b], (int32_t)__popcll(grp));
                }
            }
            if (a.queue_stats) add_by_bin(evb, valid ? b : -1, (float)evs[u], lane);
        }
    }
    ev_part[tid] = my_ev;
    __syncthreads();
    // per-bin event statistics for the propagation kernels' work queue (a
    // scheduling hint only: no result depends on it)
    if (a.queue_stats)
        for (int32_t b = tid; b < NB; b += nthr)
            if (cnt[b] > 0) {
                const int32_t c = run % a.seg_rep * NB + b;
                atomicAdd(&a.ev_bin[c], evb[b]);
                atomicAdd(&a.n_bin[c], cnt[b]);
            }
    if (evb_shared) __syncthreads();

    // wave 0: bin offsets (walkers ordered by bin, then slot)
    if (wave == 0) {
        const int32_t kb = (NB + 63) >> 6;
        const int32_t b_lo = min(lane * kb, NB), b_hi = min(b_lo + kb, NB);
        int32_t acc = 0, oacc = 0;
        for (int32_t b = b_lo; b < b_hi; ++b) {
            acc += cnt[b];
            oacc += cnt[b] > 0 ? M : 0;
        }
        int32_t tot, otot;
        acc = wave_excl_scan(acc, &tot);
        oacc = wave_excl_scan(oacc, &otot);
        for (int32_t b = b_lo; b < b_hi; ++b) {
            start[b] = acc;
            ostart[b] = oacc;
            acc += cnt[b];
            oacc += cnt[b] > 0 ? M : 0;
        }
        if (lane == 63) {
            start[NB] = tot;
            ostart[NB] = otot;
        }
    }
    // the last wave: reactions fired
    if (wave == n_waves - 1) {
        int64_t ev = 0;
        for (int32_t t = lane; t < nthr; t += 64) ev += ev_part[t];
        for (int d = 32; d > 0; d >>= 1) ev += __shfl_xor(ev, d, 64);
        if (lane == 0 && rec_slot < a.max_iters) {
            a.ev_iter[(size_t)run * a.max_iters + rec_slot] = ev;
            a.seg_iter[(size_t)run * a.max_iters + rec_slot] = n;
        }
    }
    __syncthreads();
    // row r's count of bin b becomes the position of its first walker of b
    for (int32_t b = tid; b < NB; b += nthr) {
        int32_t c = start[b];
        for (int32_t r = 0; r < P; ++r) {
            const int32_t t = cursor[r * NB + b];
            cursor[r * NB + b] = c;
            c += t;
        }
    }
    __syncthreads();

    // stable placement: waves r < P, each over its chunks in slot order; a
    // lane's place is its bin's cursor plus its rank among the bin's lanes, and
    // the cursor advances by their number.  The lanes of every bin are found at
    // once, one ballot per bit of the bin's number (a chunk holds tens of bins
    // where bins are small).  Each row also sets its recycled walkers' weights
    // side by side, for the sum below.  With a ballot per bin present, and the
    // recycled weights looked for by one wave alone, the placement took 76 us for
    // 64 runs of 465 bins x 16 walkers, 18 us for 32 runs of 80 x 32 and 11.4 us
    // for 16 of 64 x 16; this form takes 23.6, 10.6 and 8.3.
    if (wave < P) {
        int32_t *cur = cursor + wave * NB;
        const int32_t k_lo = wave * per_row, k_hi = min(n, k_lo + per_row);
        int32_t tag = k_lo + lane < k_hi ? (int32_t)wk.tag[k_lo + lane] : 0;
        int32_t n_rec = 0;
        for (int32_t c0 = k_lo; c0 < k_hi; c0 += 64) {
            const int32_t k = c0 + lane;
            const bool valid = k < k_hi;
            const int32_t b = tag & 0x7FFF;
            const bool rec = valid && (tag & 0x8000);
            const unsigned long long rm = __ballot(rec);
            if (rec) rec_w[k_lo + n_rec + lanes_below(rm)] = wr[k];
            n_rec += (int32_t)__popcll(rm);
            if (k + 64 < k_hi) tag = (int32_t)wk.tag[k + 64];
            const unsigned long long grp = match_lanes(b, valid, bits);
            if (valid) {
                const int32_t at = cur[b], rank = lanes_below(grp);
                wk.list[at + rank] = k;
                if (rank == 0) cur[b] = at + (int32_t)__popcll(grp);
            }
            wave_sync();
        }
        if (lane == 0) rec_row[wave] = n_rec;
    }
    __syncthreads();
    // the last wave: the recycled weight, summed in slot order: rows in order,
    // up to 512 weights at a time fetched into LDS
    if (wave == n_waves - 1) {
        double f = 0.0;
        int32_t rec_tot;
        const int32_t rec_lo = wave_excl_scan(lane < P ? rec_row[lane] : 0, &rec_tot);
        for (int32_t j0 = 0; j0 < rec_tot; j0 += 512) {
            const int32_t m = min(512, rec_tot - j0);
            double wv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (64 * u >= m) break;
                const int32_t j = min(j0 + 64 * u + lane, rec_tot - 1);
                int32_t at = j;   // row r's weights start at r * per_row
                for (int32_t q = 1; q < P; ++q) {
                    const int32_t lo = __builtin_amdgcn_readlane(rec_lo, q);
                    at = j >= lo ? q * per_row + (j - lo) : at;
                }
                wv[u] = rec_w[at];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (64 * u >= m) break;
                next_w[64 * u + lane] = wv[u];
            }
            wave_sync();
#pragma unroll 8
            for (int32_t i = 0; i < m; ++i) f = f + next_w[i];
            wave_sync();
        }
        if (lane == 0 && rec_slot < a.max_iters) {
            a.flux[(size_t)run * a.max_iters + rec_slot] = f;
        }
    }
    // the weights in bin-major order.  One that is infinite or not a number (sums
    // that overflowed, a reweighting of rates past the range) is a fault, and goes on
    // as 0: the hand-out of copies ends by comparing shares, and the rounds rank
    // walkers by them.
    // flux matrix of reweighting: from the second interval on (the first
    // one's walkers carry no bin yet); the start bins go to aux, which only
    // the split/merge of the same bin uses afterwards
    const bool rw_acc = a.rw_F != nullptr && iter >= 1u;
    for (int32_t p4 = tid; p4 < n; p4 += 4 * nthr) {
        int32_t ks[4], from[4] = {0, 0, 0, 0};
        double ws[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) ks[u] = wk.list[min(p4 + u * nthr, n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ws[u] = wr[ks[u]];
            if (rw_acc) from[u] = a.bin[base + ks[u]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t p = p4 + u * nthr;
            if (p < n) {
                const bool finite = ws[u] < __builtin_huge_val();
                if (!finite) atomicOr(a.err, WE_DERR_WEIGHT);
                wk.w[p] = finite ? ws[u] : 0.0;
                if (rw_acc) wk.aux[p] = (Idx)from[u];
            }
        }
    }
    __syncthreads();

    if constexpr (PLACE) {
        // bin-parallel mode: leave the bins to we_resample_bins_kernel
        int32_t *bi = binfo + (size_t)run * 3 * NB;
        for (int32_t b = tid; b < NB; b += nthr) {
            bi[b] = cnt[b];
            bi[NB + b] = start[b];
            bi[2 * NB + b] = ostart[b];
        }
        if (tid == 0) a.n_walk[run] = ostart[NB];
        return;
    }

    // split / merge: one wave per bin
    const uint64_t seed = a.seeds[run];
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    BinOut out;
    out.orig = a.origin + base;
    out.obin = a.bin + base;
    out.wn = w_nxt + base;
    for (int32_t b = wave; b < NB; b += n_waves) {
        const int32_t nb = uni(cnt[b]);
        if (nb == 0) continue;
        resample_bin<Idx, RULE, 0>(a, wk, out, run, b, nb, uni(start[b]), uni(ostart[b]), iter, k0, k1, rw_acc, lane);
    }
    __syncthreads();
    if (tid == 0) a.n_walk[run] = ostart[NB];
}

// How a run's workgroup resamples: whole, with its working arrays in LDS or in
// device memory, or placement only (bin-parallel mode).  One kernel per mode
// and rule: with every path in one, the compiler called the split/merge
// routines through a stack (784 B of scratch a lane) instead of inlining them.
enum ResampleMode { RS_LDS, RS_GLOBAL, RS_PLACE };

template <int MODE, int RULE>
__global__ __launch_bounds__(RESAMPLE_THREADS) void we_resample_kernel(SimArgs a, int32_t *__restrict__ x_cur, const double *__restrict__ w_cur,
                                                          double *__restrict__ w_nxt, int32_t *__restrict__ binfo) {
    extern __shared__ __align__(16) unsigned char lds[];
    if constexpr (MODE == RS_LDS) resample_run_t<uint16_t, true, RULE, false>(a, x_cur, w_cur, w_nxt, blockIdx.x, lds, nullptr);
    else resample_run_t<int32_t, false, RULE, MODE == RS_PLACE>(a, x_cur, w_cur, w_nxt, blockIdx.x, lds, binfo);
}

// Bin-parallel split/merge after we_resample_kernel's placement: grid
// (bins_blocks, runs), one wave per bin, the same per-bin steps on the
// run's arrays in device memory; bins of one run write disjoint ranges.
template <int RULE, int CAP>
__device__ __forceinline__ void resample_bins_wave(const SimArgs &a, double *__restrict__ w_nxt,
                                                   const int32_t *__restrict__ binfo, int32_t run, int32_t b,
                                                   unsigned char *mlds) {
    const int lane = threadIdx.x & 63;
    const int32_t NB = a.n_bins;
    if (b >= NB) return;                       // uniform over the wave
    const int32_t *bi = binfo + (size_t)run * 3 * NB;
    const int32_t nb = uni(bi[b]);
    if (nb == 0) return;
    const size_t base = (size_t)run * a.cap;
    const RunWork<int32_t> wk = global_work(a, base);
    BinOut out;
    out.orig = a.origin + base;
    out.obin = a.bin + base;
    out.wn = w_nxt + base;
    const uint32_t iter = *a.iter_dev;
    const uint64_t seed = a.seeds[run];
    resample_bin<int32_t, RULE, CAP>(a, wk, out, run, b, nb, uni(bi[NB + b]), uni(bi[2 * NB + b]), iter, (uint32_t)seed,
                                     (uint32_t)(seed >> 32), a.rw_F != nullptr && iter >= 1u, lane, mlds);
}

// Waves (bins) per workgroup: one where its LDS alone would keep others off the CU.
template <int CAP>
struct BinsBlock {
    static constexpr int WAVES = CAP >= 1024 ? 1 : 4;
    static constexpr size_t LDS = WAVES * merge_lds_bytes<CAP>();
};

// Workgroups per run.
template <int CAP>
__host__ __device__ constexpr int32_t bins_blocks(int32_t n_bins) {
    return (n_bins + BinsBlock<CAP>::WAVES - 1) / BinsBlock<CAP>::WAVES;
}

template <int RULE, int CAP>
__global__ __launch_bounds__(64 * BinsBlock<CAP>::WAVES) void we_resample_bins_kernel(SimArgs a, double *__restrict__ w_nxt,
                                                                                    const int32_t *__restrict__ binfo) {
    extern __shared__ __align__(16) unsigned char mlds[];
    const int32_t wave = (int32_t)(threadIdx.x >> 6);
    resample_bins_wave<RULE, CAP>(a, w_nxt, binfo, blockIdx.y, (int32_t)blockIdx.x * BinsBlock<CAP>::WAVES + wave,
                                  mlds + wave * merge_lds_bytes<CAP>());
}

template <int RULE, int CAP>
void launch_bins(const SimArgs &a, double *w_nxt, const int32_t *binfo, hipStream_t st) {
    hipLaunchKernelGGL((we_resample_bins_kernel<RULE, CAP>), dim3((unsigned)bins_blocks<CAP>(a.n_bins), (unsigned)a.n_runs),
                       dim3(64 * BinsBlock<CAP>::WAVES), BinsBlock<CAP>::LDS, st, a, w_nxt, binfo);
}

// New state rows from their parents: one lane per copy number.
__device__ __forceinline__ void gather_one(const SimArgs &a, const int32_t *__restrict__ x_cur,
                                           int32_t *__restrict__ x_nxt, int64_t gid) {
    const int64_t per_run = (int64_t)a.cap * a.S;
    const int32_t run = (int32_t)(gid / per_run);
    if (run >= a.n_runs) return;
    const int64_t rem = gid - (int64_t)run * per_run;
    const int32_t dst = (int32_t)(rem / a.S);
    const int32_t s = (int32_t)(rem - (int64_t)dst * a.S);
    if (dst >= a.n_walk[run]) return;
    const size_t base = (size_t)run * a.cap;
    const int32_t src = a.origin[base + dst];
    x_nxt[(base + dst) * a.S + s] = x_cur[(base + src) * a.S + s];
}

// The same with 32-bit index arithmetic, for sims whose n_runs * cap * S
// copy numbers stay below 2^31: a 64-bit division by a runtime divisor is a
// long instruction sequence, a 32-bit one a short one.
__device__ __forceinline__ void gather_one32(const SimArgs &a, const int32_t *__restrict__ x_cur,
                                             int32_t *__restrict__ x_nxt, uint32_t gid) {
    const uint32_t S = (uint32_t)a.S, per_run = (uint32_t)a.cap * S;
    const uint32_t run = gid / per_run;
    if (run >= (uint32_t)a.n_runs) return;
    const uint32_t rem = gid - run * per_run;
    const uint32_t dst = rem / S;
    const uint32_t s = rem - dst * S;
    if ((int32_t)dst >= a.n_walk[run]) return;
    const uint32_t base = run * (uint32_t)a.cap;
    const uint32_t src = (uint32_t)a.origin[base + dst];
    x_nxt[(base + dst) * S + s] = x_cur[(base + src) * S + s];
}

__global__ __launch_bounds__(256) void we_gather_rows_kernel(SimArgs a, const int32_t *__restrict__ x_cur,
                                                             int32_t *__restrict__ x_nxt, int32_t narrow) {
    if (narrow)
        gather_one32(a, x_cur, x_nxt, blockIdx.x * blockDim.x + threadIdx.x);
    else
        gather_one(a, x_cur, x_nxt, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// P(x_s = k, t) accumulated over iterations: one lane per walker, FP64 atomics.
__device__ __forceinline__ void observe_one(const SimArgs &a, const int32_t *__restrict__ xs,
                                            const double *__restrict__ ws, int64_t gid64) {
    const int32_t gid = (int32_t)gid64;
    const int32_t run = gid / a.cap;
    const int32_t k = gid - run * a.cap;
    if (run >= a.n_runs) return;
    if (k >= a.n_walk[run]) return;
    const size_t idx = (size_t)run * a.cap + k;
    const double wv = ws[idx];
    if (a.nh > 0) {
        const int32_t v = xs[idx * a.S + a.hist_species] - a.hist_lo;
        if (v >= 0 && v < a.nh) atomicAdd(&a.hist[(size_t)run * a.nh + v], wv);
    }
    if (a.n_joint > 0) {
        int32_t cell = 0, mul = 1;
        for (int d = 0; d < a.n_joint; ++d) {
            const int32_t c = min(xs[idx * a.S + a.joint_species[d]] / a.joint_width, a.joint_bins - 1);
            cell += c * mul;
            mul *= a.joint_bins;
        }
        atomicAdd(&a.jhist[(size_t)run * a.jcells + cell], wv);
    }
}

__global__ __launch_bounds__(256) void we_observe_kernel(SimArgs a, const int32_t *__restrict__ xs,
                                                         const double *__restrict__ ws) {
    observe_one(a, xs, ws, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// ---------------------------------------------------------------- batched
// The same steps for many sims in one launch each: grid y = sim, per-sim
// arguments and buffer pointers read from device memory.
struct BatchPtrs {
    const SimArgs *args;
    int32_t *const *x_cur;
    int32_t *const *x_nxt;
    const double *const *w_cur;
    double *const *w_nxt;
    int32_t *const *binfo;
    const int32_t *grid_bins;
    const int32_t *bins_cap;
};

// The members' workgroups on one variant of the split/merge: each member's first
// one and their number, and the most blocks of bins that a member has.
struct BatchBins {
    int64_t *first;    // device, [members + 1]
    int64_t total;
    int32_t max_blocks;
};

__global__ __launch_bounds__(256) void we_batch_recycle_bin_kernel(BatchPtrs b) {
    const int32_t i = blockIdx.y;
    recycle_bin_one(b.args[i], b.x_cur[i], b.grid_bins[i], (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Placement by one workgroup per run, then one wave per bin over all members'
// bins: with the split/merge in the run's workgroup, in LDS, the launch lasted
// as long as the largest member's (one run of 16 bins of 512 walkers, whose
// bins were sorted: 392 us for the batch of 64 networks).
__global__ __launch_bounds__(RESAMPLE_THREADS) void we_batch_place_kernel(BatchPtrs b) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int32_t i = blockIdx.y;
    const SimArgs &a = b.args[i];
    if ((int32_t)blockIdx.x >= a.n_runs) return;
    resample_run_t<int32_t, false, 0, true>(a, nullptr, b.w_cur[i], b.w_nxt[i], blockIdx.x, lds, b.binfo[i]);
}

// The members' split/merge, runs side by side: workgroups go to the XCDs in turn, and
// the busy bins of every run are the same few.  EVEN: grid (runs, blocks of bins,
// members), sized for the largest of each.  Else as many workgroups as the members
// on this variant have, which find their member by bisecting the members' first
// workgroups (first[n_sims]: their number).
template <int CAP, bool EVEN>
__global__ __launch_bounds__(64 * BinsBlock<CAP>::WAVES) void we_batch_bins_kernel(BatchPtrs b,
                                                                                  const int64_t *__restrict__ first,
                                                                                  int32_t n_sims) {
    extern __shared__ __align__(16) unsigned char mlds[];
    const int32_t wave = (int32_t)(threadIdx.x >> 6);
    unsigned char *wlds = mlds + wave * merge_lds_bytes<CAP>();
    if constexpr (EVEN) {
        const int32_t i = blockIdx.z;
        const SimArgs &a = b.args[i];
        if ((int32_t)blockIdx.x >= a.n_runs || b.bins_cap[i] != CAP) return;
        resample_bins_wave<-1, CAP>(a, b.w_nxt[i], b.binfo[i], blockIdx.x,
                                    (int32_t)blockIdx.y * BinsBlock<CAP>::WAVES + wave, wlds);
    } else {
        for (int64_t g = blockIdx.x; g < first[n_sims]; g += gridDim.x) {
            int32_t i = 0, end = n_sims;
            while (end - i > 1) {
                const int32_t mid = (i + end) >> 1;
                if (first[mid] <= g) i = mid;
                else end = mid;
            }
            const SimArgs &a = b.args[i];
            const int32_t at = (int32_t)(g - first[i]), block = at / a.n_runs;
            resample_bins_wave<-1, CAP>(a, b.w_nxt[i], b.binfo[i], at - block * a.n_runs,
                                        block * BinsBlock<CAP>::WAVES + wave, wlds);
        }
    }
}

// Grid-strided over each member's own cells: a grid sized for the largest
// member would spend most of its workgroups on members that have no cells
// left for them.
__global__ __launch_bounds__(256) void we_batch_gather_kernel(BatchPtrs b) {
    const int32_t i = blockIdx.y;
    const SimArgs &a = b.args[i];
    const int64_t cells = (int64_t)a.n_runs * a.cap * a.S;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; gid < cells; gid += stride)
        gather_one(a, b.x_cur[i], b.x_nxt[i], gid);
}

__global__ __launch_bounds__(256) void we_batch_observe_kernel(BatchPtrs b) {
    const int32_t i = blockIdx.y;
    const SimArgs &a = b.args[i];
    if (a.nh <= 0 && a.n_joint <= 0) return;
    observe_one(a, b.x_nxt[i], b.w_nxt[i], (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Also clears the propagation's chunk counters for the next iteration.
__global__ void we_batch_advance_kernel(BatchPtrs b, int32_t n, uint32_t *__restrict__ counters, int32_t n_counters) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) *b.args[i].iter_dev += 1u;
    if (i < n_counters) counters[(size_t)i * WE_HEAD_STRIDE] = 0u;
}

// Workgroups per member in the batched gather (each strides over its member's
// cells): 64 members then give 32768 workgroups, 128 per CU.
#define BATCH_GATHER_BLOCKS 512

// The walkers a bin may have for its merges to go in rounds, by the wave's LDS (20
// bytes each; 0: none).  Targets of at most 128 leave few bins past 256.  Above,
// room for 2048 pays as long as the waves are few: it leaves three to a CU, and
// with more waves than that the bins wait for one another, so the room is then what
// the target's bins need, and none where they are past the rounds (512 for the
// weight-equalizing rule) or so large that the serial merges of more waves win.
// us per interval without rounds / with 512, 1024, 2048 walkers' room, tau-leaping
// runs in steady state: 8 runs of 64 bins x 256 228 / 139, 153, 154; 128 such runs
// 782 / 618, 763, 1056, equalizing 1382 / 667, 842, 1224; 128 runs of 32 bins x 512
// 829 / 973, 706, 905, equalizing 1710 / 2402, 2917, 4813; 64 runs of 32 bins x
// 1000 1331 / 1336, 1792, 2427.
#define BINS_FEW_WAVES 512
static int32_t bins_cap(const SimArgs &a, int64_t waves) {
    const bool eq = a.rs_rule == 1;
    if (a.m_targ > RESAMPLE_BIG_M) {
        if (waves <= BINS_FEW_WAVES) return MERGE_ROUNDS_MAX;
        if (a.m_targ <= 384) return 512;
        if (!eq && a.m_targ <= 768) return 1024;
    }
    return eq ? 256 : 0;
}

// The batched split/merge's variants.
static constexpr int BATCH_CAPS[BATCH_BINS] = {256, 512, 1024, MERGE_ROUNDS_MAX};

// Member a's variant, and its workgroups per run; waves: batch_big_waves over the members.
int32_t batch_bins_cap(const SimArgs &a, int64_t waves) { return std::max(bins_cap(a, waves), BATCH_CAPS[0]); }
int64_t batch_big_waves(const SimArgs &a) { return a.m_targ > RESAMPLE_BIG_M ? (int64_t)a.n_runs * a.n_bins : 0; }
int32_t batch_bins_blocks(const SimArgs &a, int64_t waves, int variant) {
    if (batch_bins_cap(a, waves) != BATCH_CAPS[variant]) return 0;
    return variant == 0 ? bins_blocks<BATCH_CAPS[0]>(a.n_bins) : variant == 1 ? bins_blocks<BATCH_CAPS[1]>(a.n_bins)
           : variant == 2 ? bins_blocks<BATCH_CAPS[2]>(a.n_bins) : bins_blocks<BATCH_CAPS[3]>(a.n_bins);
}

// An empty workgroup takes 0.21 ns of a launch, finding the member about 1.1 ns per
// workgroup: the even grid where at most five in six are empty, or all are few.
// Two members of 2048 Schloegl runs 1.67 ms per step on the even grid and 1.74
// on the other, 512 runs of 16 bins with one of 4000 bins and 30 small members 3.50 and
// 0.070 ms.
#define BATCH_BINS_FEW 8192
#define BATCH_BINS_BLOCKS (1 << 20)   // workgroups stride from here on
template <int CAP>
void launch_batch_bins(const BatchPtrs &b, const BatchBins &n, int32_t n_sims, int32_t max_runs, hipStream_t st) {
    if (n.total == 0) return;
    const int64_t even = (int64_t)max_runs * n.max_blocks * n_sims;
    const dim3 block(64 * BinsBlock<CAP>::WAVES);
    if (even <= std::max<int64_t>(6 * n.total, BATCH_BINS_FEW))
        hipLaunchKernelGGL((we_batch_bins_kernel<CAP, true>), dim3(max_runs, n.max_blocks, n_sims), block,
                           BinsBlock<CAP>::LDS, st, b, n.first, n_sims);
    else
        hipLaunchKernelGGL((we_batch_bins_kernel<CAP, false>), dim3((unsigned)std::min<int64_t>(n.total, BATCH_BINS_BLOCKS)),
                           block, BinsBlock<CAP>::LDS, st, b, n.first, n_sims);
}

hipError_t launch_batch_bookkeeping(const BatchPtrs &b, int32_t n_sims, int64_t max_slots, int32_t max_runs,
                                    int64_t max_cells, const BatchBins *bins, size_t shmem, bool observe,
                                    const CmBatchModel *models,
                                    int32_t s_max_cm, uint32_t *counters, int32_t n_counters, hipStream_t st) {
    const unsigned gs = (unsigned)((max_slots + 255) / 256);
    hipLaunchKernelGGL(we_batch_recycle_bin_kernel, dim3(gs, n_sims), dim3(256), 0, st, b);
    if (models) {
        const hipError_t e = committor_bin_batch(b.args, b.x_cur, models, n_sims, max_slots, s_max_cm, st);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(we_batch_place_kernel, dim3(max_runs, n_sims),
                       dim3(resample_threads((int64_t)max_runs * n_sims)), shmem, st, b);
    launch_batch_bins<BATCH_CAPS[3]>(b, bins[3], n_sims, max_runs, st);
    launch_batch_bins<BATCH_CAPS[2]>(b, bins[2], n_sims, max_runs, st);
    launch_batch_bins<BATCH_CAPS[1]>(b, bins[1], n_sims, max_runs, st);
    launch_batch_bins<BATCH_CAPS[0]>(b, bins[0], n_sims, max_runs, st);
    const unsigned gg = (unsigned)std::max<int64_t>(1, std::min<int64_t>((max_cells + 255) / 256, BATCH_GATHER_BLOCKS));
    hipLaunchKernelGGL(we_batch_gather_kernel, dim3(gg, n_sims), dim3(256), 0, st, b);
    if (observe) hipLaunchKernelGGL(we_batch_observe_kernel, dim3(gs, n_sims), dim3(256), 0, st, b);
    hipLaunchKernelGGL(we_batch_advance_kernel, dim3((std::max(n_sims, n_counters) + 63) / 64), dim3(64), 0, st, b, n_sims,
                       counters, n_counters);
    return hipGetLastError();
}

hipError_t launch_recycle_bin(const SimArgs &a, int32_t *x_cur, bool grid_bins, hipStream_t st) {
    const int64_t total = (int64_t)a.n_runs * a.cap;
    hipLaunchKernelGGL(we_recycle_bin_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       a, x_cur, grid_bins ? 1 : 0);
    return hipGetLastError();
}

bool resample_uses_lds(const SimArgs &a);
static size_t lds_bytes_rows(const SimArgs &a, bool use_lds, int32_t rows) {
    const size_t tables = !use_lds && a.n_bins > RESAMPLE_EVB_BINS ? 3 : 4;
    size_t b = sizeof(int32_t) * ((tables + rows) * a.n_bins + 2) + 16;
    if (use_lds) b += (size_t)a.cap * (sizeof(double) + sizeof(int32_t) + 2 * sizeof(uint16_t));
    return b;
}

size_t resample_lds_bytes(const SimArgs &a, bool use_lds) {
    return lds_bytes_rows(a, use_lds, a.place_rows > 0 ? a.place_rows : 1);
}

// The per-walker arrays go to LDS when they fit beside a single cursor row.
bool resample_uses_lds(const SimArgs &a) {
    return a.cap <= RESAMPLE_LDS_CAP && lds_bytes_rows(a, true, 1) <= RESAMPLE_LDS_MAX;
}

int32_t resample_place_rows(const SimArgs &a, int64_t blocks) {
    const bool ul = resample_uses_lds(a);
    int32_t rows = (int32_t)(resample_threads(blocks) / 64);
    rows = std::min<int32_t>(rows, std::max<int32_t>(1, RESAMPLE_PLACE_INTS / std::max(1, a.n_bins)));
    while (rows > 1 && lds_bytes_rows(a, ul, rows) > RESAMPLE_LDS_MAX) --rows;
    return rows;
}

// Bin-parallel resampling pays when the runs alone leave most of the chip idle
// and a run's waves would otherwise take more than one bin each in turn
// (measured, one MI355X: 16 toggle runs x 64 bins 0.045 -> 0.033 ms, 64
// switch runs x 465 bins 0.211 -> 0.202 ms; one run of 50 bins on 16 waves
// 35.1 -> 33.3 us and eight such runs 57.2 -> 56.4 us per step, with the
// bins of up to 256 walkers merged in registers -- before those, one run
// of 50 bins went 0.063 -> 0.067 ms, its staging being in device memory).
bool resample_bins_parallel(const SimArgs &a) {
    const int64_t waves = resample_threads(a.n_runs) / 64;
    return a.n_runs < RESAMPLE_BIN_PARALLEL_RUNS && a.n_bins >= RESAMPLE_BIN_PARALLEL_BINS &&
           a.n_bins >= waves;
}

// Recycling and binning by the run's workgroup saves a launch, and costs its
// chain of fetches (row, coefficients, a search of the edges) once per walker of a
// thread.  It pays for short rows and one walker per thread: one birth-death run,
// 20 intervals 545 -> 499 us, 256 tau-leaping runs of 40 bins x 16, 50 intervals
// 4.32 -> 4.22 ms.  With two walkers per thread it is even (2048 Schloegl runs:
// 55.4 + 8.4 us -> 63.9), with 8 species or 2.5 walkers per thread it loses (16 toggle
// runs 8.2 + 4.9 us -> 16.1, 32 Schloegl runs of 80 x 32 10.4 + 4.8 -> 16.8).
bool resample_recycles(const SimArgs &a) {
    return !resample_bins_parallel(a) && resample_uses_lds(a) && a.S <= RESAMPLE_ROW_MAX &&
           a.cap <= (int32_t)resample_threads(a.n_runs);
}

// x_cur: null, or the rows to recycle and bin first (resample_recycles).
hipError_t launch_resample(const SimArgs &a, int32_t *x_cur, const double *w_cur, double *w_nxt, int32_t *binfo,
                           hipStream_t st) {
    const bool split = resample_bins_parallel(a);
    const bool use_lds = !split && resample_uses_lds(a);
    const size_t shmem = resample_lds_bytes(a, use_lds);
    const bool eq = a.rs_rule == 1;
    const dim3 gr(a.n_runs), br(resample_threads(a.n_runs));
    if (split) {
        // the placement takes no rule
        hipLaunchKernelGGL((we_resample_kernel<RS_PLACE, 0>), gr, br, shmem, st, a, x_cur, w_cur, w_nxt, binfo);
        switch (bins_cap(a, (int64_t)a.n_runs * a.n_bins)) {
        case MERGE_ROUNDS_MAX:
            if (eq) launch_bins<1, MERGE_ROUNDS_MAX>(a, w_nxt, binfo, st);
            else launch_bins<0, MERGE_ROUNDS_MAX>(a, w_nxt, binfo, st);
            break;
        case 1024: launch_bins<0, 1024>(a, w_nxt, binfo, st); break;
        case 512:
            if (eq) launch_bins<1, 512>(a, w_nxt, binfo, st);
            else launch_bins<0, 512>(a, w_nxt, binfo, st);
            break;
        case 256: launch_bins<1, 256>(a, w_nxt, binfo, st); break;
        default: launch_bins<0, 0>(a, w_nxt, binfo, st);
        }
    } else if (use_lds) {
        if (eq) hipLaunchKernelGGL((we_resample_kernel<RS_LDS, 1>), gr, br, shmem, st, a, x_cur, w_cur, w_nxt, nullptr);
        else hipLaunchKernelGGL((we_resample_kernel<RS_LDS, 0>), gr, br, shmem, st, a, x_cur, w_cur, w_nxt, nullptr);
    } else {
        if (eq) hipLaunchKernelGGL((we_resample_kernel<RS_GLOBAL, 1>), gr, br, shmem, st, a, x_cur, w_cur, w_nxt, nullptr);
        else hipLaunchKernelGGL((we_resample_kernel<RS_GLOBAL, 0>), gr, br, shmem, st, a, x_cur, w_cur, w_nxt, nullptr);
    }
    return hipGetLastError();
}

// The same with the one-species histogram summed per block in LDS first:
// block (run, i) takes walkers i*per ... (i+1)*per - 1 of one run, adds their
// weights into an LDS copy of the run's histogram row, then adds the nonzero
// entries to the row in device memory (one atomic per distinct count per
// block instead of one per walker, and none on a shared address within a
// run); the joint histogram likewise, per distinct cell.  Thread 0 of
// block (0, 0) also advances the iteration counter, which no step of this
// kernel reads, in place of the separate advance launch.  per = 1024
// walkers (four per thread) when the runs alone give enough blocks, else 256
// (one per thread: few runs, where the blocks' walkers are the whole grid).
#define OBS_WALKERS 1024
#define OBS_WALKERS_FEW 256
#define OBS_FEW_RUNS 64
#define OBS_LDS_BINS 6144
#define OBS_JOINT_LOG2 9
#define OBS_JOINT_SLOTS (1 << OBS_JOINT_LOG2)
#define OBS_JOINT_PROBES 16
// FRESH: the state rows are still the parents' (x_cur): each thread copies its
// walkers' rows to xs first, in place of the gather's launch.  What bounds both
// is the launch; a row of up to OBS_ROW_MAX counts fits one thread (longer ones
// want a lane per count).  Gather and observation of 16 runs of 64 bins x 16, 8
// species: 5.6 us, as two launches 4.4 and 4.1 and the gap between them.
#define OBS_ROW_MAX 16
template <bool FRESH>
__global__ __launch_bounds__(256) void we_observe_lds_kernel(SimArgs a, const int32_t *__restrict__ x_cur,
                                                             int32_t *__restrict__ xs,
                                                             const double *__restrict__ ws, int32_t per) {
    extern __shared__ __align__(16) unsigned char obs_lds[];
    double *h = reinterpret_cast<double *>(obs_lds);
    // joint-histogram cells of this block's walkers, summed per distinct cell
    // in an open-addressing table before one device atomic per cell (walkers
    // of one bin tend to share a cell, and device atomics on one address
    // serialize)
    __shared__ int32_t jkey[OBS_JOINT_SLOTS];
    __shared__ double jval[OBS_JOINT_SLOTS];
    const int32_t run = blockIdx.x, tid = threadIdx.x;
    if (run == 0 && blockIdx.y == 0 && tid == 0) *a.iter_dev += 1u;
    const int32_t n = a.n_walk[run];
    const int32_t k0 = (int32_t)blockIdx.y * per, k1 = min(n, k0 + per);
    if (k0 >= n) return;   // uniform over the block
    for (int32_t v = tid; v < a.nh; v += blockDim.x) h[v] = 0.0;
    for (int32_t v = tid; v < OBS_JOINT_SLOTS; v += blockDim.x) {
        jkey[v] = -1;
        jval[v] = 0.0;
    }
    __syncthreads();
    const size_t base = (size_t)run * a.cap;
    double *jrow = a.jhist + (size_t)run * a.jcells;
    for (int32_t k = k0 + tid; k < k1; k += blockDim.x) {
        const size_t idx = base + k;
        const double wv = ws[idx];
        const int32_t *row = FRESH ? x_cur + (base + (size_t)a.origin[idx]) * a.S : xs + idx * a.S;
        if constexpr (FRESH) {
            int32_t c[OBS_ROW_MAX];
#pragma unroll
            for (int sp = 0; sp < OBS_ROW_MAX; ++sp)
                if (sp < a.S) c[sp] = row[sp];
#pragma unroll
            for (int sp = 0; sp < OBS_ROW_MAX; ++sp)
                if (sp < a.S) xs[idx * a.S + sp] = c[sp];
        }
        const int32_t v = row[a.hist_species] - a.hist_lo;
        if (v >= 0 && v < a.nh) atomicAdd(&h[v], wv);
        if (a.n_joint > 0) {
            int32_t cell = 0, mul = 1;
            for (int d = 0; d < a.n_joint; ++d) {
                const int32_t c = min(row[a.joint_species[d]] / a.joint_width, a.joint_bins - 1);
                cell += c * mul;
                mul *= a.joint_bins;
            }
            const uint32_t h0 = ((uint32_t)cell * 2654435761u) >> (32 - OBS_JOINT_LOG2);
            bool done = false;
            for (int32_t p = 0; p < OBS_JOINT_PROBES && !done; ++p) {
                const int32_t slot = (int32_t)((h0 + (uint32_t)p) & (OBS_JOINT_SLOTS - 1));
                const int32_t prev = atomicCAS(&jkey[slot], -1, cell);
                if (prev == -1 || prev == cell) {
                    atomicAdd(&jval[slot], wv);
                    done = true;
                }
            }
            if (!done) atomicAdd(&jrow[cell], wv);   // table crowded: straight to the device row
        }
    }
    __syncthreads();
    double *row = a.hist + (size_t)run * a.nh;
    for (int32_t v = tid; v < a.nh; v += blockDim.x)
        if (h[v] != 0.0) atomicAdd(&row[v], h[v]);
    for (int32_t v = tid; v < OBS_JOINT_SLOTS; v += blockDim.x)
        if (jkey[v] >= 0) atomicAdd(&jrow[jkey[v]], jval[v]);
}

// New state rows (x_nxt), histograms and the end of the iteration; *advanced tells
// whether the iteration counter was advanced (else the caller launches the
// advance kernel).
hipError_t launch_gather_observe(const SimArgs &a, const int32_t *x_cur, int32_t *x_nxt, const double *ws,
                                 hipStream_t st, bool *advanced) {
    *advanced = false;
    const bool in_lds = a.nh > 0 && a.nh <= OBS_LDS_BINS;
    const bool fresh = in_lds && a.S <= OBS_ROW_MAX;
    if (!fresh) {
        const int64_t total = (int64_t)a.n_runs * a.cap * a.S;
        const int32_t narrow = total + 256 < ((int64_t)1 << 31) ? 1 : 0;
        hipLaunchKernelGGL(we_gather_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                           a, x_cur, x_nxt, narrow);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (a.nh <= 0 && a.n_joint <= 0) return hipSuccess;
    if (in_lds) {
        const int32_t per = a.n_runs < OBS_FEW_RUNS ? OBS_WALKERS_FEW : OBS_WALKERS;
        const dim3 grid((unsigned)a.n_runs, (unsigned)((a.cap + per - 1) / per));
        const size_t lds = (size_t)a.nh * sizeof(double);
        if (fresh) hipLaunchKernelGGL(we_observe_lds_kernel<true>, grid, dim3(256), lds, st, a, x_cur, x_nxt, ws, per);
        else hipLaunchKernelGGL(we_observe_lds_kernel<false>, grid, dim3(256), lds, st, a, x_cur, x_nxt, ws, per);
        *advanced = true;
        return hipGetLastError();
    }
    const int64_t total = (int64_t)a.n_runs * a.cap;
    hipLaunchKernelGGL(we_observe_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       a, x_nxt, ws);
    return hipGetLastError();
}

// End of an iteration: advance the device-side iteration counter.
__global__ void we_advance_kernel(SimArgs a) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *a.iter_dev += 1u;
}

hipError_t launch_advance(const SimArgs &a, hipStream_t st) {
    hipLaunchKernelGGL(we_advance_kernel, dim3(1), dim3(64), 0, st, a);
    return hipGetLastError();
}
