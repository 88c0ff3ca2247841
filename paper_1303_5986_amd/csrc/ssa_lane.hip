// ssa_lane.hip -- Gillespie direct-method SSA, one lane per walker (gfx950).
//
// Each lane carries one walker through one WE interval tau (Sec. II.A, the
// propagation step of the WE procedure in Sec. II.B):
//   1. all propensities a_j = c_j * prod_s C(x_s, nu_js) (divided by
//      1 + (x_r / K)^n for a Hill-type rate, Sec. III.C) and their total a0,
//      summed in reaction order;
//   2. waiting time dt = -log(1 - u1) / a0; stop when t + dt > tau (the
//      exponential is memoryless, so the overshoot is simply discarded);
//   3. reaction j = first index whose running sum exceeds u2 * a0;
//   4. x += nu_j, t += dt.
// u1, u2 come from one Philox4x32-10 block at counter (event, slot, iter, 0).
//
// Design for CDNA4: walker state and propensities live in VGPRs, the
// reaction table is wave-uniform (scalar loads), and the state change of the
// chosen reaction is an int8 delta row picked by register selects (up to 8
// reactions) or read from the wave's LDS copy of the rows, so nothing in the
// event loop waits on global memory.  HBM traffic is one read and one write
// of the state per interval.  Walkers are laid out bin-major, so neighbouring
// lanes have similar total propensity and the wave diverges little.
#include "ssa_lane_body.h"

#include <algorithm>

// Resident blocks per CU of the persistent grid, at most.
#ifndef LANE_POOL_PER_CU
#define LANE_POOL_PER_CU 5
#endif
// Idle lanes refill once at least this many of the wave's lanes are idle.
#ifndef LANE_REFILL_MIN
#define LANE_REFILL_MIN 12
#endif

// A wave's share of the work queue.  Atomics on one address (or one 128-byte
// line) take 11.4 ns each on this device, whoever asks (0.27 ns over 64 lines):
// with a single queue head the first request of 4096 waves alone took 47 us,
// and 64 switch runs (330,000 walkers of 3.4 events) waited on the head more
// than they computed.  So the queue, in tiles of 64 positions, is dealt out to
// up to 64 heads on lines of their own, block b using head b mod n (a multiple
// of 8 heads keeps each on one XCD); a wave's first 64 positions are static.
// Tiles alternate between the heads in queue order, so each head hands out the
// same mix, busiest first.  The static tiles go block by block, so that the
// busy ones spread over a CU's four SIMDs: given to wave 0 of every block first
// they all land on one SIMD of each CU (2048 Schloegl runs 743 against 675 us).
// No result depends on it.  Per launch, before and after: 64 switch runs 179 ->
// 58 us, 256 tau-leaping runs 57 -> 44 us.
#define POOL_BLOCKS_PER_HEAD 4
struct PoolQueue {
    uint32_t n, s;          // heads in use, this block's
    uint32_t first;         // this wave's static first position
    uint32_t n_first;       // positions handed out statically
    uint32_t size;          // positions of this head's tiles (its last tile may pass the queue's end)
    uint32_t *head;
    __device__ __forceinline__ PoolQueue(const SimArgs &a, uint32_t total) {
        n = min((uint32_t)a.n_heads, max(gridDim.x / POOL_BLOCKS_PER_HEAD, 1u));
        if (n >= 8) n &= ~7u;
        s = blockIdx.x % n;
        const uint32_t blocks = (gridDim.x - s + n - 1) / n, tiles = (total + 63) / 64;
        first = (blockIdx.x / n * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64u;
        n_first = (blockDim.x >> 6) * blocks * 64u;
        size = tiles > s ? (tiles - s + n - 1) / n * 64u : 0u;
        head = a.heads + s * WE_HEAD_STRIDE;
    }
    // Where the static tiles are the whole queue, a wave takes every n-th position
    // instead (n waves to a head), one from each stretch of the queue, so that
    // its walkers run out one by one and the last ones can be teamed up
    // (lane_team); tiles would give it 64 walkers of one length.
    __device__ __forceinline__ uint32_t dealt(uint32_t lane) const { return lane * (n_first / 64u) + first / 64u; }
    // queue position of this head's position i
    __device__ __forceinline__ uint32_t at(uint32_t i) const { return i < size ? ((i >> 6) * n + s) * 64u + (i & 63u) : ~0u; }
};

// Persistent lane kernel: every lane runs walkers from the work queue (see
// work_queue.hip) until it is empty; the wave takes as many queue entries as
// it has idle lanes with one atomic and hands them out in lane order.  Walkers
// differ a lot in how many events one interval takes (the total propensity
// grows steeply along the progress coordinate), so a fixed walker-per-lane
// assignment would leave most lanes of a wave idle while its slowest walker
// finishes.
// The end of a wave's work: the queue is empty and at most 32 of its walkers
// are left.  They are spread out, T = 2 ... 16 lanes (a team) per walker, and the
// lanes of a team draw the random numbers of T events at once, one event each
// (Philox, logarithm and conversions are about 70% of an event's instructions),
// then run those events side by side, every lane on the same state.  T doubles
// as walkers finish; the walkers take the same steps.  A launch lasts as long as
// its busiest walker's chain of events: with the branch-free event, one Schloegl
// run of 80 bins x 32 walkers (1158 events at most) 719 -> 304 ns per event of
// that walker, 32 such runs 783 -> 422 ns.
template <int SMAX, int RMAX, bool HILL, bool PAIR>
__device__ __forceinline__ void lane_team(const SimArgs &a, const LaneNet<SMAX, RMAX, HILL, PAIR> &net, LaneWalker &w,
                                          int32_t (&x)[SMAX], int32_t *__restrict__ xs, size_t gslot,
                                          bool active, uint32_t iter, double tau) {
    const int lane = threadIdx.x & 63;
    int T = 1;
    uint32_t g = (uint32_t)gslot;
    for (;;) {
        // teams left: their first lanes (lane 0 of a team is a multiple of T)
        const unsigned long long lead = __ballot(active && (lane & (T - 1)) == 0);
        const int n = __popcll(lead);
        if (n == 0) return;
        if (T < 16 && 2 * T * n <= 64) {
            int U = 2 * T;
            while (U < 16 && 2 * U * n <= 64) U *= 2;
            // team j of the new teams takes the j-th walker left: its first lane
            // hears from that walker's lane, the others from the first
            const int rank = __popcll(lead & ((1ull << lane) - 1ull));
            const bool is_lead = active && (lane & (T - 1)) == 0;
            // lanes that send nothing address a lane that no team's first lane is
            int src = __builtin_amdgcn_ds_permute(4 * (is_lead ? rank * U : 1), lane);
            src = __shfl(src, lane & ~(U - 1), 64);
            const bool on = lane / U < n;
            src = on ? src : lane;
            w.t = __shfl(w.t, src, 64);
            w.e = (uint32_t)__shfl((int)w.e, src, 64);
            w.fired = (uint32_t)__shfl((int)w.fired, src, 64);
            g = (uint32_t)__shfl((int)g, src, 64);
            w.k0 = (uint32_t)__shfl((int)w.k0, src, 64);
            w.k1 = (uint32_t)__shfl((int)w.k1, src, 64);
            w.slot = (uint32_t)__shfl((int)w.slot, src, 64);
#pragma unroll
            for (int s = 0; s < SMAX; ++s) x[s] = __shfl(x[s], src, 64);
            active = on;
            w.bad = false;
            w.rs.init(w.slot, iter, w.k0, w.k1);
            T = U;
        }
        const int first = lane & ~(T - 1);
        const EventDraw mine = lane_draw(w.rs, w.e + (uint32_t)(lane - first));
        w.e += (uint32_t)T;
        // the next event's pair is fetched while this one runs
        EventDraw nx{__shfl(mine.nl, first, 64), __shfl(mine.u2, first, 64)};
        for (int i = 1; i <= T; ++i) {
            const EventDraw d = nx;
            nx.nl = __shfl(mine.nl, first + i, 64);
            nx.u2 = __shfl(mine.u2, first + i, 64);
            if (active && !lane_event(net, w, x, tau, [&]() { return d; })) {
                if (lane == first) lane_finish(a, w, x, xs + (size_t)g * a.S, (size_t)g);
                active = false;
            }
            if (!__ballot(active)) return;
        }
    }
}

template <int SMAX, int RMAX, bool HILL, bool LEAP, bool PAIR>
__device__ __forceinline__ void lane_pool(const SimArgs &a, int32_t *__restrict__ xs, int32_t *wrows) {
    constexpr bool REG = RMAX <= LANE_REG_RMAX;
    if constexpr (!REG) lane_stage_rows<SMAX>(a, wrows);
    LaneNet<SMAX, RMAX, HILL, PAIR> net;
    net.load(a, wrows);
    uint32_t hor[LEAP ? SMAX : 1], hnu[LEAP ? SMAX : 1];
    if constexpr (LEAP) leap_orders(net, hor, hnu);
    LeapRng lr;
    lr.reset();
    const int lane = threadIdx.x & 63;
    const uint32_t iter = *a.iter_dev;
    const double tau = a.tau;
    const uint32_t M = (uint32_t)a.m_targ;
    const uint32_t total = a.queue[1] * M;
    const PoolQueue pq(a, total);
    const unsigned long long below = lane ? ((1ull << lane) - 1ull) : 0ull;
    LaneWalker w;
    int32_t x[SMAX];
    w.bad = false;
    bool active = false, exhausted = false, first = true;
    size_t gslot = 0;
    int32_t *xr = xs;
    for (;;) {
        const unsigned long long need = __ballot(!active);
        const int nneed = __popcll(need);
        if (!exhausted && (nneed >= LANE_REFILL_MIN || nneed == 64)) {
            // every lane executes the atomic (only the leader adds), so no
            // lane takes a path of its own around the wave-wide steps
            const int leader = __ffsll((long long)need) - 1;
            uint32_t base = pq.first;
            if (!first) {
                const uint32_t got = atomicAdd(pq.head, lane == leader ? (uint32_t)nneed : 0u);
                base = pq.n_first + (uint32_t)__shfl((int)got, leader, 64);
            }
            if ((uint64_t)(first ? pq.n_first : base + (uint32_t)nneed) >= pq.size) exhausted = true;
            if (!active) {
                const uint32_t rank = (uint32_t)__popcll(need & below);
                const uint32_t q = pq.at(!LEAP && first && pq.size <= pq.n_first ? pq.dealt(rank) : base + rank);
                if (q < total) {
                    const uint32_t sg = q / M, o = q - sg * M;
                    const int2 seg = a.seg[sg];
                    if ((int32_t)o < seg.y) {
                        const uint32_t g = (uint32_t)seg.x + o;   // below 2^30
                        const uint32_t run = g / (uint32_t)a.cap;
                        const uint32_t k = g - run * (uint32_t)a.cap;
                        gslot = g;
                        xr = xs + gslot * a.S;
                        w.begin(x, xr, a.S, k, a.seeds[run], iter);
                        if constexpr (LEAP) lr.reset();
                        active = true;
                    }
                }
            }
            first = false;
        }
        if (!__ballot(active) && exhausted) break;
        if constexpr (LEAP) {
            if (active && !lane_leap_step(net, w, lr, x, hor, hnu, iter, tau, a.leap_eps)) {
                lane_finish(a, w, x, xr, gslot);
                active = false;
            }
        } else {
            if (exhausted && nneed >= 32) {
                lane_team<SMAX, RMAX, HILL, PAIR>(a, net, w, x, xs, gslot, active, iter, tau);
                break;
            }
            if (active && !lane_event(net, w, x, tau, [&]() { return lane_draw(w.rs, w.e++); })) {
                lane_finish(a, w, x, xr, gslot);
                active = false;
            }
        }
    }
}

// Five waves per SIMD for the smallest networks, whose registers allow it.
// PAIR: reactions of at most two molecules (LanePair).
template <int SMAX, int RMAX, bool PAIR>
__global__ __launch_bounds__(256, SMAX == 1 ? 5 : 1) void ssa_lane_pool_kernel(SimArgs a, int32_t *__restrict__ xs) {
    constexpr int ROWS = RMAX <= LANE_REG_RMAX ? 1 : RMAX * LaneRow<SMAX>::W;
    __shared__ int32_t rows[4 * ROWS];
    lane_pool<SMAX, RMAX, false, false, PAIR>(a, xs, rows + (threadIdx.x >> 6) * ROWS);
}

// The same for networks with Hill-type rates (Sec. III.C).
template <int SMAX, int RMAX>
__global__ __launch_bounds__(256) void ssa_lane_hill_kernel(SimArgs a, int32_t *__restrict__ xs) {
    constexpr int ROWS = RMAX <= LANE_REG_RMAX ? 1 : RMAX * LaneRow<SMAX>::W;
    __shared__ int32_t rows[4 * ROWS];
    lane_pool<SMAX, RMAX, true, false, false>(a, xs, rows + (threadIdx.x >> 6) * ROWS);
}

// The same with tau-leaping instead of the exact direct method.
template <int SMAX, int RMAX>
__global__ __launch_bounds__(256) void ssa_lane_leap_kernel(SimArgs a, int32_t *__restrict__ xs) {
    constexpr int ROWS = RMAX <= LANE_REG_RMAX ? 1 : RMAX * LaneRow<SMAX>::W;
    __shared__ int32_t rows[4 * ROWS];
    lane_pool<SMAX, RMAX, false, true, false>(a, xs, rows + (threadIdx.x >> 6) * ROWS);
}

// Fixed assignment, one walker per lane: used for the two largest variants,
// whose register footprint leaves no room for the queue state.
template <int SMAX, int RMAX>
__global__ __launch_bounds__(256) void ssa_lane_kernel(SimArgs a, int32_t *__restrict__ xs) {
    constexpr bool REG = RMAX <= LANE_REG_RMAX;
    constexpr int ROWS = REG ? 1 : RMAX * LaneRow<SMAX>::W;
    __shared__ int32_t rows[4 * ROWS];
    int32_t *wrows = rows + (threadIdx.x >> 6) * ROWS;
    if constexpr (!REG) lane_stage_rows<SMAX>(a, wrows);
    const int32_t gid = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    const int32_t run = gid / a.cap;
    const int32_t k = gid - run * a.cap;
    if (run >= a.n_runs) return;
    if (k >= a.n_walk[run]) return;
    lane_walker<SMAX, RMAX>(a, xs, run, k, *a.iter_dev, wrows);
}


namespace {
// Persistent grid: as many blocks as stay resident on the device, capped at
// LANE_POOL_PER_CU per CU.
template <int SMAX, int RMAX, int VARIANT, bool PAIR>   // 0: exact, 1: Hill-type rates, 2: tau-leaping
unsigned pool_blocks(const SimArgs &a) {
    static int per_cu = -1, n_cu = 0;   // one cache per kernel
    void (*kernel)(SimArgs, int32_t *);
    if constexpr (VARIANT == 1) kernel = ssa_lane_hill_kernel<SMAX, RMAX>;
    else if constexpr (VARIANT == 2) kernel = ssa_lane_leap_kernel<SMAX, RMAX>;
    else kernel = ssa_lane_pool_kernel<SMAX, RMAX, PAIR>;
    if (per_cu < 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess || per_cu < 1) {
            per_cu = 1;
            n_cu = std::max(n_cu, 1);
        }
        // More resident blocks are not faster: on Schloegl at 2048 x 60 x 8
        // walkers, when <1,4> could hold 7 per CU, a launch took 1.188 ms at 5
        // per CU against 1.215 at 4, 1.268 at 3, 1.243 at 6 and 1.230 at 7.
        if (per_cu > LANE_POOL_PER_CU) per_cu = LANE_POOL_PER_CU;
    }
    // Where the chip has more room than walkers: up to four times the waves, each
    // with fewer walkers, which start as teams (one Schloegl run of 80 bins x 32
    // walkers 433 -> 352 us); past one block per CU, whole blocks per CU, since
    // the SIMDs with one wave more would finish last (32 such runs: 320 blocks
    // 597, 256 482, 512 533, 1024 798 us).
    int64_t need = ((int64_t)a.n_runs * a.cap + 255) / 256;
    if (VARIANT != 2) need = need < n_cu ? need * std::min<int64_t>(4, n_cu / need) : (need + n_cu / 2) / n_cu * n_cu;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(need, (int64_t)per_cu * n_cu));
}

template <int SMAX, int RMAX>
hipError_t launch_fixed(const SimArgs &a, int32_t *xs, hipStream_t st) {
    const int64_t total = (int64_t)a.n_runs * a.cap;
    hipLaunchKernelGGL((ssa_lane_kernel<SMAX, RMAX>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a,
                       xs);
    return hipGetLastError();
}

template <int SMAX, int RMAX, bool PAIR = false>
hipError_t launch_pool(const SimArgs &a, int32_t *xs, hipStream_t st) {
    hipLaunchKernelGGL((ssa_lane_pool_kernel<SMAX, RMAX, PAIR>), dim3(pool_blocks<SMAX, RMAX, 0, PAIR>(a)),
                       dim3(256), 0, st, a, xs);
    return hipGetLastError();
}

template <int SMAX, int RMAX>
hipError_t launch_hill(const SimArgs &a, int32_t *xs, hipStream_t st) {
    hipLaunchKernelGGL((ssa_lane_hill_kernel<SMAX, RMAX>), dim3(pool_blocks<SMAX, RMAX, 1, false>(a)),
                       dim3(256), 0, st, a, xs);
    return hipGetLastError();
}
template <int SMAX, int RMAX>
hipError_t launch_leap(const SimArgs &a, int32_t *xs, hipStream_t st) {
    hipLaunchKernelGGL((ssa_lane_leap_kernel<SMAX, RMAX>), dim3(pool_blocks<SMAX, RMAX, 2, false>(a)),
                       dim3(256), 0, st, a, xs);
    return hipGetLastError();
}
}  // namespace

// Launch helper: picks the smallest register footprint that holds the
// network.  The queue variants need the queue built by launch_work_queue.
hipError_t launch_ssa_lane(const SimArgs &a, int32_t *xs, hipStream_t st) {
    if (a.engine == 1) {
        if (a.hill) return hipErrorInvalidValue;
        if (a.S <= 1 && a.R <= 4) return launch_leap<1, 4>(a, xs, st);
        if (a.S <= 2 && a.R <= 8) return launch_leap<2, 8>(a, xs, st);
        if (a.S <= 8 && a.R <= 16) return launch_leap<8, 16>(a, xs, st);
        return hipErrorInvalidValue;
    }
    if (a.hill) {
        if (a.S <= 2 && a.R <= 8) return launch_hill<2, 8>(a, xs, st);
        if (a.S <= 8 && a.R <= 16) return launch_hill<8, 16>(a, xs, st);
        return hipErrorInvalidValue;
    }
    if (a.S <= 1 && a.R <= 4) return launch_pool<1, 4>(a, xs, st);
    if (a.S <= 2 && a.R <= 8) return launch_pool<2, 8>(a, xs, st);
    // Up to eight reactions: tables in scalar registers (10 futile-cycle runs of 101
    // bins x 100 walkers, 6 species: <8,16> 61.4 us per interval, <8,8> 41.8), and
    // where no reaction takes three molecules the pair form (26.5).  Networks of two
    // species keep the general form: its branches cost them less than the picks (64
    // switch runs of 465 bins x 16, Hill-type rates: 59 us, in pair form 66).
    if (a.S <= 8 && a.R <= 8) return a.desc2 ? launch_pool<8, 8, true>(a, xs, st) : launch_pool<8, 8>(a, xs, st);
    if (a.S <= 8 && a.R <= 16) return launch_pool<8, 16>(a, xs, st);
    if (a.S <= 16 && a.R <= 32) return launch_fixed<16, 32>(a, xs, st);
    if (a.S <= 32 && a.R <= 64) return launch_fixed<32, 64>(a, xs, st);
    return hipErrorInvalidValue;
}

// The name of the kernel launch_ssa_lane runs for these arguments (a third
// template argument, the pair form, only where it is set).
const char *ssa_lane_name(const SimArgs &a) {
    if (a.engine == 1)
        return a.S <= 1 && a.R <= 4 ? "ssa_lane_leap_kernel<1,4>"
               : a.S <= 2 && a.R <= 8 ? "ssa_lane_leap_kernel<2,8>" : "ssa_lane_leap_kernel<8,16>";
    if (a.hill) return a.S <= 2 && a.R <= 8 ? "ssa_lane_hill_kernel<2,8>" : "ssa_lane_hill_kernel<8,16>";
    if (a.S <= 1 && a.R <= 4) return "ssa_lane_pool_kernel<1,4>";
    if (a.S <= 2 && a.R <= 8) return "ssa_lane_pool_kernel<2,8>";
    if (a.S <= 8 && a.R <= 8) return a.desc2 ? "ssa_lane_pool_kernel<8,8,true>" : "ssa_lane_pool_kernel<8,8>";
    if (a.S <= 8 && a.R <= 16) return "ssa_lane_pool_kernel<8,16>";
    if (a.S <= 16 && a.R <= 32) return "ssa_lane_kernel<16,32>";
    return "ssa_lane_kernel<32,64>";
}

// Deltas travel as int8, so every change must lie in [-128, 127].
bool lane_kernel_fits(int32_t S, int32_t R, int32_t max_delta) {
    return S <= 32 && R <= 64 && max_delta <= 127;
}
