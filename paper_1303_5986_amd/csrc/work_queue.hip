// work_queue.hip -- the walker work queue of the persistent propagation
// kernels (gfx950).
//
// Before each propagation step three small kernels (one, for few runs) list
// the walkers as segments of up to m_targ consecutive slots (one occupied
// bin after resampling) and order the segments by the mean events per walker
// seen in their bin during the last interval, busiest first -- longest-
// processing-time-first scheduling, so the long walkers start early and the
// short ones fill the tail.  The propagation kernels then take walkers from the front
// of the queue (the lane kernels' has several heads) with one atomic per request.  The order is a scheduling hint
// only: every result depends on (seed, iteration, slot, event), never on
// which lane or wave runs a walker.
#include "we_common.h"

// The lane kernels' queue heads (a.queue[0] itself when there is only that).
__device__ __forceinline__ void clear_heads(const SimArgs &a, int32_t tid) {
    if (tid < a.n_heads) a.heads[tid * WE_HEAD_STRIDE] = 0u;
}

// Segments per bin: one thread per (run, segment).
__global__ __launch_bounds__(256) void queue_count_kernel(SimArgs a) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t run = (int32_t)(gid / a.n_bins), j = (int32_t)(gid - (int64_t)run * a.n_bins);
    if (run >= a.n_runs) return;
    const int64_t first = (int64_t)j * a.m_targ;
    if (first >= a.n_walk[run]) return;
    const int32_t b = min(max(a.bin[(size_t)run * a.cap + first], 0), a.n_bins - 1);
    atomicAdd(&a.occ_bin[run % a.seg_rep * a.n_bins + b], 1);
}

// Bitonic sort of 64 (key, bin) pairs held one per lane, descending by key
// and, for equal keys, by bin.
__device__ __forceinline__ void wave_sort_desc(float &key, int32_t &idx, int lane) {
    for (int size = 2; size <= 64; size <<= 1)
        for (int d = size >> 1; d > 0; d >>= 1) {
            const float ko = __shfl_xor(key, d, 64);
            const int32_t io = __shfl_xor(idx, d, 64);
            const bool lower = (lane & d) == 0;
            const float ki = lower ? key : ko, kj = lower ? ko : key;
            const int32_t bi = lower ? idx : io, bj = lower ? io : idx;
            const bool i_first = ki > kj || (ki == kj && bi > bj);
            const bool desc = (lane & size) == 0;
            if (i_first != desc) {
                key = ko;
                idx = io;
            }
        }
}

// Bin order and queue offsets: one block.  Orders the bins by mean events per
// walker, descending, lays out their segments in that order, and clears the
// statistics and the queue.  SMALL (few runs, queue_small below): the same
// block first counts the segments into LDS and afterwards lists them itself,
// so the three steps are one launch.
// Counters lie [replica][bin], so that a run's adds and the reads here are of
// consecutive words.  The order needs no sort: keys are binary floats >= 0, so
// their bits order them, and a histogram over the distance to the largest key in
// steps of 2^-7 of a factor of two (1024 of them: down to 1/256 of the largest)
// gives every bin its place with one LDS atomic.  Bins of one step come in any
// order.  What bounds it is the latency of its few phases: 465 bins, 64 runs
// took 36 us, 60 bins, 2048 runs 16.8, 80 bins, 32 runs 17.7 and 100 bins, 10 runs
// 16 us with a bitonic sort over the block (a barrier per step, one wave per bin
// for the sums); this form takes 5.1, 8.5, 7.6 and 6.1 us.  The counters' layout
// also took the runs' adds in resampling (2048 runs: 61 -> 55.5 us with them).
#define QUEUE_MAX_BINS 8192
#define QUEUE_SMALL_SEGS 4096
#define QUEUE_SMALL_BINS 1024
#define QUEUE_STEPS 1024
#define QUEUE_STEP_SHIFT 16
template <bool SMALL>
__global__ __launch_bounds__(1024) void queue_order_kernel(SimArgs a) {
    constexpr int32_t KB = SMALL ? QUEUE_SMALL_BINS : QUEUE_MAX_BINS;
    __shared__ uint32_t key[KB];         // mean events per walker, as bits
    __shared__ int32_t at[KB];           // the bin's segments, then their place within its step
    __shared__ int32_t step[QUEUE_STEPS];
    __shared__ float part_ev[1024];      // several threads per bin: their sums
    __shared__ int32_t part_n[1024], part_occ[1024];
    __shared__ uint32_t key_max;
    __shared__ int32_t wave_tot[16];
    // SMALL only: segments and next position per counter; per thread, up to
    // PER (run, segment) pairs' walkers and counter (-1: none) and one counter's
    // statistics, all fetched at once
    __shared__ int32_t s_occ[SMALL ? QUEUE_SMALL_BINS : 1];
    __shared__ int32_t s_off[SMALL ? QUEUE_SMALL_BINS : 1];
    constexpr int PER = SMALL ? QUEUE_SMALL_SEGS / 1024 : 1;
    int32_t sg_n[PER], sg_c[PER];
    float my_ev = 0.0f;
    int32_t my_nw = 0;
    const int32_t NB = a.n_bins, tid = threadIdx.x, nthr = blockDim.x;
    const int32_t rep = a.seg_rep, NC = NB * rep;
    const int lane = tid & 63, wv = tid >> 6;
    const int32_t n_seg = a.n_runs * NB;
    step[tid] = 0;
    if (tid == 0) key_max = 0u;
    if constexpr (SMALL) {
        if (tid < NC) {
            s_occ[tid] = 0;
            my_ev = a.ev_bin[tid];
            my_nw = a.n_bin[tid];
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int32_t sg = tid + u * nthr;
            sg_n[u] = sg < n_seg ? a.n_walk[sg / NB] : 0;
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int32_t sg = tid + u * nthr, run = sg / NB;
            const int64_t first = (int64_t)(sg - run * NB) * a.m_targ;
            sg_c[u] = -1;
            if (first < sg_n[u])
                sg_c[u] = run % rep * NB + min(max(a.bin[(size_t)run * a.cap + first], 0), NB - 1);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (sg_c[u] >= 0) atomicAdd(&s_occ[sg_c[u]], 1);
    }
    __syncthreads();
    auto occ = [&](int32_t c) { return SMALL ? s_occ[SMALL ? c : 0] : a.occ_bin[c]; };
    // G threads per bin, each over every G-th replica
    const int32_t G = max(1, min(1024 / NB, rep));
    uint32_t my_max = 0u;
    for (int32_t i = tid; i < G * NB; i += nthr) {
        const int32_t sub = i / NB, b = i - sub * NB;
        float ev = 0.0f;
        int32_t nw = 0, oc = 0;
        if constexpr (SMALL) {   // NB * rep <= 1024: a thread per counter
            ev = my_ev;
            nw = my_nw;
            oc = s_occ[i];
        } else {
#pragma unroll 8
            for (int32_t r = sub; r < rep; r += G) {
                ev += a.ev_bin[r * NB + b];
                nw += a.n_bin[r * NB + b];
                oc += occ(r * NB + b);
            }
        }
        if (G > 1) {
            part_ev[i] = ev;
            part_n[i] = nw;
            part_occ[i] = oc;
        } else {
            key[b] = __float_as_uint(nw > 0 ? ev / (float)nw : 0.0f);
            at[b] = oc;
            my_max = max(my_max, key[b]);
        }
    }
    if (G > 1) {
        __syncthreads();
        if (tid < NB) {
            float ev = 0.0f;
            int32_t nw = 0, before = 0;
            for (int32_t sub = 0; sub < G; ++sub) {
                const int32_t i = sub * NB + tid, oc = part_occ[i];
                ev += part_ev[i];
                nw += part_n[i];
                part_occ[i] = before;
                before += oc;
            }
            key[tid] = __float_as_uint(nw > 0 ? ev / (float)nw : 0.0f);
            at[tid] = before;
            my_max = key[tid];
        }
    }
    for (int d = 32; d > 0; d >>= 1) my_max = max(my_max, (uint32_t)__shfl_xor((int)my_max, d, 64));
    if (lane == 0 && my_max > 0u) atomicMax(&key_max, my_max);
    __syncthreads();
    auto step_of = [&](int32_t b) {
        return (int32_t)min((uint32_t)(QUEUE_STEPS - 1), (key_max - key[b]) >> QUEUE_STEP_SHIFT);
    };
    for (int32_t b = tid; b < NB; b += nthr) at[b] = atomicAdd(&step[step_of(b)], at[b]);
    __syncthreads();
    // first position of each step
    const int32_t mine = step[tid];
    int32_t incl = mine;
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) wave_tot[wv] = incl;
    __syncthreads();
    for (int w = 0; w < wv; ++w) incl += wave_tot[w];
    step[tid] = incl - mine;
    if (tid == nthr - 1) {
        a.queue[0] = 0u;
        a.queue[1] = (uint32_t)incl;
    }
    clear_heads(a, tid);
    __syncthreads();
    for (int32_t i = tid; i < G * NB; i += nthr) {
        const int32_t sub = i / NB, b = i - sub * NB;
        int32_t pos = step[step_of(b)] + at[b] + (G > 1 ? part_occ[i] : 0);
        for (int32_t r0 = sub; r0 < rep; r0 += 8 * G) {
            int32_t oc[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) oc[u] = r0 + u * G < rep ? occ((r0 + u * G) * NB + b) : 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int32_t r = r0 + u * G, c = r * NB + b;
                if (r >= rep) break;
                if (SMALL) {
                    s_off[c] = pos;
                } else {
                    a.seg_off[c] = pos;
                    a.occ_bin[c] = 0;
                    a.seg_cur[c] = 0;
                }
                a.ev_bin[c] = 0.0f;
                a.n_bin[c] = 0;
                pos += oc[u];
            }
        }
    }
    if constexpr (SMALL) {
        __syncthreads();
        // the segment list, as queue_fill_kernel lays it out
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (sg_c[u] < 0) continue;
            const int32_t sg = tid + u * nthr, run = sg / NB;
            const int64_t first = (int64_t)(sg - run * NB) * a.m_targ;
            const int32_t pos = atomicAdd(&s_off[sg_c[u]], 1);
            a.seg[pos] =
                make_int2((int32_t)((size_t)run * a.cap + first), (int32_t)min((int64_t)a.m_targ, sg_n[u] - first));
        }
    }
}

// Tiny case (queue_tiny: at most 64 segments and 64 counters, e.g. one run of
// up to 64 bins): the same three steps in one wave, with no block barrier
// in the sort -- lane b holds bin b's key, a bitonic sort over the 64 lanes
// by shuffles (padding keys -1 last), then a wave prefix over the counters in
// sorted order.
__global__ __launch_bounds__(64) void queue_order_wave_kernel(SimArgs a) {
    __shared__ int32_t s_occ[64], s_off[64], s_cur[64];
    const int lane = threadIdx.x & 63;
    const int32_t NB = a.n_bins, rep = a.seg_rep, NC = NB * rep, n_seg = a.n_runs * NB;
    s_occ[lane] = 0;
    s_cur[lane] = 0;
    __syncthreads();
    // each segment's bin (lane = run * NB + segment)
    int32_t b = -1, run = 0, j = 0;
    if (lane < n_seg) {
        run = lane / NB;
        j = lane - run * NB;
        if ((int64_t)j * a.m_targ < a.n_walk[run]) {
            b = min(max(a.bin[(size_t)run * a.cap + (size_t)j * a.m_targ], 0), NB - 1);
            atomicAdd(&s_occ[run % rep * NB + b], 1);
        }
    }
    // bin keys: mean events per walker over the bin's replica counters
    float key = -1.0f;
    int32_t idx = lane;
    if (lane < NB) {
        float ev = 0.0f;
        int32_t nw = 0;
        for (int32_t r = 0; r < rep; ++r) {
            ev += a.ev_bin[r * NB + lane];
            nw += a.n_bin[r * NB + lane];
        }
        key = nw > 0 ? ev / (float)nw : 0.0f;
    }
    wave_sort_desc(key, idx, lane);
    __syncthreads();
    // exclusive prefix of the counters in sorted bin order (replicas of a
    // bin consecutive): lane i holds counter i of that sequence
    const int32_t bin_at = __shfl(idx, rep > 0 ? lane / rep : 0, 64);
    const int32_t c = lane % rep * NB + bin_at;
    const int32_t cnt = lane < NC ? s_occ[c] : 0;
    int32_t incl = cnt;
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane < NC) s_off[c] = incl - cnt;
    const int32_t total = __shfl(incl, 63, 64);
    if (lane == 0) {
        a.queue[0] = 0u;
        a.queue[1] = (uint32_t)total;
    }
    clear_heads(a, lane);
    __syncthreads();
    // the segment list, as queue_fill_kernel lays it out
    if (b >= 0) {
        const int32_t n = a.n_walk[run];
        const int64_t first = (int64_t)j * a.m_targ;
        const int32_t cc = run % rep * NB + b;
        const int32_t pos = s_off[cc] + atomicAdd(&s_cur[cc], 1);
        a.seg[pos] = make_int2((int32_t)((size_t)run * a.cap + first), (int32_t)min((int64_t)a.m_targ, n - first));
    }
    if (lane < NC) {
        a.ev_bin[lane] = 0.0f;
        a.n_bin[lane] = 0;
    }
}

// Segment list: one thread per (run, segment), same grid as the count.
__global__ __launch_bounds__(256) void queue_fill_kernel(SimArgs a) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t run = (int32_t)(gid / a.n_bins), j = (int32_t)(gid - (int64_t)run * a.n_bins);
    if (run >= a.n_runs) return;
    const int32_t n = a.n_walk[run];
    const int64_t first = (int64_t)j * a.m_targ;
    if (first >= n) return;
    const size_t g = (size_t)run * a.cap + first;
    const int32_t b = min(max(a.bin[g], 0), a.n_bins - 1);
    const int32_t c = run % a.seg_rep * a.n_bins + b;
    const int32_t pos = a.seg_off[c] + atomicAdd(&a.seg_cur[c], 1);
    a.seg[pos] = make_int2((int32_t)g, (int32_t)min((int64_t)a.m_targ, n - first));
}

// Few runs (at most QUEUE_SMALL_SEGS segments, QUEUE_SMALL_BINS counters):
// one block does all three steps; else three launches.
bool queue_small(const SimArgs &a) {
    return (int64_t)a.n_runs * a.n_bins <= QUEUE_SMALL_SEGS && a.n_bins <= QUEUE_SMALL_BINS &&
           (int64_t)a.n_bins * a.seg_rep <= QUEUE_SMALL_BINS;
}

// At most 64 segments and 64 counters: one wave does everything.
bool queue_tiny(const SimArgs &a) {
    return (int64_t)a.n_runs * a.n_bins <= 64 && a.n_bins <= 64 && (int64_t)a.n_bins * a.seg_rep <= 64;
}

hipError_t launch_work_queue(const SimArgs &a, hipStream_t st) {
    if (queue_tiny(a)) {
        hipLaunchKernelGGL(queue_order_wave_kernel, dim3(1), dim3(64), 0, st, a);
        return hipGetLastError();
    }
    if (queue_small(a)) {
        hipLaunchKernelGGL(queue_order_kernel<true>, dim3(1), dim3(1024), 0, st, a);
        return hipGetLastError();
    }
    const int64_t total = (int64_t)a.n_runs * a.n_bins;
    const unsigned g = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(queue_count_kernel, dim3(g), dim3(256), 0, st, a);
    hipLaunchKernelGGL(queue_order_kernel<false>, dim3(1), dim3(1024), 0, st, a);
    hipLaunchKernelGGL(queue_fill_kernel, dim3(g), dim3(256), 0, st, a);
    return hipGetLastError();
}
