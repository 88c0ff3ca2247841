// reweight.hip -- steady-state reweighting (Sec. II.B.2, Eq. ss), gfx950.
//
// One workgroup per run, launched after the resampling of every iteration;
// it returns at once unless (iteration + 1) is a multiple of the period.
// The flux matrix F[i][j] (weight moved from bin j into bin i, summed from
// the second interval on) is accumulated by the resampling kernel.
//
//   1. W_j = sum_i F[i][j] (ascending i), the weight that started intervals
//      in bin j; the current weight w_i of every bin (its walkers in slot
//      order; the resampled ensemble is bin-major).
//   2. Candidates: bins that are occupied, weigh more than zero and have
//      W_j > 0, in ascending order; the pivot is the one holding the most
//      weight (ties: the lowest bin).
//   3. The pivot's strongly connected component among the candidates, edge
//      j -> i where F[i][j] > 0: forward and backward reachability over
//      64-bit adjacency masks, one wave each (OR-reductions, no barriers).
//   4. Eq. ss on the component, with rates r(a -> b) = F[b][a] / W_a, by
//      state reduction (Grassmann, Taksar and Heyman 1985): states are
//      removed from the highest index down, each time with
//          s_m = sum_{j<m} r(m -> j),  r(i -> j) += r(i -> m) r(m -> j) / s_m,
//      then pi_0 = 1, pi_m = sum_{i<m} pi_i r(i -> m) / s_m.  Every term is
//      non-negative, so there is no cancellation; on a strongly connected
//      set every s_m and pi_m is positive.
//   5. Bin a's walkers are scaled by (pi_a / Z * W_A) / w_a, Z = sum pi,
//      W_A the component's current weight, which it keeps; every other bin
//      is scaled by 1 (exactly unchanged).  Optionally F is cleared, so that
//      the next event sees only the intervals after this one.
// The rate matrix lives in LDS when it fits, else in a per-run global
// scratch.  What bounds an event is the latency of the elimination's steps, one
// after another over the component's states: each step reads its row (one wave)
// and its column (the others) at once and lists the rows with a nonzero entry,
// and the 16 waves update those rows (rates join neighbouring bins, so most
// rows have none).  64 runs of 465 bins take 1.6 ms per event, 32 runs of 80
// bins 110 us; with 4 waves, each testing its share of the rows one load after
// another, and walkers, column sums and bit masks fetched one at a time, it was
// 7.1 ms and 141 us.  Sums over
// lanes use fixed trees, so the result is deterministic (graph replays equal
// eager runs bit for bit).
#include "we_internal.h"

#define RW_THREADS 1024
#define RW_LDS_LIMIT (128 * 1024)

namespace {

__host__ __device__ inline size_t rw_align8(size_t b) { return (b + 7) & ~(size_t)7; }

// Bytes of the small per-run tables: W, w, pi, s, factor (double), candidate
// and component lists and a bin -> candidate map (int32), the two adjacency
// bit matrices (uint64), 4 ints of scalars and the forward and backward
// reach masks (8 words each; n_bins <= 512).
#define RW_MISC_BYTES (16 + 2 * 8 * 8)
__host__ __device__ inline size_t rw_small_bytes(int32_t NB) {
    const size_t nw = (size_t)(NB + 63) / 64;
    return rw_align8(40 * (size_t)NB + 12 * (size_t)NB) + 16 * (size_t)NB * nw + RW_MISC_BYTES;
}

// Sum over the 64 lanes as the butterfly over lane bits 5, 4, 3, 2, 1, 0 adds it
// (every lane gets it): lane halves and rows swapped, then rotations in a
// 16-lane row, which reach the partner of bit 3, and, the lanes 8 apart being
// equal by then, of bit 2.
union RwBits {
    double d;
    uint32_t w[2];
};
template <int CTRL>
__device__ __forceinline__ double rw_dpp(double v) {
    RwBits in, out;
    in.d = v;
    out.w[0] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)in.w[0], CTRL, 0xF, 0xF, false);
    out.w[1] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)in.w[1], CTRL, 0xF, 0xF, false);
    return out.d;
}
__device__ __forceinline__ double rw_wave_sum(double v) {
    RwBits x, y, z;
    x.d = v;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(x.w[k], x.w[k], false, false);
        y.w[k] = r[0];
        z.w[k] = r[1];
    }
    x.d = y.d + z.d;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto r = __builtin_amdgcn_permlane16_swap(x.w[k], x.w[k], false, false);
        y.w[k] = r[0];
        z.w[k] = r[1];
    }
    v = y.d + z.d;
    v = v + rw_dpp<0x128>(v);   // row_ror:8
    v = v + rw_dpp<0x124>(v);   // row_ror:4
    v = v + rw_dpp<0x4E>(v);    // quad_perm [2,3,0,1]
    v = v + rw_dpp<0xB1>(v);    // quad_perm [1,0,3,2]
    return v;
}

__device__ __forceinline__ uint32_t rw_wave_or(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = r[0] | r[1];
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return q[0] | q[1];
}

__device__ __forceinline__ void rw_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave: grows `reach` (nw words over candidate indices) along the rows of
// `adj` (adj[c * nw + word]: the candidates one step from c) until nothing
// changes.  Inlined, so that every access stays an LDS access: a generic
// pointer would turn them into flat accesses, which the wave-level sync does
// not order against the caller's LDS reads.
__device__ __forceinline__ void rw_reach(unsigned long long *reach, const unsigned long long *adj, int32_t nc, int32_t nw,
                         int lane) {
    for (;;) {
        unsigned long long acc[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) acc[w] = 0ull;
        for (int32_t c = lane; c < nc; c += 64) {
            if ((reach[c >> 6] >> (c & 63)) & 1ull) {
#pragma unroll
                for (int w = 0; w < 8; ++w)
                    if (w < nw) acc[w] |= adj[(size_t)c * nw + w];
            }
        }
        bool changed = false;
        unsigned long long nr[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const unsigned long long r = w < nw ? reach[w] : 0ull;
            nr[w] = r | rw_wave_or((uint32_t)acc[w]) | ((unsigned long long)rw_wave_or((uint32_t)(acc[w] >> 32)) << 32);
            changed |= nr[w] != r;
        }
        rw_wave_sync();
#pragma unroll
        for (int w = 0; w < 8; ++w)
            if (w < nw && lane == 0) reach[w] = nr[w];
        rw_wave_sync();
        if (!changed) break;
    }
}

}  // namespace

// RL: the rate matrix in LDS (else in the run's global scratch); a template
// parameter so that the compiler knows the address space of every access.
template <bool RL>
__global__ __launch_bounds__(RW_THREADS) void we_reweight_kernel(SimArgs a, double *__restrict__ w_nxt) {
    extern __shared__ __align__(16) unsigned char lds[];
    const uint32_t iter = *a.iter_dev;
    if ((iter + 1u) % (uint32_t)a.rw_period != 0u) return;
    const int32_t run = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, n_waves = nthr >> 6;
    // one elimination step: the state's row over its sum, the rows with a
    // nonzero entry in its column and those entries, how many, and the row's
    // first nonzero entry
    __shared__ double row_m[WE_RW_MAX_BINS], col_m[WE_RW_MAX_BINS];
    __shared__ int32_t rows_m[WE_RW_MAX_BINS], n_rows[2], row_lo;   // counts by the step's parity
    const int32_t NB = a.n_bins, NW = (NB + 63) >> 6;
    const size_t base = (size_t)run * a.cap;
    const int32_t n = a.n_walk[run];
    const double *__restrict__ F = a.rw_F + (size_t)run * NB * NB;
    const int32_t *__restrict__ bins = a.bin + base;
    double *__restrict__ w = w_nxt + base;

    double *Wc = reinterpret_cast<double *>(lds);   // [NB]
    double *wb = Wc + NB;                             // [NB]
    double *pi = wb + NB;                             // [NB] over the component
    double *sm = pi + NB;                             // [NB] over the component
    double *fac = sm + NB;                            // [NB]
    int32_t *cand = reinterpret_cast<int32_t *>(fac + NB);  // [NB] candidate -> bin
    int32_t *act = cand + NB;                               // [NB] component -> bin
    int32_t *pos = act + NB;                                // [NB] a bin's end, then its walkers
    unsigned long long *succ =
        reinterpret_cast<unsigned long long *>(lds + rw_align8(40 * (size_t)NB + 12 * (size_t)NB));
    unsigned long long *pred = succ + (size_t)NB * NW;
    int32_t *misc = reinterpret_cast<int32_t *>(pred + (size_t)NB * NW);   // 4 ints
    unsigned long long *fw = reinterpret_cast<unsigned long long *>(misc + 4);   // 8 words
    unsigned long long *bw = fw + 8;                                              // 8 words
    double *R = RL ? reinterpret_cast<double *>(lds + rw_small_bytes(NB)) : a.rw_R + (size_t)run * NB * NB;

    // 1. W_j, and where each bin's walkers start and end (act and pos double as
    // these tables)
    for (int32_t j = tid; j < NB; j += nthr) {
        double acc = 0.0;
#pragma unroll 16
        for (int32_t i = 0; i < NB; ++i) acc = acc + F[(size_t)i * NB + j];
        Wc[j] = acc;
        act[j] = 0;
        pos[j] = 0;
        fac[j] = 1.0;
    }
    __syncthreads();
    for (int32_t k = tid; k < n; k += nthr) {
        const int32_t b = bins[k], before = k > 0 ? bins[k - 1] : -1, after = k + 1 < n ? bins[k + 1] : -1;
        if (b != before) act[b] = k;
        if (b != after) pos[b] = k + 1;
    }
    __syncthreads();
    for (int32_t i = tid; i < NB; i += nthr) {
        double acc = 0.0;
        const int32_t k0 = act[i], k1 = pos[i];
#pragma unroll 16
        for (int32_t k = k0; k < k1; ++k) acc = acc + w[k];
        wb[i] = acc;
        pos[i] = k1 - k0;
    }
    __syncthreads();

    // 2. candidates (ascending) and the pivot
    if (wave == 0) {
        int32_t nc = 0;
        for (int32_t c0 = 0; c0 < NB; c0 += 64) {
            const int32_t i = c0 + lane;
            const bool is = i < NB && pos[i] > 0 && wb[i] > 0.0 && Wc[i] > 0.0;
            const unsigned long long m = __ballot(is);
            const int32_t idx = nc + __popcll(m & ((1ull << lane) - 1ull));
            if (is) cand[idx] = i;
            nc += __popcll(m);
        }
        rw_wave_sync();
        double bv = -1.0;
        int32_t bc = INT32_MAX;
        for (int32_t c = lane; c < nc; c += 64) {
            const double v = wb[cand[c]];
            if (v > bv) { bv = v; bc = c; }
        }
        for (int d = 32; d > 0; d >>= 1) {
            const double ov = __shfl_xor(bv, d, 64);
            const int32_t oc = __shfl_xor(bc, d, 64);
            if (ov > bv || (ov == bv && oc < bc)) { bv = ov; bc = oc; }
        }
        if (lane == 0) {
            misc[0] = nc;
            misc[2] = bc;
            misc[3] = 0;
        }
    }
    __syncthreads();
    const int32_t nc = misc[0];
    bool ok = false;
    if (nc >= 2) {
        // 3. adjacency among the candidates, then the pivot's component
        for (size_t t = tid; t < (size_t)nc * NW; t += nthr) {
            succ[t] = 0ull;
            pred[t] = 0ull;
        }
        __syncthreads();
        for (int32_t to = wave; to < nc; to += n_waves) {
            const double *Frow = F + (size_t)cand[to] * NB;
            bool edge[WE_RW_MAX_BINS / 64];
#pragma unroll
            for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q) {
                const int32_t from = 64 * q + lane;
                edge[q] = from < nc && to != from && Frow[cand[min(from, nc - 1)]] > 0.0;
            }
#pragma unroll
            for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q) {
                const unsigned long long m = __ballot(edge[q]);
                if (edge[q]) atomicOr(&succ[(size_t)(64 * q + lane) * NW + (to >> 6)], 1ull << (to & 63));
                if (lane == 0 && q < NW) pred[(size_t)to * NW + q] = m;
            }
        }
        __syncthreads();
        // wave 0 forward, wave 1 backward
        if (wave < 2) {
            const int32_t pv = misc[2];
            unsigned long long *reach = fw + 8 * wave;
            for (int32_t q = lane; q < NW; q += 64) reach[q] = q == (pv >> 6) ? 1ull << (pv & 63) : 0ull;
            rw_wave_sync();
            rw_reach(reach, succ + (size_t)wave * NB * NW, nc, NW, lane);
        }
        __syncthreads();
        if (wave == 0) {
            int32_t na = 0;
            for (int32_t c0 = 0; c0 < nc; c0 += 64) {
                const int32_t c = c0 + lane;
                const bool in = c < nc && ((fw[c >> 6] & bw[c >> 6]) >> (c & 63)) & 1ull;
                const unsigned long long m = __ballot(in);
                if (in) act[na + __popcll(m & ((1ull << lane) - 1ull))] = cand[c];
                na += __popcll(m);
            }
            if (lane == 0) misc[1] = na;
        }
        __syncthreads();
        const int32_t na = misc[1];
        if (na >= 2) {
            // 4. rates on the component, state reduction, back substitution
            for (int32_t to = wave; to < na; to += n_waves) {
                const double *Frow = F + (size_t)act[to] * NB;
                double f[WE_RW_MAX_BINS / 64];
#pragma unroll
                for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q) {
                    const int32_t from = min(64 * q + lane, na - 1);
                    f[q] = 64 * q < na ? Frow[act[from]] : 0.0;
                }
#pragma unroll
                for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q) {
                    const int32_t from = 64 * q + lane;
                    if (from < na) R[(size_t)from * na + to] = from == to ? 0.0 : f[q] / Wc[act[from]];
                }
            }
            if (tid < 2) n_rows[tid] = 0;
            __syncthreads();
            for (int32_t m = na - 1; m >= 1; --m) {
                for (int32_t i0 = wave * 64; i0 < m; i0 += nthr) {
                    const int32_t i = i0 + lane;
                    const double rim = i < m ? R[(size_t)i * na + m] : 0.0;
                    const unsigned long long nz = __ballot(rim != 0.0);
                    int32_t at = 0;
                    if (lane == 0 && nz) at = atomicAdd(&n_rows[m & 1], (int32_t)__popcll(nz));
                    at = __shfl(at, 0, 64) + (int32_t)__popcll(nz & ((1ull << lane) - 1ull));
                    if (rim != 0.0) {
                        rows_m[at] = i;
                        col_m[at] = rim;
                    }
                }
                if (wave == n_waves - 1) {   // the last wave has no part of the column (m < 512)
                    double v[WE_RW_MAX_BINS / 64];
                    double p = 0.0;
                    int32_t lo = m;
#pragma unroll
                    for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q) {
                        const int32_t j = 64 * q + lane;
                        v[q] = j < m ? R[(size_t)m * na + j] : 0.0;
                    }
#pragma unroll
                    for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q) {
                        if (64 * q + lane < m) p = p + v[q];
                        const unsigned long long nz = __ballot(v[q] != 0.0);
                        if (nz) lo = min(lo, 64 * q);
                    }
                    const double s = rw_wave_sum(p);
#pragma unroll
                    for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q)
                        if (64 * q + lane < m) row_m[64 * q + lane] = s > 0.0 ? v[q] / s : v[q];
                    if (lane == 0) {
                        sm[m] = s;
                        row_lo = lo;
                        if (!(s > 0.0)) misc[3] = 1;
                    }
                }
                __syncthreads();
                if (misc[3]) break;
                const int32_t nr = n_rows[m & 1], lo = row_lo;
                if (tid == 0) n_rows[(m & 1) ^ 1] = 0;
                for (int32_t q = wave; q < nr; q += n_waves) {
                    const int32_t i = rows_m[q];
                    const double rim = col_m[q];
                    double *Ri = R + (size_t)i * na;
                    for (int32_t j0 = lo + lane; j0 < m; j0 += 256) {
                        double v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = j0 + 64 * u < m ? Ri[j0 + 64 * u] : 0.0;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int32_t j = j0 + 64 * u;
                            if (j < m && j != i) Ri[j] = v[u] + rim * row_m[j];
                        }
                    }
                }
                __syncthreads();
            }
            if (wave == 0 && !misc[3]) {
                if (lane == 0) pi[0] = 1.0;
                rw_wave_sync();
                bool pos_ok = true;
                // the next state's column is read while this one's sum is formed
                double col[WE_RW_MAX_BINS / 64], nxt[WE_RW_MAX_BINS / 64];
                auto column = [&](int32_t m, double (&c)[WE_RW_MAX_BINS / 64]) {
#pragma unroll
                    for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q) {
                        const int32_t i = 64 * q + lane;
                        c[q] = i < m && m < na ? R[(size_t)i * na + m] : 0.0;
                    }
                };
                column(1, nxt);
                for (int32_t m = 1; m < na; ++m) {
#pragma unroll
                    for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q) col[q] = nxt[q];
                    column(m + 1, nxt);
                    double p = 0.0;
#pragma unroll
                    for (int q = 0; q < WE_RW_MAX_BINS / 64; ++q)
                        if (64 * q + lane < m) p = p + pi[64 * q + lane] * col[q];
                    const double v = rw_wave_sum(p) / sm[m];
                    pos_ok = pos_ok && v > 0.0;
                    if (lane == 0) pi[m] = v;
                    rw_wave_sync();
                }
                if (pos_ok) {
                    double zp = 0.0, wp = 0.0;
                    for (int32_t q = lane; q < na; q += 64) {
                        zp = zp + pi[q];
                        wp = wp + wb[act[q]];
                    }
                    const double Z = rw_wave_sum(zp), WA = rw_wave_sum(wp);
                    for (int32_t q = lane; q < na; q += 64) fac[act[q]] = (pi[q] / Z * WA) / wb[act[q]];
                    if (lane == 0) misc[3] = 2;
                }
            }
            __syncthreads();
            ok = misc[3] == 2;
        }
    }

    // 5. rescale; with rw_reset the flux matrix starts over (every read of
    // it lies before the last barrier)
    if (ok)
        for (int32_t k = tid; k < n; k += nthr) w[k] = w[k] * fac[bins[k]];
    if (a.rw_reset) {
        double *Fw = a.rw_F + (size_t)run * NB * NB;
        for (size_t t = tid; t < (size_t)NB * NB; t += nthr) Fw[t] = 0.0;
    }
    if (tid == 0) a.rw_stat[2 * (size_t)run + (ok ? 0 : 1)] += 1;
}

bool rw_solve_in_lds(int32_t NB) {
    return rw_small_bytes(NB) + 8 * (size_t)NB * NB <= RW_LDS_LIMIT;
}

hipError_t launch_reweight(const SimArgs &a, double *w_nxt, hipStream_t st) {
    const size_t shmem = rw_small_bytes(a.n_bins) + (a.rw_R ? 0 : 8 * (size_t)a.n_bins * a.n_bins);
    if (a.rw_R) hipLaunchKernelGGL(we_reweight_kernel<false>, dim3(a.n_runs), dim3(RW_THREADS), shmem, st, a, w_nxt);
    else hipLaunchKernelGGL(we_reweight_kernel<true>, dim3(a.n_runs), dim3(RW_THREADS), shmem, st, a, w_nxt);
    return hipGetLastError();
}
