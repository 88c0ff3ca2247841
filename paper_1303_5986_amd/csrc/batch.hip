// batch.hip -- many independent WE runs of different networks stepped
// together (gfx950).
//
// Runs are independent (the paper runs independent replicas for its error
// bars, Sec. IV), so a batch is a set of ordinary sims sharing one stream.
// What is batched is the propagation: instead of one SSA launch per run --
// each too small to fill 256 CUs when a run holds a few hundred walkers --
// every kernel variant gets ONE persistent launch whose workgroups pull chunks
// (a member, a run, a range of walker slots) until the list is exhausted.  A
// workgroup copies its chunk's reaction tables to LDS when the member changes
// and its waves then share the chunk's slots:
//   lane variants: 64 slots per wave at a time, one per lane;
//   group variants: 64 / L slots, L lanes each;
//   wave variant:  one slot, one wave.
// Chunks hold about equal work (slots times the work of a walker of their
// network), the networks with the most reactions first, so uneven runs balance
// across the chip.  The bookkeeping is batched the same way: recycle/bin,
// resample (placement by one workgroup per run of every member, then one wave
// per bin), gather, observe and the
// iteration counters are one launch each, with the member index on grid y;
// a member's arguments and buffers are read from device tables.  The whole
// iteration can be captured as a HIP graph (the work counters are cleared
// by a kernel, not a memset, so replays are safe).  Members may record their
// ensembles (eager steps only) and, once a member's committor is trained and
// switched on, bin on it: one batched launch evaluates every such member's
// model after the batched recycle/bin.
//
// Autotuning: every kernel a network fits -- lane (64 walkers per wave),
// group with 32, 16, 8, 4 or 2 walkers per wave, wave (one) -- runs a short
// pilot (one interval with every slot filled, timed with HIP events, best of
// autotune_iters) and the fastest is kept; the choice is cached in a JSON
// file keyed by (species, reactions, walker slots, runs, tau).
#include <algorithm>
#include <cstdio>
#include <fstream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "ssa_group_body.h"
#include "ssa_lane_body.h"
#include "ssa_wave_body.h"
#include "we_internal.h"

namespace {

// V_GROUP_L: the group kernel with L lanes per walker, the tables in LDS;
// V_GROUPR_L: the same for members whose lane blocks hold at most
// BATCH_GROUP_REG reactions (descriptors and propensities in registers);
// V_GROUPG_L: tables read through the cache, for members whose tables take
// more than BATCH_GROUP_TABLES bytes.  The order within a group is L = 2 .. 32.
enum Variant {
    V_LANE_1_4 = 0, V_LANE_2_8, V_LANE_8_16, V_LANE_16_32,
    V_GROUP, V_GROUPR = V_GROUP + 5, V_GROUPG = V_GROUPR + 5,
    V_WAVE = V_GROUPG + 5, V_COUNT
};
#define BATCH_GROUP_REG 8
#define BATCH_GROUP_TABLES (48 * 1024)
#define BATCH_WAVES 8                       // waves per workgroup of the wave variant, at most
// Dynamic LDS of a workgroup, at most: a CU's 160 KB less next_chunk's word, which
// takes a 16-byte unit (the dynamic part starts on 16 bytes).
#define BATCH_LDS (160 * 1024 - 16)
// Species of any member, at most.
#define BATCH_MAX_SPECIES 3968
// The largest wave-variant member (4096 descriptors and a wave's 64 chunk sums
// and counts) leaves room for five waves.
static_assert(16 * 4096 + 5 * (64 * 8 + 4 * (BATCH_MAX_SPECIES + 4)) <= BATCH_LDS, "wave variant");
// Chunk counters per variant, on 128-byte lines of their own: one counter for
// every walker tile bound the launches (an atomic on one address takes 11.4 ns).
// Batch of 64 networks of 8 to 3680 reactions, by chunks with tables in LDS: wave
// leg 706 -> 242 us, the three group legs 457 -> 107 us per step.
#define BATCH_HEADS 8

// Walker slots a workgroup works on at a time.
int32_t slots_per_round(int v, int32_t waves) {
    if (v == V_WAVE) return waves;
    if (v >= V_GROUP) return 4 * (32 >> ((v - V_GROUP) % 5));
    return 256;
}

struct Chunk {
    int32_t sim, run, slot, n;
};

Variant variant_of(const we_sim *s) {
    const int32_t S = s->S, R = s->net->R;
    if (s->kernel == WE_KERNEL_WAVE) return V_WAVE;
    if (s->kernel == WE_KERNEL_GROUP) {
        const bool lds = group_tables_bytes(R, s->args.n_chg) <= BATCH_GROUP_TABLES;
        const bool reg = (R + s->group_lanes - 1) / s->group_lanes <= BATCH_GROUP_REG;
        int32_t l = 0;
        while ((2 << l) < s->group_lanes) ++l;
        return (Variant)((lds ? reg ? V_GROUPR : V_GROUP : V_GROUPG) + l);
    }
    if (S <= 1 && R <= 4) return V_LANE_1_4;
    if (S <= 2 && R <= 8) return V_LANE_2_8;
    if (S <= 8 && R <= 16) return V_LANE_8_16;
    if (S <= 16 && R <= 32) return V_LANE_16_32;
    return V_WAVE;
}

}  // namespace

// The calling workgroup's next chunk, or -1: a static first one, then from its
// counter (block b uses counter b mod BATCH_HEADS; chunks alternate between
// the counters in list order).  Every thread calls it; on the way it waits for
// the workgroup, so the tables in LDS may be replaced afterwards.
__device__ __forceinline__ int32_t next_chunk(int32_t n_chunks, bool first, uint32_t *__restrict__ counters) {
    __shared__ uint32_t got;
    const uint32_t H = min((uint32_t)BATCH_HEADS, gridDim.x), s = blockIdx.x % H;
    uint32_t i = blockIdx.x / H;
    if (!first) {
        __syncthreads();
        if (threadIdx.x == 0) got = atomicAdd(counters + s * WE_HEAD_STRIDE, 1u);
        __syncthreads();
        i = (gridDim.x - s + H - 1) / H + got;
    }
    i = i * H + s;
    return i < (uint32_t)n_chunks ? (int32_t)i : -1;
}

template <int SMAX, int RMAX>
__global__ __launch_bounds__(256) void batch_lane_kernel(const SimArgs *__restrict__ args,
                                                         int32_t *const *__restrict__ xptr,
                                                         const Chunk *__restrict__ chunks, int32_t n_chunks,
                                                         uint32_t *__restrict__ counters) {
    constexpr bool REG = RMAX <= LANE_REG_RMAX;
    constexpr int ROWS = REG ? 1 : RMAX * LaneRow<SMAX>::W;
    __shared__ int32_t rows[4 * ROWS];
    int32_t *wrows = rows + (threadIdx.x >> 6) * ROWS;
    for (bool first = true;; first = false) {
        const int32_t c = next_chunk(n_chunks, first, counters);
        if (c < 0) break;
        const Chunk ch = chunks[c];
        const SimArgs &a = args[ch.sim];
        if constexpr (!REG) lane_stage_rows<SMAX>(a, wrows);
        const int32_t hi = min(ch.slot + ch.n, a.n_walk[ch.run]);
        for (int32_t k = ch.slot + (int32_t)threadIdx.x; k < hi; k += 256)
            lane_walker<SMAX, RMAX>(a, xptr[ch.sim], ch.run, k, *a.iter_dev, wrows);
    }
}

// Wave variant: descriptors in LDS (in the pair form where the member's
// network has it), reaction headers, changes and dependency lists from global
// memory.  Members' walkers fire few events per interval, so the chunk sums
// from scratch at its start, 64 propensities per chunk, weigh most: with the
// descriptors read through the cache, one slot per work item, the leg of the
// 64-network batch took 706 us.
template <class D>
__device__ __forceinline__ void batch_wave_chunk(const SimArgs &a, const D *gdesc, const Chunk &ch, bool stage,
                                                 int32_t *xs, unsigned char *smem, double *lchunk, int32_t *lx) {
    if (stage) {
        const uint4 *gd = reinterpret_cast<const uint4 *>(gdesc);
        uint4 *ld = reinterpret_cast<uint4 *>(smem);
        for (int32_t i = threadIdx.x; i < a.R; i += blockDim.x) ld[i] = gd[i];
        __syncthreads();
    }
    LdsTables<D> tab;
    tab.d = reinterpret_cast<const D *>(smem);
    tab.h = a.rinfo;
    tab.ids = a.dep;
    const uint32_t iter = *a.iter_dev;
    const int32_t hi = min(ch.slot + ch.n, a.n_walk[ch.run]);
    for (int32_t k = ch.slot + (int32_t)(threadIdx.x >> 6); k < hi; k += (int32_t)(blockDim.x >> 6)) {
        wave_walker_t(a, tab, xs, ch.run, k, iter, lchunk, lx);
        __builtin_amdgcn_wave_barrier();
    }
}

__global__ __launch_bounds__(64 * BATCH_WAVES, 4) void batch_wave_kernel(const SimArgs *__restrict__ args,
                                                                       int32_t *const *__restrict__ xptr,
                                                                       const Chunk *__restrict__ chunks, int32_t n_chunks,
                                                                       uint32_t *__restrict__ counters, int32_t s_pad,
                                                                       int32_t tables) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    double *lchunk = reinterpret_cast<double *>(smem + tables) + wv * 64;
    int32_t *lx = reinterpret_cast<int32_t *>(smem + tables + (size_t)nw * 64 * sizeof(double)) + wv * s_pad;
    int32_t staged = -1;
    for (bool first = true;; first = false) {
        const int32_t c = next_chunk(n_chunks, first, counters);
        if (c < 0) break;
        const Chunk ch = chunks[c];
        const SimArgs &a = args[ch.sim];
        if (a.desc2) batch_wave_chunk(a, a.desc2, ch, staged != ch.sim, xptr[ch.sim], smem, lchunk, lx);
        else batch_wave_chunk(a, a.desc, ch, staged != ch.sim, xptr[ch.sim], smem, lchunk, lx);
        staged = ch.sim;
    }
}

// Group variant: 64 / L consecutive slots per wave, one group of L lanes per
// slot; slices of s_max ints (the largest group_slice among the members on
// this variant).  BR > 0: the members' lane blocks hold at most BR reactions,
// kept in registers (group_walker).  LT: the member's tables in LDS.
template <int L, int BR, bool LT, class D>
__device__ __forceinline__ void batch_group_chunk(const SimArgs &a, const D *gdesc, const Chunk &ch, bool stage,
                                                  int32_t *xs, unsigned char *smem, int32_t *lx) {
    constexpr int G = 64 / L;
    GroupTables<D> tb{gdesc, a.chg_ptr, a.chg};
    if constexpr (LT) tb = group_stage(a, gdesc, smem, stage);
    const uint32_t iter = *a.iter_dev;
    const int32_t hi = min(ch.slot + ch.n, a.n_walk[ch.run]);
    for (int32_t k0 = ch.slot + (int32_t)(threadIdx.x >> 6) * G; k0 < hi; k0 += 4 * G) {
        const int32_t k = k0 + (int32_t)(threadIdx.x & 63) / L;
        group_walker<L, BR, D>(a, tb, xs, ch.run, k, k < hi, iter, lx);
    }
}

// BR > 0: three waves a SIMD (167 registers; left to itself the compiler takes 174
// and the longest of these launches goes from 50.4 to 53.7 us).
template <int L, int BR, bool LT>
__global__ __launch_bounds__(256, BR > 0 ? 3 : 1) void batch_group_kernel(const SimArgs *__restrict__ args,
                                                          int32_t *const *__restrict__ xptr,
                                                          const Chunk *__restrict__ chunks, int32_t n_chunks,
                                                          uint32_t *__restrict__ counters, int32_t s_max, int32_t tables) {
    extern __shared__ __align__(16) unsigned char bgsm[];
    constexpr int G = 64 / L;
    int32_t *lx = reinterpret_cast<int32_t *>(bgsm + tables) +
                  ((size_t)(threadIdx.x >> 6) * G + (threadIdx.x & 63) / L) * s_max;
    int32_t staged = -1;
    for (bool first = true;; first = false) {
        const int32_t c = next_chunk(n_chunks, first, counters);
        if (c < 0) break;
        const Chunk ch = chunks[c];
        const SimArgs &a = args[ch.sim];
        if (a.desc2) batch_group_chunk<L, BR, LT>(a, a.desc2, ch, staged != ch.sim, xptr[ch.sim], bgsm, lx);
        else batch_group_chunk<L, BR, LT>(a, a.desc, ch, staged != ch.sim, xptr[ch.sim], bgsm, lx);
        staged = ch.sim;
    }
}

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
struct BatchBins {
    int64_t *first;
    int64_t total;
    int32_t max_blocks;
};
hipError_t launch_batch_bookkeeping(const BatchPtrs &b, int32_t n_sims, int64_t max_slots, int32_t max_runs,
                                    int64_t max_cells, const BatchBins *bins, size_t shmem, bool observe,
                                    const CmBatchModel *models,
                                    int32_t s_max_cm, uint32_t *counters, int32_t n_counters, hipStream_t st);
int32_t batch_bins_cap(const SimArgs &a, int64_t waves);
int64_t batch_big_waves(const SimArgs &a);
int32_t batch_bins_blocks(const SimArgs &a, int64_t waves, int variant);
size_t resample_lds_bytes(const SimArgs &a, bool use_lds);
int32_t resample_place_rows(const SimArgs &a, int64_t blocks);

struct we_batch {
    hipStream_t stream = nullptr;
    ReadStage stage;
    std::vector<we_sim *> sims;
    std::vector<Variant> var;
    // per variant: its chunks, dynamic LDS bytes (tables in front) and workgroups
    int32_t n_chunks[V_COUNT] = {};
    Chunk *d_chunks[V_COUNT] = {};
    size_t shmem[V_COUNT] = {};
    int32_t tables[V_COUNT] = {}, s_max[V_COUNT] = {}, blocks[V_COUNT] = {};
    int32_t wave_waves = BATCH_WAVES;  // waves per workgroup of the wave variant
    uint32_t *d_counters = nullptr;    // [V_COUNT][BATCH_HEADS], WE_HEAD_STRIDE words apart; zero between iterations
    SimArgs *d_args = nullptr;
    int32_t **d_xptr[2] = {nullptr, nullptr};
    double **d_wptr[2] = {nullptr, nullptr};
    int32_t **d_binfo = nullptr;
    int32_t *d_grid_bins = nullptr;
    int64_t max_slots = 0, max_cells = 0;
    int32_t max_runs = 0;
    BatchBins bins[BATCH_BINS] = {};   // split/merge, by variant
    int32_t *d_bins_cap = nullptr;     // each member's
    size_t resample_shmem = 0;
    bool observe = false;
    int32_t iter = 0, max_iters = 0;
    hipGraphExec_t graph_exec = nullptr;
    hipStream_t capture_stream = nullptr;
    int32_t graph_iters = 0;
    bool capturing = false;
    // learned bins: each member's active model as the device tables hold it
    std::vector<CmBatchModel> cm_host, cm_graph;
    std::vector<int32_t> grid_bins_host;
    CmBatchModel *d_models = nullptr;
    int32_t s_max_cm = 0;
    bool any_cm = false;
};

namespace {

// Pilot timing of one kernel choice.  Each of `reps` throw-away sims starts
// with every slot of every run holding a walker at x0 (weight 1 / cap) and
// times its first interval: propagation at full occupancy, the regime a WE
// run spends most of its time near once its bins fill, rather than the
// sparse initial ensemble (a few walkers per run favour the kernels with
// the fewest walkers per wave, which lose once the bins fill).  The fastest
// repetition counts.
we_status pilot_ms(const we_network *net, const we_grid *g, const we_params *p, int32_t kernel,
                   int32_t walkers_per_wave, int32_t reps, hipStream_t st, double *ms) {
    we_params q = *p;
    q.kernel = kernel;
    q.walkers_per_wave = walkers_per_wave;
    q.max_iters = 1;
    q.record_iters = 0;
    q.n_joint = 0;
    q.hist_hi = q.hist_lo - 1;
    *ms = 0.0;
    for (int32_t rep = 0; rep < std::max(reps, 1); ++rep) {
        we_sim *s = nullptr;
        we_status r = we_init(net, g, &q, st, nullptr, 0, &s);
        if (r != WE_OK) return r;
        const int32_t cap = s->cap, S = s->S;
        std::vector<int32_t> xs((size_t)cap * S);
        for (int32_t k = 0; k < cap; ++k) std::copy(p->x0, p->x0 + S, xs.begin() + (size_t)k * S);
        const std::vector<double> ws(cap, 1.0 / cap);
        for (int32_t run = 0; run < s->n_runs && r == WE_OK; ++run)
            r = we_set_ensemble(s, run, cap, xs.data(), ws.data());
        hipEvent_t e0 = nullptr, e1 = nullptr;
        float t = 0.f;
        if (r == WE_OK && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
            r = we_fail(WE_EDEVICE, "hipEventCreate failed");
        if (r == WE_OK && hipEventRecord(e0, st) != hipSuccess) r = we_fail(WE_EDEVICE, "hipEventRecord failed");
        if (r == WE_OK) r = we_step_intervals(s, 1);
        if (r == WE_OK && (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                           hipEventElapsedTime(&t, e0, e1) != hipSuccess))
            r = we_fail(WE_EDEVICE, "pilot timing failed");
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        if (r == WE_OK) r = we_synchronize(s);
        we_destroy(s);
        if (r != WE_OK) return r;
        if (rep == 0 || t < *ms) *ms = t;
    }
    return WE_OK;
}

std::map<std::string, int> read_cache(const char *path) {
    std::map<std::string, int> m;
    if (!path || !*path) return m;
    std::ifstream f(path);
    if (!f) return m;
    std::stringstream ss;
    ss << f.rdbuf();
    const std::string t = ss.str();
    // flat object of "key": value pairs
    size_t pos = 0;
    while ((pos = t.find('"', pos)) != std::string::npos) {
        const size_t end = t.find('"', pos + 1);
        if (end == std::string::npos) break;
        const std::string key = t.substr(pos + 1, end - pos - 1);
        const size_t colon = t.find(':', end);
        if (colon == std::string::npos) break;
        m[key] = std::atoi(t.c_str() + colon + 1);
        pos = t.find_first_of(",}", colon);
        if (pos == std::string::npos) break;
    }
    return m;
}

void write_cache(const char *path, const std::map<std::string, int> &m) {
    if (!path || !*path) return;
    std::ofstream f(path);
    f << "{";
    bool first = true;
    for (const auto &kv : m) {
        f << (first ? "" : ",") << "\n  \"" << kv.first << "\": " << kv.second;
        first = false;
    }
    f << "\n}\n";
}

// Work of one walker of a member, in units of a wave's time: the chunk sums (or
// the lane blocks) it evaluates and a constant for the rest.
double walker_cost(int v, const we_sim *s) {
    if (v == V_WAVE) return s->net->R / 64.0 + 16.0;
    if (v >= V_GROUP) return (double)((s->net->R + s->group_lanes - 1) / s->group_lanes) + 8.0;
    return s->net->R + 8.0;
}

using ChunkKernel = void (*)(const SimArgs *, int32_t *const *, const Chunk *, int32_t, uint32_t *);
using TableKernel = void (*)(const SimArgs *, int32_t *const *, const Chunk *, int32_t, uint32_t *, int32_t, int32_t);

ChunkKernel lane_kernel_of(int v) {
    return v == V_LANE_1_4 ? batch_lane_kernel<1, 4> : v == V_LANE_2_8 ? batch_lane_kernel<2, 8>
           : v == V_LANE_8_16 ? batch_lane_kernel<8, 16> : batch_lane_kernel<16, 32>;
}

template <int BR, bool LT>
TableKernel group_kernel_of(int l) {
    return l == 0 ? batch_group_kernel<2, BR, LT> : l == 1 ? batch_group_kernel<4, BR, LT>
           : l == 2 ? batch_group_kernel<8, BR, LT> : l == 3 ? batch_group_kernel<16, BR, LT>
                                                             : batch_group_kernel<32, BR, LT>;
}

TableKernel table_kernel_of(int v) {
    if (v == V_WAVE) return batch_wave_kernel;
    const int l = (v - V_GROUP) % 5;
    return v < V_GROUPR ? group_kernel_of<0, true>(l) : v < V_GROUPG ? group_kernel_of<BATCH_GROUP_REG, true>(l)
                                                                      : group_kernel_of<0, false>(l);
}

// The variants' LDS, workgroups and chunk lists.  About BATCH_CHUNKS chunks of
// equal work per resident workgroup: enough to balance, few enough that the
// tables are copied and the waves of a workgroup waited for seldom.
#define BATCH_CHUNKS 4
we_status build_chunks(we_batch *b) {
    int dev = 0, cus = 1;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    for (int v = 0; v < V_COUNT; ++v) {
        std::vector<int32_t> of;       // members, most reactions first
        for (size_t i = 0; i < b->sims.size(); ++i)
            if (b->var[i] == v) of.push_back((int32_t)i);
        if (of.empty()) continue;
        std::stable_sort(of.begin(), of.end(), [&](int32_t x, int32_t y) { return b->sims[x]->net->R > b->sims[y]->net->R; });
        int threads = 256;
        if (v >= V_GROUP) {
            for (int32_t i : of) {
                const we_sim *s = b->sims[i];
                const size_t t = v == V_WAVE ? 16 * (size_t)s->net->R
                                 : v < V_GROUPG ? group_tables_bytes(s->net->R, s->args.n_chg) : 0;
                b->tables[v] = std::max(b->tables[v], (int32_t)((t + 15) & ~(size_t)15));
                b->s_max[v] = std::max(b->s_max[v], v == V_WAVE ? (s->S + 4) & ~3 : group_slice(s->S));
            }
            if (v == V_WAVE) {
                const size_t per = 64 * sizeof(double) + sizeof(int32_t) * (size_t)b->s_max[v];
                b->wave_waves = (int32_t)std::min<size_t>(BATCH_WAVES, (BATCH_LDS - b->tables[v]) / per);
                b->shmem[v] = b->tables[v] + b->wave_waves * per;
                threads = 64 * b->wave_waves;
            } else {
                b->shmem[v] = b->tables[v] + sizeof(int32_t) * (size_t)slots_per_round(v, 0) * b->s_max[v];
            }
        }
        const int32_t round = slots_per_round(v, b->wave_waves);
        int per_cu = 0;
        const void *fn = v < V_GROUP ? (const void *)lane_kernel_of(v) : (const void *)table_kernel_of(v);
        HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, b->shmem[v]));
        if (per_cu < 1) return we_fail(WE_EINVAL, "a batched propagation kernel's workgroup does not fit a CU");
        double total = 0.0;
        for (int32_t i : of) total += walker_cost(v, b->sims[i]) * b->sims[i]->n_runs * b->sims[i]->cap;
        const double aim = total / ((double)BATCH_CHUNKS * per_cu * cus);
        std::vector<Chunk> ch;
        for (int32_t i : of) {
            const we_sim *s = b->sims[i];
            const int32_t n = (int32_t)std::max(1.0, std::min(aim / walker_cost(v, s) / round, 1e6)) * round;
            for (int32_t r = 0; r < s->n_runs; ++r)
                for (int32_t k = 0; k < s->cap; k += n) ch.push_back(Chunk{i, r, k, std::min(n, s->cap - k)});
        }
        b->n_chunks[v] = (int32_t)ch.size();
        b->blocks[v] = (int32_t)std::min<int64_t>(b->n_chunks[v], (int64_t)per_cu * cus);
        HIP_TRY(hipMalloc(&b->d_chunks[v], sizeof(Chunk) * ch.size()));
        HIP_TRY(hipMemcpy(b->d_chunks[v], ch.data(), sizeof(Chunk) * ch.size(), hipMemcpyHostToDevice));
    }
    return WE_OK;
}

bool same_models(const std::vector<CmBatchModel> &x, const std::vector<CmBatchModel> &y) {
    if (x.size() != y.size()) return false;
    for (size_t i = 0; i < x.size(); ++i)
        if (x[i].params != y[i].params || x[i].wt != y[i].wt || x[i].feat != y[i].feat || x[i].qedges != y[i].qedges)
            return false;
    return true;
}

std::vector<CmBatchModel> current_models(const we_batch *b) {
    std::vector<CmBatchModel> m;
    for (const we_sim *s : b->sims) m.push_back(committor_batch_model(s));
    return m;
}

// Bring the device tables of learned bins up to date with the members'
// committors (trained and switched on since the last iteration, or off).
we_status refresh_models(we_batch *b) {
    std::vector<CmBatchModel> m = current_models(b);
    if (same_models(m, b->cm_host)) return WE_OK;
    HIP_TRY(hipStreamSynchronize(b->stream));
    b->any_cm = false;
    b->s_max_cm = 0;
    for (size_t i = 0; i < m.size(); ++i) {
        const bool on = m[i].params != nullptr;
        b->grid_bins_host[i] = on ? 0 : 1;
        if (on) {
            b->any_cm = true;
            b->s_max_cm = std::max(b->s_max_cm, b->sims[i]->S);
        }
    }
    HIP_TRY(hipMemcpy(b->d_models, m.data(), sizeof(CmBatchModel) * m.size(), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(b->d_grid_bins, b->grid_bins_host.data(), sizeof(int32_t) * m.size(), hipMemcpyHostToDevice));
    b->cm_host = m;
    return WE_OK;
}

we_status launch_batch_iteration(we_batch *b, hipStream_t st, bool capture) {
    if (!capture) {
        we_status r = refresh_models(b);
        if (r != WE_OK) return r;
    }
    const int32_t parity = b->sims[0]->cur;
    int32_t *const *xp = b->d_xptr[parity];
    for (int v = 0; v < V_COUNT; ++v) {
        if (b->n_chunks[v] == 0) continue;
        const dim3 grid((unsigned)b->blocks[v]);
        uint32_t *cnt = b->d_counters + (size_t)v * BATCH_HEADS * WE_HEAD_STRIDE;
        if (v < V_GROUP)
            hipLaunchKernelGGL(lane_kernel_of(v), grid, dim3(256), 0, st, b->d_args, xp, b->d_chunks[v], b->n_chunks[v], cnt);
        else
            hipLaunchKernelGGL(table_kernel_of(v), grid, dim3(v == V_WAVE ? 64 * b->wave_waves : 256), b->shmem[v], st,
                               b->d_args, xp, b->d_chunks[v], b->n_chunks[v], cnt, b->s_max[v], b->tables[v]);
        HIP_TRY(hipGetLastError());
    }
    // recycle/bin, committor bins where active, resample, gather, observe,
    // advance: one launch per step for all members
    BatchPtrs bp{b->d_args, b->d_xptr[parity], b->d_xptr[1 - parity],
                 (const double *const *)b->d_wptr[parity], b->d_wptr[1 - parity], b->d_binfo,
                 b->d_grid_bins, b->d_bins_cap};
    HIP_TRY(launch_batch_bookkeeping(bp, (int32_t)b->sims.size(), b->max_slots, b->max_runs, b->max_cells,
                                     b->bins, b->resample_shmem, b->observe, b->any_cm ? b->d_models : nullptr,
                                     b->s_max_cm, b->d_counters, V_COUNT * BATCH_HEADS, st));
    for (we_sim *s : b->sims) s->cur = 1 - s->cur;
    if (!capture)
        for (we_sim *s : b->sims) HIP_TRY(committor_record(s, st));
    return WE_OK;
}

bool recording(const we_batch *b) {
    for (const we_sim *s : b->sims)
        if (s->rec.cap_iters > 0 && s->rec.n_iters < s->rec.cap_iters) return true;
    return false;
}

}  // namespace

extern "C" we_status we_batch_create(int32_t n, const we_network *const *nets, const we_grid *grids,
                                     const we_params *params, void *hip_stream, int32_t autotune_iters,
                                     const char *cache_path, we_batch **out) {
    if (!out || n <= 0 || !nets || !grids || !params) return we_fail(WE_EINVAL, "bad arguments");
    *out = nullptr;
    we_batch *b = new we_batch();
    b->stream = (hipStream_t)hip_stream;
    std::map<std::string, int> cache = read_cache(cache_path);
    bool cache_dirty = false;
    int32_t s_most = 0;
    for (int32_t i = 0; i < n; ++i) {
        we_params p = params[i];
        if (p.rw_period > 0) {
            we_batch_destroy(b);
            return we_fail(WE_EINVAL, "reweighting is not supported inside a batch");
        }
        if (p.engine != 0) {
            we_batch_destroy(b);
            return we_fail(WE_EINVAL, "tau-leaping is not supported inside a batch");
        }
        if (!nets[i]->hill.empty()) {
            we_batch_destroy(b);
            return we_fail(WE_EINVAL, "Hill-type rates are not supported inside a batch");
        }
        const int32_t S = nets[i]->S, R = nets[i]->R;
        if (p.kernel == WE_KERNEL_AUTO) {
            const bool lane_ok = lane_kernel_fits(S, R, nets[i]->max_delta);
            if (autotune_iters > 0) {
                char key[128];
                std::snprintf(key, sizeof key, "S%d_R%d_cap%d_runs%d_tau%g", S, R, p.m_targ * grids[i].n_bins,
                              p.n_runs, p.tau);
                auto it = cache.find(key);
                if (it != cache.end()) {
                    // value: kernel + 16 * walkers per wave (group kernel)
                    p.kernel = it->second % 16;
                    p.walkers_per_wave = it->second / 16;
                } else {
                    std::vector<std::pair<int32_t, int32_t>> cand;
                    if (lane_ok) cand.push_back({WE_KERNEL_LANE, 0});
                    for (int32_t wpw : {32, 16, 8, 4, 2})
                        if (group_kernel_fits(S, R, 64 / wpw)) cand.push_back({WE_KERNEL_GROUP, wpw});
                    if (wave_kernel_fits(S, R) && nets[i]->max_chg <= 64) cand.push_back({WE_KERNEL_WAVE, 0});
                    double best = 0.0;
                    for (size_t c = 0; c < cand.size(); ++c) {
                        double t = 0.0;
                        we_status r = pilot_ms(nets[i], &grids[i], &p, cand[c].first, cand[c].second, autotune_iters,
                                               b->stream, &t);
                        if (r != WE_OK) { we_batch_destroy(b); return r; }
                        if (c == 0 || t < best) {
                            best = t;
                            p.kernel = cand[c].first;
                            p.walkers_per_wave = cand[c].second;
                        }
                    }
                    cache[key] = p.kernel + 16 * p.walkers_per_wave;
                    cache_dirty = true;
                }
            } else {
                p.kernel = (lane_ok && R <= 32) ? WE_KERNEL_LANE : WE_KERNEL_WAVE;
            }
        }
        we_sim *s = nullptr;
        we_status r = we_init(nets[i], &grids[i], &p, b->stream, nullptr, 0, &s);
        if (r != WE_OK) { we_batch_destroy(b); return r; }
        s->stage = &b->stage;
        b->sims.push_back(s);
        b->var.push_back(variant_of(s));
        s_most = std::max(s_most, S);
        b->max_iters = (i == 0) ? s->max_iters : std::min(b->max_iters, s->max_iters);
    }
    if (cache_dirty) write_cache(cache_path, cache);
    if (s_most > BATCH_MAX_SPECIES) {
        we_batch_destroy(b);
        return we_fail(WE_EINVAL, "species count too large for the batched wave kernel");
    }
    std::vector<SimArgs> args;
    std::vector<int32_t *> xp0, xp1;
    std::vector<double *> wp0, wp1;
    std::vector<int32_t *> binfo;
    std::vector<int32_t> grid_bins;
    int32_t runs_hi = 0;
    for (we_sim *s : b->sims) runs_hi = std::max(runs_hi, s->n_runs);
    for (we_sim *s : b->sims) {
        args.push_back(s->args);
        args.back().queue_stats = 0;   // the batched kernels keep their own work queue
        // cursor rows for the batched launch's block size
        args.back().place_rows = resample_place_rows(s->args, (int64_t)runs_hi * (int64_t)b->sims.size());
        xp0.push_back(s->x[0]);
        xp1.push_back(s->x[1]);
        wp0.push_back(s->w[0]);
        wp1.push_back(s->w[1]);
        binfo.push_back(s->rs_binfo);
        grid_bins.push_back(1);
        b->resample_shmem = std::max(b->resample_shmem, resample_lds_bytes(args.back(), false));
        b->max_slots = std::max<int64_t>(b->max_slots, (int64_t)s->n_runs * s->cap);
        b->max_cells = std::max<int64_t>(b->max_cells, (int64_t)s->n_runs * s->cap * s->S);
        b->max_runs = std::max(b->max_runs, s->n_runs);
        b->observe = b->observe || s->args.nh > 0 || s->args.n_joint > 0;
    }
    int64_t big_waves = 0;
    for (we_sim *s : b->sims) big_waves += batch_big_waves(s->args);
    std::vector<int32_t> caps;
    for (we_sim *s : b->sims) caps.push_back(batch_bins_cap(s->args, big_waves));
    HIP_TRY(hipMalloc(&b->d_bins_cap, sizeof(int32_t) * n));
    HIP_TRY(hipMemcpy(b->d_bins_cap, caps.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice));
    for (int v = 0; v < BATCH_BINS; ++v) {
        BatchBins &bb = b->bins[v];
        std::vector<int64_t> first(1, 0);
        for (we_sim *s : b->sims) {
            const int32_t blocks = batch_bins_blocks(s->args, big_waves, v);
            first.push_back(first.back() + (int64_t)s->n_runs * blocks);
            bb.max_blocks = std::max(bb.max_blocks, blocks);
        }
        bb.total = first.back();
        HIP_TRY(hipMalloc(&bb.first, sizeof(int64_t) * first.size()));
        HIP_TRY(hipMemcpy(bb.first, first.data(), sizeof(int64_t) * first.size(), hipMemcpyHostToDevice));
    }
    HIP_TRY(hipMalloc(&b->d_wptr[0], sizeof(double *) * n));
    HIP_TRY(hipMalloc(&b->d_wptr[1], sizeof(double *) * n));
    HIP_TRY(hipMemcpy(b->d_wptr[0], wp0.data(), sizeof(double *) * n, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(b->d_wptr[1], wp1.data(), sizeof(double *) * n, hipMemcpyHostToDevice));
    HIP_TRY(hipMalloc(&b->d_models, sizeof(CmBatchModel) * n));
    b->cm_host.assign(n, CmBatchModel{});
    b->grid_bins_host.assign(n, 1);
    HIP_TRY(hipMemcpy(b->d_models, b->cm_host.data(), sizeof(CmBatchModel) * n, hipMemcpyHostToDevice));
    HIP_TRY(hipMalloc(&b->d_binfo, sizeof(int32_t *) * n));
    HIP_TRY(hipMalloc(&b->d_grid_bins, sizeof(int32_t) * n));
    HIP_TRY(hipMemcpy(b->d_binfo, binfo.data(), sizeof(int32_t *) * n, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(b->d_grid_bins, grid_bins.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice));
    HIP_TRY(hipMalloc(&b->d_args, sizeof(SimArgs) * n));
    HIP_TRY(hipMemcpy(b->d_args, args.data(), sizeof(SimArgs) * n, hipMemcpyHostToDevice));
    HIP_TRY(hipMalloc(&b->d_xptr[0], sizeof(int32_t *) * n));
    HIP_TRY(hipMalloc(&b->d_xptr[1], sizeof(int32_t *) * n));
    HIP_TRY(hipMemcpy(b->d_xptr[0], xp0.data(), sizeof(int32_t *) * n, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(b->d_xptr[1], xp1.data(), sizeof(int32_t *) * n, hipMemcpyHostToDevice));
    HIP_TRY(hipMalloc(&b->d_counters, sizeof(uint32_t) * V_COUNT * BATCH_HEADS * WE_HEAD_STRIDE));
    HIP_TRY(hipMemset(b->d_counters, 0, sizeof(uint32_t) * V_COUNT * BATCH_HEADS * WE_HEAD_STRIDE));
    HIP_TRY(hipDeviceSynchronize());
    we_status r = build_chunks(b);
    if (r != WE_OK) { we_batch_destroy(b); return r; }
    *out = b;
    return WE_OK;
}

extern "C" we_status we_batch_step(we_batch *b, int32_t n) {
    if (!b) return we_fail(WE_EINVAL, "NULL batch");
    if (n < 0 || (int64_t)b->iter + n > b->max_iters) return we_fail(WE_ECAPACITY, "max_iters exceeded");
    for (int32_t i = 0; i < n; ++i) {
        we_status r = launch_batch_iteration(b, b->stream, false);
        if (r != WE_OK) return r;
        b->iter += 1;
        for (we_sim *s : b->sims) {
            s->iter += 1;
            if (s->args.nh > 0) s->hist_iters += 1;
        }
    }
    return WE_OK;
}

extern "C" we_status we_batch_graph_capture(we_batch *b, int32_t n) {
    if (!b) return we_fail(WE_EINVAL, "NULL batch");
    if (n <= 0 || (n & 1)) return we_fail(WE_EINVAL, "capture an even, positive number of iterations");
    if (b->graph_exec) { (void)hipGraphExecDestroy(b->graph_exec); b->graph_exec = nullptr; }
    if (!b->capture_stream) HIP_TRY(hipStreamCreateWithFlags(&b->capture_stream, hipStreamNonBlocking));
    HIP_TRY(hipStreamSynchronize(b->stream));
    if (recording(b)) return we_fail(WE_ESTATE, "a member is recording: step eagerly until its record buffer is full");
    {
        we_status r = refresh_models(b);
        if (r != WE_OK) return r;
    }
    std::vector<int32_t> cur0;
    for (we_sim *s : b->sims) { cur0.push_back(s->cur); s->capturing = true; }
    HIP_TRY(hipStreamBeginCapture(b->capture_stream, hipStreamCaptureModeThreadLocal));
    we_status r = WE_OK;
    for (int32_t i = 0; i < n && r == WE_OK; ++i) r = launch_batch_iteration(b, b->capture_stream, true);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(b->capture_stream, &g);
    for (size_t i = 0; i < b->sims.size(); ++i) { b->sims[i]->cur = cur0[i]; b->sims[i]->capturing = false; }
    if (r != WE_OK) { if (g) (void)hipGraphDestroy(g); return r; }
    if (e != hipSuccess) return we_hip_fail(e, "hipStreamEndCapture");
    e = hipGraphInstantiate(&b->graph_exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) return we_hip_fail(e, "hipGraphInstantiate");
    b->graph_iters = n;
    b->cm_graph = b->cm_host;
    return WE_OK;
}

extern "C" we_status we_batch_graph_replay(we_batch *b, int32_t times) {
    if (!b) return we_fail(WE_EINVAL, "NULL batch");
    if (!b->graph_exec) return we_fail(WE_ESTATE, "no captured graph");
    if (times < 0 || (int64_t)b->iter + (int64_t)times * b->graph_iters > b->max_iters)
        return we_fail(WE_ECAPACITY, "max_iters exceeded");
    if (!same_models(current_models(b), b->cm_graph))
        return we_fail(WE_ESTATE, "a member's bins changed since the capture: capture again");
    for (int32_t t = 0; t < times; ++t) {
        HIP_TRY(hipGraphLaunch(b->graph_exec, b->stream));
        b->iter += b->graph_iters;
        for (we_sim *s : b->sims) {
            s->iter += b->graph_iters;
            if (s->args.nh > 0) s->hist_iters += b->graph_iters;
        }
    }
    return WE_OK;
}

extern "C" we_sim *we_batch_sim(we_batch *b, int32_t i) {
    if (!b || i < 0 || i >= (int32_t)b->sims.size()) return nullptr;
    return b->sims[i];
}

extern "C" we_status we_batch_info(we_batch *b, int32_t *n_sims, int32_t *kernels, int32_t *walkers_per_wave) {
    if (!b) return we_fail(WE_EINVAL, "NULL batch");
    if (n_sims) *n_sims = (int32_t)b->sims.size();
    for (size_t i = 0; i < b->sims.size(); ++i) {
        const we_sim *s = b->sims[i];
        if (kernels) kernels[i] = s->kernel;
        if (walkers_per_wave)
            walkers_per_wave[i] = s->kernel == WE_KERNEL_GROUP ? 64 / s->group_lanes
                                  : s->kernel == WE_KERNEL_WAVE ? 1 : 64;
    }
    return WE_OK;
}

extern "C" void we_batch_destroy(we_batch *b) {
    if (!b) return;
    if (b->stream) (void)hipStreamSynchronize(b->stream);
    for (we_sim *s : b->sims) we_destroy(s);
    for (int v = 0; v < V_COUNT; ++v) (void)hipFree(b->d_chunks[v]);
    (void)hipFree(b->d_counters);
    (void)hipFree(b->d_args);
    (void)hipFree(b->d_xptr[0]);
    (void)hipFree(b->d_xptr[1]);
    (void)hipFree(b->d_wptr[0]);
    (void)hipFree(b->d_wptr[1]);
    (void)hipFree(b->d_binfo);
    for (BatchBins &bb : b->bins) (void)hipFree(bb.first);
    (void)hipFree(b->d_bins_cap);
    (void)hipFree(b->d_grid_bins);
    (void)hipFree(b->d_models);
    if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
    if (b->capture_stream) (void)hipStreamDestroy(b->capture_stream);
    delete b;
}
