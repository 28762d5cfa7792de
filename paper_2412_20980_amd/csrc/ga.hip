// Genetic operators on the device (Section III-B): initial population (eq. 2),
// tournament selection, positional crossover (eq. 3-6) with duplicate repair,
// swap mutation (eq. 7-9) and elitism (eq. 10-11).
//
// One workgroup builds one individual.  Its membership bit set over the nodes
// lives in LDS while the row is built; the finished row is written out sorted
// for the fitness kernels.  Every random decision is a Philox draw keyed by
// (seed, generation, individual, slot), so the result is a pure function of
// the seed and does not depend on the launch geometry.  The parts that are
// sequential by definition (rejection draws that depend on the current
// membership, in ascending slot order) are resolved by one wave over LDS only;
// repairs' first-attempt draws are computed by the whole block beforehand.
//
// A launch serves one GA or a batch of independent GAs (one per instance
// graph): blockIdx.y selects the instance, whose sizes, seed and buffer
// offsets come from a device table, so every instance follows exactly the
// rules (and draws) of a GA run alone.  The generation number is read from
// device memory, which lets a whole generation be captured once and replayed.
#include <algorithm>
#include <climits>

#include "operators.h"

namespace gapa {
namespace {

constexpr int kOpBlock = 512;  // threads of an operator block, at most

// Initial individual i (eq. 2): slot j takes the first INIT draw that is not
// already in the row; the row is then sorted.
__global__ __launch_bounds__(kOpBlock) void k_init(OpArgs args)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const Op a = resolve(args);
    const int32_t i = blockIdx.x;
    if (i >= a.P) return;
    __shared__ OpSums sm;
    const OpLds l = carve(smem, a);
    clear_lds(l, a);
    __syncthreads();
    if (threadIdx.x < 64) wave_draw_in_order(l, a, nullptr, a.k, false, i, 0, kStreamInit);
    emit(l, a, sm, i);
}

__global__ __launch_bounds__(kOpBlock, 8) void k_offspring(OpArgs args)
{
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ OpSums sm;
    const Op a = resolve(args);
    const int32_t o = blockIdx.x;
    if (o >= a.L) return;
    make_child(carve(smem, a), a, sm, o, *args.gen_ctr + 1u, [&](int32_t p) { return a.pop + (int64_t)p * a.k; });
}

// Fitness of every slot from the pass's MCN (GAPA_MINIMISE_MCN).
__global__ void k_mcn_objective(const int32_t *__restrict__ mcn, int64_t *__restrict__ fit, int32_t count)
{
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) fit[i] = mcn[i];
}

// Elitism (eq. 10-11) as a merge by ranks, per instance (blockIdx.y).
// Keys: parents (PC, tag r) for the npar rows already ordered by (PC, tag),
// pooled offspring (PC, tag npar + o) for o = pool[q] (q < npool; pool NULL:
// o = q).  At generation 0 there are no parents and the P initial
// individuals are the pool.  A key's output position is the number of keys
// smaller in (PC, tag) order: the pooled offspring below it plus the
// parents below it (they are sorted: its own index, or a binary search for
// an offspring).  The first P positions are written.
//
// A block takes kRankKeys keys.  Each of its waves holds a 64-entry slice of
// the pool, one entry per lane, and compares it with one key at a time: a
// ballot and a bit count give the slice's entries below the key.  The waves'
// counts meet in LDS, and the block places its keys and copies their rows in
// the same launch, kRowLanes threads a row.  At P = lambda = 1024, k = 2000 the
// ranks take 5.7 us with 8 keys a block (6.9 with 16, 11.8 with 64: the keys'
// loop is a chain of LDS reads; more blocks share it); the row copies in a
// launch of their own took 5.2 us more, and at n = 200 (P = 32, k = 10) 3.9 us
// after 4.6.
// Slower: counting the parents by ballot too, and the comparison loop
// written without branches, eight keys a batch.
struct RankArgs {
    const GaInst *inst;
    const int64_t *f_par;   // current fitness (instance base fit_off)
    const int64_t *f_pool;  // pooled offspring fitness (instance base slot_off)
    const int32_t *pool;    // NULL, or [npool] offspring of each pooled entry (one instance)
    int32_t npool;          // with pool
    int32_t init;           // generation 0: no parents
    int64_t *f_out;         // next fitness (instance base fit_off)
    const int32_t *parents;   // rows of the current population (instance base pop_off)
    const int32_t *children;  // rows of the offspring (instance base child_off)
    int32_t *rows_out;        // rows of the next population (instance base pop_off)
    uint32_t *gen_ctr;        // [1] advanced by gens after generation 0
    uint32_t gens;
};

struct RankView {
    const int64_t *f_par, *f_pool;
    int32_t npar, npool;
};

__device__ __forceinline__ RankView rank_view(const RankArgs &a, int32_t b)
{
    const GaInst &I = a.inst[b];
    RankView v;
    v.npar = a.init ? 0 : I.P;
    v.npool = a.init ? I.P : (a.pool ? a.npool : I.L);
    v.f_par = a.f_par + I.fit_off;
    v.f_pool = a.f_pool + I.slot_off;
    return v;
}

constexpr int kRankKeys = 8;    // keys per block
constexpr int kRankWaves = 16;  // waves per block
constexpr int kRowLanes = 64 * kRankWaves / kRankKeys;

__global__ __launch_bounds__(64 * kRankWaves) void k_rank_rows(RankArgs a)
{
    __shared__ int64_t kf[kRankKeys];
    __shared__ int32_t kt[kRankKeys], kc[kRankKeys];
    __shared__ int32_t s_to[kRankKeys], s_tag[kRankKeys];  // position (or P and beyond: dropped) and source of each key
    const GaInst &I = a.inst[blockIdx.y];
    const RankView r = rank_view(a, blockIdx.y);
    const int32_t total = r.npar + r.npool;
    const int32_t k0 = blockIdx.x * kRankKeys;
    // (every reader of the counter in this generation has finished: stream order)
    if (!a.init && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) a.gen_ctr[0] += a.gens;
    if (k0 >= total) return;  // uniform over the block
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (threadIdx.x < kRankKeys) {
        const int32_t t = k0 + threadIdx.x;
        int64_t f = INT64_MAX;
        int32_t tag = INT_MAX;
        if (t < total) {
            f = t < r.npar ? r.f_par[t] : r.f_pool[t - r.npar];
            tag = t < r.npar ? -1 : (a.pool ? a.pool[t - r.npar] : t - r.npar);
        }
        kf[threadIdx.x] = f;
        kt[threadIdx.x] = tag;
        kc[threadIdx.x] = 0;
    }
    __syncthreads();
    int32_t mine = 0;
    for (int32_t q0 = wv * 64; q0 < r.npool; q0 += 64 * kRankWaves) {
        const int32_t q = q0 + lane;
        const bool in = q < r.npool;
        const int64_t g = in ? r.f_pool[q] : 0;
        const int32_t gt = in ? (a.pool ? a.pool[q] : q) : 0;
#pragma unroll 8
        for (int k = 0; k < kRankKeys; ++k) {
            const int64_t f = kf[k];
            const int32_t tag = kt[k];
            const int32_t c = __popcll(__ballot(in && (g < f || (g == f && gt < tag))));
            mine += lane == k ? c : 0;
        }
    }
    if (mine) atomicAdd(&kc[lane], mine);
    __syncthreads();
    if (threadIdx.x < kRankKeys) {
        const int32_t t = k0 + threadIdx.x;
        int32_t p = INT_MAX, tag = 0;
        if (t < total) {
            const int64_t f = kf[threadIdx.x];
            p = kc[threadIdx.x];
            if (t < r.npar) {
                p += t;
                tag = t;
            } else {
                int32_t lo = 0, hi = r.npar;
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (r.f_par[mid] <= f) lo = mid + 1;
                    else hi = mid;
                }
                p += lo;
                tag = r.npar + kt[threadIdx.x];
            }
            if (p < I.P) a.f_out[I.fit_off + p] = f;
        }
        s_to[threadIdx.x] = p;
        s_tag[threadIdx.x] = tag;
    }
    __syncthreads();
    const int32_t q = threadIdx.x / kRowLanes, p = s_to[q], tag = s_tag[q], k = I.k;
    if (p >= I.P) return;
    const int32_t *s = tag < r.npar ? a.parents + I.pop_off + (int64_t)tag * k
                                    : a.children + I.child_off + (int64_t)(tag - r.npar) * k;
    int32_t *d = a.rows_out + I.pop_off + (int64_t)p * k;
    if (((reinterpret_cast<uintptr_t>(s) | reinterpret_cast<uintptr_t>(d) | (uintptr_t)k * 4) & 15) == 0) {
        for (int32_t j = threadIdx.x % kRowLanes; j < k / 4; j += kRowLanes)
            reinterpret_cast<int4 *>(d)[j] = reinterpret_cast<const int4 *>(s)[j];
    } else {
        for (int32_t j = threadIdx.x % kRowLanes; j < k; j += kRowLanes) d[j] = s[j];
    }
}

}  // namespace

int ga_rank_and_gather(gapa_ga *ga, bool init, const int64_t *f_pool, const int32_t *pool, int32_t npool,
                       hipStream_t s, int32_t gens)
{
    const int nxt = init ? ga->cur : 1 - ga->cur;
    const int32_t count = ga->count;
    RankArgs a;
    a.inst = ga->inst.as<GaInst>();
    a.f_par = ga->fit[ga->cur].as<int64_t>();
    a.f_pool = f_pool;
    a.pool = pool;
    a.npool = npool;
    a.init = init ? 1 : 0;
    a.f_out = ga->fit[nxt].as<int64_t>();
    a.parents = ga->pop[ga->cur].as<int32_t>();
    a.children = ga->children.as<int32_t>();
    a.rows_out = ga->pop[nxt].as<int32_t>();
    a.gen_ctr = ga->gen_ctr.as<uint32_t>();
    a.gens = (uint32_t)gens;
    // launch extents: the largest instance
    const int32_t max_total = init ? ga->max_pop : (pool ? ga->max_pop + npool : ga->max_pop_lambda);
    TimedScope pass(&ga->timer, "elitism", s, 1);
    hipLaunchKernelGGL(k_rank_rows, dim3((max_total + kRankKeys - 1) / kRankKeys, count), dim3(64 * kRankWaves), 0, s,
                       a);
    GAPA_HIP(hipGetLastError());
    ga->cur = nxt;
    return GAPA_OK;
}

// Threads of an operator block: 256 for short rows (k = 100: 11.0 us against 11.4
// with 512; 32 GAs of k = 10 to 500 together 27.4 against 38), 512 for long ones
// (n = 200k, k = 2000: 1024 children 31.8 us against 32.2, 4096 87.2 against 90.9;
// 300 of k = 3000 33 against 44).  That takes the registers down to 64, for eight
// waves a SIMD; with more, 37.5 and 98.2.
static int32_t op_threads(const gapa_ga *ga)
{
    int32_t k = INT_MAX;
    for (const GaInst &I : ga->hinst) k = std::min(k, I.k);
    return k > 1024 ? kOpBlock : kOpBlock / 2;
}

int ga_prepare_kernels(size_t lds)
{
    if (lds > 64 * 1024) {
        GAPA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_init),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        GAPA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_offspring),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    }
    return GAPA_OK;
}

int ga_launch_init(gapa_ga *ga, hipStream_t s)
{
    OpArgs a = op_args(ga, nullptr);
    TimedScope ts(&ga->timer, "ga_init", s, 1);
    hipLaunchKernelGGL(k_init, dim3(ga->max_pop, ga->count),
                       dim3(op_threads(ga)), ga->op_lds_bytes, s, a);
    GAPA_HIP(hipGetLastError());
    return GAPA_OK;
}

int ga_launch_offspring(gapa_ga *ga, hipStream_t s, bool rows_only)
{
    OpArgs a = op_args(ga, ga->pop[ga->cur].as<int32_t>());
    a.rows_only |= rows_only ? 1 : 0;
    TimedScope ts(&ga->timer, "ga_offspring", s, 1);
    hipLaunchKernelGGL(k_offspring, dim3(ga->max_lambda, ga->count),
                       dim3(op_threads(ga)), ga->op_lds_bytes, s, a);
    GAPA_HIP(hipGetLastError());
    return GAPA_OK;
}

static int ga_eval(gapa_ga *ga, bool init, bool breed, hipStream_t s)
{
    int32_t *mcn = ga->objective_mcn ? ga->child_mcn.as<int32_t>() : nullptr;
    const Measure measure = ga->objective_forest ? kMeasureForest : kMeasurePC;
    int rc;
    if (breed)
        rc = breed_rows_components(ga, mcn, s, measure);
    else if (ga->by_rows && ga->count > 1)
        rc = eval_rows_components_batch(ga, init, mcn, s, measure);
    else if (ga->by_rows)
        rc = eval_rows_components_ws(ga->graph, ga->children.as<int32_t>(), init ? ga->params.pop : ga->lambda,
                                     ga->params.k, ga->child_fit.as<int64_t>(), mcn, ga->flag.as<int32_t>() + 3,
                                     ga->ws, &ga->timer, s, measure);
    else if (ga->count > 1)
        rc = eval_masks(ga->graph, ga->masks.as<uint32_t>(), ga->alive.as<int32_t>(), 0, ga->child_fit.as<int64_t>(),
                        mcn, ga->ws, &ga->timer, s, init ? &ga->tab_init : &ga->tab_gen, measure);
    else
        rc = eval_masks(ga->graph, ga->masks.as<uint32_t>(), ga->alive.as<int32_t>(),
                        init ? ga->params.pop : ga->lambda, ga->child_fit.as<int64_t>(), mcn, ga->ws, &ga->timer, s,
                        nullptr, measure);
    if (rc != GAPA_OK || !mcn) return rc;
    // the objective is MCN: it replaces PC as the fitness of every slot
    hipLaunchKernelGGL(k_mcn_objective, dim3((ga->slots + 255) / 256), dim3(256), 0, s, mcn,
                       ga->child_fit.as<int64_t>(), ga->slots);
    GAPA_HIP(hipGetLastError());
    return GAPA_OK;
}

int ga_eval_children(gapa_ga *ga, bool init, hipStream_t s) { return ga_eval(ga, init, false, s); }

int ga_init_population(gapa_ga *ga, hipStream_t s)
{
    int rc = launch_fill_u32(ga->gen_ctr.ptr, 0u, 1, s);
    if (rc == GAPA_OK) rc = ga_launch_init(ga, s);
    if (rc == GAPA_OK) rc = ga_eval_children(ga, true, s);
    if (rc == GAPA_OK) rc = ga_rank_and_gather(ga, true, ga->child_fit.as<int64_t>(), nullptr, 0, s);
    return rc;
}

int ga_generation(gapa_ga *ga, hipStream_t s)
{
    // (with timing on, breeding and evaluation are launches of their own)
    const bool breed = ga->by_rows && ga->count == 1 && !ga->timer.level && components_breed(ga);
    int rc = breed ? GAPA_OK : ga_launch_offspring(ga, s);
    if (rc == GAPA_OK) rc = ga_eval(ga, false, breed, s);
    if (rc == GAPA_OK) rc = ga_rank_and_gather(ga, false, ga->child_fit.as<int64_t>(), nullptr, 0, s);
    if (rc != GAPA_OK) return rc;
    ga->generation += 1;
    return GAPA_OK;
}

int ga_generations(gapa_ga *ga, int32_t n, hipStream_t s)
{
    const Measure measure = ga->objective_forest ? kMeasureForest : kMeasurePC;
    int rc = GAPA_OK;
    // (an even number of swaps: the last children are where recordings, too, put theirs)
    if ((n & 1) == 0) ga->swap_children();
    for (int32_t i = 0; i < n && rc == GAPA_OK; ++i) rc = breed_rows_components(ga, nullptr, s, measure, i);
    if (rc == GAPA_OK) rc = ga_rank_and_gather(ga, false, ga->child_fit.as<int64_t>(), nullptr, 0, s, n);
    if (rc == GAPA_OK) ga->generation += n;
    return rc;
}

}  // namespace gapa
