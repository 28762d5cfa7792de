// Host-side internals of the HIP library: handle layouts, device buffers,
// kernel-timing bookkeeping and the launchers each kernel file provides.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "gapa.h"

namespace gapa {

// ---------------------------------------------------------------- errors ----

void set_error(const char *fmt, ...);

struct Status {
    int code = GAPA_OK;
    bool ok() const { return code == GAPA_OK; }
};

// ------------------------------------------------------- device buffers -----

// Grow-only device allocation (contents not preserved on growth).  A
// borrowed buffer is a view of memory owned elsewhere: reserve() never
// allocates for it (a request beyond its size is an error) and release()
// only forgets it.
struct DevBuf {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool borrowed = false;
    int reserve(size_t want);  // GAPA_OK, GAPA_E_OOM, or GAPA_E_INVALID_ARG for a borrowed view too small
    void release();
    void borrow(void *p, size_t n)
    {
        ptr = p;
        bytes = n;
        borrowed = true;
    }
    template <class T> T *as() const { return static_cast<T *>(ptr); }
};

// ---------------------------------------------------------------- mailbox ---

// Page-locked host memory through which a handle's small host arrays pass:
// kernels read its inputs and write its results in place, so that a call with
// host arrays waits once, for its stream, instead of once a copy (a copy from or
// to ordinary memory is one of 12 to 17 us, whatever its size).  100 rows of 20
// genes, n = 2018: 32 us a call against 66 by copies; a GA's best individual 14
// against 45, its population of 1000 genes 14 against 46, of 77,000 29 against 56.
// From 1 MiB on the copies' own staging takes over.
//
// Handles take a mailbox at their first such call and give it back when they
// are destroyed; the process keeps kSpare of those for the next handles (page
// locking one takes longer than many calls) and frees the others.
struct Mailbox {
    static constexpr size_t kBytes = 1 << 20;
    static constexpr size_t kSpare = 8;
    unsigned char *host = nullptr;  // what the host sees
    unsigned char *dev = nullptr;   // the same memory for kernels on the handle's device
    bool open();                    // false if there is none to be had (the copies serve then)
    void close();
};

// Up to three device arrays (bytes a multiple of 4) to the front of the mailbox,
// one after the other, and waits for them (and all else on the stream).  clear: the
// first array again, to be cleared once copied, or NULL.
struct MailItem {
    const void *src;
    size_t bytes;
};
int mail_collect(const Mailbox &m, MailItem a, MailItem b, MailItem c, hipStream_t s, uint32_t *clear = nullptr);

// ---------------------------------------------------------------- timing ----

// While enabled, named scopes are bracketed by a pair of HIP events recorded
// on their stream; totals are folded in on collect().  Level 1 times whole
// passes (the batched fitness of a chunk, the operator kernel, elitism);
// level 2 also times every kernel launch inside them (the extra events add
// gaps between kernels, so pass totals are only exact at level 1).
class KernelTimer {
public:
    int level = 0;
    void begin(const char *name, hipStream_t s);
    void end(hipStream_t s);
    int collect(gapa_kernel_time *out, int cap, int *count);
    ~KernelTimer();

private:
    struct Pending {
        std::string name;
        hipEvent_t a, b;
    };
    std::vector<Pending> pending_;
    std::vector<hipEvent_t> free_;
    std::map<std::string, std::pair<int64_t, double>> totals_;
    std::vector<std::string> names_;  // stable storage for returned names
    std::vector<size_t> open_;        // indices into pending_ of open scopes
    hipEvent_t take();
};

struct TimedScope {
    KernelTimer *t;
    hipStream_t s;
    bool on;
    TimedScope(KernelTimer *timer, const char *name, hipStream_t stream, int level = 2)
        : t(timer), s(stream), on(timer && timer->level >= level)
    {
        if (on) t->begin(name, s);
    }
    ~TimedScope()
    {
        if (on) t->end(s);
    }
};

// ----------------------------------------------------------------- graph ----

// Scratch for the batched fitness of one chunk of individuals.
struct FitnessWorkspace {
    DevBuf parent;   // int32 [B][n]  union-find parents
    DevBuf count;    // int32 [B][n]  component sizes at roots (union-find path)
    DevBuf dead;     // uint32 [n][Wd] removed bits, node-major (bit-parallel path)
    DevBuf reach;    // uint32 [n][Wd] root-component bits
    DevBuf ucount;   // int32 [B][n]  set sizes of the leftover union-find, kept zero
    DevBuf pairs;    // int64 [B * n_noniso] pending (individual, node) keys
    DevBuf worklist; // int4 [n_noniso] records (node, first edge, edge end) of the nodes still pending after the ordered sweep
    DevBuf pflag;    // uint8 [n_noniso] 1: the node at this band position is still pending after the ordered sweep (then: at this worklist position, after the last follow-up sweep)
    bool pflag_clear = false;  // pflag zeroed since it was (re)allocated
    DevBuf small;    // int32 roots, root-set sizes, counters, count partials
    int32_t *stats_ctr = nullptr;  // device counters of the last bit-parallel chunk
    int32_t stats_B = 0;
    DevBuf masks;    // uint32 [P][W] removed-node bit sets (eval_population)
    DevBuf alive;    // int32 [P]    surviving non-isolated nodes (eval_population)
    DevBuf genes;    // int32 [P][k]  staged host genes
    DevBuf spill;    // int32 union-find parents of eval_rows_components beyond LDS
    DevBuf fitness;  // int64 [P]
    DevBuf mcn;      // int32 [P]
    DevBuf flag;     // int32 [4]     device error flags, and as many of trusted rows, which nobody reads
    DevBuf six_mats; // int8 [3][chunk][n_pad][n_pad] dense reachability matrices
    DevBuf six_tot;  // uint64 [chunk] their entry sums
    // extra lanes (owned): chunks of a population wider than one pass run
    // side by side, each with its own workspace and stream
    std::vector<FitnessWorkspace *> lanes;
    std::vector<hipStream_t> lane_streams;
    std::vector<hipEvent_t> lane_done;
    hipEvent_t fork = nullptr;
};

// Launch shapes of the bit-parallel fitness pass (results do not depend on
// them; only speed does).
// (The defaults against a grid of 4096 and bands of 8192 blocks: power law n =
// 200k, P = 1024, uniform rows 148 us a pass against 175, hub rows 191 and 202; P =
// 32 86 and 92; BA m = 3 165 and 186; random graph of mean degree 8 222 and 240; two
// sweeps or 16 neighbours are up to 5 % faster on these and ten times slower
// without hubs, or 20 % on BA with m = 2.)
struct Tuning {
    int32_t sweep_grid = 2048;   // blocks of the worklist and pair kernels (twice as many hook pairs)
    int32_t band_scan = 32;      // neighbours read per node in the ordered sweep
    int32_t sweeps = 3;          // follow-up sweeps over the pending nodes
    int32_t band_blocks = 2048;  // block cap of one band launch
};

}  // namespace gapa

struct gapa_graph {
    std::atomic<int32_t> refs{1};  // the caller's handle, plus one per GA or batch using the graph
    int device = 0;
    uint64_t content_hash = 0;     // FNV-1a of n, row_ptr and col_idx (checkpoints name their graph by it)
    int32_t n = 0;
    int64_t nnz = 0;
    int32_t words = 0;          // ceil(n / 32): words of a node bit set
    int32_t *d_row_ptr = nullptr;
    int32_t *d_col = nullptr;
    int32_t *d_src = nullptr;   // source node of every CSR entry (COO rows)
    int32_t *d_order = nullptr; // [n] nodes by (degree desc, id)
    int32_t *d_colD = nullptr;  // [nnz] each neighbour list by (degree desc, id)
    int4 *d_band_rec = nullptr;   // [n_noniso] non-isolated nodes by (BFS level, id) as records
                                  // (node, row_ptr[node], row_ptr[node + 1], 0)
    uint32_t *d_noniso = nullptr; // [words] bit v set: v has at least one edge
    int8_t *d_src_idx = nullptr;  // [n] index of a band source among its instance's (order[voff + t]), else -1
    std::vector<int32_t> band_off;  // host: band b is d_band_rec[band_off[b], band_off[b+1])
    bool deep = false;          // with d_lists: many nodes, and long paths from the first of d_order
    bool loose = false;         // with d_lists: many nodes outside the component of the first of d_order
    int32_t levels = 0;         // breadth-first levels from the highest-degree nodes
    int32_t src_band = 0;       // size of band 0 when it holds exactly the sources, else 0
    int32_t n_noniso = 0;       // nodes with at least one edge
    // NeighbourLists of a one-instance graph of at most kListsMaxN nodes:
    // the n first chunks of four 16-bit ids, all list_chunks chunks, the int32
    // [n + 1] first chunk of each node, the uint16 [n] new number of each node
    unsigned char *d_lists = nullptr;
    int32_t list_chunks = 0;
    int32_t n_hub = 0;          // nodes of more than kHubDegree neighbours
    bool far = false;           // most nodes are kFarLevel hops or more from every high-degree node
    bool sparse = false;        // not far, but kSparseDegree neighbours or fewer a node that has any
    int32_t algorithm = 0;      // 0: bit-parallel sweeps, 1: edge-parallel union-find
    gapa::Tuning tune;
    int32_t tune_version = 0;   // bumped by every tuning change (recorded graphs are re-recorded)
    gapa::FitnessWorkspace ws;
    gapa::KernelTimer timer;
    gapa::Mailbox mail;
    gapa::Mailbox check;        // its device's slot for the checked allocation-free call (not owned), or empty
    bool flag_clear = false;    // the first four words of ws.flag hold zeros
    bool failed = false;
};

namespace gapa {

// Node words per tile of the dead-row transpose (32 nodes each); the tile
// lists of instance tables step by it.
constexpr int kTransposeWords = 4;

// Node words per transposer tile for chunks of Wd words per node row (Wd a
// power of two <= 32): kTransposeWords * 32 / Wd.
inline int32_t transpose_tile_words(int32_t Wd)
{
    return kTransposeWords * 32 / Wd;
}

// Several instances (disjoint node ranges of one graph, each with its own
// individuals) evaluated in one bit-parallel fitness pass.  All arrays are on
// the device.  Slot i of instance b is entry b * bseg + i of the alive,
// fitness and mcn arrays; its removed-node bit set (local node ids, W_b =
// ceil(n_b / 32) words) starts at word moff[b] + i * W_b of the mask array.
struct InstTable {
    int32_t count = 0;
    int32_t bseg = 0;                    // slots per instance: 32 * Wd, Wd a power of two <= 32
    const int32_t *voff = nullptr;       // [count + 1] first node of each instance
    const int32_t *live = nullptr;       // [count] slots in use
    const int64_t *moff = nullptr;       // [count]
    const int32_t *node_inst = nullptr;  // [n] instance of each node
    const int32_t *tiles = nullptr;      // [2 * ntiles] (instance, first node word) of each 8-word tile
    int32_t ntiles = 0;
};

// What the fitness sums over the components C of G - S: |C|(|C| - 1)/2
// (pairwise connectivity), or |C| - 1, whose sum is |V minus S| minus the
// number of components (the size of a spanning forest of G - S).
enum Measure : int32_t { kMeasurePC = 0, kMeasureForest = 1 };

// Fitness of P individuals given as removed-node bit sets masks[P][W]
// (device) with alive[P] = surviving non-isolated nodes of each.  Writes
// fitness[P] (int64, the sum selected by `measure`) and, if mcn != nullptr,
// mcn[P] (int32).  Runs the graph's selected algorithm.
// With an instance table of count > 1 (bit-parallel algorithm only), P is
// ignored and all slots of all instances are evaluated in one pass.
int eval_masks(gapa_graph *g, const uint32_t *masks, const int32_t *alive, int32_t P, int64_t *fitness, int32_t *mcn,
               FitnessWorkspace &ws, KernelTimer *timer, hipStream_t s, const InstTable *it = nullptr,
               Measure measure = kMeasurePC);
int eval_masks_bits(gapa_graph *g, const uint32_t *masks, const int32_t *alive, int32_t P, int64_t *fitness,
                    int32_t *mcn, FitnessWorkspace &ws, KernelTimer *timer, hipStream_t s,
                    const InstTable *it = nullptr, Measure measure = kMeasurePC);
// Bytes of scratch the bit-parallel fitness needs for chunks of 32 * Wd
// individuals on graph g (every buffer of one pass plus the chunk's bit sets,
// each part 256-byte aligned).
size_t bits_scratch_bytes(const gapa_graph *g, int32_t Wd);
// Fitness of P gene rows (device, [P][k]) with every buffer carved from
// `scratch` (`bytes` long), by workgroups (components_fit) or the bit-parallel
// pass: chunks of 32 * Wd rows, Wd the widest power of two <= 32 that fits, one
// after another on stream s; a gene outside [0, n) sets flag[0] (flag: 4 int32
// in the scratch, cleared here unless flag_out is NULL: then nobody reads it).
// Nothing is allocated; GAPA_E_INVALID_ARG if not even 32 rows fit.
int eval_genes_bits_scratch(gapa_graph *g, const int32_t *genes, int32_t P, int32_t k, int64_t *fitness,
                            int32_t *mcn, Measure measure, void *scratch, size_t bytes, int32_t **flag_out,
                            hipStream_t s);
int eval_masks_unionfind(gapa_graph *g, const uint32_t *masks, int32_t P, int64_t *fitness, int32_t *mcn,
                         FitnessWorkspace &ws, KernelTimer *timer, hipStream_t s, Measure measure = kMeasurePC);
// Same from gene rows genes[P][k] (device node ids; a repeated id in a row is
// one removal); a gene outside [0, n) sets flag[0] and is ignored.
int eval_genes(gapa_graph *g, const int32_t *genes, int32_t P, int32_t k, int64_t *fitness, int32_t *mcn,
               int32_t *flag, FitnessWorkspace &ws, KernelTimer *timer, hipStream_t s, Measure measure = kMeasurePC);

// Removed-node bit sets masks[P][W] of P = 32 Wd individuals (Wd a power of
// two <= 32) to node-major rows rows[n][Wd]: bit i of row v is set when
// individual i removes v.
int launch_bits_transpose(const uint32_t *masks, int32_t P, int32_t W, int32_t n, uint32_t *rows, hipStream_t s);

// Fills count 32-bit words at p with value (a kernel, not a memset node).
int launch_fill_u32(void *p, uint32_t value, int64_t count, hipStream_t s);
// A graph's neighbour lists for the kernels that keep per-node state of whole
// individuals in LDS.  Nodes are renumbered by descending degree (`rank`;
// fitness values do not depend on the numbering), so that neighbouring
// threads walk lists of similar lengths, and isolated nodes come last.  Node
// v's list is chunks [off[v], off[v + 1]) of four 16-bit ids, ascending (so
// by descending degree), the last one filled up with its first neighbour; head[v]
// is its first chunk (all v for an isolated node).
struct NeighbourLists {
    const uint16_t *rank;  // [n]
    const int32_t *off;    // [n + 1]
    const uint2 *ids;      // [off[n]]
    const uint2 *head;     // [n]
    int32_t n;
    int32_t n_hub;         // nodes of more than kHubDegree neighbours: the first n_hub
};
constexpr int32_t kListsMaxN = 65535;
constexpr int32_t kHubDegree = 24;

// The lists laid out from `base` on (in the order of gapa_graph::d_lists).
__host__ __device__ inline NeighbourLists neighbour_lists(const unsigned char *base, int32_t n, int32_t chunks,
                                                          int32_t n_hub)
{
    const size_t ids_at = (size_t)n * 8, off_at = ids_at + (size_t)chunks * 8, rank_at = off_at + ((size_t)n + 1) * 4;
    return NeighbourLists{reinterpret_cast<const uint16_t *>(base + rank_at),
                          reinterpret_cast<const int32_t *>(base + off_at),
                          reinterpret_cast<const uint2 *>(base + ids_at), reinterpret_cast<const uint2 *>(base), n,
                          n_hub};
}

inline size_t neighbour_lists_bytes(int32_t n, int32_t chunks)
{
    return (size_t)n * 8 + (size_t)chunks * 8 + ((size_t)n + 1) * 4 + (size_t)n * 2;
}

inline NeighbourLists neighbour_lists(const gapa_graph *g)
{
    return neighbour_lists(g->d_lists, g->n, g->list_chunks, g->n_hub);
}

// Fitness of P gene rows (device, [P][k]) by one workgroup each
// (components.hip), on graphs with neighbour lists: one launch.  A gene outside
// [0, n) sets flag[0] and is ignored.  spill: components_spill_bytes of
// device memory (fewer: fewer workgroups side by side).  components_fit: whether
// that is the way for P individuals at a time.
bool components_fit(const gapa_graph *g, int64_t P);
size_t components_spill_bytes(const gapa_graph *g, int32_t P);
int eval_rows_components(gapa_graph *g, const int32_t *genes, int32_t P, int32_t k, int64_t *fitness, int32_t *mcn,
                         int32_t *flag, void *spill, size_t spill_bytes, KernelTimer *timer, hipStream_t s,
                         Measure measure);
// The same with the spill in ws (grown as needed).
int eval_rows_components_ws(gapa_graph *g, const int32_t *genes, int32_t P, int32_t k, int64_t *fitness, int32_t *mcn,
                            int32_t *flag, FitnessWorkspace &ws, KernelTimer *timer, hipStream_t s, Measure measure);

// The same for the instances of a batch, in one launch (plans made at creation,
// one for the initial population and one for a generation's children).
struct CompBatch {
    DevBuf insts, tasks, lists;  // (lists: of the graphs, once for both plans)
    int32_t ntasks = 0, threads = 0, blocks = 0, spill_stride = 0;
    size_t lds = 0;
};
int components_batch_plan(gapa_ga *ga, gapa_graph *const *graphs, bool init);
bool components_breed(const gapa_ga *ga);
// (ahead > 0: the ahead-th generation since the last elitism, merged in first)
int breed_rows_components(gapa_ga *ga, int32_t *mcn, hipStream_t s, Measure measure, int32_t ahead = 0);
int eval_rows_components_batch(gapa_ga *ga, bool init, int32_t *mcn, hipStream_t s, Measure measure);

// Dense reachability fitness (sixdst.hip).
bool sixdst_sparse(const gapa_graph *g, int32_t hops);
int sixdst_eval_genes(gapa_graph *g, const int32_t *genes, int32_t P, int32_t k, int32_t hops, int64_t *pc,
                      int32_t *mcn, int32_t *flag, hipStream_t s);
size_t sixdst_bytes_per_individual(int32_t n);
int sixdst_eval_masks(gapa_graph *g, const uint32_t *masks, int32_t P, int32_t hops, int32_t chunk, uint8_t *mats,
                      unsigned long long *tot, int64_t *pc, int32_t *mcn, hipStream_t s);

// P rows of genes[.][k] (device; rows[0 .. P), or the first P when rows is NULL)
// -> masks[P][W] and alive[P]; out-of-range genes raise flag[0].
int launch_mask_build(const int32_t *genes, const int32_t *rows, int32_t P, int32_t k, int32_t n, int32_t W,
                      const uint32_t *noniso, int32_t n_noniso, uint32_t *masks, int32_t *alive, int32_t *flag, hipStream_t s);

// ------------------------------------------------------------------- GA -----

// LDS a compute unit has for a block of the operators, and what their kernels take
// of it besides the dynamic part (the flags of a block and the sums of its waves).
constexpr size_t kOpLdsMax = 160 * 1024, kOpStaticLds = 48;

// Dynamic LDS of the operator kernels for n nodes and budget k (the membership
// bits in whole 16 bytes, the row, three bit sets over its slots and the list of
// slots, whose room takes the member counts of the quads later), and the words
// of a quad as a power of two.  Quads of more than four words keep the counts
// within the room that there is on the largest graphs (more than a million
// nodes).  Sizes that fit no block come out above kOpLdsMax - kOpStaticLds.
inline size_t ga_op_lds_layout(int32_t n, int32_t k, int32_t *log_q)
{
    const size_t W4 = ((size_t)n + 127) / 128, k2 = ((size_t)k + 1) & ~(size_t)1;
    const size_t fixed = 16 * W4 + 4 * ((size_t)k + 3 * (((size_t)k + 31) / 32));
    for (*log_q = 2;; ++*log_q) {
        const size_t quads = (W4 >> (*log_q - 2)) + 1;
        const size_t bytes = fixed + 2 * std::max(k2, (quads + 1) & ~(size_t)1);
        if (bytes + kOpStaticLds <= kOpLdsMax || quads <= k2) return bytes;
    }
}
int ga_prepare_kernels(size_t lds);

// Device table entry of one GA instance: where its rows live in the shared
// buffers, its sizes and its random-stream parameters.  A single GA is a
// one-entry table with every offset 0.
struct GaInst {
    int64_t pop_off;    // first element of its rows in pop[*] (row stride k)
    int64_t child_off;  // first element of its rows in children (row stride k)
    int64_t mask_off;   // first word of its child masks (row stride W)
    int32_t fit_off;    // first entry in fit[*]
    int32_t slot_off;   // first entry in child_fit and alive
    int32_t noniso_off; // first word of its non-isolated node bit set
    uint64_t seed, t_pc, t_pm;
    int32_t P, L, k, n, W, KW, T, n_noniso;
    int32_t log_q;      // words of a quad in the operators' LDS, as a power of two
};

int ga_init_population(gapa_ga *ga, hipStream_t s);
// One generation of every instance; the generation number is read on the
// device, so the launches can be captured into a graph and replayed.
int ga_generation(gapa_ga *ga, hipStream_t s);
// n >= 2 generations at a launch each, one elitism at the end; for GAs that
// ga_merges allows.
constexpr int32_t kMergeKeys = 256;  // parents and children together, at most
bool ga_merges(const gapa_ga *ga);
int ga_generations(gapa_ga *ga, int32_t n, hipStream_t s);
int ga_launch_init(gapa_ga *ga, hipStream_t s);
// rows_only: the children's rows only; their bit sets and alive counts are
// left for the caller to build (for the few it evaluates).
int ga_launch_offspring(gapa_ga *ga, hipStream_t s, bool rows_only = false);
// Elitism of every instance over its current parents (none at generation 0,
// `init`) and its evaluated offspring (f_pool[q] is the fitness of child
// pool[q], or of child q when pool is NULL; a pool only with one instance);
// writes the next population buffer and, after generation 0, advances the
// device generation counter.
int ga_rank_and_gather(gapa_ga *ga, bool init, const int64_t *f_pool, const int32_t *pool, int32_t npool,
                       hipStream_t s, int32_t gens = 1);
// Exact fitness of the children currently held (the initial population at
// generation 0) into child_fit.
int ga_eval_children(gapa_ga *ga, bool init, hipStream_t s);

// ------------------------------------------------------------ surrogate -----

struct SurrogateState;
// Allocates and initialises the learned screening model of a one-instance GA.
int surrogate_attach(gapa_ga *ga, const gapa_surrogate_params *sp, hipStream_t s);
void surrogate_release(SurrogateState *st);
// One generation with screening (or a full one during warm-up / fallback).
int surrogate_generation(gapa_ga *ga, hipStream_t s);
int surrogate_predict(gapa_ga *ga, const int32_t *genes, int32_t P, float *yhat, hipStream_t s);
int surrogate_train_batch(gapa_ga *ga, const int32_t *genes, const float *target, int32_t B, bool keep_grads,
                          hipStream_t s);
int surrogate_tensor(gapa_ga *ga, int32_t which, int32_t kind, float *host, int64_t count, bool set);
int surrogate_stats(gapa_ga *ga, gapa_surrogate_report *out);
int surrogate_last_pool(gapa_ga *ga, int32_t *pool, int32_t cap, int32_t *count);
int surrogate_last_predictions(gapa_ga *ga, float *yhat, int32_t cap, int32_t *count);
// The judge's statistics of m predictions against exact fitness (device
// arrays), written to host out[2]; waits on s.
int surrogate_judge(const float *yhat, const int32_t *pool, const int64_t *F, int32_t m, double mu, double sd,
                    double *out, hipStream_t s);

// Error reporting for HIP calls.
int hip_fail(hipError_t e, const char *what);
#define GAPA_HIP(call)                                                  \
    do {                                                                \
        hipError_t _e = (call);                                         \
        if (_e != hipSuccess) return ::gapa::hip_fail(_e, #call);       \
    } while (0)

}  // namespace gapa

struct gapa_ga {
    gapa_graph *graph = nullptr;  // for a batch: the disjoint union of the instance graphs
    gapa_params params{};         // first instance's parameters
    int32_t lambda = 0;
    uint64_t t_pc = 0, t_pm = 0;  // Bernoulli thresholds floor(p * 2^32)
    int64_t generation = 0;
    int cur = 0;                  // which population buffer is current
    int32_t count = 1;            // instances
    std::vector<gapa::GaInst> hinst;
    gapa::DevBuf inst;            // GaInst [count]
    int32_t max_pop = 0, max_lambda = 0, max_pop_lambda = 0;
    gapa::DevBuf pop[2];          // int32 rows of every instance
    gapa::DevBuf fit[2];          // int64 [sum P]
    gapa::DevBuf children;        // int32 rows
    gapa::DevBuf child_fit;       // int64 slots
    gapa::DevBuf children_prev, child_fit_prev;  // of the generation before, when generations run at a launch each
    void swap_children()
    {
        std::swap(children, children_prev);
        std::swap(child_fit, child_fit_prev);
    }
    gapa::DevBuf child_mcn;       // int32 slots (GAPA_MINIMISE_MCN: the pass's MCN, copied into child_fit)
    int32_t slots = 0;
    bool objective_mcn = false;
    bool objective_forest = false;  // GAPA_MAXIMISE_COMPONENTS: fitness = |V minus S| - components
    bool by_rows = false;         // fitness by eval_rows_components(_batch): no bit sets are made
    gapa::CompBatch comp_init, comp_gen;  // a batch evaluated that way
    gapa::DevBuf masks;           // uint32 removed-node bit sets of the children
    gapa::DevBuf alive;           // int32 slots: surviving non-isolated nodes
    gapa::DevBuf flag;            // int32 [4] device error flags
    gapa::DevBuf gen_ctr;         // uint32 [1] generations completed (read by the operator kernel)
    uint32_t *noniso = nullptr;   // batch: per-instance non-isolated bit sets (else the graph's)
    gapa::DevBuf noniso_buf;
    // batch: instance tables of the fitness pass at generation 0 and later
    gapa::InstTable tab_init, tab_gen;
    gapa::DevBuf tab_voff, tab_live_init, tab_live_gen, tab_moff, tab_node_inst, tab_tiles;
    gapa::FitnessWorkspace ws;
    gapa::KernelTimer timer;
    gapa::Mailbox mail;
    hipStream_t last_stream = nullptr;
    size_t op_lds_bytes = 0;      // dynamic LDS of the operator kernels
    bool failed = false;
    // graph replay of one generation (one per current-buffer parity)
    bool use_graph = false;
    bool warm = false;            // a generation has run eagerly: buffers are sized
    int32_t captured_version = -1;  // graph tuning the recorded generations were made with
    hipStream_t cap_stream = nullptr;
    struct Replay {
        int parity;        // current population buffer the recording starts from
        int32_t gens;      // generations it runs
        hipGraph_t graph;
        hipGraphExec_t exec;
    };
    std::vector<Replay> replays;
    gapa::SurrogateState *surr = nullptr;  // learned screening, when attached
};

struct gapa_batch {
    gapa_ga *ga = nullptr;
    // owned: the disjoint union of the instance graphs, or, where workgroups
    // evaluate the individuals on the graphs' neighbour lists, only its device,
    // sizes and tuning
    gapa_graph *super = nullptr;
};
