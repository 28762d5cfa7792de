// Fitness by one workgroup for every few individuals, for graphs whose node
// states fit LDS: the whole evaluation from gene rows to PC (and MCN) is one
// launch.  The bit-parallel pass of fitness_bits.hip shares every graph read
// among up to 2048 individuals, but takes a dozen dependent launches and
// keeps its rows in global memory; here a workgroup takes up to eight
// individuals (one while there are compute units to spare), keeps a byte of
// removed bits and a byte of reached bits per node, and needs about two sweeps
// of LDS reads.
//
// Nodes are renumbered by descending degree (NeighbourLists).
//   1. The genes' nodes are removed.  Each individual's root is its first
//      survivor; the root and its neighbours are reached.
//   2. Pull sweeps: a node is reached in the individuals one of its
//      neighbours is reached in, if it survives there.  Sweeps over all nodes,
//      hubs first, read the four neighbours of highest degree and settle most
//      of a graph with a giant component; a few more go over a list of the
//      nodes still open in some individual and over their whole lists.
//   3. The rest is exact whatever the sweeps left: per individual a
//      union-find over the surviving edges between open nodes, with the
//      reached ones contracted into one entry.  Its entries are the listed
//      nodes in rank order (a prefix count over the words of listed bits
//      gives a node's entry), so it needs room only for them: in LDS, for as
//      many individuals at a time as fit, or, if one does not, in a slice of
//      global memory the workgroup owns.
//   4. Every set of the union-find is counted at its representative; the
//      root's component is every survivor but the open nodes outside the
//      reached set.
//
// Bound by LDS: a sweep over all nodes reads four bytes at random for every
// node that is open (about 8 clocks for a wave's 64, bank conflicts included)
// and takes 8 us for n = 30k, of 34 (random graph of mean degree 8, three
// sweeps) or 20 us (BA, m = 3, two) for the whole evaluation of one individual;
// eight individuals in a byte cost a block 1.4 times one.  Whole calls against
// the bit-parallel pass: n = 200, P = 32: 9.7 against 53 us; BA n = 10k: P = 256
// 16 against 78 us, P = 2048 28 against 133; random graph n = 30k: P = 203 34
// us against 2.4 ms (few individuals left that pass a large union-find around
// the roots), P = 2048 44 against 136 us; power law n = 65k: P = 256 48 against
// 115 us, P = 2048 116 against 179; 32 graphs of 1000 to 50,000 nodes, 128
// individuals each: 82 against 200 us, bound by the largest graphs' blocks.
// Bits instead of bytes for the states: 1.5 times slower sweeps (ten more
// instructions a neighbour).  One individual a block whatever the population:
// n = 30k, P = 2048 336 us.  Pushing on from hubs, too: BA n = 10k 26 instead of
// 20 us.
#include <algorithm>
#include <vector>

#include "operators.h"

namespace gapa {
namespace {

constexpr int32_t kFullSweeps = 12;    // sweeps over all nodes, at most
constexpr int32_t kSweepNodes = 4;     // nodes a thread has in flight in one
constexpr int32_t kSweeps = 8;         // sweeps over the list of open nodes, at most
constexpr int32_t kLaterChunks = 32;   // chunks of neighbours an open node reads in one
constexpr int32_t kWaveChunks = 8;     // longer lists are united by a whole wave
constexpr int32_t kPushLanes = 4;      // lanes that push one newly reached node
constexpr int32_t kPushLevels = 4;     // levels pushed after the root's neighbours, at most

// Union-find parents of the open nodes: in LDS, or in global memory.
template <bool kLds>
struct Parents {
    int32_t *p;
    __device__ __forceinline__ int32_t get(int32_t x) const
    {
        if constexpr (kLds) return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void set(int32_t x, int32_t v) const
    {
        if constexpr (kLds) __hip_atomic_store(p + x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else __hip_atomic_store(p + x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Root of x, re-pointing visited entries at their grandparents.
    __device__ __forceinline__ int32_t find(int32_t x) const
    {
        int32_t q = get(x);
        while (q != x) {
            const int32_t gp = get(q);
            if (gp != q) set(x, gp);
            x = q;
            q = gp;
        }
        return x;
    }
    // Root of x, changing nothing.
    __device__ __forceinline__ int32_t root(int32_t x) const
    {
        int32_t q = get(x);
        while (q != x) {
            x = q;
            q = get(x);
        }
        return x;
    }
    // The larger root is hooked under the smaller (parents only decrease).
    __device__ __forceinline__ void unite(int32_t a, int32_t b) const
    {
        a = find(a);
        b = find(b);
        while (a != b) {
            if (a < b) {
                const int32_t t = a;
                a = b;
                b = t;
            }
            const int32_t old = atomicCAS(p + a, a, b);
            if (old == a) return;
            a = find(old);
            b = find(b);
        }
    }
};

constexpr int32_t kGroup = 8;  // individuals of a workgroup at most

// A population on one graph, as a workgroup sees it.
struct CompView {
    const int32_t *genes;  // [P][k]
    int32_t k;
    NeighbourLists g;
    int32_t n1;            // nodes with an edge: the first n1 ranks
    int32_t cap;           // entries (listed nodes, union-find parents) LDS holds
    int32_t *spill;        // [n1 + 1] parents of this workgroup beyond it, or NULL when cap > n1
    int64_t *fitness;      // [P]
    int32_t *mcn;          // [P] or NULL
    int32_t forest;
    int32_t *flag;         // [0] set for a gene outside [0, n)
};

// Node states in LDS: a bit for every individual that the node is reached in,
// and one for every individual it is removed in.  Up to four individuals share
// a byte (reached below, removed above), so that a node's own state is one
// read and n bytes are enough; up to eight take two arrays of bytes.
template <int kBits>
struct States {
    static constexpr uint32_t kAll = (1u << kBits) - 1u;
    uint8_t *s;    // [n16] kBits 4: both, kBits 8: reached
    uint8_t *rem;  // [n16] kBits 8: removed

    static size_t bytes(int32_t n) { return ((size_t)n + 15) / 16 * 16 * (kBits == 4 ? 1 : 2); }

    // Word to fill both arrays with: the individuals of `unused` removed everywhere.
    __device__ __forceinline__ void clear(int32_t n, uint32_t unused) const
    {
        const uint32_t f = (kBits == 4 ? unused << 4 : 0u) * 0x01010101u, g = unused * 0x01010101u;
        for (int32_t i = threadIdx.x; i < (n + 15) / 16; i += blockDim.x) {
            reinterpret_cast<uint4 *>(s)[i] = uint4{f, f, f, f};
            if constexpr (kBits == 8) reinterpret_cast<uint4 *>(rem)[i] = uint4{g, g, g, g};
        }
    }
    // (reached, removed) of a node
    __device__ __forceinline__ uint2 get(int32_t v) const
    {
        if constexpr (kBits == 4) {
            const uint32_t x = s[v];
            return uint2{x & 15u, x >> 4};
        } else {
            return uint2{s[v], rem[v]};
        }
    }
    __device__ __forceinline__ uint32_t removed(int32_t v) const
    {
        if constexpr (kBits == 4) return s[v] >> 4;
        else return rem[v];
    }
    __device__ __forceinline__ uint32_t open(int32_t v) const
    {
        const uint2 x = get(v);
        return ~(x.x | x.y) & kAll;
    }
    // Individuals in which one of the four nodes of a chunk is reached.
    __device__ __forceinline__ uint32_t any_reached(const uint2 c) const
    {
        return (s[c.x & 0xFFFFu] | s[c.x >> 16] | s[c.y & 0xFFFFu] | s[c.y >> 16]) & kAll;
    }
    // Writes a node's state; no other thread may be writing it.
    __device__ __forceinline__ void put(int32_t v, uint32_t reached, uint32_t removed) const
    {
        if constexpr (kBits == 4) {
            s[v] = (uint8_t)(reached | removed << 4);
        } else {
            s[v] = (uint8_t)reached;
            rem[v] = (uint8_t)removed;
        }
    }
    // Set bits that other threads may be setting bits beside; the old ones.
    __device__ __forceinline__ uint32_t or_reached(int32_t v, uint32_t bits) const
    {
        return or_byte(s, v, bits) & kAll;
    }
    __device__ __forceinline__ uint32_t or_removed(int32_t v, uint32_t bits) const
    {
        if constexpr (kBits == 4) return or_byte(s, v, bits << 4) >> 4;
        else return or_byte(rem, v, bits);
    }

private:
    static __device__ __forceinline__ uint32_t or_byte(uint8_t *bytes, int32_t v, uint32_t bits)
    {
        const int32_t sh = 8 * (v & 3);
        return (atomicOr(reinterpret_cast<uint32_t *>(bytes) + (v >> 2), bits << sh) >> sh) & 0xFFu;
    }
};

// One instance of a batch (device table).
struct CompInst {
    int64_t lists_off;  // first byte of its neighbour lists
    int64_t child_off;  // of its rows in the children
    int32_t slot_off;   // of its slots in the fitness values
    int32_t n, chunks, n_hub, k, n1, cap, bits;
};

// LDS: the states; of the n1 nodes with an edge, the listed ones (a bit each)
// and their number before each word [ceil(n1 / 32) each]; parents [cap] and
// the list [cap].
template <int kBits>
struct CompLds {
    States<kBits> st;
    uint32_t *listed;
    int32_t *before, *parents;
    uint16_t *list;
};

template <int kBits>
size_t comp_lds_fixed(int32_t n, int32_t n1)
{
    return States<kBits>::bytes(n) + ((size_t)n1 + 31) / 32 * 8;
}

// Sums of a workgroup, most with one entry an individual.
struct CompSums {
    int32_t root[kGroup], removed[kGroup], outside[kGroup], big[kGroup];
    unsigned long long sum[kGroup];
    int32_t added[3], seen[3];  // of a sweep, three in turn: the next one's is cleared while unused
    int32_t queued, hub;        // nodes pushed on from; whether one is a hub
    int32_t wave[16];
};

// Lists the nodes open in some individual, in rank order, as many as fit;
// returns how many there are.  Whole block.
template <int kBits>
__device__ __forceinline__ int32_t list_open(const CompLds<kBits> &l, CompSums &sm, int32_t n1, int32_t cap)
{
    const int32_t W1 = (n1 + 31) / 32, T = blockDim.x, tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    for (int32_t b = 0; b < n1; b += 8 * T) {
        uint32_t open[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) open[u] = l.st.open(min(b + u * T + tid, n1 - 1));
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int32_t v = b + u * T + tid;
            const uint64_t m = __ballot(v < n1 && open[u]);
            if ((tid & 31) == 0 && v < n1) l.listed[v >> 5] = (tid & 32) ? (uint32_t)(m >> 32) : (uint32_t)m;
        }
    }
    if (tid < 16) sm.wave[tid] = 0;
    __syncthreads();
    const int32_t per = (W1 + T - 1) / T;
    const int32_t w0 = min(W1, tid * per), w1 = min(W1, w0 + per);
    int32_t cnt = 0;
    for (int32_t w = w0; w < w1; ++w) cnt += __popc(l.listed[w]);
    const int32_t incl = wave_scan(cnt);
    if (lane == 63) sm.wave[wv] = incl;
    __syncthreads();
    int32_t at = incl - cnt, total = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int32_t x = sm.wave[q];
        at += q < wv ? x : 0;
        total += x;
    }
    for (int32_t w = w0; w < w1; ++w) {
        l.before[w] = at;
        for (uint32_t x = l.listed[w]; x; x &= x - 1, ++at)
            if (at < cap) l.list[at] = (uint16_t)(w * 32 + __ffs(x) - 1);
    }
    __syncthreads();
    return total;
}

// The i-th listed node (from the list, or past its end by a search of the
// counts before each word).
template <int kBits>
__device__ __forceinline__ int32_t listed_node(const CompLds<kBits> &l, int32_t i, int32_t cap, int32_t W1)
{
    if (i < cap) return l.list[i];
    int32_t lo = 0, hi = W1 - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (l.before[mid] <= i) lo = mid;
        else hi = mid - 1;
    }
    uint32_t x = l.listed[lo];
    for (int32_t q = i - l.before[lo]; q > 0; --q) x &= x - 1;
    return lo * 32 + __ffs(x) - 1;
}

// Union-finds of the individuals [i0, i1) over the `count` listed nodes:
// entry (i - i0)(count + 1) is individual i's reached set, the count entries
// after it the listed nodes (those not open in i stay alone and are left out).
// Adds the sizes of their sets to sm.
template <int kBits, bool kLds>
__device__ __forceinline__ void count_open(const CompView &a, const CompLds<kBits> &l, CompSums &sm,
                                           const Parents<kLds> par, int32_t count, int32_t i0, int32_t i1, bool settled)
{
    const int32_t T = blockDim.x, tid = threadIdx.x, W1 = (a.n1 + 31) / 32;
    const int32_t stride = count + 1, entries = (i1 - i0) * stride;
    const uint2 *ids = a.g.ids;
    __syncthreads();
    for (int32_t e = tid; e < entries; e += T) par.set(e, e);
    __syncthreads();
    // an edge to a reached node unites with that set (there is none once the
    // sweeps have settled); one between open nodes is taken from its smaller end
    auto edge = [&](int32_t v, int32_t e, int32_t base, uint32_t bit, int32_t u) {
        const uint2 x = l.st.get(u);
        if (x.y & bit) return;
        if (x.x & bit) {
            if (!settled) par.unite(e, base);
        } else if (v < u) {
            par.unite(e, base + 1 + l.before[u >> 5] + __popc(l.listed[u >> 5] & ((1u << (u & 31)) - 1u)));
        }
    };
    auto chunk = [&](int32_t v, int32_t e, int32_t base, uint32_t bit, const uint2 q) {
        edge(v, e, base, bit, q.x & 0xFFFFu);
        edge(v, e, base, bit, q.x >> 16);
        edge(v, e, base, bit, q.y & 0xFFFFu);
        edge(v, e, base, bit, q.y >> 16);
    };
    for (int32_t i = i0; i < i1; ++i) {
        const uint32_t bit = 1u << i;
        const int32_t base = (i - i0) * stride;
        // lists come longest first: a wave each, then a thread each
        for (int32_t t = tid >> 6; t < count; t += T >> 6) {
            const int32_t v = listed_node(l, t, a.cap, W1);
            const int32_t c0 = a.g.off[v], c1 = a.g.off[v + 1];
            if (c1 - c0 <= kWaveChunks) break;
            if (!(l.st.open(v) & bit)) continue;
            for (int32_t c = c0 + (tid & 63); c < c1; c += 64) chunk(v, base + 1 + t, base, bit, ids[c]);
        }
    }
    for (int32_t i = i0; i < i1; ++i) {
        const uint32_t bit = 1u << i;
        const int32_t base = (i - i0) * stride;
        for (int32_t t = tid; t < count; t += T) {
            const int32_t v = listed_node(l, t, a.cap, W1);
            if (!(l.st.open(v) & bit)) continue;
            const int32_t c0 = a.g.off[v], c1 = a.g.off[v + 1];
            if (c1 - c0 > kWaveChunks) continue;
            for (int32_t c = c0; c < c1; ++c) chunk(v, base + 1 + t, base, bit, ids[c]);
        }
    }
    __syncthreads();
    // (no re-pointing on the way: it could undo an entry already at its root)
    for (int32_t e = tid; e < entries; e += T) par.set(e, par.root(e));
    __syncthreads();
    // a representative's entry becomes its count, kept below zero so that it
    // is not taken for a parent
    constexpr int32_t kCount = INT32_MIN;
    for (int32_t e = tid; e < entries; e += T)
        if (par.get(e) == e) par.set(e, kCount + 1);
    __syncthreads();
    for (int32_t e = tid; e < entries; e += T) {
        const int32_t r = par.get(e);
        if (r >= 0) atomicAdd(par.p + r, 1);
    }
    __syncthreads();
    for (int32_t i = i0; i < i1; ++i) {
        const uint32_t bit = 1u << i;
        const int32_t base = (i - i0) * stride;
        for (int32_t t0 = 0; t0 < count; t0 += T) {
            const int32_t t = t0 + tid;
            int32_t s = 0;  // the set this entry represents
            bool out = false;
            if (t < count && (l.st.open(listed_node(l, t, a.cap, W1)) & bit)) {
                const int32_t r = par.get(base + 1 + t);
                out = r != base;
                if (r < 0) s = r - kCount;
            }
            const uint64_t m = __ballot(out);
            if (m && (tid & 63) == 0) {
                atomicAdd(&sm.outside[i], __popcll(m));
                atomicMax(&sm.big[i], 1);
            }
            if (s > 1) {
                atomicMax(&sm.big[i], s);
                atomicAdd(&sm.sum[i], a.forest ? (unsigned long long)(s - 1)
                                               : (unsigned long long)s * (unsigned long long)(s - 1) / 2);
            }
        }
    }
}

// Counts pairs (node, individual) whose node is a component of its own, one
// node a lane: it counts as removed from here on.  Whole wave.
__device__ __forceinline__ void count_singles(CompSums &sm, uint32_t single, int32_t members)
{
    if (__ballot(single != 0) == 0) return;
    for (int32_t i = 0; i < members; ++i) {
        const uint64_t m = __ballot((single >> i) & 1u);
        if (m && (threadIdx.x & 63) == 0) {
            atomicAdd(&sm.removed[i], __popcll(m));
            atomicMax(&sm.big[i], 1);
        }
    }
}

// One sweep over all nodes with an edge, in rank order: a node is reached in
// the individuals one of its first four neighbours is.  kSweepNodes nodes a
// thread at a time, the chunks of the next ones loaded meanwhile; nothing here
// waits for a second load.  Returns the (node, individual) pairs the thread
// reached.
template <int kBits>
__device__ __forceinline__ int32_t sweep_heads(const CompView &a, const CompLds<kBits> &l)
{
    const int32_t T = blockDim.x, tid = threadIdx.x, n1 = a.n1;
    int32_t added = 0;
    if (n1 == 0) return 0;
    uint2 next[kSweepNodes];
#pragma unroll
    for (int u = 0; u < kSweepNodes; ++u) next[u] = a.g.head[min(u * T + tid, n1 - 1)];
    for (int32_t b = 0; b < n1; b += kSweepNodes * T) {
        uint2 head[kSweepNodes];
#pragma unroll
        for (int u = 0; u < kSweepNodes; ++u) {
            head[u] = next[u];
            next[u] = a.g.head[min(b + (kSweepNodes + u) * T + tid, n1 - 1)];
        }
#pragma unroll
        for (int u = 0; u < kSweepNodes; ++u) {
            const int32_t v = b + u * T + tid;
            if (v >= n1) break;
            const uint2 x = l.st.get(v);
            const uint32_t open = ~(x.x | x.y) & States<kBits>::kAll;
            if (open) {
                const uint32_t gain = l.st.any_reached(head[u]) & open;
                if (gain) l.st.put(v, x.x | gain, x.y);  // no other thread writes it now
                added += __popc(gain);
            }
        }
    }
    return added;
}

// Fitness of the individuals [z0, z0 + members) of a view, members <= kBits.
// Whole block; ends with a barrier.
template <int kBits>
__device__ __forceinline__ void eval_group(const CompView &a, const CompLds<kBits> &l, CompSums &sm, int32_t z0, int32_t members)
{
    constexpr uint32_t kAll = States<kBits>::kAll;
    const int32_t n = a.g.n, n1 = a.n1;
    const int32_t T = blockDim.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = T >> 6;
    const int32_t *off = a.g.off;
    const uint2 *ids = a.g.ids;
    // members past the last count as removing every node
    l.st.clear(n, kAll & ~((1u << members) - 1u));
    if (tid < 3) sm.added[tid] = sm.seen[tid] = 0;
    if (tid == 0) sm.queued = sm.hub = 0;
    if (tid < kGroup) {
        sm.root[tid] = n1;
        sm.removed[tid] = a.k;
        sm.outside[tid] = sm.big[tid] = 0;
        sm.sum[tid] = 0;
    }
    __syncthreads();
    // the removed nodes; every gene counts as a removed node with an edge, less
    // the repeated ones, the isolated ones and those that are no nodes
    const int32_t *rows = a.genes + (int64_t)z0 * a.k;
    for (int32_t e = tid; e < members * a.k; e += T) {
        const int32_t i = e / a.k, v = rows[e];
        bool counts = false;
        if (v >= 0 && v < n) {
            const int32_t r = a.g.rank[v];
            counts = !((l.st.or_removed(r, 1u << i) >> i) & 1u) && r < n1;
        } else {
            atomicOr(a.flag, 1);
        }
        if (!counts) atomicSub(&sm.removed[i], 1);
    }
    __syncthreads();
    // roots: the first surviving rank, a wave an individual
    for (int32_t i = wv; i < members; i += nw) {
        int32_t root = n1;
        for (int32_t b = 0; b < n1; b += 64) {
            const uint64_t m = __ballot(b + lane < n1 && !((l.st.removed(b + lane) >> i) & 1u));
            if (m) {
                root = b + (int32_t)__ffsll((unsigned long long)m) - 1;
                break;
            }
        }
        if (lane == 0 && root < n1) {
            sm.root[i] = root;
            l.st.or_reached(root, 1u << i);
        }
    }
    __syncthreads();
    // The roots' surviving neighbours are reached, and queued; while they are
    // few and no hub among them, their neighbours in turn (without hubs, a
    // sweep that starts from a handful of reached nodes gets little further;
    // with one, it gets most of the way, and pushing the hub's list is slow).
    auto push = [&](int32_t u, uint32_t bits) {
        const uint32_t alive = bits & ~l.st.removed(u);
        if (!alive) return;
        if (alive & ~l.st.or_reached(u, alive)) {
            if (u < a.g.n_hub) sm.hub = 1;
            const int32_t at = atomicAdd(&sm.queued, 1);
            if (at < a.cap) l.list[at] = (uint16_t)u;
        }
    };
    auto push_chunk = [&](const uint2 q, uint32_t bits) {
        push(q.x & 0xFFFFu, bits);
        push(q.x >> 16, bits);
        push(q.y & 0xFFFFu, bits);
        push(q.y >> 16, bits);
    };
    // (the waves share the individuals out evenly, or a wave takes several)
    const int32_t ways = min(members, nw);
    for (int32_t i = wv % ways; i < members; i += ways) {
        const int32_t root = sm.root[i];
        if (root >= n1) continue;
        const int32_t sharing = (nw - 1 - wv % ways) / ways + 1, c0 = off[root], c1 = off[root + 1];
        const bool many = c1 - c0 > T / 8;  // too many to push on from
        for (int32_t c = c0 + wv / ways * 64 + lane; c < c1; c += sharing * 64) {
            const uint2 q = ids[c];
            if (!many) {
                push_chunk(q, 1u << i);
                continue;
            }
            const uint32_t u[4] = {q.x & 0xFFFFu, q.x >> 16, q.y & 0xFFFFu, q.y >> 16};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (!((l.st.removed(u[e]) >> i) & 1u)) l.st.or_reached(u[e], 1u << i);
        }
        if (many && lane == 0) sm.hub = 1;
    }
    __syncthreads();
    for (int32_t level = 0, q0 = 0; n1 > T && level < kPushLevels; ++level) {
        const int32_t q1 = min(sm.queued, a.cap);
        const bool hub = sm.hub;
        __syncthreads();  // everyone has read it before it grows again
        if (q1 == q0 || q1 - q0 > T || hub) break;
        for (int32_t q = q0 + tid / kPushLanes; q < q1; q += T / kPushLanes) {
            const int32_t v = l.list[q];
            const uint32_t bits = l.st.get(v).x;
            const int32_t c1 = off[v + 1];
            for (int32_t c = off[v] + tid % kPushLanes; c < c1; c += kPushLanes) push_chunk(ids[c], bits);
        }
        q0 = q1;
        __syncthreads();
    }
    // Sweeps over all nodes, until a round or two of the list hold the rest,
    // while the last one reached an eighth of the open pairs, or half as many
    // as had been reached before.
    const int32_t few = min(2 * T, max(T, n1 / 6));
    int32_t open = 0, found = 0;
    for (int32_t i = 0; i < members; ++i) open += n1 - sm.removed[i];
    for (int32_t s = 0; n1 > T && s < kFullSweeps; ++s) {
        const int32_t added = wave_sum(sweep_heads(a, l));
        if (lane == 0 && added) atomicAdd(&sm.added[s % 3], added);
        if (tid == 0) sm.added[(s + 1) % 3] = 0;
        __syncthreads();
        const int32_t now = sm.added[s % 3];
        open -= now;
        if (open <= few || now == 0 || (now < open / 8 && now < found / 2)) break;
        found += now;
    }
    // A look at node v's list: reaches it in the individuals one of its neighbours
    // is reached in.  One whose neighbours are all removed is a component of its
    // own; it counts as removed from here on, and is returned.  Sets seen's bit 0 if
    // something was reached, 1 if the node stays open, 2 if its list was cut short.
    auto look = [&](int32_t v, int32_t &seen) {
        const uint2 x = l.st.get(v);
        const uint32_t want = ~(x.x | x.y) & kAll;
        uint32_t single = 0;
        if (want) {
            const int32_t c0 = off[v], c1 = off[v + 1], ce = min(c1, c0 + kLaterChunks);
            uint32_t acc = 0, gone = kAll;  // reached in some neighbour; removed in every neighbour
            for (int32_t c = c0; c < ce && (acc & want) != want; ++c) {
                const uint2 q = ids[c];
                const uint2 y0 = l.st.get(q.x & 0xFFFFu), y1 = l.st.get(q.x >> 16);
                const uint2 y2 = l.st.get(q.y & 0xFFFFu), y3 = l.st.get(q.y >> 16);
                acc |= y0.x | y1.x | y2.x | y3.x;
                gone &= y0.y & y1.y & y2.y & y3.y;
            }
            acc &= want;
            if (ce == c1) single = want & ~acc & gone;
            if (acc | single) l.st.put(v, x.x | acc, x.y | single);
            seen |= (acc ? 1 : 0) | ((acc | single) == want ? 0 : ce < c1 ? 6 : 2);
        }
        return single;
    };
    // Sweeps over the list of the nodes still open (those that fit it; if they do
    // not, after one over all nodes.  A star of 60k nodes without its centre, 8
    // individuals 73 us, 1024 126; without that sweep 264 and 951).
    int32_t count = n1;
    if (n1 <= T) {
        // one round holds every node
        if (tid < n1) l.list[tid] = (uint16_t)tid;
        for (int32_t w = tid; w < (n1 + 31) / 32; w += T) {
            l.listed[w] = ~0u;
            l.before[w] = 32 * w;
        }
        __syncthreads();
    } else {
        count = list_open(l, sm, n1, a.cap);
        if (count > a.cap) {
            for (int32_t v0 = 0; v0 < n1; v0 += T) {
                int32_t seen = 0;
                const uint32_t single = v0 + tid < n1 ? look(v0 + tid, seen) : 0u;
                count_singles(sm, single, members);
            }
            __syncthreads();
            count = list_open(l, sm, n1, a.cap);
        }
    }
    bool settled = count <= a.cap;  // no open node touches a reached one
    bool left = count > a.cap;      // some node is open
    for (int32_t s = 0; count > 0 && s < kSweeps; ++s) {
        int32_t seen = 0;
        for (int32_t t0 = 0; t0 < min(count, a.cap); t0 += T) {
            const int32_t t = t0 + tid;
            const uint32_t single = t < min(count, a.cap) ? look(l.list[t], seen) : 0u;
            count_singles(sm, single, members);
        }
        const uint64_t m0 = __ballot(seen & 1), m1 = __ballot(seen & 2), m2 = __ballot(seen & 4);
        if (lane == 0 && (m0 | m1 | m2)) atomicOr(&sm.seen[s % 3], (m0 ? 1 : 0) | (m1 ? 2 : 0) | (m2 ? 4 : 0));
        if (tid == 0) sm.seen[(s + 1) % 3] = 0;
        __syncthreads();
        const int32_t all = sm.seen[s % 3];
        if (s + 1 == kSweeps || !(all & 1)) {
            settled = settled && !(all & 5);
            left = left || (all & 2);
            break;
        }
    }
    if (left) {  // uniform over the block
        // a list that is mostly closed again, or did not fit, is made anew
        if (count > a.cap || count * members > 2 * T) count = list_open(l, sm, n1, a.cap);
        const int32_t at_once = a.cap / (count + 1);
        if (at_once > 0)
            for (int32_t i = 0; i < members; i += at_once)
                count_open<kBits, true>(a, l, sm, Parents<true>{l.parents}, count, i, min(members, i + at_once), settled);
        else
            for (int32_t i = 0; i < members; ++i)
                count_open<kBits, false>(a, l, sm, Parents<false>{a.spill}, count, i, i + 1, settled);
        __syncthreads();
    }
    // MCN where nothing with an edge survives: 1 if an isolated node does
    int32_t least = 0;
    if (wv == 0 && a.mcn)
        for (uint64_t bare = __ballot(lane < members && sm.root[min(lane, kGroup - 1)] >= n1); bare; bare &= bare - 1) {
            const int32_t i = (int32_t)__ffsll((unsigned long long)bare) - 1;
            bool any = false;
            for (int32_t v = n1; v < n && !any; v += 64)
                any = __ballot(v + lane < n && !((l.st.removed(min(v + lane, n - 1)) >> i) & 1u)) != 0;
            if (lane == i) least = any;
        }
    if (tid < members) {
        const int32_t z = z0 + tid;
        const int64_t s = sm.root[tid] < n1 ? n1 - sm.removed[tid] - sm.outside[tid] : 0;
        a.fitness[z] = (int64_t)sm.sum[tid] + (s > 0 ? (a.forest ? s - 1 : s * (s - 1) / 2) : 0);
        if (a.mcn) a.mcn[z] = max(max((int32_t)s, sm.big[tid]), least);
    }
    __syncthreads();
}

template <int kBits>
__device__ __forceinline__ CompLds<kBits> comp_carve(uint8_t *lds, const CompView &a)
{
    const int32_t n16 = (a.g.n + 15) / 16 * 16, W1 = (a.n1 + 31) / 32;
    CompLds<kBits> l;
    l.st.s = lds;
    l.st.rem = kBits == 8 ? lds + n16 : nullptr;
    l.listed = reinterpret_cast<uint32_t *>(lds + (kBits == 8 ? 2 : 1) * n16);
    l.before = reinterpret_cast<int32_t *>(l.listed + W1);
    l.parents = l.before + W1;
    l.list = reinterpret_cast<uint16_t *>(l.parents + a.cap);
    return l;
}

// P individuals of one graph, `group` to a workgroup at a time.
template <int kBits>
__global__ __launch_bounds__(1024) void k_components(CompView a, int32_t P, int32_t group)
{
    extern __shared__ __align__(16) uint8_t comp_lds[];
    __shared__ CompSums sm;
    const CompLds<kBits> l = comp_carve<kBits>(comp_lds, a);
    if (a.spill) a.spill += (int64_t)blockIdx.x * (a.n1 + 1);
    for (int32_t z = blockIdx.x * group; z < P; z += gridDim.x * group) eval_group(a, l, sm, z, min(group, P - z));
}

// The elitism of the generation before, not launched by itself: every block
// finds the merged order of the parents and their children for itself.
struct MergeArgs {
    const int64_t *f_par, *f_child;  // fitness of the parents, ascending, and of their children
    const int32_t *children;         // the children's rows
    int32_t *pop_out;                // out: the merged population, P rows
    int64_t *fit_out;                // and its fitness
    int32_t lds_at;                  // bytes of LDS before this
    uint32_t ahead;                  // generations since the counter was advanced
};

// Sources of the P positions of the merged population (parent t: t, child c:
// P + c), in LDS, and the fitness of all keys by source.  A parent's position
// is its own and the children below it; a child's the children below it, by
// (fitness, index), and the parents not above it (as k_rank_rows has it).  The
// threads share the children a key is compared with evenly.
__device__ __forceinline__ const int32_t *merged_order(const MergeArgs &m, int32_t P, int32_t L, uint8_t *lds,
                                                       const int64_t *&fitness)
{
    const int32_t T = blockDim.x, tid = threadIdx.x, keys = P + L;
    int64_t *f = reinterpret_cast<int64_t *>(lds + m.lds_at);
    int32_t *pos = reinterpret_cast<int32_t *>(f + keys), *src = pos + keys;
    for (int32_t t = tid; t < keys; t += T) {
        f[t] = t < P ? m.f_par[t] : m.f_child[t - P];
        pos[t] = 0;
    }
    __syncthreads();
    const int32_t parts = T / keys, t = tid % keys, part = tid / keys;  // (keys <= T)
    if (part < parts) {
        const int64_t mine = f[t];
        int32_t below = 0;
#pragma unroll 4
        for (int32_t j = part; j < L; j += parts) {
            const int64_t x = f[P + j];
            below += x < mine || (x == mine && j < t - P);
        }
        if (part == 0) {
            int32_t lo = 0, hi = P;
            while (t >= P && lo < hi) {
                const int32_t mid = (lo + hi) >> 1;
                if (f[mid] <= mine) lo = mid + 1;
                else hi = mid;
            }
            below += t < P ? t : lo;
        }
        if (below) atomicAdd(&pos[t], below);
    }
    __syncthreads();
    for (int32_t x = tid; x < keys; x += T)
        if (pos[x] < P) src[pos[x]] = x;
    __syncthreads();
    fitness = f;
    return src;
}

// A generation's children, one to a workgroup: bred and evaluated in one launch
// (the operators' LDS and the evaluation's share the block's, one after the
// other; the child's row comes back from the lines just written).  With kMerge
// the population they come from is first merged from the one before and its
// children, and written out by the blocks, a row or a few each.
template <bool kMerge>
__global__ __launch_bounds__(1024) void k_breed_components(CompView a, OpArgs args, MergeArgs m)
{
    extern __shared__ __align__(16) uint8_t comp_lds[];
    __shared__ CompSums sm;
    __shared__ OpSums os;
    const Op op = resolve(args);
    const int32_t o = blockIdx.x;
    const int64_t *f = nullptr;
    const int32_t *src = kMerge ? merged_order(m, op.P, op.L, comp_lds, f) : nullptr;
    auto row = [&](int32_t p) {
        if constexpr (kMerge) {
            const int32_t t = src[p];
            return t < op.P ? op.pop + (int64_t)t * op.k : m.children + (int64_t)(t - op.P) * op.k;
        } else {
            return op.pop + (int64_t)p * op.k;
        }
    };
    if constexpr (kMerge)
        for (int32_t p = o; p < op.P; p += gridDim.x) {
            const int32_t *from = row(p);
            for (int32_t j = threadIdx.x; j < op.k; j += blockDim.x) m.pop_out[(int64_t)p * op.k + j] = from[j];
            if (threadIdx.x == 0) m.fit_out[p] = f[src[p]];
        }
    make_child(carve(reinterpret_cast<uint32_t *>(comp_lds), op), op, os, o, *args.gen_ctr + 1u + m.ahead, row);
    if (a.spill) a.spill += (int64_t)o * (a.n1 + 1);
    __syncthreads();
    eval_group(a, comp_carve<4>(comp_lds, a), sm, o, 1);
}

// Tasks (instance, first individual, individuals, 0) of many instances, the
// largest graphs first.  A block takes one of every gridDim.x, forwards and
// backwards in turn, so that large tasks meet small ones.
__global__ __launch_bounds__(1024) void k_components_batch(const CompInst *__restrict__ insts,
                                                           const int4 *__restrict__ tasks, int32_t ntasks,
                                                           const unsigned char *__restrict__ lists,
                                                           const int32_t *__restrict__ children,
                                                           int64_t *__restrict__ fitness, int32_t *__restrict__ mcn,
                                                           int32_t forest, int32_t *__restrict__ flag,
                                                           int32_t *__restrict__ spill, int32_t spill_stride)
{
    extern __shared__ __align__(16) uint8_t comp_lds[];
    __shared__ CompSums sm;
    const int32_t B = gridDim.x;
    for (int32_t r = 0; r * B < ntasks; ++r) {
        const int32_t t = r * B + ((r & 1) ? B - 1 - (int32_t)blockIdx.x : (int32_t)blockIdx.x);
        if (t >= ntasks) continue;
        const int4 task = tasks[t];
        const CompInst &I = insts[task.x];
        const CompView a{children + I.child_off, I.k, neighbour_lists(lists + I.lists_off, I.n, I.chunks, I.n_hub),
                         I.n1, I.cap, spill + (int64_t)blockIdx.x * spill_stride, fitness + I.slot_off,
                         mcn ? mcn + I.slot_off : nullptr, forest, flag};
        if (I.bits == 4) eval_group(a, comp_carve<4>(comp_lds, a), sm, task.y, task.z);
        else eval_group(a, comp_carve<8>(comp_lds, a), sm, task.y, task.z);
    }
}

// Launch shape for P individuals: threads enough for a few rounds over the
// nodes; a workgroup a compute unit (small ones: two or four) before a
// workgroup takes more than one individual; four individuals a workgroup at
// most where two bytes a node would leave little LDS for leftover nodes; room
// in LDS for every node to be left over, as far as it goes.
struct CompShape {
    int32_t bits, threads, group, blocks, cap;
    size_t lds;
};

constexpr size_t kCompLds = 156 * 1024;
constexpr int32_t kWideNodes = 40000;

// Threads of a block for P individuals: one a node on the smallest graphs (their
// one round over the nodes needs no list: n = 200 8.4 us against 10.3, n = 500
// 13.0 against 13.8), as long as that leaves no compute unit short of blocks.
int32_t comp_threads(int32_t n, int64_t P)
{
    return n <= 256 ? 256 : n <= 512 ? 512 : n <= 1024 && P <= 256 ? 1024 : n <= 4096 ? 512 : 1024;
}

// Individuals of a workgroup, to fill `room` workgroups with P.
int32_t comp_group(int32_t n, int64_t P, int32_t room)
{
    return (int32_t)std::min<int64_t>(n <= kWideNodes ? kGroup : 4, (P + room - 1) / room);
}

// LDS entries for leftover nodes (all a graph of n1 nodes with an edge can
// have, as far as `lds` bytes go), and the LDS bytes with them.
int32_t comp_cap(int32_t bits, int32_t n, int32_t n1, size_t lds, size_t *used)
{
    const size_t fixed = bits == 4 ? comp_lds_fixed<4>(n, n1) : comp_lds_fixed<8>(n, n1);
    const int32_t cap = (int32_t)std::min<size_t>((size_t)n1 + 1, (lds - fixed) / 6);
    *used = fixed + (size_t)cap * 6;
    return cap;
}

int32_t comp_per_cu(int32_t threads, size_t lds)
{
    return (int32_t)std::min<size_t>(2048 / threads, (160 * 1024) / (lds + 1024));
}

CompShape comp_shape(const gapa_graph *g, int32_t P, size_t spill_bytes)
{
    CompShape c{};
    c.threads = comp_threads(g->n, P);
    const int32_t per_cu = 1024 / c.threads;
    c.group = comp_group(g->n, P, 256 * per_cu);
    c.bits = c.group <= 4 ? 4 : 8;
    c.cap = comp_cap(c.bits, g->n, g->n_noniso, kCompLds / per_cu, &c.lds);
    const int32_t groups = (P - 1) / c.group + 1;
    c.blocks = std::min(groups, 256 * comp_per_cu(c.threads, c.lds));
    if (c.cap <= g->n_noniso)
        c.blocks = (int32_t)std::min<size_t>((size_t)c.blocks, spill_bytes / (((size_t)g->n_noniso + 1) * 4));
    return c;
}

template <int kBits>
int launch_components(const CompShape &c, const CompView &a, int32_t P, hipStream_t s)
{
    if (c.lds > 60 * 1024)  // (always the same limit: threads on other graphs launch the kernel too)
        GAPA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_components<kBits>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCompLds));
    hipLaunchKernelGGL(k_components<kBits>, dim3((unsigned)c.blocks), dim3(c.threads), c.lds, s, a, P, c.group);
    GAPA_HIP(hipGetLastError());
    return GAPA_OK;
}

}  // namespace

// On a graph of long paths (a lattice, a road network) the sweeps leave most
// nodes to the union-find; where LDS does not hold them all, the bit-parallel
// pass, which spreads the union-finds over the whole chip, is kept (shuffled
// lattice of 240 x 240: 8 individuals 1.3 ms against 2.2, 1024 3.4 against 12.8).
//
// So it is for few individuals on graphs with more nodes than LDS lists outside
// the component of the node of highest degree: they go through a slice of global
// memory of each workgroup, which pays once enough workgroups do that side by
// side.  n = 60k, bit-parallel pass against workgroups: stars of 50 nodes, 8
// individuals 209 us against 979, 64 630 against 1053, 128 1173 against 1191, 256
// 2224 against 1477; paths of 20, 64 776 against 1152, 256 2436 against 1609;
// random graph of mean degree 0.8, 8 305 against 538, 64 550 against 567, 128 800
// against 630; a star beside a path, 64 846 against 1177, 128 1448 against 1347;
// beside a lattice, 32 1.4 ms against 2.2, 1024 13.9 against 12.0.
//
// (Trees fall into pieces only without their hubs.  With and without most of
// those, 8 individuals: BA m = 1 0.98 ms against 0.21, 0.67 against 0.82; random
// recursive tree 0.84 against 1.41, 0.40 against 0.93.  From 64 individuals on
// workgroups are 0.9 to 4 times as fast.)
bool components_fit(const gapa_graph *g, int64_t P)
{
    constexpr int64_t kLooseRows = 128;
    return g->d_lists && (g->loose ? P >= kLooseRows : !g->deep);
}

size_t components_spill_bytes(const gapa_graph *g, int32_t P)
{
    const CompShape c = comp_shape(g, P, SIZE_MAX);
    return c.cap > g->n_noniso ? 0 : (size_t)c.blocks * ((size_t)g->n_noniso + 1) * 4;
}

int eval_rows_components(gapa_graph *g, const int32_t *genes, int32_t P, int32_t k, int64_t *fitness, int32_t *mcn,
                         int32_t *flag, void *spill, size_t spill_bytes, KernelTimer *timer, hipStream_t s,
                         Measure measure)
{
    if (P <= 0) return GAPA_OK;
    constexpr int32_t kMost = 1 << 30;  // of a launch: its blocks step past the last individual
    if (P > kMost) {
        const int rc = eval_rows_components(g, genes, kMost, k, fitness, mcn, flag, spill, spill_bytes, timer, s, measure);
        if (rc != GAPA_OK) return rc;
        return eval_rows_components(g, genes ? genes + (int64_t)kMost * k : nullptr, P - kMost, k, fitness + kMost,
                                    mcn ? mcn + kMost : nullptr, flag, spill, spill_bytes, timer, s, measure);
    }
    const CompShape c = comp_shape(g, P, spill_bytes);
    if (c.blocks < 1) return GAPA_E_INVALID_ARG;
    const CompView a{genes, k, neighbour_lists(g), g->n_noniso, c.cap,
                     c.cap > g->n_noniso ? nullptr : static_cast<int32_t *>(spill), fitness, mcn, (int32_t)measure, flag};
    TimedScope pass(timer, "fitness_pass", s, 1);
    TimedScope ts(timer, "k_components", s);
    return c.bits == 4 ? launch_components<4>(c, a, P, s) : launch_components<8>(c, a, P, s);
}

int eval_rows_components_ws(gapa_graph *g, const int32_t *genes, int32_t P, int32_t k, int64_t *fitness, int32_t *mcn,
                            int32_t *flag, FitnessWorkspace &ws, KernelTimer *timer, hipStream_t s, Measure measure)
{
    const size_t spill = components_spill_bytes(g, P);
    const int rc = ws.spill.reserve(spill);
    if (rc != GAPA_OK) return rc;
    return eval_rows_components(g, genes, P, k, fitness, mcn, flag, ws.spill.ptr, spill, timer, s, measure);
}

// One launch breeds and evaluates a generation of one GA while every child has a
// workgroup of its own (a workgroup that takes several would breed them one
// after the other).  n = 200, P = 32: a generation 15.8 us against 18.4; n = 10k,
// P = 256: 27.7 against 29.1 (its launch and the row's way through memory are
// saved, but a block of 1024 threads breeds more slowly than one of 256).
bool components_breed(const gapa_ga *ga)
{
    const CompShape c = comp_shape(ga->graph, ga->lambda, SIZE_MAX);
    return c.group == 1 && c.blocks == ga->lambda && ga->op_lds_bytes <= c.lds;
}

// Several generations of one call run at a launch each, the elitism of one in the
// next one's launch, while the blocks find the merged order sooner than a launch
// of its own does: while a thread compares its key with 32 children at the most.
// n = 200: P = 8 15.1 us a generation against 13.2, P = 32 15.6 and 14.0, P = 64
// (32 comparisons) 16.4 and 15.9; n = 10k, P = 128 (32) 27.1 and 26.1; n = 2000, P
// = 128 (64) 21.7 and 22.3.
bool ga_merges(const gapa_ga *ga)
{
    if (!ga->by_rows || ga->count != 1 || ga->surr || ga->objective_mcn || ga->timer.level ||
        ga->max_pop_lambda > kMergeKeys || ga->op_lds_bytes > kCompLds / 2)
        return false;
    const int32_t parts = comp_threads(ga->graph->n, ga->lambda) / ga->max_pop_lambda;
    return ga->lambda <= 32 * parts && components_breed(ga);
}

template <bool kMerge>
static int launch_breed(const CompShape &c, size_t lds, const CompView &a, const OpArgs &args, const MergeArgs &m,
                        hipStream_t s)
{
    if (lds > 60 * 1024)
        GAPA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_breed_components<kMerge>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCompLds));
    hipLaunchKernelGGL(k_breed_components<kMerge>, dim3((unsigned)c.blocks), dim3(c.threads), lds, s, a, args, m);
    GAPA_HIP(hipGetLastError());
    return GAPA_OK;
}

int breed_rows_components(gapa_ga *ga, int32_t *mcn, hipStream_t s, Measure measure, int32_t ahead)
{
    const gapa_graph *g = ga->graph;
    const size_t spill = components_spill_bytes(g, ga->lambda);
    const CompShape c = comp_shape(g, ga->lambda, spill);
    const int rc = ga->ws.spill.reserve(spill);
    if (rc != GAPA_OK) return rc;
    MergeArgs m{};
    size_t lds = c.lds;
    if (ahead > 0) {
        ga->swap_children();
        m.f_par = ga->fit[ga->cur].as<int64_t>();
        m.f_child = ga->child_fit_prev.as<int64_t>();
        m.children = ga->children_prev.as<int32_t>();
        m.pop_out = ga->pop[1 - ga->cur].as<int32_t>();
        m.fit_out = ga->fit[1 - ga->cur].as<int64_t>();
        m.lds_at = (int32_t)((ga->op_lds_bytes + 15) & ~(size_t)15);
        m.ahead = (uint32_t)ahead;
        lds = std::max(lds, m.lds_at + 12 * (size_t)ga->max_pop_lambda + 4 * (size_t)ga->max_pop);
    }
    const OpArgs args = op_args(ga, ga->pop[ga->cur].as<int32_t>());
    const CompView a{args.children, ga->params.k, neighbour_lists(g), g->n_noniso, c.cap,
                     c.cap > g->n_noniso ? nullptr : ga->ws.spill.as<int32_t>(), ga->child_fit.as<int64_t>(), mcn,
                     (int32_t)measure, ga->flag.as<int32_t>() + 3};
    if (ahead > 0) ga->cur = 1 - ga->cur;
    return ahead > 0 ? launch_breed<true>(c, lds, a, args, m, s) : launch_breed<false>(c, lds, a, args, m, s);
}

// Instance table and tasks of a batch: `init` for the initial population, else
// for a generation's children.
int components_batch_plan(gapa_ga *ga, gapa_graph *const *graphs, bool init)
{
    CompBatch &cb = init ? ga->comp_init : ga->comp_gen;
    const int32_t count = ga->count;
    int32_t n_max = 0;
    int64_t total = 0;
    for (const GaInst &I : ga->hinst) {
        n_max = std::max(n_max, I.n);
        total += init ? I.P : I.L;
    }
    cb.threads = comp_threads(n_max, total);
    const int32_t per_cu = 1024 / cb.threads;
    std::vector<CompInst> insts((size_t)count);
    std::vector<int4> tasks;
    std::vector<int32_t> by_size((size_t)count);
    for (int32_t b = 0; b < count; ++b) by_size[b] = b;
    std::sort(by_size.begin(), by_size.end(), [&](int32_t x, int32_t y) {
        return ga->hinst[x].n != ga->hinst[y].n ? ga->hinst[x].n > ga->hinst[y].n : x < y;
    });
    cb.lds = 0;
    cb.spill_stride = 0;
    int64_t lists_bytes = 0;
    for (int32_t b = 0; b < count; ++b) {
        insts[b].lists_off = lists_bytes;
        lists_bytes += (int64_t)((neighbour_lists_bytes(graphs[b]->n, graphs[b]->list_chunks) + 255) & ~(size_t)255);
    }
    for (int32_t b : by_size) {
        const GaInst &I = ga->hinst[b];
        CompInst &c = insts[b];
        const int32_t group = comp_group(I.n, total, 256 * per_cu), live = init ? I.P : I.L;
        c.n = I.n;
        c.chunks = graphs[b]->list_chunks;
        c.n_hub = graphs[b]->n_hub;
        c.k = I.k;
        c.n1 = I.n_noniso;
        c.bits = group <= 4 ? 4 : 8;
        size_t used = 0;
        c.cap = comp_cap(c.bits, I.n, c.n1, kCompLds / per_cu, &used);
        c.child_off = I.child_off;
        c.slot_off = I.slot_off;
        cb.lds = std::max(cb.lds, used);
        if (c.cap <= c.n1) cb.spill_stride = std::max(cb.spill_stride, c.n1 + 1);
        for (int32_t z = 0; z < live; z += group) tasks.push_back(make_int4(b, z, std::min(group, live - z), 0));
    }
    cb.ntasks = (int32_t)tasks.size();
    cb.blocks = std::min(cb.ntasks, 256 * comp_per_cu(cb.threads, cb.lds));
    int rc;
    if ((rc = cb.insts.reserve(insts.size() * sizeof(CompInst))) != GAPA_OK) return rc;
    if ((rc = cb.tasks.reserve(tasks.size() * sizeof(int4))) != GAPA_OK) return rc;
    if ((rc = ga->ws.spill.reserve((size_t)cb.blocks * cb.spill_stride * 4)) != GAPA_OK) return rc;
    DevBuf &lists = ga->comp_init.lists;
    if (!lists.ptr) {
        if ((rc = lists.reserve((size_t)lists_bytes)) != GAPA_OK) return rc;
        for (int32_t b = 0; b < count; ++b)
            GAPA_HIP(hipMemcpyAsync(lists.as<unsigned char>() + insts[b].lists_off, graphs[b]->d_lists,
                                    neighbour_lists_bytes(graphs[b]->n, graphs[b]->list_chunks),
                                    hipMemcpyDeviceToDevice, nullptr));
        GAPA_HIP(hipStreamSynchronize(nullptr));
    }
    GAPA_HIP(hipMemcpy(cb.insts.ptr, insts.data(), insts.size() * sizeof(CompInst), hipMemcpyHostToDevice));
    GAPA_HIP(hipMemcpy(cb.tasks.ptr, tasks.data(), tasks.size() * sizeof(int4), hipMemcpyHostToDevice));
    return GAPA_OK;
}

int eval_rows_components_batch(gapa_ga *ga, bool init, int32_t *mcn, hipStream_t s, Measure measure)
{
    const CompBatch &cb = init ? ga->comp_init : ga->comp_gen;
    if (cb.lds > 60 * 1024)
        GAPA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_components_batch),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCompLds));
    TimedScope pass(&ga->timer, "fitness_pass", s, 1);
    TimedScope ts(&ga->timer, "k_components", s);
    hipLaunchKernelGGL(k_components_batch, dim3((unsigned)cb.blocks), dim3(cb.threads), cb.lds, s,
                       cb.insts.as<CompInst>(), cb.tasks.as<int4>(), cb.ntasks,
                       ga->comp_init.lists.as<unsigned char>(), ga->children.as<int32_t>(),
                       ga->child_fit.as<int64_t>(), mcn, (int32_t)measure, ga->flag.as<int32_t>() + 3,
                       ga->ws.spill.as<int32_t>(), cb.spill_stride);
    GAPA_HIP(hipGetLastError());
    return GAPA_OK;
}

}  // namespace gapa
