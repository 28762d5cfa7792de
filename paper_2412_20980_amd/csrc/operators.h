// The genetic operators of one workgroup: the initial individual's draws, and a
// child from selection to its sorted row.  Every function here is called by all
// threads of the block (a multiple of 64, at most 1024).
#pragma once

#include <climits>

#include "device_common.h"
#include "internal.h"

namespace gapa {
namespace {

// Launch arguments: buffer bases shared by all instances of the launch.
struct OpArgs {
    const GaInst *inst;       // [instances]
    const int32_t *pop;       // current population rows, ascending
    const uint32_t *noniso;   // non-isolated node bit sets
    int32_t *children;        // out: child rows, ascending
    uint32_t *masks;          // out: removed-node bit set of each child
    int32_t *alive;           // out: surviving non-isolated nodes of each child
    int32_t *flag;            // [1] attempts exhausted
    const uint32_t *gen_ctr;  // [1] generations completed
    int32_t rows_only;        // emit only the rows (no bit sets, no alive counts)
};

// One instance's view, resolved by each block from the table.
struct Op {
    const int32_t *pop;     // [P][k]
    const uint32_t *noniso; // [W] bit v set: v has an edge
    int32_t *children;      // [L][k]
    uint32_t *masks;        // [L][W]
    int32_t *alive;         // [L]
    int32_t *flag;
    uint64_t seed, t_pc, t_pm;
    int32_t P, L, k, n, W, KW, T, n_noniso, log_q;
    int32_t rows_only;
};

__device__ __forceinline__ Op resolve(const OpArgs &a)
{
    const GaInst &I = a.inst[blockIdx.y];
    Op o;
    o.pop = a.pop ? a.pop + I.pop_off : nullptr;
    o.noniso = a.noniso + I.noniso_off;
    o.children = a.children + I.child_off;
    o.masks = a.masks + I.mask_off;
    o.alive = a.alive + I.slot_off;
    o.flag = a.flag;
    o.seed = I.seed;
    o.t_pc = I.t_pc;
    o.t_pm = I.t_pm;
    o.P = I.P;
    o.L = I.L;
    o.k = I.k;
    o.n = I.n;
    o.W = I.W;
    o.KW = I.KW;
    o.T = I.T;
    o.n_noniso = I.n_noniso;
    o.log_q = I.log_q;
    o.rows_only = a.rows_only;
    return o;
}

// LDS of one operator block: membership bits over the nodes, the row by slot,
// a list of slots (16-bit: the LDS limit keeps k far below 65536), and three
// bit sets over the slots.  Once the row is complete the list's room holds the
// number of members before each quad of the set's words.  Kept small so that
// four blocks fit a compute unit at n = 200k, k = 2000.
struct OpLds {
    uint32_t *U;          // [W, rounded up to a multiple of 4]
    int32_t *row;         // [k]
    uint32_t *from_donor; // [KW]
    uint32_t *dup;        // [KW]
    uint32_t *mut;        // [KW]
    uint16_t *list;       // [max(k, quads)]
};

__device__ __forceinline__ OpLds carve(uint32_t *smem, const Op &a)
{
    OpLds l;
    l.U = smem;
    l.row = reinterpret_cast<int32_t *>(smem + ((a.W + 3) & ~3));
    l.from_donor = reinterpret_cast<uint32_t *>(l.row + a.k);
    l.dup = l.from_donor + a.KW;
    l.mut = l.dup + a.KW;
    l.list = reinterpret_cast<uint16_t *>(l.mut + a.KW);
    return l;
}

__device__ __forceinline__ bool lds_test(const uint32_t *U, uint32_t v)
{
    return (U[v >> 5] >> (v & 31)) & 1u;
}

__device__ __forceinline__ void lds_set(uint32_t *U, uint32_t v)
{
    U[v >> 5] |= 1u << (v & 31);
}

// Starting from candidate u (attempt t0), the first attempt of
// (slot, ind, gen, stream | t) that is not a member; -1 if attempts run out.
__device__ __forceinline__ int32_t first_non_member(const uint32_t *U, uint32_t u, uint32_t t0, uint64_t seed, uint32_t slot,
                                    uint32_t ind, uint32_t gen, uint32_t stream, uint32_t n)
{
    uint32_t t = t0;
    while (lds_test(U, u)) {
        if (++t >= kMaxAttempts) return -1;
        u = bounded(draw(seed, slot, ind, gen, stream, t).w0, n);
    }
    return (int32_t)u;
}

// The defining rule, in slot order: slot list[a] (a = 0, 1, ...) takes the
// first draw (slot, ind, gen, stream | t), t = 0, 1, ..., that is not in the
// membership set U; U gains it and, with `swap`, loses the slot's previous
// value.  One wave resolves 64 slots at a time: every lane takes its attempt
// 0, and lane l's draw is accepted if it is not a member (checked against U
// as it stood before the batch) and no earlier lane drew the same value.  All
// lanes before the first rejected one are committed at once; the rejected
// one is resolved alone with further attempts from its attempt 0, exactly as
// the sequential rule would given the committed lanes; the next batch starts
// after it.  A draw equal to a value an earlier lane frees (swap) is
// rejected too and then accepted by the lone resolution: the same result.
//
// With `pre` (no swap), slot j's attempt-0 value was computed beforehand by
// the whole block and stored in row[j] (the slot's old value is not needed).
//
// Equal draws within the batch are found through U itself: every candidate
// not yet a member sets its bit with an atomic OR, and a lane that finds its
// bit already set by another lane of the batch marks a collision.  Without
// one (the usual case) no lane is taken; with one the lanes compare values
// directly.  Bits set for lanes that are not committed are cleared again.
__device__ __forceinline__ void wave_draw_in_order(const OpLds &l, const Op &a, const uint16_t *list, int32_t count, bool swap,
                                   uint32_t ind, uint32_t gen, uint32_t stream, bool pre = false)
{
    const int lane = threadIdx.x & 63;
    int32_t pos = 0;
    while (pos < count) {
        const int32_t nvalid = min(64, count - pos);
        const bool valid = lane < nvalid;
        const int32_t j = valid ? (list ? list[pos + lane] : pos + lane) : 0;
        // attempt 0 of slot j: drawn here, or (pre, no swap) already in row[j]
        const uint32_t c = !valid ? 0u : pre ? (uint32_t)l.row[j] : bounded(draw(a.seed, j, ind, gen, stream, 0).w0, a.n);
        const int32_t old = (valid && swap) ? l.row[j] : -1;
        const uint32_t w = c >> 5, bit = 1u << (c & 31);
        // membership before the batch: every lane reads before any lane writes
        const bool in_u = valid && (l.U[w] & bit);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        bool mine = false, clash = false;
        if (valid && !in_u) {
            const uint32_t prev = atomicOr(&l.U[w], bit);
            mine = !(prev & bit);
            clash = !mine;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        bool taken = false;
        if (__ballot(clash) != 0) {
            // q is uniform across the wave: lane q's value is read with readlane
            for (int q = 0; q < nvalid; ++q) {
                const uint32_t cq = (uint32_t)__builtin_amdgcn_readlane((int)c, q);
                taken |= q < lane && cq == c;
            }
        }
        const bool reject = valid && (in_u || taken);
        const uint64_t rej = __ballot(reject);
        const int32_t f = rej ? (int32_t)__ffsll((unsigned long long)rej) - 1 : nvalid;
        // lanes from f on are not committed: clear the bits they set
        if (mine && lane >= f) atomicAnd(&l.U[w], ~bit);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (lane < f) {
            // (a committed value whose bit a later, uncommitted lane with the
            // same draw had set and just cleared is set again)
            atomicOr(&l.U[w], bit);
            if (swap) atomicAnd(&l.U[old >> 5], ~(1u << (old & 31)));
            l.row[j] = (int32_t)c;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (f < nvalid) {
            if (lane == f) {
                const int32_t u = first_non_member(l.U, c, 0, a.seed, j, ind, gen, stream, a.n);
                if (u < 0) {
                    atomicOr(a.flag, 1);
                } else {
                    if (swap) l.U[old >> 5] &= ~(1u << (old & 31));
                    lds_set(l.U, u);
                    l.row[j] = u;
                }
            }
            pos += f + 1;
        } else {
            pos += nvalid;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
}

constexpr int kScanWaves = 16;  // waves of a block, at most

// Exclusive prefix sum over the block (blockDim.x <= 1024, a multiple of 64) of
// counts that add up to less than 65536; also returns the block total.  Every thread must call it.
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t x, int32_t *total)
{
    __shared__ uint16_t s_wave[kScanWaves];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int32_t incl = wave_scan(x);
    if (lane == 63) s_wave[wv] = (uint16_t)incl;
    __syncthreads();
    int32_t before = 0, sum = 0;
    for (int q = 0; q < (int)(blockDim.x >> 6); ++q) {
        if (q < wv) before += s_wave[q];
        sum += s_wave[q];
    }
    __syncthreads();
    *total = sum;
    return before + incl - x;
}

// Slots whose bit is set in bits[0 .. ceil(k/32)), ascending, into list[];
// returns how many.  Whole block: each thread enumerates a contiguous run of
// words at the offset a block scan of their popcounts gives.  The list is
// visible to every thread on return.
__device__ __forceinline__ int32_t block_list_slots(const uint32_t *bits, int32_t k, uint16_t *list)
{
    const int32_t KW = (k + 31) / 32;
    const int32_t per = (KW + (int32_t)blockDim.x - 1) / (int32_t)blockDim.x;
    const int32_t w0 = min(KW, (int32_t)threadIdx.x * per), w1 = min(KW, w0 + per);
    int32_t cnt = 0;
    for (int32_t w = w0; w < w1; ++w) cnt += __popc(bits[w]);
    int32_t total = 0;
    int32_t off = block_exclusive_scan(cnt, &total);
    for (int32_t w = w0; w < w1; ++w)
        for (uint32_t x = bits[w]; x; x &= x - 1) list[off++] = (uint16_t)(w * 32 + __ffs(x) - 1);
    __syncthreads();
    return total;
}

__device__ __forceinline__ void clear_lds(const OpLds &l, const Op &a)
{
    for (int32_t w = threadIdx.x; w < (a.W + 3) / 4; w += blockDim.x)
        reinterpret_cast<uint4 *>(l.U)[w] = uint4{0u, 0u, 0u, 0u};
    for (int32_t w = threadIdx.x; w < a.KW; w += blockDim.x) l.from_donor[w] = l.dup[w] = l.mut[w] = 0u;
}

__device__ __forceinline__ int32_t popc4(const uint4 x)
{
    return __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w);
}

// Flags of one operator block.
struct OpSums {
    int32_t donor;
    int32_t dups, muts;  // whether any slot is a duplicate, or mutates
    int32_t gone;        // removed non-isolated nodes
};
static_assert(sizeof(OpSums) + sizeof(uint16_t) * kScanWaves == kOpStaticLds, "LDS declared in the operator kernels");

// The finished individual leaves as its row in ascending order and, where the
// fitness kernels consume them, its membership bit set (the removed-node mask)
// and its count of surviving non-isolated nodes (n_noniso minus the genes that
// have an edge).
//
// A gene's place in the row is the number of members below it: the members
// before its quad of words (2^log_q words, four unless LDS is short), from one
// pass over the set, and those of the quad below it.  That is a read of 16
// bytes or two a gene; enumerating the set's bits in order instead, every thread
// over its own run of words, takes a read and a loop over bits for each of the
// n / 32 words, mostly empty ones, one after the other (n = 200k, k = 2000: 10.0 of
// a block's 23.5 us, against 5.6 of 16.8).
__device__ __forceinline__ void emit(const OpLds &l, const Op &a, OpSums &sm, int32_t idx)
{
    const int32_t T = blockDim.x;
    if (threadIdx.x == 0) sm.gone = 0;
    __syncthreads();
    if (!a.rows_only) {
        uint32_t *m = a.masks + (int64_t)idx * a.W;
        int32_t w = threadIdx.x;
        for (; w + 7 * T < a.W; w += 8 * T) {
            uint32_t x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = l.U[w + u * T];
#pragma unroll
            for (int u = 0; u < 8; ++u) m[w + u * T] = x[u];
        }
        for (; w < a.W; w += T) m[w] = l.U[w];
    }
    const uint4 *U4 = reinterpret_cast<const uint4 *>(l.U);
    uint16_t *before = l.list;
    const int32_t W4 = (a.W + 3) / 4, per_q = 1 << (a.log_q - 2), quads = (W4 + per_q - 1) / per_q;
    // (an odd number of quads each: threads side by side read different banks)
    const int32_t per = ((quads + T - 1) / T) | 1;
    const int32_t q0 = min(quads, (int32_t)threadIdx.x * per), q1 = min(quads, q0 + per);
    int32_t cnt = 0;
    for (int32_t w = q0 * per_q; w < min(W4, q1 * per_q); ++w) cnt += popc4(U4[w]);
    int32_t total = 0;
    int32_t off = block_exclusive_scan(cnt, &total);
    for (int32_t q = q0; q < q1; ++q) {
        before[q] = (uint16_t)off;
        for (int32_t w = q * per_q; w < min(W4, (q + 1) * per_q); ++w) off += popc4(U4[w]);
    }
    __syncthreads();
    int32_t *dst = a.children + (int64_t)idx * a.k;
    const bool whole = total == a.k;  // not if attempts ran out: the row is no permutation of the set then
    int32_t gone = 0;
#pragma unroll 4
    for (int32_t j = threadIdx.x; j < a.k; j += T) {
        const int32_t c = l.row[j], w = c >> 7;
        int32_t r = before[c >> (a.log_q + 5)];
        for (int32_t x = c >> (a.log_q + 5) << (a.log_q - 2); x < w; ++x) r += popc4(U4[x]);
        const uint4 x = U4[w];
        const uint64_t lo = (uint64_t)x.y << 32 | x.x, hi = (uint64_t)x.w << 32 | x.z;
        const uint64_t below = (1ull << (c & 63)) - 1ull;
        r += __popcll((c & 64 ? hi : lo) & below) + (c & 64 ? __popcll(lo) : 0);
        dst[whole ? r : j] = c;
        if (!a.rows_only) gone += (a.noniso[c >> 5] >> (c & 31)) & 1u;
    }
    if (!a.rows_only) {
        gone = wave_sum(gone);
        if ((threadIdx.x & 63) == 0 && gone) atomicAdd(&sm.gone, gone);
        __syncthreads();
        if (threadIdx.x == 0) a.alive[idx] = a.n_noniso - sm.gone;
    }
    if (threadIdx.x == 0 && !whole) atomicOr(a.flag, 1);
}

// Position of value c in the ascending base row staged in bs[0, k): galloping
// from slot j (the rows of a converged population differ by small shifts),
// then a binary search inside the bracket.  c must be in the row.
__device__ __forceinline__ int32_t base_position(const int32_t *bs, int32_t k, int32_t j, int32_t c)
{
    int32_t lo, hi;
    if (bs[j] < c) {
        int32_t b = 1;
        while (j + b < k && bs[j + b] < c) b <<= 1;
        lo = j + (b >> 1) + 1;
        hi = min(j + b, k);
    } else {
        int32_t b = 1;
        while (j - b >= 0 && bs[j - b] >= c) b <<= 1;
        lo = max(j - b + 1, 0);
        hi = j - (b >> 1);
    }
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (bs[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Rows up to kOpSlots genes a thread keep each thread's base and donor
// genes in registers from the crossover to the row fill (slot j = thread +
// T i, T the block's threads); longer rows read them again from global memory.
constexpr int kOpSlots = 8;

// Offspring o of generation gen >= 1.
//   base  = POP[o mod P]; donor = tournament winner (smallest (PC, position)
//           among T uniform draws with replacement; contestant c is word c mod 4
//           of SELECT draw slot c / 4).  The population is ordered by (PC,
//           position), so the winner is the smallest position drawn.
//   eq. 6 gene j = donor[j] where the crossover mask (eq. 4) word-0 coin of
//           XOVER draw j is below floor(pc 2^32), else base[j]; word 1 of the
//           same draw is the mutation coin of eq. 8.
//   repair  a slot whose value already sits at a lower slot gets a uniform
//           non-member (REPAIR draws), slots ascending.
//   eq. 9   each mutated slot, ascending, swaps its gene for a uniform
//           non-member (MUTATE draws).
//   sort    the row ascending.
// row(p) points at the row at position p of the population.
template <class Row>
__device__ __forceinline__ void make_child(const OpLds &l, const Op &a, OpSums &sm, int32_t o, uint32_t gen,
                                           const Row &row)
{
    const int32_t T = blockDim.x;
    if (threadIdx.x < 64) {
        int32_t best = INT_MAX;
        const int32_t c = threadIdx.x;
        if (c < a.T) {  // (at most 64)
            const Words4 w = draw(a.seed, (uint32_t)(c >> 2), o, gen, kStreamSelect, 0);
            best = (int32_t)bounded((c & 3) == 0 ? w.w0 : (c & 3) == 1 ? w.w1 : (c & 3) == 2 ? w.w2 : w.w3, (uint32_t)a.P);
        }
        for (int32_t x = 1; x < a.T; x <<= 1) best = min(best, __shfl_xor(best, x, 64));
        if (threadIdx.x == 0) {
            sm.donor = best;
            sm.dups = sm.muts = 0;
        }
    }
    clear_lds(l, a);
    __syncthreads();

    const int32_t *base = row(o % a.P);
    const int32_t *donor = row(sm.donor);
    const bool regs = a.k <= T * kOpSlots;
    int32_t bv[kOpSlots], dv[kOpSlots];
    uint32_t takes = 0u;  // bit i: slot threadIdx.x + T i takes the donor gene
    // Crossover coins; the base row is staged in LDS (row[] holds it while
    // duplicates are located), values taken from it enter the membership set.
    if (regs) {
#pragma unroll
        for (int i = 0; i < kOpSlots; ++i) {
            const int32_t j = threadIdx.x + T * i;
            bv[i] = j < a.k ? base[j] : 0;
            dv[i] = j < a.k ? donor[j] : 0;
        }
#pragma unroll
        for (int i = 0; i < kOpSlots; ++i) {
            const int32_t j = threadIdx.x + T * i;
            if (j >= a.k) break;
            const Words4 x = draw(a.seed, j, o, gen, kStreamXover, 0);
            const bool take = (uint64_t)x.w0 < a.t_pc;
            l.row[j] = bv[i];
            if (take) takes |= 1u << i;
            else atomicOr(&l.U[bv[i] >> 5], 1u << (bv[i] & 31));
            if ((uint64_t)x.w1 < a.t_pm) {
                atomicOr(&l.mut[j >> 5], 1u << (j & 31));
                sm.muts = 1;
            }
        }
    } else {
#pragma unroll 4
        for (int32_t j = threadIdx.x; j < a.k; j += blockDim.x) {
            const Words4 x = draw(a.seed, j, o, gen, kStreamXover, 0);
            const bool take = (uint64_t)x.w0 < a.t_pc;
            const int32_t b = base[j];
            l.row[j] = b;
            if (take) atomicOr(&l.from_donor[j >> 5], 1u << (j & 31));
            else atomicOr(&l.U[b >> 5], 1u << (b & 31));
            if ((uint64_t)x.w1 < a.t_pm) {
                atomicOr(&l.mut[j >> 5], 1u << (j & 31));
                sm.muts = 1;
            }
        }
    }
    __syncthreads();

    // Base and donor rows are ascending and distinct, so a value occurs at most
    // twice in the child: once from each row.  A donor value c that is already
    // a member came from the base row at the slot p where base[p] = c; the
    // later of p and j is the copy.  Other donor values join the set.
    if (regs) {
#pragma unroll
        for (int i = 0; i < kOpSlots; ++i) {
            if (!((takes >> i) & 1u)) continue;
            const int32_t j = threadIdx.x + T * i;
            const int32_t c = dv[i];
            if (lds_test(l.U, c)) {
                const int32_t p = base_position(l.row, a.k, j, c);
                const int32_t later = p < j ? j : p;
                atomicOr(&l.dup[later >> 5], 1u << (later & 31));
                sm.dups = 1;
            } else {
                atomicOr(&l.U[c >> 5], 1u << (c & 31));
            }
        }
    } else {
#pragma unroll 2
        for (int32_t j = threadIdx.x; j < a.k; j += blockDim.x) {
            if (!((l.from_donor[j >> 5] >> (j & 31)) & 1u)) continue;
            const int32_t c = donor[j];
            if (lds_test(l.U, c)) {
                const int32_t p = base_position(l.row, a.k, j, c);
                const int32_t later = p < j ? j : p;
                atomicOr(&l.dup[later >> 5], 1u << (later & 31));
                sm.dups = 1;
            } else {
                atomicOr(&l.U[c >> 5], 1u << (c & 31));
            }
        }
    }
    __syncthreads();
    // the child's row by slot: donor values where the coin took the donor
    if (regs) {
#pragma unroll
        for (int i = 0; i < kOpSlots; ++i)
            if ((takes >> i) & 1u) l.row[threadIdx.x + T * i] = dv[i];
    } else {
        for (int32_t j = threadIdx.x; j < a.k; j += blockDim.x)
            if ((l.from_donor[j >> 5] >> (j & 31)) & 1u) l.row[j] = donor[j];
    }
    __syncthreads();

    // Repair, then mutation, each in ascending slot order by one wave.  The
    // slot lists are built by the whole block, and so are the repair slots'
    // attempt-0 draws (a repaired slot's duplicate value is not needed, so the
    // draw takes its place in row[]).
    if (sm.dups) {
        const int32_t nd = block_list_slots(l.dup, a.k, l.list);
        for (int32_t q = threadIdx.x; q < nd; q += T) {
            const int32_t j = l.list[q];
            l.row[j] = (int32_t)bounded(draw(a.seed, j, o, gen, kStreamRepair, 0).w0, a.n);
        }
        __syncthreads();
        if (threadIdx.x < 64) wave_draw_in_order(l, a, l.list, nd, false, o, gen, kStreamRepair, true);
        __syncthreads();
    }
    if (sm.muts) {
        const int32_t nm = block_list_slots(l.mut, a.k, l.list);
        if (threadIdx.x < 64) wave_draw_in_order(l, a, l.list, nm, true, o, gen, kStreamMutate);
    }
    emit(l, a, sm, o);
}

// Arguments of a launch for every instance of ga, breeding from the rows in pop.
inline OpArgs op_args(gapa_ga *ga, const int32_t *pop)
{
    OpArgs a;
    a.inst = ga->inst.as<GaInst>();
    a.pop = pop;
    a.noniso = ga->noniso ? ga->noniso : ga->graph->d_noniso;
    a.children = ga->children.as<int32_t>();
    a.masks = ga->masks.as<uint32_t>();
    a.alive = ga->alive.as<int32_t>();
    a.flag = ga->flag.as<int32_t>();
    a.gen_ctr = ga->gen_ctr.as<uint32_t>();
    a.rows_only = ga->by_rows ? 1 : 0;
    return a;
}

}  // namespace
}  // namespace gapa
