// The paper's dense reachability fitness (Sec. III-D, eq. 13-17).  For each
// removal set S:
//
//   M1 = A_S + I     A_S: the adjacency with every edge of a removed node
//                    deleted (eq. 13)
//   M  = Normalizer(M1^hops)   (entries > 0 become 1)
//   pc = (sum M - n) / 2,  mcn = the largest row sum over surviving nodes
//
// With hops at least the diameter of every component this is (PC, MCN)
// exactly; the paper's hops = 6 (eq. 15) truncates.  Exact integers.  Two
// ways to the same numbers, chosen by what each would cost (sixdst_sparse):
//
//   - k_six_reach: row v of M is the set of nodes within `hops` hops of v, so
//     the product with the sparse M1 is an OR over v's neighbours.  A block
//     keeps the sets of every node, restricted to 32 NW sources, as bits in
//     LDS and advances them hop by hop.
//   - k_six_gemm: M1 as an n_pad x n_pad 0/1 int8 matrix (n_pad = n rounded
//     up to 128; padding rows and columns are zero) raised to the power by
//     binary exponentiation on the matrix cores, the products
//     (A+I)(A+I)^2(A+I)^4... of the paper, each normalised.  Its cost grows
//     with log(hops) and not with the edges: for many hops on dense graphs.
//     Every matrix is a power of one symmetric matrix, so every product is
//     symmetric and column j of the right operand is its row j: both
//     operands of the int8 products (v_mfma_i32_16x16x64_i8) are read as
//     rows.
#include <algorithm>

#include "device_common.h"
#include "internal.h"

namespace gapa {
namespace {

constexpr int kTile = 128;   // output tile of a block; matrices are padded to a multiple of it
constexpr int kLd = 80;      // LDS row stride of a 64-byte k-step (16 rows of one read fall in distinct banks)
typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bool removed(const uint32_t *mask, int32_t v)
{
    return (mask[v >> 5] >> (v & 31)) & 1u;
}

// Row i of M1 for individual z (block (i, z)).
__global__ __launch_bounds__(256) void k_six_build(const uint32_t *__restrict__ masks, int32_t W,
                                                   const int32_t *__restrict__ row_ptr,
                                                   const int32_t *__restrict__ col, int32_t n, int32_t np,
                                                   uint8_t *__restrict__ M)
{
    const int32_t i = blockIdx.x, z = blockIdx.y;
    uint8_t *row = M + ((int64_t)z * np + i) * np;
    const uint32_t *mask = masks + (int64_t)z * W;
    for (int32_t c = threadIdx.x; c < np / 16; c += blockDim.x) reinterpret_cast<uint4 *>(row)[c] = uint4{0, 0, 0, 0};
    __syncthreads();
    if (i >= n) return;
    if (threadIdx.x == 0) row[i] = 1;
    if (removed(mask, i)) return;
    for (int32_t e = row_ptr[i] + threadIdx.x; e < row_ptr[i + 1]; e += blockDim.x) {
        const int32_t j = col[e];
        if (!removed(mask, j)) row[j] = 1;
    }
}

// C = Normalizer(A B) for individual blockIdx.y, A and B symmetric powers of
// one matrix, so C is symmetric: block t computes the 128 x 128 tile
// (bi, bj), bi <= bj, the t-th of the upper triangle, and writes it and its
// mirror image.  The four waves take 64 x 64 quadrants (4 x 4 MFMA tiles
// each).  Per k-step of 64 bytes the 128 A rows and the 128 B rows (B
// columns) of the step are staged in LDS (80-byte pitch: the 16 rows one
// operand read touches fall in distinct banks), double-buffered: the next
// step's global loads are in flight during the products.  MFMA operands:
// lane l holds bytes 16 (l / 16) .. + 15 of the step for row / column
// l % 16 (the same byte order on both sides); C[4 (l / 16) + r][l % 16].
constexpr int kStage = kTile * kLd;    // one operand tile of one k-step
constexpr int kOutPitch = kTile + 16;  // output tile pitch in LDS
__global__ __launch_bounds__(256) void k_six_gemm(const uint8_t *__restrict__ A, const uint8_t *__restrict__ B,
                                                  uint8_t *__restrict__ C, int32_t np)
{
    __shared__ __align__(16) uint8_t smem[4 * kStage];  // [buffer][A, B][128][kLd]
    const int64_t base = (int64_t)blockIdx.y * np * np;
    // t = bj (bj + 1) / 2 + bi
    const int32_t t_lin = blockIdx.x;
    int32_t bj = (int32_t)((sqrtf(8.f * (float)t_lin + 1.f) - 1.f) * 0.5f);
    while ((bj + 1) * (bj + 2) / 2 <= t_lin) ++bj;
    while (bj * (bj + 1) / 2 > t_lin) --bj;
    const int32_t bi = t_lin - bj * (bj + 1) / 2;
    const int32_t i0 = bi * kTile, j0 = bj * kTile;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lg = lane >> 4;
    const int wr = wv >> 1, wc = wv & 1;
    // loader: thread t moves bytes 16 (t % 4) .. + 15 of rows t / 4 and 64 + t / 4 of both tiles
    const int lrow = t >> 2, lcol = (t & 3) * 16;
    const uint8_t *ga = A + base + (int64_t)(i0 + lrow) * np + lcol;
    const uint8_t *gb = B + base + (int64_t)(j0 + lrow) * np + lcol;
    const int64_t half = (int64_t)64 * np;
    uint4 ra0 = *reinterpret_cast<const uint4 *>(ga), ra1 = *reinterpret_cast<const uint4 *>(ga + half);
    uint4 rb0 = *reinterpret_cast<const uint4 *>(gb), rb1 = *reinterpret_cast<const uint4 *>(gb + half);
    i32x4 acc[4][4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[x][y] = i32x4{0, 0, 0, 0};
    const int32_t steps = np / 64;
    for (int32_t s = 0; s < steps; ++s) {
        uint8_t *sA = smem + (s & 1) * 2 * kStage, *sB = sA + kStage;
        *reinterpret_cast<uint4 *>(&sA[lrow * kLd + lcol]) = ra0;
        *reinterpret_cast<uint4 *>(&sA[(64 + lrow) * kLd + lcol]) = ra1;
        *reinterpret_cast<uint4 *>(&sB[lrow * kLd + lcol]) = rb0;
        *reinterpret_cast<uint4 *>(&sB[(64 + lrow) * kLd + lcol]) = rb1;
        __syncthreads();
        if (s + 1 < steps) {
            const int64_t o = (int64_t)(s + 1) * 64;
            ra0 = *reinterpret_cast<const uint4 *>(ga + o);
            ra1 = *reinterpret_cast<const uint4 *>(ga + half + o);
            rb0 = *reinterpret_cast<const uint4 *>(gb + o);
            rb1 = *reinterpret_cast<const uint4 *>(gb + half + o);
        }
        i32x4 a[4], b[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) a[x] = *reinterpret_cast<const i32x4 *>(&sA[(wr * 64 + 16 * x + lr) * kLd + lg * 16]);
#pragma unroll
        for (int y = 0; y < 4; ++y) b[y] = *reinterpret_cast<const i32x4 *>(&sB[(wc * 64 + 16 * y + lr) * kLd + lg * 16]);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y) acc[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[x], b[y], acc[x][y], 0, 0, 0);
    }
    // normalised tile through LDS, then written as 16-byte row pieces
    __syncthreads();
    uint8_t *out = smem;
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                out[(wr * 64 + 16 * x + 4 * lg + r) * kOutPitch + wc * 64 + 16 * y + lr] = acc[x][y][r] > 0 ? 1 : 0;
    __syncthreads();
    const int orow = t >> 1, ocol = (t & 1) * 64;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint4 *>(C + base + (int64_t)(i0 + orow) * np + j0 + ocol + 16 * q) =
            *reinterpret_cast<const uint4 *>(&out[orow * kOutPitch + ocol + 16 * q]);
    if (bi != bj) {
        // the mirror tile: row orow of it is column orow of this one
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t w[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                w[d] = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[d] |= (uint32_t)out[(ocol + 16 * q + 4 * d + e) * kOutPitch + orow] << (8 * e);
            }
            *reinterpret_cast<uint4 *>(C + base + (int64_t)(j0 + orow) * np + i0 + ocol + 16 * q) =
                uint4{w[0], w[1], w[2], w[3]};
        }
    }
}

// Row sums of M: block (g, z) takes rows 32 g .. 32 g + 31 of individual z,
// one wave per row at a time; the block adds its rows' total and largest
// surviving row into the individual's counters (integer atomics, order-free).
constexpr int kRowsPerBlock = 32;
__global__ __launch_bounds__(256) void k_six_rows(const uint8_t *__restrict__ M, const uint32_t *__restrict__ masks,
                                                  int32_t W, int32_t n, int32_t np,
                                                  unsigned long long *__restrict__ total, int32_t *__restrict__ mcn)
{
    __shared__ uint32_t s_sum[4], s_max[4];
    const int32_t z = blockIdx.y;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t *mask = masks + (int64_t)z * W;
    uint32_t bsum = 0, bmax = 0;
    for (int32_t r = wv; r < kRowsPerBlock; r += 4) {
        const int32_t i = blockIdx.x * kRowsPerBlock + r;
        if (i >= n) break;
        const uint4 *row = reinterpret_cast<const uint4 *>(M + ((int64_t)z * np + i) * np);
        uint32_t sum = 0;
        for (int32_t c = lane; c < np / 16; c += 64) {
            const uint4 q = row[c];
            // entries are 0 or 1: the byte sum of a word is its popcount
            sum += __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        bsum += sum;
        if (!removed(mask, i)) bmax = max(bmax, sum);
    }
    if (lane == 0) {
        s_sum[wv] = bsum;
        s_max[wv] = bmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t t = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
        const uint32_t m = max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3]));
        if (t) atomicAdd(total + z, (unsigned long long)t);
        if (m) atomicMax(mcn + z, (int32_t)m);
    }
}

__global__ void k_six_final(const unsigned long long *__restrict__ total, int32_t count, int32_t n,
                            int64_t *__restrict__ pc)
{
    const int32_t z = blockIdx.x * blockDim.x + threadIdx.x;
    if (z < count) pc[z] = ((int64_t)total[z] - n) / 2;
}

// Clears the outputs of P individuals and the gene flag.
__global__ void k_six_clear(int64_t *__restrict__ pc, int32_t *__restrict__ mcn, int32_t P, int32_t *__restrict__ flag)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < P) {
        pc[i] = 0;
        mcn[i] = 0;
    }
    if (i < 4) flag[i] = 0;
}

// NW words of one node's reached sources.
template <int NW>
struct Bits {
    uint32_t w[NW];
};

template <int NW>
__device__ __forceinline__ Bits<NW> ld_bits(const uint32_t *p)
{
    Bits<NW> b;
    if constexpr (NW == 4) {
        const uint4 q = *reinterpret_cast<const uint4 *>(p);
        b.w[0] = q.x, b.w[1] = q.y, b.w[2] = q.z, b.w[3] = q.w;
    } else {
        const uint2 q = *reinterpret_cast<const uint2 *>(p);
        b.w[0] = q.x, b.w[1] = q.y;
    }
    return b;
}

template <int NW>
__device__ __forceinline__ void st_bits(uint32_t *p, const Bits<NW> &b)
{
    if constexpr (NW == 4) *reinterpret_cast<uint4 *>(p) = uint4{b.w[0], b.w[1], b.w[2], b.w[3]};
    else *reinterpret_cast<uint2 *>(p) = uint2{b.w[0], b.w[1]};
}

// OR over the 16 lanes of a row, in every lane.
__device__ __forceinline__ uint32_t row_or(uint32_t x)
{
    x |= lane_xor<1>(x);
    x |= lane_xor<2>(x);
    x |= lane_xor<4>(x);
    return x | lane_xor<8>(x);
}

// Full adder on 32 bit columns: a becomes the sum, the carry is returned.
__device__ __forceinline__ uint32_t add_bits(uint32_t &a, uint32_t b, uint32_t c)
{
    const uint32_t carry = (a & b) | (c & (a | b));
    a ^= b ^ c;
    return carry;
}

// Bit counts of the 32 columns of 15 words: plane p holds bit p of each count.
struct Planes {
    uint32_t p0, p1, p2, p3;
};

__device__ __forceinline__ Planes count_bits15(const uint32_t (&x)[15])
{
    uint32_t ones = x[0], c[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) c[i] = add_bits(ones, x[2 * i + 1], x[2 * i + 2]);
    uint32_t twos = c[0], d[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) d[i] = add_bits(twos, c[2 * i + 1], c[2 * i + 2]);
    uint32_t fours = d[0];
    const uint32_t eights = add_bits(fours, d[1], d[2]);
    return Planes{ones, twos, fours, eights};
}

// ORs into acc the sets of the four nodes of one chunk of a neighbour list.
template <int NW>
__device__ __forceinline__ void or_chunk(Bits<NW> &acc, const uint32_t *sets, const uint2 c)
{
    const Bits<NW> a = ld_bits<NW>(sets + (c.x & 0xFFFFu) * NW), b = ld_bits<NW>(sets + (c.x >> 16) * NW);
    const Bits<NW> d = ld_bits<NW>(sets + (c.y & 0xFFFFu) * NW), e = ld_bits<NW>(sets + (c.y >> 16) * NW);
#pragma unroll
    for (int q = 0; q < NW; ++q) acc.w[q] |= a.w[q] | b.w[q] | d.w[q] | e.w[q];
}

// Whether b holds every bit of full.
template <int NW>
__device__ __forceinline__ bool covers(const Bits<NW> &b, const Bits<NW> &full)
{
    uint32_t miss = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) miss |= full.w[q] & ~b.w[q];
    return miss == 0;
}

constexpr int kHubLanes = 16;  // lanes that pull a node of more than kHubDegree neighbours

// Reachability from 32 NW sources of one removal set, a task a time: task t
// takes the sources [32 NW sb, 32 NW (sb + 1)), sb = t mod nsb, of individual
// t / nsb, and a block a contiguous run of tasks.  LDS: the sets of all n
// nodes twice (the hop being read and the hop being written), rows of NW
// words padded to a multiple of 32 rows; the removed-node bit set; with
// kLdsGraph also the offsets and neighbour lists, so that a task reads nothing
// from global memory but its genes.  Removed nodes have empty sets
// throughout, so no neighbour needs a test (M's 1 on their diagonal cancels
// in sum M - n).
//
// The state after hop 1 is set from the sources' own neighbour lists (one
// atomic OR an edge); every later hop is a pull: a node ORs its neighbours'
// sets, unless it has every surviving source already.  The first n_hub nodes
// are pulled by kHubLanes lanes each, the others by one.  A hop that changes
// nothing is the last.
//
// M is symmetric: the row sum of source s is the number of nodes that hold
// bit s.
//
// Bound by LDS: a hop of the BA graph (n = 2000, m = 2) reads 195 KB of sets
// and ids a task, 16-byte rows at random (about three to a bank), and takes
// 2.3 us of a task's 15 (six hops); the other 4 us are hop 1 and the counts.
// Adjacency read from global memory (order, row pointers, columns: a chain of
// three loads a node): 0.72 ms for 512 individuals against 0.48.  Two blocks of
// half the sources a compute unit: 0.78; 512 threads: 0.73.  Row sums by
// transposing every word instead of the bit planes: 0.51.
constexpr int kSumBits = 40;  // n^2 <= 2^26 for GAPA_SIXDST_MAX_N
constexpr unsigned long long kTaskDone = 1ull << kSumBits;

template <int NW, bool kLdsGraph>
__global__ __launch_bounds__(1024) void k_six_reach(const int32_t *__restrict__ genes, int32_t k, const NeighbourLists g,
                                                    int32_t hops, int32_t nsb, int64_t tasks,
                                                    unsigned long long *__restrict__ pc, int32_t *__restrict__ mcn,
                                                    int32_t *__restrict__ flag)
{
    extern __shared__ __align__(16) uint32_t six_lds[];
    __shared__ int32_t s_cnt[32 * NW];
    __shared__ int32_t s_changed[3];
    const int32_t n = g.n, W = (n + 31) / 32, rows = W * 32;
    const int32_t T = blockDim.x, tid = threadIdx.x;
    uint32_t *dead = six_lds + 2 * rows * NW;
    const int32_t *off = g.off;
    const uint2 *ids = g.ids;
    if constexpr (kLdsGraph) {
        uint2 *l_ids = reinterpret_cast<uint2 *>(dead + (W + 1) / 2 * 2);
        const int32_t chunks = g.off[n];
        int32_t *l_off = reinterpret_cast<int32_t *>(l_ids + chunks);
        for (int32_t i = tid; i < chunks; i += T) l_ids[i] = g.ids[i];
        for (int32_t i = tid; i <= n; i += T) l_off[i] = g.off[i];
        off = l_off;
        ids = l_ids;
    }
    const int32_t sub = tid % kHubLanes;
    // this block's tasks
    const int64_t per = tasks / gridDim.x, extra = tasks % gridDim.x;
    const int64_t t0 = blockIdx.x * per + min((int64_t)blockIdx.x, extra);
    const int64_t t1 = t0 + per + (blockIdx.x < extra ? 1 : 0);
    int32_t z_dead = -1;  // individual the removed-node set is of
    for (int64_t task = t0; task < t1; ++task) {
        const int32_t z = (int32_t)(task / nsb), w0 = (int32_t)(task % nsb) * NW;
        uint32_t *cur = six_lds, *nxt = six_lds + rows * NW;
        for (int32_t i = tid; i < rows * NW / 4; i += T) reinterpret_cast<uint4 *>(cur)[i] = uint4{0, 0, 0, 0};
        for (int32_t i = tid; i < 32 * NW; i += T) s_cnt[i] = 0;
        if (tid < 3) s_changed[tid] = 0;
        if (z != z_dead) {
            z_dead = z;
            // the last word's padding nodes count as removed
            for (int32_t w = tid; w < W; w += T) dead[w] = w == W - 1 && (n & 31) ? ~0u << (n & 31) : 0u;
            __syncthreads();
            for (int32_t j = tid; j < k; j += T) {
                const int32_t v = genes[(int64_t)z * k + j];
                if (v >= 0 && v < n) {
                    const int32_t r = g.rank[v];
                    atomicOr(&dead[r >> 5], 1u << (r & 31));
                } else {
                    atomicOr(flag, 1);
                }
            }
        }
        __syncthreads();
        Bits<NW> full;
#pragma unroll
        for (int q = 0; q < NW; ++q) full.w[q] = w0 + q < W ? ~dead[w0 + q] : 0u;

        // after hop 1: every surviving source and its surviving neighbours
        for (int32_t t = tid / kHubLanes; t < 32 * NW; t += T / kHubLanes) {
            const int32_t s = w0 * 32 + t;
            if (s >= n || removed(dead, s)) continue;
            const uint32_t bit = 1u << (t & 31);
            uint32_t *word = cur + (t >> 5);
            const int32_t c1 = off[s + 1];
            for (int32_t c = off[s] + sub; c < c1; c += kHubLanes) {
                const uint2 q = ids[c];
                const int32_t u[4] = {(int32_t)(q.x & 0xFFFFu), (int32_t)(q.x >> 16), (int32_t)(q.y & 0xFFFFu),
                                      (int32_t)(q.y >> 16)};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (!removed(dead, u[e])) atomicOr(word + u[e] * NW, bit);
            }
            if (sub == 0) atomicOr(word + s * NW, bit);
        }
        __syncthreads();

        for (int32_t h = 2; h <= hops; ++h) {
            bool changed = false;
            for (int32_t v = tid / kHubLanes; v < g.n_hub; v += T / kHubLanes) {
                Bits<NW> acc = ld_bits<NW>(cur + v * NW);
                const Bits<NW> mine = acc;
                if (!removed(dead, v) && !covers<NW>(mine, full)) {
                    const int32_t c1 = off[v + 1];
                    for (int32_t c = off[v] + sub; c < c1; c += kHubLanes) or_chunk<NW>(acc, cur, ids[c]);
#pragma unroll
                    for (int q = 0; q < NW; ++q) acc.w[q] = row_or(acc.w[q]);
#pragma unroll
                    for (int q = 0; q < NW; ++q) changed |= acc.w[q] != mine.w[q];
                }
                if (sub == 0) st_bits<NW>(nxt + v * NW, acc);
            }
            for (int32_t v = g.n_hub + tid; v < n; v += T) {
                Bits<NW> acc = ld_bits<NW>(cur + v * NW);
                const Bits<NW> mine = acc;
                if (!removed(dead, v) && !covers<NW>(mine, full)) {
                    const int32_t c1 = off[v + 1];
                    for (int32_t c = off[v]; c < c1; ++c) or_chunk<NW>(acc, cur, ids[c]);
#pragma unroll
                    for (int q = 0; q < NW; ++q) changed |= acc.w[q] != mine.w[q];
                }
                st_bits<NW>(nxt + v * NW, acc);
            }
            // three flags in turn: the one the hop after next will use is
            // cleared while nobody reads or sets it
            if (changed) s_changed[h % 3] = 1;
            if (tid == 0) s_changed[(h + 1) % 3] = 0;
            __syncthreads();
            uint32_t *t = cur;
            cur = nxt;
            nxt = t;
            if (!s_changed[h % 3]) break;
        }

        // row sums of the sources: a half-wave takes one word of 480 nodes,
        // 15 a lane, as bit planes of their counts; transposed, lane c of
        // plane p has the bits of source c
        const int l32 = tid & 31;
        const int32_t word_tasks = (n + 479) / 480 * NW;
        for (int32_t t = tid >> 5; t < word_tasks; t += T >> 5) {
            const int32_t q = t % NW, v0 = t / NW * 480 + l32;
            uint32_t x[15];
#pragma unroll
            for (int i = 0; i < 15; ++i) x[i] = v0 + 32 * i < n ? cur[(v0 + 32 * i) * NW + q] : 0u;
            const Planes p = count_bits15(x);
            const int32_t cnt = __popc(transpose32(p.p0, l32)) + 2 * __popc(transpose32(p.p1, l32)) +
                                4 * __popc(transpose32(p.p2, l32)) + 8 * __popc(transpose32(p.p3, l32));
            if (cnt) atomicAdd(&s_cnt[q * 32 + l32], cnt);
        }
        __syncthreads();
        if (tid < 64) {
            // row sums less the sources themselves: twice the pairs, over all
            // tasks of the individual; its last task to finish (the task count
            // is kept in the high bits of the sum) halves it
            int32_t best = 0, sum = 0;
            for (int32_t i = tid; i < 32 * NW; i += 64) {
                best = max(best, s_cnt[i]);
                sum += max(s_cnt[i] - 1, 0);
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                best = max(best, __shfl_xor(best, o, 64));
                sum += __shfl_xor(sum, o, 64);
            }
            if (tid == 0) {
                if (best) atomicMax(mcn + z, best);
                const unsigned long long old = atomicAdd(pc + z, kTaskDone + (unsigned long long)sum);
                if (old >> kSumBits == (unsigned long long)nsb - 1) pc[z] = ((old & (kTaskDone - 1)) + sum) / 2;
            }
        }
        __syncthreads();  // the sums and sets are read before the next task clears them
    }
}

// Rates the two ways are priced at: words ORed a second by the pulls (a path
// of 2000 nodes, nothing saturated, 5.8e12), multiply-adds a second by the
// products (n = 2000: 1.24e15 to 1.3e15).
constexpr double kPullRate = 6e12, kMacRate = 1.3e15;

// Launch shape of k_six_reach.  A block takes four words of sources where two
// copies of the sets (and, if they fit beside them, the neighbour lists) leave
// room for that in LDS, else two.
constexpr size_t kReachLds = 158 * 1024;
struct ReachShape {
    int32_t NW, threads;
    bool lds_graph;
    size_t lds;
};

ReachShape reach_shape(const gapa_graph *g)
{
    const size_t W = (size_t)g->words;
    const size_t graph = (size_t)g->list_chunks * 8 + ((size_t)g->n + 1) * 4;
    auto sets = [&](int32_t NW) { return 2 * W * 32 * NW * 4 + (W + 1) / 2 * 8; };
    ReachShape r{};
    r.NW = g->n > 64 && sets(4) <= kReachLds ? 4 : 2;
    if (r.NW == 4 && sets(4) + graph > kReachLds && sets(2) + graph <= kReachLds) r.NW = 2;
    r.lds_graph = sets(r.NW) + graph <= kReachLds;
    r.lds = sets(r.NW) + (r.lds_graph ? graph : 0);
    r.threads = g->n <= 384 ? 256 : r.lds <= kReachLds / 2 && g->n <= 1536 ? 512 : 1024;
    return r;
}

template <int NW, bool kLdsGraph>
int launch_reach(const ReachShape &r, int32_t blocks, const int32_t *genes, int32_t k, const gapa_graph *g,
                 int32_t hops, int32_t nsb, int64_t tasks, int64_t *pc, int32_t *mcn, int32_t *flag, hipStream_t s)
{
    // (always the same limit: threads on other graphs launch the kernel too)
    if (r.lds > 64 * 1024)
        GAPA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_six_reach<NW, kLdsGraph>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kReachLds));
    hipLaunchKernelGGL((k_six_reach<NW, kLdsGraph>), dim3((unsigned)blocks), dim3(r.threads), r.lds, s, genes, k,
                       neighbour_lists(g), hops, nsb, tasks, reinterpret_cast<unsigned long long *>(pc), mcn, flag);
    GAPA_HIP(hipGetLastError());
    return GAPA_OK;
}

}  // namespace

// Which of the two ways is taken.  The reachable sets pay for every edge at
// every hop until nothing changes, the products for the dense matrix log2(hops)
// times.  How many hops change something is not known beforehand: four times
// the breadth-first levels of G is allowed for, and at most eight times the
// products' cost if all of them did.  Measured, reachable sets against
// products: BA n = 2000 (m = 2), 512 individuals, hops = 6: 0.48 against 11.4
// ms, hops = 2: 0.21 against 4.2; random graph of mean degree 200 (256
// individuals, hops = 6): 0.98 against 5.8 ms; path of 2000 nodes (64
// individuals), 100 hops: 0.55 against 3.5 ms; n = 8192, mean degree 6 (64
// individuals, hops = 6): 1.1 against 83.7 ms.  A clique of half the nodes
// with the others as a path on it, all hops: the products (each hop changes
// every set of the clique).  What removing S does to the paths is not seen: a
// clique of 300 of 2000 nodes and a path of the others, joined by a hub that is
// removed (64 individuals), takes 6.2 ms against 3.0 with 128 hops, 3.1 against 2.6
// with 64; a tighter bound would cost sparse graphs asked for all hops more (BA m =
// 4, n = 2000: a few us an individual against 110).
bool sixdst_sparse(const gapa_graph *g, int32_t hops)
{
    const double np = (double)((g->n + kTile - 1) / kTile * kTile);
    const double hop = ((double)g->nnz + 2.0 * g->n) * g->words / kPullRate;
    int32_t products = 0;
    for (int32_t h = hops; h > 1; h >>= 1) products += 1 + (h & 1);
    const double dense = products * np * np * np / kMacRate;
    const int32_t most = std::min(hops - 1, g->n);
    return std::min(most, 4 * g->levels) * hop <= dense && most * hop <= 8.0 * dense;
}

// pc[P], mcn[P] (device) of P gene rows by reachable sets; a gene outside
// [0, n) sets flag[0].  Needs no workspace.
int sixdst_eval_genes(gapa_graph *g, const int32_t *genes, int32_t P, int32_t k, int32_t hops, int64_t *pc,
                      int32_t *mcn, int32_t *flag, hipStream_t s)
{
    const ReachShape r = reach_shape(g);
    const int32_t nsb = (g->words + r.NW - 1) / r.NW;
    const int64_t tasks = (int64_t)P * nsb;
    // as many blocks as the chip holds at once, each with its run of tasks
    const int32_t per_cu = (int32_t)std::max<size_t>(1, std::min<size_t>(2048 / r.threads, (160 * 1024) / (r.lds + 1024)));
    const int32_t blocks = (int32_t)std::min<int64_t>(tasks, 256 * per_cu);
    hipLaunchKernelGGL(k_six_clear, dim3((unsigned)((std::max<int64_t>(P, 4) + 255) / 256)), dim3(256), 0, s, pc, mcn,
                       P, flag);
    GAPA_HIP(hipGetLastError());
    if (r.NW == 4)
        return r.lds_graph ? launch_reach<4, true>(r, blocks, genes, k, g, hops, nsb, tasks, pc, mcn, flag, s)
                           : launch_reach<4, false>(r, blocks, genes, k, g, hops, nsb, tasks, pc, mcn, flag, s);
    return r.lds_graph ? launch_reach<2, true>(r, blocks, genes, k, g, hops, nsb, tasks, pc, mcn, flag, s)
                       : launch_reach<2, false>(r, blocks, genes, k, g, hops, nsb, tasks, pc, mcn, flag, s);
}

size_t sixdst_bytes_per_individual(int32_t n)
{
    const size_t np = ((size_t)n + kTile - 1) / kTile * kTile;
    return 3 * np * np;
}

// pc[P], mcn[P] (device) of the P removal sets given as bit sets masks[P][W]
// (device); mats holds three np x np matrices for each of `chunk`
// individuals, tot `chunk` counters.
int sixdst_eval_masks(gapa_graph *g, const uint32_t *masks, int32_t P, int32_t hops, int32_t chunk, uint8_t *mats,
                      unsigned long long *tot, int64_t *pc, int32_t *mcn, hipStream_t s)
{
    const int32_t n = g->n, W = g->words;
    const int32_t np = (n + kTile - 1) / kTile * kTile;
    const int64_t mat = (int64_t)np * np;
    for (int32_t z0 = 0; z0 < P; z0 += chunk) {
        const int32_t cnt = std::min(chunk, P - z0);
        const uint32_t *mk = masks + (int64_t)z0 * W;
        uint8_t *buf[3] = {mats, mats + (int64_t)cnt * mat, mats + 2 * (int64_t)cnt * mat};
        hipLaunchKernelGGL(k_six_build, dim3(np, cnt), dim3(256), 0, s, mk, W, g->d_row_ptr, g->d_col, n, np, buf[0]);
        // binary exponentiation: b holds M1^(2^j), r the product of the powers taken so far
        int b = 0, r = -1;
        const int32_t nt = np / kTile;
        const dim3 grid(nt * (nt + 1) / 2, cnt);
        for (int32_t h = hops;;) {
            if (h & 1) {
                if (r < 0) {
                    r = b;
                } else {
                    const int f = 3 - r - b;  // the free buffer
                    hipLaunchKernelGGL(k_six_gemm, grid, dim3(256), 0, s, buf[r], buf[b], buf[f], np);
                    r = f;
                }
            }
            h >>= 1;
            if (h == 0) break;
            int f = 0;
            while (f == r || f == b) ++f;
            hipLaunchKernelGGL(k_six_gemm, grid, dim3(256), 0, s, buf[b], buf[b], buf[f], np);
            b = f;
        }
        GAPA_HIP(hipGetLastError());
        int rc = launch_fill_u32(tot, 0u, 2 * (int64_t)cnt, s);
        if (rc == GAPA_OK) rc = launch_fill_u32(reinterpret_cast<uint32_t *>(mcn + z0), 0u, cnt, s);
        if (rc != GAPA_OK) return rc;
        hipLaunchKernelGGL(k_six_rows, dim3((n + kRowsPerBlock - 1) / kRowsPerBlock, cnt), dim3(256), 0, s, buf[r],
                           mk, W, n, np, tot, mcn + z0);
        hipLaunchKernelGGL(k_six_final, dim3((cnt + 255) / 256), dim3(256), 0, s, tot, cnt, n, pc + z0);
        GAPA_HIP(hipGetLastError());
    }
    return GAPA_OK;
}

}  // namespace gapa
