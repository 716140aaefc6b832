// pc_blocks.hip -- the counting kernel of pruned launches: pairs of 512-point
// tiles as 16 x 16 blocks of 32 x 32 points, squared chords from the matrix cores
// (mixed mode) or in binary64 (F64, at the end of this comment).
//
// A survivor of the prune pass is a pair of tiles (I, J) whose chord interval
// meets some edges.  One workgroup of four waves takes it:
//   * classification: one lane per block bounds the block's chords from the
//     bounding spheres of its two 32-point groups; a block inside one bin is
//     counted whole, the others ("open") get the first edge k0 and the number m
//     of edges inside their interval;
//   * the i-tile sits in LDS in the form the matrix instruction reads, shared
//     by the four waves and kept while the i-tile stays the same; each wave
//     takes four of the J tile's sixteen columns of blocks, one after the
//     other, with the column's 32 j-points in registers;
//   * an open block is four v_mfma_f32_16x16x32_bf16, each giving
//     d = h - c for 256 pairs (c the squared chord, h the threshold of the
//     block's first edge); the sign of d is the count, and d within a bounded
//     width of 0 (see below) sends the pair to binary64.
//
// Chords.  With o_I, o_J the tiles' sphere centres, D = o_I - o_J, and the
// points centred on their own tile (a' = RN32(a - o_I), b' = RN32(b - o_J)),
//   c = |D|^2 + s_a + s_b - 2 a'.b',  s_a = |a'|^2 + 2 D.a',
//                                     s_b = |b'|^2 - 2 D.b'.
// s_a and s_b are formed in binary32 once per point and tile pair.  Every
// binary32 operand is split exactly into three bf16 limbs (truncation leaves
// at most 8 bits at each step), and one K = 32 product holds per coordinate
// the eight limb products that reach binary32 accuracy (all but the 3rd x 3rd,
// below 2^-30), and s_a, s_b as limbs against ones; the threshold is the
// accumulator's starting value.
//
// Why the matrix cores, and why 32 x 32.  The vector form of the same chord
// needs four or five instructions per pair before it is binned; the product
// takes 16 cycles of a SIMD per 256 pairs, a quarter of that, and leaves the
// vector unit the binning alone (per two pairs one byte permute that spreads
// the two sign bits, half an add, one three-operand minimum).  Finer blocks
// meet fewer edges: of the 1M workload's pairs 14% are visited at 256 x 64
// points, 10% at 32 x 32, and most of those meet one edge instead of two.  The
// tiles are 512 points because an item's fixed work (its centre and bounds, a
// column's operands, a run's bookkeeping) is shared by all its blocks: at 256
// points it was 70% of the kernel's vector instructions.
//
// What bounds it: vector instructions and matrix products, which a SIMD does
// not overlap: together some 85% of the cycles, the rest waits for LDS and at
// the tile pair's barriers.  A block of one edge takes 34 vector instructions
// and four products (about 47 cycles of a CU), of two 57, through the table 115 or 135,
// by differences 97 per half; the item's and the columns' shares are 15 to 27 per
// block.  Counting kernel, this one against the vector kernel of 256-point tiles
// on the same ordering: 21.9 / 42.7 ms on the 1M workload, 103 / 212 ms for 1M x 1M
// points in 254 bins, 13.0 / 21.0 ms for 64 mocks x 300,000 randoms, 1.51 / 2.2 ms
// for 300,000 x 400,000 resident points in 24 even bins, 0.10 / 0.29 ms for 10,000
// + 10,000 points, 0.024 / 0.134 ms for 1003 points.
//
// Error bound (u = 2^-24, v = 2^-53, R = r_I + r_J the tiles' radii, D = |D|).
// For an edge inside the tile pair's interval |h - D^2| <= R (2D + R) to
// rounding.  Against the exact chord of the binary64 unit vectors:
//   * rounding a', b':            <= 2 (D + R) u R + (u R)^2
//   * D rounded to binary32:      <= 2 u D R
//   * s_a, s_b (|.|^2, three fused multiply-adds, three roundings in |.|^2):
//                                 <= 7 u (R^2 + 2 D R)
//   * the threshold rounded:      <= u R (2D + R)
//   * the product, M = sum of |terms| <= 4 D R + 2.5 R^2 (see below):
//                                 <= 13 u M
//   * a higher edge of the block, d_t = RN(d + RN(h_t - h)): <= u (8 D R + 2 R^2)
// in all below u (80 D R + 45 R^2).  E = u R (88 D + 50 R) + 2^-48 (D + R)^2 +
// 2^-110 lies 10% above that; its second term covers the binary64 steps and the
// binary64 chord itself (5 v c), the third underflow.  With h = e + E: d < 0
// proves the binary64 chord at or above e, d > W = 2E proves it below, and 0 <=
// d <= W is recomputed in binary64 in the reference's order.  Measured against
// binary64 over tile pairs of catalogues of 1003 to 1M points: at most 0.05 E;
// 2.7 u (D + R)^2 at most and 0.05 to 0.17 in the mean square, where the vector
// kernel's forms have 28 and 0.5 to 2.2 (differences), 2.8 and 0.23 to 0.76
// (tile-centred Gram).
//
// The product's term.  How v_mfma_f32_16x16x32_bf16 rounds is not documented; it
// was found by probes, and this model gives its results bit for bit (2 10^6 sums of
// operands like these and of random ones; a test holds the model to the hardware).
// The four groups of eight slots are added to the accumulator one after the other.
// In a group with 2^p the largest product of its operands' powers of two, each
// product is cut toward zero to a multiple of 2^(p - 24), which only products 2^11
// below 2^p can lose by; with 2^q the larger of 2^p and the accumulator's power, the
// accumulator is cut downward to a multiple of 2^(q - 24), the products' sum to one
// of 2^(q - 31), and their sum rounded to nearest.  Here a coordinate's group has
// one large product, at most p_k = |2 a'_k b'_k|, and seven that lose at most u p_k
// each; the last group six products, of which five lose at most u S, S = max(|s_a|,
// |s_b|) <= 2 D R + R^2; the accumulator loses u p_k and u S; and the four roundings
// u each of at most H + P, three times, and H + P + |s_a| + |s_b|, where H <= 2 D R + R^2
// is the threshold, P = sum of p_k <= R^2 / 2 and |s_a| + |s_b| <= 2 D R + R^2.  In all
// 22 D R + 17 R^2 in units of u, the cut sums and the dropped 3rd x 3rd products less
// than 0.2 more: below 13 M = 52 D R + 32.5 R^2.  (Largest error seen: 3.9 M.)  With
// |D|^2 as the accumulator's start the roundings add four times |D|^2, of 13.
//
// Blocks of three edges and more (near tiles, sparse catalogues) look each chord
// up in a table instead.  There the product starts at RN(D^2) and takes the
// j-points negated, so that it is the chord itself: |D|^2 joins M (13 u D^2) and is
// rounded (u D^2), the table's edge is (2 u (D + R)^2), so the chord is within E_t =
// E + 14 u D^2 + 2 u (D + R)^2 (measured: at most 0.18 E_t, 3.7 u (D + R)^2 and 0.24 to
// 0.76 in the mean square, where the cell table of the vector kernel has the
// differences' 28 and 0.5 to 2.2).  Its cell holds at most one edge, and a chord within
// E_t of that edge goes to binary64.  The table needs E_t below an eighth of a cell (see
// build_lutb); blocks that reach below that (near ones: E grows with the tiles'
// size, not with the chord) form their chords from differences, (D - b') + a'
// per coordinate, whose error follows the chord: the difference vector is off
// by at most u (2D + 2R + sqrt(c)) <= 3 u (D + R), three roundings square it, and
// the table's edge and the final difference add two: below A sqrt(c) + B with
// A = 16 u (D + R), B = 64 u^2 (D + R)^2.
//
// F64 (PC_FP64_PLAIN): every pair of an open block gets its squared chord in
// binary64, in the reference's order of operations and without fused
// multiply-adds, from the unit vectors themselves; blocks, classification and
// work units are the same.  A lane holds 4 x 4 pairs, the i-tile lies in LDS as
// three arrays.  Few edges are compared with the chord and the lanes counted by
// scalar instructions, which run beside the vector ones; more edges go through
// the chord table with the chord rounded to binary32, and where that is within
// rounding of the cell's edge the chord itself decides.  Bound by the eight
// binary64 operations of a chord (11.3 instructions a pair, 14 cycles of a CU
// per wave of pairs, of 17 in the vector kernel, at 75% of its pairs): 2.32 ms
// for 100,000 + 100,000 points in 30 bins, the vector kernel of 256-point tiles
// 3.26.
#include <algorithm>
#include <array>
#include <type_traits>

#include "pc_internal.hpp"

namespace pc {

namespace blk {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kT = kBlockTile;              // points per tile
constexpr int kWaves = 4;                   // waves per workgroup
constexpr int kThreads = kWave * kWaves;
constexpr int kG = kGroup;                  // points per block side
constexpr int kN = kT / kG;                 // blocks per tile side
constexpr int kPer = kT / kThreads;         // i-points per thread
static_assert(kN * kN == kThreads, "one lane classifies one block");
constexpr uint32_t kColMask = (1u << kN) - 1u;
constexpr float kNever = 1e30f;             // added to d of a pair that counts nowhere
constexpr uint32_t kDiagBlock = 1u << 31;   // block descriptor: on the diagonal, only i < j counts
constexpr uint32_t kTableBlock = 1u << 30;  // block descriptor: chords go through the table
constexpr uint32_t kInRange = 1u << 28;     // with kTableBlock: every chord falls into the table's cells
constexpr uint32_t kNearBlock = 1u << 29;   // with kTableBlock: chords from differences
// Edges from which a whole block goes through the table: one edge costs a block
// the same half add and minimum per pair, the table nine instructions and two
// LDS accesses per pair whatever their number.  Counting kernel with the line at
// 3 / 4 / 5 / 6: 1.63 / 1.68 / 1.67 / 1.77 ms for 300,000 x 400,000 points, 13.8 / 14.0 /
// 14.6 / 15.1 ms for 64 mocks, 22.5 / 22.6 / 22.7 / 23.0 ms on the 1M workload.  With
// eight lane columns the line lies at 4: 18.9 / 17.2 / 17.7 ms at 3 / 4 / 5 for 300,000 x
// 300,000 points in 254 bins.
constexpr uint32_t table_edges(int32_t cols) { return cols >= 16 ? 3u : 4u; }
// The same with the table in global memory, by the histogram's lane columns: the
// fewer there are, the more of 64 lanes' adds meet in one word.  Whole calls with the
// line at 4 / 5 / 6 / 8 / 12, ms: eight columns (125 log bins, 300,000 x 300,000 points)
// 9.58 / 9.68 / 9.88 / 10.3 / 10.9; four (150 and 200) 11.8 / 11.3 / 11.4 / 11.9 / 12.6 and
// 15.3 / 14.2 / 14.3 / 14.9 / 16.1; two (254) 28.6 / 21.0 / 18.7 / 18.4 / 19.8, and 1M x 1M
// points 115.2 / - / 103.0 / 102.8 / 105; one (300 bins, 100,000 x 100,000 points)
// - / 10.0 / - / 4.70 / 4.15, in 500 bins - / - / - / 7.69 / 5.70 (without a table 19.2).
constexpr uint32_t table_edges_global(int32_t cols) { return cols >= 4 ? 5u : cols == 2 ? 8u : 12u; }
// The same in binary64, where an edge costs a pair a comparison: counting kernel with
// the line at 3 / 4 / 5 / 6 / 8, ms: 1M x 1M points in 40 log bins (sixteen columns)
// 32.6 / 32.7 / 32.9 / 33.0 / 33.1, 100,000 x 100,000 in 30 1.12 / 1.15 / 1.16 / 1.18 / 1.21,
// 200,000 x 200,000 in 40 even bins to half the field's width 9.53 / 9.47 / 10.5 / 10.7 /
// 10.7; 1M x 1M in 254 log bins (eight columns) 118 / 120 / 124 / 128 / 134.  Whole calls
// of 50,000 x 50,000 at 4 / 5 / 8 / 12 in 400 bins (four) 1.57 / 1.46 / 1.32 / 1.54, in 500
// (two) 2.01 / 1.93 / 1.83 / 1.59.
constexpr uint32_t table_edges64(int32_t cols) { return cols >= 8 ? 3u : cols == 4 ? 8u : 12u; }
constexpr uint32_t kOnes = 0x3F803F80u;     // two bf16 ones

struct BParams {
    const SegDesc *segs;
    const TableDesc *tabs;
    const uint64_t *items;                  // survivors: seg | K0 << 32 | M << 43
    const uint64_t *tiles;                  // beside them: t | u << 32
    const unsigned long long *n_items;
    unsigned long long *queue;              // 8 zeroed counters kQueueStride words apart
    unsigned long long *rechecked;
    unsigned long long *stats;              // the statistics stripes (see k_prune)
    unsigned long long *counts;             // all jobs' counters, count_words of them, and
    const unsigned long long *copies;       // kPruneStripes copies with the prune pass's whole tile pairs
    int64_t count_words;
    uint32_t flush_every;                   // items between flushes, so that no 32-bit word can wrap
    int32_t max_edges, max_cells;           // of the launch's tables: LDS layout (max_cells 0: no table)
    int32_t cols;                           // lane columns of the histogram (power of two)
    uint32_t table_edges;                   // edges from which a block goes through the table
    int32_t chunk;                          // work units taken from the queue at a time, at most
};

// Loads through the constant address space: wave-uniform addresses, scalar loads.
template <typename T>
__device__ __forceinline__ T ld_uniform(const T *p) {
    static_assert(sizeof(T) % 4 == 0, "size");
    using CU = const __attribute__((address_space(4))) uint32_t;
    CU *q = (CU *)(p);
    T out;
    uint32_t *o = reinterpret_cast<uint32_t *>(&out);
#pragma unroll
    for (int i = 0; i < static_cast<int>(sizeof(T) / 4); ++i) o[i] = q[i];
    return out;
}

__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t uni64(uint64_t x) {
    return static_cast<uint64_t>(uni(static_cast<uint32_t>(x))) | (static_cast<uint64_t>(uni(static_cast<uint32_t>(x >> 32))) << 32);
}
__device__ __forceinline__ float uni_f(float x) { return __uint_as_float(uni(__float_as_uint(x))); }
__device__ __forceinline__ float pow2(uint32_t k) { return __uint_as_float((127u + k) << 23); }
__device__ __forceinline__ uint32_t ballot32(bool b) { return static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(b)); }

// The three bf16 limbs of x, exact, each in the upper half of a word.
struct Limbs {
    uint32_t a, b, c;
};
__device__ __forceinline__ Limbs split(float x) {
    Limbs l;
    l.a = __float_as_uint(x) & 0xFFFF0000u;
    const float r = x - __uint_as_float(l.a);
    l.b = __float_as_uint(r) & 0xFFFF0000u;
    l.c = __float_as_uint(r - __uint_as_float(l.b));
    return l;
}
// upper halves of (lo, hi) as one word
__device__ __forceinline__ uint32_t pack(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }

// A point's eight K slots of one lane group (16 bytes): a coordinate as the i
// side (1,1,2,2,1,3,2,3) and as the j side (1,2,1,2,3,1,3,2); the last group
// carries s_a and s_b against ones.
__device__ __forceinline__ u32x4 slots_i(float x) {
    const Limbs l = split(x);
    return u32x4{pack(l.a, l.a), pack(l.b, l.b), pack(l.a, l.c), pack(l.b, l.c)};
}
__device__ __forceinline__ u32x4 slots_si(float x) {
    const Limbs l = split(x);
    return u32x4{pack(l.a, l.b), pack(l.c, kOnes), kOnes, 0u};
}
// the j side of both kinds (last = the lane is of the last group)
__device__ __forceinline__ u32x4 slots_j(float x, bool last) {
    const Limbs l = split(x);
    const uint32_t ab = pack(l.a, l.b);
    return u32x4{last ? kOnes : ab, last ? pack(kOnes, l.a) : ab, last ? pack(l.b, l.c) : pack(l.c, l.a),
                 last ? 0u : pack(l.c, l.b)};
}

__device__ __forceinline__ f32x4 product(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}

// Two values of d against one edge: the permute turns their sign bits into two
// bytes (0xFF when negative), the lower two of the word for the run's first
// edge (kSelLo) or the upper two for the next (kSelHi), and subtracting it
// counts them: with n_k the count in byte k, the word is n_0 + 2^8 (n_1 - n_0) +
// 2^16 (n_2 - n_1) + 2^24 (n_3 - n_2).  A byte takes 255, a block adds at most 8
// to one: kRunBlocks blocks in a run.  mn keeps the smallest d (as
// unsigned bits: negative ones are large).
constexpr uint32_t kSelLo = 0x0C0C0B09u, kSelHi = 0x0B090C0Cu;
constexpr int kRunBlocks = 31;
template <uint32_t SEL>
__device__ __forceinline__ void tally(float d1, float d2, uint32_t &n, uint32_t &mn) {
    const uint32_t b1 = __float_as_uint(d1), b2 = __float_as_uint(d2);
    n -= __builtin_amdgcn_perm(b2, b1, SEL);
    mn = min(min(mn, b1), b2);
}
// the counts of the first and the next edge
__device__ __forceinline__ void counts_of(uint32_t n, uint32_t &first, uint32_t &next) {
    uint32_t w = n + (n << 8);  // n 0x01010101 = n_0 + 2^8 n_1 + 2^16 n_2 + 2^24 n_3,
    w += w << 16;               // without the quarter-rate multiply
    first = (w & 0xFFu) + ((w >> 8) & 0xFFu);
    next = ((w >> 16) & 0xFFu) + (w >> 24);
}

// d of the 16 pairs a lane holds of a block: D[2 ri + cj] for rows 16 ri +
// 4 (lane / 16) + v and column 16 cj + lane % 16.
struct BlockD {
    f32x4 d[4];
};

// LDS histogram: T[row] pairs put into a row (whole blocks into their bin, open
// ones into the row below their first edge, chords of the table), a word per
// lane column; N[edge] pairs above an edge.  The count of row r is T[r] +
// N[r - 1] - N[r].
struct Hist {
    uint32_t *T, *N;
    int32_t n_edges, cols;
};

__device__ __forceinline__ void add_row(const Hist &h, uint32_t row, uint32_t n) {
    atomicAdd(h.T + row * static_cast<uint32_t>(h.cols) + (threadIdx.x & static_cast<uint32_t>(h.cols - 1)), n);
}

// Sum of x over the wave (every lane active), uniform.
__device__ __forceinline__ uint32_t wave_total(uint32_t x) {
#define PC_DPP_ADD(ctrl, rows) x += __builtin_amdgcn_update_dpp(0, x, ctrl, rows, 0xF, false)
    PC_DPP_ADD(0x111, 0xF);  // row_shr 1, 2, 4, 8
    PC_DPP_ADD(0x112, 0xF);
    PC_DPP_ADD(0x114, 0xF);
    PC_DPP_ADD(0x118, 0xF);
    PC_DPP_ADD(0x142, 0xA);  // row_bcast 15, 31
    PC_DPP_ADD(0x143, 0xC);
#undef PC_DPP_ADD
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), kWave - 1));
}

__device__ void clear_hist(const Hist &h) {
    // N follows T
    for (int r = static_cast<int>(threadIdx.x); r < (h.n_edges + 1) * h.cols + h.n_edges; r += kThreads) h.T[r] = 0u;
}

__device__ void flush_hist(const Hist &h, unsigned long long *counts) {
    __syncthreads();
    for (int r = static_cast<int>(threadIdx.x); r <= h.n_edges; r += kThreads) {
        uint32_t v = 0;
        for (int c = 0; c < h.cols; ++c) v += h.T[r * h.cols + ((c + r) & (h.cols - 1))];
        if (r > 0) v += h.N[r - 1];
        if (r < h.n_edges) v -= h.N[r];
        if (v) atomicAdd(counts + r, static_cast<unsigned long long>(v));
    }
    __syncthreads();
    clear_hist(h);
}

// Pairs too near an edge wait in LDS for their binary64 chord: the loads of a
// pair's two points take some two thousand cycles, and a wave that fetched them
// at once would hold up its workgroup in most items.  One pair per thread is
// then done at a time, in the reference's order of operations.
constexpr uint32_t kQueued = 64;
struct Pending {
    const double4 *a[kQueued], *b[kQueued];
    uint32_t edge[kQueued];     // the edge, or kTableRow | the row the pair was counted in
    uint32_t n;                 // may pass kQueued: the pairs beyond were done at once
};
constexpr uint32_t kTableRow = 1u << 31;
// Table look-ups of a lane in flight: one at a time each waits for its LDS read
// (with 4 / 8 / 16: 1.83 / 1.78 / 1.70 ms for 300,000 x 400,000 points, 16.0 / 15.6 /
// 15.6 ms for 64 mocks; 16 leaves no registers for the rest).
constexpr int kLook = 8;

__device__ __forceinline__ void recheck(const Hist &h, const double4 *pa, const double4 *pb, uint32_t edge,
                                        const double *e64) {
#pragma clang fp contract(off)
    const double4 a = *pa, b = *pb;
    const double dx = a.x - b.x, dy = a.y - b.y, dz = a.z - b.z;
    double c = dx * dx;
    c = c + dy * dy;
    c = c + dz * dz;
    if (edge & kTableRow) {
        int lo = 0, hi = h.n_edges;  // number of edges at or below c
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (e64[mid] <= c) lo = mid + 1;
            else hi = mid;
        }
        const uint32_t prov = edge & ~kTableRow;
        if (static_cast<uint32_t>(lo) != prov) {
            add_row(h, static_cast<uint32_t>(lo), 1u);
            add_row(h, prov, 0xFFFFFFFFu);
        }
    } else {
        if (c >= e64[edge]) atomicAdd(h.N + edge, 1u);
    }
}

__device__ __forceinline__ void send(const Hist &h, Pending &pend, const double4 *a, const double4 *b, uint32_t edge,
                                     const double *e64) {
    const uint32_t at = atomicAdd(&pend.n, 1u);
    if (at < kQueued) {
        pend.a[at] = a;
        pend.b[at] = b;
        pend.edge[at] = edge;
    } else {
        recheck(h, a, b, edge, e64);
    }
}

// One block against an edge del above the product's.
template <uint32_t SEL, bool ADD>
__device__ __forceinline__ void block_tally(const BlockD &D, float del, uint32_t &n, uint32_t &mn) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 4; v += 2) {
            if (ADD) tally<SEL>(D.d[q][v] + del, D.d[q][v + 1] + del, n, mn);
            else tally<SEL>(D.d[q][v], D.d[q][v + 1], n, mn);
        }
}

// The products of block row bi against the column's j-points.
__device__ __forceinline__ void block_products(const u32x4 (*As)[kWave], int bi, const u32x4 (&B)[2], float H, BlockD &D) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const u32x4 a0 = As[2 * bi][lane], a1 = As[2 * bi + 1][lane];
    const f32x4 C = {H, H, H, H};
    D.d[0] = product(a0, B[0], C);
    D.d[1] = product(a0, B[1], C);
    D.d[2] = product(a1, B[0], C);
    D.d[3] = product(a1, B[1], C);
}

// The edge set's chord table (8 bytes a cell: the edge, the row below it): in
// LDS, or with GT in global memory, where the lookups of a block, a few adjacent
// cells, come from the nearest cache.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
using LdsU = __attribute__((address_space(3))) uint32_t;
using LdsCell = const __attribute__((address_space(3))) u32x2;
__device__ __forceinline__ uint32_t lds_addr(const void *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void *)(p)));
}
struct ChordTable {
    const unsigned char *cells; // GT: cell 0
    uint32_t base;              // otherwise its LDS address, less 8 key0
    uint32_t shift, key0;
    uint32_t row_shift;         // a row's bytes in the histogram, as a power of two
    float lo, hi;               // cells' range
};
template <bool GT, bool CLAMP>
__device__ __forceinline__ u32x2 cell_of(const ChordTable &t, float c) {
    const uint32_t key = __float_as_uint(CLAMP ? __builtin_amdgcn_fmed3f(c, t.lo, t.hi) : c);
    if (GT) return *reinterpret_cast<const u32x2 *>(t.cells + static_cast<uint32_t>((key >> t.shift) - t.key0) * 8u);
    return *(LdsCell *)(uintptr_t)(((key >> t.shift) << 3) + t.base);
}
// the byte offset of the row of a chord that differs from its cell's edge by x
__device__ __forceinline__ uint32_t row_offset(const ChordTable &t, u32x2 e, float x) {
    return ((__float_as_uint(x) >> 31) + e.y) << t.row_shift;
}
__device__ __forceinline__ void add_offset(uint32_t lds, uint32_t n) {
    __hip_atomic_fetch_add((LdsU *)(uintptr_t)lds, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <bool GT, bool F64>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) k_count_blocks(BParams p) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ u32x4 As[F64 ? 1 : kT / 16][kWave];  // 16 rows x 4 lane groups per set
    __shared__ double Ai[3][F64 ? kT : 1];    // F64: the i-tile's coordinates
    __shared__ uint32_t blk[kThreads];        // open blocks: k0 - K0 | m << 16 | flags; 0: nothing to do
    __shared__ Pending pend;
    __shared__ uint64_t sh_next[2];
    __shared__ unsigned long long sh_stat[7]; // pairs by edges (1, 2, 3, more), of near blocks; items with open, with few-edge blocks
    // a bit per item, of 32 items and the 32 before: it has open blocks, blocks of a few edges
    __shared__ uint32_t sh_open[2], sh_few[2];
    const int tid0 = static_cast<int>(threadIdx.x);
    const int wave = static_cast<int>(uni(threadIdx.x / kWave));

    Hist h;
    double *const e_lds = reinterpret_cast<double *>(lds);
    ChordTable tbl;
    uint2 *const cells = reinterpret_cast<uint2 *>(lds + 8 * p.max_edges);
    h.T = reinterpret_cast<uint32_t *>(lds + 8 * (p.max_edges + p.max_cells));
    h.cols = p.cols;
    h.n_edges = 0;
    tbl.cells = nullptr;
    tbl.base = tbl.shift = tbl.key0 = 0;
    tbl.row_shift = 2u + static_cast<uint32_t>(__builtin_ctz(static_cast<uint32_t>(p.cols)));
    tbl.lo = tbl.hi = 0.0f;
    int cur_tab = -1, cur_job = -1;
    bool has_table = false;
    unsigned long long *cur_counts = nullptr;
    uint32_t since_flush = 0, cur_seg = 0xFFFFFFFFu, cur_t = 0;
    uint32_t seen = 0;                        // pairs this lane sent to the re-check
    uint32_t xs = 0;                          // thread 0's place in the queue's slices
    uint64_t wi = 0, end = 0;
    // A unit of work is a survivor, or where there are few of them a quarter (a
    // column of blocks per wave) or a sixteenth (four blocks per wave) of one: a
    // whole survivor is some 40 blocks per wave, and a launch needs several
    // units per workgroup to end evenly.  Cut and whole: 28 / 73 us at 3
    // survivors (1003 points), 120 / 141 us at 820 (10,000 + 10,000 points) with
    // 1024 workgroups; from 4 survivors a workgroup on a whole one pays its
    // fixed work once (no difference either way at 38,861).
    const uint64_t total = ld_uniform(p.n_items);
    const uint32_t part_bits = total >= 4ull * gridDim.x ? 0u : total * 2u >= gridDim.x ? 2u : 4u;
    if (tid0 < 7) sh_stat[tid0] = 0ull;
    for (int64_t w = static_cast<int64_t>(blockIdx.x) * kThreads + tid0; w < p.count_words;
         w += static_cast<int64_t>(gridDim.x) * kThreads) {
        unsigned long long v = 0;
#pragma unroll
        for (int s = 0; s < kPruneStripes; ++s) v += p.copies[s * p.count_words + w];
        if (v) atomicAdd(p.counts + w, v);
    }
    if (tid0 == 0) pend.n = sh_open[0] = sh_open[1] = sh_few[0] = sh_few[1] = 0u;
    auto add_items = [&](uint32_t r) {        // thread 0
        sh_stat[5] += __popc(sh_open[r]);
        sh_stat[6] += __popc(sh_few[r]);
        sh_open[r] = sh_few[r] = 0u;
    };

    for (;; ++wi) {
        // opaque per item: addresses made from it are recomputed rather than
        // kept (and spilled) across the loop
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        const int lane = tid & (kWave - 1);
        const int grp = lane >> 4;            // lane group: x, y, z, s
        const bool last = grp == 3;
        if (wi >= end) {
            // Work queue: the units in eight slices, one per XCD; a workgroup
            // takes a chunk at a time from its own slice, then from the
            // others (consecutive survivors share the i-tile).
            __syncthreads();
            if (tid == 0) {
                const uint64_t units = total << part_bits;
                const uint64_t chunk = max<uint64_t>(1, min<uint64_t>(p.chunk, units / (8ull * gridDim.x)));
                uint64_t a = 0, b = 0;
                for (; xs < 8u; ++xs) {
                    const uint32_t x = (blockIdx.x + xs) & 7u;
                    const uint64_t s0 = units * x / 8u, s1 = units * (x + 1u) / 8u;
                    const uint64_t c = atomicAdd(p.queue + x * kQueueStride, static_cast<unsigned long long>(chunk));
                    if (s0 + c < s1) {
                        a = s0 + c;
                        b = min<uint64_t>(s1, a + chunk);
                        break;
                    }
                }
                sh_next[0] = a;
                sh_next[1] = b;
            }
            __syncthreads();
            wi = uni64(sh_next[0]);
            end = uni64(sh_next[1]);
            if (wi >= end) break;
        }
        // the unit's columns of blocks, and the wave's rows of them
        const uint32_t part = static_cast<uint32_t>(wi) & ((1u << part_bits) - 1u);
        const int first_col = part_bits == 0 ? wave : part_bits == 2 ? static_cast<int>(part) * kWaves + wave : static_cast<int>(part);
        const uint32_t rows = part_bits == 4 ? 0xFu << (4 * wave) : kColMask;
        // the wave that classifies the unit's blocks (all do their own where a unit is a whole survivor; in a
        // survivor's first unit the others look at the rest, for its statistics)
        const bool classifies = part_bits == 0 || wave == static_cast<int>(part_bits == 2 ? part : part >> 2);
        const uint64_t w0 = ld_uniform(p.items + (wi >> part_bits)), w1 = ld_uniform(p.tiles + (wi >> part_bits));
        const uint32_t seg = static_cast<uint32_t>(w0);
        const uint32_t K0 = static_cast<uint32_t>(w0 >> 32) & 2047u, M = static_cast<uint32_t>(w0 >> 43) & 2047u;
        const uint32_t t = static_cast<uint32_t>(w1), u = static_cast<uint32_t>(w1 >> 32);
        const SegDesc *sp = p.segs + seg;     // its fields come through scalar loads where they are used
        const bool new_i = seg != cur_seg || t != cur_t;
        cur_seg = seg;
        cur_t = t;
        const int64_t ibeg = static_cast<int64_t>(t) * kT, jbeg = static_cast<int64_t>(u) * kT;
        const int32_t i_lim = static_cast<int32_t>(min<int64_t>(kT, ld_uniform(&sp->ni) - ibeg));
        const int32_t j_lim = static_cast<int32_t>(min<int64_t>(kT, ld_uniform(&sp->nj) - jbeg));
        const bool diag = ld_uniform(&sp->tri) != 0 && t == u;
        // what the item reads: its i-points (kept while the i-tile stays), the
        // wave's first column of j-points, the bounds
        const float4 *jg = ld_uniform(&sp->jg) + jbeg;
        float4 gi[kPer], gj[2];
        double4 di[kPer];
        if constexpr (F64) {
#pragma unroll
            for (int r = 0; r < kPer; ++r) di[r] = (ld_uniform(&sp->i64) + ibeg)[min(r * kThreads + tid, i_lim - 1)];
        } else {
#pragma unroll
            for (int r = 0; r < kPer; ++r) gi[r] = (ld_uniform(&sp->ig) + ibeg)[min(r * kThreads + tid, i_lim - 1)];
#pragma unroll
            for (int c = 0; c < 2; ++c) gj[c] = jg[min(first_col * kG + 16 * c + (lane & 15), j_lim - 1)];
        }
        const int cbi = lane & (kN - 1), cbj = wave * (kWave / kN) + lane / kN;  // the block this lane classifies
        const float4 si = (ld_uniform(&sp->ib32) + static_cast<int64_t>(t) * kN)[cbi];
        const float4 sj = (ld_uniform(&sp->jb32) + static_cast<int64_t>(u) * kN)[cbj];
        const double4 oi = ld_uniform(ld_uniform(&sp->ib) + t), oj = ld_uniform(ld_uniform(&sp->jb) + u);
        const double Dx = oi.x - oj.x, Dy = oi.y - oj.y, Dz = oi.z - oj.z;
        const double D2 = Dx * Dx + Dy * Dy + Dz * Dz;
        // E in binary32, raised by 2^-16 for the roundings
        const float R = uni_f(static_cast<float>(oi.w + oj.w) * (1.0f + 0x1p-20f));
        const float Dl = uni_f(__builtin_amdgcn_sqrtf(static_cast<float>(D2)) * (1.0f + 0x1p-20f));
        const float E = (R * (88.0f * Dl + 50.0f * R) * 0x1p-24f + (Dl + R) * (Dl + R) * 0x1p-48f + 0x1p-110f) * (1.0f + 0x1p-16f);
        const double h_off = static_cast<double>(E) - D2;  // threshold of edge k: RN32(e64[k] + h_off)
        const float fx = uni_f(static_cast<float>(Dx)), fy = uni_f(static_cast<float>(Dy)),
                    fz = uni_f(static_cast<float>(Dz));
        const uint32_t wbits = uni(__float_as_uint(2.0f * E * (1.0f + 0x1p-20f)));
        __syncthreads();  // every wave is done with the last item's LDS

        const int tab = ld_uniform(&sp->tab), job = ld_uniform(&sp->job);
        const bool switched = tab != cur_tab || job != cur_job || since_flush >= p.flush_every;
        const uint32_t waiting = min(uni(pend.n), kQueued);
        if (waiting >= kQueued / 2 || (switched && waiting != 0u)) {
            if (tid < static_cast<int>(waiting)) recheck(h, pend.a[tid], pend.b[tid], pend.edge[tid], e_lds);
            __syncthreads();
            if (tid == 0) pend.n = 0u;
        }
        if (switched) {
            if (cur_job >= 0) flush_hist(h, cur_counts);
            if (tid == 0) {
                add_items(0u);
                add_items(1u);
            }
            if (tab != cur_tab) {
                const TableDesc *td = p.tabs + tab;
                h.n_edges = ld_uniform(&td->n_edges);
                h.N = h.T + (h.n_edges + 1) * h.cols;
                const double *e64 = ld_uniform(&td->e64);
                const uint2 *src = reinterpret_cast<const uint2 *>(ld_uniform(&td->lutb));
                const int n_cells = ld_uniform(&td->b_cells);
                has_table = n_cells > 0 && (GT || n_cells <= p.max_cells);
                tbl.shift = ld_uniform(&td->b_shift);
                tbl.key0 = ld_uniform(&td->b_key0);
                tbl.base = lds_addr(cells) - 8u * tbl.key0;
                tbl.lo = __uint_as_float(tbl.key0 << tbl.shift);
                tbl.hi = __uint_as_float(((tbl.key0 + static_cast<uint32_t>(n_cells)) << tbl.shift) - 1u);
                __syncthreads();
                for (int k = tid; k < h.n_edges; k += kThreads) e_lds[k] = e64[k];
                if (GT) tbl.cells = reinterpret_cast<const unsigned char *>(src);
                else if (has_table)
                    for (int k = tid; k < n_cells; k += kThreads) cells[k] = src[k];
                clear_hist(h);
                cur_tab = tab;
            }
            cur_job = job;
            cur_counts = ld_uniform(&sp->counts);
            since_flush = 0;
            __syncthreads();  // the table and the cleared histogram
        }
        ++since_flush;
        const uint32_t ring = (since_flush >> 5) & 1u, item_bit = 1u << (since_flush & 31u);
        if (tid == 0 && (since_flush & 31u) == 0u) add_items(ring ^ 1u);

        // ---- the i-tile, in the product's form
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int i = r * kThreads + tid;
            if constexpr (F64) {
                Ai[0][i] = di[r].x;
                Ai[1][i] = di[r].y;
                Ai[2][i] = di[r].z;
                continue;
            }
            u32x4 *const at = &As[i >> 4][i & 15];
            if (new_i) {
                at[0] = slots_i(gi[r].x);
                at[16] = slots_i(gi[r].y);
                at[32] = slots_i(gi[r].z);
            }
            // g = (-2 a', |a'|^2): the product takes -s_a = D.g - |a'|^2
            const float s = fmaf(fx, gi[r].x, fmaf(fy, gi[r].y, fmaf(fz, gi[r].z, -gi[r].w)));
            at[48] = slots_si(i < i_lim ? s : kNever);
        }
        // ---- classification of the wave's 64 blocks
        const float E_t = (E + 0x1p-23f * (7.0f * Dl * Dl + (Dl + R) * (Dl + R))) * (1.0f + 0x1p-16f);
        // (opaque: with the condition itself the binary64 instance took 3.5% longer, 32.5 / 31.4 ms for
        // 1M x 1M points in 40 bins)
        if (uni(classifies || part == 0)) {
            const float vx = fx + (si.x - sj.x), vy = fy + (si.y - sj.y), vz = fz + (si.z - sj.z);
            const float d = __builtin_amdgcn_sqrtf(fmaf(vx, vx, fmaf(vy, vy, vz * vz)));
            // outward: 12 u (D + R) covers the roundings above
            const float rs = (si.w + sj.w) * (1.0f + 0x1p-20f) + 0x1p-20f * (Dl + R);
            const float lo = fmaxf(d - rs, 0.0f), hi = d + rs;
            const double c_lo = static_cast<double>(lo * lo * (1.0f - 0x1p-18f));
            const double c_hi = static_cast<double>(hi * hi * (1.0f + 0x1p-18f) + 0x1p-120f);
            // edges of [K0, K0 + M) at or below each bound
            uint32_t a = 0, b = 0;
            for (uint32_t step = 1u << (31 - __builtin_clz(M)); step > 0; step >>= 1) {
                if (a + step <= M && e_lds[K0 + a + step - 1] <= c_lo) a += step;
                if (b + step <= M && e_lds[K0 + b + step - 1] <= c_hi) b += step;
            }
            const int32_t ni = min(max(i_lim - cbi * kG, 0), kG), nj = min(max(j_lim - cbj * kG, 0), kG);
            uint32_t np = static_cast<uint32_t>(ni * nj);
            const bool on_diag = diag && cbi == cbj;
            if (diag && cbi >= cbj) np = on_diag ? static_cast<uint32_t>(ni * (ni - 1) / 2) : 0u;
            if (part == 0) {
                const uint32_t m = np ? b - a : 0u;
                const uint64_t any = __builtin_amdgcn_ballot_w64(m != 0u), few = __builtin_amdgcn_ballot_w64(m - 1u < 3u);
                if (lane == 0 && any) atomicOr(sh_open + ring, item_bit);
                if (lane == 0 && few) atomicOr(sh_few + ring, item_bit);
            }
            if (!classifies || (part_bits == 4 && cbj != static_cast<int>(part))) np = 0u;
            const uint32_t m = np ? b - a : 0u;
            const bool near = !F64 && has_table && lo * lo < E_t * pow2(27u - tbl.shift);
            const bool by_table = m && (near || m >= p.table_edges && has_table && (F64 || np == kG * kG && !on_diag));
            const bool in_range = lo * lo * (1.0f - 0x1p-18f) - E_t > tbl.lo && hi * hi * (1.0f + 0x1p-18f) + E_t < tbl.hi;
            blk[cbj * kN + cbi] = m ? a | (m << 16) | (on_diag ? kDiagBlock : 0u) | (by_table ? kTableBlock : 0u) | (near ? kNearBlock : 0u) | (by_table && in_range ? kInRange : 0u) : 0u;
            if (np && !by_table) add_row(h, K0 + a, np);
            const bool full = !diag && i_lim == kT && j_lim == kT && part_bits != 4;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint64_t s = __builtin_amdgcn_ballot_w64(k < 3 ? m == static_cast<uint32_t>(k + 1) : m > 3u);
                uint32_t v = static_cast<uint32_t>(__builtin_popcountll(s)) * (kG * kG);
                if (!full) {
                    v = (s >> lane) & 1u ? np : 0u;
                    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
                }
                if (lane == 0 && v) atomicAdd(sh_stat + k, static_cast<unsigned long long>(v));
            }
            if (near && m) atomicAdd(sh_stat + 4, static_cast<unsigned long long>(np));
        }
        __syncthreads();

        // ---- the wave's columns of blocks; lane k holds the threshold of edge K0 + k
        const float h_lane = static_cast<float>(e_lds[min(K0 + static_cast<uint32_t>(lane), static_cast<uint32_t>(h.n_edges - 1))] + h_off);
        auto threshold = [&](uint32_t k) {
            if (k < kWave) return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(h_lane), static_cast<int>(k)));
            return uni_f(static_cast<float>(e_lds[K0 + k] + h_off));
        };
        const double e_lane = F64 ? e_lds[min(K0 + static_cast<uint32_t>(lane), static_cast<uint32_t>(h.n_edges - 1))] : 0.0;
        auto edge = [&](uint32_t k) {  // F64: edge K0 + k
            const uint64_t bits = __double_as_longlong(e_lane);
            if (k < kWave)
                return __hiloint2double(__builtin_amdgcn_readlane(static_cast<int>(bits >> 32), static_cast<int>(k)),
                                        __builtin_amdgcn_readlane(static_cast<int>(bits), static_cast<int>(k)));
            return __longlong_as_double(static_cast<long long>(uni64(static_cast<uint64_t>(__double_as_longlong(e_lds[K0 + k])))));
        };
        uint32_t cnt = 0u;         // lane k: the wave's pairs above edge K0 + k
        const uint32_t column = lds_addr(h.T) + 4u * static_cast<uint32_t>(tid & (h.cols - 1));
        auto add_above = [&](uint32_t k, uint32_t pairs) {
            if (k < kWave) cnt += lane == static_cast<int>(k) ? pairs : 0u;
            else if (lane == 0)
                atomicAdd(h.N + K0 + k, pairs);
        };
        // the lanes' counts of a pair of edges, K0 + k and the next
        auto add_pair = [&](uint32_t n, uint32_t k) {
            uint32_t c0, c1;
            counts_of(n, c0, c1);
            const uint32_t both = wave_total(c0 | (c1 << 16));  // at most 31 x 1024 each
            add_above(k, both & 0xFFFFu);
            if (both >> 16) add_above(k + 1u, both >> 16);
        };
        uint32_t n = 0u, kb = 0u;  // the run's counts of edges K0 + kb and the next (see tally)
        int run = 0;               // blocks in it
        auto flush_run = [&]() {
            if (run) add_pair(n, kb);
            n = 0u;
            run = 0;
        };
        for (int cb = first_col; cb < kN; cb += part_bits == 0 ? kWaves : kN) {
            const uint32_t desc = blk[cb * kN + (lane & (kN - 1))];
            uint32_t open = ballot32(desc != 0u) & rows;
            if constexpr (F64) {
                // lane (li, lj) holds the block's pairs (li + 8 a, lj + 8 b)
                const int li = lane & 7, lj = lane >> 3;
                double jx[4], jy[4], jz[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const double4 q = (ld_uniform(&sp->j64) + jbeg)[min(cb * kG + lj + 8 * b, j_lim - 1)];
                    jx[b] = q.x;
                    jy[b] = q.y;
                    jz[b] = q.z;
                }
                while (open) {
                    const int bi = __builtin_ctz(open);
                    open &= open - 1u;
                    const uint32_t key = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(desc), bi));
                    const uint32_t k0 = key & 0xFFFFu, m = (key >> 16) & 0xFFFu;
                    double c[16];
                    {
#pragma clang fp contract(off)
#pragma unroll
                        for (int a = 0; a < 4; ++a) {
                            const int i = bi * kG + li + 8 * a;
                            const double x = Ai[0][i], y = Ai[1][i], z = Ai[2][i];
#pragma unroll
                            for (int b = 0; b < 4; ++b) {
                                const double dx = x - jx[b], dy = y - jy[b], dz = z - jz[b];
                                double v = dx * dx;
                                v = v + dy * dy;
                                c[4 * a + b] = v + dz * dz;
                            }
                        }
                    }
                    uint32_t none = 0;  // the lane's pairs that are none: below every edge
                    if ((key & kDiagBlock) || (bi + 1) * kG > i_lim || (cb + 1) * kG > j_lim) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int i = bi * kG + li + 8 * (v >> 2), j = cb * kG + lj + 8 * (v & 3);
                            if (i >= i_lim || j >= j_lim || ((key & kDiagBlock) && i >= j)) {
                                c[v] = -1.0;
                                ++none;
                            }
                        }
                    }
                    if (key & kTableBlock) {
#pragma unroll
                        for (int q = 0; q < 16; q += kLook) {
                            u32x2 e[kLook];
                            float x[kLook];
                            uint32_t at[kLook];
                            float least = INFINITY;
#pragma unroll
                            for (int v = 0; v < kLook; ++v) {
                                x[v] = static_cast<float>(c[q + v]);
                                e[v] = cell_of<GT, true>(tbl, x[v]);
                            }
#pragma unroll
                            for (int v = 0; v < kLook; ++v) {
                                const float d = __uint_as_float(e[v].x) - x[v];
                                at[v] = row_offset(tbl, e[v], d);
                                add_offset(at[v] + column, 1u);
                                // x and the edge are rounded to binary32: within 2^-22 x the chord itself decides
                                least = fminf(least, fmaf(-0x1p-22f, x[v], fabsf(d)));
                            }
                            if (__builtin_amdgcn_ballot_w64(least <= 0x1p-120f) != 0) {
#pragma unroll
                                for (int v = 0; v < kLook; ++v) {
                                    const float d = __uint_as_float(e[v].x) - x[v];
                                    if (fmaf(-0x1p-22f, x[v], fabsf(d)) <= 0x1p-120f) {
                                        const uint32_t row = (e[v].y + (c[q + v] >= e_lds[e[v].y] ? 1u : 0u)) << tbl.row_shift;
                                        if (row != at[v]) {
                                            add_offset(row + column, 1u);
                                            add_offset(at[v] + column, 0xFFFFFFFFu);
                                        }
                                    }
                                }
                            }
                        }
                        if (none) {
                            const u32x2 e = cell_of<GT, true>(tbl, -1.0f);
                            add_offset(row_offset(tbl, e, __uint_as_float(e.x) + 1.0f) + column, 0u - none);
                        }
                        continue;
                    }
                    for (uint32_t r = 0; r < m; ++r) {
                        const double e = edge(k0 + r);
                        uint32_t pairs = 0;
#pragma unroll
                        for (int v = 0; v < 16; ++v) pairs += static_cast<uint32_t>(__builtin_popcountll(__builtin_amdgcn_ballot_w64(c[v] >= e)));
                        add_above(k0 + r, pairs);
                    }
                }
                continue;
            }
            // the column's j-points as the product reads them
            u32x4 B[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float4 g = gj[c];
                const bool ok = cb * kG + 16 * c + (lane & 15) < j_lim;
                // -s_b = -D.g - |b'|^2; the coordinates as -b' = g / 2
                const float s = ok ? -fmaf(fx, g.x, fmaf(fy, g.y, fmaf(fz, g.z, g.w))) : kNever;
                const float x = 0.5f * (grp == 0 ? g.x : grp == 1 ? g.y : g.z);
                B[c] = slots_j(last ? s : x, last);
            }
            if (part_bits == 0 && cb + kWaves < kN) {
#pragma unroll
                for (int c = 0; c < 2; ++c) gj[c] = jg[min((cb + kWaves) * kG + 16 * c + (lane & 15), j_lim - 1)];
            }
            // a block's points in the tiles' ordered copies
            auto point_i = [&](int bi, int s) { return ld_uniform(&sp->i64) + ibeg + (bi * kG + 16 * (s >> 3) + 4 * (lane >> 4) + (s & 3)); };
            auto point_j = [&](int s) { return ld_uniform(&sp->j64) + jbeg + (cb * kG + 16 * ((s >> 2) & 1) + (lane & 15)); };
            auto send_near = [&](const BlockD &D, float del, uint32_t k, int bi) {
                uint32_t hits = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) hits |= __float_as_uint(D.d[q][v] + del) <= wbits ? 1u << (4 * q + v) : 0u;
                seen += __popc(hits);
                for (; hits; hits &= hits - 1u) {
                    const int s = __builtin_ctz(hits);
                    send(h, pend, point_i(bi, s), point_j(s), K0 + k, e_lds);
                }
            };
            // of the lane's pairs s0 .. s0 + kLook - 1, counted at `at`, those of hits
            auto send_rows = [&](uint32_t hits, const auto &at, int bi, int s0) {
                seen += __popc(hits);
                for (; hits; hits &= hits - 1u) {
                    const int v = __builtin_ctz(hits);
                    uint32_t o = at[0];
#pragma unroll
                    for (int w = 1; w < static_cast<int>(sizeof(at) / sizeof(at[0])); ++w) {
                        asm("" : "+v"(o));  // no indexed array: it would be written to scratch on every pass
                        o = v == w ? at[w] : o;
                    }
                    send(h, pend, point_i(bi, s0 + v), point_j(s0 + v), (o >> tbl.row_shift) | kTableRow, e_lds);
                }
            };
            // blocks of one or two edges, those of the same edges together: a
            // run holds edge kb, the next one, or both; its counts stay in n
            // until another kb comes
            uint32_t narrow = open & ~ballot32(desc >= (3u << 16));
            open &= ~narrow;
            while (narrow) {
                const uint32_t key = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(desc), __builtin_ctz(narrow)));
                uint32_t same = ballot32(desc == key) & narrow;
                narrow &= ~same;
                const uint32_t k0 = key & 0xFFFFu;
                const bool two = (key >> 17) != 0u;
                if (run + kN > kRunBlocks || (k0 != kb && (two || k0 != kb + 1u))) {
                    flush_run();
                    kb = k0;
                }
                run += __builtin_popcount(same);
                const float H = threshold(k0);
                if (two) {
                    const float del = uni_f(threshold(k0 + 1u) - H);
                    while (same) {
                        const int bi = __builtin_ctz(same);
                        same &= same - 1u;
                        BlockD D;
                        block_products(As, bi, B, H, D);
                        uint32_t mn = 0xFFFFFFFFu;
                        block_tally<kSelLo, false>(D, 0.0f, n, mn);
                        block_tally<kSelHi, true>(D, del, n, mn);
                        if (__builtin_expect(__builtin_amdgcn_ballot_w64(mn <= wbits) != 0, 0)) {
#pragma unroll 1
                            for (uint32_t r = 0; r < 2; ++r) send_near(D, r ? del : 0.0f, k0 + r, bi);
                        }
                    }
                } else if (k0 == kb) {
                    while (same) {
                        const int bi = __builtin_ctz(same);
                        same &= same - 1u;
                        BlockD D;
                        block_products(As, bi, B, H, D);
                        uint32_t mn = 0xFFFFFFFFu;
                        block_tally<kSelLo, false>(D, 0.0f, n, mn);
                        if (__builtin_expect(__builtin_amdgcn_ballot_w64(mn <= wbits) != 0, 0)) send_near(D, 0.0f, k0, bi);
                    }
                } else {
                    while (same) {
                        const int bi = __builtin_ctz(same);
                        same &= same - 1u;
                        BlockD D;
                        block_products(As, bi, B, H, D);
                        uint32_t mn = 0xFFFFFFFFu;
                        block_tally<kSelHi, false>(D, 0.0f, n, mn);
                        if (__builtin_expect(__builtin_amdgcn_ballot_w64(mn <= wbits) != 0, 0)) send_near(D, 0.0f, k0, bi);
                    }
                }
            }
            // far blocks of the table last
            uint32_t look = ballot32((desc & (kTableBlock | kNearBlock)) == kTableBlock) & open;
            open &= ~look;
            // blocks of more edges, and those on the diagonal
            while (open) {
                const int bi = __builtin_ctz(open);
                open &= open - 1u;
                const uint32_t key = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(desc), bi));
                const uint32_t k0 = key & 0xFFFFu, m = (key >> 16) & 0xFFFu;
                BlockD D;
                if (key & kNearBlock) {
                    const float S = Dl + R, A = 0x1p-20f * S, A2 = 2.0f * A * A, B2 = 0x1p-83f * (S * S) * (S * S);
                    const float q = A * pow2(28u - tbl.shift);
                    const float floor_c = fmaxf(q * q, 0x1p-42f * S * S * pow2(28u - tbl.shift)) * (1.0f + 0x1p-10f);
                    const float A2n = -A2;
                    float px[2], py[2], pz[2];
                    int32_t below[2];  // i-points (of the tile) that the lane's j-points pair with
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int j = cb * kG + 16 * c + (lane & 15);
                        const float4 g = jg[min(j, j_lim - 1)];
                        px[c] = fmaf(0.5f, g.x, fx);
                        py[c] = fmaf(0.5f, g.y, fy);
                        pz[c] = fmaf(0.5f, g.z, fz);
                        below[c] = j >= j_lim ? 0 : (key & kDiagBlock) ? min(j, i_lim) : i_lim;
                    }
#pragma unroll 1
                    for (int r = 0; r < 8; r += 4) {
                        float4 g[4];
                        const int i0 = bi * kG + 4 * r + 4 * grp;
#pragma unroll
                        for (int v = 0; v < 4; ++v) g[v] = (ld_uniform(&sp->ig) + ibeg)[min(i0 + v, i_lim - 1)];
                        float x[8], d[8];
                        u32x2 e[8];
                        uint32_t at[8], hits = 0;
#pragma unroll
                        for (int v = 0; v < 8; ++v) {
                            const float4 &a = g[v & 3];
                            const float dx = fmaf(-0.5f, a.x, px[v >> 2]), dy = fmaf(-0.5f, a.y, py[v >> 2]),
                                        dz = fmaf(-0.5f, a.z, pz[v >> 2]);
                            x[v] = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                            e[v] = cell_of<GT, true>(tbl, x[v]);
                        }
#pragma unroll
                        for (int v = 0; v < 8; ++v) {
                            d[v] = __uint_as_float(e[v].x) - x[v];
                            at[v] = row_offset(tbl, e[v], d[v]);
                            const bool ok = i0 + (v & 3) < below[v >> 2];
                            add_offset(at[v] + column, ok ? 1u : 0u);
                            if (ok && (fmaf(d[v], d[v], A2n * x[v]) <= B2 || x[v] <= floor_c)) hits |= 1u << v;
                        }
                        send_rows(hits, at, bi, 2 * r);
                    }
                    continue;
                }
                const float H0 = threshold(k0);
                block_products(As, bi, B, H0, D);
                if (key & kDiagBlock) {
                    // only i < j counts
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (16 * (q >> 1) + 4 * grp + v >= 16 * (q & 1) + (lane & 15)) D.d[q][v] = kNever;
                }
                // the first two edges, then two at a time
                uint32_t nq = 0u, mn = 0xFFFFFFFFu;
                float d0 = 0.0f, d1 = m > 1 ? uni_f(threshold(k0 + 1u) - H0) : kNever;
                block_tally<kSelLo, false>(D, 0.0f, nq, mn);
                block_tally<kSelHi, true>(D, d1, nq, mn);
                for (uint32_t q = 0;;) {
                    add_pair(nq, k0 + q);
                    if (__builtin_expect(__builtin_amdgcn_ballot_w64(mn <= wbits) != 0, 0)) {
#pragma unroll 1
                        for (uint32_t r = q; r < min(q + 2, m); ++r) send_near(D, r == q ? d0 : d1, k0 + r, bi);
                    }
                    q += 2;
                    if (q >= m) break;
                    nq = 0u;
                    mn = 0xFFFFFFFFu;
                    d0 = uni_f(threshold(k0 + q) - H0);
                    block_tally<kSelLo, true>(D, d0, nq, mn);
                    d1 = kNever;
                    if (q + 1 < m) {
                        d1 = uni_f(threshold(k0 + q + 1) - H0);
                        block_tally<kSelHi, true>(D, d1, nq, mn);
                    }
                }
            }
            // The product of the negated j-points is the chord less |D|^2: a
            // subtraction per pair less than from d, 15.2 / 14.6 ms for 64 mocks,
            // 1.70 / 1.64 ms for 300,000 x 400,000 points.
            if (look) {
#pragma unroll
                for (int c = 0; c < 2; ++c) B[c] ^= 0x80008000u;
                const float D2f = uni_f(static_cast<float>(D2));
                do {
                    const int bi = __builtin_ctz(look);
                    look &= look - 1u;
                    const uint32_t key = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(desc), bi));
                    BlockD D;
                    block_products(As, bi, B, D2f, D);
                    auto look_up = [&](auto clamp) {
#pragma unroll
                        for (int q = 0; q < 16; q += kLook) {
                            float c[kLook];
                            u32x2 e[kLook];
                            uint32_t at[kLook];
                            float least = INFINITY;
#pragma unroll
                            for (int v = 0; v < kLook; ++v) {
                                c[v] = D.d[(q + v) >> 2][v & 3];
                                e[v] = cell_of<GT, decltype(clamp)::value>(tbl, c[v]);
                            }
#pragma unroll
                            for (int v = 0; v < kLook; ++v) {
                                c[v] = __uint_as_float(e[v].x) - c[v];
                                at[v] = row_offset(tbl, e[v], c[v]);
                                add_offset(at[v] + column, 1u);
                                least = fminf(least, fabsf(c[v]));
                            }
                            if (__builtin_expect(__builtin_amdgcn_ballot_w64(least <= E_t) != 0, 0)) {
                                uint32_t hits = 0;
#pragma unroll
                                for (int v = 0; v < kLook; ++v) hits |= fabsf(c[v]) <= E_t ? 1u << v : 0u;
                                send_rows(hits, at, bi, q);
                            }
                        }
                    };
                    // (without the clamp 115 instructions a block instead of 135: 1.61 / 1.66 ms
                    // for 300,000 x 400,000 points, 13.5 / 13.8 ms for 64 mocks)
                    if (key & kInRange) look_up(std::false_type());
                    else look_up(std::true_type());
                } while (look);
            }
        }
        flush_run();
        if (cnt) atomicAdd(h.N + K0 + lane, cnt);
    }
    __syncthreads();
    if (tid0 < static_cast<int>(min(pend.n, kQueued))) recheck(h, pend.a[tid0], pend.b[tid0], pend.edge[tid0], e_lds);
    if (cur_job >= 0) flush_hist(h, cur_counts);
    if (tid0 == 0) {
        add_items(0u);
        add_items(1u);
    }
    for (int o = 32; o > 0; o >>= 1) seen += __shfl_xor(seen, o, kWave);
    if ((tid0 & (kWave - 1)) == 0 && seen) atomicAdd(p.rechecked, static_cast<unsigned long long>(seen));
    __syncthreads();
    const unsigned long long pairs = sh_stat[0] + sh_stat[1] + sh_stat[2] + sh_stat[3];
    if (tid0 == 0 && (pairs | sh_stat[5])) {
        unsigned long long *st = p.stats + (blockIdx.x % kPruneStripes) * kPruneStripeWords;
        atomicAdd(st + 1, pairs);
        if (!F64) atomicAdd(st + 11, pairs - sh_stat[4]);
        atomicAdd(st + 6, sh_stat[3]);
        for (int k = 0; k < 3; ++k) atomicAdd(st + 7 + k, sh_stat[k]);
        atomicAdd(st + 3, sh_stat[6]);
        atomicAdd(st + 4, sh_stat[5]);
        atomicAdd(st + 5, sh_stat[5]);
    }
}

// ------------------------------------------------ the product, for its test

__global__ void __launch_bounds__(kWave) k_products(const uint16_t *__restrict__ a, const uint16_t *__restrict__ b,
                                                    const float *__restrict__ c, float *__restrict__ out) {
    const size_t at = static_cast<size_t>(blockIdx.x) * 32 + 8 * (threadIdx.x >> 4);
    u32x4 x, y;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        x[k] = a[at + 2 * k] | (static_cast<uint32_t>(a[at + 2 * k + 1]) << 16);
        y[k] = b[at + 2 * k] | (static_cast<uint32_t>(b[at + 2 * k + 1]) << 16);
    }
    const float s = c[blockIdx.x];
    const f32x4 d = product(x, y, f32x4{s, s, s, s});
    if (threadIdx.x == 0) out[blockIdx.x] = d[0];
}

hipError_t launch_products(int32_t n, const uint16_t *a, const uint16_t *b, const float *c, float *out) {
    if (n > 0) k_products<<<dim3(static_cast<uint32_t>(n)), dim3(kWave), 0, nullptr>>>(a, b, c, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- bounds

// Per tile of an ordered view, one workgroup: centre (normalised mean) and
// radius, rounded outward; the Gram form of its points centred on it, (-2 b'_x,
// -2 b'_y, -2 b'_z, |b'|^2) with b' = RN32(b - c); and per 32-point group the
// mean relative to the tile centre, rounded to binary32, and the largest
// distance from it.
__global__ void __launch_bounds__(kThreads) k_block_bounds(const ViewDesc *__restrict__ views, int n_views) {
    __shared__ double sh[kWaves][4];
    int lo = 0, hi = n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile0 <= static_cast<int64_t>(blockIdx.x)) lo = mid;
        else hi = mid - 1;
    }
    const ViewDesc &vw = views[lo];
    const double4 *__restrict__ a64s = vw.a64s;
    const int64_t n = vw.n, t = static_cast<int64_t>(blockIdx.x) - vw.tile0, b = t * kT;
    const int tid = static_cast<int>(threadIdx.x), lane = tid & (kWave - 1), wave = tid / kWave;
    double4 p[kPer];
    bool ok[kPer];
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int64_t i = b + r * kThreads + tid;
        ok[r] = i < n;
        p[r] = a64s[ok[r] ? i : b];
        s[0] += ok[r] ? p[r].x : 0.0;
        s[1] += ok[r] ? p[r].y : 0.0;
        s[2] += ok[r] ? p[r].z : 0.0;
    }
    auto all = [&](double v, int k, bool largest) {
        for (int o = 32; o > 0; o >>= 1) {
            const double x = __shfl_xor(v, o, kWave);
            v = largest ? fmax(v, x) : v + x;
        }
        if (lane == 0) sh[wave][k] = v;
    };
    for (int k = 0; k < 3; ++k) all(s[k], k, false);
    __syncthreads();
    for (int k = 0; k < 3; ++k) {
        s[k] = 0.0;
        for (int w = 0; w < kWaves; ++w) s[k] += sh[w][k];
    }
    const double norm = sqrt(s[0] * s[0] + s[1] * s[1] + s[2] * s[2]);
    const double4 first = a64s[b];
    const bool good = norm > 1e-6;
    const double cx = good ? s[0] / norm : first.x, cy = good ? s[1] / norm : first.y, cz = good ? s[2] / norm : first.z;
    double m = 0.0;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const double dx = p[r].x - cx, dy = p[r].y - cy, dz = p[r].z - cz;
        if (ok[r]) m = fmax(m, dx * dx + dy * dy + dz * dz);
    }
    all(m, 3, true);
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) m = fmax(m, sh[w][3]);
    if (tid == 0) vw.bounds[t] = make_double4(cx, cy, cz, sqrt(m) * (1.0 + 0x1p-40) + 0x1p-60);
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const double ex = p[r].x - cx, ey = p[r].y - cy, ez = p[r].z - cz;
        if (ok[r] && vw.g32s) {
            const float x = static_cast<float>(ex), y = static_cast<float>(ey), z = static_cast<float>(ez);
            vw.g32s[b + r * kThreads + tid] = make_float4(-2.0f * x, -2.0f * y, -2.0f * z, fmaf(z, z, fmaf(y, y, x * x)));
        }
        const uint64_t in = __ballot(ok[r]) & (lane < kG ? 0xFFFFFFFFull : ~0xFFFFFFFFull);
        double gx = ok[r] ? ex : 0.0, gy = ok[r] ? ey : 0.0, gz = ok[r] ? ez : 0.0;
        for (int o = kG / 2; o > 0; o >>= 1) {
            gx += __shfl_xor(gx, o, kWave);
            gy += __shfl_xor(gy, o, kWave);
            gz += __shfl_xor(gz, o, kWave);
        }
        const double inv = 1.0 / fmax(static_cast<double>(__popcll(in)), 1.0);
        const float mx = static_cast<float>(gx * inv), my = static_cast<float>(gy * inv), mz = static_cast<float>(gz * inv);
        const double dx = ex - mx, dy = ey - my, dz = ez - mz;
        double g2 = ok[r] ? dx * dx + dy * dy + dz * dz : 0.0;
        for (int o = kG / 2; o > 0; o >>= 1) g2 = fmax(g2, __shfl_xor(g2, o, kWave));
        if ((lane & (kG - 1)) == 0)
            vw.groups[t * kN + (r * kThreads + tid) / kG] =
                make_float4(mx, my, mz, __double2float_ru(sqrt(g2) * (1.0 + 0x1p-40) + 0x1p-60));
    }
}

hipError_t launch_bounds(const ViewDesc *views, int n_views, int64_t tiles, hipStream_t st) {
    if (n_views <= 0 || tiles <= 0) return hipSuccess;
    if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
    k_block_bounds<<<dim3(static_cast<uint32_t>(tiles)), dim3(kThreads), 0, st>>>(views, n_views);
    return hipGetLastError();
}

// ------------------------------------------------------------------ launch

// The launch's LDS layout: the histogram's lane columns (at most `cols`) and
// whether the chord tables come along.
// Four workgroups share a CU where that is possible, else three (40 or 53 KB each;
// the largest edge set, 1024 edges, takes 52 KB, under the 64 KB any kernel may
// have): 500 log bins, which leave no room for a column at four, take 15.6 ms for
// 200,000 x 200,000 points with three workgroups' four columns, 18.8 with one.
// Beside a mixed launch's i-tile the tables come along where they leave eight
// columns: with fewer, the adds that meet in one word cost more than look-ups from
// the cache.  Whole calls of 100,000 x 100,000 points, table in LDS / in global memory:
// 1.45 / 1.48 ms for 80 log bins (eight columns beside the table), 2.37 / 1.68 for 100
// (four), 5.1 / 1.92 for 125 (two), 11.5 / 2.31 for 150 (one).
// Where most blocks go through the table three workgroups with it are better than
// four without.  edges_met tells (see run_batch): four without / three with, ms, at
// 0.16 (254 bins, 1M x 1M) 103 / 110, 0.14 (100, 300,000 x 300,000) 8.13 / 8.65, 0.18 (125)
// 9.68 / 9.96, 0.21 (150) 11.3 / 11.1, 0.28 (200) 14.2 / 13.2, 0.35 (254) 18.4 / 17.2, 0.80
// (200 over 1.5 decades, 250,000 x 125,000) 8.98 / 6.62; even bins: 0.47 (45) 8.03 / 7.13,
// 1.04 (100) 10.7 / 7.47.
// Small calls take any column there is: the table in LDS spares them the ordering
// (few_pairs, see run_batch).  Mixed ones, whose workgroups don't fill the chip, take
// three workgroups' room for eight columns: 3000 points on the sky in 167 bins of 37 to
// 123 degrees 105 us, 265 with the columns that four leave.
constexpr int32_t kLdsCols = 8;
constexpr double kEdgesMet = 0.2;
void lds_layout(bool fp64, bool few_pairs, double edges_met, int32_t max_edges, int32_t max_cells, int32_t cols,
                int32_t *cols_out, int32_t *cells_out, uint32_t *lds_bytes) {
    auto bytes = [&](int32_t c, int32_t cells) { return static_cast<uint32_t>(8 * (max_edges + cells) + 4 * ((max_edges + 1) * c + max_edges)); };
    static const std::array<uint32_t, 2> fixed = [] {
        hipFuncAttributes a;
        std::array<uint32_t, 2> f = {36u * 1024u, 36u * 1024u};
        if (hipFuncGetAttributes(&a, reinterpret_cast<const void *>(k_count_blocks<false, false>)) == hipSuccess)
            f[0] = static_cast<uint32_t>(a.sharedSizeBytes);
        if (hipFuncGetAttributes(&a, reinterpret_cast<const void *>(k_count_blocks<false, true>)) == hipSuccess)
            f[1] = static_cast<uint32_t>(a.sharedSizeBytes);
        return f;
    }();
    auto room_of = [&](uint32_t workgroups) {
        const uint32_t each = 160u * 1024u / workgroups;
        return each - std::min(fixed[fp64], each);
    };
    uint32_t room = room_of(4);
    if (bytes(1, 0) > room) room = room_of(3);
    if (few_pairs && !fp64 && bytes(std::min(cols, kLdsCols), max_cells) > room) room = room_of(3);
    int32_t c = 1;
    const int32_t least = fp64 || few_pairs ? 1 : std::min(cols, kLdsCols);
    if (max_cells > 0 && bytes(least, max_cells) > room) {
        if (!fp64 && !few_pairs && edges_met >= kEdgesMet && bytes(least, max_cells) <= room_of(3)) room = room_of(3);
        else max_cells = 0;
    }
    while (c < cols && bytes(2 * c, max_cells) <= room) c *= 2;
    *cols_out = c;
    *cells_out = max_cells;
    *lds_bytes = bytes(c, max_cells);
}

// (global_table: the sets' chord tables are not in LDS)
hipError_t occupancy(bool fp64, bool global_table, uint32_t lds_bytes, int *per_cu) {
    const auto k = fp64 ? (global_table ? k_count_blocks<true, true> : k_count_blocks<false, true>)
                        : (global_table ? k_count_blocks<true, false> : k_count_blocks<false, false>);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k, kThreads, lds_bytes);
}

hipError_t launch_count(bool fp64, bool global_table, const SegDesc *segs, const TableDesc *tabs, const uint64_t *items, const uint64_t *tiles,
                        const unsigned long long *n_items, unsigned long long *queue, unsigned long long *rechecked,
                        unsigned long long *stats, unsigned long long *counts, const unsigned long long *copies,
                        int64_t count_words, int32_t max_edges, int32_t max_cells, int32_t cols, uint32_t lds_bytes, int chunk, uint64_t flush_cap, int grid, hipStream_t st) {
    BParams p;
    p.segs = segs;
    p.tabs = tabs;
    p.items = items;
    p.tiles = tiles;
    p.n_items = n_items;
    p.queue = queue;
    p.rechecked = rechecked;
    p.stats = stats;
    p.counts = counts;
    p.copies = copies;
    p.count_words = count_words;
    // a word of the histogram grows by at most 512 x 512 per item
    constexpr uint64_t kCap = 0xFFFFFFFFull / (static_cast<uint64_t>(kT) * kT);
    p.flush_every = static_cast<uint32_t>(flush_cap > 0 && flush_cap < kCap ? flush_cap : kCap);
    p.max_edges = max_edges;
    p.max_cells = max_cells;
    p.cols = cols;
    p.table_edges = fp64 ? table_edges64(cols) : global_table ? table_edges_global(cols) : table_edges(cols);
    p.chunk = chunk;
    const auto k = fp64 ? (global_table ? k_count_blocks<true, true> : k_count_blocks<false, true>)
                        : (global_table ? k_count_blocks<true, false> : k_count_blocks<false, false>);
    k<<<dim3(grid), dim3(kThreads), lds_bytes, st>>>(p);
    return hipGetLastError();
}

}  // namespace blk

}  // namespace pc
