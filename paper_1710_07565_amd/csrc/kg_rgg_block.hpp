// kg_rgg_block.hpp -- the edge passes of the random geometric graphs (two and
// three dimensions) for grids with few points per cell, a wave per block of
// cells (Sec. 5.3: every point against its cell and the neighbours).
//
// A block is one cell or 2^D cells (an aligned group of Morton indices, so its
// points are consecutive vertices u).  Its candidates are the points of the
// cells of its window (the block and one cell around it) with Morton index
// >= the block's first, in ascending index, so in ascending id; the block's own
// points come first.  Testing more than the 3^D window of a point's own cell
// changes nothing: points of cells that do not touch are at least one cell
// side apart, which is at least r.
//
// Task u G + g tests point u against the g-th of G equal parts of the
// candidates, a bit per candidate; task order is output order.  The test is
// made on the points' positions inside their cells, rounded down to 2^-13 or
// 2^-14 of a cell (two 16-bit numbers to a word, written by the points kernel).
// The rounding moves a distance by less than sqrt(D) units, so only squares
// within [lo, lo + band] are open; a word that holds one (a few in 100) is tested
// again, the open candidates in binary64.
//
// Two dimensions: a pass runs 64 tasks, a lane each, and G (1 to 8) is the one
// that needs the fewest instructions for the block's points and candidates;
// all lanes of a part read the same LDS address, one packed subtraction and one
// dot product give d^2 minus the threshold, whose sign bit is shifted into the
// lane's result word.  Three dimensions: the matrix units form these
// differences, G = 4 (rgg_block_count3_kernel).
//
// Count pass: the result words and the block's edge count.  Write pass: the
// words' set bits are the edges, in output order; they are gathered in LDS and
// stored with consecutive lanes on consecutive edges.  A block with more
// candidates than its words hold (the path's rule has how often) is tested in
// binary64 in both passes.
//
// What bounds it: vector instructions (in two dimensions 3.5 per test of about
// 80 per vertex, and more than that again for the window, the lists and the
// masks), in the write pass also latency.  n = 2^26 at
// r = 0.55 (ln n / n)^(1/d), lane per vertex before: two dimensions count 4.4 ->
// 1.9 ms, write 2.6 -> 2.2 ms (call 7.8 -> 4.4 ms); three dimensions count
// 10.7 -> 2.9 ms, write 8.3 -> 1.6 ms (20.8 -> 5.6 ms).
#pragma once
#include "kg_rgg.hpp"
#include "kg_rgg3.hpp"
#include "kg_tile.hpp"

namespace kg {

struct RggBlockJob {
    double r2;
    uint64_t nb;               // blocks
    uint32_t G;                // cells per side
    uint32_t Q;                // position bits per cell
    uint32_t lo, band;         // open squares of quantised distances
    const uint64_t *coff;      // first vertex of every cell
    const uint32_t *q;         // D = 2: (x, y) per vertex; D = 3: (x, y), z
    uint32_t *bits;            // words x n
    uint64_t *bcnt;            // edges per block
    const uint64_t *boff;      // their offsets
    const uint64_t *status;    // [1] overflow
    uint32_t *list;            // D = 3: the candidate lists for the write pass (RggWindow::LIST words per block)
    const double *pts;
    uint2 *edges;
};

constexpr uint32_t kBlockStage = 320;                // edges gathered in LDS (a block has 140 to 200 on average)
constexpr uint32_t kBlocksPerWave = 4;

typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
typedef short short2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));     // 16-byte aligned: one LDS read

// dx^2 + dy^2 + c of two packed positions (no sum leaves 32 bits; the
// saturating form takes c as a third operand instead of a copy of it)
__device__ __forceinline__ int32_t dist2_packed(uint32_t a, uint32_t b, int32_t c)
{
    const ushort2v d = __builtin_bit_cast(ushort2v, a) - __builtin_bit_cast(ushort2v, b);
    const short2v s = __builtin_bit_cast(short2v, d);
    return __builtin_amdgcn_sdot2(s, s, c, true);
}

template <int D>
__device__ __forceinline__ uint32_t cell_spread(uint32_t x) { return D == 2 ? spread_bits(x) : spread3(x); }
template <int D>
__device__ __forceinline__ uint32_t cell_gather(uint32_t z) { return D == 2 ? gather_bits(z) : gather3(z); }

// The bits from position `first` on (any, also below 0 or above 31).
__device__ __forceinline__ uint32_t bits_from(int32_t first)
{
    return (uint32_t)(0xFFFFFFFFull << (uint32_t)min(max(first, 0), 32));
}

// v of lane (lane xor X) within groups of 16 by DPP, across them by a shuffle
template <int X>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    if (X == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);    // quad_perm 1,0,3,2
    if (X == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);    // quad_perm 2,3,0,1
    if (X == 3) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x1B, 0xF, 0xF, false);    // quad_perm 3,2,1,0
    if (X == 7) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    if (X == 15) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false);  // row_mirror
    if (X == 4) return lane_xor<3>(lane_xor<7>(v));
    if (X == 8) return lane_xor<7>(lane_xor<15>(v));
    return (uint32_t)__shfl_xor((int)v, X, 64);
}

// The median of two values and 0 is their minimum, of two and 2^32 - 1 their
// maximum: one instruction for both sides of an exchange.
__device__ __forceinline__ uint32_t median(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Ascending sort of one value per lane inside groups of 16, 32 or 64 lanes: a
// merge first compares each lane with its mirror image, then at halving
// distances, always with the smaller value to the lower lane.
struct LaneSort {
    uint32_t upper[6];       // all ones in the lanes with bit 1, 2, 4, 8, 16, 32

    __device__ __forceinline__ LaneSort()
    {
#pragma unroll
        for (int i = 0; i < 6; ++i) upper[i] = (threadIdx.x >> i & 1) ? ~0u : 0u;
    }

    // lane against lane xor X, the smaller value to the lane without bit i
    template <int X>
    __device__ __forceinline__ void cx(uint32_t &v, int i) const { v = median(v, lane_xor<X>(v), upper[i]); }

    template <int N>
    __device__ __forceinline__ uint32_t sort(uint32_t v) const
    {
        cx<1>(v, 0);
        cx<3>(v, 1); cx<1>(v, 0);
        cx<7>(v, 2); cx<2>(v, 1); cx<1>(v, 0);
        cx<15>(v, 3); cx<4>(v, 2); cx<2>(v, 1); cx<1>(v, 0);
        if (N >= 32) {
            cx<31>(v, 4); cx<8>(v, 3); cx<4>(v, 2); cx<2>(v, 1); cx<1>(v, 0);
        }
        if (N >= 64) {
            cx<63>(v, 5); cx<16>(v, 4); cx<8>(v, 3); cx<4>(v, 2); cx<2>(v, 1); cx<1>(v, 0);
        }
        return v;
    }
};

// Inclusive prefix sums over groups of 16 lanes, or the wave.
template <bool ROWS>
__device__ __forceinline__ uint32_t group_incl_scan32(uint32_t v)
{
    if (!ROWS) return wave_incl_scan32(v);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);   // row_shr:8
    return v;
}

// The candidates of the blocks in hand.  The cells of a window that hold
// points, in ascending order: the vertex at position p of the list is p + base,
// for len positions.  Windows of up to 16 cells are found four at a time (16 lanes and 16
// entries each), larger ones one at a time.
struct RggCells {
    uint32_t base[64], len[64], pos[64], posz[64];
    uint32_t map[4][16];       // one block, or four: bit off - 1 of every cell but the first
};

template <int D, int B, int WORDS>
struct RggWindow {
    static constexpr int W = (1 << B) + 2;                       // window side
    static constexpr int NC = D == 2 ? W * W : W * W * W;        // its cells (9, 16, 27 or 64)
    static constexpr bool ROWS = NC <= 16;
    static constexpr uint32_t LANES = ROWS ? 16 : 64, BLOCKS = 64 / LANES;
    static constexpr uint32_t MAP = ROWS ? 16 : 64;              // map words of a block
    static constexpr uint32_t CAND = 32 * WORDS + 64;            // room of the candidate lists
    // large windows are kept for the write pass: bases, then map, k, C and the cells
    static constexpr uint32_t BASES = NC <= 32 ? 32 : 64, LIST = BASES + 32;
    static_assert(CAND <= 32 * MAP, "a bit per candidate");
    uint32_t st, incl;         // per lane: first vertex of its cell, points up to it
    uint32_t split;            // per lane: parts() of its block
    uint64_t full;             // lanes whose cell holds points
    LaneSort order;

    // The parts of a block's candidates (k, C the same in each 8 lanes): in two
    // dimensions the G of 1 .. 8 with the fewest vector instructions, about 4
    // per candidate and 60 per pass.  Returns G and, above bit
    // 4, the candidates of a part (a multiple of 4); 0 if the result words or
    // the lists are too small.
    static __device__ __forceinline__ uint32_t parts(uint32_t k, uint32_t C)
    {
        if (D == 3) {
            // four parts, as the matrix units' rows take them; an odd multiple
            // of 4 spreads the parts' reads over the LDS banks
            if (C > 32 * WORDS) return 0;
            const uint32_t q = (C + 15) / 16;
            return (q < 2 * WORDS ? q | 1 : q) << 6 | 4;
        }
        const uint32_t g = (threadIdx.x & 7) + 1;
        const uint32_t c = 4 * (uint32_t)((float)(C + 4 * g - 1) * __builtin_amdgcn_rcpf((float)(4 * g)) + 0.0001f);
        uint32_t cost = ((k * g + 63) >> 6) * (4 * c + 60);
        if (C > 32 * WORDS || g * ((c + 31) >> 5) > WORDS || g * c > CAND) cost = 0xFFFF;
        // c <= CAND < 2^10, cost < 2^16: the least cost, its c and g
        uint32_t v = cost << 14 | c << 4 | g;
        v = min(v, lane_xor<1>(v));
        v = min(v, lane_xor<2>(v));
        v = min(v, lane_xor<7>(v));
        return v >> 14 == 0xFFFF ? 0 : v & 0x3FFF;
    }

    // the last two bits of the first coordinate of a Morton index
    static __device__ __forceinline__ uint32_t low2(uint32_t z) { return (z & 1) | (z >> (D - 1) & 2); }

    // the windows of blocks b, b + 1, ... (BLOCKS of them)
    __device__ __forceinline__ void find(const RggBlockJob &J, uint64_t b, RggCells &s)
    {
        const uint32_t lane = threadIdx.x, i = lane % LANES, row = lane / LANES;
        const uint64_t mine = b + row;
        const uint32_t z0 = (uint32_t)(mine << (D * B));
        const uint32_t bx = cell_gather<D>(z0), by = cell_gather<D>(z0 >> 1), bz = D == 3 ? cell_gather<D>(z0 >> 2) : 0;
        uint32_t zz = kRggNone;
        if (i < NC && mine < J.nb) {
            const uint32_t x = bx + i % W - 1, y = by + (i / W) % W - 1, z = D == 3 ? bz + i / (W * W) - 1 : 0;
            if (x < J.G && y < J.G && z < J.G) {
                const uint32_t m = cell_spread<D>(x) | (cell_spread<D>(y) << 1) | (D == 3 ? cell_spread<D>(z) << 2 : 0);
                if (m >= z0) zz = m;
            }
        }
        zz = order.sort<(NC <= 16 ? 16 : NC <= 32 ? 32 : 64)>(zz);
        uint32_t len = 0;
        st = 0;
        if (zz != kRggNone) {
            st = (uint32_t)J.coff[zz];
            len = (uint32_t)J.coff[zz + 1] - st;
        }
        incl = group_incl_scan32<ROWS>(len);
        const uint32_t off = incl - len;
        split = parts((uint32_t)__shfl((int)incl, (int)(row * LANES + (1 << (D * B)) - 1), 64),
                      (uint32_t)__shfl((int)incl, (int)(row * LANES + LANES - 1), 64));
        full = __ballot(len != 0);
        (&s.map[0][0])[lane] = 0;
        __syncthreads();
        if (len != 0) {
            const uint64_t before = full & lanemask_lt(lane);
            const uint32_t n = (uint32_t)__popcll(ROWS ? before >> (16 * row) : before);
            const uint32_t at = row * LANES + n;
            s.base[at] = st - off;
            s.len[at] = len;
            // 0 .. 3 in each dimension: the coordinates' last two bits tell
            const uint32_t ox = (low2(zz) - bx + 1) & 3, oy = (low2(zz >> 1) - by + 1) & 3;
            s.pos[at] = (ox << J.Q) | (oy << J.Q << 16);
            if (D == 3) s.posz[at] = ((low2(zz >> 2) - bz + 1) & 3) << J.Q;
            if (n && off <= 32 * MAP)
                atomicOr(&(&s.map[0][0])[row * MAP + ((off - 1) >> 5)], 1u << ((off - 1) & 31));
        }
        __syncthreads();
    }
};

// One block of a window set: row j.
template <int D, int B, int WORDS>
struct RggBlock {
    typedef RggWindow<D, B, WORDS> Window;
    static constexpr uint32_t CAND = Window::CAND;
    uint32_t j, u0, k, C, cells;      // row, first vertex, points, candidates, cells with points
    uint32_t G, Cg, live;             // parts, candidates of a part (a multiple of 4), tasks
    uint32_t magic;                   // task / G = task * magic >> 16
    bool light;

    __device__ __forceinline__ RggBlock(const Window &w, uint32_t row)
    {
        constexpr uint32_t L = Window::LANES;
        j = row;
        u0 = __builtin_amdgcn_readlane(w.st, L * row);           // the block's first cell is the smallest
        k = __builtin_amdgcn_readlane(w.incl, L * row + (1 << (D * B)) - 1);
        C = __builtin_amdgcn_readlane(w.incl, L * row + L - 1);
        cells = (uint32_t)__popcll(Window::ROWS ? w.full >> (16 * row) & 0xFFFF : w.full);
        tasks(__builtin_amdgcn_readlane(w.split, L * row));
    }

    // a block whose list the count pass kept
    __device__ __forceinline__ RggBlock(const uint32_t *list, RggCells &s)
    {
        const uint32_t lane = threadIdx.x;
        const uint32_t a = lane < Window::BASES ? list[lane] : 0, t = list[Window::BASES + (lane & 31)];
        s.base[lane] = a;
        if (lane < 32) (&s.map[0][0])[lane] = t;
        j = 0;
        u0 = __builtin_amdgcn_readfirstlane(a);
        k = __builtin_amdgcn_readlane(t, 29);
        C = __builtin_amdgcn_readlane(t, 30);
        cells = __builtin_amdgcn_readlane(t, 31);
        tasks(__builtin_amdgcn_readlane(t, 28));
        __syncthreads();
    }

    __device__ __forceinline__ void keep(uint32_t *list, const RggCells &s) const
    {
        static_assert(CAND <= 28 * 32, "map words beside the four counts");
        const uint32_t lane = threadIdx.x;
        if (lane < cells) list[lane] = s.base[lane];
        if (lane < 32)
            list[Window::BASES + lane] = lane == 28 ? Cg << 4 | G : lane == 29 ? k : lane == 30 ? C : lane == 31 ? cells
                                                         : (&s.map[0][0])[lane];
    }

    __device__ __forceinline__ void tasks(uint32_t split)
    {
        G = split & 15;
        Cg = split >> 4;
        light = G != 0;
        live = k * G;
        // floor(65536 / G) + 1, or 65536 / G where that is whole: exact for task * G < 65536
        magic = D == 2 && light ? uni((uint32_t)(65536.0f * __builtin_amdgcn_rcpf((float)G)) + 1) : 0;
    }

    // Three dimensions: a part's words (1, 2 or 4, so their number is a shift)
    // and the candidates of a word but a part's last (a multiple of 4).  Word
    // w of task t is word t << word_log() + w of the block, in output order.
    __device__ __forceinline__ uint32_t word_log() const { return Cg <= 32 ? 0 : Cg <= 64 ? 1 : 2; }
    __device__ __forceinline__ uint32_t word_len() const
    {
        const uint32_t l = word_log();
        return ((Cg / 4 + (1u << l) - 1) >> l) * 4;
    }

    // point and first candidate of a task
    __device__ __forceinline__ uint32_t point(uint32_t task) const { return task < live ? task * magic >> 16 : 0; }
    __device__ __forceinline__ uint32_t part(uint32_t task, uint32_t u) const { return task < live ? (task - u * G) * Cg : 0; }

    // f(p, v, c) for every candidate: position, vertex, cell entry
    template <class F>
    __device__ __forceinline__ void each(const RggCells &s, F f) const
    {
        const uint32_t lane = threadIdx.x;
        const uint32_t *map = &s.map[0][0] + Window::MAP * j;
        uint32_t before = Window::LANES * j;
        for (uint32_t t = 0; t < C; t += 64) {
            const uint32_t m0 = map[t / 32], m1 = map[t / 32 + 1];
            const uint32_t c = __builtin_amdgcn_mbcnt_hi(m1, __builtin_amdgcn_mbcnt_lo(m0, before));
            before += __builtin_popcount(m0) + __builtin_popcount(m1);
            const uint32_t p = t + lane;
            if (p < C) f(p, p + s.base[c], c);
        }
    }

    // the vertex at position p of the candidates
    __device__ __forceinline__ uint32_t vertex(const RggCells &s, uint32_t p) const
    {
        const uint32_t *map = &s.map[0][0] + Window::MAP * j;
        uint32_t c = Window::LANES * j + __builtin_popcount(map[p / 32] & ((1u << (p & 31)) - 1));
        for (uint32_t w = 0; w < p / 32; ++w) c += __builtin_popcount(map[w]);
        return p + s.base[c];
    }

    // binary64 predicate of two vertices
    static __device__ __forceinline__ bool near(const RggBlockJob &J, uint32_t u, uint32_t v)
    {
        const double *a = J.pts + (uint64_t)D * u, *b = J.pts + (uint64_t)D * v;
        const double dx = a[0] - b[0], dy = a[1] - b[1];
        double d2 = dx * dx + dy * dy;
        if (D == 3) {
            const double dz = a[2] - b[2];
            d2 = d2 + dz * dz;
        }
        return d2 < J.r2;
    }

    // every edge of a heavy block's vertex u (ids ascend): f(v)
    template <class F>
    __device__ __forceinline__ void heavy(const RggBlockJob &J, const RggCells &s, uint32_t u, F f) const
    {
        uint32_t p = 0;
        for (uint32_t c = Window::LANES * j; c < Window::LANES * j + cells; ++c) {
            for (const uint32_t end = p + s.len[c]; p != end; ++p) {
                const uint32_t v = p + s.base[c];
                if (v > u && near(J, u, v)) f(v);
            }
        }
    }
};

template <int B, int WORDS>
__global__ __launch_bounds__(64) void rgg_block_count2_kernel(RggBlockJob J)
{
    typedef RggWindow<2, B, WORDS> Window;
    typedef RggBlock<2, B, WORDS> Block;
    __shared__ RggCells s;
    __shared__ __attribute__((aligned(16))) uint32_t s_xy[Block::CAND];
    __shared__ uint32_t s_id[Block::CAND];
    const uint32_t lane = threadIdx.x;
    const uint64_t b0 = (uint64_t)blockIdx.x * kBlocksPerWave;
    Window win;
    for (uint32_t bi = 0; bi < kBlocksPerWave && b0 + bi < J.nb; ++bi) {
        if (bi % Window::BLOCKS == 0) win.find(J, b0 + bi, s);
        const Block K(win, bi % Window::BLOCKS);
        uint32_t cnt = 0;
        if (K.k && K.light) {
            K.each(s, [&](uint32_t p, uint32_t v, uint32_t c) {
                s_id[p] = v;
                s_xy[p] = J.q[v] + s.pos[c];
            });
            // padding: the window's corner, at squares of at least lo, which
            // are open at most, and open candidates are checked against C
            for (uint32_t p = K.C + lane; p < K.G * K.Cg; p += 64) s_xy[p] = 0;
            __syncthreads();
            const int32_t base = -(int32_t)J.lo;
            auto square = [&](uint32_t xy, uint32_t axy) { return (uint32_t)dist2_packed(xy, axy, base); };
            for (uint32_t t = 0; t < K.live; t += 64) {
                const uint32_t task = t + lane;
                const uint32_t u = K.point(task), g0 = K.part(task, u);
                const uint32_t uxy = s_xy[u];
                const uint64_t own = __ballot(task < K.live);
                uint32_t *out = J.bits + (uint64_t)K.u0 * WORDS + task;
                for (uint32_t w = 0; w < K.Cg; w += 32, out += K.live) {
                    const uint32_t quads = uni(min(8u, (K.Cg - w) / 4)), p0 = g0 + w;
                    uint32_t acc = 0, open = ~0u;
                    for (uint32_t i = 0; i < quads; ++i) {
                        const uint4v c = *reinterpret_cast<const uint4v *>(s_xy + p0 + 4 * i);
                        const uint32_t t0 = square(c.x, uxy), t1 = square(c.y, uxy), t2 = square(c.z, uxy),
                                       t3 = square(c.w, uxy);
                        acc = __builtin_amdgcn_alignbit(acc, t0, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t1, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t2, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t3, 31);
                        open = min(open, min(t0, t1));
                        open = min(open, min(t2, t3));
                    }
                    // bit i: candidate p0 + i
                    uint32_t m = __builtin_bitreverse32(acc << ((32 - 4 * quads) & 31));
                    // a lane whose word holds an open square: its candidates, a
                    // lane each, by the quantised and, if open, the exact test
                    for (uint64_t mo = __ballot(open <= J.band) & own; mo; mo &= mo - 1) {
                        const int l = __builtin_ctzll(mo);
                        const uint32_t lu = __builtin_amdgcn_readlane(u, l), lp = __builtin_amdgcn_readlane(p0, l);
                        const uint32_t p = lp + (lane & 31);
                        bool hit = false;
                        if (lane < 4 * quads && p < K.C) {
                            if (square(s_xy[p], s_xy[lu]) <= J.band) hit = Block::near(J, K.u0 + lu, s_id[p]);
                        }
                        const uint32_t found = (uint32_t)__ballot(hit);
                        if ((int)lane == l) m |= found;
                    }
                    m &= bits_from((int32_t)(u + 1) - (int32_t)p0);      // after u
                    if (task < K.live) {
                        cnt += __builtin_popcount(m);
                        *out = m;
                    }
                }
            }
            cnt = wave_incl_scan32(cnt);
            if (lane == 63) J.bcnt[b0 + bi] = cnt;
        } else {
            for (uint32_t u = lane; u < K.k; u += 64) K.heavy(J, s, K.u0 + u, [&](uint32_t) { ++cnt; });
            const uint64_t total = wave_incl_scan64(cnt);
            if (lane == 63) J.bcnt[b0 + bi] = total;
        }
        __syncthreads();
    }
}

// Three dimensions: |u|^2 - 2 u.c + |c|^2 is a product of a column (x, y, z, 1)
// per point and a row (-2x, -2y, -2z, |c|^2) per candidate, so the matrix
// units form d^2 minus the threshold for 16 points x 16 candidates in one
// binary32 instruction (K = 4, the sum starts from |u|^2 - lo).  Rows 4h .. 4h + 3 of a
// product come out in lanes 16 h .. 16 h + 15: they take candidates of part h,
// so lane 16 h + c holds the results of point c against part h, in order.
// Coordinates count from the window's centre: with cell side 2^Q every partial
// sum is below 48 4^Q, and the roundings together below 2^(2Q - 15.7); `open`
// squares are taken 2^(2Q - 14) further to both sides.  A product and 6 vector
// instructions per 256 tests, where the packed form of two dimensions takes
// 30: 594 vector instructions per block instead of 1056.  n = 2^26,
// r = 0.55 (ln n / n)^(1/3): 3.9 -> 2.9 ms (products and vector instructions of a
// SIMD hardly overlap: 23 and 70 % of the time).
template <int B, int WORDS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void rgg_block_count3_kernel(RggBlockJob J)
{
    typedef RggWindow<3, B, WORDS> Window;
    typedef RggBlock<3, B, WORDS> Block;
    typedef float float4v __attribute__((ext_vector_type(4)));
    constexpr uint32_t S = 32 * WORDS + 16;     // 16 words past a multiple of 64: the components' reads
                                                // fall into different banks; also room for the last 16 points
    __shared__ RggCells s;
    __shared__ float s_f[4 * S];                // -2x, -2y, -2z, x^2 + y^2 + z^2 of every candidate
    const uint32_t lane = threadIdx.x, col = lane & 15, h = lane >> 4;
    const uint64_t b0 = (uint64_t)blockIdx.x * kBlocksPerWave;
    const float mid2 = (float)(Window::W << J.Q);               // twice the centre
    const float margin = (float)(1u << (2 * J.Q - 14));
    const float thr = (float)J.lo - margin;
    const float wide_f = (float)J.band + 2.0f * margin;
    const uint32_t wide = __float_as_uint(wide_f);
    Window win;
    for (uint32_t bi = 0; bi < kBlocksPerWave && b0 + bi < J.nb; ++bi) {
        win.find(J, b0 + bi, s);
        const Block K(win, 0);
        K.keep(J.list + (b0 + bi) * Window::LIST, s);
        uint32_t cnt = 0;
        if (K.k && K.light) {
            K.each(s, [&](uint32_t p, uint32_t v, uint32_t c) {
                const uint2 w = reinterpret_cast<const uint2 *>(J.q)[v];
                const uint32_t xy = w.x + s.pos[c];
                const float x = __builtin_fmaf((float)(xy & 0xFFFF), -2.0f, mid2);
                const float y = __builtin_fmaf((float)(xy >> 16), -2.0f, mid2);
                const float z = __builtin_fmaf((float)(w.y + s.posz[c]), -2.0f, mid2);
                s_f[p] = x;
                s_f[S + p] = y;
                s_f[2 * S + p] = z;
                s_f[3 * S + p] = 0.25f * __builtin_fmaf(x, x, __builtin_fmaf(y, y, z * z));
            });
            // padding: far away
            for (uint32_t p = K.C + lane; p < 4 * K.Cg; p += 64) {
                s_f[p] = s_f[S + p] = s_f[2 * S + p] = 0.0f;
                s_f[3 * S + p] = 1e15f;
            }
            __syncthreads();
            const uint32_t wlog = K.word_log(), wlen = K.word_len();
            const float *row = s_f + h * S + (col >> 2) * K.Cg + (col & 3);
            for (uint32_t t = 0; t < K.k; t += 16) {
                const uint32_t u = t + col;
                const float b = h == 3 ? 1.0f : u < K.k ? -0.5f * s_f[h * S + u] : 0.0f;
                const float c0 = u < K.k ? s_f[3 * S + u] - thr : 1e15f;      // no point: far from all
                const float4v from = {c0, c0, c0, c0};
                uint32_t *out = J.bits + (uint64_t)K.u0 * WORDS + ((4 * u + h) << wlog);
                for (uint32_t w = 0; w < K.Cg; w += wlen, ++out) {
                    const uint32_t quads = uni(min(wlen, K.Cg - w) / 4), p0 = h * K.Cg + w;
                    uint32_t acc = 0, open = ~0u;
                    auto take = [&](const float4v &d) {
                        const uint32_t t0 = __float_as_uint(d.x), t1 = __float_as_uint(d.y),
                                       t2 = __float_as_uint(d.z), t3 = __float_as_uint(d.w);
                        acc = __builtin_amdgcn_alignbit(acc, t0, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t1, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t2, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t3, 31);
                        open = min(min(open, t0), t1);
                        open = min(min(open, t2), t3);
                    };
                    uint32_t i = 0;
                    for (; i + 2 <= quads; i += 2) {
                        const float a0 = row[w + 4 * i], a1 = row[w + 4 * i + 4];
                        const float4v d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b, from, 0, 0, 0);
                        const float4v d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b, from, 0, 0, 0);
                        take(d0);
                        take(d1);
                    }
                    if (i < quads) take(__builtin_amdgcn_mfma_f32_16x16x4f32(row[w + 4 * i], b, from, 0, 0, 0));
                    // bit i: candidate p0 + i
                    uint32_t m = __builtin_bitreverse32(acc << ((32 - 4 * quads) & 31));
                    // a lane whose word holds an open square: its candidates, a
                    // lane each, by a direct square and, if open, the exact test
                    for (uint64_t mo = __ballot(open <= wide); mo; mo &= mo - 1) {
                        const int l = __builtin_ctzll(mo);
                        const uint32_t lu = __builtin_amdgcn_readlane(u, l), lp = __builtin_amdgcn_readlane(p0, l);
                        const uint32_t p = lp + (lane & 31);
                        bool hit = false;
                        if (lane < 4 * quads && p < K.C) {
                            const float dx = s_f[p] - s_f[lu], dy = s_f[S + p] - s_f[S + lu], dz = s_f[2 * S + p] - s_f[2 * S + lu];
                            const float d = 0.25f * __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz)) - thr;
                            if (d <= wide_f) hit = d < 0.0f || Block::near(J, K.u0 + lu, K.vertex(s, p));
                        }
                        const uint32_t found = (uint32_t)__ballot(hit);
                        if ((int)lane == l) m |= found;
                    }
                    m &= bits_from((int32_t)(u + 1) - (int32_t)p0);      // after u
                    cnt += __builtin_popcount(m);
                    if (u < K.k) *out = m;
                }
            }
            cnt = wave_incl_scan32(cnt);
            if (lane == 63) J.bcnt[b0 + bi] = cnt;
        } else {
            for (uint32_t u = lane; u < K.k; u += 64) K.heavy(J, s, K.u0 + u, [&](uint32_t) { ++cnt; });
            const uint64_t total = wave_incl_scan64(cnt);
            if (lane == 63) J.bcnt[b0 + bi] = total;
        }
        __syncthreads();
    }
}

template <int D, int B, int WORDS>
__global__ __launch_bounds__(64) void rgg_block_write_kernel(RggBlockJob J)
{
    typedef RggWindow<D, B, WORDS> Window;
    typedef RggBlock<D, B, WORDS> Block;
    __shared__ RggCells s;
    __shared__ uint32_t s_id[Block::CAND];
    __shared__ uint2 s_e[kBlockStage];
    if (ld_uni(J.status + 1)) return;
    const uint32_t lane = threadIdx.x;
    const uint64_t b0 = (uint64_t)blockIdx.x * kBlocksPerWave;
    Window win;
    uint32_t first[Window::BLOCKS];      // the first result words of the blocks in hand, read together
    for (uint32_t bi = 0; bi < kBlocksPerWave && b0 + bi < J.nb; ++bi) {
        const uint64_t o = ld_uni(J.boff + b0 + bi);
        const uint64_t total = ld_uni(J.boff + b0 + bi + 1) - o;
        if (D == 2 && bi % Window::BLOCKS == 0) {
            win.find(J, b0 + bi, s);
#pragma unroll
            for (uint32_t j = 0; j < Window::BLOCKS; ++j) {
                const Block K(win, j);
                first[j] = lane < K.live ? J.bits[(uint64_t)K.u0 * WORDS + lane] : 0;
            }
        }
        if (total == 0) continue;
        const Block K = D == 2 ? Block(win, bi % Window::BLOCKS) : Block(J.list + (b0 + bi) * Window::LIST, s);
        if (K.light) {
            const bool staged = total <= kBlockStage;
            // a word's edges, in order: two per trip, their ids are read together
            auto put = [&](uint32_t u, uint32_t m, const uint32_t *id, uint32_t &at) {
                if (staged) {
                    while (m) {
                        const uint32_t i0 = __builtin_ctz(m);
                        m &= m - 1;
                        const uint32_t i1 = m ? __builtin_ctz(m) : i0;
                        const uint32_t v0 = id[i0], v1 = id[i1];
                        s_e[at] = make_uint2(u, v0);
                        if (m) s_e[at + 1] = make_uint2(u, v1);
                        at += m ? 2 : 1;
                        m &= m - 1;
                    }
                } else {
                    for (; m; m &= m - 1) J.edges[o + at++] = make_uint2(u, id[__builtin_ctz(m)]);
                }
            };
            if (D == 3) {
                // a lane takes n consecutive words of the block; the first
                // kRowWords stay in registers for the second look
                const uint32_t wlog = K.word_log(), wlen = K.word_len(), words = K.live << wlog, n = (words + 63) / 64;
                const uint32_t *in = J.bits + (uint64_t)K.u0 * WORDS + lane * n;
                const uint32_t mine = lane * n < words ? min(n, words - lane * n) : 0;
                constexpr uint32_t kRowWords = 8;
                uint32_t m[kRowWords];
#pragma unroll
                for (uint32_t i = 0; i < kRowWords; ++i) m[i] = i < mine ? in[i] : 0;
                K.each(s, [&](uint32_t p, uint32_t v, uint32_t) { s_id[p] = v; });
                __syncthreads();
                uint32_t cnt = 0;
#pragma unroll
                for (uint32_t i = 0; i < kRowWords; ++i) cnt += __builtin_popcount(m[i]);
                for (uint32_t i = kRowWords; i < mine; ++i) cnt += __builtin_popcount(in[i]);
                uint32_t at = wave_incl_scan32(cnt) - cnt;
                auto word = [&](uint32_t i, uint32_t m) {
                    const uint32_t x = lane * n + i, t = x >> wlog;
                    put(K.u0 + (t >> 2), m, s_id + (t & 3) * K.Cg + (x & ((1u << wlog) - 1)) * wlen, at);
                };
#pragma unroll
                for (uint32_t i = 0; i < kRowWords; ++i)
                    if (i < n) word(i, m[i]);
                for (uint32_t i = kRowWords; i < mine; ++i) word(i, in[i]);
            } else {
                const uint32_t nw = (K.Cg + 31) / 32;
                uint32_t done = 0;
                uint32_t m = first[0];
#pragma unroll
                for (uint32_t j = 1; j < Window::BLOCKS; ++j) m = bi % Window::BLOCKS == j ? first[j] : m;
                K.each(s, [&](uint32_t p, uint32_t v, uint32_t) { s_id[p] = v; });
                __syncthreads();
                for (uint32_t t = 0; t < K.live; t += 64) {
                    const uint32_t task = t + lane;
                    const uint32_t *in = J.bits + (uint64_t)K.u0 * WORDS + task;
                    const bool own = task < K.live;
                    const uint32_t lu = K.point(task), u = K.u0 + lu;
                    if (t != 0) m = own ? in[0] : 0;
                    uint32_t cnt = __builtin_popcount(m);
                    for (uint32_t w = 1; w < nw; ++w) cnt += own ? __builtin_popcount(in[w * K.live]) : 0;
                    const uint32_t incl = wave_incl_scan32(cnt);
                    uint32_t at = done + incl - cnt;
                    done += __builtin_amdgcn_readlane(incl, 63);
                    const uint32_t *id = s_id + K.part(task, lu);
                    for (uint32_t w = 0;; id += 32) {
                        put(u, m, id, at);
                        if (++w == nw) break;
                        m = own ? in[w * K.live] : 0;
                    }
                }
            }
            __syncthreads();
            if (staged)
                for (uint32_t i = lane; i < (uint32_t)total; i += 64) J.edges[o + i] = s_e[i];
        } else {
            if (D == 3) win.find(J, b0 + bi, s);
            uint64_t before = o;
            for (uint32_t ub = 0; ub < K.k; ub += 64) {
                const uint32_t u = K.u0 + ub + lane;
                const bool in = ub + lane < K.k;
                uint64_t cnt = 0;
                if (in) K.heavy(J, s, u, [&](uint32_t) { ++cnt; });
                const uint64_t incl = wave_incl_scan64(cnt);
                uint64_t at = before + incl - cnt;
                if (in) K.heavy(J, s, u, [&](uint32_t v) { J.edges[at++] = make_uint2(u, v); });
                before += __shfl(incl, 63, 64);
            }
        }
        __syncthreads();
    }
}

}  // namespace kg
