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
// candidates; a pass runs 64 tasks, a lane each, and G (1 to 8) is the one that
// needs the fewest instructions for the block's points and candidates.  All
// lanes of a part read the same LDS address, and task order is output order.  The test is made on the points' positions inside
// their cells, rounded down to 2^-13 or 2^-14 of a cell (two 16-bit numbers
// to a word, written by the points kernel): one packed subtraction and one
// dot product give d^2 minus the threshold, whose sign bit is shifted into the
// lane's result word.  The rounding moves a distance by less than sqrt(D)
// units, so only squares within [lo, lo + band] are open; a word that holds
// one (a few in 100) is tested again, the open candidates in binary64.
//
// Count pass: the result words and the block's edge count.  Write pass: the
// words' set bits are the edges, in output order; they are gathered in LDS and
// stored with consecutive lanes on consecutive edges.  A block with more
// candidates than its words hold (hardly ever at the densities this path is
// chosen for) is tested in binary64 in both passes.
//
// What bounds it: vector instructions in the count pass (3.5 per test in two
// dimensions, 5.5 in three, of about 80 and 144 tests per vertex, and as much
// again for the window, the lists and the masks), latency in the write pass.
// n = 2^26 at r = 0.55 (ln n / n)^(1/d), lane per vertex before: two
// dimensions count 4.4 -> 2.0 ms, write 2.6 -> 2.2 ms (call 7.8 -> 4.8 ms);
// three dimensions count 10.7 -> 3.8 ms, write 8.3 -> 2.2 ms (20.8 -> 7.1 ms).
#pragma once
#include "kg_rgg.hpp"
#include "kg_rgg3.hpp"
#include "kg_tile.hpp"

namespace kg {

struct RggBlockJob {
    uint64_t n, capacity;
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

template <int X>
__device__ __forceinline__ void lane_cx(uint32_t &v, uint32_t bit)
{
    const uint32_t t = lane_xor<X>(v);
    const uint32_t a = min(v, t), b = max(v, t);
    v = (threadIdx.x & bit) ? b : a;
}

// Ascending sort of one value per lane inside groups of 16, 32 or 64 lanes: a
// merge first compares each lane with its mirror image, then at halving
// distances, always with the smaller value to the lower lane.
template <int N>
__device__ __forceinline__ uint32_t lane_sort(uint32_t v)
{
    lane_cx<1>(v, 1);
    lane_cx<3>(v, 2); lane_cx<1>(v, 1);
    lane_cx<7>(v, 4); lane_cx<2>(v, 2); lane_cx<1>(v, 1);
    lane_cx<15>(v, 8); lane_cx<4>(v, 4); lane_cx<2>(v, 2); lane_cx<1>(v, 1);
    if (N >= 32) {
        lane_cx<31>(v, 16); lane_cx<8>(v, 8); lane_cx<4>(v, 4); lane_cx<2>(v, 2); lane_cx<1>(v, 1);
    }
    if (N >= 64) {
        lane_cx<63>(v, 32); lane_cx<16>(v, 16); lane_cx<8>(v, 8); lane_cx<4>(v, 4); lane_cx<2>(v, 2); lane_cx<1>(v, 1);
    }
    return v;
}

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

    // The parts of a block's candidates (k, C the same in each 8 lanes): the G
    // of 1 .. 8 with the fewest vector instructions, about 4 (6 in three
    // dimensions) per candidate and 60 per pass.  Returns G and, above bit
    // 4, the candidates of a part (a multiple of 4); 0 if the result words or
    // the lists are too small.
    static __device__ __forceinline__ uint32_t parts(uint32_t k, uint32_t C)
    {
        const uint32_t g = (threadIdx.x & 7) + 1;
        const uint32_t c = 4 * (uint32_t)((float)(C + 4 * g - 1) * __builtin_amdgcn_rcpf((float)(4 * g)) + 0.0001f);
        uint32_t cost = ((k * g + 63) >> 6) * ((D == 2 ? 4 : 6) * c + 60);
        if (C > 32 * WORDS || g * ((c + 31) >> 5) > WORDS || g * c > CAND) cost = 0xFFFF;
        // c <= CAND < 2^10, cost < 2^16: the least cost, its c and g
        uint32_t v = cost << 14 | c << 4 | g;
        v = min(v, lane_xor<1>(v));
        v = min(v, lane_xor<2>(v));
        v = min(v, lane_xor<7>(v));
        return v >> 14 == 0xFFFF ? 0 : v & 0x3FFF;
    }

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
        zz = lane_sort<(NC <= 16 ? 16 : NC <= 32 ? 32 : 64)>(zz);
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
            const uint32_t ox = cell_gather<D>(zz) - bx + 1, oy = cell_gather<D>(zz >> 1) - by + 1;
            s.pos[at] = (ox << J.Q) | (oy << J.Q << 16);
            if (D == 3) s.posz[at] = (cell_gather<D>(zz >> 2) - bz + 1) << J.Q;
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
        magic = light ? uni((uint32_t)(65536.0f * __builtin_amdgcn_rcpf((float)G)) + 1) : 0;
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

template <int D, int B, int WORDS>
__global__ __launch_bounds__(64) void rgg_block_count_kernel(RggBlockJob J)
{
    typedef RggWindow<D, B, WORDS> Window;
    typedef RggBlock<D, B, WORDS> Block;
    __shared__ RggCells s;
    __shared__ __attribute__((aligned(16))) uint32_t s_xy[Block::CAND];
    __shared__ __attribute__((aligned(16))) uint32_t s_z[D == 3 ? Block::CAND : 4];
    __shared__ uint32_t s_id[Block::CAND];
    const uint32_t lane = threadIdx.x;
    const uint64_t b0 = (uint64_t)blockIdx.x * kBlocksPerWave;
    Window win;
    for (uint32_t bi = 0; bi < kBlocksPerWave && b0 + bi < J.nb; ++bi) {
        if (bi % Window::BLOCKS == 0) win.find(J, b0 + bi, s);
        const Block K(win, bi % Window::BLOCKS);
        if (D == 3) K.keep(J.list + (b0 + bi) * Window::LIST, s);
        uint32_t cnt = 0;
        if (K.k && K.light) {
            K.each(s, [&](uint32_t p, uint32_t v, uint32_t c) {
                s_id[p] = v;
                if (D == 2) {
                    s_xy[p] = J.q[v] + s.pos[c];
                } else {
                    const uint2 w = reinterpret_cast<const uint2 *>(J.q)[v];
                    s_xy[p] = w.x + s.pos[c];
                    s_z[p] = w.y + s.posz[c];
                }
            });
            // padding: the window's corner, further from the block than r
            for (uint32_t p = K.C + lane; p < K.G * K.Cg; p += 64) {
                s_xy[p] = 0;
                if (D == 3) s_z[p] = 0;
            }
            __syncthreads();
            const int32_t base = -(int32_t)J.lo;
            auto square = [&](uint32_t xy, uint32_t z, uint32_t axy, uint32_t az) -> uint32_t {
                const int32_t dz = D == 3 ? (int32_t)(z - az) : 0;
                return (uint32_t)dist2_packed(xy, axy, D == 3 ? __mul24(dz, dz) + base : base);
            };
            for (uint32_t t = 0; t < K.live; t += 64) {
                const uint32_t task = t + lane;
                const uint32_t u = K.point(task), g0 = K.part(task, u);
                const uint32_t uxy = s_xy[u], uz = D == 3 ? s_z[u] : 0;
                uint32_t *out = J.bits + (uint64_t)K.u0 * WORDS + task;
                for (uint32_t w = 0; w < K.Cg; w += 32, out += K.live) {
                    const uint32_t quads = uni(min(8u, (K.Cg - w) / 4)), p0 = g0 + w;
                    uint32_t acc = 0, open = ~0u;
                    for (uint32_t i = 0; i < quads; ++i) {
                        const uint4v c = *reinterpret_cast<const uint4v *>(s_xy + p0 + 4 * i);
                        uint4v cz = {0, 0, 0, 0};
                        if (D == 3) cz = *reinterpret_cast<const uint4v *>(s_z + p0 + 4 * i);
                        const uint32_t t0 = square(c.x, cz.x, uxy, uz), t1 = square(c.y, cz.y, uxy, uz),
                                       t2 = square(c.z, cz.z, uxy, uz), t3 = square(c.w, cz.w, uxy, uz);
                        acc = __builtin_amdgcn_alignbit(acc, t0, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t1, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t2, 31);
                        acc = __builtin_amdgcn_alignbit(acc, t3, 31);
                        open = min(open, min(t0, t1));
                        open = min(open, min(t2, t3));
                    }
                    // bit i: candidate p0 + i, after u and in the list
                    uint32_t m = __builtin_bitreverse32(acc << ((32 - 4 * quads) & 31));
                    const int32_t first = (int32_t)(u + 1) - (int32_t)p0, end = (int32_t)K.C - (int32_t)p0;
                    uint32_t ok = first <= 0 ? ~0u : first >= 32 ? 0u : ~0u << first;
                    ok &= end >= 32 ? ~0u : end <= 0 ? 0u : (1u << end) - 1;
                    if (task >= K.live) ok = 0;
                    // a lane whose word holds an open square: its candidates, a
                    // lane each, by the quantised and, if open, the exact test
                    for (uint64_t mo = __ballot(open <= J.band && ok != 0); mo; mo &= mo - 1) {
                        const int l = __builtin_ctzll(mo);
                        const uint32_t lu = __builtin_amdgcn_readlane(u, l), lp = __builtin_amdgcn_readlane(p0, l);
                        const uint32_t p = lp + (lane & 31);
                        bool hit = false;
                        if (lane < 4 * quads && p < K.C) {
                            const uint32_t t = square(s_xy[p], D == 3 ? s_z[p] : 0, s_xy[lu], D == 3 ? s_z[lu] : 0);
                            if (t <= J.band) hit = Block::near(J, K.u0 + lu, s_id[p]);
                        }
                        const uint32_t found = (uint32_t)__ballot(hit);
                        if ((int)lane == l) m |= found;
                    }
                    m &= ok;
                    cnt += __builtin_popcount(m);
                    if (task < K.live) *out = m;
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
            const uint32_t nw = (K.Cg + 31) / 32;
            const bool staged = total <= kBlockStage;
            uint32_t done = 0;
            uint32_t m = first[0];
#pragma unroll
            for (uint32_t j = 1; j < Window::BLOCKS; ++j) m = bi % Window::BLOCKS == j ? first[j] : m;
            if (D == 3) m = lane < K.live ? J.bits[(uint64_t)K.u0 * WORDS + lane] : 0;
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
                    if (staged) {
                        // two edges per trip: their ids are read together
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
                    if (++w == nw) break;
                    m = own ? in[w * K.live] : 0;
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
