// kg_tile.hpp -- the sampler's two kernels.
//
//   tile_kernel  : the common case.  One wavefront per tile; a tile whose
//                  base case needs at most kFastDraws draws keeps them in
//                  registers (16 per lane), sorts them in LDS and streams the
//                  decoded edges out.  Any other tile is appended to a queue.
//   queue_kernel : the queued tiles, with the general base case (key
//                  sub-ranges when the draws exceed the LDS capacity).
//
// Both produce the same bits for a tile: the sorted distinct set of the
// first J draws of the tile's stream with J the smallest count giving k
// distinct valid values (Sec. 2.2 base case; Sec. 4.1, 4.2 offsets).
#pragma once
#include "kg_kernels.hpp"

namespace kg {

constexpr uint32_t kFastDraws = 1280;   // draws of one wave's base case (at most 5 Philox blocks per lane)
constexpr uint32_t kFastRounds = 5;     // rounds of 256 draws (one Philox block per lane each)
constexpr uint32_t kKeyWords = 1288;    // LDS key words: >= kFastDraws + 3 and >= the widest sort span (64 x 20)
constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr uint64_t kGrabBig = 32;       // tiles per range a workgroup takes from the shared counter ...
constexpr uint64_t kGrabSmall = 8;      // ... and near the end of the walk
constexpr uint64_t kTailTiles = 64;     // tiles per workgroup handed out in small ranges
constexpr uint32_t kStripeBig = 8;      // tiles of a batch's fixed ranges ...
constexpr uint32_t kStripeSmall = 4;    // ... and where all of them are fixed
constexpr uint64_t kStaticTiles = 16;   // fewer tiles per workgroup than this are shared out in advance

// Wave-uniform 64-bit load through the scalar data cache.  Only for data
// that no lane writes while the kernel runs (sizes and offsets written by
// the earlier kernels of the pass).
__device__ __forceinline__ uint64_t ld_uni(const uint64_t *p)
{
    return *(const __attribute__((address_space(4))) uint64_t *)p;
}

// The chunk of tile t (wave-uniform): the last g with tstart[g] <= t.  A
// 64-way search: at each level the lanes probe 64 evenly spaced entries of
// the candidate range and the count of those <= t (a prefix of the lanes,
// the starts being sorted) picks the sub-range, so the wave waits for
// ceil(log64 G) loads, not log2 G.  Keeps tstart[lo] <= t (tstart[0] = 0).
__device__ __forceinline__ uint64_t chunk_of_tile(const Job &job, uint64_t t)
{
    const uint64_t lane = threadIdx.x & 63;
    uint64_t lo = 0, n = job.G;
    while (n > 1) {
        const uint64_t step = (n + 63) >> 6;
        const uint64_t p = lo + lane * step;
        const bool le = p < lo + n && job.tstart[p] <= t;
        const uint64_t c = (uint64_t)__popcll(__ballot(le));   // >= 1: lane 0 probes lo
        const uint64_t end = lo + n;
        lo += (c - 1) * step;
        n = end - lo < step ? end - lo : step;
    }
    return lo;
}

// Ranges of tiles for a persistent grid: workgroup b takes fixed ranges
// first, then the next one not yet handed out, from the counter status[5]
// (cleared by the scan kernel), so a workgroup whose tiles were cheap takes
// more and none waits on a slow tail.  The counter is one address for all
// dies: a take costs about 17 ns of everybody's time, as much as ten tiles of
// the whole grid, so it is kept for what balancing needs.  Grids with fewer
// than kStaticTiles tiles per workgroup take none (an equal share each; a view
// of 16,640 tiles on 4,096 workgroups, which took four ranges each from the
// counter: whole call 287 -> 119 us); up to 4 x kGrabBig, three
// quarters of the share are fixed and the rest goes in ranges of kGrabSmall
// (n = 3,000,017: 235 us with half of it fixed, 223 with three quarters);
// beyond that the first range has kGrabBig tiles, then ranges of kGrabBig, and
// of kGrabSmall for the last kTailTiles tiles per workgroup, so that the walk
// ends evenly while the counter, the chunk search and the chunk set-up are paid
// once per kGrabBig tiles for most of it.
// A graph's tiles cost about the same, but those of a batch differ several
// times between its graphs, and neighbours are alike: there a fixed share is
// not one piece but every W-th range of kStripeSmall or kStripeBig tiles (batches of
// 73, 16 and 10 uneven graphs 1248 -> 799, 226 -> 181 and 325 -> 341 us).
// The bounds are formed anew at each take (a few scalar instructions) instead
// of being held in scalar registers, which the tile loop has none to spare of.
struct TileGrab {
    uint32_t taken = 0;      // fixed ranges so far

    // the next range [t0, t1) of T tiles; false once every range has been handed out
    __device__ __forceinline__ bool next(const Job &job, uint64_t &t0, uint64_t &t1)
    {
        const uint64_t T = ld_uni(job.status + 2);
        const uint32_t W = gridDim.x, b = blockIdx.x;
        // fixed ranges of `each` tiles, workgroups with one more
        uint32_t each = kGrabBig, more = 0, ranges = 1;
        uint64_t tail = (uint64_t)W * kTailTiles;
        if (T < (uint64_t)W * 4 * kGrabBig) {
            each = (uint32_t)T / W;
            const bool all = each < kStaticTiles;
            if (all) {
                more = (uint32_t)T - each * W;
            } else {
                each -= each / 4;
                tail = T;
            }
            if (job.ninst > 1) {
                const uint32_t sub = all ? kStripeSmall : kStripeBig;
                ranges = each / sub + (all ? 1u : 0u);
                each = sub;
                more = 0;
            }
        }
        uint64_t fixed = ((uint64_t)each * W + more) * ranges;
        if (taken < ranges) {
            t0 = (uint64_t)each * (taken * W + b) + (b < more ? b : more);
            t1 = t0 + each + (b < more ? 1 : 0);
            t1 = t1 < T ? t1 : T;
            ++taken;
            return t0 < t1;
        }
        if (fixed >= T) return false;
        const uint64_t rest = T - fixed;
        const uint64_t head = rest > tail ? rest - tail : 0;    // tiles in large ranges
        const uint64_t qh = (head + kGrabBig - 1) / kGrabBig;
        uint64_t q = 0;
        if (threadIdx.x == 0) q = atomicAdd((unsigned long long *)(job.status + 5), 1ull);
        q = uni64(q);
        if (q < qh) {
            t0 = fixed + q * kGrabBig;
            t1 = t0 + kGrabBig < fixed + head ? t0 + kGrabBig : fixed + head;
            return true;
        }
        t0 = fixed + head + (q - qh) * kGrabSmall;
        t1 = t0 + kGrabSmall < T ? t0 + kGrabSmall : T;
        return t0 < T;
    }
};

// The chunk a wave is in: chunk constants, the stream and the decoder of
// its tiles (enter), the chunk of a tile (locate) and the context of one
// tile (tile).  The tile kernel advances the decoder from tile to tile itself;
// the queue kernel places every tile from scratch.
struct TileWalk {
    uint64_t g, gstart, gend;   // current chunk, its first tile, first tile of the next
    uint64_t N;                 // slots of the chunk
    uint64_t qs;                // 2^s = qs * dv + rs
    uint32_t s;                 // tile exponent
    uint32_t row0;              // first row of the chunk (directed) or its row section
    uint32_t rs;
    TileCtx tc;

    __device__ __forceinline__ void enter(const Job &job, uint64_t gg)
    {
        enter(job, gg, ld_uni(job.tstart + gg), ld_uni(job.tstart + gg + 1));
    }

    __device__ __forceinline__ void enter(const Job &job, uint64_t gg, uint64_t start, uint64_t end)
    {
        g = gg;
        gstart = start;
        gend = end;
        // the fields the sampler needs, through the scalar cache for batches
        Inst I;
        memset(&I, 0, sizeof(I));
        if (job.ninst == 1) {
            I.n = job.one.n; I.seed = job.one.seed; I.chunk_base = job.one.chunk_base;
            I.directed = job.one.directed; I.P = job.one.P; I.s = job.one.s; I.view = job.one.view;
        } else {
            const __attribute__((address_space(4))) Inst *q =
                (const __attribute__((address_space(4))) Inst *)(job.insts + inst_of_chunk(job, g));
            I.n = q->n; I.seed = q->seed; I.chunk_base = q->chunk_base;
            I.directed = q->directed; I.P = q->P; I.s = q->s; I.view = q->view;
        }
        const uint32_t c = uni((uint32_t)chunk_ordinal(I, g - I.chunk_base));
        s = uni(I.s);
        const Chunk ch = chunk_geometry(I, c);
        N = uni64(ch.N);
        Decoder &d = tc.dec;
        d.r0 = d.c0 = d.b = 0;
        d.lbase = 0;
        d.wide = 0;
        uint64_t dv;
        if (I.directed) {
            d.type = 0; dv = I.n - 1; row0 = uni((uint32_t)ch.row0);
        } else if (!ch.diag) {
            d.type = 1; dv = ch.w; d.b = uni((uint32_t)ch.b); row0 = uni((uint32_t)ch.a);
        } else {
            d.type = 2; dv = 1; row0 = uni((uint32_t)ch.a);
            d.r0 = row0; d.b = uni((uint32_t)ch.h);
        }
        if (dv == 0) dv = 1;
        d.type = uni(d.type);
        d.dv = uni((uint32_t)dv);
        d.pow2 = uni((dv & (dv - 1)) == 0);
        d.sh = uni(63 - __clzll(dv));
        d.rcp = unid(1.0 / (double)dv);
        {
            // with m = floor(2^(32 + sh) / dv) and e the remainder, y / dv below
            // 2^32 is the high part of m y + m shifted by sh where e <= 2^sh, and
            // of (m + 1) y elsewhere (dv - e < 2^sh): Robison, "N-bit unsigned
            // division via N-bit multiply-add" (2005)
            uint64_t m = (uint64_t)ldexp(d.rcp, (int)(32 + d.sh));
            int64_t e = (int64_t)((1ull << (32 + d.sh)) - m * dv);
            if (e < 0) { --m; e += (int64_t)dv; }
            else if (e >= (int64_t)dv) { ++m; e -= (int64_t)dv; }
            const bool down = e <= (int64_t)(1ull << d.sh);
            d.mul = uni((uint32_t)(down ? m : m + 1));
            d.add = uni((uint32_t)(down ? m : 0));
        }
        qs = uni64(div_est(1ull << s, dv, d.rcp));
        rs = uni((uint32_t)((1ull << s) - qs * dv));
        tc.st = Stream{uni((uint32_t)I.seed), uni((uint32_t)(I.seed >> 32)), c, 0, TAG_TLEAF};
    }

    // the chunk of tile t, entered
    __device__ __forceinline__ void locate(const Job &job, uint64_t t) { enter(job, chunk_of_tile(job, t)); }

    // stream counter and decoder at tile t of the current chunk, from which
    // tiles advance by 2^s slots; returns the slots of the chunk's last tile
    // (0: 2^32)
    __device__ __forceinline__ uint32_t place(uint64_t t)
    {
        Decoder &d = tc.dec;
        tc.st.b = uni((uint32_t)(t - gstart));
        d.lbase = (t - gstart) << s;
        if (d.type != 2) {
            const uint64_t q = div_est(d.lbase, d.dv, d.rcp);
            d.c0 = uni((uint32_t)(d.lbase - q * d.dv));
            d.r0 = uni(row0 + (uint32_t)q);
        }
        return (uint32_t)(N - ((gend - 1 - gstart) << s));
    }

    // slot count, stream counter and decoding constants of tile t (of the
    // current chunk)
    __device__ __forceinline__ void tile(uint64_t t)
    {
        Decoder &d = tc.dec;
        const uint64_t tl = t - gstart;
        const uint64_t lstart = tl << s;
        if (d.type == 2) {
            d.lbase = lstart;
        } else {
            const uint64_t q = div_est(lstart, d.dv, d.rcp);
            d.c0 = uni((uint32_t)(lstart - q * d.dv));
            d.r0 = uni(row0 + (uint32_t)q);
        }
        d.lbase = uni64(d.lbase);
        tc.S = uni64((N - lstart) < (1ull << s) ? (N - lstart) : (1ull << s));
        tc.bits = uni(tc.S <= 1 ? 0 : 64 - __clzll(tc.S - 1));
        tc.mask = uni(tc.bits >= 32 ? 0xFFFFFFFFu : ((1u << tc.bits) - 1));
        tc.full = uni(tc.S == (1ull << tc.bits));
        tc.st.b = uni((uint32_t)tl);
        d.wide = uni((uint64_t)d.c0 + tc.S > (1ull << 32));
    }
};

// Lane-to-lane moves of the sort (wave-wide DPP shifts by one lane); the
// lane without a source keeps `edge`.
__device__ __forceinline__ uint32_t from_next_lane(uint32_t x, uint32_t edge)
{
    return __builtin_amdgcn_update_dpp(edge, x, 0x130, 0xF, 0xF, false);   // wave_shl:1, lane 63 keeps edge
}
__device__ __forceinline__ uint32_t from_prev_lane(uint32_t x, uint32_t edge)
{
    return __builtin_amdgcn_update_dpp(edge, x, 0x138, 0xF, 0xF, false);   // wave_shr:1, lane 0 keeps edge
}

template <int W>
__device__ __forceinline__ void wload(const uint32_t *s, uint32_t p0, uint32_t *v)
{
#pragma unroll
    for (int i = 0; i < W; ++i) v[i] = s[p0 + i];
}
template <int W>
__device__ __forceinline__ void wstore(uint32_t *s, uint32_t p0, const uint32_t *v)
{
#pragma unroll
    for (int i = 0; i < W; ++i) s[p0 + i] = v[i];
}

// The lane index as a fresh register value: addresses derived from it are
// formed where they are used instead of being kept (and spilled) across the
// whole tile loop.
__device__ __forceinline__ uint32_t lane_here()
{
    uint32_t r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(threadIdx.x));
    return r;
}

__device__ __forceinline__ void cx(uint32_t &a, uint32_t &b)
{
    const uint32_t x = a, y = b;
    a = x < y ? x : y;
    b = x < y ? y : x;
}

// Sort of s[0, 64 W) (W even) after the bucket placement: the keys are in
// bucket order (bucket = top bits), arbitrary inside a bucket, and no bucket
// holds more than R keys.  Lane L holds positions [W L, W L + W) in
// registers and the wave runs R rounds of odd-even transposition sort:
// even rounds compare-exchange the pairs (2j, 2j + 1), all inside a lane;
// odd rounds the pairs (2j + 1, 2j + 2), the pair across two lanes by DPP
// (each lane computes its own side from the old values).  A pair of keys
// from two buckets is already in order and never exchanged, so every bucket
// is sorted on its own, as a sequence of at most R elements, which R rounds
// of odd-even transposition sort (Knuth, TAOCP vol. 3, 5.3.4) always sort.
// Returns whether two adjacent positions are equal (repeats; count_repeats
// counts them); with PADS, other than `pads` pairs of equal padding.
template <int W, bool PADS>
__device__ __forceinline__ bool oddeven(uint32_t *s, uint32_t R, uint32_t pads)
{
    const uint32_t lane = lane_here();
    const uint32_t p0 = W * lane;
    uint32_t v[W];
    wload<W>(s, p0, v);
    // rounds in pairs (an extra round leaves a sorted sequence sorted)
    for (uint32_t r = 0; r < R; r += 2) {
#pragma unroll
        for (int i = 0; i < W; i += 2) cx(v[i], v[i + 1]);
        const uint32_t nx = from_next_lane(v[0], kNone);     // lane 63: the padding bound
        const uint32_t pv = from_prev_lane(v[W - 1], 0u);    // lane 0: no predecessor
#pragma unroll
        for (int i = 1; i + 1 < W; i += 2) cx(v[i], v[i + 1]);
        v[W - 1] = v[W - 1] < nx ? v[W - 1] : nx;
        v[0] = v[0] > pv ? v[0] : pv;
    }
    wstore<W>(s, p0, v);
    const uint32_t nx = from_next_lane(v[0], ~v[W - 1]);       // lane 63: a value unequal to its last key
    if (PADS) {
        uint32_t n = (uint32_t)__popcll(__ballot(v[W - 1] == nx));
#pragma unroll
        for (int i = 0; i + 1 < W; ++i) n += (uint32_t)__popcll(__ballot(v[i] == v[i + 1]));
        return n != pads;
    }
    uint64_t eq = __ballot(v[W - 1] == nx);
#pragma unroll
    for (int i = 0; i + 1 < W; ++i) eq |= __ballot(v[i] == v[i + 1]);
    return eq != 0;
}

// The number of repeats in the sorted keys s[0..V); `dup` is the place of the
// last one.
__device__ __forceinline__ uint32_t count_repeats(const uint32_t *s, uint32_t V, uint32_t &dup)
{
    const uint32_t lane = lane_here();
    uint32_t n = 0;
    for (uint32_t b = 0; b < V; b += 64) {
        const uint32_t p = b + lane;
        const uint64_t m = __ballot(p > 0 && p < V && s[p] == s[p - 1]);
        if (m) dup = b + 63 - (uint32_t)__builtin_clzll(m);
        n += (uint32_t)__popcll(m);
    }
    return n;
}

// Maximum over the 64 lanes (DPP row shifts, then row broadcasts; lane 63
// ends with the maximum).
__device__ __forceinline__ uint32_t wave_max32(uint32_t v)
{
    uint32_t t;
    t = __builtin_amdgcn_update_dpp(0u, v, 0x111, 0xF, 0xF, false); v = v > t ? v : t;   // row_shr:1
    t = __builtin_amdgcn_update_dpp(0u, v, 0x112, 0xF, 0xF, false); v = v > t ? v : t;   // row_shr:2
    t = __builtin_amdgcn_update_dpp(0u, v, 0x114, 0xF, 0xF, false); v = v > t ? v : t;   // row_shr:4
    t = __builtin_amdgcn_update_dpp(0u, v, 0x118, 0xF, 0xF, false); v = v > t ? v : t;   // row_shr:8
    t = __builtin_amdgcn_update_dpp(0u, v, 0x142, 0xA, 0xF, false); v = v > t ? v : t;   // row_bcast:15
    t = __builtin_amdgcn_update_dpp(0u, v, 0x143, 0xC, 0xF, false); v = v > t ? v : t;   // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// Base case of the common tiles.  Pass 1 (one Philox block per lane and
// round; lane L computes blocks L + 64 e, i.e. draws 256 e + 4 L + q) counts
// every valid draw in its bucket -- the top min(9, bits) bits of the key,
// 512 32-bit counters -- and keeps the draws in registers (rejected ones as
// ~0), together with its rank among the draws of its bucket (the value
// the LDS atomic returned).  An exclusive scan turns the counters into bucket
// starts; pass 2 places each draw at its bucket start plus its rank; as
// many rounds of odd-even transposition as the fullest bucket has keys (8 to
// 14 keys per lane) then sort inside buckets, and repeats are counted.
// The set is that of the first J draws with J the least count giving ke
// distinct valid values.  J starts at ke, or, where rejections or repeats are
// expected (a chunk's partial last tile, a dense tile), three standard
// deviations below the expected count; while more than kMissing values are
// missing the pass is repeated with a larger J, again by a low estimate (a
// guess that turns out too large falls back to steps that cannot be), and
// the last kMissing are drawn one by one and inserted (add_missing).  Leaves
// the sorted set in s[0..ke) and returns true, or returns false once J would
// exceed lim (or in the rare cases the queue kernel handles); the counters
// are zero again whenever it returns.
// Jobs with tiles of 2^32 slots (s = 32, fewer than 1120 keys on average) have
// copies of their own (SPARSE).  Keys of 32 bits leave no values for a padding
// without repeats, and to look all keys through for repeats on that account made
// these tiles slower than a form without insertions; the copies count the equal
// pairs.  Up to kSparseDraws - 16 keys (room for repeats) a copy of three rounds
// also saves the steps over the other two.  n = 2^28, 2^23 tiles of 32, 300, 500 and
// 1000 keys: 7.0, 9.9, 11.4 and 17.7 ms without the copies, 6.2, 8.3, 9.3 and 15.1 with.
constexpr uint32_t kBucketWords = 512;   // one 32-bit counter per bucket
constexpr uint32_t kMaxRounds = 32;      // a fuller bucket sends the tile to the queue
constexpr int kSparseRounds = 3;
constexpr uint32_t kSparseDraws = 256 * kSparseRounds;
constexpr uint32_t kMissing = 6;         // values inserted one by one (a pass costs about as much as six)

// Draws J, J + 1, ... of the tile one by one until the sorted keys s[0..V)
// hold ke distinct values: a new value takes the place of a repeat (`dup`: the
// later position of one, if V exceeds the D distinct values), or the array
// grows by one.  An insertion moves the keys between the two places by one
// position.  Without it every tile with a repeat (12 % of the tiles at
// 1024 keys of 2^22 slots) drew, placed and sorted all its keys a second time.
// Returns the new V; kNone for a key equal to the padding value.
__device__ __forceinline__ uint32_t add_missing(const TileCtx &t, uint32_t *s, uint32_t J, uint32_t V, uint32_t D,
                                                uint32_t ke, uint32_t dup)
{
    const uint32_t lane = lane_here();
    uint32_t base = J >> 2;
    U4 w = t.st.block_uniform_key(base + lane);
    bool known = true;                  // dup is the place of a repeat
    while (D < ke) {
        const uint32_t l = (J >> 2) - base;
        if (l >= 64) {
            base += 64;
            w = t.st.block_uniform_key(base + lane);
            continue;
        }
        const uint32_t q = J & 3;
        const uint32_t wq = q == 0 ? w.x : q == 1 ? w.y : q == 2 ? w.z : w.w;
        const uint32_t x = __builtin_amdgcn_readlane(wq, l) & t.mask;
        ++J;
        if (!t.full && x >= (uint32_t)t.S) continue;
        if (x == kNone) return kNone;
        // r: the keys below x, by two probes of 64 lanes
        const uint32_t st = (V + 63) >> 6;
        uint32_t p = lane * st;
        uint32_t r = (uint32_t)__popcll(__ballot(p < V && s[p] < x));
        if (r) {
            const uint32_t lo = (r - 1) * st;
            p = lo + lane;
            r = lo + (uint32_t)__popcll(__ballot(lane < st && p < V && s[p] < x));
        }
        if (r < V && uni(s[r]) == x) continue;
        uint32_t a = V;                 // the place that the new key's neighbours move into
        if (V > D) {
            if (!known) (void)count_repeats(s, V, dup);
            known = false;
            a = dup;
        } else {
            ++V;
        }
        if (a < r) {
            for (uint32_t b = a; b + 1 < r; b += 64) {
                p = b + lane;
                const bool in = p + 1 < r;
                const uint32_t y = in ? s[p + 1] : 0;
                __syncthreads();
                if (in) s[p] = y;
            }
            __syncthreads();
            if (lane == 0) s[r - 1] = x;
        } else {
            for (uint32_t b = 0; r + b < a; b += 64) {
                const bool in = r + b + lane < a;
                p = a - b - lane;
                const uint32_t y = in ? s[p - 1] : 0;
                __syncthreads();
                if (in) s[p] = y;
            }
            __syncthreads();
            if (lane == 0) s[r] = x;
        }
        __syncthreads();
        ++D;
    }
    return V;
}

// Draws to add, at least, when e values are missing and a draw is a new one
// with probability f: three standard deviations below the mean e / f.
__device__ __forceinline__ uint32_t draws_for(float e, float f)
{
    const float g = __builtin_amdgcn_rcpf(f);
    const float x = e * g - 3.0f * __builtin_amdgcn_sqrtf(e * (1.0f - f)) * g - 1.0f;
    return (uint32_t)fmaxf(e, x);
}

template <int ROUNDS, bool SPARSE>
__device__ __forceinline__ bool fast_set(const TileCtx &t, uint32_t *s, uint32_t *cnt, uint32_t ke, uint32_t lim)
{
    const uint32_t lane = threadIdx.x;
    const uint32_t S32 = (uint32_t)t.S;                 // used only when S < 2^bits <= 2^32
    const uint32_t shift = t.bits > 9 ? t.bits - 9 : 0;
    uint4 *cw = reinterpret_cast<uint4 *>(cnt) + 2 * lane;   // this lane's 8 counter words
    uint32_t J = ke;             // draws of this pass
    uint32_t sure = ke;          // draws that are needed for certain
    const bool sparse = t.full && (uint64_t)ke * ke <= 8 * t.S;    // at most 4 repeats expected
    bool guess = !sparse;
    if (guess) {
        // on average a draw is valid and new with probability (S - ke / 2) / 2^bits
        const float f = ((float)S32 - 0.5f * (float)ke) * __builtin_amdgcn_ldexpf(1.0f, -(int)t.bits);
        const uint32_t g = uni(draws_for((float)ke, f));
        J = g < lim ? g : lim;
        J = J < ke ? ke : J;
    }
    for (;;) {
        if (J > lim) return false;
        // the counters are zero here: cleared at the start of the kernel and
        // after every use (below)
        const uint32_t nit = uni((J + 255) >> 8);
        // rounds whose 256 draws all lie below J: in a full tile with keys
        // below 2^31 every such draw is valid and needs no checks
        const bool nclean_tile = t.full && t.bits < 32;
        const uint32_t nclean = nclean_tile ? uni(J >> 8) : 0u;
        uint64_t coll = 0;      // a valid key equal to ~0 (2^32-slot tiles only)
        bool hit = false;
        // the draws stay in registers (x[4 e + q] = draw 256 e + 4 lane + q)
        uint32_t x[4 * ROUNDS], rk[4 * ROUNDS];
#pragma unroll
        for (int e = 0; e < ROUNDS; ++e) {
#pragma unroll
            for (int q = 0; q < 4; ++q) { x[4 * e + q] = kNone; rk[4 * e + q] = 0; }
            const uint32_t blk = lane + 64u * e;
            if ((uint32_t)e < nclean) {
                const U4 w = t.st.block_uniform_key(blk);     // the tile's key is wave-uniform
                const uint32_t v[4] = {w.x & t.mask, w.y & t.mask, w.z & t.mask, w.w & t.mask};
#pragma unroll
                for (int q = 0; q < 4; ++q) rk[4 * e + q] = atomicAdd(&cnt[v[q] >> shift], 1u);
#pragma unroll
                for (int q = 0; q < 4; ++q) x[4 * e + q] = v[q];
            } else if ((uint32_t)e < nit && 4 * blk < J) {
                // only the lanes whose block holds draws below J compute it
                const U4 w = t.st.block_uniform_key(blk);
                uint32_t v[4] = {w.x & t.mask, w.y & t.mask, w.z & t.mask, w.w & t.mask};
                if (nclean_tile) {
                    // a full tile with keys below 2^31: only draws past J drop out
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const bool ok = 4 * blk + q < J;
                        rk[4 * e + q] = atomicAdd(&cnt[v[q] >> shift], ok ? 1u : 0u);
                        v[q] = ok ? v[q] : kNone;
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        // a draw past J or rejected adds 0 and is kept as ~0
                        const bool ok = (4 * blk + q < J) & (t.full | (v[q] < S32));
                        hit |= ok & (v[q] == kNone);
                        rk[4 * e + q] = atomicAdd(&cnt[v[q] >> shift], ok ? 1u : 0u);
                        v[q] = ok ? v[q] : kNone;
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) x[4 * e + q] = v[q];
            }
        }
        coll = __ballot(hit);
        __syncthreads();
        if (coll) {
            cw[0] = make_uint4(0, 0, 0, 0);
            cw[1] = make_uint4(0, 0, 0, 0);
            return false;
        }
        uint32_t V;             // valid draws
        uint32_t R;             // keys in the fullest bucket
        {
            const uint4 c0 = cw[0], c1 = cw[1];
            uint32_t w[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
            uint32_t sum = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += w[i];
            uint32_t mx = w[0];
#pragma unroll
            for (int i = 1; i < 8; ++i) mx = mx > w[i] ? mx : w[i];
            R = wave_max32(mx);
            const uint32_t incl = wave_incl_scan32(sum);
            uint32_t run = incl - sum;
#pragma unroll
            for (int i = 0; i < 8; ++i) { const uint32_t c = w[i]; w[i] = run; run += c; }
            cw[0] = make_uint4(w[0], w[1], w[2], w[3]);
            cw[1] = make_uint4(w[4], w[5], w[6], w[7]);
            V = __builtin_amdgcn_readlane(incl, 63);
        }
        __syncthreads();
        {
#pragma unroll
            for (int e = 0; e < ROUNDS; ++e) {
                if ((uint32_t)e < nclean) {
                    // every entry of a clean round is a valid key
                    uint32_t old[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) old[q] = cnt[x[4 * e + q] >> shift] + rk[4 * e + q];
#pragma unroll
                    for (int q = 0; q < 4; ++q) s[old[q]] = x[4 * e + q];
                } else if ((uint32_t)e < nit) {
                    uint32_t old[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t xv = x[4 * e + q];
                        const bool ok = xv != kNone;
                        old[q] = cnt[ok ? xv >> shift : 0u] + rk[4 * e + q];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t xv = x[4 * e + q];
                        // a ~0 entry lands in the padding after the V keys, which is
                        // rewritten below or lies past the sorted span (kKeyWords >= V + 4)
                        const uint32_t pos = xv != kNone ? old[q] : V + (lane & 3);
                        s[pos] = xv;
                    }
                }
            }
        }
        // the wave's LDS operations complete in order, so the bucket starts
        // read above are read before they are cleared here
        cw[0] = make_uint4(0, 0, 0, 0);
        cw[1] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        if (R > kMaxRounds) return false;
        uint32_t ndup, dup = 0;
        {
            // keys per lane from V: 4, 8, 12, 16, 18 or 20; [V, 64 W) is padded
            const int mode = V <= 256 ? 0 : V <= 512 ? 1 : V <= 768 ? 2 : V <= 1024 ? 3 : V <= 1152 ? 4 : 5;
            constexpr uint32_t kSpan[6] = {256, 512, 768, 1024, 1152, 1280};
            const uint32_t span = kSpan[mode];
            // ascending above every key, so that no two are equal (in a tile of
            // 2^32 slots they all are ~0: the sparse copy counts the equal pairs
            // among them, the common one the repeats always)
            const uint32_t pads = t.bits < 32 || V == span ? 0u : span - 1 - V;
            for (uint32_t p = V + lane; p < span; p += 64) s[p] = t.bits < 32 ? 0x80000000u | p : kNone;
            __syncthreads();
            bool rep;
            if (mode == 0) rep = oddeven<4, SPARSE>(s, R, pads);
            else if (mode == 1) rep = oddeven<8, SPARSE>(s, R, pads);
            else if (ROUNDS <= 3 || mode == 2) rep = oddeven<12, SPARSE>(s, R, pads);
            else if (mode == 3) rep = oddeven<16, SPARSE>(s, R, pads);
            else if (mode == 4) rep = oddeven<18, SPARSE>(s, R, pads);
            else rep = oddeven<20, SPARSE>(s, R, pads);
            __syncthreads();
            ndup = rep ? count_repeats(s, V, dup) : 0u;
        }
        if (SPARSE && __builtin_expect(V == ke && ndup == 0, 1)) return true;
        const uint32_t D = V - ndup;
        if (D > ke) {
            guess = false;
            J = sure;
            continue;
        }
        if (D + kMissing < ke) {
            const uint32_t e = ke - D;
            sure = J + e;
            J = sure;
            if (guess) {
                const float f = ((float)S32 - (float)D) * __builtin_amdgcn_ldexpf(1.0f, -(int)t.bits);
                J = sure - e + uni(draws_for((float)e, f));
                J = J < lim ? J : sure < lim ? lim : sure;
            }
            continue;
        }
        if (D < ke) {
            V = add_missing(t, s, J, V, D, ke, dup);
            if (V == kNone) return false;
        }
        if (V > ke) {
            // repeats are left: squeeze them out
            uint32_t kept = 0;
            for (uint32_t b0 = 0; b0 < V; b0 += 64) {
                const uint32_t p = b0 + lane;
                uint32_t xv = 0;
                bool keep = false;
                if (p < V) {
                    xv = s[p];
                    keep = p == 0 || s[p - 1] != xv;
                }
                const uint64_t bal = __ballot(keep);
                __syncthreads();
                if (keep) s[kept + __popcll(bal & lanemask_lt(lane))] = xv;
                kept += __popcll(bal);
                __syncthreads();
            }
        }
        return true;
    }
}

// Decoding constants of a tile copied into vector registers: they are read
// by every key of the emission loop, and scalar registers are scarce there.
__device__ __forceinline__ uint32_t vreg(uint32_t x)
{
    uint32_t r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(x));
    return r;
}

struct DecV {
    uint32_t dv, r0, c0, b, sh, msk, mul, add;
};

__device__ __forceinline__ DecV dec_vregs(const Decoder &d)
{
    DecV v;
    v.dv = vreg(d.dv); v.r0 = vreg(d.r0); v.c0 = vreg(d.c0); v.b = vreg(d.b);
    v.sh = vreg(d.sh); v.msk = vreg(d.dv - 1);
    v.mul = vreg(d.mul); v.add = vreg(d.add);
    return v;
}

// Directed (TYPE 0) or rectangle (TYPE 1) slot with a 32-bit dividend:
// quotient by shift or by the reciprocal multiplier (Decoder::mul): one product
// and a shift, exact, instead of two conversions, a binary64 product and a
// correction to both sides, 30 vector instructions and 4 wide products per 256
// edges instead of 66 in all.  Directed n = 2^25, 2^16 chunks 1081 -> 1011 us, a
// batch of 64 instances 1986 -> 1906 us.
template <int TYPE, bool POW2, bool ALIGNED = false>
__device__ __forceinline__ uint2 dec_narrow(const DecV &d, uint32_t x)
{
    if (ALIGNED) {
        // rectangle, width 2^sh, tile starting at a row start, first column a
        // multiple of the width: row offset by shift, column by mask and OR
        return make_uint2(d.r0 + (x >> d.sh), d.b | (x & d.msk));
    }
    const uint32_t y = d.c0 + x;
    uint32_t q, r;
    if (POW2) {
        q = y >> d.sh;
        r = y & d.msk;
    } else {
        q = (uint32_t)(((uint64_t)y * d.mul + d.add) >> 32) >> d.sh;
        r = y - q * d.dv;
    }
    const uint32_t u = d.r0 + q;
    return TYPE == 0 ? make_uint2(u, r + (r >= u ? 1u : 0u)) : make_uint2(u, d.b + r);
}

// Triangle slots (rows of a section counted down by one slot each) relative
// to the tile's first row: slot y of rows of L, L - 1, ... slots lies in row
// r = floor(B - sqrt(B^2 - 2 y)), B = L + 1/2, as r = 2 y / (B + sqrt(...))
// without the cancellation.  y < 2^32 keeps r below 92,682 (rows that all hold
// at least one slot, the r-th from the end r of them), so with the hardware's
// square root and reciprocal (2^29 ulp, 2^-23, each at worst) the estimate is off by
// one at most, and the row's integer bounds correct it.  32-bit products suffice while
// y + L < 2^32 and L < 2^26 (larger tiles and sections: emit_sorted).  About
// 20 vector instructions per slot against 150 for the 64-bit formula:
// undirected n = 4,194,381, m = 67,108,867 in one section 409 -> 252 us, in
// 37 sections with m = 48,000,271 245 -> 235 us.
struct TriV {
    uint32_t L, row, off;    // slots of the tile's first row, that row, its slots before the tile
    double B, BB;
};

__device__ __forceinline__ uint2 dec_tri(const TriV &d, uint32_t x)
{
    const uint32_t y = d.off + x;
    const double yy = 2.0 * (double)y;
    const double D = d.BB - yy;
    const double s = __builtin_amdgcn_sqrt(D > 0.0 ? D : 0.0);
    uint32_t r = (uint32_t)(yy * __builtin_amdgcn_rcp(d.B + s));
    // slots before row r: r L - r (r - 1) / 2 (the even factor halved)
    uint32_t st = r * d.L - (r >> 1) * ((r - 1) | 1);
    if ((int32_t)(y - st) < 0) { --r; st -= d.L - r; }
    else if (y - st >= d.L - r) { st += d.L - r; ++r; }
    const uint32_t u = d.row + r;
    return make_uint2(u, u + 1 + (y - st));
}
// Sorted keys s[0..n) out as edges o0 .. o0 + n - 1, four keys per lane per
// round (lane-strided, so each store instruction covers 512 contiguous bytes).
template <class Dec>
__device__ __forceinline__ void emit_keys(const TileCtx &t, const uint32_t *s, uint32_t n, const Dec &dec)
{
    uint2 *out = reinterpret_cast<uint2 *>(t.edges) + t.o0;
    const uint32_t lane = lane_here();
    const uint32_t nfull = n & ~255u;
    // one 64-bit lane pointer advanced per round; the four stores of a round
    // sit at fixed byte offsets from it (0, 512, 1024, 1536)
    uint2 *ol = out + lane;
    for (uint32_t b = 0; b < nfull; b += 256, ol += 256) {
        uint32_t x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = s[b + lane + 64 * i];
#pragma unroll
        for (int i = 0; i < 4; ++i) ol[64 * i] = dec(x[i]);
    }
    if (nfull < n) {
        uint32_t x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t p = nfull + lane + 64 * i;
            x[i] = p < n ? s[p] : 0;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t p = nfull + lane + 64 * i;
            if (p < n) out[p] = dec(x[i]);
        }
    }
}

template <int TYPE, bool POW2, bool ALIGNED = false>
__device__ __forceinline__ void emit_narrow(const TileCtx &t, const uint32_t *s, uint32_t n)
{
    const DecV d = dec_vregs(t.dec);
    emit_keys(t, s, n, [&](uint32_t x) { return dec_narrow<TYPE, POW2, ALIGNED>(d, x); });
}

__device__ __forceinline__ void emit_tile(const TileCtx &t, const uint32_t *s, uint32_t n)
{
    const Decoder &d = t.dec;
    if (d.type == 2) {
        // the tile's first slot by the general formula, once per tile
        const uint2 e = d(0);
        TriV v;
        v.row = uni(e.x);
        v.off = uni(e.y - e.x - 1);
        v.L = d.r0 + d.b - 1 - v.row;
        if (v.L < (1u << 26) && (uint64_t)v.off + t.S + v.L < (1ull << 32)) {
            v.B = (double)v.L + 0.5;
            v.BB = v.B * v.B;
            emit_keys(t, s, n, [&](uint32_t x) { return dec_tri(v, x); });
            return;
        }
    }
    if (d.type == 2 || d.wide) emit_sorted(t, s, n);
    else if (d.type == 0) {
        if (d.pow2) emit_narrow<0, true>(t, s, n); else emit_narrow<0, false>(t, s, n);
    } else {
        if (d.pow2 && d.c0 == 0 && (d.b & (d.dv - 1)) == 0) emit_narrow<1, true, true>(t, s, n);
        else if (d.pow2) emit_narrow<1, true>(t, s, n);
        else emit_narrow<1, false>(t, s, n);
    }
}

// Slots of the tile whose stream and decoder the context holds, and its edges:
// `last_S` slots if it is the chunk's `last` tile (0: 2^32), else 2^s.  SPARSE: with
// the copy of the base case for s = 32 (few tiles of a wave each do without).
template <bool SPARSE>
__device__ __forceinline__ bool sample_tile(TileCtx &tc, uint32_t *s_key, uint32_t *s_cnt, uint64_t o0, uint64_t k,
                                            uint32_t s, bool last, uint32_t last_S, uint32_t fast_cap)
{
    Decoder &d = tc.dec;
    tc.S = 1ull << s;
    tc.bits = s;
    tc.full = 1;
    if (last && last_S != (uint32_t)tc.S) {
        tc.S = last_S;
        tc.bits = uni(last_S <= 1 ? 0 : 32 - __clz(last_S - 1));
        tc.full = uni(tc.S == (1ull << tc.bits));
    }
    tc.mask = (uint32_t)((1ull << tc.bits) - 1);
    d.wide = uni((uint64_t)d.c0 + tc.S > (1ull << 32));      // rows of more than 2^32 - 2^s slots
    tc.o0 = o0;
    const uint32_t lim = fast_cap < kFastDraws ? fast_cap : kFastDraws;
    const bool comp = 2 * k > tc.S;
    const uint64_t ke = comp ? tc.S - k : k;
    if (ke == 0) {
        emit_complement(tc, s_key, 0, 0, tc.S, 0);
    } else if (ke <= lim &&
               ((SPARSE && s == 32 && ke <= kSparseDraws - 16 &&
                 fast_set<kSparseRounds, true>(tc, s_key, s_cnt, (uint32_t)ke, lim < kSparseDraws ? lim : kSparseDraws)) ||
                fast_set<(int)kFastRounds, SPARSE>(tc, s_key, s_cnt, (uint32_t)ke, lim))) {
        // (a triangle's tiles of 2^32 slots are too large for dec_tri)
        if (!comp && SPARSE && d.type == 2 && s == 32) emit_sorted(tc, s_key, (uint32_t)ke);
        else if (!comp) emit_tile(tc, s_key, (uint32_t)ke);
        else emit_complement(tc, s_key, (uint32_t)ke, 0, tc.S, 0);
    } else {
        return false;
    }
    return true;
}

__device__ __forceinline__ void clear_counters(uint32_t *s_cnt)
{
    uint4 *cw = reinterpret_cast<uint4 *>(s_cnt) + 2 * threadIdx.x;
    cw[0] = make_uint4(0, 0, 0, 0);
    cw[1] = make_uint4(0, 0, 0, 0);
    __syncthreads();
}

// A workgroup's ranges of tiles.
template <bool SPARSE>
__device__ __forceinline__ void sample_ranges(const Job &job, uint32_t *s_key, uint32_t *s_cnt)
{
    if (ld_uni(job.status + 1)) return;
    clear_counters(s_cnt);
    TileWalk w;
    TileCtx &tc = w.tc;
    Decoder &d = tc.dec;
    tc.edges = job.edges;
    TileGrab grab;
    uint64_t t, t1;
    while (grab.next(job, t, t1)) {
        uint64_t g = chunk_of_tile(job, t);
        // tile offsets are read two tiles ahead: they come from HBM (the output
        // stream evicts them from the caches), so a tile never waits for its own
        // (the read after the last offset lands in the queue behind them, unused)
        uint64_t o_next = ld_uni(job.tile_off + t);
        uint64_t o_pre = ld_uni(job.tile_off + t + 1);
        for (;;) {
            // chunk constants, then the decoder at the wave's first tile of the chunk
            w.enter(job, g);
            const uint32_t s = w.s;
            // tiles of the range in this chunk; after `full` of them comes the
            // chunk's last tile
            const uint64_t tend = w.gend < t1 ? w.gend : t1;
            const uint32_t count = (uint32_t)(tend - t), full = (uint32_t)(w.gend - 1 - t);
            const uint32_t last_S = w.place(t);
            const uint32_t qs32 = (uint32_t)w.qs;
            for (uint32_t i = 0; i < count; ++i) {
                const uint64_t o0 = o_next;
                o_next = o_pre;
                o_pre = ld_uni(job.tile_off + t + i + 2);
                const uint64_t k = o_next - o0;
                if (k != 0) {
                    if (!sample_tile<SPARSE>(tc, s_key, s_cnt, o0, k, s, i == full, last_S, job.fast_cap) &&
                        threadIdx.x == 0) {
                        const uint64_t q = atomicAdd((unsigned long long *)(job.status + 4), 1ull);
                        job.queue[q] = t + i;
                    }
                    __syncthreads();
                }
                // next tile of the chunk: 2^s = qs dv + rs slots further
                ++tc.st.b;
                d.lbase += 1ull << s;
                if (d.type != 2) {
                    const uint32_t room = d.dv - w.rs;      // c0 + rs may pass 2^32
                    uint32_t c0 = d.c0 + w.rs, r0 = d.r0 + qs32;
                    if (d.c0 >= room) { c0 = d.c0 - room; ++r0; }
                    d.c0 = c0;
                    d.r0 = r0;
                }
            }
            t = tend;
            if (t >= t1) break;
            // next chunk that has tiles
            ++g;
            while (ld_uni(job.tstart + g + 1) <= t) ++g;
        }
    }
}

// 4 waves per SIMD (up to 128 VGPRs, no spills); the LDS of a wave (keys of
// up to 1280 draws and 512 bucket counters, 7.2 KB) would allow 5
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void tile_kernel(Job job)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_key[kKeyWords];
    __shared__ __attribute__((aligned(16))) uint32_t s_cnt[kBucketWords];   // bucket counters, then starts
    sample_ranges<false>(job, s_key, s_cnt);
}

// The same for jobs with tiles of 2^32 slots: a kernel of its own, since the second
// copy of the base case costs the others' tiles about 1 %.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void tile_sparse_kernel(Job job)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_key[kKeyWords];
    __shared__ __attribute__((aligned(16))) uint32_t s_cnt[kBucketWords];
    sample_ranges<true>(job, s_key, s_cnt);
}

// The sampler of small jobs (at most a tile per workgroup): the wave walks
// the tile tree's path to its tile itself, 64 proposals of each variate at
// once, and takes the general base case where the register one does not do,
// so the job needs neither the planner's nor the queue's launch.  Where the
// chunk tree's left counts are the chunks' offsets (directed G(n,m)), the wave
// walks that path first and the count kernel's launch is not needed either
// (job.whole): the chain of variates is the same, but not cut by a launch.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8))) void tile_one_kernel(Job job)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_key[kKeyWords];
    __shared__ __attribute__((aligned(16))) uint32_t s_cnt[kBucketWords];
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kCapMax + 8];
    const uint64_t t = blockIdx.x;
    uint64_t g, gs, ge, o0 = 0, k = job.one.m;
    if (job.whole) {
        // a lane per chunk: the chunk of tile t by the chunks' tiles
        const Sections at(job.one);
        gs = ge = 0;
        for (g = 0;; g += 64) {
            if (g >= job.G) return;
            const uint64_t c = g + threadIdx.x;
            const uint64_t T = c < job.G ? tiles_of((at(c + 1) - at(c)) * (job.one.n - 1), job.one.s) : 0;
            const uint64_t incl = ge + wave_incl_scan64(T);
            const uint64_t past = __ballot(incl > t);
            if (past) {
                const int l = __builtin_ctzll(past);
                g += l;
                ge = __shfl(incl, l, 64);
                gs = ge - __shfl(T, l, 64);
                break;
            }
            ge = __shfl(incl, 63, 64);
        }
        g = uni64(g); gs = uni64(gs); ge = uni64(ge);
    } else {
        if (ld_uni(job.status + 1) || t >= ld_uni(job.status + 2)) return;
        g = chunk_of_tile(job, t);
        gs = ld_uni(job.tstart + g);
        ge = ld_uni(job.tstart + g + 1);
        o0 = ld_uni(job.off + g);
        k = ld_uni(job.off + g + 1) - o0;
    }
    clear_counters(s_cnt);
    TileWalk w;
    TileCtx &tc = w.tc;
    tc.edges = job.edges;
    w.enter(job, g, gs, ge);
    const uint32_t last_S = w.place(t);
    // two trees in one loop (the variate's code appears once): the chunks'
    // rows [lo, hi) where they are not known yet, then the chunk's tiles
    bool rows = job.whole != 0;
    const Sections at(job.one);
    uint32_t at_me = rows ? (uint32_t)g : tc.st.b;
    uint32_t lo = 0, hi = rows ? (uint32_t)job.G : (uint32_t)(ge - gs), heap = 1;
    uint64_t A = 0, B = job.one.n;
    for (;;) {
        if (hi - lo <= 1) {
            if (!rows) break;
            rows = false;
            at_me = tc.st.b;
            lo = 0;
            hi = (uint32_t)(ge - gs);
            heap = 1;
            continue;
        }
        const uint32_t mid = lo + (hi - lo + 1) / 2;
        uint64_t all, left, M = 0;
        if (rows) {
            M = at(mid);
            all = (B - A) * (job.one.n - 1);
            left = (M - A) * (job.one.n - 1);
        } else {
            all = tile_range_slots(lo, hi, w.s, w.N);
            left = tile_range_slots(lo, mid, w.s, w.N);
        }
        const Stream st{tc.st.k0, tc.st.k1, rows ? heap : tc.st.a, rows ? 0 : heap, rows ? TAG_DTREE : TAG_TTREE};
        const uint64_t X = uni64(hyp<64>(st, all, left, k));
        if (at_me < mid) { hi = mid; B = M; k = X; heap = 2 * heap; }
        else { lo = mid; A = M; o0 += X; k -= X; heap = 2 * heap + 1; }
    }
    if (k == 0) return;
    if (!sample_tile<false>(tc, s_key, s_cnt, o0, k, w.s, t + 1 == ge, last_S, job.fast_cap)) {
        __syncthreads();
        leaf_sample<kCapMax>(tc, s_key, s_hist, k, job.leaf_cap < kCapMax ? job.leaf_cap : kCapMax);
    }
}

// Tiles the fast kernel queued: one wave per queued tile, general base case.
template <int CAP>
__global__ __launch_bounds__(64) void queue_kernel(Job job)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_bkt[CAP + 8];
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[CAP + 8];
    if (ld_uni(job.status + 1)) return;
    const uint64_t nq = ld_uni(job.status + 4);
    const uint32_t cap = job.leaf_cap < CAP ? job.leaf_cap : CAP;
    for (uint64_t i = blockIdx.x; i < nq; i += gridDim.x) {
        const uint64_t t = ld_uni(job.queue + i);
        const uint64_t o0 = ld_uni(job.tile_off + t);
        const uint64_t k = ld_uni(job.tile_off + t + 1) - o0;
        TileWalk w;
        w.locate(job, t);
        w.tile(t);
        TileCtx &tc = w.tc;
        tc.o0 = o0;
        tc.edges = job.edges;
        leaf_sample<CAP>(tc, s_bkt, s_hist, k, cap);
        __syncthreads();
    }
}

}  // namespace kg
