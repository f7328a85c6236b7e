// kg_skip.hpp -- the geometric-skip G(n,p) variant: a second sampler for the
// law of Sec. 2.1.1 / 4.3 (every slot an independent Bernoulli(p) trial)
// with its own bits.  Each tile of each chunk (the 2^s-slot tiles of the
// main path) runs its trials by waiting times: the number of failures before
// the next success is floor(log U / log(1 - p)), one 64-bit draw of the
// tile's stream (seed, chunk ordinal, tile, TAG_SKIP) per gap; for p > 1/2
// the waiting times are those of the failures and the other slots are the
// successes.  Count pass -> scan of the tile counts -> write pass.  When
// the workspace holds a row of positions per tile, the count pass keeps the
// events' positions and the write pass only decodes them (skip_gen_kernel,
// skip_emit_kernel); otherwise the write pass generates the same trials again
// (skip_write_kernel), which costs no more (directed n = 2^25, 536 million
// edges: 2.65 ms a call, with the rows 2.73) and reads and writes no rows; there
// many tiles of few events are counted by a lane each (skip_count_kernel).  The
// chunk and tile layout comes from the main path's count and offset kernels.
#pragma once
#include "kg_tile.hpp"

namespace kg {

constexpr uint32_t TAG_SKIP = 7;

// Scan of the wave sums (one workgroup of 1024 lanes, rounds of 1024); the
// total edges and the overflow flag.
__global__ __launch_bounds__(1024) void skip_scan_kernel(Job job, uint64_t nwaves)
{
    __shared__ uint64_t s_w[16];
    const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint64_t carry = 0;
    for (uint64_t base = 0; base < nwaves; base += 1024) {
        const uint64_t i = base + t;
        const uint64_t v = i < nwaves ? job.queue[i] : 0;
        const uint64_t incl = wave_incl_scan64(v);
        if (lane == 63) s_w[wv] = incl;
        __syncthreads();
        uint64_t before = carry, total = 0;
        for (int w = 0; w < 16; ++w) {
            const uint64_t x = s_w[w];
            if ((uint32_t)w < wv) before += x;
            total += x;
        }
        if (i < nwaves) job.queue[i] = before + incl - v;
        carry += total;
        __syncthreads();
    }
    if (t == 0) {
        job.status[0] = carry;
        job.status[1] = carry > job.capacity ? 1 : 0;
        job.status[5] = 0;
        if (job.out_total) *job.out_total = carry;
    }
}

// The scanned counts as tile offsets: tile_off[t] = the wave's prefix plus
// the in-wave prefix of the counts, tile_off[T] = the total (the layout the
// write pass walks, as the main path's sampler does).
__global__ __launch_bounds__(64) void skip_fix_kernel(Job job)
{
    const uint64_t t = (uint64_t)blockIdx.x * 64 + threadIdx.x;
    const uint64_t T = job.status[2];
    const uint64_t k = t < T ? job.tile_off[t] : 0;
    const uint64_t ex = wave_incl_scan64(k) - k;
    if (t < T) job.tile_off[t] = job.queue[blockIdx.x] + ex;
    else if (t == T) job.tile_off[T] = job.status[0];
}

// Write pass: a persistent grid walks ranges of tiles chunk by chunk, each
// workgroup taking the next range from the shared counter (as the main
// sampler does, with its decoders).  The waiting times of a tile are
// independent draws, so the positions of its events (successes, or
// failures when p > 1/2) are prefix sums: x_d = x_{d-1} + 1 + g_d.  A round
// takes 128 draws (lane L: block 64 r + L, draws 128 r + 2 L and + 1), forms
// the gaps, scans them across the wave and appends the events below S to
// LDS; full batches and the tile's last one are decoded and stored with
// consecutive lanes on consecutive edges (the main sampler's emission).
constexpr uint32_t kSkipKeys = 1408;   // LDS batch (11 rounds of 128 events)

// One round of a tile's waiting times: the positions x0, x1 of lane L's two
// events (tile-local, counted from `pos`), whether they fall below S, how
// many of the round's 128 events do (they are a prefix in lane order), and
// the wave's inclusive sum of the advances for the next round's `pos`.
// `next` holds only where all 128 do.
struct SkipRound {
    uint64_t x0, x1, next;
    bool v0, v1;
    uint32_t nv;
};

// Inclusive sum over the wave's lanes that stays at 2^32 - 1 once it reaches it.
__device__ __forceinline__ uint32_t wave_incl_scan_sat(uint32_t v)
{
    v = __builtin_elementwise_add_sat(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false));
    v = __builtin_elementwise_add_sat(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false));
    v = __builtin_elementwise_add_sat(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false));
    v = __builtin_elementwise_add_sat(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false));
    v = __builtin_elementwise_add_sat(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));
    v = __builtin_elementwise_add_sat(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));
    return v;
}

// The gap floor(log U / L), log U / L rounded as the project's binary64
// routines round it.  Quick form (a table in LDS): log U = E ln 2 + log m with
// m = c (1 + r), |r| < 2^-9, four terms of log(1 + r): off by less than 2^-46,
// so the quotient is off by less than 2^-45 / |L| plus 2^-50 of itself (the
// roundings on both sides).  Where a whole number is nearer than `open`
// (2^-44 / |L| + 2^-49 S; about one gap in 10^5), the full form decides.
// 18 binary64 operations and a 16-byte LDS read instead of about 60.  The gap
// pass is bound by vector instructions; with this form, the sums below and
// one 8-byte store a pair, directed n = 2^25, 536 million edges: 2204 ->
// 1280 us (0.42 million gaps a microsecond), the call 3570 -> 2700 us.
struct GapLaw {
    double L, iL, open;
    const double2 *tab;      // LDS copy of g_gap_tab, or null (full form only)

    __device__ __forceinline__ double operator()(double U) const
    {
        if (tab) {
            const double2 c = tab[(uint32_t)((uint64_t)__double_as_longlong(U) >> 44) & (kGapTab - 1)];
            const double r = __builtin_fma(__builtin_amdgcn_frexp_mant(U), c.x, -1.0);
            double q = __builtin_fma(r, -0.25, 1.0 / 3.0);
            q = __builtin_fma(r, q, -0.5);
            q = __builtin_fma(r * r, q, r);
            const double e = (__builtin_fma((double)__builtin_amdgcn_frexp_exp(U), 0x1.62e42fefa39efp-1, c.y) + q) * iL;
            const double f = floor(e);
            if (__builtin_expect(fabs((e - f) - 0.5) < 0.5 - open, 1)) return f;
        }
        return floor(log_f64(U) / L);
    }
};

__device__ __forceinline__ GapLaw gap_law(double L, uint32_t s, const double2 *tab)
{
    return GapLaw{L, 1.0 / L, 0x1p-44 / fabs(L) + (double)(1ull << s) * 0x1p-49, tab};
}

// The quick logarithm's table into LDS (one wave).
__device__ __forceinline__ void load_gap_tab(double2 *tab)
{
    for (uint32_t i = threadIdx.x; i < kGapTab; i += 64) tab[i] = g_gap_tab[i];
    __syncthreads();
}

__device__ __forceinline__ SkipRound skip_round(const TileCtx &tc, uint32_t r, uint64_t pos, const GapLaw &gap)
{
    const uint32_t lane = threadIdx.x;
    const uint64_t S = tc.S;
    const U4 q = tc.st.block_uniform_key(64 * r + lane);
    const double g0 = gap(unit_of(((uint64_t)q.y << 32) | q.x)), g1 = gap(unit_of(((uint64_t)q.w << 32) | q.z));
    // a gap of S or more ends the tile wherever it starts
    const double cap = (double)S;
    const double c0 = g0 < cap ? g0 : cap, c1 = g1 < cap ? g1 : cap;
    SkipRound o;
    if (S <= (1ull << 31)) {
        // 32-bit sums that stay at 2^32 - 1 once they reach it (past any S)
        const uint32_t a0 = (uint32_t)c0 + 1, a1 = (uint32_t)c1 + 1, at = (uint32_t)pos;
        const uint32_t incl = wave_incl_scan_sat(__builtin_elementwise_add_sat(a0, a1));
        const uint32_t ex = __builtin_amdgcn_update_dpp(0, (int)incl, 0x138, 0xF, 0xF, false);   // wave_shr:1
        const uint32_t x0 = __builtin_elementwise_add_sat(__builtin_elementwise_add_sat(at, ex), a0) - 1;
        const uint32_t x1 = __builtin_elementwise_add_sat(at, incl) - 1;
        o.x0 = x0;
        o.x1 = x1;
        o.v0 = x0 < (uint32_t)S;
        o.v1 = x1 < (uint32_t)S;
        o.next = at + __builtin_amdgcn_readlane(incl, 63);
    } else {
        const uint64_t a0 = (uint64_t)c0 + 1, a1 = (uint64_t)c1 + 1, sum = a0 + a1;
        const uint64_t incl = wave_incl_scan64(sum);
        o.x0 = pos + (incl - sum) + a0 - 1;
        o.x1 = o.x0 + a1;
        o.v0 = o.x0 < S;
        o.v1 = o.x1 < S;
        // (the builtin's result is signed: no sign bit may reach the upper half)
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)incl, 63);
        const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(incl >> 32), 63);
        o.next = pos + ((uint64_t)hi << 32 | lo);
    }
    o.nv = (uint32_t)(__popcll(__ballot(o.v0)) + __popcll(__ballot(o.v1)));
    return o;
}

// A tile's events generated and stored at output offset o0, in LDS batches
// of up to kSkipKeys (for p > 1/2 the complement of the failures is stored).
__device__ __forceinline__ void skip_write_tile(TileCtx &tc, uint32_t *s_key, uint64_t o0, bool flip, const GapLaw &gap)
{
    const uint32_t lane = threadIdx.x;
    const uint64_t S = tc.S;
    uint64_t pos = 0, rlo = 0, done = 0;
    uint32_t nb = 0;
    for (uint32_t r = 0;; ++r) {
        const SkipRound R = skip_round(tc, r, pos, gap);
        if (nb + R.nv > kSkipKeys) {
            // batch full: out with it (a wave-uniform decision)
            __syncthreads();
            if (!flip) {
                TileCtx tb = tc;
                tb.o0 = o0 + done;
                emit_tile(tb, s_key, nb);
                done += nb;
            } else {
                const uint64_t rhi = (uint64_t)s_key[nb - 1] + 1;
                done += emit_complement(tc, s_key, nb, rlo, rhi, done);
                rlo = rhi;
            }
            __syncthreads();
            nb = 0;
        }
        if (R.v0) s_key[nb + 2 * lane] = (uint32_t)R.x0;
        if (R.v1) s_key[nb + 2 * lane + 1] = (uint32_t)R.x1;
        nb += R.nv;
        if (R.nv < 128) break;
        pos = R.next;
    }
    __syncthreads();
    if (!flip) {
        TileCtx tb = tc;
        tb.o0 = o0 + done;
        emit_tile(tb, s_key, nb);
    } else {
        emit_complement(tc, s_key, nb, rlo, S, done);
    }
    __syncthreads();
}

__global__ __launch_bounds__(64) void skip_write_kernel(Job job)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_key[kSkipKeys];
    if (ld_uni(job.status + 1)) return;
    const double p = job.one.p;
    const bool flip = p > 0.5;
    const bool all = p >= 1.0;
    __shared__ double2 s_tab[kGapTab];
    load_gap_tab(s_tab);
    const GapLaw gap = gap_law(all ? -1.0 : log1p_f64(flip ? -(1.0 - p) : -p), job.one.s, s_tab);
    TileWalk w;
    TileCtx &tc = w.tc;
    tc.edges = job.edges;
    TileGrab grab;
    uint64_t t, t1;
    while (grab.next(job, t, t1)) {
        uint64_t g = chunk_of_tile(job, t);
        for (;;) {
            w.enter(job, g);
            const uint64_t tend = w.gend < t1 ? w.gend : t1;
            for (; t < tend; ++t) {
                const uint64_t o0 = ld_uni(job.tile_off + t);
                const uint64_t k = ld_uni(job.tile_off + t + 1) - o0;
                if (k == 0) continue;
                w.tile(t);
                tc.st.tag = TAG_SKIP;
                tc.o0 = o0;
                if (all) emit_complement(tc, s_key, 0, 0, tc.S, 0);
                else skip_write_tile(tc, s_key, o0, flip, gap);
            }
            if (t >= t1) break;
            ++g;
            while (ld_uni(job.tstart + g + 1) <= t) ++g;
        }
    }
}

// Gap pass: generates each tile's events once, and, where the workspace holds
// a slab of rows (cap > 0), keeps the positions of up to `cap` of them in the
// tile's row (slab + t cap, ascending) and writes the tile's edge count;
// after the scan an emission pass only decodes the stored positions, so the
// Philox block and logarithm of a gap are paid once instead of twice.  A tile
// with more events than its row holds is generated again by the write path.
__global__ __launch_bounds__(64) void skip_gen_kernel(Job job, uint32_t *slab, uint32_t cap)
{
    const double p = job.one.p;
    const bool flip = p > 0.5;
    const bool all = p >= 1.0;
    __shared__ double2 s_tab[kGapTab];
    load_gap_tab(s_tab);
    const GapLaw gap = gap_law(all ? -1.0 : log1p_f64(flip ? -(1.0 - p) : -p), job.one.s, s_tab);
    const uint32_t lane = threadIdx.x;
    TileWalk w;
    TileCtx &tc = w.tc;
    TileGrab grab;
    uint64_t t, t1;
    while (grab.next(job, t, t1)) {
        uint64_t g = chunk_of_tile(job, t);
        for (;;) {
            w.enter(job, g);
            const uint64_t tend = w.gend < t1 ? w.gend : t1;
            for (; t < tend; ++t) {
                w.tile(t);
                tc.st.tag = TAG_SKIP;
                const uint64_t S = tc.S;
                uint64_t nev = 0;
                if (!all && p > 0.0) {
                    uint32_t *row = slab + t * (uint64_t)cap;
                    uint64_t pos = 0;
                    for (uint32_t r = 0;; ++r) {
                        const SkipRound R = skip_round(tc, r, pos, gap);
                        // i0 and cap are even: the pair fits or none of it
                        // does; the row's end past its events is not read
                        const uint64_t i0 = nev + 2 * lane;
                        if (R.v0 && i0 < cap)
                            *reinterpret_cast<uint2 *>(row + i0) = make_uint2((uint32_t)R.x0, (uint32_t)R.x1);
                        nev += R.nv;
                        if (R.nv < 128) break;
                        pos = R.next;
                    }
                }
                const uint64_t k = all ? S : !(p > 0.0) ? 0 : flip ? S - nev : nev;
                if (lane == 0) job.tile_off[t] = k;
            }
            if (t >= t1) break;
            ++g;
            while (ld_uni(job.tstart + g + 1) <= t) ++g;
        }
    }
}

// Counts without positions, a lane per tile: for many tiles of few events, where
// most of a wave's 128 gaps would lie past its tile's end (kg_gnp_skip's rule).
__global__ __launch_bounds__(64) void skip_count_kernel(Job job)
{
    const Inst I = job.one;
    const bool flip = I.p > 0.5;
    const bool all = I.p >= 1.0;
    __shared__ double2 s_tab[kGapTab];
    load_gap_tab(s_tab);
    const GapLaw gap = gap_law(all ? -1.0 : log1p_f64(flip ? -(1.0 - I.p) : -I.p), I.s, s_tab);
    const uint64_t t = (uint64_t)blockIdx.x * 64 + threadIdx.x;
    if (t >= job.status[2]) return;
    const uint64_t g = last_le(job.tstart, job.G, t), tl = t - job.tstart[g];
    const uint64_t lo = tl << I.s, end = lo + (1ull << I.s), N = chunk_geometry(I, g).N;
    const uint64_t S = (end < N ? end : N) - lo;
    uint64_t nev = 0, pos = 0;
    if (!all && I.p > 0.0) {
        Draws64 d(make_stream(I.seed, (uint32_t)g, (uint32_t)tl, TAG_SKIP));
        for (;; ++nev) {
            const double w = gap(unit_of(d.get()));
            if (w >= (double)(S - pos)) break;
            pos += (uint64_t)w + 1;
        }
    }
    job.tile_off[t] = all ? S : !(I.p > 0.0) ? 0 : flip ? S - nev : nev;
}

// The gap pass's tile counts summed per wave of 64 tiles (for the scan).
__global__ __launch_bounds__(64) void skip_sums_kernel(Job job)
{
    const uint64_t t = (uint64_t)blockIdx.x * 64 + threadIdx.x;
    const uint64_t T = job.status[2];
    const uint64_t k = t < T ? job.tile_off[t] : 0;
    const uint64_t incl = wave_incl_scan64(k);
    if (threadIdx.x == 63) job.queue[blockIdx.x] = incl;
}

// Emission pass of the slab variant: each tile's stored positions through
// LDS to the decoders (the complement of them for p > 1/2).  Bound by memory:
// 4 bytes read and 8 written per edge, 1.40 ms for 536 million edges
// (4.6 TB/s, what a large copy reaches).
__global__ __launch_bounds__(64) void skip_emit_kernel(Job job, const uint32_t *slab, uint32_t cap)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_key[kSkipKeys];
    if (ld_uni(job.status + 1)) return;
    const double p = job.one.p;
    const bool flip = p > 0.5;
    const bool all = p >= 1.0;
    // (rarely used: no table)
    const GapLaw gap = gap_law(all ? -1.0 : log1p_f64(flip ? -(1.0 - p) : -p), job.one.s, nullptr);
    const uint32_t lane = threadIdx.x;
    TileWalk w;
    TileCtx &tc = w.tc;
    tc.edges = job.edges;
    TileGrab grab;
    uint64_t t, t1;
    while (grab.next(job, t, t1)) {
        uint64_t g = chunk_of_tile(job, t);
        for (;;) {
            w.enter(job, g);
            const uint64_t tend = w.gend < t1 ? w.gend : t1;
            for (; t < tend; ++t) {
                const uint64_t o0 = ld_uni(job.tile_off + t);
                const uint64_t k = ld_uni(job.tile_off + t + 1) - o0;
                if (k == 0) continue;
                w.tile(t);
                tc.st.tag = TAG_SKIP;
                tc.o0 = o0;
                const uint64_t S = tc.S;
                if (all) {
                    emit_complement(tc, s_key, 0, 0, S, 0);
                    continue;
                }
                const uint64_t nev = flip ? S - k : k;
                if (nev > cap) {
                    skip_write_tile(tc, s_key, o0, flip, gap);
                    continue;
                }
                // the row to LDS, 16 bytes per lane (rows start 16-byte
                // aligned: cap is a multiple of 4), then the tail word by word
                const uint32_t *row = slab + t * (uint64_t)cap;
                const uint32_t n4 = (uint32_t)nev & ~3u;
                for (uint32_t i = 4 * lane; i < n4; i += 256)
                    *reinterpret_cast<uint4 *>(s_key + i) = *reinterpret_cast<const uint4 *>(row + i);
                if (n4 + lane < (uint32_t)nev) s_key[n4 + lane] = row[n4 + lane];
                __syncthreads();
                if (!flip) emit_tile(tc, s_key, (uint32_t)nev);
                else emit_complement(tc, s_key, (uint32_t)nev, 0, S, 0);
                __syncthreads();
            }
            if (t >= t1) break;
            ++g;
            while (ld_uni(job.tstart + g + 1) <= t) ++g;
        }
    }
}

}  // namespace kg
