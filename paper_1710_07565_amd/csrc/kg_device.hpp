// kg_device.hpp -- device building blocks of the generator: counter-based
// random streams, the binary64 logarithm kernel, hypergeometric and binomial
// variates, and the geometry of chunks, tiles and edge slots.
//
// Method: Funke et al., "Communication-free Massively Distributed Graph
// Generation" (arXiv 1710.07565).  Every recursion node draws from its own
// stream so that any chunk can recompute its sample size alone (Sec. 2.2);
// sample sizes of sub-universes are hypergeometric (Sec. 2.2) or binomial
// (Sec. 4.3); variates come from acceptance-rejection (Sec. 2.2).
//
// Bit reproducibility: only IEEE binary64 + - * / sqrt and exact conversions
// are used, in a fixed order, with contraction disabled at build time
// (-ffp-contract=off).  log is computed here from those operations; no
// device math library routine decides a variate.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kg {

// ---------------------------------------------------------------------------
// Constants of the method
// ---------------------------------------------------------------------------
constexpr uint32_t kLambda = 560;       // tiles hold [560, 1120) samples in expectation (1024 at power-of-two densities)
constexpr uint32_t kUnitTiles = 64;     // most tiles of one planner unit (one lane expands it)
constexpr uint32_t kLnfTab = 1024;      // ln k! tabulated for k <= kLnfTab

enum : uint32_t { TAG_DTREE = 1, TAG_UTREE = 2, TAG_CBIN = 3, TAG_TTREE = 4, TAG_TLEAF = 5, TAG_INST = 6 };

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 32x32
// multiplications with the bijection keyed by (k0, k1), bumped by the Weyl
// constants between rounds.
// ---------------------------------------------------------------------------
struct U4 { uint32_t x, y, z, w; };

__host__ __device__ __forceinline__ U4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return U4{c0, c1, c2, c3};
}

// The same rounds for a key held in scalar registers (the same key in every
// lane of the wave): the three-way xor of a round is one v_bitop3_b32 (a
// three-input bitwise function given by its truth table; 0x96 is a ^ b ^ c)
// with the round key as its scalar operand.
__device__ __forceinline__ uint32_t xor3_sk(uint32_t a, uint32_t b, uint32_t k)
{
    uint32_t r;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "s"(k));
    return r;
}

// Philox4x32-10 of counter (a, j, b, tag) under a wave-uniform key, with a,
// b and tag wave-uniform and the block j per lane: the first round's products
// are both uniform, the second and third have one uniform product each, so
// they are formed by the scalar unit.
__device__ __forceinline__ U4 philox_wave(uint32_t a, uint32_t j, uint32_t b, uint32_t tag, uint32_t k0,
                                         uint32_t k1)
{
    uint32_t z;
    asm volatile("s_mov_b32 %0, 0" : "=s"(z));
    k0 += z;
    k1 += z;
    // round 1: c0 = a, c1 = j, c2 = b, c3 = tag
    uint64_t p0 = (uint64_t)0xD2511F53u * a;
    uint64_t p1 = (uint64_t)0xCD9E8D57u * b;
    uint32_t c0 = ((uint32_t)(p1 >> 32) ^ k0) ^ j;     // lane
    uint32_t c1 = (uint32_t)p1;                        // uniform
    uint32_t c2 = (uint32_t)(p0 >> 32) ^ tag ^ k1;     // uniform
    uint32_t c3 = (uint32_t)p0;                        // uniform
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    // round 2: c0 lane, c2 uniform
    p0 = (uint64_t)0xD2511F53u * c0;
    p1 = (uint64_t)0xCD9E8D57u * c2;
    {
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;        // uniform
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ (c3 ^ k1);      // lane
        c1 = (uint32_t)p1;                                       // uniform
        c3 = (uint32_t)p0;                                       // lane
        c0 = n0;
        c2 = n2;
    }
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    // round 3: c0 uniform, c2 lane
    p0 = (uint64_t)0xD2511F53u * c0;
    p1 = (uint64_t)0xCD9E8D57u * c2;
    {
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ (c1 ^ k0);      // lane
        const uint32_t n2 = c3 ^ ((uint32_t)(p0 >> 32) ^ k1);      // lane
        c1 = (uint32_t)p1;                                       // lane
        c3 = (uint32_t)p0;                                       // uniform
        c0 = n0;
        c2 = n2;
    }
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
#pragma unroll
    for (int r = 3; r < 10; ++r) {
        p0 = (uint64_t)0xD2511F53u * c0;
        p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3_sk((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = r == 3 ? (uint32_t)(p0 >> 32) ^ (c3 ^ k1) : xor3_sk((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return U4{c0, c1, c2, c3};
}

// A random stream: Philox keyed by the seed, counter (a, block, b, tag).
struct Stream {
    uint32_t k0, k1, a, b, tag;
    __device__ __forceinline__ U4 block(uint32_t j) const { return philox(a, j, b, tag, k0, k1); }
    // only when k0, k1 are wave-uniform (scalar registers)
    __device__ __forceinline__ U4 block_uniform_key(uint32_t j) const
    {
        return philox_wave(a, j, b, tag, k0, k1);
    }
};

__device__ __forceinline__ Stream make_stream(uint64_t seed, uint32_t a, uint32_t b, uint32_t tag)
{
    return Stream{(uint32_t)seed, (uint32_t)(seed >> 32), a, b, tag};
}

// Sequential 64-bit draws: draw d is (w1:w0) of block d/2 if d is even,
// (w3:w2) otherwise.
struct Draws64 {
    Stream s;
    uint64_t next;
    uint32_t cj;
    U4 buf;
    __device__ __forceinline__ explicit Draws64(const Stream &st) : s(st), next(0), cj(0xFFFFFFFFu), buf{0, 0, 0, 0} {}
    __device__ __forceinline__ uint64_t get()
    {
        const uint64_t d = next++;
        const uint32_t j = (uint32_t)(d >> 1);
        if (j != cj) { buf = s.block(j); cj = j; }
        return (d & 1) ? (((uint64_t)buf.w << 32) | buf.z) : (((uint64_t)buf.y << 32) | buf.x);
    }
};

// Top 52 bits plus half an ulp, (a + 1/2) 2^-52: exact, strictly inside
// (0, 1).  The bits are placed as the fraction of a number in [1, 2); both
// additions are exact.
__device__ __forceinline__ double unit_of(uint64_t x)
{
    return (__longlong_as_double((long long)((x >> 12) | 0x3FF0000000000000ull)) - 1.0) + 0x1p-53;
}

// Uniform integer in [0, R) by power-of-two mask and rejection.
__device__ __forceinline__ uint64_t draw_below(Draws64 &d, uint64_t R)
{
    const uint64_t mask = R <= 1 ? 0ull : (~0ull >> __clzll(R - 1));
    for (;;) {
        const uint64_t x = d.get() & mask;
        if (x < R) return x;
    }
}

// ---------------------------------------------------------------------------
// Natural logarithm from + - * / (binary64).  x = 2^e f, f in [sqrt(1/2),
// sqrt(2)); with u = f - 1 (exact) and s = u / (2 + u),
//   log f = 2 atanh(s) = u - (u^2/2 - s (u^2/2 + R(s^2))),
//   R(z) = sum_{i=1..11} 2 z^i / (2i + 1)  (Horner, innermost term first);
// e ln 2 is added as e*hi (exact: hi has 32 fraction bits) and e*lo.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double atanh_series(double z)
{
    double r = 2.0 / 23.0;
    r = 2.0 / 21.0 + z * r;
    r = 2.0 / 19.0 + z * r;
    r = 2.0 / 17.0 + z * r;
    r = 2.0 / 15.0 + z * r;
    r = 2.0 / 13.0 + z * r;
    r = 2.0 / 11.0 + z * r;
    r = 2.0 / 9.0 + z * r;
    r = 2.0 / 7.0 + z * r;
    r = 2.0 / 5.0 + z * r;
    r = 2.0 / 3.0 + z * r;
    return z * r;
}

__device__ __forceinline__ double log_f64(double x)
{
    const double kLn2Hi = 0x1.62e42fee00000p-1;
    const double kLn2Lo = 0x1.a39ef35793c76p-33;
    const uint64_t bits = (uint64_t)__double_as_longlong(x);
    int e = (int)((bits >> 52) & 0x7ffu) - 1023;
    const uint64_t mant = bits & 0x000FFFFFFFFFFFFFull;
    uint64_t fb;
    if (mant > 0x6A09E667F3BCDull) { fb = mant | (1022ull << 52); e += 1; }   // above sqrt(2)
    else                           { fb = mant | (1023ull << 52); }
    const double f = __longlong_as_double((long long)fb);
    const double u = f - 1.0;
    const double s = u / (2.0 + u);
    const double z = s * s;
    const double R = atanh_series(z);
    const double hfsq = 0.5 * u * u;
    const double dk = (double)e;
    return dk * kLn2Hi - ((hfsq - (s * (hfsq + R) + dk * kLn2Lo)) - u);
}

__device__ __forceinline__ double log1p_f64(double x)
{
    if (x > -0.25 && x < 0.25) {
        const double s = x / (2.0 + x);
        const double z = s * s;
        const double R = atanh_series(z);
        const double hfsq = 0.5 * x * x;
        return x - (hfsq - s * (hfsq + R));
    }
    return log_f64(1.0 + x);
}

// ---------------------------------------------------------------------------
// ln k!: table T[k] = T[k-1] + log k for k <= 1024 (built on the device by
// kg_lnf_init_kernel); above it only differences are needed, from Stirling's
// series with three correction terms in z = k + 1:
//   lnf(a+d) - lnf(a) = (z - 1/2) log1p(d/z) + d (log(z + d) - 1)
//                       + corr(z + d) - corr(z),
//   corr(z) = 1/(12 z) - 1/(360 z^3) + 1/(1260 z^5),
// so that two large log-factorials are never subtracted.
// ---------------------------------------------------------------------------
extern __device__ double g_lnf_tab[kLnfTab + 1];

__device__ __forceinline__ double stirling_corr(double z)
{
    const double r = 1.0 / z;
    const double r2 = r * r;
    return r * (1.0 / 12.0 - r2 * (1.0 / 360.0 - r2 * (1.0 / 1260.0)));
}

__device__ __forceinline__ double stirling_diff(uint64_t a, uint64_t d)
{
    const double z = (double)(a + 1);
    const double zd = (double)(a + d + 1);
    const double dd = (double)d;
    const double t1 = (z - 0.5) * log1p_f64(dd / z);
    const double t2 = dd * (log_f64(zd) - 1.0);
    const double t3 = stirling_corr(zd) - stirling_corr(z);
    return (t1 + t2) + t3;
}

// lnf(y) - lnf(x).  Both cases above the table go through one Stirling
// difference (lanes of a wave often differ in the case): from x itself, or
// from the end of the table with the tabulated part below it added; in the
// first case the added part is +0.0, which leaves the value unchanged.
__device__ __forceinline__ double lnf_diff(uint64_t x, uint64_t y)
{
    if (x == y) return 0.0;
    const bool neg = x > y;
    const uint64_t lo = neg ? y : x, hi = neg ? x : y;
    double r;
    if (hi <= kLnfTab) {
        r = g_lnf_tab[hi] - g_lnf_tab[lo];
    } else {
        const bool part = lo < kLnfTab;
        const uint64_t a = part ? (uint64_t)kLnfTab : lo;
        const double tp = part ? g_lnf_tab[kLnfTab] - g_lnf_tab[part ? lo : 0] : 0.0;
        r = tp + stirling_diff(a, hi - a);
    }
    return neg ? -r : r;
}

// floor(a * b / d) for a*b < 2^117, d >= 1 and a quotient below 2^53,
// exactly: an estimate `est` (off by 2^-45 of itself and one), corrected by the
// remainder.  Below d = 2^60 and a quotient of 2^45 the remainder of the estimate
// fits a signed 64-bit word, so the products are needed modulo 2^64 only.
__device__ __forceinline__ uint64_t muldiv_floor(uint64_t a, uint64_t b, uint64_t d, double est)
{
    uint64_t q = est <= 0.0 ? 0ull : (uint64_t)est;
    if (((uint32_t)(d >> 60) | (uint32_t)(q >> 45)) == 0) {
        int64_t r = (int64_t)(a * b - q * d);
        while (r < 0) { --q; r += (int64_t)d; }
        while (r >= (int64_t)d) { ++q; r -= (int64_t)d; }
        return q;
    }
    typedef unsigned __int128 u128;
    const u128 num = (u128)a * b;
    while ((u128)q * d > num) --q;
    while ((u128)(q + 1) * d <= num) ++q;
    return q;
}

// ---------------------------------------------------------------------------
// Discrete ratio of uniforms (Kinderman-Monahan; centre mu + 1/2 and
// half-width (D1 sqrt(var + 1/2) + D2)/2 as in Stadlober's samplers).
// Proposal j uses block j: U from (w1:w0), V from (w3:w2);
// X = floor(a + h (V - 1/2) / U), accepted iff 2 log U <= log f(X)/f(M),
// with the squeezes 4U - U^2 - 3 <= T (accept) and T <= U - 1/U (reject).
// ---------------------------------------------------------------------------
constexpr double kRouD1 = 0x1.b72cd3f331398p+0;   // 2 sqrt(2/e)
constexpr double kRouD2 = 0x1.cc3ebd3bc711ap-1;   // 3 - 2 sqrt(3/e)

// log f(x) - log f(M) of the hypergeometric law.
struct HypRatio {
    uint64_t N, K, k, M;
    __device__ __forceinline__ double operator()(uint64_t X) const
    {
        // one copy of the difference's code (rarely run: see RouQuick)
        double T = 0.0;
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const uint64_t b = i == 0 ? 0 : i == 1 ? k : i == 2 ? K : N - K - k;
            const bool up = i == 0 || i == 3;
            T = T + lnf_diff(up ? b + X : b - X, up ? b + M : b - M);
        }
        return T;
    }
};

// log f(x) - log f(M) of the binomial law.
struct BinRatio {
    uint64_t N, M;
    double p;
    __device__ __forceinline__ double operator()(uint64_t X) const
    {
        double T = 0.0;
#pragma unroll 1
        for (int i = 0; i < 2; ++i) T = T + lnf_diff(i ? N - X : X, i ? N - M : M);
        if (p != 0.5) {                    // log p - log(1 - p) is zero at 1/2
            const double lq = log_f64(p) - log1p_f64(-p);
            T = T + ((double)X - (double)M) * lq;
        }
        return T;
    }
};

// ---------------------------------------------------------------------------
// The acceptance decision in binary32.  A proposal is accepted iff
// 2 log U <= T = log f(X) - log f(M) (the squeezes lie on either side of
// 2 log U, so away from equality they never change the decision).  The four
// (hypergeometric) or two (binomial) log-factorial differences of T, the
// arguments A_i moving by +d or -d, d = X - M, are with y_i = A_i + 1/2
//   ln (A_i + d)! - ln A_i! = d ln y_i + y_i phi(d / y_i) + (t - t^2) / (24 y_i) + ...,
//   phi(t) = (1 + t) ln(1 + t) - t = t^2 (1/2 - t/6 + t^2/12 - ...),
// (Stirling's series about A + 1/2).  The d ln y_i add up to d times the
// logarithm of a ratio that is 1 + q with |q| <= sum 1 / y_i because M is the
// mode, so nothing large is subtracted and binary32 holds T to
// 2e-6 of the sum of its terms plus the neglected 2e-5 of the smallest
// arguments taken (y = 16, t = 0.2; measured at most 0.37 of the margin
// below).  Proposals with |t| > 0.2 or |d| >= 2^24 (a few per cent: the
// ratio of uniforms has a heavy tail) are rejected by a bound on phi.
// Decisions closer than the margin, and laws outside y >= 16, |q| <= 1/16, go
// to the binary64 ratio above (about one proposal in 10^4 of the tile
// tree's), so the variates are those of the binary64 test bit for bit.  Measured, headline call: planner 0.38 ->
// 0.15 ms, count kernel 0.167 -> 0.069 ms (under the profiler; the binary64
// ratio is about 500 vector instructions, this one about 50).
// ---------------------------------------------------------------------------
template <int NT>
struct RouQuick {
    static_assert(NT == 2 || NT == 4, "binomial: two factorials, hypergeometric: four");
    float lam, iy[NT];

    static __device__ __forceinline__ constexpr bool up(int i) { return i == 0 || i == 3; }

    // y_i, and the ratio's q = num / den
    __device__ __forceinline__ void init(const double (&y)[NT], double num, double den)
    {
        float c = 0.0f, most = 0.0f;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            iy[i] = __builtin_amdgcn_rcpf((float)y[i]);
            c = __builtin_fmaf(up(i) ? iy[i] : -iy[i], iy[i], c);
            most = fmaxf(most, iy[i]);
        }
        const float q = (float)num * __builtin_amdgcn_rcpf((float)den);
        float l = __builtin_fmaf(q, -1.0f / 6.0f, 0.2f);
        l = __builtin_fmaf(q, l, -0.25f);
        l = __builtin_fmaf(q, l, 1.0f / 3.0f);
        l = __builtin_fmaf(q, l, -0.5f);
        l = __builtin_fmaf(q, l, 1.0f);
        lam = __builtin_fmaf(c, 1.0f / 24.0f, q * l);
        if (!(most <= 1.0f / 16.0f && fabsf(q) <= 1.0f / 16.0f)) iy[0] = 1e30f;   // every t is out of range
    }

    // 1: accepted, 0: rejected, -1: too close to say.  X = M + dd is in
    // range, so every A_i + d is at least 0 and every t above -1.
    __device__ __forceinline__ int decide(double dd, double U) const
    {
        const float d = (float)dd;
        // 2 ln U; the hardware's base-2 logarithm is good to 1 ulp
        const float lu = 1.3862943611f * __builtin_amdgcn_logf((float)U);
        float most = iy[0];
#pragma unroll
        for (int i = 1; i < NT; ++i) most = fmaxf(most, iy[i]);
        const float ad = fabsf(d);
        if (!(ad * most <= 0.2f && ad < 0x1p24f)) {
            // far from the mode (a small U): phi(t) >= t^2 / (2 + 2 |t| / 3)
            // (Bernstein) bounds T from above; the neglected terms are below 1
            if (most > 1.0f) return -1;
            float low = 0.0f;
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const float t = ad * iy[i];
                low = __builtin_fmaf(ad * t, __builtin_amdgcn_rcpf(__builtin_fmaf(t, 0.66666669f, 2.0f)), low);
            }
            return 0.9999f * low - 1.0001f * fabsf(d * lam) + lu > 1.0f ? 0 : -1;
        }
        const float d2 = d * d;
        float S = 0.0f;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const float t = (up(i) ? d : -d) * iy[i];
            float P = __builtin_fmaf(t, -1.0f / 72.0f, 1.0f / 56.0f);
            P = __builtin_fmaf(t, P, -1.0f / 42.0f);
            P = __builtin_fmaf(t, P, 1.0f / 30.0f);
            P = __builtin_fmaf(t, P, -1.0f / 20.0f);
            P = __builtin_fmaf(t, P, 1.0f / 12.0f);
            P = __builtin_fmaf(t, P, -1.0f / 6.0f);
            P = __builtin_fmaf(t, P, __builtin_fmaf(iy[i] * iy[i], -1.0f / 24.0f, 0.5f));
            S = __builtin_fmaf(d2 * iy[i], P, S);
        }
        const float gap = __builtin_fmaf(d, lam, S) + lu;
        const float eps = __builtin_fmaf(2e-6f, S - lu, 5e-5f);
        return gap < -eps ? 1 : gap > eps ? 0 : -1;
    }
};

// The binary64 test of one proposal, with the squeezes.
template <class Ratio>
__device__ __forceinline__ bool rou_accept(const Ratio &ratio, uint64_t X, double U)
{
    const double T = ratio(X);
    if (U * (4.0 - U) - 3.0 <= T) return true;
    if (U * (U - T) >= 1.0) return false;
    return 2.0 * log_f64(U) <= T;
}

// Proposal j of a variate: accepted or not, and its X (a whole number).
// Md is the mode, excl = upper + 1.
template <class Ratio, class Quick>
__device__ __forceinline__ bool rou_try(const Stream &s, uint32_t j, double a, double h, uint64_t upper, double excl,
                                        double Md, const Ratio &ratio, const Quick &quick, double &X)
{
    const U4 w = s.block(j);
    const double U = unit_of(((uint64_t)w.y << 32) | w.x);
    const double V = unit_of(((uint64_t)w.w << 32) | w.z);
    const double t = a + h * (V - 0.5) / U;
    if (!(t >= 0.0 && t < excl)) return false;
    X = floor(t);
    if (upper >> 53 && (uint64_t)X > upper) return false;      // upper + 1 rounds in binary64
    const int dec = quick.decide(X - Md, U);
    return __builtin_expect(dec < 0, 0) ? rou_accept(ratio, (uint64_t)X, U) : dec != 0;
}

// Aligned groups of PAR lanes: the lowest lane of the caller's group with
// `acc` set decides; its X to the whole group.  False when no lane has it.
template <int PAR>
__device__ __forceinline__ bool group_first(bool acc, double &X)
{
    const uint64_t all = __ballot(acc);
    const uint64_t bits = (uint64_t)__double_as_longlong(X);
    uint32_t lo, hi;
    if (PAR == 64) {
        if (!all) return false;
        const int src = __builtin_ctzll(all);
        lo = __builtin_amdgcn_readlane((uint32_t)bits, src);
        hi = __builtin_amdgcn_readlane((uint32_t)(bits >> 32), src);
    } else {
        const uint32_t base = __lane_id() & ~(uint32_t)(PAR - 1);
        const uint32_t won = (uint32_t)(all >> base) & (uint32_t)((1ull << (PAR & 63)) - 1);
        if (!won) return false;
        const int src = (int)(base + __builtin_ctz(won));
        lo = (uint32_t)__shfl((int)(uint32_t)bits, src);
        hi = (uint32_t)__shfl((int)(uint32_t)(bits >> 32), src);
    }
    X = __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    return true;
}

// PAR = 1: one proposal at a time.  Otherwise an aligned group of PAR lanes
// works on one variate (the same arguments in every lane of the group) and
// tries proposals j0 .. j0 + PAR - 1 at once; the lowest accepted one wins,
// so the variate is the one the sequential loop returns.  Used where a
// variate's latency, not the lanes' throughput, bounds a kernel.
template <int PAR, class Ratio, class Quick>
__device__ __forceinline__ uint64_t rou_sample(const Stream &s, double a, double h, uint64_t upper, double Md,
                                               const Ratio &ratio, const Quick &quick)
{
    static_assert(PAR == 1 || PAR == 2 || PAR == 4 || PAR == 8 || PAR == 64, "lanes per variate");
    const uint32_t q = __lane_id() & (PAR - 1);
    const double excl = (double)upper + 1.0;
    for (uint32_t j0 = 0;; j0 += PAR) {
        double X = 0.0;
        const bool acc = rou_try(s, j0 + q, a, h, upper, excl, Md, ratio, quick, X);
        if (PAR == 1 ? acc : group_first<PAR>(acc, X)) return (uint64_t)X;
    }
}

// The quick test's arguments of HYP(N, K, k) and BIN(N, p).
// (The differences of the binary64 values are exact or lose nothing that
// matters: k and M are below 2^53, and M is at most half of K.)
__device__ __forceinline__ RouQuick<4> quick_of(const HypRatio &r, double Kd, double kd, double Md)
{
    const double y1 = Md + 0.5, y2 = (kd - Md) + 0.5, y3 = (Kd - Md) + 0.5;
    const double y4 = (double)(r.N - r.K - r.k + r.M) + 0.5;
    RouQuick<4> q;
    const double den = y2 * y3;
    q.init({y1, y2, y3, y4}, y1 * y4 - den, den);
    return q;
}
__device__ __forceinline__ RouQuick<2> quick_of(const BinRatio &r, double Nd, double Md)
{
    const double y1 = Md + 0.5, y2 = (Nd - Md) + 0.5;
    RouQuick<2> q;
    const double den = y2 * r.p;
    q.init({y1, y2}, y1 * (1.0 - r.p) - den, den);
    return q;
}

// The mode floor((k + 1)(K + 1) / (N + 2)).
__device__ __forceinline__ uint64_t hyp_mode(uint64_t N, uint64_t K, uint64_t k, double Nd, double Kd, double kd)
{
    // the quotient to 2^-45 of itself at worst: the hardware's reciprocal (2^29 ulp,
    // 2^-23), one step
    const double d = Nd + 2.0;
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    return muldiv_floor(k + 1, K + 1, N + 2, floor((kd + 1.0) * (Kd + 1.0) * r));
}

// Hypergeometric: how many of k draws without replacement from N items land
// among K marked ones (the sample size of a sub-universe, Sec. 2.2).
template <int PAR = 1>
__device__ __forceinline__ uint64_t hyp(const Stream &s, uint64_t N, uint64_t K, uint64_t k)
{
    // symmetries: complement the draws, complement the marked set, swap roles
    uint64_t k1 = k, K1 = K;
    bool c1 = false, c2 = false;
    if (k1 > N - k1) { k1 = N - k1; c1 = true; }
    if (K1 > N - K1) { K1 = N - K1; c2 = true; }
    const uint64_t lo = k1 < K1 ? k1 : K1;   // draws
    const uint64_t hi = k1 < K1 ? K1 : k1;   // marked
    uint64_t x;
    if (lo == 0) {
        x = 0;
    } else if (lo <= 16) {
        // direct simulation: the i-th draw picks one of the N - i items left
        Draws64 d(s);
        x = 0;
        for (uint64_t i = 0; i < lo; ++i)
            if (draw_below(d, N - i) < hi - x) ++x;
    } else {
        const double Nd = (double)N, Kd = (double)hi, kd = (double)lo;
        const double pp = Kd / Nd;
        const double mu = kd * pp;
        const double var = (((Nd - kd) * kd) * pp) * (1.0 - pp) / (Nd - 1.0);
        const double c = sqrt(var + 0.5);
        const double h = kRouD1 * c + kRouD2;
        const double a = mu + 0.5;
        const HypRatio r{N, hi, lo, hyp_mode(N, hi, lo, Nd, Kd, kd)};
        const double Md = (double)r.M;
        x = rou_sample<PAR>(s, a, h, lo, Md, r, quick_of(r, Kd, kd, Md));
    }
    if (c2) x = k1 - x;
    if (c1) x = K - x;
    return x;
}

// The same hypergeometric variate as hyp(), consumed one ratio-of-uniforms
// proposal per step() so that lanes of a wave working on different variates
// do not wait for each other's rejection loops.  Identical draws and result.
struct HypRun {
    Stream s;
    HypRatio r;           // r.K marked items, r.k draws, after the symmetries
    RouQuick<4> quick;
    uint64_t K, k1, x;
    double a, h, Md, excl;
    uint32_t j;
    bool c1, c2, done;

    __device__ __forceinline__ void init(const Stream &st, uint64_t N, uint64_t K_, uint64_t k)
    {
        s = st;
        K = K_;
        k1 = k;
        uint64_t K1 = K_;
        c1 = c2 = false;
        if (k1 > N - k1) { k1 = N - k1; c1 = true; }
        if (K1 > N - K1) { K1 = N - K1; c2 = true; }
        const uint64_t lo = k1 < K1 ? k1 : K1;
        const uint64_t hi = k1 < K1 ? K1 : k1;
        r.N = N;
        r.K = hi;
        r.k = lo;
        j = 0;
        done = true;
        if (lo == 0) {
            x = 0;
        } else if (lo <= 16) {
            Draws64 d(s);
            x = 0;
            for (uint64_t i = 0; i < lo; ++i)
                if (draw_below(d, N - i) < hi - x) ++x;
        } else {
            const double Nd = (double)N, Kd = (double)hi, kd = (double)lo;
            const double pp = Kd / Nd;
            const double mu = kd * pp;
            const double var = (((Nd - kd) * kd) * pp) * (1.0 - pp) / (Nd - 1.0);
            const double c = sqrt(var + 0.5);
            h = kRouD1 * c + kRouD2;
            a = mu + 0.5;
            r.M = hyp_mode(N, hi, lo, Nd, Kd, kd);
            Md = (double)r.M;
            excl = kd + 1.0;
            quick = quick_of(r, Kd, kd, Md);
            done = false;
        }
    }

    // one trip of proposals; true once the variate is known.  PAR > 1: the
    // aligned group of PAR lanes holding the same state tries PAR proposals
    // at once (the lowest accepted one is the sequential walk's).
    template <int PAR = 1>
    __device__ __forceinline__ bool step()
    {
        if (done) return true;
        double X = 0.0;
        const bool acc = rou_try(s, j + (__lane_id() & (PAR - 1)), a, h, r.k, excl, Md, r, quick, X);
        j += PAR;
        if (PAR == 1 ? acc : group_first<PAR>(acc, X)) { x = (uint64_t)X; done = true; }
        return done;
    }

    __device__ __forceinline__ uint64_t result() const
    {
        uint64_t y = x;
        if (c2) y = k1 - y;
        if (c1) y = K - y;
        return y;
    }
};

// Waiting time of Bernoulli(1/2) trials, floor(log U / log(1/2)): the
// exponent of U, unless U is within 2^-20 of a power of two, where the
// rounding of the quotient decides.
__device__ __forceinline__ uint64_t half_gap(double U)
{
    const uint32_t hi = (uint32_t)((uint64_t)__double_as_longlong(U) >> 32);
    const uint32_t top = hi & 0xFFFFFu;
    if (top == 0 || top == 0xFFFFFu) return (uint64_t)floor(log_f64(U) / log1p_f64(-0.5));
    return 1022u - (hi >> 20);
}

// Binomial(N, p): a G(n,p) chunk's edge count (Sec. 4.3).  Small means by
// geometric waiting times floor(log U / log(1-p)); otherwise ratio of uniforms.
template <int PAR = 1>
__device__ __forceinline__ uint64_t bin_core(const Stream &s, uint64_t N, double p)
{
    const double Nd = (double)N;
    if (Nd * p < 16.0) {
        Draws64 d(s);
        uint64_t X = 0, pos = 0;
        if (p == 0.5) {
            for (;;) {
                const uint64_t g = half_gap(unit_of(d.get()));
                if (g >= N - pos) return X;
                pos += g + 1;
                ++X;
            }
        }
        const double L = log1p_f64(-p);
        for (;;) {
            const double U = unit_of(d.get());
            const double g = floor(log_f64(U) / L);
            if (g >= (double)(N - pos)) return X;
            pos += (uint64_t)g + 1;
            ++X;
        }
    }
    const double q = 1.0 - p;
    const double mu = Nd * p;
    const double var = mu * q;
    const double c = sqrt(var + 0.5);
    const double h = kRouD1 * c + kRouD2;
    const double a = mu + 0.5;
    const double Md = floor((Nd + 1.0) * p);
    const BinRatio r{N, (uint64_t)Md, p};
    return rou_sample<PAR>(s, a, h, N, Md, r, quick_of(r, Nd, Md));
}

template <int PAR = 1>
__device__ __forceinline__ uint64_t binom(const Stream &s, uint64_t N, double p)
{
    if (N == 0 || p <= 0.0) return 0;
    if (p >= 1.0) return N;
    if (p > 0.5) return N - bin_core<PAR>(s, N, 1.0 - p);
    return bin_core<PAR>(s, N, p);
}

// ---------------------------------------------------------------------------
// Instances and chunk geometry (Sec. 4.1 row chunks; Sec. 4.2 sections and
// the upper-triangular chunk matrix, ordered row-major).
// ---------------------------------------------------------------------------
struct Inst {
    uint64_t n, m;
    double p;
    uint64_t seed;
    uint32_t model, directed, P, s;   // s: tile exponent, tiles of 2^s slots
    uint64_t nchunks;                 // chunks generated: P (directed) or P(P+1)/2; 1 or P for a view
    uint64_t chunk_base;              // first global chunk index of the instance
    uint32_t view;                    // 0: the whole graph; r + 1: the edges incident to section r
    uint32_t pad_;
};

__host__ __device__ __forceinline__ uint64_t section_bound(const Inst &I, uint64_t i)
{
    // floor(i n / P); i n < 2^64 because i <= P <= 2^31 and n <= 2^32
    return (i * I.n) / I.P;
}

// floor(x / d) where the quotient is below 2^50, from rcp = 1 / d in
// binary64: the estimate is off by less than one, so one step corrects it
// (a 64-bit integer division takes about 130 instructions here).
__device__ __forceinline__ uint64_t div_est(uint64_t x, uint64_t d, double rcp)
{
    uint64_t q = (uint64_t)((double)x * rcp);
    const int64_t r = (int64_t)(x - q * d);
    if (r < 0) --q;
    else if ((uint64_t)r >= d) ++q;
    return q;
}

// section_bound(I, i) on the device: floor(i n / P) = i floor(n / P) +
// floor(i (n mod P) / P).  floor(n / P) is the floor of the binary64
// quotient, because n <= 2^32 keeps a fraction 2^-32 away from an integer.
struct Sections {
    uint64_t q, r, P;
    double rcp;
    __device__ __forceinline__ explicit Sections(const Inst &I) : P(I.P), rcp(1.0 / (double)I.P)
    {
        q = (uint64_t)((double)I.n / (double)I.P);
        r = I.n - q * P;
    }
    __device__ __forceinline__ uint64_t operator()(uint64_t i) const
    {
        return i * q + div_est(i * r, P, rcp);
    }
};

__host__ __device__ __forceinline__ uint64_t uord(uint64_t P, uint64_t i)
{
    return i * P - i * (i - 1) / 2;   // ordinal of diagonal chunk (i, i)
}

// Row of the undirected chunk matrix that ordinal c lies in: the largest i
// with uord(i) <= c.  The binary64 root is within one of it (c < 2^30).
__device__ __forceinline__ uint64_t urow(uint64_t P, uint64_t c)
{
    const double b = (double)(2 * P + 1);
    int64_t i = (int64_t)((b - sqrt(b * b - 8.0 * (double)c)) * 0.5);
    i = i < 0 ? 0 : i >= (int64_t)P ? (int64_t)P - 1 : i;
    while (uord(P, (uint64_t)i) > c) --i;
    while (i + 1 < (int64_t)P && uord(P, (uint64_t)i + 1) <= c) ++i;
    return (uint64_t)i;
}

struct Chunk {
    uint64_t N;       // slots
    uint64_t row0;    // directed: first row
    uint64_t a, h;    // undirected: row section start / size
    uint64_t b, w;    // undirected: column section start / size
    uint32_t ci, cj;  // row chunk; undirected: cell of the chunk matrix
    uint32_t diag;    // undirected triangle chunk
};

// Ordinal (in the instance's canonical chunk order) of the instance's k-th
// generated chunk.  A view of section r (the per-PE partition of Sec. 4.1
// and 4.2) generates, directed, row chunk r alone; undirected, the chunks
// (i, r) for i < r and (r, j) for j >= r of the upper-triangular chunk
// matrix, in canonical order -- every edge with an endpoint in section r.
__host__ __device__ __forceinline__ uint64_t chunk_ordinal(const Inst &I, uint64_t k)
{
    if (I.view == 0) return k;
    const uint64_t r = I.view - 1;
    if (I.directed) return r;
    return k < r ? uord(I.P, k) + (r - k) : uord(I.P, r) + (k - r);
}

__device__ __forceinline__ Chunk chunk_geometry(const Inst &I, uint64_t c)
{
    Chunk g;
    g.diag = 0; g.a = g.h = g.b = g.w = 0; g.row0 = 0;
    const Sections at(I);
    if (I.directed) {
        g.ci = (uint32_t)c;
        g.cj = 0;
        g.row0 = at(c);
        g.N = (at(c + 1) - g.row0) * (I.n - 1);
        return g;
    }
    const uint64_t ci = urow(I.P, c), cj = ci + (c - uord(I.P, ci));
    g.ci = (uint32_t)ci;
    g.cj = (uint32_t)cj;
    g.a = at(ci); g.h = at(ci + 1) - g.a;
    g.b = at(cj); g.w = at(cj + 1) - g.b;
    g.diag = ci == cj;
    g.N = g.diag ? g.h * (g.h - (g.h > 0)) / 2 : g.h * g.w;
    return g;
}

// Tiles of chunk with N slots; planner units (subtrees of <= kUnitTiles
// tiles): 2^d with d minimal such that ceil(T / 2^d) <= kUnitTiles.
__device__ __forceinline__ uint64_t tiles_of(uint64_t N, uint32_t s)
{
    return (N + ((1ull << s) - 1)) >> s;
}

__device__ __forceinline__ uint32_t unit_depth(uint64_t T, uint32_t ulog)
{
    uint32_t d = 0;
    while (((T + (1ull << d) - 1) >> d) > (1ull << ulog)) ++d;
    return d;
}

// ---------------------------------------------------------------------------
// Chunk counts by walking one root-to-leaf path (what a single PE does in the
// paper; Sec. 2.2, 4.1, 4.2).  The split of a range [lo, hi) of chunks or
// sections is at lo + ceil((hi - lo)/2).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t tri_slots(uint64_t A) { return A * (A - (A > 0)) / 2; }

// A node splits its count over its parts one conditional variate at a time:
// part r gets HYP(slots left, slots of part r, count left), until the part
// that holds the chunk, and the last part gets the rest.  Directed: two
// halves of the row chunks [a, b).  Undirected: a triangle [a, b) has the
// parts T1 = [a, l), R = [a, l) x [l, b), T2 = [l, b); a rectangle
// [a, b) x [c, d) its four quadrants, or two halves where a side has one section.
// One loop over all levels and parts, so that the variate's code (the path's
// whole time is its latency, about 1.7 us per variate) appears once: 37 KB for
// the count kernel, which fits the instruction cache, where a copy per kind of
// split and a division per section bound took 146 KB.
template <int PAR = 1>
__device__ __forceinline__ uint64_t path_count(const Inst &I, uint64_t ci, uint64_t cj)
{
    const Sections at(I);
    // rows [a, b) start and end at slots' rows A, B; columns [c, d) at C, D
    uint64_t k = I.m, a = 0, b = I.P, c = 0, d = 0, A = 0, B = I.n, C = 0, D = 0;
    uint32_t code = 1;
    const bool dir = I.directed != 0;
    bool tri = !dir;
    for (;;) {
        const uint64_t l = a + (b - a + 1) / 2, q = c + (d - c + 1) / 2;
        const bool rows = b - a > 1, cols = !dir && !tri && d - c > 1;
        if (!rows && !cols) return k;
        // the node's parts: slots of the first three, their number, the chunk's
        uint64_t Lb = 0, Qb = 0, left, n0, n1 = 0, n2 = 0;
        uint32_t parts = 2, mine;
        if (rows) Lb = at(l);
        if (cols) Qb = at(q);
        if (tri) {
            left = tri_slots(B - A);
            n0 = tri_slots(Lb - A);
            n1 = (Lb - A) * (B - Lb);
            parts = 3;
            mine = cj < l ? 0 : ci < l ? 1 : 2;
        } else {
            const uint64_t w = dir ? I.n - 1 : D - C;        // slots of a row
            left = (B - A) * w;
            if (rows && cols) {
                n0 = (Lb - A) * (Qb - C);
                n1 = (Lb - A) * (D - Qb);
                n2 = (B - Lb) * (Qb - C);
                parts = 4;
                mine = (ci >= l ? 2u : 0u) + (cj >= q ? 1u : 0u);
            } else if (rows) {
                n0 = (Lb - A) * w;
                mine = ci < l ? 0 : 1;
            } else {
                n0 = (B - A) * (Qb - C);
                mine = cj < q ? 0 : 1;
            }
        }
        for (uint32_t r = 0; r + 1 < parts; ++r) {
            const uint64_t nr = r == 0 ? n0 : r == 1 ? n1 : n2;
            const uint64_t X = hyp<PAR>(make_stream(I.seed, code, dir ? 0 : r, dir ? TAG_DTREE : TAG_UTREE), left,
                                        nr, k);
            if (r == mine) { k = X; break; }
            left -= nr;
            k -= X;
        }
        code = (dir ? 2 : 4) * code + mine;
        if (tri && mine == 1) {
            tri = false;
            c = l; C = Lb; d = b; D = B;
            b = l; B = Lb;
        } else {
            const bool low = tri ? mine == 0 : parts == 4 ? mine < 2 : mine == 0;
            if (rows) { if (low) { b = l; B = Lb; } else { a = l; A = Lb; } }
            if (cols) {
                if (parts == 4 ? (mine & 1) != 0 : mine != 0) { c = q; C = Qb; } else { d = q; D = Qb; }
            }
        }
    }
}

// Slots of tile range [lo, hi) of a chunk with Nc slots.
__device__ __forceinline__ uint64_t tile_range_slots(uint64_t lo, uint64_t hi, uint32_t s, uint64_t Nc)
{
    const uint64_t e = hi << s;
    return (e > Nc ? Nc : e) - (lo << s);
}

}  // namespace kg
