// Device-side random numbers and samplers of the diffusion and reaction steps.
//
// Every floating-point expression here is evaluated exactly as written
// (the library is built with -ffp-contract=off and no fast-math), so a CPU
// program that follows the same definitions in the same order reproduces
// every draw bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#pragma clang fp contract(off)

namespace rdos {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11): ten rounds of the
// 4x32 S-box with multipliers 0xD2511F53 / 0xCD9E8D57 and a Weyl key
// schedule (0x9E3779B9, 0xBB67AE85).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint4 x, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * x.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * x.z;
        x = make_uint4((uint32_t)(p1 >> 32) ^ x.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ x.w ^ k1, (uint32_t)p0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return x;
}

// One counter-based stream: counter (draw block, stream id, tet, period),
// key (k0, k1).  Draw j takes the block j/2 and, within it, words (x, y)
// for even j or (z, w) for odd j, mapped to a 53-bit uniform in [0, 1).
// Draws are taken in order, so a new block is generated exactly at even j.
struct Stream {
    uint32_t k0, k1, id, tet, period;
    uint32_t j;
    uint4 words;

    __device__ __forceinline__ Stream(uint32_t key0, uint32_t key1, uint32_t stream_id,
                                      uint32_t tet_id, uint32_t period_id)
        : k0(key0), k1(key1), id(stream_id), tet(tet_id), period(period_id), j(0),
          words(make_uint4(0, 0, 0, 0))
    {
    }

    __device__ __forceinline__ double uniform()
    {
        if (!(j & 1u)) words = philox4x32_10(make_uint4(j >> 1, id, tet, period), k0, k1);
        return take();
    }

    __device__ __forceinline__ double take()
    {
        const uint32_t hi = (j & 1u) ? words.z : words.x;
        const uint32_t lo = (j & 1u) ? words.w : words.y;
        ++j;
        return ((double)(hi >> 5) * 67108864.0 + (double)(lo >> 6)) * 0x1p-53;
    }
};

// The same stream with its first block generated at construction, for callers
// that always draw and have loads in flight meanwhile.
struct PrimedStream : Stream {
    __device__ __forceinline__ PrimedStream(uint32_t key0, uint32_t key1, uint32_t stream_id, uint32_t tet_id,
                                            uint32_t period_id)
        : Stream(key0, key1, stream_id, tet_id, period_id)
    {
        words = philox4x32_10(make_uint4(0, id, tet, period), k0, k1);
    }

    __device__ __forceinline__ double uniform()
    {
        if (!(j & 1u) && j != 0) words = philox4x32_10(make_uint4(j >> 1, id, tet, period), k0, k1);
        return take();
    }
};

// ---------------------------------------------------------------------------
// Natural logarithm from add/sub/mul/div only (no hardware transcendental):
// reduce x = 2^e m with m in [sqrt(1/2), sqrt(2)); with f = m - 1 and
// s = f / (2 + f), ln m = 2 atanh s = f - s (f - 2 R(s^2)) where
// R(z) = z/3 + z^2/5 + ... + z^11/23 (Horner); add e ln 2 with ln 2 split into
// a head whose products with e are exact and a rounded tail.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double log_basic(double x)
{
    constexpr double kLn2Head = 0x1.62e42fee00000p-1;
    constexpr double kLn2Tail = 0x1.a39ef35793c76p-33;
    constexpr double kSqrt2 = 0x1.6a09e667f3bcdp+0;
    uint64_t bits = (uint64_t)__double_as_longlong(x);
    int e = (int)((bits >> 52) & 0x7ffu);
    if (e == 0) {  // subnormal input
        x = x * 0x1p54;
        bits = (uint64_t)__double_as_longlong(x);
        e = (int)((bits >> 52) & 0x7ffu) - 54;
    }
    e -= 1023;
    double m = __longlong_as_double((long long)((bits & 0x000fffffffffffffull) | 0x3ff0000000000000ull));
    if (m > kSqrt2) {
        m = m * 0.5;
        e += 1;
    }
    const double f = m - 1.0;
    const double s = f / (2.0 + f);
    const double z = s * s;
    const double R =
        z * (1.0 / 3.0 + z * (1.0 / 5.0 + z * (1.0 / 7.0 + z * (1.0 / 9.0 + z * (1.0 / 11.0 +
        z * (1.0 / 13.0 + z * (1.0 / 15.0 + z * (1.0 / 17.0 + z * (1.0 / 19.0 + z * (1.0 / 21.0 +
        z * (1.0 / 23.0)))))))))));
    const double lnm = f - s * (f - 2.0 * R);
    const double de = (double)e;
    return de * kLn2Head + (lnm + de * kLn2Tail);
}

// ---------------------------------------------------------------------------
// Binomial(n, p), exact in law:
//   BINV  sequential inversion from P(0) = q^n (Kachitvichyanukul &
//         Schmeiser, 1988) when n p < 10,
//   BTRD  transformed rejection with decomposition (Hoermann, 1993)
//         otherwise;
// p > 1/2 is sampled as n - Binomial(n, 1 - p).
// ---------------------------------------------------------------------------

// a / x for a whole x below 2^31, y = 1 / x to within a few ulp: the product
// a y corrected once by its exact residual.  A quotient by such an x lies at
// least 2^-32 ulp from the midpoint of two doubles (or is one of them), far
// more than the correction's own error, so the result is the correctly
// rounded quotient, as a / x is; it needs 3 operations beside y where the
// division takes 11.  For quotients clear of under- and overflow.
__device__ __forceinline__ double divide_by_whole(double a, double x, double y)
{
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-x, q, a), y, q);
}

// 1 / x to within a few ulp (the hardware estimate and two Newton steps).
__device__ __forceinline__ double reciprocal_near(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
    return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}

// q^n by squaring, low bits first, two bits a pass; the lanes of a wavefront
// share the passes (products past a lane's highest bit are not kept).
__device__ __forceinline__ double pow_by_squaring(double q, int32_t n)
{
    double acc = 1.0;
    while (__ballot(n > 0) != 0) {
        acc = n & 1 ? acc * q : acc;
        q = q * q;
        acc = n & 2 ? acc * q : acc;
        q = q * q;
        n >>= 2;
    }
    return acc;
}

// The walk u -= P(x), P(x + 1) = P(x) ((n + 1) p / (q (x + 1)) - p / q) runs
// four steps at a time: the four ratios do not depend on the walk, so their
// latencies overlap, and only a compare, a subtraction and a product per
// step are serial.  The lanes of a wavefront walk in step, so x + 1 .. x + 4
// are uniform.  A lane whose walk has ended keeps its values, since u <= P
// stays true.  Ratios past x = n are never kept: x > n starts again.
template <class Rng>
__device__ __forceinline__ int32_t binomial_inversion(int32_t n, double p, Rng &rng)
{
    const double q = 1.0 - p;
    const double odds = p / q;
    const double np1_odds = (double)(n + 1) * odds;
    const double p_zero = pow_by_squaring(q, n);
    for (;;) {
        double u = rng.uniform();
        double pk = p_zero;
        int32_t x = 0;
        for (int32_t base = 1; __ballot(u > pk && x <= n) != 0; base += 4) {
            double ratio[4];
            if (base == 1) {
                ratio[0] = np1_odds - odds;
                ratio[1] = np1_odds * 0.5 - odds;
                ratio[2] = divide_by_whole(np1_odds, 3.0, 1.0 / 3.0) - odds;
                ratio[3] = np1_odds * 0.25 - odds;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double xj = (double)(base + j);
                    ratio[j] = divide_by_whole(np1_odds, xj, reciprocal_near(xj)) - odds;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool go = u > pk;
                u = go ? u - pk : u;
                pk = go ? pk * ratio[j] : pk;
                x += go ? 1 : 0;
            }
        }
        if (x <= n) return x;
    }
}

// Binomial(1, p) as binomial_inversion (after the reflection) draws it.  Its
// walk ends at 0 for u <= q and at 1 for u - q <= q RN(p / q), which is p but
// for rounding: only draws within a few ulp of 1 need the quotient, and start
// again if they pass it.
template <class Rng>
__device__ __forceinline__ bool bernoulli_as_binomial(double p, Rng &rng)
{
    if (p <= 0.0) return false;
    if (p >= 1.0) return true;
    const bool reflect = p > 0.5;
    const double pp = reflect ? 1.0 - p : p;
    const double q = 1.0 - pp;
    for (;;) {
        const double u = rng.uniform();
        if (!(u > q)) return reflect;
        const double rest = u - q;
        if (rest <= pp * (1.0 - 0x1p-50) || rest <= q * (pp / q)) return !reflect;
    }
}

// Stirling-series remainder ln k! - ((k + 1/2) ln(k + 1) - (k + 1) + ln(2 pi)/2):
// correctly rounded values for k <= 9, the series 1/12 - 1/360 + 1/1260 in
// 1/(k+1) beyond.
__constant__ const double kStirlingExact[10] = {
    0x1.4c071bcda0a5bp-4, 0x1.52a9b923ea649p-5, 0x1.c579a268d80b3p-6, 0x1.54a2662fd78a9p-6,
    0x1.10b4e513fcbedp-6, 0x1.c6b167bebdf36p-7, 0x1.85d4d612e4a86p-7, 0x1.552805e7b3076p-7,
    0x1.2f4871b12ab64p-7, 0x1.10f9d4c0743a7p-7,
};

__device__ __forceinline__ double stirling_tail(int32_t k)
{
    if (k < 10) return kStirlingExact[k];
    const double v = 1.0 / (double)(k + 1);
    const double v2 = v * v;
    return (1.0 / 12.0 - (1.0 / 360.0 - (1.0 / 1260.0) * v2) * v2) * v;
}

// One pass of BTRD's rejection: true and *x on acceptance.
template <class Rng>
__device__ __forceinline__ bool btrd_pass(int32_t n, double p, Rng &rng, int32_t *x)
{
    const double nd = (double)n;
    const double q = 1.0 - p;
    const double npq = (nd * p) * q;
    const double spq = sqrt(npq);
    const double b = 1.15 + 2.53 * spq;
    const double a = (-0.0873 + 0.0248 * b) + 0.01 * p;
    const double c = nd * p + 0.5;
    const double vr = 0.92 - 4.2 / b;
    const double urvr = 0.86 * vr;
    double v = rng.uniform();
    const bool box = v <= urvr;  // inside the box: accept at once
    double u;
    if (box) {
        u = v / vr - 0.43;
    } else {
        const double draw = rng.uniform();
        if (v >= vr) {
            u = draw - 0.5;
        } else {
            u = v / vr - 0.93;
            u = (u < 0.0 ? -0.5 : 0.5) - u;
            v = draw * vr;
        }
    }
    const double us = 0.5 - fabs(u);
    const double kd = floor(((2.0 * a) / us + b) * u + c);
    if (kd < 0.0 || kd > nd) return false;
    *x = (int32_t)kd;
    if (box) return true;
    const double alpha = (2.83 + 5.1 / b) * spq;
    v = v * alpha / (a / (us * us) + b);
    const double mode = floor((nd + 1.0) * p);
    const double r = p / q;
    const double km = fabs(kd - mode);
    if (km <= 15.0) {
        // ratio f(k)/f(mode) by the recurrence f(i)/f(i-1) = nr/i - r: from
        // the mode up, multiplied up from 1, or from k up to the mode,
        // multiplied into v.  Four ratios at a time (they are independent).
        const double nr = (nd + 1.0) * r;
        const bool up = mode < kd;
        const double low = up ? mode : kd;
        const int32_t steps = (int32_t)km;
        double f = up ? 1.0 : v;
        for (int32_t i = 0; __ballot(i < steps) != 0; i += 4) {
            double ratio[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double ij = low + (double)(i + j + 1);
                ratio[j] = divide_by_whole(nr, ij, reciprocal_near(ij)) - r;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) f = i + j < steps ? f * ratio[j] : f;
        }
        return up ? v <= f : f <= 1.0;
    }
    v = log_basic(v);
    const double rho = (km / npq) * (((km / 3.0 + 0.625) * km + 1.0 / 6.0) / npq + 0.5);
    const double t = -(km * km) / (2.0 * npq);
    if (v < t - rho) return true;
    if (v > t + rho) return false;
    const int32_t m_i = (int32_t)mode, k_i = (int32_t)kd;
    const double nm = nd - mode + 1.0;
    const double h = (mode + 0.5) * log_basic((mode + 1.0) / (r * nm)) + stirling_tail(m_i) + stirling_tail(n - m_i);
    const double nk = nd - kd + 1.0;
    return v <= h + (nd + 1.0) * log_basic(nm / nk) + (kd + 0.5) * log_basic(nk * r / (kd + 1.0)) -
                    stirling_tail(k_i) - stirling_tail(n - k_i);
}

// ---------------------------------------------------------------------------
// Steps 3.2-3.3 for one species of one tet: n = min(Binomial(ni, zeta), Ns)
// molecules leave and are split over the interior faces (Sec. II.B).  Below
// the threshold (10 in the paper): one categorical draw per molecule against
// the running sum of the weights, the last interior face closing the
// interval; otherwise
// n_i = Binomial(n - sum_{j<i} n_j, w_i / (1 - sum_{j<i} w_j)) face by face,
// the last interior face taking what is left (a single interior face takes
// everything without a draw), so that weight 3 is read by the scaled form only.
//
// scaled (ANY_SCALED instances; the alternative at the end of Sec. II.B): the
// whole population ni is split at once with weights zeta w_i, and a molecule
// that draws no face stays; if more than Ns would leave, the Ns present are
// split as above.  1.0 * w == w exactly, so the plain split is the same there.
//
// The thinning and the faces' binomials share one loop: each pass draws once
// (one inversion, or one attempt of BTRD's rejection) and a lane that accepts
// goes on to its next binomial in the next pass, whatever the others do.  A
// wavefront then runs as many passes as its slowest lane needs in all, not
// the sum over the binomials of each one's slowest lane, and the samplers are
// in the code once instead of five times (the update kernel 41 -> 21 KB).
// Bound: the serial chain of one lane.  A bar of 1080 tets holding 93
// molecules each took 64.7 us per period with one binomial after the other
// and 41.5 us with this loop (queue-based one-launch path); tets of a few
// molecules draw once or twice and took the same (the 750-tet cube 14.9 and
// 14.7 us, the 384,000-tet batch 0.2373 and 0.2373 ms).  Returns n, and
// out[].
// ---------------------------------------------------------------------------
template <bool ANY_SCALED, class Rng>
__device__ __forceinline__ int32_t leave_and_split(int32_t ni, int32_t Ns, double zeta, bool scaled,
                                                   const int32_t nbr[4], const double weights[4],
                                                   int32_t threshold, Rng &rng, int32_t out[4])
{
    // scalars, selected by face: an index into the arrays would put them in memory
    const double w0 = weights[0], w1 = weights[1], w2 = weights[2], w3 = weights[3];
    const uint32_t faces = (nbr[0] >= 0 ? 1u : 0u) | (nbr[1] >= 0 ? 2u : 0u) | (nbr[2] >= 0 ? 4u : 0u) |
                           (nbr[3] >= 0 ? 8u : 0u);  // the interior ones
    const int interior = __popc(faces), last = 31 - __clz((int)faces);
    bool thin = !(ANY_SCALED && scaled);
    int32_t n = ni;
    int32_t o0, o1, o2, o3;
    const auto add = [&](int k, int32_t m) {
        o0 += k == 0 ? m : 0;
        o1 += k == 1 ? m : 0;
        o2 += k == 2 ? m : 0;
        o3 += k == 3 ? m : 0;
    };
    for (;;) {
        const bool all = !(ANY_SCALED && scaled);  // every molecule of n leaves
        const double z = all ? 1.0 : zeta;
        o0 = o1 = o2 = o3 = 0;
        int f = -1;
        int32_t left = n;
        double taken = 0.0;
        double p = zeta;
        bool draw = thin || (n >= threshold && n > 0 && interior > (all ? 1 : 0));
        bool face = !thin;  // the next thing to do is to pick a face
        if (thin && __ballot(ni > 1) == 0) {
            // no lane holds more than one molecule: a single Bernoulli draw
            n = ni > 0 && Ns > 0 && bernoulli_as_binomial(zeta, rng) ? 1 : 0;
            draw = n >= threshold && n > 0 && interior > 1;
            left = n;
            face = true;
        }
        while (__ballot(draw) != 0) {
            if (!draw) continue;
            if (face) {
                // the next interior face and its probability
                const uint32_t rest = f < 0 ? faces : faces & (0xfffffffeu << f);
                f = rest ? __builtin_ctz(rest) : 4;
                if (f > last || left == 0 || (all && f == last)) {
                    if (all) add(last, left);
                    draw = false;
                    continue;
                }
                const double wf = f == 0 ? w0 : f == 1 ? w1 : f == 2 ? w2 : w3;
                p = (z * wf) / (1.0 - taken);
                if (p > 1.0) p = 1.0;
                taken = taken + z * wf;
            }
            int32_t x = 0;
            bool accepted = true;
            if (left > 0 && p > 0.0) {
                if (p >= 1.0) {
                    x = left;
                } else {
                    const bool reflect = p > 0.5;
                    const double pp = reflect ? 1.0 - p : p;
                    if ((double)left * pp < 10.0)
                        x = binomial_inversion(left, pp, rng);
                    else
                        accepted = btrd_pass(left, pp, rng, &x);
                    if (reflect) x = left - x;
                }
            }
            face = accepted;
            if (!accepted) continue;
            if (f < 0) {  // the thinning
                n = x < Ns ? x : Ns;
                left = n;
                draw = n >= threshold && n > 0 && interior > 1;
            } else {
                add(f, x);
                left -= x;
            }
        }
        if (n > 0 && all && interior == 1) {
            add(last, n);
        } else if (n > 0 && n < threshold && interior > 0) {
            // a face's interval ends at the running sum of the weights; a draw
            // past them all closes on the last face, or stays (scaled).  The
            // sums do not fall, so the draws below each of them give the
            // faces' shares by differences: a compare and an addition a face
            // and draw, a quarter of what finding each draw's face takes (the
            // 750-tet cube 6.1 to 5.2 us per period)
            const uint32_t drawn = all ? faces & ~(1u << last) : faces;
            const double e0 = drawn & 1u ? z * w0 : 0.0, e1 = drawn & 2u ? e0 + z * w1 : e0,
                         e2 = drawn & 4u ? e1 + z * w2 : e1, e3 = drawn & 8u ? e2 + z * w3 : e2;
            int32_t c0 = 0, c1 = 0, c2 = 0, c3 = 0;
            for (int32_t i = 0; i < n; ++i) {
                const double u = rng.uniform();
                c0 += u < e0 ? 1 : 0;
                c1 += u < e1 ? 1 : 0;
                c2 += u < e2 ? 1 : 0;
                c3 += u < e3 ? 1 : 0;
            }
            o0 = c0;
            o1 = c1 - c0;
            o2 = c2 - c1;
            o3 = c3 - c2;
            if (all) add(last, n - c3);
        }
        out[0] = o0;
        out[1] = o1;
        out[2] = o2;
        out[3] = o3;
        if (all) return n;
        const int32_t moved = (o0 + o1) + (o2 + o3);
        if (moved <= Ns) return moved;
        n = Ns;  // more would leave than are present: those present, split in the plain form
        scaled = false;
    }
}

}  // namespace rdos
