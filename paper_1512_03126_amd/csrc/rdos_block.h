// What the kernels that keep counts in LDS share: reactions packed for LDS,
// the SSA of one lane's tet, and lists filled by wavefronts.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rdos_cell.h"
#include "rdos_internal.h"

#pragma clang fp contract(off)

namespace rdos {

// A reaction as the SSA reads it: one 16-byte LDS load.
struct alignas(16) BlockReaction {
    double k;
    uint32_t shape;   // order, then five bits each: r0, r1, p0, p1, p2 (kNoSpecies: none)
    uint32_t masks;   // low half: species involved; high half: species that must be present
    static constexpr uint32_t kNoSpecies = 31;
    __device__ __forceinline__ int order() const { return (int)(shape & 3u); }
    __device__ __forceinline__ int species(int i) const { return (int)((shape >> (2 + 5 * i)) & 31u); }
    __device__ __forceinline__ uint32_t involved() const { return masks & 0xffffu; }
    __device__ __forceinline__ uint32_t needed() const { return masks >> 16; }
};

__device__ __forceinline__ uint32_t pack_species(int32_t n, int i, int32_t id)
{
    return (i < n ? (uint32_t)id : BlockReaction::kNoSpecies);
}

__device__ __forceinline__ BlockReaction pack_reaction(const DevSim &sm, int q)
{
    BlockReaction r;
    const int32_t rn = sm.rn[q], pn = sm.pn[q];
    const uint32_t a = pack_species(rn, 0, sm.r0[q]), b = pack_species(rn, 1, sm.r1[q]);
    r.k = sm.k[q];
    r.shape = (uint32_t)rn | (a << 2) | (b << 7) | (pack_species(pn, 0, sm.p0[q]) << 12) |
              (pack_species(pn, 1, sm.p1[q]) << 17) | (pack_species(pn, 2, sm.p2[q]) << 22);
    r.masks = sm.involved[q] | ((rn > 0 ? 1u << a : 0u) | (rn > 1 ? 1u << b : 0u)) << 16;
    return r;
}

// One lane's tet in the SSA: its counts are the block's own, the rest belongs
// to the lane.
struct BlockCell {
    int32_t *N;
    double *lane;      // occ[S], last[S], c[R], a[R], `lanes` apart
    int32_t stride;    // between species of N
    int32_t lanes;
    int32_t S, R;
    __device__ __forceinline__ int32_t &n(int s) const { return N[s * stride]; }
    __device__ __forceinline__ double &occ(int s) const { return lane[s * lanes]; }
    __device__ __forceinline__ double &last(int s) const { return lane[(S + s) * lanes]; }
    __device__ __forceinline__ double &c(int q) const { return lane[(2 * S + q) * lanes]; }
    __device__ __forceinline__ double &a(int q) const { return lane[(2 * S + R + q) * lanes]; }
};

// Step 2 for one tet (as cell_ssa, the same operations in the same order):
// the constants c_r are computed once for the tet, when their reactants are
// first present, the propensities of an event are kept for the choice of its
// reaction, and a reaction's fields come from LDS in one load.  Returns the species some event touched.
__device__ __forceinline__ uint32_t block_ssa(const DevSim &sm, const BlockReaction *rx, int32_t t,
                                                 uint32_t period32, double tau_k, uint32_t key1,
                                                 const BlockCell &cell)
{
    const int R = cell.R;
    const double nav = sm.mesh[t].nav;  // waited for where a constant needs it
    const uint32_t allowed = sm.allowed ? sm.allowed[t] : 0xffffffffu;
    uint32_t touched = 0, known = 0;    // known: reactions whose constant c_r has been computed
    PrimedStream ssa(sm.key0, key1, kSsaStream, (uint32_t)t, period32);
    double now = 0.0;
    for (uint32_t events = 0;; ++events) {
        if (events >= kMaxEventsPerPeriod) {  // runaway rates: stop and report, never hang
            atomicOr(sm.flags, 2);
            break;
        }
        double a0 = 0.0;
        for (int q0 = 0; q0 < R; q0 += 2) {  // two at a time, their loads in flight together
            double a[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int q = min(q0 + j, R - 1);
                const BlockReaction x = rx[q];
                const int order = x.order();
                const int32_t na = cell.n(order > 0 ? x.species(0) : 0);
                const int32_t nb = cell.n(order > 1 ? x.species(1) : 0);
                double h = order > 0 ? (double)na : 1.0;
                if (order == 2) h = h * (double)(x.species(0) == x.species(1) ? na - 1 : nb);
                a[j] = 0.0;
                if (h != 0.0) {
                    double c;
                    if ((known >> q) & 1u) {
                        c = cell.c(q);
                    } else {
                        c = order == 1 ? x.k : (order == 0 ? x.k * nav : x.k / nav);
                        if (!((allowed >> q) & 1u)) c = 0.0;
                        cell.c(q) = c;
                        known |= 1u << q;
                    }
                    a[j] = c * h;
                }
                cell.a(q) = a[j];
            }
            a0 = a0 + a[0];
            if (q0 + 1 < R) a0 = a0 + a[1];
        }
        if (!(a0 > 0.0)) break;
        // -ln(1 - u) >= u: no event before tau_k where u / a0 reaches it with
        // more to spare than the roundings of dt and now + dt take.  That is
        // most tets of a period, and then the logarithm and the division are
        // not waited for (with the constants computed only where needed:
        // 384,000 tets of four species 11.9 to 11.4 us per period)
        const double u = ssa.uniform();
        if (u > (tau_k - now) * a0 * (1.0 + 0x1p-30)) break;
        const double dt = -log_basic(1.0 - u) / a0;
        if (now + dt >= tau_k) break;
        now = now + dt;
        const double x = ssa.uniform() * a0;
        int chosen = -1;
        double cum = 0.0;
        for (int q = 0; q < R; ++q) {
            cum = cum + cell.a(q);
            if (x < cum) {
                chosen = q;
                break;
            }
        }
        if (chosen < 0) {  // x rounded up to a0: the last reaction able to fire
            for (int q = R - 1; q >= 0; --q)
                if (cell.a(q) > 0.0) {
                    chosen = q;
                    break;
                }
        }
        const BlockReaction r = rx[chosen];
        for (uint32_t inv = r.involved(); inv; inv &= inv - 1u) {
            const int s = __builtin_ctz(inv);
            const bool seen = (touched >> s) & 1u;
            const double o = seen ? cell.occ(s) : 0.0;
            const double l = seen ? cell.last(s) : 0.0;
            int32_t ns = cell.n(s);
            cell.occ(s) = o + (double)ns * (now - l);
            cell.last(s) = now;
            ns += (int)(s == r.species(2)) + (int)(s == r.species(3)) + (int)(s == r.species(4)) -
                  (int)(s == r.species(0)) - (int)(s == r.species(1));
            cell.n(s) = ns;
            if (ns > 0x3fffffff) atomicOr(sm.flags, 1);
        }
        touched |= r.involved();
    }
    return touched;
}

// The lanes' exclusive prefix sum of v (v < 2^bits), and the total.
__device__ __forceinline__ int32_t wave_prefix(uint32_t v, int bits, int32_t *total)
{
    int32_t before = 0, sum = 0;
    for (int k = 0; k < bits; ++k) {
        const uint64_t plane = __ballot((v >> k) & 1u);
        before += (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(plane >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)plane, 0u))
                  << k;
        sum += __popcll(plane) << k;
    }
    *total = sum;
    return before;
}

// Room for `total` entries of a block's list (one LDS atomic for the lanes
// that are here).
__device__ __forceinline__ int32_t reserve(int32_t *count, int32_t total)
{
    int32_t base = 0;
    const int32_t lane = (int32_t)__lane_id();
    if (lane == __builtin_amdgcn_readfirstlane(lane)) base = atomicAdd(count, total);
    return __builtin_amdgcn_readfirstlane(base);
}

}  // namespace rdos
