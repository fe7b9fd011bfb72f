// One cell's share of a period (Algorithm 1, Steps 2-3): the arithmetic that
// every step kernel runs, whatever memory its counts live in.
//
// A kernel's per-lane state is a `Cell`: n(s) the count of species s, occ(s)
// and last(s) its occupancy integral and the time of its last change (both
// meaningful only for species an event touched).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rdos_internal.h"
#include "rdos_sampling.h"

#pragma clang fp contract(off)

namespace rdos {

typedef int32_t v4i __attribute__((ext_vector_type(4)));

// A pointer into device (global) memory.  Accesses through generic pointers
// become flat instructions, which also count against the scalar-load wait
// counter, so a wait for a scalar load would wait for them too.
template <typename T>
using gptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ gptr<T> global(T *p)
{
    return (gptr<T>)p;
}

// propensity a_r = c_r h_r of reaction q with the tet's counts (mass action);
// zero where the reaction is not allowed in tet t (bit q of its `allowed`
// word).  The counts are tested first, and the tet's N_A V and allowed word
// are read from memory only when they matter: most tets hold no reactant
// pair, and then their update does not wait for those loads.
template <class Cell>
__device__ __forceinline__ double propensity(const DevSim &sm, int q, const Cell &c, const MeshRec *mr, int32_t t)
{
    const int order = sm.rn[q];
    double h;
    if (order == 0) {
        h = 1.0;
    } else {
        const int32_t na = c.n(sm.r0[q]);
        if (order == 1) {
            h = (double)na;
        } else if (sm.r0[q] == sm.r1[q]) {
            h = (double)na * (double)(na - 1);
        } else {
            h = (double)na * (double)c.n(sm.r1[q]);
        }
    }
    if (h == 0.0) return 0.0;  // c_r * 0 == 0 for every finite c_r
    if (sm.allowed && !((sm.allowed[t] >> q) & 1u)) return 0.0;
    if (order == 1) return sm.k[q] * h;
    const double nav = mr->nav;
    const double k = order == 0 ? sm.k[q] * nav : sm.k[q] / nav;
    return k * h;
}

// Step 2: Gillespie direct method over [0, tau_k); the first event at or past
// tau_k is discarded.  Step 2.1: on each event the occupancy integral of
// every reactant and product is brought up to the event time.  Returns the
// species some event touched: occ and last of the others stand for 0 and
// are never stored.
template <class Cell>
__device__ __forceinline__ uint32_t cell_ssa(const DevSim &sm, const MeshRec *mr, int32_t t, uint32_t period32,
                                             double tau_k, uint32_t key1, const Cell &ls)
{
    const int S = sm.S;
    const int R = sm.R;
    uint32_t touched = 0;
    Stream ssa(sm.key0, key1, kSsaStream, (uint32_t)t, period32);
    double now = 0.0;
    for (uint32_t events = 0;; ++events) {
        if (events >= kMaxEventsPerPeriod) {  // runaway rates: stop and report, never hang
            atomicOr(sm.flags, 2);
            break;
        }
        double a0 = 0.0;
        for (int q = 0; q < R; ++q) a0 = a0 + propensity(sm, q, ls, mr, t);
        if (!(a0 > 0.0)) break;
        const double dt = -log_basic(1.0 - ssa.uniform()) / a0;
        if (now + dt >= tau_k) break;
        now = now + dt;
        const double x = ssa.uniform() * a0;
        int chosen = -1;
        double cum = 0.0;
        for (int q = 0; q < R; ++q) {
            cum = cum + propensity(sm, q, ls, mr, t);
            if (x < cum) {
                chosen = q;
                break;
            }
        }
        if (chosen < 0) {  // x rounded up to a0: the last reaction able to fire
            for (int q = R - 1; q >= 0; --q)
                if (propensity(sm, q, ls, mr, t) > 0.0) {
                    chosen = q;
                    break;
                }
        }
        // the chosen reaction's fields, read with a wavefront-uniform index
        // (scalar loads) and selected per lane
        uint32_t inv = 0;
        int a = -1, b = -1, c0 = -1, c1 = -1, c2 = -1;
        for (int q = 0; q < R; ++q) {
            const int rn = sm.rn[q], pn = sm.pn[q];
            const bool is = q == chosen;
            inv = is ? sm.involved[q] : inv;
            a = is && rn > 0 ? sm.r0[q] : a;
            b = is && rn > 1 ? sm.r1[q] : b;
            c0 = is && pn > 0 ? sm.p0[q] : c0;
            c1 = is && pn > 1 ? sm.p1[q] : c1;
            c2 = is && pn > 2 ? sm.p2[q] : c2;
        }
        for (int s = 0; s < S; ++s) {
            if (!((inv >> s) & 1u)) continue;
            const bool seen = (touched >> s) & 1u;
            const double o = seen ? ls.occ(s) : 0.0;
            const double l = seen ? ls.last(s) : 0.0;
            int32_t &ns = ls.n(s);
            ls.occ(s) = o + (double)ns * (now - l);
            ls.last(s) = now;
            ns += (int)(s == c0) + (int)(s == c1) + (int)(s == c2) - (int)(s == a) - (int)(s == b);
            if (ns > 0x3fffffff) atomicOr(sm.flags, 1);
        }
        touched |= inv;
    }
    return touched;
}

// eq. 2: the time-mean population of a species that events touched, Ns its
// count at the end of the period.
template <class Cell>
__device__ __forceinline__ double mean_occupancy(const Cell &ls, int s, int32_t Ns, double tau_k)
{
    return (ls.occ(s) + (double)Ns * (tau_k - ls.last(s))) / tau_k;
}

}  // namespace rdos
