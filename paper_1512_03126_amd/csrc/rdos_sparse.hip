// Periods of Algorithm 1 for batches of sparsely occupied realizations: one
// block per realization keeps its occupied (tet, species) pairs in a hash
// table in LDS for a whole run of periods.
//
// Why: over the queue a period of such a batch is bound by lines, not by
// molecules: at 2% occupancy nearly every count, occupancy byte, queue entry
// and atomic has a line of memory to itself, and the atomics run at the memory
// side.  A realization of 384,000 tets and 7,600 molecules has 61 KB of keys
// and counts; its table of 16,384 slots fits one compute unit, so a batch of
// 256 of them fills the device and a period touches memory only for the mesh
// records of the occupied tets and for the block's own lists (streamed, read
// back by the same block).
//   * A period: list the table's pairs; where two species share a tet, or one
//     reacts alone, look the tet's counts up and list the tet for the SSA;
//     clear the table; draw every listed pair's transfers (64 pairs per
//     wavefront and turn, the SSA's lanes in the first wavefronts meanwhile)
//     and add them to the emptied table.
//   * The state in memory is left as it is until the run ends; then a second
//     kernel writes the final states back, unless some table was full: then
//     no realization has moved, and the caller runs the periods otherwise.
// What bounds it: vector instructions of the drawing loop (about 500 per
// wavefront of 64 pairs, four wavefronts per SIMD) and its gathers of mesh
// records.  Cycles per period of one 384,000-tet realization (7,600 pairs):
// list 14,000, lookups 10,000, clear 2,000, draws 66,000, waits 5,000.  With
// linear probing and a species at a time the lookups took 36,000 and the
// listing 26,000.
// Measured, us per period over the queue and here: 256 + 64 realizations of
// 384,000 and 48,000 tets 228 and 63; 128 of 384,000 109 and 46; 600 of
// 48,000 72 and 25.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "rdos_block.h"
#include "rdos_internal.h"

#pragma clang fp contract(off)

namespace rdos {

namespace {

typedef uint32_t v2u __attribute__((ext_vector_type(2)));

struct SparseHead {
    double D[kMaxSpecies];
    BlockReaction rx[kMaxReactions];
    int32_t n_pairs;     // pairs listed for Step 3
    int32_t n_maybe;     // pairs whose tet may react
    int32_t n_ssa;       // tets listed for the SSA
    int32_t n_fire;      // those with an event in the period
    int32_t next;        // pairs handed out to wavefronts
    int32_t n_start;     // pairs of the run's first state
    int32_t failed;      // the table is full
    int32_t n_heavy;     // listed pairs of several molecules
};
static_assert(sizeof(SparseHead) == kSparseHeadBytes, "LDS head");

// A (tet, species) pair: species in the high bits, tet + 1 below (never 0).
__device__ __forceinline__ uint32_t pair_key(int s, uint32_t t) { return ((uint32_t)s << kSparseTetBits) | (t + 1u); }
__device__ __forceinline__ uint32_t key_tet(uint32_t key) { return (key & ((1u << kSparseTetBits) - 1u)) - 1u; }
__device__ __forceinline__ int key_species(uint32_t key) { return (int)(key >> kSparseTetBits); }

constexpr int kMaxProbes = 512;

// Open addressing with double hashing (linear probing's clusters cost the
// wavefront its worst lane: 2.5 times as long lookups at half load): slot h
// holds {key (0: empty), count}.  `seen` and `many` are one-hash filters over
// tets: a tet whose bit in `many` is clear holds one species at most.
struct SparseTable {
    uint32_t *slot;
    uint32_t size;
    uint32_t *seen, *many;
    int bit_shift;  // 32 - log2 of the bits in `seen`

    __device__ __forceinline__ uint32_t tet_bit(uint32_t t) const { return (t * 0x85EBCA6Bu) >> bit_shift; }
    __device__ __forceinline__ bool crowded(uint32_t t) const
    {
        const uint32_t b = tet_bit(t) >> 1;
        return (many[b >> 5] >> (b & 31u)) & 1u;
    }
    __device__ __forceinline__ uint32_t home(uint32_t key) const { return __umulhi(key * 0x9E3779B1u, size); }
    __device__ __forceinline__ uint32_t next(uint32_t h, uint32_t key) const
    {
        h += ((key * 0xC2B2AE35u) >> 20) | 1u;  // below 4096, the smallest table
        return h >= size ? h - size : h;
    }
    // Adds c molecules; false when no room was found.
    __device__ __forceinline__ bool add(uint32_t key, int32_t c, uint32_t t, bool track) const
    {
        uint32_t h = home(key);
#pragma unroll 1
        for (int tries = 0; tries < kMaxProbes; ++tries) {
            const uint32_t old = atomicCAS(&slot[2 * h], 0u, key);
            if (old == 0u || old == key) {
                atomicAdd(reinterpret_cast<int32_t *>(&slot[2 * h + 1]), c);
                if (old == 0u && track) {
                    const uint32_t b = tet_bit(t), bit = 1u << (b & 31u), half = b >> 1;
                    if (atomicOr(&seen[b >> 5], bit) & bit) atomicOr(&many[half >> 5], 1u << (half & 31u));
                }
                return true;
            }
            h = next(h, key);
        }
        return false;
    }
    // The counts of four species of a tet, s0 .. s0 + 3 (those past the last
    // are looked up too, and absent): four probes in flight, and the
    // wavefront waits for the longest of the lookups, not for each in turn.
    __device__ __forceinline__ void counts(int s0, uint32_t t, int32_t c[4]) const
    {
        uint32_t key[4], h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            key[j] = pair_key(s0 + j, t);
            h[j] = home(key[j]);
            c[j] = 0;
        }
        uint32_t open = 15u;
#pragma unroll 1
        for (int tries = 0; tries < kMaxProbes && __ballot(open != 0) != 0; ++tries) {
            uint32_t k[4];
            int32_t v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                k[j] = slot[2 * h[j]];
                v[j] = (int32_t)slot[2 * h[j] + 1];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool mine = ((open >> j) & 1u) && k[j] == key[j];
                c[j] = mine ? v[j] : c[j];
                if (mine || k[j] == 0u) open &= ~(1u << j);
                h[j] = next(h[j], key[j]);
            }
        }
    }
};

// A wavefront's entries in a list that the block fills.
__device__ __forceinline__ int32_t append_one(bool active, int32_t *count)
{
    int32_t total;
    const int32_t before = wave_prefix(active ? 1u : 0u, 1, &total);
    return total > 0 ? before + reserve(count, total) : 0;
}

}  // namespace

// n_periods periods of unit blockIdx.x (a realization), the iterations
// iter0 .. of its simulation.  Reads the state in memory and leaves it as it
// is; the state after the run goes to the unit's pair list
// (launch_sparse_commit writes it back), or *fail is raised.
template <bool ANY_SCALED>
__global__ __launch_bounds__(kSparseMaxThreads) void sparse_kernel(const DevSim *__restrict__ sims,
                                                                const WorkUnit *__restrict__ units, int64_t iter0,
                                                                int32_t n_periods, SparsePlan plan)
{
    extern __shared__ __align__(16) unsigned char lds[];
    SparseHead &head = *reinterpret_cast<SparseHead *>(lds);
    const int32_t tid = (int32_t)threadIdx.x, lane = (int32_t)__lane_id(), nt = (int32_t)blockDim.x;
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WorkUnit un = units[blockIdx.x];
    using ConstSim = const __attribute__((address_space(4))) DevSim;
    ConstSim *desc = (ConstSim *)sims + un.sim;
    const DevSim &sm0 = *(const DevSim *)desc;
    const int32_t S = sm0.S, R = sm0.R, T = sm0.T;
    const int64_t first = sm0.step0 + iter0;
    const int32_t Tp = (T + 3) & ~3;
    const uint32_t key1 = sm0.key1 ^ (uint32_t)un.realization;

    SparseTable table;
    table.slot = reinterpret_cast<uint32_t *>(lds + kSparseHeadBytes);
    table.size = (uint32_t)plan.slots;
    table.seen = table.slot + 2 * plan.slots;
    table.many = table.seen + 2 * plan.filter_words;
    table.bit_shift = __builtin_clz((uint32_t)plan.filter_words) - 5;  // 2 x 32 bits a word of `many`
    // the SSA's lane state: counts [S], then occ, last, c, a
    const int32_t lanes = plan.lanes;
    double *lane_state = reinterpret_cast<double *>(table.many + plan.filter_words);
    int32_t *lane_counts = reinterpret_cast<int32_t *>(lane_state + 2 * (S + R) * lanes);
    const bool track = R > 0 && S > 1;

    // the unit's lists in memory
    char *mem = plan.scratch + (int64_t)blockIdx.x * plan.unit_bytes;
    const gptr<v2u> pairs = (gptr<v2u>)mem;                                 // [slots] {key, count}
    const gptr<v2u> maybe = (gptr<v2u>)(mem + 8 * (int64_t)plan.slots);     // [slots]
    const gptr<uint32_t> start = (gptr<uint32_t>)(mem + 16 * (int64_t)plan.slots);  // [slots] key
    const gptr<int32_t> ssa = (gptr<int32_t>)(mem + 20 * (int64_t)plan.slots);  // [slots][1 + S] tet, counts
    const gptr<int32_t> after =                                                 // [waves][64 S][3]
        (gptr<int32_t>)(mem + (24 + 4 * (int64_t)S) * plan.slots) + (int64_t)wave * 64 * S * 3;

    if (tid < S) head.D[tid] = sm0.D[tid];
    if (tid < R) head.rx[tid] = pack_reaction(sm0, tid);
    if (tid == 0) head.n_pairs = head.n_maybe = head.n_ssa = head.n_fire = head.next = head.n_start = head.failed = head.n_heavy = 0;
    const auto clear_table = [&]() {
        v4i *p = reinterpret_cast<v4i *>(table.slot);
        for (int32_t i = tid; i < plan.slots / 2 + 3 * plan.filter_words / 4; i += nt) p[i] = v4i{0, 0, 0, 0};
    };
    clear_table();
    __syncthreads();

    // the state of period `first`
    {
        const int32_t words = (T + 15) >> 4;
        const gptr<const uint8_t> marks =
            global((const uint8_t *)sm0.mask[first & 1]) + (int64_t)un.realization * S * sm0.mstride;
        const gptr<const int32_t> src =
            global((const int32_t *)sm0.buf[first & 1]) + (int64_t)un.realization * S * Tp;
        const uint32_t tag = occupancy_tag(first);
        for (int32_t s = 0; s < S; ++s)
            for (int32_t w = tid; w < words; w += nt) {
                const uint32_t m = *(gptr<const uint32_t>)(marks + (int64_t)s * sm0.mstride + 4 * w);
                for (int b = 0; b < 4; ++b) {
                    if (((m >> (8 * b)) & 0xffu) != tag) continue;
                    const int32_t t = 16 * w + 4 * b;
                    const v4i c = *(gptr<const v4i>)(src + s * Tp + t);
                    for (int i = 0; i < 4; ++i) {
                        const int32_t n = i == 0 ? c.x : i == 1 ? c.y : i == 2 ? c.z : c.w;
                        if (n == 0) continue;
                        const uint32_t key = pair_key(s, (uint32_t)(t + i));
                        const int32_t at = atomicAdd(&head.n_start, 1);
                        if (at >= plan.slots || !table.add(key, n, (uint32_t)(t + i), track))
                            head.failed = 1;
                        else
                            start[at] = key;
                    }
                }
            }
    }
    __syncthreads();

    // Pairs of one molecule are listed from the front, others from the back: a
    // wavefront of single molecules draws once per lane, without the loops of
    // the samplers (us per period without and with: 100 realizations of 93,750
    // tets at 0.03 molecules per species and tet 40.4 and 37.8, 256 of 384,000
    // at 0.01 51.7 and 51.0).
    const auto list_pair = [&](bool active, const v2u &e) {
        const bool heavy = active && (int32_t)e.y > 1;
        const int32_t at = append_one(active && !heavy, &head.n_pairs);
        if (active && !heavy) pairs[at] = e;
        if (__ballot(heavy) == 0) return;
        const int32_t back = append_one(heavy, &head.n_heavy);
        if (heavy) pairs[plan.slots - 1 - back] = e;
    };

    // species that react alone, and in pairs of themselves
    uint32_t alone = 0, twins = 0;
    for (int q = 0; q < R; ++q) {
        if (sm0.rn[q] == 1) alone |= 1u << sm0.r0[q];
        if (sm0.rn[q] == 2 && sm0.r0[q] == sm0.r1[q]) twins |= 1u << sm0.r0[q];
    }

    // the species each reaction needs, reaction q's in lane q
    const uint32_t need_of_lane = lane < R ? head.rx[lane].needed() : 0u;

    for (int32_t k = 0;; ++k) {
        if (head.failed) {  // uniform over the block
            if (tid == 0) atomicOr(plan.fail, 1u);
            return;
        }
        ConstSim *now = desc;
        asm volatile("" : "+s"(now));
        const DevSim &sm = *(const DevSim *)now;
        const bool last = k == n_periods;
        const uint32_t period32 = (uint32_t)(first + k);
        const double tau_k = sm.tau;

        // List the pairs: those of tets where nothing can react go to `pairs`
        // (after the last period all do), the others to `maybe`.  Four slots
        // per lane and round, without branches: half the slots are empty.
        for (int32_t h0 = 0; h0 < plan.slots; h0 += 4 * nt) {
            const int32_t h = h0 + 4 * tid;
            const v4i a = *reinterpret_cast<const v4i *>(table.slot + 2 * h);
            const v4i b = *reinterpret_cast<const v4i *>(table.slot + 2 * h + 4);
            const uint32_t key[4] = {(uint32_t)a.x, (uint32_t)a.z, (uint32_t)b.x, (uint32_t)b.z};
            const int32_t cnt[4] = {a.y, a.w, b.y, b.w};
            // a count wrapped by an overflowing addition is reported, and dropped
            if ((cnt[0] | cnt[1] | cnt[2] | cnt[3]) < 0) atomicOr(sm.flags, 1);
            uint32_t held = 0, can = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) held |= (uint32_t)(cnt[j] > 0) << j;
            if (R > 0 && !last) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int s = key_species(key[j]) & 31;
                    uint32_t c = (alone >> s) & 1u;
                    c |= cnt[j] > 1 ? (twins >> s) & 1u : 0u;
                    if (track) c |= (uint32_t)table.crowded(key_tet(key[j]));
                    can |= c << j;
                }
                can &= held;
            }
            uint32_t plain = held & ~can, heavy = 0;
            if (!last) {
#pragma unroll
                for (int j = 0; j < 4; ++j) heavy |= (uint32_t)(cnt[j] > 1) << j;
                heavy &= plain;
                plain &= ~heavy;
            }
            int32_t total;
            int32_t at = wave_prefix(__popc(plain), 3, &total);
            if (total > 0) {
                at += reserve(&head.n_pairs, total);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((plain >> j) & 1u) pairs[at + __popc(plain & ((1u << j) - 1u))] = v2u{key[j], (uint32_t)cnt[j]};
            }
            if (__ballot(heavy != 0) != 0) {
                at = wave_prefix(__popc(heavy), 3, &total);
                at = plan.slots - 1 - at - reserve(&head.n_heavy, total);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((heavy >> j) & 1u) pairs[at--] = v2u{key[j], (uint32_t)cnt[j]};
            }
            if (__ballot(can != 0) != 0) {
                at = wave_prefix(__popc(can), 3, &total);
                at += reserve(&head.n_maybe, total);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((can >> j) & 1u) maybe[at++] = v2u{key[j], (uint32_t)cnt[j]};
            }
        }
        __syncthreads();
        if (last) break;

        // The tets of `maybe`: where some reaction's reactants are present the
        // lane of the lowest species lists the tet, with its counts, for the
        // SSA; elsewhere each lane lists its pair.
        const int32_t n_maybe = head.n_maybe;
        for (int32_t j0 = 0; j0 < n_maybe; j0 += nt) {
            const int32_t j = j0 + tid;
            bool can = false, owner = true;
            v2u e = v2u{0, 0};
            uint32_t t = 0;
            int32_t c[4] = {0, 0, 0, 0};  // the tet's counts of the first four species
            if (j < n_maybe) {
                e = maybe[j];
                t = key_tet(e.x);
                const int s = key_species(e.x);
                uint32_t held = 1u << s;
#pragma unroll
                for (int q = 0; q < 4; ++q) c[q] = q == s ? (int32_t)e.y : 0;
                if (track && table.crowded(t))
                    for (int q0 = 0; q0 < S; q0 += 4) {
                        int32_t d[4];
                        table.counts(q0, t, d);
#pragma unroll
                        for (int q = 0; q < 4; ++q) held |= (uint32_t)(d[q] > 0) << (q0 + q);
                        if (q0 == 0) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) c[q] = d[q];
                        }
                    }
                owner = (held & ((1u << s) - 1u)) == 0u;
                const uint32_t allowed = sm.allowed ? sm.allowed[t] : 0xffffffffu;
                for (int q = 0; q < R; ++q) {
                    const uint32_t need = __builtin_amdgcn_readlane(need_of_lane, q);
                    can |= ((allowed >> q) & 1u) && (held & need) == need;
                }
            }
            int32_t at;
            list_pair(j < n_maybe && !can, e);
            const bool lead = j < n_maybe && can && owner;
            if (__ballot(lead) == 0) continue;
            at = append_one(lead, &head.n_ssa);
            if (lead) {
                const gptr<int32_t> p = ssa + (int64_t)at * (1 + S);
                p[0] = (int32_t)t;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (q < S) p[1 + q] = c[q];
                for (int q0 = 4; q0 < S; q0 += 4) {
                    table.counts(q0, t, c);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (q0 + q < S) p[1 + q0 + q] = c[q];
                }
            }
        }
        __syncthreads();
        int32_t n_ssa = head.n_ssa;
        clear_table();
        // A few tets go to the SSA's lanes as they are, while the other
        // wavefronts work on.  Of many (an abundant species with a slow
        // first-order reaction) the block first sorts out those whose first
        // event, as the SSA draws it, falls past the period: nothing reacts
        // there, and their pairs join the list.
        const bool sorted_out = n_ssa > 2 * lanes;  // uniform over the block
        if (sorted_out) {
            for (int32_t j0 = 0; j0 < n_ssa; j0 += nt) {
                const int32_t j = j0 + tid;
                const gptr<const int32_t> p = (gptr<const int32_t>)ssa + (int64_t)j * (1 + S);
                bool fire = false;
                uint32_t t = 0;
                if (j < n_ssa) {
                    t = (uint32_t)p[0];
                    const double nav = sm.mesh[t].nav;
                    const uint32_t allowed = sm.allowed ? sm.allowed[t] : 0xffffffffu;
                    double a0 = 0.0;
                    for (int q = 0; q < R; ++q) {
                        const BlockReaction x = head.rx[q];
                        const int32_t na = p[1 + x.species(0)];
                        double h = (double)na, c = x.k;
                        if (x.order() == 2) {
                            h = h * (double)(x.species(0) == x.species(1) ? na - 1 : p[1 + x.species(1)]);
                            c = x.k / nav;
                        }
                        a0 = a0 + (h == 0.0 || !((allowed >> q) & 1u) ? 0.0 : c * h);
                    }
                    if (a0 > 0.0) {
                        Stream rng(sm.key0, key1, kSsaStream, t, period32);
                        fire = -log_basic(1.0 - rng.uniform()) / a0 < tau_k;
                    }
                }
                for (int s = 0; s < S; ++s) {
                    const int32_t c = j < n_ssa && !fire ? p[1 + s] : 0;
                    list_pair(c > 0, v2u{pair_key(s, t), (uint32_t)c});
                }
                const int32_t at = append_one(fire, &head.n_fire);
                if (fire) maybe[at] = v2u{(uint32_t)j, 0u};
            }
        }
        __syncthreads();
        if (sorted_out) n_ssa = head.n_fire;

        // Step 3 (and Step 2 before it, in the first wavefronts): the next
        // state fills the table.  Pairs are handed out 64 at a time (a fixed
        // share per wavefront left the block waiting for its slowest, 14,000
        // cycles against 4,600 of a period's 110,000; reading pairs and mesh
        // records a round ahead gained nothing, as the loop is bound by
        // instructions).
        const int32_t n_pairs = head.n_pairs, n_heavy = head.n_heavy, heavies = (n_heavy + 63) & ~63;
        const int32_t ssa_waves = lanes / 64;
        int32_t tet0 = wave < ssa_waves ? 64 * wave : n_ssa;  // this wavefront's next tets for the SSA
        int32_t n_after = 0, at_after = 0;                    // and the pairs its last ones left
        for (;;) {
            uint32_t key = 0, code = 0;
            int32_t Ns = 0;
            if (at_after < n_after) {
                const int32_t j = at_after + lane;
                at_after += 64;
                if (j < n_after) {
                    key = (uint32_t)after[3 * j];
                    Ns = after[3 * j + 1];
                    code = (uint32_t)after[3 * j + 2];
                }
            } else if (tet0 < n_ssa) {
                const int32_t j = tet0 + lane;
                tet0 += 64 * ssa_waves;
                n_after = at_after = 0;
                uint32_t held = 0, touched = 0;
                int32_t t = 0;
                const BlockCell cell{lane_counts + tid, lane_state + tid, lanes, lanes, S, R};
                if (j < n_ssa) {
                    const int32_t i = sorted_out ? (int32_t)maybe[j].x : j;
                    const gptr<const int32_t> p = (gptr<const int32_t>)ssa + (int64_t)i * (1 + S);
                    t = p[0];
                    for (int s = 0; s < S; ++s) cell.n(s) = p[1 + s];
                    touched = block_ssa(sm, head.rx, t, period32, tau_k, key1, cell);
                    for (int s = 0; s < S; ++s) held |= (uint32_t)(cell.n(s) > 0) << s;
                }
                // eq. 2 and the stochastic rounding of the touched species
                for (int s = 0; s < S; ++s) {
                    int32_t total;
                    const bool here = (held >> s) & 1u;
                    const int32_t before = wave_prefix(here ? 1u : 0u, 1, &total);
                    if (here) {
                        const int32_t n = cell.n(s);
                        uint32_t c = (uint32_t)n;
                        if (((touched & sm.diff_mask) >> s) & 1u && !sm.first_order) {
                            const double nbar = mean_occupancy(cell, s, n, tau_k);
                            int32_t ni = (int32_t)floor(nbar);
                            const double frac = nbar - (double)ni;
                            c = 0u;
                            if (frac > 0.0) {
                                Stream rng(sm.key0, key1, (uint32_t)s, (uint32_t)t, period32);
                                if (rng.uniform() < frac) ni += 1;
                                c = 0x80000000u;
                            }
                            c |= (uint32_t)ni;
                        }
                        const int32_t i = 3 * (n_after + before);
                        after[i] = (int32_t)pair_key(s, (uint32_t)t);
                        after[i + 1] = n;
                        after[i + 2] = (int32_t)c;
                    }
                    n_after += total;
                }
                // read back by other lanes of this wavefront
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                continue;
            } else {
                int32_t j = 0;
                if (lane == 0) j = atomicAdd(&head.next, 64);
                j = __builtin_amdgcn_readfirstlane(j);
                if (j >= heavies + n_pairs) break;
                const bool first_ones = j < heavies;  // those of several molecules take longest
                j += lane - (first_ones ? 0 : heavies);
                if (j < (first_ones ? n_heavy : n_pairs)) {
                    const v2u e = pairs[first_ones ? plan.slots - 1 - j : j];
                    key = e.x;
                    Ns = (int32_t)e.y;
                    code = e.y;
                }
            }
            if (key == 0) continue;
            const uint32_t t = key_tet(key);
            const int s = key_species(key);
            int32_t out[4] = {0, 0, 0, 0};
            int32_t nb[4] = {0, 0, 0, 0};
            int32_t stay = Ns;
            if ((sm.diff_mask >> s) & 1u) {
                const MeshRec *mr = sm.mesh + t;
                const int4 n4 = *reinterpret_cast<const int4 *>(mr->nbr);
                nb[0] = n4.x;
                nb[1] = n4.y;
                nb[2] = n4.z;
                nb[3] = n4.w;
                const double w[4] = {mr->w[0], mr->w[1], mr->w[2], ANY_SCALED ? mr->w3 : 0.0};
                const double g = mr->g;
                PrimedStream rng(sm.key0, key1, (uint32_t)s, t, period32);
                const int32_t ni = (int32_t)(code & 0x7fffffffu);
                if (code >> 31) (void)rng.uniform();  // the rounding's draw
                double zeta = (tau_k * head.D[s]) * g;
                if (zeta > 1.0) zeta = 1.0;
                const int32_t n = leave_and_split<ANY_SCALED>(ni, Ns, zeta, sm.transfer_form == 1, nb, w,
                                                              sm.split_threshold, rng, out);
                stay = Ns - n;
            }
            // one destination per round: as many rounds as the busiest lane has
#pragma unroll 1
            for (uint32_t left = (stay > 0 ? 16u : 0u) | (out[0] > 0 ? 1u : 0u) | (out[1] > 0 ? 2u : 0u) |
                                 (out[2] > 0 ? 4u : 0u) | (out[3] > 0 ? 8u : 0u);
                 left; left &= left - 1u) {
                const int f = __builtin_ctz(left);
                const uint32_t u = f == 4 ? t : (uint32_t)(f == 0 ? nb[0] : f == 1 ? nb[1] : f == 2 ? nb[2] : nb[3]);
                const int32_t c = f == 4 ? stay : f == 0 ? out[0] : f == 1 ? out[1] : f == 2 ? out[2] : out[3];
                if (!table.add(pair_key(s, u), c, u, track)) head.failed = 1;
            }
        }
        __syncthreads();
        if (tid == 0) head.n_pairs = head.n_heavy = head.n_maybe = head.n_ssa = head.n_fire = head.next = 0;
        __syncthreads();
    }
    if (tid == 0) {
        plan.counts[2 * blockIdx.x] = head.n_start;
        plan.counts[2 * blockIdx.x + 1] = head.n_pairs;
    }
}

// Writes the runs' final states back (one block per unit), unless a unit of
// the launch failed: then every unit's state stays as it was before the run.
__global__ __launch_bounds__(kSparseMaxThreads) void sparse_commit_kernel(const DevSim *__restrict__ sims,
                                                                       const WorkUnit *__restrict__ units,
                                                                       int64_t iter0, int32_t n_periods,
                                                                       SparsePlan plan)
{
    if (*plan.fail != 0u) return;
    const WorkUnit un = units[blockIdx.x];
    const DevSim &sm = sims[un.sim];
    const int32_t Tp = (sm.T + 3) & ~3;
    const int64_t first = sm.step0 + iter0, end = first + n_periods;
    const char *mem = plan.scratch + (int64_t)blockIdx.x * plan.unit_bytes;
    const gptr<const v2u> pairs = (gptr<const v2u>)mem;
    const gptr<const uint32_t> start = (gptr<const uint32_t>)(mem + 16 * (int64_t)plan.slots);
    const int64_t base = (int64_t)un.realization * sm.S * Tp;
    const gptr<int32_t> from = global(sm.buf[first & 1]) + base;
    const gptr<int32_t> to = global(sm.buf[end & 1]) + base;
    const gptr<uint8_t> marks = global(sm.mask[end & 1]) + (int64_t)un.realization * sm.S * sm.mstride;
    const int32_t n0 = plan.counts[2 * blockIdx.x], n1 = plan.counts[2 * blockIdx.x + 1];
    for (int32_t j = threadIdx.x; j < n0; j += blockDim.x)
        from[(int64_t)key_species(start[j]) * Tp + key_tet(start[j])] = 0;
    // the zeros reach memory before counts are written over them
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const uint8_t mark = occupancy_tag(end);
    for (int32_t j = threadIdx.x; j < n1; j += blockDim.x) {
        const v2u e = pairs[j];
        const uint32_t t = key_tet(e.x);
        const int s = key_species(e.x);
        to[(int64_t)s * Tp + t] = (int32_t)e.y;
        marks[(int64_t)s * sm.mstride + (t >> 2)] = mark;
    }
}

hipError_t launch_sparse(const DevSim *sims, const WorkUnit *units, int64_t iter0, int32_t n_periods,
                         const SparsePlan &plan, hipStream_t st)
{
    if (plan.units < 1 || n_periods < 1 || plan.lds_bytes > kResidentLdsMax || plan.threads < 64 ||
        plan.threads > kSparseMaxThreads || plan.slots % (4 * plan.threads) != 0)
        return hipErrorInvalidValue;
    if (plan.scaled)
        sparse_kernel<true><<<plan.units, plan.threads, plan.lds_bytes, st>>>(sims, units, iter0, n_periods, plan);
    else
        sparse_kernel<false><<<plan.units, plan.threads, plan.lds_bytes, st>>>(sims, units, iter0, n_periods, plan);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    sparse_commit_kernel<<<plan.units, kSparseMaxThreads, 0, st>>>(sims, units, iter0, n_periods, plan);
    return hipGetLastError();
}

bool sparse_shape(int32_t S, int32_t R, int64_t pairs, bool many_units, SparsePlan *plan)
{
    const int32_t lane = R > 0 ? resident_lane_bytes(S, R) + 4 * S : 0;
    // 16,384 slots at most: 20,480 do not fit beside the head
    for (int32_t step = 1; step <= 4; ++step) {
        const int32_t slots = 4096 * step;
        if (pairs > slots * 6 / 10) continue;
        // the filters: some 16 bits of `seen` a pair where they fit
        int32_t filter = R > 0 && S > 1 ? (step == 1 ? 512 : 2048) : 4;
        if (kSparseHeadBytes + 8 * slots + 12 * filter + 64 * lane > kResidentLdsMax) filter = min(filter, 1024);
        const int32_t fixed = kSparseHeadBytes + 8 * slots + 12 * filter;
        if (fixed + 64 * lane > kResidentLdsMax) break;
        plan->slots = slots;
        plan->filter_words = filter;
        // blocks of a quarter of the wavefronts share a compute unit where
        // there are more units than it takes to give each its own
        plan->threads = step == 1 && many_units ? 256 : kSparseMaxThreads;
        const int32_t budget = plan->threads == 256 ? kResidentLdsMax / 4 : kResidentLdsMax;
        plan->lanes = R > 0 ? max(64, min(min(plan->threads, 256), ((budget - fixed) / lane) & ~63)) : 0;
        plan->lds_bytes = fixed + plan->lanes * lane;
        // pairs, maybe, start, tets for the SSA, pairs after the SSA
        plan->unit_bytes = ((24 + 4 * (int64_t)S) * slots + 12 * (int64_t)S * plan->lanes + 255) & ~(int64_t)255;
        return true;
    }
    return false;
}

}  // namespace rdos
