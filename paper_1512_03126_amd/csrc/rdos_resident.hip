// Periods of Algorithm 1 with the state held in LDS: one launch runs a whole
// run of periods, each block keeping the counts of its own tets in LDS.
//
// What bounds it: the serial chain of a period in one block, about ten cycles
// per instruction with a wavefront or two per SIMD.  The two-launch path pays
// two launches and five dependent trips to memory on top of the same chain,
// and one lane per tet works its species in turn; here the counts never leave
// LDS, a lane takes a (tet, species) pair (the SSA, which couples the
// species, runs before, one lane per tet), and only molecules that cross into
// another block's tets go through memory.
//   * Split.  A realization is cut into as many blocks as the device holds at
//     once (16 tets at least): crowded tets gain from every split (1080 tets
//     of 93 molecules: 64, 33, 27, 23.5 us per period with 1, 8, 34 and 68
//     blocks), sparse ones hardly lose (the 750-tet cube 6.0 us with one
//     block, 6.5 with 47; 384,000 tets at 2% occupancy 10.2 us with 128
//     blocks, 9.4 with 256).  Realizations beyond that run one block each,
//     up to eight on a compute unit.
//   * Exchange.  Arrivals from other blocks are added to the realization's
//     own count buffer of the next period (all zero until then) by agent-scope
//     atomics; a block publishes the period it has finished, waits for the
//     blocks that share a face with it only, and moves what arrived into LDS.
//     Waiting for every block cost 4.1 us per period on the 384,000-tet mesh,
//     waiting for neighbours 2.5.  Nothing else is written during a run, so
//     no cache has to be written back: all shared words are read and written
//     by agent-scope atomics.
//   * Layout.  Full: two count buffers in LDS and lists with room for every
//     pair.  Where a block's tets need more than that, short: one buffer (the
//     counts of listed pairs are taken out before any molecule moves) and
//     lists with room for a part of its tets, which hold nearly twice as many
//     tets, and slower where both fit (384,000 tets at 2%: full 8.7, short 9.4
//     us per period).  A period whose pairs overflow short lists is
//     worked through in parts, every addition through memory.
//   * Diffusion alone, in blocks with a lane for every pair (EVERY): nothing is
//     listed, an empty pair's lane idles.  The 750-tet cube 5.2 and 4.7 us per
//     period with the list and without, a bar of 192 tets 3.9 and 3.2.
//   * The list pass is bound by its instructions on large blocks (a wavefront
//     takes 256 tets): a group's occupancy is one word with four bits per
//     species, which a reaction tests for four tets at once (5,000 tets of
//     three species in a block: 9,300 cycles with a word per tet, 7,200 so).
//   * Two count buffers alternate by parity, as in memory.  A neighbour adds
//     to the buffer of period k + 2 only after this block has published
//     period k + 1, by when it has emptied that buffer of period k's arrivals.
// Measured, us per period, two launches (or the queue-based one launch) and
// this kernel: 750-tet cube 14.4 and 4.7; 1080-tet bar at 93 molecules per
// tet 41.5 and 22.9; ten species on that bar 105 and 21.8; 600 realizations of
// the cube with production 26 and 8.4; 384,000 tets at 2% 14.8 and 8.5, with a
// fourth species and jitter 20.3 and 11.3; 162,000 tets at 30 molecules per
// species and tet 292 and 104.  Short layout: 998,250 tets of four species at
// 0.03 and 0.1 molecules per tet 23.3 and 15.5, 43.9 and 24.7; 16 realizations
// of 80,400 triangles 28 and 14.2.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "rdos_block.h"
#include "rdos_internal.h"

#pragma clang fp contract(off)

namespace rdos {

namespace {

// Block-wide LDS words before the arrays (see resident_lds_bytes).
struct ResidentHead {
    double D[kMaxSpecies];
    BlockReaction rx[kMaxReactions];
    int32_t n_ssa;    // tets listed for the SSA
    int32_t n_pairs;  // (tet, species) pairs listed for Step 3
    int32_t stop;     // a wait for other blocks failed
    int32_t spills;   // periods in which short lists overflowed
};
static_assert(sizeof(ResidentHead) == kResidentHeadBytes, "LDS head");

// What was added through memory to four tets: read, and moved into the block's
// counts d.
struct Arrivals {
    gptr<unsigned long long> p;
    unsigned long long lo, hi;
    __device__ __forceinline__ explicit Arrivals(gptr<unsigned long long> at)
        : p(at), lo(__hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)),
          hi(__hip_atomic_load(at + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    {
    }
    __device__ __forceinline__ void take(int32_t *d) const
    {
        if ((lo | hi) == 0) return;
        __hip_atomic_store(p, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p + 1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        d[0] += (int32_t)(uint32_t)lo;
        d[1] += (int32_t)(uint32_t)(lo >> 32);
        d[2] += (int32_t)(uint32_t)hi;
        d[3] += (int32_t)(uint32_t)(hi >> 32);
    }
};

// Adds n molecules to tet t in the count buffer of `period`, and marks its
// four-tet group.
__device__ __forceinline__ void add_in_memory(const DevSim &sm, int64_t period, int64_t base, int64_t mbase,
                                              int64_t Tp, int32_t s, int32_t t, int32_t n, bool mark)
{
    const gptr<int32_t> next = global(sm.buf[period & 1]) + base;
    __hip_atomic_fetch_add(next + (uint32_t)(s * (int32_t)Tp + t), n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!mark) return;
    const gptr<uint8_t> marks = global(sm.mask[period & 1]) + mbase;
    __hip_atomic_store(marks + (uint32_t)(s * sm.mstride + (t >> 2)), occupancy_tag(period), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// Blocks of up to this many four-tet groups (over all species) read every
// group for arrivals; larger ones read the occupancy bytes first.
constexpr int32_t kDirectGroups = 2048;

// Waits until every neighbouring block has published `target` (first
// wavefront; each lane watches one of them, mine, and any beyond 64 in turn).
// Bounded: a wait past its limit raises *fail, which ends every other wait.
constexpr uint32_t kWaitSpins = 1u << 28;  // minutes: a neighbour may be deep in a long SSA
__device__ __forceinline__ bool wait_neighbours(const unsigned long long *done, const uint16_t *list, int32_t n,
                                                int32_t mine, unsigned long long target, uint32_t *fail)
{
    const int32_t lane = (int32_t)__lane_id();
    for (uint32_t spins = 0;; ++spins) {
        bool all = lane >= n || __hip_atomic_load(&done[(int64_t)mine * kResidentFlagStride], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT) >= target;
        for (int32_t j = lane + 64; j < n; j += 64)
            all &= __hip_atomic_load(&done[(int64_t)list[j] * kResidentFlagStride], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT) >= target;
        if (__ballot(!all) == 0) return true;
        if ((spins & 63u) == 63u) {
            if (__hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) return false;
            if (spins > kWaitSpins) {
                if (lane == 0) atomicOr(fail, 1u);
                return false;
            }
        }
    }
}

}  // namespace

// Fills parts[blockIdx.x] from the realization it belongs to, its list of
// neighbours (the blocks that hold a face neighbour of one of its tets: their
// places among the realization's blocks, plan.max_parts entries per block)
// and its period counter.
__global__ __launch_bounds__(256) void resident_layout_kernel(const DevSim *__restrict__ sims,
                                                              const ResidentUnit *__restrict__ units,
                                                              int32_t n_units, ResidentUnit same, ResidentPlan plan)
{
    __shared__ uint32_t seen[kResidentMaxParts / 32];
    __shared__ int32_t n;
    const int32_t b = (int32_t)blockIdx.x;
    ResidentUnit u = same;  // one simulation: its realizations are cut alike
    if (units) {            // the last unit that starts at or before this block
        int32_t lo = 0, hi = n_units - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (units[mid].first <= b)
                lo = mid;
            else
                hi = mid - 1;
        }
        u = units[lo];
    } else {
        u.realization = b / u.blocks;
        u.first = u.realization * u.blocks;
    }
    ResidentPart pt{};
    pt.sim = u.sim;
    pt.realization = u.realization;
    pt.part = b - u.first;
    pt.parts = u.blocks;
    pt.stride = u.len;
    pt.t0 = pt.part * u.len;
    pt.len = min(u.len, u.T - pt.t0);
    pt.flag0 = u.first;
    for (int k = threadIdx.x; k < kResidentMaxParts / 32; k += blockDim.x) seen[k] = 0;
    if (threadIdx.x == 0) n = 0;
    __syncthreads();
    if (u.blocks > 1) {
        const MeshRec *mesh = sims[u.sim].mesh;
        for (int32_t i = threadIdx.x; i < pt.len; i += blockDim.x) {
            const int4 nb = *reinterpret_cast<const int4 *>(mesh[pt.t0 + i].nbr);
            const int32_t other[4] = {nb.x, nb.y, nb.z, nb.w};
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                if (other[f] < 0 || (uint32_t)(other[f] - pt.t0) < (uint32_t)pt.len) continue;
                const int32_t q = other[f] / u.len;
                atomicOr(&seen[q >> 5], 1u << (q & 31));
            }
        }
        __syncthreads();
        for (int32_t q = threadIdx.x; q < u.blocks; q += blockDim.x)
            if ((seen[q >> 5] >> (q & 31)) & 1u)
                plan.neighbours[(int64_t)b * plan.max_parts + atomicAdd(&n, 1)] = (uint16_t)q;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        pt.neighbours = n;
        plan.parts[b] = pt;
        plan.done[(int64_t)b * kResidentFlagStride] = 0;
        if (b == 0) plan.done[(int64_t)plan.blocks * kResidentFlagStride] = 0;  // both words
    }
}

hipError_t launch_resident_layout(const DevSim *sims, const ResidentPlan &plan, const ResidentUnit *units,
                                  int32_t n_units, const ResidentUnit &same, hipStream_t st)
{
    if (plan.blocks < 1) return hipErrorInvalidValue;
    resident_layout_kernel<<<plan.blocks, 256, 0, st>>>(sims, units, n_units, same, plan);
    return hipGetLastError();
}

size_t resident_plan_bytes(int64_t blocks, int64_t max_parts)
{
    return (size_t)blocks * (sizeof(ResidentPart) + kResidentFlagStride * sizeof(unsigned long long)) + 128 +
           (max_parts > 1 ? (size_t)blocks * max_parts * sizeof(uint16_t) : 0);
}

void resident_place(ResidentPlan *plan, void *memory)
{
    char *p = static_cast<char *>(memory);
    plan->done = reinterpret_cast<unsigned long long *>(p);  // the counters, then the failure word
    p += (size_t)plan->blocks * kResidentFlagStride * sizeof(unsigned long long) + 128;
    plan->parts = reinterpret_cast<ResidentPart *>(p);
    p += (size_t)plan->blocks * sizeof(ResidentPart);
    plan->neighbours = plan->max_parts > 1 ? reinterpret_cast<uint16_t *>(p) : nullptr;
}

// n_periods periods of the block's part (parts[blockIdx.x]) of one
// realization, the iterations iter0 .. of its simulation.
template <bool ANY_SCALED, bool FULL, bool EVERY>
__global__ __launch_bounds__(kResidentMaxThreads) void resident_kernel(
    const DevSim *__restrict__ sims, const ResidentPart *__restrict__ parts,
    const uint16_t *__restrict__ neighbours, int32_t max_parts, int64_t iter0, int32_t n_periods, int64_t partial,
    double tau_last, unsigned long long *done_all, unsigned long long epoch, uint32_t *fail, int32_t lds_bytes,
    LaunchEnd launch_end)
{
    extern __shared__ __align__(16) unsigned char lds[];
    ResidentHead &head = *reinterpret_cast<ResidentHead *>(lds);
    const int32_t tid = (int32_t)threadIdx.x, nt = (int32_t)blockDim.x;
    const ResidentPart pt = parts[blockIdx.x];
    using ConstSim = const __attribute__((address_space(4))) DevSim;
    ConstSim *desc = (ConstSim *)sims + pt.sim;
    const DevSim &sm = *(const DevSim *)desc;
    const int32_t S = sm.S, R = sm.R;
    const int64_t first = sm.step0 + iter0;
    const int64_t left = sm.step_end - first;
    if (left <= 0) {  // uniform over the unit's blocks
        end_block(fail + 1, launch_end);
        return;
    }
    if (left < n_periods) n_periods = (int32_t)left;

    const int32_t len = pt.len, t0 = pt.t0;
    const int32_t ls = (len + 3) & ~3;  // stride between species rows
    const int32_t P = S * ls;
    const uint32_t per_species = (uint32_t)(0xffffffffu / (uint32_t)ls + 1u);  // e / ls == umulhi(e, per_species)
    const int32_t range = FULL ? ls : resident_range(S, R, ls, lds_bytes);  // tets the lists are sure to hold
    const int32_t room = S * range;                                         // pairs
    const int32_t used = resident_lds_bytes(S, R, ls, FULL, range, 0);
    const int32_t lanes = resident_lanes(S, R, lds_bytes, used, nt);
    int32_t *counts = reinterpret_cast<int32_t *>(lds + kResidentHeadBytes);  // [2][P] or [P]
    int32_t *taken = counts + (FULL ? 2 : 1) * P;  // [room] short: counts of the listed pairs from the nt-th on
    int32_t *pop = taken + (FULL ? 0 : room);      // [room] rounded mean populations of the pairs the SSA listed
    uint16_t *list = reinterpret_cast<uint16_t *>(pop + (R > 0 ? room : 0));  // [room] pairs
    uint16_t *ssa_list = list + room;              // [range] tets
    double *lane_state = reinterpret_cast<double *>(lds + used);

    const int64_t Tp = ((int64_t)sm.T + 3) & ~(int64_t)3;
    const int64_t base = (int64_t)pt.realization * S * Tp;
    const int64_t mbase = (int64_t)pt.realization * S * sm.mstride;
    const uint32_t key1 = sm.key1 ^ (uint32_t)pt.realization;
    const bool alone = pt.parts == 1;
    const bool direct = S * ((pt.stride + 3) / 4) <= kDirectGroups;
    unsigned long long *done = done_all + (int64_t)pt.flag0 * kResidentFlagStride;
    const uint16_t *nlist = neighbours + (int64_t)blockIdx.x * max_parts;
    const int32_t my_neighbour = !alone && tid < 64 && tid < pt.neighbours ? nlist[tid] : 0;

    if (tid < S) head.D[tid] = sm.D[tid];
    if (tid < R) head.rx[tid] = pack_reaction(sm, tid);
    if (tid == 0) head.n_ssa = head.n_pairs = head.stop = head.spills = 0;
    {
        const gptr<int32_t> src = global(sm.buf[first & 1]) + base + t0;
        for (int32_t v = tid; v < P / 4; v += nt) {
            const int32_t s = (int32_t)__umulhi(4u * (uint32_t)v, per_species);
            const gptr<v4i> p = (gptr<v4i>)(src + s * Tp + (4 * v - s * ls));
            *reinterpret_cast<v4i *>(counts + 4 * v) = *p;
            if (FULL) *reinterpret_cast<v4i *>(counts + P + 4 * v) = v4i{0, 0, 0, 0};
            if (!alone || !FULL) {  // additions through memory reach this buffer from the second period on
                const gptr<unsigned long long> z = (gptr<unsigned long long>)p;
                __hip_atomic_store(z, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(z + 1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if (!FULL) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the buffer is empty before additions to it
    __syncthreads();

    // the reactants of reaction q in lane q, as shifts of a group's occupancy
    // (four bits per species); a reaction without reactants: bit 16
    uint32_t reactants = 0;
    if ((int32_t)__lane_id() < R) {
        const BlockReaction x = head.rx[__lane_id()];
        const int a = x.order() > 0 ? x.species(0) : 0, b = x.order() > 1 ? x.species(1) : a;
        reactants = x.order() > 0 ? (uint32_t)(4 * a) | (uint32_t)(4 * b) << 8 : 1u << 16;
    }

    for (int32_t k = 0; k < n_periods; ++k) {
        // read the descriptor's fields in the period that uses them: held
        // across the loop they are more than the scalar registers hold
        ConstSim *now = desc;
        asm volatile("" : "+s"(now));
        const DevSim &sm = *(const DevSim *)now;
        const int64_t period = first + k;
        const uint32_t period32 = (uint32_t)period;
        const double tau_k = period == partial ? tau_last : sm.tau;
        int32_t *cur = FULL ? counts + (k & 1) * P : counts;
        int32_t *nxt = FULL ? counts + ((k & 1) ^ 1) * P : counts;
        bool spill = false;  // short lists that would overflow

        for (int32_t from = 0, to = ls; from < ls;) {
            // List the tets where a reaction's reactants are all present, and
            // the (tet, species) pairs that hold molecules in the others.  A
            // lane takes the four tets of a group, every species (one 16-byte
            // LDS load each).
            for (int32_t i0 = from; i0 < to && !EVERY; i0 += 4 * nt) {
                const int32_t i = i0 + 4 * tid;
                uint64_t held = 0;  // bit 4 s + b: species s in tet i + b
                if (i < to) {
                    int32_t sign = 0;
                    const auto group = [&sign](const v4i &c) {
                        sign |= c.x | c.y | c.z | c.w;
                        return min((uint32_t)c.x, 1u) | min((uint32_t)c.y, 1u) << 1 | min((uint32_t)c.z, 1u) << 2 |
                               min((uint32_t)c.w, 1u) << 3;
                    };
                    int s0 = 0;
                    for (; s0 + 1 < S; s0 += 4) {  // four loads in flight; past the last species it repeats
                        v4i c[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            c[j] = *reinterpret_cast<const v4i *>(cur + min(s0 + j, S - 1) * ls + i);
                        uint32_t four = 0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) four |= group(c[j]) << 4 * (min(s0 + j, S - 1) - s0);
                        held |= (uint64_t)four << 4 * s0;
                    }
                    if (s0 < S) held |= (uint64_t)group(*reinterpret_cast<const v4i *>(cur + s0 * ls + i)) << 4 * s0;
                    if (sign < 0) {  // a count wrapped by an overflowing addition: reported, and dropped
                        atomicOr(sm.flags, 1);
                        for (int s = 0; s < S; ++s)
                            for (int b = 0; b < 4; ++b) cur[s * ls + i + b] = max(cur[s * ls + i + b], 0);
                    }
                }
                if (__ballot(held != 0) == 0 && !sm.zeroth) continue;  // uniform over the wavefront
                int32_t total;
                if (R > 0) {
                    uint32_t fire = 0;  // the tets where some reaction may
                    if (!sm.allowed) {
                        for (int q = 0; q < R; ++q) {
                            const uint32_t x = __builtin_amdgcn_readlane(reactants, q);
                            fire |= ((uint32_t)(held >> (x & 63u)) & (uint32_t)(held >> (x >> 8 & 63u))) |
                                    (x >> 16 ? 15u : 0u);
                        }
                    } else {
                        for (int q = 0; q < R; ++q) {
                            const uint32_t x = __builtin_amdgcn_readlane(reactants, q);
                            const uint32_t f = ((uint32_t)(held >> (x & 63u)) & (uint32_t)(held >> (x >> 8 & 63u))) |
                                               (x >> 16 ? 15u : 0u);
                            for (int b = 0; b < 4; ++b)
                                if ((f >> b & 1u) && i + b < len) fire |= (sm.allowed[t0 + i + b] >> q & 1u) << b;
                        }
                    }
                    fire &= (1u << min(max(min(len, to) - i, 0), 4)) - 1u;
                    const int32_t at = wave_prefix(__popc(fire), 3, &total);
                    if (total > 0) {
                        held &= ~(0x1111111111111111ull * fire);  // the SSA's lane lists them
                        int32_t j = at + reserve(&head.n_ssa, total);
                        for (; fire; fire &= fire - 1u, ++j)
                            if (FULL || j < range) ssa_list[j] = (uint16_t)(i + __builtin_ctz(fire));
                    }
                }
                int32_t at = wave_prefix(__popcll(held), 32 - __builtin_clz(4 * S), &total);
                if (total > 0) {
                    at += reserve(&head.n_pairs, total);
                    const auto put = [&](uint32_t m, int s0) {
                        for (; m; m &= m - 1u, ++at) {
                            const int32_t bit = __builtin_ctz(m);
                            if (FULL || at < room) list[at] = (uint16_t)((s0 + (bit >> 2)) * ls + i + (bit & 3));
                        }
                    };
                    put((uint32_t)held, 0);
                    if (S > 8) put((uint32_t)(held >> 32), 8);
                }
            }
            if (!EVERY) __syncthreads();
            int32_t n_ssa = head.n_ssa;
            if (!FULL && to - from > range) {
                // over the whole range with short lists: where the pairs may
                // not fit, go on in parts, every addition through memory
                spill = n_ssa > range || head.n_pairs + S * n_ssa > room;
                __syncthreads();  // all have read the lengths before the SSA adds to them
                if (spill) {      // uniform over the block
                    if (tid == 0) {
                        head.n_ssa = head.n_pairs = 0;
                        head.spills += 1;
                    }
                    __syncthreads();
                    to = range;
                    continue;
                }
            }
            n_ssa = min(n_ssa, range);

            // Step 2
            if (R > 0) {
                if (n_ssa > 0) {  // uniform over the block
                    for (int32_t j = tid; j < n_ssa && tid < lanes; j += lanes) {
                        const int32_t i = ssa_list[j], t = t0 + i;
                        const BlockCell cell{cur + i, lane_state + tid, ls, lanes, S, R};
                        const uint32_t touched = block_ssa(sm, head.rx, t, period32, tau_k, key1, cell);
                        // its pairs, the wavefront's species by species: lanes
                        // of Step 3 that share a species draw alike (162,000
                        // tets at 30 molecules per species and tet: 150,000
                        // cycles for Step 3 in the order of the tets, 118,000
                        // so).  Touched: eq. 2 and the stochastic rounding;
                        // bit 31 of the count tells Step 3 to take them from
                        // pop[].
                        uint32_t held = 0;
                        int32_t total = 0;  // of the lanes that are here
                        for (int s = 0; s < S; ++s) {
                            const bool here = cell.n(s) > 0;
                            held |= (uint32_t)here << s;
                            total += (int32_t)__popcll(__ballot(here));
                        }
                        int32_t next_at = reserve(&head.n_pairs, total);
                        for (int s = 0; s < S; ++s) {
                            const bool here = (held >> s) & 1u;
                            const int32_t at = next_at + wave_prefix(here ? 1u : 0u, 1, &total);
                            next_at += total;
                            if (!here) continue;
                            list[at] = (uint16_t)(s * ls + i);
                            if (!((touched >> s) & 1u) || sm.first_order || !((sm.diff_mask >> s) & 1u)) continue;
                            const int32_t Ns = cell.n(s);
                            const double nbar = mean_occupancy(cell, s, Ns, tau_k);
                            int32_t ni = (int32_t)floor(nbar);
                            const double frac = nbar - (double)ni;
                            uint32_t drew = 0;
                            if (frac > 0.0) {
                                Stream rng(sm.key0, key1, (uint32_t)s, (uint32_t)t, period32);
                                if (rng.uniform() < frac) ni += 1;
                                drew = 0x80000000u;
                            }
                            pop[at] = (int32_t)((uint32_t)ni | drew);
                            cell.n(s) = (int32_t)((uint32_t)Ns | 0x80000000u);
                        }
                    }
                    __syncthreads();
                }
            }

            // Step 3: one lane per pair.  Short layout: the counts of listed
            // pairs are taken out first (the first nt stay in registers), so
            // that what moves or stays is added to the same array.
            const int32_t n_pairs = EVERY ? P : head.n_pairs;
            uint32_t first_raw = 0;
            if (!FULL && !spill) {
                for (int32_t j = tid; j < n_pairs; j += nt) {
                    const uint32_t e = list[j], c = (uint32_t)cur[e];
                    cur[e] = 0;
                    if (j < nt)
                        first_raw = c;
                    else
                        taken[j] = (int32_t)c;
                }
                __syncthreads();
            }
            for (int32_t j = tid; j < n_pairs; j += nt) {
                const uint32_t e = EVERY ? (uint32_t)j : list[j];
                const int32_t s = (int32_t)__umulhi(e, per_species);
                const int32_t t = t0 + (int32_t)e - s * ls;
                uint32_t raw;
                if (FULL) {
                    raw = (uint32_t)cur[e];
                    cur[e] = 0;
                    if (EVERY && (int32_t)raw < 0) {  // as in the scan
                        atomicOr(sm.flags, 1);
                        raw = 0;
                    }
                } else {
                    raw = spill ? (uint32_t)cur[e] : j < nt ? first_raw : (uint32_t)taken[j];
                }
                const int32_t Ns = (int32_t)(raw & 0x7fffffffu);
                int32_t stay = Ns;
                if (Ns > 0 && ((sm.diff_mask >> s) & 1u)) {
                    const MeshRec *mr = sm.mesh + t;
                    const int4 n4 = *reinterpret_cast<const int4 *>(mr->nbr);
                    const int32_t nb[4] = {n4.x, n4.y, n4.z, n4.w};
                    const double w[4] = {mr->w[0], mr->w[1], mr->w[2], ANY_SCALED ? mr->w3 : 0.0};
                    const double g = mr->g;
                    PrimedStream rng(sm.key0, key1, (uint32_t)s, (uint32_t)t, period32);
                    int32_t ni = Ns;
                    if (raw >> 31) {
                        const uint32_t code = (uint32_t)pop[j];
                        ni = (int32_t)(code & 0x7fffffffu);
                        if (code >> 31) (void)rng.uniform();  // the rounding's draw
                    }
                    double zeta = (tau_k * head.D[s]) * g;
                    if (zeta > 1.0) zeta = 1.0;
                    int32_t out[4];
                    const int32_t n = leave_and_split<ANY_SCALED>(ni, Ns, zeta, sm.transfer_form == 1, nb, w,
                                                                  sm.split_threshold, rng, out);
                    if (n > 0) {
                        stay = Ns - n;
#pragma unroll
                        for (int f = 0; f < 4; ++f) {
                            if (out[f] <= 0) continue;
                            const int32_t i = nb[f] - t0;
                            if ((uint32_t)i < (uint32_t)len && !spill)
                                atomicAdd(&nxt[s * ls + i], out[f]);
                            else  // another block's tet
                                add_in_memory(sm, period + 1, base, mbase, Tp, s, nb[f], out[f], !direct);
                        }
                    }
                }
                if (stay > 0) {
                    if (!spill)
                        atomicAdd(&nxt[e], stay);
                    else
                        add_in_memory(sm, period + 1, base, mbase, Tp, s, t, stay, !direct);
                }
            }
            __syncthreads();
            if (tid == 0) head.n_ssa = head.n_pairs = 0;
            if (FULL) break;
            from = to;
            to = min(ls, to + range);
            if (from < ls) __syncthreads();
        }
        // additions through memory reach it before this block publishes the
        // period
        if (!alone || spill) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (spill)
                for (int32_t v = tid; v < P / 4; v += nt) *reinterpret_cast<v4i *>(cur + 4 * v) = v4i{0, 0, 0, 0};
            __syncthreads();
            if (!alone) {
                const unsigned long long target = epoch + (unsigned long long)k + 1ull;
                if (tid < 64) {
                    if (tid == 0)
                        __hip_atomic_store(&done[(int64_t)pt.part * kResidentFlagStride], target, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    if (!wait_neighbours(done, nlist, pt.neighbours, my_neighbour, target, fail) && tid == 0)
                        head.stop = 1;
                }
                __syncthreads();
            }
            // what was added to this block's tets
            const gptr<int32_t> next = global(sm.buf[(period + 1) & 1]) + base + t0;
            if (direct) {
                // two groups per pass, their loads in flight together
                for (int32_t v = tid; v < P / 4; v += 2 * nt) {
                    const int32_t u = min(v + nt, P / 4 - 1);
                    const int32_t sv = (int32_t)__umulhi(4u * (uint32_t)v, per_species),
                                  su = (int32_t)__umulhi(4u * (uint32_t)u, per_species);
                    const Arrivals one((gptr<unsigned long long>)(next + sv * Tp + (4 * v - sv * ls))),
                        two((gptr<unsigned long long>)(next + su * Tp + (4 * u - su * ls)));
                    one.take(nxt + 4 * v);
                    if (v + nt < P / 4) two.take(nxt + 4 * u);
                }
            } else {
                const gptr<uint8_t> marks = global(sm.mask[(period + 1) & 1]) + mbase + (t0 >> 2);
                const uint32_t mark = occupancy_tag(period + 1);
                const int32_t words = (len + 15) >> 4;
                for (int32_t v = tid; v < S * words; v += nt) {
                    const int32_t s = v / words, wd = v - s * words;
                    const uint32_t m =
                        __hip_atomic_load((gptr<uint32_t>)(marks + (int64_t)s * sm.mstride + 4 * wd),
                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        if (((m >> (8 * b)) & 0xffu) != mark) continue;
                        const int32_t i = 16 * wd + 4 * b;
                        const Arrivals here((gptr<unsigned long long>)(next + s * Tp + i));
                        here.take(nxt + s * ls + i);
                    }
                }
            }
        }
        __syncthreads();
        if (head.stop) break;  // uniform over the block
    }

    // the state of the next period, its occupancy bytes, and an empty other buffer
    const int64_t end = first + n_periods;
    const int32_t *fin = FULL ? counts + (n_periods & 1) * P : counts;
    const gptr<int32_t> dst = global(sm.buf[end & 1]) + base + t0;
    const gptr<int32_t> other = global(sm.buf[(end & 1) ^ 1]) + base + t0;
    const gptr<uint8_t> mdst = global(sm.mask[end & 1]) + mbase + (t0 >> 2);
    const uint8_t mark = occupancy_tag(end);
    for (int32_t v = tid; v < P / 4; v += nt) {
        const int32_t s = (int32_t)__umulhi(4u * (uint32_t)v, per_species);
        const int32_t i = 4 * v - s * ls;
        const v4i c = *reinterpret_cast<const v4i *>(fin + 4 * v);
        *(gptr<v4i>)(dst + s * Tp + i) = c;
        mdst[(int64_t)s * sm.mstride + (i >> 2)] = (c.x | c.y | c.z | c.w) != 0 ? mark : (uint8_t)0;
        if (alone && FULL && (n_periods & 1)) *(gptr<v4i>)(other + s * Tp + i) = v4i{0, 0, 0, 0};
    }
    if (head.stop && tid == 0) atomicOr(sm.flags, 8);
    if (!FULL && tid == 0 && 4 * (int64_t)head.spills > n_periods) {
        atomicOr(sm.flags, kFlagCrowded);
        if (launch_end.crowded)
            __hip_atomic_store(launch_end.crowded, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    end_block(fail + 1, launch_end);
}

hipError_t launch_resident(const DevSim *sims, const ResidentPlan &plan, int64_t iter0, int32_t n_periods,
                           int64_t partial, double tau_last, unsigned long long epoch, const LaunchEnd &end,
                           hipStream_t st)
{
    if (n_periods <= 0) return hipSuccess;
    if (plan.blocks < 1 || plan.threads < 64 || plan.threads > kResidentMaxThreads ||
        plan.lds_bytes > kResidentLdsMax)
        return hipErrorInvalidValue;
    const void *fn;
    if (plan.full && plan.every)
        fn = plan.scaled ? reinterpret_cast<const void *>(&resident_kernel<true, true, true>)
                         : reinterpret_cast<const void *>(&resident_kernel<false, true, true>);
    else if (plan.full)
        fn = plan.scaled ? reinterpret_cast<const void *>(&resident_kernel<true, true, false>)
                         : reinterpret_cast<const void *>(&resident_kernel<false, true, false>);
    else
        fn = plan.scaled ? reinterpret_cast<const void *>(&resident_kernel<true, false, false>)
                         : reinterpret_cast<const void *>(&resident_kernel<false, false, false>);
    uint32_t *fail = reinterpret_cast<uint32_t *>(plan.done + (int64_t)plan.blocks * kResidentFlagStride);
    const uint16_t *neighbours = plan.neighbours;
    int32_t max_parts = plan.max_parts;
    unsigned long long *done = plan.done;
    const ResidentPart *parts = plan.parts;
    int32_t lds = plan.lds_bytes;
    void *args[] = {(void *)&sims,      (void *)&parts,   (void *)&neighbours, (void *)&max_parts,
                    (void *)&iter0,     (void *)&n_periods, (void *)&partial,  (void *)&tau_last,
                    (void *)&done,      (void *)&epoch,   (void *)&fail,       (void *)&lds,
                    (void *)&end};
    if (plan.max_parts > 1)
        return hipLaunchCooperativeKernel(fn, dim3(plan.blocks), dim3(plan.threads), args, (unsigned)lds, st);
    return hipLaunchKernel(fn, dim3(plan.blocks), dim3(plan.threads), args, (size_t)lds, st);
}

}  // namespace rdos
