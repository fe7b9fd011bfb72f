// Shared host/device definitions of the rdos library (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "../../include/rdos.h"

namespace rdos {

constexpr int kMaxSpecies = RDOS_MAX_SPECIES;
constexpr int kMaxReactions = RDOS_MAX_REACTIONS;
constexpr uint32_t kSsaStream = 0x80000000u;   // Philox stream id of the SSA draws
constexpr int kSplitOneByOne = 10;             // Sec. II.B: n below this moves one by one
constexpr double kAvogadro = 6.02214076e23;    // 1/mol (SI 2019)
constexpr uint32_t kMaxEventsPerPeriod = 1u << 24;  // SSA events of one tet in one period

// One tetrahedron's tables: one 64-byte line, read only when the tet holds
// molecules (or has a 0th-order reaction).
struct alignas(64) MeshRec {
    int32_t nbr[4];   // neighbour across face f (opposite local vertex f), -1 = boundary
    double w[3];      // direction weights of faces 0..2; with w3 they sum to 1 over the interior faces
    double g;         // sum_f A_f / (V delta_f), 1/m^2; local rate d = D g
    double w3;        // face 3, which closes the split when it is interior: only transfer form 1 reads it
    double nav;       // N_A * volume in litres
};
static_assert(sizeof(MeshRec) == 64, "MeshRec must be one cache line");

// The value an occupancy byte holds to mark period k (1..255, never 0).
// Bytes are not cleared after they are read: a byte marks its group only in
// the period whose tag it holds.  A byte left from 510 periods earlier (the
// tags repeat every 255 periods, and each of the two maps serves every other
// period) can match again; the scan then reads an all-zero count vector and
// queues nothing, so a stale byte costs a read, never a result.
__host__ __device__ inline uint8_t occupancy_tag(int64_t period) { return (uint8_t)(period % 255 + 1); }

// One simulation as the step kernel sees it (device memory).
struct alignas(16) DevSim {
    const MeshRec *mesh;       // [T]
    int32_t *buf[2];           // [Rz][S][Tp] counts; period k reads buf[k & 1] and fills buf[(k + 1) & 1]
    uint8_t *mask[2];          // [Rz][S][mstride] occupancy of buf[k & 1]: byte t >> 2 of row (r, s)
                               // equals occupancy_tag(k) when species s of tets 4 (t >> 2) .. + 3 may
                               // be non-zero in period k
    int32_t *flags;            // bit 0: count overflow; bit 1: SSA event cap; bit 2: queue overflow; bit 3: a
                               // wait between blocks failed; bit 4: kFlagCrowded
    int32_t T, S, R, Rz;
    int32_t mstride;           // occupancy bytes per species row (Tp / 4 rounded up to 16)
    uint32_t key0, key1;       // Philox key words before the realization is mixed in
    double tau;                // full period
    int64_t step0;             // period index of launch iteration 0
    int64_t step_end;          // periods >= step_end are not run
    double D[kMaxSpecies];
    uint32_t diff_mask;        // species with D > 0
    uint32_t zeroth;           // 1 if some reaction has no reactant (every tet active)
    uint32_t first_order;      // 1: n from the count at the end of the period instead of Nbar
    int32_t split_threshold;   // below this n molecules are split one by one (Sec. II.B: 10)
    int32_t transfer_form;     // 0: n = binomial then split (eq. 3); 1: one split scaled by zeta
    const uint32_t *allowed;   // [T] bit r: reaction r may fire in the tet (null: everywhere)
    // reactions
    int32_t rn[kMaxReactions], r0[kMaxReactions], r1[kMaxReactions];
    int32_t pn[kMaxReactions], p0[kMaxReactions], p1[kMaxReactions], p2[kMaxReactions];
    uint32_t involved[kMaxReactions];   // bit m: species m is a reactant or a product
    double k[kMaxReactions];
};

// A block's unit of work: up to kTetsPerTile consecutive tets of one
// realization of one simulation.
struct Tile {
    int32_t sim;
    int32_t realization;
    int32_t tet0;
    int32_t ntet;
};

constexpr int kBlock = 256;        // threads per block (4 wavefronts)
constexpr int kTetsPerLane = 4;    // one 16-byte load per species and lane
constexpr int kTetsPerTile = kBlock * kTetsPerLane;

// One realization of one simulation in a work list, for building the tile
// list on the device: its tiles are tiles[first .. first + ceil(T / kTetsPerTile)).
struct WorkUnit {
    int32_t sim;
    int32_t realization;
    int32_t T;
    int32_t first;
};

// Held while a graph is captured and around device allocations and frees
// made by other threads, so neither can interfere with a capture.
inline std::mutex &device_api_mutex()
{
    static std::mutex m;
    return m;
}

// What a launch says in host memory (pinned; null: nobody asks).  One whose
// blocks wait for each other: its last block to end writes `number` to *word.
// One with short lists: it writes 1 to *crowded where it raises kFlagCrowded.
struct LaunchEnd {
    unsigned long long *word = nullptr;
    unsigned long long number = 0;
    uint32_t *crowded = nullptr;
};
// A block's end (every thread of it): the launch's last one says so on the
// host.  `ended` counts blocks, and is 0 between launches.
__device__ __forceinline__ void end_block(uint32_t *ended, const LaunchEnd &end)
{
    if (!end.word) return;
    __syncthreads();
    if (threadIdx.x != 0 || atomicAdd(ended, 1u) + 1u != gridDim.x) return;
    __hip_atomic_store(ended, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(end.word, end.number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Kernel launchers (rdos_kernels.hip).
hipError_t launch_geometry(const double *xyz, const int32_t *tet_verts, const int32_t *nbr,
                           int32_t T, double *scratch_vol, double *scratch_bc,
                           double *scratch_area, MeshRec *mesh, int32_t *bad_volume,
                           hipStream_t st);
// The same for triangles (surface diffusion): area instead of volume, edge
// lengths instead of face areas, N_A A as the unit of amount.
hipError_t launch_geometry_tri(const double *xyz, const int32_t *tri_verts, const int32_t *nbr, int32_t T,
                               double *scratch_area, double *scratch_bc, double *scratch_len, MeshRec *mesh,
                               int32_t *bad_area, hipStream_t st);
// Face matching on the device for cells of cell_verts (4: tetrahedra, 3:
// triangles) vertices with ids below 2^bits (bits <= 21 for tetrahedra, <= 31
// for triangles): nbr[4 T] (filled with -1 by the caller) gets the cell
// across each face; *err (zero on entry) becomes non-zero when a face lies on
// more than two cells or twice on one.  scratch holds
// face_match_scratch_bytes(T, cell_verts) bytes.
size_t face_match_scratch_bytes(int32_t T, int32_t cell_verts);
hipError_t launch_face_match(const int32_t *cells, int32_t T, int32_t cell_verts, int32_t bits, int32_t *nbr,
                             void *scratch, int32_t *err, hipStream_t st);
hipError_t launch_tau_min(const MeshRec *mesh, int32_t T, const double *D, int32_t S,
                          unsigned long long *out_bits, hipStream_t st);
// Writes the k-th smallest (0-based, clamped to the last) of 1/(D_m g_t)
// over diffusing species and connected tets to *out_bits (as its bit
// pattern); scratch must hold tau_select_scratch_bytes(T, S) bytes.
size_t tau_select_scratch_bytes(int32_t T, int32_t S);
hipError_t launch_tau_select(const MeshRec *mesh, int32_t T, const double *D, int32_t S, int64_t k, void *scratch,
                             unsigned long long *out_bits, hipStream_t st);
// Work-list sizes and queue geometry, read by the kernels from device memory
// so that a captured graph stays valid when the work list changes.
struct alignas(16) WorkHeader {
    int32_t n_tiles;   // tiles in the work list
    int32_t n_sims;    // simulation descriptors
    int32_t nseg;      // queue segments in use, 1..kMaxSegments
    int32_t seg_cap;   // entries per segment
    int64_t qcap;      // stride between the count rows of the queue (allocated entries)
    int32_t tile0;     // this work list starts at tiles[tile0] (kernels get the array's base)
    int32_t pad;
};

// Occupied-tet queue of one launch pair (device memory, see the scan kernel).
struct QueueView {
    int32_t *tet;       // [qcap] tile * kTetsPerTile + offset
    int32_t *counts;    // [species][qcap] counts at the start of the period
    int32_t *len;       // [2][kMaxSegments] segment lengths, one per kLenStride ints (own cache
                        // line); both halves zero before the first launch
    WorkHeader *hdr;    // device copy of the sizes below
    int32_t nseg;       // host copies
    int32_t seg_cap;
    int64_t qcap;       // allocated entries per count row
    int32_t species;    // allocated count rows
    int32_t scaled;     // some simulation of the work list uses transfer form 1 (picks the update kernel)
    uint32_t *sync;     // [kPersistSyncWords] of the one-launch path: grid-barrier counters, failure word, blocks ended
    unsigned long long *work;  // null, or [3] device totals the update kernel adds to: tets, count additions,
                               // additions that are transfers across a face
    int32_t owned;      // the work lists launched on it have a segment per tile and a scan wavefront per
                        // tile (at most kMaxSegments tiles): the scan instance that fills segments by its
                        // own count (checked again on the device)
};
constexpr int kMaxSegments = 1024;
constexpr int kPersistSyncWords = 64 * 32 + 32;  // 64 barrier counters on lines of their own, then two words
constexpr int kLenStride = 32;  // 128 bytes between segment lengths: no two share a line

// Queue geometry for a work list of n_tiles tiles: tiles ti with
// ti % nseg == k fill segment k.
inline void queue_shape(int64_t n_tiles, int32_t *nseg, int32_t *seg_cap)
{
    const int64_t ns = n_tiles < kMaxSegments ? (n_tiles > 0 ? n_tiles : 1) : kMaxSegments;
    *nseg = (int32_t)ns;
    *seg_cap = (int32_t)(((n_tiles + ns - 1) / ns) * kTetsPerTile);
}

// One period for every tile: period index = sims[i].step0 + iter; the period
// whose index equals `partial` lasts tau_last instead of tau.  Consecutive
// launches on one queue alternate qsel = 0, 1, 0, ...
// scan_grid blocks stride over the tiles named in q.hdr (> 0 required).
hipError_t launch_scan(const DevSim *sims, const Tile *tiles, int64_t iter, const QueueView &q, int32_t qsel,
                       int32_t scan_grid, hipStream_t st);
// The update grid is grid_segments (1..kMaxSegments) x blocks_per_segment
// blocks, one block column per queue segment: grid_segments must be at least
// the segments of the work list (else the kernel updates nothing and raises
// bit 2 of the first simulation's flags).
hipError_t launch_update(const DevSim *sims, const Tile *tiles, int64_t iter, int64_t partial, double tau_last,
                         const QueueView &q, int32_t qsel, int32_t blocks_per_segment, int32_t grid_segments,
                         hipStream_t st);
hipError_t launch_step(const DevSim *sims, const Tile *tiles, int64_t iter, int64_t partial, double tau_last,
                       const QueueView &q, int32_t qsel, int32_t scan_grid, int32_t blocks_per_segment,
                       int32_t grid_segments, hipStream_t st);
// One launch per period (scan and update fused; no queue in device memory):
// grid blocks of four wavefronts stride over the tiles named in q.hdr; the
// queue supplies the header, the species bound and the work tallies only.
// Queues of up to kFusedSpecies species rows (hipErrorInvalidValue beyond).
constexpr int kFusedSpecies = 8;
hipError_t launch_fused(const DevSim *sims, const Tile *tiles, int64_t iter, int64_t partial, double tau_last,
                        const QueueView &q, int32_t grid, hipStream_t st);
// Scan blocks needed to give every tile of a work list its own wavefront.
inline int32_t scan_blocks_for(int64_t n_tiles)
{
    const int64_t b = (n_tiles + kBlock / 64 - 1) / (kBlock / 64);
    return (int32_t)(b < 1 ? 1 : (b > (1 << 20) ? (1 << 20) : b));
}
// The work list of one simulation alone: its descriptor, header and tiles.
hipError_t launch_own_work(const DevSim &d, DevSim *desc, const WorkHeader &h, WorkHeader *hdr, Tile *tiles,
                           hipStream_t st);
hipError_t launch_advance(DevSim *sims, const WorkHeader *hdr, int64_t by, hipStream_t st);
// Writes tiles[0 .. n_tiles) from n_units work units whose `first` fields
// ascend from 0 and leave no gaps (each unit has at least one tile).
hipError_t launch_expand_tiles(const WorkUnit *units, int32_t n_units, int32_t n_tiles, Tile *tiles, hipStream_t st);
// Small work lists: n_periods periods in one cooperative launch of `grid`
// blocks (at most persist_grid_limit(q), every block resident), grid-wide
// barriers between the scan and update phases.  Period i uses queue half
// (phase + i) & 1.  sync points at kPersistSyncWords words of device memory
// (barrier counters, failure word) that no other launch uses meanwhile; a
// barrier that times out raises bit 3 of every simulation's flags.
int32_t persist_grid_limit(const QueueView &q);
hipError_t launch_persist(const DevSim *sims, const Tile *tiles, int64_t iter0, int32_t n_periods, int32_t phase,
                          int64_t partial, double tau_last, const QueueView &q, int32_t grid, uint32_t *sync,
                          const LaunchEnd &end, hipStream_t st);
// State held in LDS (rdos_resident.hip).  A realization is cut into `parts`
// ranges of consecutive tets, one block each; a block keeps its range's
// counts in LDS for a whole run of periods.
struct ResidentPart {
    int32_t sim;
    int32_t realization;
    int32_t t0, len;      // its tets; t0 a multiple of 16, len too except at the end of the mesh
    int32_t part, parts;  // its place among the realization's blocks
    int32_t stride;       // tets per block of the realization (the last may hold fewer)
    int32_t flag0;        // the realization's first block
    int32_t neighbours;   // blocks it exchanges molecules with
    int32_t pad[3];
};
// One realization of a work list, for building the parts on the device.
struct ResidentUnit {
    int32_t sim;
    int32_t realization;
    int32_t T;
    int32_t first;   // its first block
    int32_t blocks;
    int32_t len;     // tets per block
};
struct ResidentPlan {
    unsigned long long *done;   // [blocks][kResidentFlagStride] last period finished by each block, then the
                                // failure word and the number of blocks that have ended (device)
    ResidentPart *parts;        // [blocks] (device)
    uint16_t *neighbours;       // [blocks][max_parts] (device; max_parts > 1)
    int32_t blocks;
    int32_t max_parts;          // blocks of the realization with the most; above 1 the launches are cooperative
    int32_t threads;
    int32_t lds_bytes;
    int32_t full;               // layout
    int32_t every;              // no reactions, full, and a lane for every pair of a block
    int32_t scaled;             // some simulation uses transfer form 1
};
constexpr int kResidentMaxThreads = 1024;
constexpr int kResidentMaxParts = 1024;
constexpr int64_t kResidentMaxUnits = 1 << 16;  // of an engine's work list
constexpr int32_t kResidentLdsMax = 160 * 1024;
// Raised by a run whose short lists overflowed in over a quarter of its
// periods: no error, but the queue is faster then.
constexpr int32_t kFlagCrowded = 16;
constexpr int kResidentFlagStride = 16;  // 128 bytes between blocks' period counters
constexpr int32_t kResidentHeadBytes = kMaxSpecies * 8 + kMaxReactions * 16 + 16;
// Two layouts of a block whose species rows hold `ls` tets (a multiple of 4).
// Full: two count buffers and lists that hold every pair.  Short: one count
// buffer, and lists for `range` tets, an eighth of the block's at least (whole
// four-tet groups).
__host__ __device__ inline int32_t resident_least(int32_t ls) { return 4 * ((ls / 4 + 7) / 8); }
// A lane's share in the SSA: occupancy integrals, times, constants and
// propensities.
__host__ __device__ inline int32_t resident_lane_bytes(int32_t S, int32_t R) { return 16 * (S + R); }
// The lists for `range` tets: the pairs (short layout: and their counts), and
// with reactions the rounded mean populations and the tets for the SSA.
__host__ __device__ inline int32_t resident_list_bytes(int32_t S, int32_t R, bool full, int32_t range)
{
    return (((full ? 2 * S : 6 * S) + (R > 0 ? 4 * S + 2 : 0)) * range + 15) & ~15;
}
// LDS with `lanes` lanes in the SSA (64 at least; none without reactions).
__host__ __device__ inline int32_t resident_lds_bytes(int32_t S, int32_t R, int32_t ls, bool full, int32_t range,
                                                      int32_t lanes)
{
    return kResidentHeadBytes + (full ? 8 : 4) * S * ls + resident_list_bytes(S, R, full, range) +
           (R > 0 ? resident_lane_bytes(S, R) * lanes : 0);
}
// The tets the short layout's lists hold in `lds` bytes: up to 256 lanes in
// the SSA (a wavefront per SIMD) come first.
__host__ __device__ inline int32_t resident_range(int32_t S, int32_t R, int32_t ls, int32_t lds)
{
    const int32_t least = resident_least(ls);
    int32_t left = lds - resident_lds_bytes(S, R, ls, false, least, 64);
    if (R > 0) {
        const int32_t more = (left / resident_lane_bytes(S, R)) & ~63;
        left -= (more < 192 ? more : 192) * resident_lane_bytes(S, R);
    }
    if (left < 16) return least;
    const int32_t range = least + ((left - 15) / (6 * S + (R > 0 ? 4 * S + 2 : 0)) & ~3);
    return range < ls ? range : ls;
}
// The lanes of the SSA with `used` of the LDS taken by the rest.
__host__ __device__ inline int32_t resident_lanes(int32_t S, int32_t R, int32_t lds, int32_t used, int32_t threads)
{
    if (R == 0) return 0;
    const int32_t most = ((lds - used) / resident_lane_bytes(S, R)) & ~63;
    return most < threads ? most : threads;
}
__host__ __device__ inline bool resident_every(int32_t S, int32_t R, int32_t ls, int32_t threads)
{
    return R == 0 && S * ls <= threads;
}
// Device memory of a plan, and its arrays' places in it (16-byte aligned).
size_t resident_plan_bytes(int64_t blocks, int64_t max_parts);
void resident_place(ResidentPlan *plan, void *memory);
// Fills the arrays of a plan: its blocks are those of n_units units whose
// `first` fields ascend from 0 without gaps, or (units null) of the
// realizations of one simulation, each cut like `same`.
hipError_t launch_resident_layout(const DevSim *sims, const ResidentPlan &plan, const ResidentUnit *units,
                                  int32_t n_units, const ResidentUnit &same, hipStream_t st);
// n_periods periods of every part: the iterations iter0 .. of its simulation
// (the period equal to `partial` lasts tau_last).  `epoch` is at least every
// value in plan.done; the launch raises them to at most epoch + n_periods.
hipError_t launch_resident(const DevSim *sims, const ResidentPlan &plan, int64_t iter0, int32_t n_periods,
                           int64_t partial, double tau_last, unsigned long long epoch, const LaunchEnd &end,
                           hipStream_t st);
// Batches of sparse realizations (rdos_sparse.hip): one block per unit of the
// work list keeps its occupied (tet, species) pairs in a hash table in LDS.
struct SparsePlan {
    int32_t units;
    int32_t threads;      // per block
    int32_t slots;        // of the table: the most pairs a realization may hold (a multiple of 4 threads)
    int32_t filter_words; // of each of the two filters over tets (a power of two)
    int32_t lanes;        // in the SSA at a time (a multiple of 64; 0 without reactions)
    int32_t lds_bytes;
    int32_t scaled;       // some simulation uses transfer form 1
    int64_t unit_bytes;   // of scratch per unit
    char *scratch;        // [units][unit_bytes] (device)
    int32_t *counts;      // [units][2] pairs before and after the run (device)
    uint32_t *fail;       // raised when a table was full (device)
};
constexpr int kSparseMaxThreads = 1024;
constexpr int kSparseTetBits = 27;        // tets below 2^27 - 1
// Their scratch is (24 + 4 S) bytes a slot: 1.2 GB for 2048 units of 16,384 slots
// and three species, 2.4 GB for twelve.
constexpr size_t kSparseMaxUnits = 2048;
constexpr int32_t kSparseHeadBytes = kMaxSpecies * 8 + kMaxReactions * 16 + 32;
// The table and lane state for units of up to S species, R reactions and
// about `pairs` occupied pairs, and for more or fewer units than the device
// has compute units; false where they do not fit the LDS.
bool sparse_shape(int32_t S, int32_t R, int64_t pairs, bool many_units, SparsePlan *plan);
// n_periods periods of every unit; no simulation ends among them, and none
// has a reaction without reactants.  All units' states move on, or, when
// *plan.fail is set (it must be 0 before), none does.
hipError_t launch_sparse(const DevSim *sims, const WorkUnit *units, int64_t iter0, int32_t n_periods,
                         const SparsePlan &plan, hipStream_t st);
// Rebuilds the occupancy bytes of buf[parity] from the counts of every
// realization and species and clears those of the other buffer (after
// counts were set from the host).
hipError_t launch_mask_build(const int32_t *counts, uint8_t *mask_cur, uint8_t *mask_other, uint8_t tag, int32_t Rz,
                             int32_t S,
                             int64_t Tp, hipStream_t st);
// Bytes of one species row of the occupancy map: one per four tets, padded
// to 16 bytes so that the scan reads four bytes at a time.
inline int32_t mask_stride(int64_t Tp) { return (int32_t)(((Tp / 4) + 15) & ~(int64_t)15); }
// counts[0 .. T) and the flags word to out[0 .. T] (pinned host memory).
hipError_t launch_read_counts(const int32_t *counts, const int32_t *flags, int32_t *out, int32_t T, hipStream_t st);
// Takes `bits` off the flags word.
hipError_t launch_clear_flags(int32_t *flags, int32_t bits, hipStream_t st);
// The mesh records taken apart: nbr[T][4], w[T][4], g[T], nav[T].
hipError_t launch_unpack_mesh(const MeshRec *mesh, int32_t T, int32_t *nbr, double *w, double *g, double *nav,
                              hipStream_t st);
hipError_t launch_copy(const void *src, void *dst, size_t bytes, hipStream_t st);
// blocks x 256 lanes each split n molecules reps times, one-by-one or by
// sequential binomials; sink holds blocks * 256 int64.
hipError_t launch_split_cost(bool one_by_one, int64_t n, int32_t reps, int64_t *sink, int32_t blocks, hipStream_t st);


}  // namespace rdos
