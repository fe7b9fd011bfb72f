// Host side of the rdos C ABI: handles, call-order checks, mesh topology,
// device set-up and the stepping loop (Algorithm 1, Steps 1 and 4).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <limits>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "rdos_internal.h"
#include "rdos_sim.h"
#include "rdos_turn.h"

using namespace rdos;

namespace rdos {

rdos_status fail(rdos_sim *s, rdos_status code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (s) s->error = buf;
    return code;
}

rdos_status hip_fail(rdos_sim *s, hipError_t e, const char *what)
{
    return fail(s, e == hipErrorOutOfMemory ? RDOS_ENOMEM : RDOS_EDEVICE, "%s: %s", what,
                hipGetErrorString(e));
}

#define HIP_TRY(sim, expr, what)                         \
    do {                                                 \
        hipError_t e__ = (expr);                         \
        if (e__ != hipSuccess) return hip_fail(sim, e__, what); \
    } while (0)

int64_t padded_tets(int32_t T) { return ((int64_t)T + 3) & ~(int64_t)3; }

// Device memory of simulations, their queues and their set-up comes from a
// stream-ordered pool per device: allocation and release are ordered on the
// simulation's stream and never synchronise the whole device (hipFree can,
// which stalled admissions behind the engine's running chunks), and freed
// memory stays in the pool for the next simulation.
static hipMemPool_t pool_for(int device)
{
    static std::mutex mu;
    static hipMemPool_t pools[64] = {};
    if (device < 0 || device >= 64) return nullptr;
    std::lock_guard<std::mutex> g(mu);
    if (!pools[device]) {
        hipMemPoolProps props{};
        props.allocType = hipMemAllocationTypePinned;
        props.handleTypes = hipMemHandleTypeNone;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = device;
        hipMemPool_t pool = nullptr;
        if (hipMemPoolCreate(&pool, &props) != hipSuccess) return nullptr;
        uint64_t keep = ~0ull;  // never hand freed memory back to the driver
        (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
        pools[device] = pool;
    }
    return pools[device];
}

hipError_t dev_alloc(void **p, size_t bytes, hipStream_t st)
{
    *p = nullptr;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    hipMemPool_t pool = pool_for(device);
    if (!pool) return hipErrorOutOfMemory;
    return hipMallocFromPoolAsync(p, bytes ? bytes : 16, pool, st);
}

void dev_free(void *p, hipStream_t st)
{
    if (p) (void)hipFreeAsync(p, st);
}

size_t queue_bytes(int64_t n_tiles, int32_t n_species)
{
    int32_t nseg, seg_cap;
    queue_shape(n_tiles, &nseg, &seg_cap);
    return (size_t)nseg * seg_cap * (1 + (size_t)n_species) * sizeof(int32_t) +
           2 * (size_t)kMaxSegments * kLenStride * sizeof(int32_t) + sizeof(WorkHeader) +
           kPersistSyncWords * sizeof(uint32_t);
}

// Room for a work list of up to capacity_tiles tiles and n_species count rows.
hipError_t alloc_queue(QueueView *q, int64_t capacity_tiles, int32_t n_species, hipStream_t st)
{
    *q = QueueView{};
    queue_shape(capacity_tiles, &q->nseg, &q->seg_cap);
    q->qcap = (int64_t)q->nseg * q->seg_cap;
    q->species = std::max(n_species, 1);
    hipError_t e = dev_alloc((void **)&q->tet, (size_t)q->qcap * sizeof(int32_t), st);
    if (e == hipSuccess) e = dev_alloc((void **)&q->counts, (size_t)q->qcap * q->species * sizeof(int32_t), st);
    const size_t len_bytes = 2 * (size_t)kMaxSegments * kLenStride * sizeof(int32_t);
    if (e == hipSuccess) e = dev_alloc((void **)&q->len, len_bytes, st);
    if (e == hipSuccess) e = dev_alloc((void **)&q->hdr, sizeof(WorkHeader), st);
    if (e == hipSuccess) e = dev_alloc((void **)&q->sync, kPersistSyncWords * sizeof(uint32_t), st);
    if (e == hipSuccess) e = hipMemsetAsync(q->len, 0, len_bytes, st);
    return e;
}

// Points the queue at a work list of n_tiles tiles (<= its capacity) and
// n_sims descriptors; the kernels read these sizes from q->hdr.
WorkHeader queue_header(QueueView *q, int64_t n_tiles, int32_t n_sims, int32_t tile0)
{
    int32_t nseg, seg_cap;
    queue_shape(n_tiles, &nseg, &seg_cap);
    q->nseg = nseg;
    q->seg_cap = seg_cap;
    WorkHeader h{};
    h.n_tiles = (int32_t)n_tiles;
    h.n_sims = n_sims;
    h.nseg = nseg;
    h.seg_cap = seg_cap;
    h.qcap = q->qcap;
    h.tile0 = tile0;
    return h;
}
hipError_t set_queue_work(QueueView *q, int64_t n_tiles, int32_t n_sims, hipStream_t st, int32_t tile0)
{
    int32_t nseg, seg_cap;
    queue_shape(n_tiles, &nseg, &seg_cap);
    if ((int64_t)nseg * seg_cap > q->qcap) return hipErrorInvalidValue;
    const WorkHeader h = queue_header(q, n_tiles, n_sims, tile0);
    hipError_t e = hipMemcpyAsync(q->hdr, &h, sizeof h, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);  // h lives on this stack frame
    return e;
}

void free_queue(QueueView *q, hipStream_t st)
{
    dev_free(q->tet, st);
    dev_free(q->counts, st);
    dev_free(q->len, st);
    dev_free(q->hdr, st);
    dev_free(q->sync, st);
    *q = QueueView{};
}

// Validation scans.  They accumulate over blocks without leaving early, so
// that they run at memory speed, and name the first offender only when there
// is one (a million tets set up and read, with the tables taken apart on the
// device: 32 ms before both, 16.5 after).
constexpr int64_t kScanBlock = 4096;
static int64_t first_not_finite(const double *v, int64_t n)
{
    for (int64_t b = 0; b < n; b += kScanBlock) {
        const int64_t e = std::min(n, b + kScanBlock);
        int bad = 0;
        for (int64_t i = b; i < e; ++i) bad |= !(std::fabs(v[i]) <= std::numeric_limits<double>::max());
        if (bad)
            for (int64_t i = b; i < e; ++i)
                if (!std::isfinite(v[i])) return i;
    }
    return -1;
}
static int64_t first_not_below(const int32_t *v, int64_t n, int32_t bound)
{
    for (int64_t b = 0; b < n; b += kScanBlock) {
        const int64_t e = std::min(n, b + kScanBlock);
        int bad = 0;
        for (int64_t i = b; i < e; ++i) bad |= (uint32_t)v[i] >= (uint32_t)bound;
        if (bad)
            for (int64_t i = b; i < e; ++i)
                if ((uint32_t)v[i] >= (uint32_t)bound) return i;
    }
    return -1;
}
// The sum of counts, or the first negative one in *bad.
static int64_t sum_counts(const int32_t *v, int64_t n, int64_t *bad)
{
    int64_t total = 0;
    *bad = -1;
    for (int64_t b = 0; b < n; b += kScanBlock) {
        const int64_t e = std::min(n, b + kScanBlock);
        int32_t sign = 0;
        for (int64_t i = b; i < e; ++i) {
            sign |= v[i];
            total += v[i];
        }
        if (sign < 0)
            for (int64_t i = b; i < e; ++i)
                if (v[i] < 0) {
                    *bad = i;
                    return total;
                }
    }
    return total;
}

int32_t compute_units(int device)
{
    static std::atomic<int32_t> known[64] = {};
    if (device < 0 || device >= 64) return 0;
    int32_t n = known[device].load(std::memory_order_relaxed);
    if (n > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 0;
    known[device].store(n, std::memory_order_relaxed);
    return n;
}

ResidentCut resident_cut(int32_t T, int32_t S, int32_t R, int32_t max_blocks)
{
    ResidentCut c;
    // 16 tets: the occupancy bytes of a block's range are whole words
    const int32_t k = std::max(1, std::min(max_blocks, (T + 15) / 16));
    const int32_t len = k == 1 ? T : ((T + k - 1) / k + 15) & ~15;
    const int64_t ls = ((int64_t)len + 3) & ~(int64_t)3;
    const int32_t rows = (int32_t)std::min<int64_t>(ls, 0xffff);
    c.full = resident_lds_bytes(S, R, rows, true, rows, 64) <= kResidentLdsMax;
    if (S * ls > 0xffff || resident_lds_bytes(S, R, rows, c.full, resident_least(rows), 64) > kResidentLdsMax) return c;
    c.len = len;
    c.blocks = (T + len - 1) / len;
    // a lane per (tet, species) pair, up to a block's limit
    c.threads = (int32_t)std::min<int64_t>(kResidentMaxThreads, (S * ls + 63) & ~(int64_t)63);
    c.lds_bytes = c.full ? std::min(kResidentLdsMax, resident_lds_bytes(S, R, rows, true, rows, c.threads))
                         : kResidentLdsMax;
    return c;
}

// Pairs that a realization is expected to hold: the counts last set, spread
// evenly.
double expected_pairs(const rdos_sim *s)
{
    const int32_t S = (int32_t)s->D.size();
    double pairs = 0.0;
    for (int32_t m = 0; m < S; ++m) {
        const double total = (double)s->species_totals[m];
        pairs += (double)s->T * (1.0 - std::exp(-total / ((double)s->Rz * s->T)));
    }
    return pairs;
}

// Whether the short layout's lists hold what a block is expected to, with room
// to spare.  Blocks whose lists overflow move every molecule through memory,
// which is slower than the two-launch path: us per period, two launches and
// this, 998,250 tets of four species at 0.3 and 1 molecules per tet 71 and
// 101, 121 and 167; below that, at 0.1 and 0.03: 44 and 25, 23 and 15.5.  What
// is expected goes by the counts last set: where they were written through a
// device view, or grew, the kernel raises kFlagCrowded (998,250 tets of four
// species, written with one molecule per pair: 221 us per period, 195 over
// the queue).
bool resident_lists_hold(const rdos_sim *s, const ResidentCut &c)
{
    if (c.full) return true;
    if (s->crowded) return false;
    if (s->desc.zeroth) return false;  // every tet is listed for the SSA
    const int32_t S = (int32_t)s->D.size(), R = (int32_t)s->rx.size(), ls = (c.len + 3) & ~3;
    return expected_pairs(s) * c.len <= 0.5 * (double)s->T * S * resident_range(S, R, ls, c.lds_bytes);
}

// Tets of a block of `len` that may react, at most: those expected to hold a
// pair, or all.
static double expected_tets(const rdos_sim *s, int32_t len)
{
    if (s->desc.zeroth) return len;
    return std::min((double)len, expected_pairs(s) * len / s->T);
}

// Whether blocks of `len` tets of a simulation, which have the device `turns`
// times one after the other (1: all at once), are faster than the queue.  A
// compute unit has 768 of the queue's lanes in the SSA (512 above ten species)
// whatever the model, and as many of a block's as the LDS holds beside its
// counts: 64 at 16 species and 32 reactions.  Many reactions over few lanes,
// or many turns for little work, leave these paths behind.  Measured, us per
// period, two launches and this path, with so many passes of the lanes over
// the tets: one turn, 20 realizations of 10,368 tets, 16 reactions, 7 passes
// 217 and 124, 24 reactions, 13 passes 344 and 408; 200 of 750 tets, 24
// reactions, 12 passes 276 and 354; two turns, 1000 of 384 tets, 16 reactions, 3
// passes 131 and 119; 400 of 750, 24 reactions, 12 passes 298 and 685; three,
// 3000 of 162 tets, 8 reactions, 2.5 passes 92 and 80, 16 reactions 142 and 153;
// four, 1000 of 384 tets, 32 reactions, 6 passes 385 and 699.  More turns: 10,000
// realizations of 162 tets, 3 species and 2 reactions, five turns, 126 pairs in a
// block 72 and 36, 5 pairs 23 and 23; 20,000 of 48 tets, ten turns, one pair 25
// and 37; 30,000 of 6 tets, eight turns 45 and 80.
static bool resident_pays(const rdos_sim *s, int32_t len, double turns, int32_t lanes)
{
    const int32_t R = (int32_t)s->rx.size();
    const double tets = expected_tets(s, len), pairs = s->desc.zeroth ? len : expected_pairs(s) * len / s->T;
    if (turns > 4.0 && !(R == 0 && turns <= 5.0) && !(R <= 6 && turns <= 10.0 && pairs >= 100.0)) return false;
    if (R < 8) return true;
    const double passes = std::max(1.0, tets / std::max(lanes, 1));
    if (turns <= 1.0) return passes <= 8.0;
    return turns * passes * R <= (turns <= 2.0 ? 104.0 : 72.0);
}

bool resident_pays(const rdos_sim *s, const ResidentCut &c)
{
    const int32_t S = (int32_t)s->D.size(), R = (int32_t)s->rx.size(), ls = (c.len + 3) & ~3;
    const int32_t range = c.full ? ls : resident_range(S, R, ls, c.lds_bytes);
    const int32_t used = resident_lds_bytes(S, R, ls, c.full, range, 0);
    return resident_pays(s, c.len, 1.0, resident_lanes(S, R, c.lds_bytes, used, c.threads));
}

// One block per realization, more of them (n) than compute units: the widest
// blocks of which enough share a compute unit.  Narrower blocks finish later
// but more run at once, which pays while a lane has a few pairs to itself and
// the number of turns falls; a block that has its compute unit alone takes all
// its lanes.  Measured, us per period with 512 lanes (two blocks per compute
// unit), 256 (four) and 128 (eight): 600 realizations of 750 tets at 0.02
// molecules per species and tet 8.3, 4.9 and 6.2, at 0.3 14.9, 12.5 and 18, at
// 2 50, 69 and 89; 1500 of them at 0.02 13.4, 9.1 and 7.2.  1024 lanes against
// 512, one block per compute unit: 1500 realizations of 1944 tets at 2
// molecules 216 and 297.  Light blocks with a compute unit each are slower than
// the sparse kernel (`light` false: left to it): 600 realizations of 6000 tets
// of three species with 180 pairs in each 21.9 and 12.4, with 1200 36 and 33;
// 400 of 3072 tets with 1900 pairs 25.8 and 49.5.
bool resident_in_turn(const rdos_sim *const *sims, size_t n_sims, int64_t n, int32_t cus, bool light,
                      ResidentPlan *plan)
{
    double work = 0.0;  // items of the fullest block: pairs, and tets that always run the SSA
    for (size_t i = 0; i < n_sims; ++i)
        work = std::max(work, expected_pairs(sims[i]) + (sims[i]->desc.zeroth ? sims[i]->T : 0.0));
    for (int32_t per_cu = 8; per_cu >= 1; per_cu /= 2) {
        const int32_t threads = kResidentMaxThreads / per_cu;
        if (per_cu == 1 && !light && work < 1500.0) break;
        if (per_cu > 2 && (n <= (int64_t)cus * per_cu / 2 || work > (per_cu == 8 ? 2.0 : 4.0) * threads)) continue;
        // whole units of the hardware's LDS allocation (1280 bytes)
        const int32_t most = kResidentLdsMax / per_cu / 1280 * 1280, lanes = per_cu == 2 ? 128 : 64;
        int32_t lds = 0, full = 1, widest = 0;
        for (size_t i = 0; i < n_sims; ++i) {
            const int32_t S = (int32_t)sims[i]->D.size(), R = (int32_t)sims[i]->rx.size(),
                          rows = (sims[i]->T + 3) & ~3;
            lds = std::max(lds, resident_lds_bytes(S, R, rows, true, rows, threads));
            if (resident_lds_bytes(S, R, rows, true, rows, lanes) > most) full = 0;
            widest = std::max(widest, (S * rows + 63) & ~63);
        }
        lds = full ? std::min(lds, most) : most;
        bool fits = true;
        for (size_t i = 0; i < n_sims && !full; ++i) {
            const int32_t S = (int32_t)sims[i]->D.size(), R = (int32_t)sims[i]->rx.size(),
                          rows = (sims[i]->T + 3) & ~3;
            ResidentCut c;
            c.len = sims[i]->T;
            c.lds_bytes = lds;
            fits &= resident_lds_bytes(S, R, rows, false, resident_least(rows), 64) <= lds &&
                    resident_lists_hold(sims[i], c);
        }
        if (!fits) continue;
        const int32_t used_threads = std::min(threads, widest);
        const int32_t together = std::min(kResidentLdsMax / lds, kResidentMaxThreads / used_threads);
        for (size_t i = 0; i < n_sims; ++i) {
            const int32_t S = (int32_t)sims[i]->D.size(), R = (int32_t)sims[i]->rx.size(),
                          rows = (sims[i]->T + 3) & ~3, range = full ? rows : resident_range(S, R, rows, lds);
            const int32_t lanes_of =
                resident_lanes(S, R, lds, resident_lds_bytes(S, R, rows, full, range, 0), used_threads);
            if (!resident_pays(sims[i], sims[i]->T, (double)n / ((double)cus * together), lanes_of)) return false;
        }
        plan->threads = used_threads;
        plan->lds_bytes = lds;
        plan->full = plan->every = full;
        for (size_t i = 0; i < n_sims; ++i)
            plan->every &= resident_every((int32_t)sims[i]->D.size(), (int32_t)sims[i]->rx.size(),
                                          (sims[i]->T + 3) & ~3, plan->threads);
        return true;
    }
    return false;
}

// The cuts of a simulation's realizations for the resident kernel, alone and
// over the device.  Several blocks per realization wait for each other, so
// all must be on the device at once: no more than its compute units (a block
// fills one).
static ResidentCut cut_one(const rdos_sim *s)
{
    return resident_cut(s->T, (int32_t)s->D.size(), (int32_t)s->rx.size(), 1);
}
static ResidentCut cut_many(const rdos_sim *s)
{
    const int32_t k = compute_units(s->device) / s->Rz;
    ResidentCut c;
    if (k > 1) c = resident_cut(s->T, (int32_t)s->D.size(), (int32_t)s->rx.size(), k);
    if (c.blocks < 2) c.blocks = 0;
    return c;
}

static size_t resident_bytes(const rdos_sim *s)
{
    const int64_t one = cut_one(s).blocks, many = cut_many(s).blocks;
    return (one ? resident_plan_bytes(s->Rz, 1) : 0) + (many ? resident_plan_bytes(many * s->Rz, many) : 0);
}

// Lays out the block list of one cut on the device (finalize; the caller has
// uploaded the descriptor on the same stream).
static rdos_status plan_resident(rdos_sim *s, const ResidentCut &c, ResidentPlan *plan)
{
    *plan = ResidentPlan{};
    if (c.blocks == 0) return RDOS_OK;
    ResidentPlan p{};
    p.blocks = c.blocks * s->Rz;
    p.max_parts = c.blocks;
    p.threads = c.threads;
    p.lds_bytes = c.lds_bytes;
    p.full = c.full;
    p.every = c.full && resident_every((int32_t)s->D.size(), (int32_t)s->rx.size(), (c.len + 3) & ~3, c.threads);
    p.scaled = s->transfer_form == 1;
    void *memory = nullptr;
    {
        std::lock_guard<std::mutex> g(device_api_mutex());
        if (dev_alloc(&memory, resident_plan_bytes(p.blocks, p.max_parts), s->stream) != hipSuccess) {
            (void)hipGetLastError();
            return RDOS_OK;  // no room: the queue runs the periods
        }
    }
    resident_place(&p, memory);
    *plan = p;
    HIP_TRY(s, launch_resident_layout(s->d_desc, p, nullptr, 0, ResidentUnit{0, 0, s->T, 0, c.blocks, c.len},
                                      s->stream),
            "block list");
    return RDOS_OK;
}

static bool capturing(const rdos_sim *s)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s->stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone;
}

// Whether n periods pay for the reading and writing of every count around them
// (and, with several blocks, for the cooperative launch), which the queue does
// not need: it reads the occupancy bytes and the counts of occupied tets.
// Lists of at most kPersistTiles tiles always do, and four periods.  Of larger
// ones, by the share of pairs that hold molecules, us for n periods and the
// wait, over the queue and in LDS, at so many molecules per pair.  Several
// blocks, n = 2: 12,096 tets at 0.01 40 and 46, 2,058,000 at 0.01 43 and 58, at
// 0.1 65 and 65, 262,440 of three species at 0.1 104 and 72; n = 3: 2,058,000
// at 0.01 54 and 65, 384,000 of three species at 0.02 90 and 80; n = 4:
// 2,058,000 at 0.01 78 and 72.  A block each, n = 1: 3000 realizations of 162
// tets at 0.01 32 and 38, 200 of 4374 at 0.001 39 and 43, at 0.1 71 and 59; n =
// 2: 3000 of 162 45 and 42, 200 of 4374 at 0.001 55 and 50.
static bool long_enough(const rdos_sim *s, int64_t n, bool several_blocks)
{
    if (s->n_tiles <= kPersistTiles || n >= 4) return true;
    const double cells = (double)s->T * (double)s->D.size();
    const double share = s->desc.zeroth ? 1.0 : expected_pairs(s) / cells;
    if (several_blocks) return n >= (share >= 0.08 ? 2 : share >= 0.015 ? 3 : 4);
    return n >= (share >= 0.08 ? 1 : 2);
}

// The resident launch for n periods, or null: the two-launch (or one-launch)
// path.  Several blocks per realization, unless one does as well: light
// tets (on average two molecules per pair or fewer, by the counts last set)
// with a lane each.  Measured: the cube of 750 tets at 1.3 molecules per tet
// 6.0 us per period with one block, 6.5 with 47; a bar of 1080 tets at 93
// molecules per tet 64 and 23.5.
static const ResidentPlan *resident_for(rdos_sim *s, int64_t n)
{
    if (s->launch_mode != 0) return nullptr;
    if (capturing(s)) return nullptr;  // the period counters of a replay would start over
    const ResidentPlan *one = s->resident_one.blocks ? &s->resident_one : nullptr;
    const ResidentPlan *many = s->resident_many.blocks ? &s->resident_many : nullptr;
    const int32_t cus = compute_units(s->device);
    if (one && s->Rz > cus) {
        const rdos_sim *sim = s;
        if (!resident_in_turn(&sim, 1, s->Rz, cus, true, &s->resident_one)) one = nullptr;
    } else if (one) {
        const ResidentCut c = cut_one(s);
        if (!resident_lists_hold(s, c) || !resident_pays(s, c)) one = nullptr;
    }
    if (many) {
        const ResidentCut c = cut_many(s);
        if (!resident_lists_hold(s, c) || !resident_pays(s, c)) many = nullptr;
    }
    if (one && many) {
        int64_t molecules = 0;
        for (int64_t t : s->species_totals) molecules += t;
        const int64_t pairs = (int64_t)s->T * (int64_t)s->D.size();
        if (pairs > kResidentMaxThreads || molecules > 2 * pairs * s->Rz)
            one = nullptr;
        else
            many = nullptr;
    }
    const ResidentPlan *plan = many ? many : one;
    return plan && long_enough(s, n, many != nullptr) ? plan : nullptr;
}

static int64_t tiles_of(const rdos_sim *s) { return (int64_t)s->Rz * ((s->T + kTetsPerTile - 1) / kTetsPerTile); }

size_t state_bytes(const rdos_sim *s)
{
    const int64_t Tp = padded_tets(s->T);
    const size_t counts = (size_t)s->Rz * s->D.size() * (size_t)Tp * sizeof(int32_t);
    const size_t tiles = (size_t)tiles_of(s) * sizeof(Tile);
    const size_t masks = s->regions.empty() ? 0 : (size_t)s->T * sizeof(uint32_t);
    const size_t occupancy = 2 * (size_t)s->Rz * s->D.size() * mask_stride(Tp);
    return (size_t)s->T * sizeof(MeshRec) + 2 * counts + tiles + queue_bytes(tiles_of(s), (int32_t)s->D.size()) +
           masks + occupancy + resident_bytes(s) + sizeof(DevSim) + 64;
}

// Face-matching results are cached by mesh connectivity (the cell array):
// requests that share a lattice but move its vertices reuse them.  An entry
// shares the cell array of the simulation that made it and its neighbour
// table ([T][4] ints) with the simulations set up from it; nothing is copied.
struct TopologyCache {
    struct Entry {
        int32_t cell_verts = 4;
        std::shared_ptr<const std::vector<int32_t>> cells;
        std::shared_ptr<const int32_t> nbr;
        uint64_t last_use = 0;
    };
    std::mutex mu;
    std::multimap<uint64_t, Entry> entries;  // by hash of the cell array
    size_t bytes = 0;
    uint64_t clock = 0;
    static constexpr size_t kMaxBytes = size_t(1) << 30;
};

static TopologyCache &topology_cache()
{
    static TopologyCache c;
    return c;
}

static uint64_t hash_tets(const std::vector<int32_t> &tv)
{
    // Four independent multiply-rotate lanes over 64-bit words, folded at the
    // end: a hit is confirmed by comparing the arrays, so the hash only has to
    // spread keys, and independent lanes keep it near memory speed (a
    // byte-serial hash took about 15 ms for a million tetrahedra).
    const uint64_t m = 0x9e3779b97f4a7c15ull;
    const size_t nb = tv.size() * sizeof(int32_t);
    const unsigned char *p = reinterpret_cast<const unsigned char *>(tv.data());
    uint64_t h[4] = {0x243f6a8885a308d3ull, 0x13198a2e03707344ull, 0xa4093822299f31d0ull, 0x082efa98ec4e6c89ull};
    size_t i = 0;
    for (; i + 32 <= nb; i += 32)
        for (int j = 0; j < 4; ++j) {
            uint64_t w;
            std::memcpy(&w, p + i + 8 * j, 8);
            const uint64_t x = h[j] ^ w;
            h[j] = ((x << 29) | (x >> 35)) * m;
        }
    uint64_t r = nb;
    for (; i < nb; ++i) r = (r ^ p[i]) * 1099511628211ull;
    for (int j = 0; j < 4; ++j) {
        r = (r ^ h[j]) * m;
        r ^= r >> 31;
    }
    return r;
}

// A neighbour table of n ints, left uninitialized for its producer to fill.
static std::shared_ptr<int32_t> new_table(size_t n)
{
    return std::shared_ptr<int32_t>(new int32_t[n], std::default_delete<int32_t[]>());
}

// The cached neighbour table of this simulation's connectivity, or null;
// *hash receives the key for topology_insert.
static std::shared_ptr<const int32_t> topology_lookup(rdos_sim *s, uint64_t *hash)
{
    TopologyCache &c = topology_cache();
    const uint64_t h = hash_tets(*s->tet_verts) ^ (uint64_t)s->cell_verts;
    *hash = h;
    std::lock_guard<std::mutex> g(c.mu);
    auto range = c.entries.equal_range(h);
    for (auto it = range.first; it != range.second; ++it)
        if (it->second.cell_verts == s->cell_verts &&
            (it->second.cells == s->tet_verts || *it->second.cells == *s->tet_verts)) {
            it->second.last_use = ++c.clock;
            return it->second.nbr;
        }
    return nullptr;
}

// Adds a table made for this simulation's connectivity (least recently used
// entries make room).
static void topology_insert(rdos_sim *s, uint64_t h, std::shared_ptr<const int32_t> nbr)
{
    TopologyCache &c = topology_cache();
    std::lock_guard<std::mutex> g(c.mu);
    const size_t add = (s->tet_verts->size() + 4 * (size_t)s->T) * sizeof(int32_t);
    while (!c.entries.empty() && c.bytes + add > TopologyCache::kMaxBytes) {
        auto old = c.entries.begin();
        for (auto it = c.entries.begin(); it != c.entries.end(); ++it)
            if (it->second.last_use < old->second.last_use) old = it;
        c.bytes -= (old->second.cells->size() + 4 * (old->second.cells->size() / old->second.cell_verts)) *
                   sizeof(int32_t);
        c.entries.erase(old);
    }
    if (add > TopologyCache::kMaxBytes) return;
    TopologyCache::Entry en;
    en.cell_verts = s->cell_verts;
    en.cells = s->tet_verts;
    en.nbr = std::move(nbr);
    en.last_use = ++c.clock;
    c.entries.emplace(h, std::move(en));
    c.bytes += add;
}

// Face matching runs on the device (launch_face_match) for meshes of at least
// 16384 cells whose vertex ids pack into a 64-bit key (*bits: bits per vertex
// id).  The sort makes it O(T) where the host sort is O(T log T): about a
// second on the host for a million tetrahedra.
static bool device_match_applies(const rdos_sim *s, int32_t *bits)
{
    int32_t b = 1;
    while (b < 31 && ((int64_t)1 << b) < (int64_t)s->n_verts) ++b;
    *bits = b;
    return s->T >= 16384 && !(s->cell_verts == 4 && b > 21) && (int64_t)s->T * 4 <= 0x7fffffff;
}

rdos_status build_topology_uncached(rdos_sim *s, std::vector<int32_t> &nbr);

// Edge matching for a surface of triangles: each edge (opposite local vertex
// e) keyed by its sorted vertex pair; slot 3 of every triangle is a boundary.
static rdos_status build_edges(rdos_sim *s, std::vector<int32_t> &nbr)
{
    struct EdgeKey {
        int32_t a, b;
        int32_t slot;  // 4 * triangle + edge
    };
    const int32_t T = s->T;
    std::vector<EdgeKey> keys((size_t)T * 3);
    for (int32_t t = 0; t < T; ++t) {
        const int32_t *v = &(*s->tet_verts)[3 * (size_t)t];
        for (int e = 0; e < 3; ++e) {
            const int32_t p = v[e == 0 ? 1 : 0], q = v[e <= 1 ? 2 : 1];
            keys[3 * (size_t)t + e] = {std::min(p, q), std::max(p, q), 4 * t + e};
        }
    }
    std::sort(keys.begin(), keys.end(), [](const EdgeKey &x, const EdgeKey &y) {
        if (x.a != y.a) return x.a < y.a;
        if (x.b != y.b) return x.b < y.b;
        return x.slot < y.slot;
    });
    nbr.assign((size_t)T * 4, -1);
    for (size_t i = 0; i < keys.size();) {
        size_t j = i + 1;
        while (j < keys.size() && keys[j].a == keys[i].a && keys[j].b == keys[i].b) ++j;
        if (j - i > 2)
            return fail(s, RDOS_EINVAL, "edge (%d,%d) is shared by %zu triangles", keys[i].a, keys[i].b, j - i);
        if (j - i == 2) {
            const int32_t t0 = keys[i].slot / 4, t1 = keys[i + 1].slot / 4;
            if (t0 == t1) return fail(s, RDOS_EINVAL, "triangle %d repeats an edge", t0);
            nbr[keys[i].slot] = t1;
            nbr[keys[i + 1].slot] = t0;
        }
        i = j;
    }
    return RDOS_OK;
}

// Face matching: each face is keyed by its sorted vertex triple; two tets with
// the same key are neighbours across it.  A key seen three times is an error.
rdos_status build_topology_uncached(rdos_sim *s, std::vector<int32_t> &nbr)
{
    if (s->cell_verts == 3) return build_edges(s, nbr);
    struct FaceKey {
        int32_t a, b, c;
        int32_t slot;  // 4 * tet + face
    };
    const int32_t T = s->T;
    std::vector<FaceKey> keys((size_t)T * 4);
    for (int32_t t = 0; t < T; ++t) {
        const int32_t *v = &(*s->tet_verts)[4 * (size_t)t];
        for (int f = 0; f < 4; ++f) {
            std::array<int32_t, 3> tri;
            int q = 0;
            for (int i = 0; i < 4; ++i)
                if (i != f) tri[q++] = v[i];
            std::sort(tri.begin(), tri.end());
            keys[4 * (size_t)t + f] = {tri[0], tri[1], tri[2], 4 * t + f};
        }
    }
    std::sort(keys.begin(), keys.end(), [](const FaceKey &x, const FaceKey &y) {
        if (x.a != y.a) return x.a < y.a;
        if (x.b != y.b) return x.b < y.b;
        if (x.c != y.c) return x.c < y.c;
        return x.slot < y.slot;
    });
    nbr.assign((size_t)T * 4, -1);
    const size_t nF = keys.size();
    for (size_t i = 0; i < nF;) {
        size_t j = i + 1;
        while (j < nF && keys[j].a == keys[i].a && keys[j].b == keys[i].b && keys[j].c == keys[i].c) ++j;
        if (j - i > 2)
            return fail(s, RDOS_EINVAL, "face (%d,%d,%d) is shared by %zu tetrahedra", keys[i].a, keys[i].b,
                        keys[i].c, j - i);
        if (j - i == 2) {
            const int32_t t0 = keys[i].slot / 4, t1 = keys[i + 1].slot / 4;
            if (t0 == t1) return fail(s, RDOS_EINVAL, "tetrahedron %d repeats a face", t0);
            nbr[keys[i].slot] = t1;
            nbr[keys[i + 1].slot] = t0;
        }
        i = j;
    }
    return RDOS_OK;
}

rdos_status upload_desc(rdos_sim *s)
{
    HIP_TRY(s, hipMemcpyAsync(s->d_desc, &s->desc, sizeof(DevSim), hipMemcpyHostToDevice, s->stream),
            "upload simulation descriptor");
    HIP_TRY(s, hipStreamSynchronize(s->stream), "upload simulation descriptor");
    return RDOS_OK;
}

// The kernels read the state of period k from buf[k & 1]; the descriptor's
// buf[] follows the handle's buffers, which swap when set_state changes the
// parity of the period index (the other buffer is all zero between periods).
rdos_status match_parity(rdos_sim *s)
{
    if (s->desc.buf[0] == s->d_buf[0] && s->desc.buf[1] == s->d_buf[1] && s->desc.mask[0] == s->d_mask[0] &&
        s->desc.mask[1] == s->d_mask[1])
        return RDOS_OK;
    s->desc.buf[0] = s->d_buf[0];
    s->desc.buf[1] = s->d_buf[1];
    s->desc.mask[0] = s->d_mask[0];
    s->desc.mask[1] = s->d_mask[1];
    return upload_desc(s);
}

// The scan reads only count vectors whose occupancy byte is set; after the
// host wrote counts, the map of the current buffer is rebuilt from them
// (and the other one cleared) before the next period runs.
rdos_status ensure_mask(rdos_sim *s)
{
    if (!s->mask_dirty) return RDOS_OK;
    const int64_t Tp = padded_tets(s->T);
    const int p = (int)(s->step & 1);
    HIP_TRY(s, launch_mask_build(s->d_buf[p], s->d_mask[p], s->d_mask[p ^ 1], occupancy_tag(s->step), s->Rz,
                                 (int32_t)s->D.size(), Tp, s->stream),
            "rebuild occupancy");
    s->mask_dirty = false;
    return RDOS_OK;
}

static rdos_status flags_status(rdos_sim *s, int32_t flags)
{
    if (flags & kFlagCrowded) s->crowded = true;
    if (flags & 1) return fail(s, RDOS_EOVERFLOW, "a molecule count overflowed int32");
    if (flags & 4) return fail(s, RDOS_EDEVICE, "occupied-tet queue overflowed (internal error)");
    if (flags & 8)
        return fail(s, RDOS_EDEVICE, "a wait between blocks of the one-launch path timed out (internal error)");
    if (flags & 2)
        return fail(s, RDOS_EOVERFLOW, "a tet fired more than %u reactions in one period; shorten tau",
                    kMaxEventsPerPeriod);
    return RDOS_OK;
}

rdos_status check_flags(rdos_sim *s)
{
    int32_t flags = 0;
    HIP_TRY(s, hipMemcpyAsync(&flags, s->d_flags, sizeof flags, hipMemcpyDeviceToHost, s->stream),
            "read flags");
    HIP_TRY(s, hipStreamSynchronize(s->stream), "synchronize");
    return flags_status(s, flags);
}

// Pinned buffers for small read-outs: a kernel writes the counts and the flags
// into one, and a single wait replaces two copies with theirs (the 750-tet
// cube, one period and its counts: 41 us a pass, 62 with the copies).  At most
// kReadBuffers of kReadBytes each while simulations are alive, taken and
// returned under a lock; a caller that finds none free copies instead.  Making
// one costs as much as several reads, so a simulation copies in its first four,
// also where a buffer made for another is free (a new simulation's first such
// pass 56 us, 91 with the queue's kernels and the copies).
class ReadBuffers {
public:
    static constexpr int kReadBuffers = 16, kFirstReads = 4;
    static constexpr size_t kReadBytes = size_t(64) << 10;
    void *take()
    {
        std::lock_guard<std::mutex> g(mu_);
        if (!free_.empty()) {
            void *p = free_.back();
            free_.pop_back();
            return p;
        }
        if (made_ >= kReadBuffers) return nullptr;
        void *p = nullptr;
        std::lock_guard<std::mutex> dg(device_api_mutex());
        if (hipHostMalloc(&p, kReadBytes, hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        ++made_;
        return p;
    }
    void give(void *p)
    {
        std::lock_guard<std::mutex> g(mu_);
        free_.push_back(p);
    }
    void simulation_made()
    {
        std::lock_guard<std::mutex> g(mu_);
        ++alive_;
    }
    void simulation_gone()  // with the last one the buffers go back
    {
        std::lock_guard<std::mutex> g(mu_);
        if (--alive_ > 0 || free_.empty()) return;
        std::lock_guard<std::mutex> dg(device_api_mutex());
        for (void *p : free_) (void)hipHostFree(p);
        made_ -= (int)free_.size();
        free_.clear();
    }

private:
    std::mutex mu_;
    std::vector<void *> free_;
    int made_ = 0;
    int64_t alive_ = 0;
};
// Not destroyed: simulations may be, at the end of the process, after what was
// made with the first of them.
static ReadBuffers &read_buffers()
{
    alignas(ReadBuffers) static unsigned char room[sizeof(ReadBuffers)];
    static ReadBuffers &b = *new (room) ReadBuffers;
    return b;
}

rdos_status enqueue_period(rdos_sim *s, int64_t period, int64_t partial, double tau_last)
{
    rdos_status st = ensure_mask(s);
    if (st != RDOS_OK) return st;
    if (s->launch_mode == 3 && s->queue.species <= kFusedSpecies) {
        // one fused launch; the queue's length halves stay as they are, so
        // the two-launch path that may follow keeps its parity
        HIP_TRY(s, launch_fused(s->d_desc, s->d_tiles, period, partial, tau_last, s->queue,
                                scan_blocks_for(s->n_tiles), s->stream),
                "launch period");
        return RDOS_OK;
    }
    HIP_TRY(s, launch_step(s->d_desc, s->d_tiles, period, partial, tau_last, s->queue, (int32_t)(s->launches & 1),
                           scan_blocks_for(s->n_tiles), s->update_bps, s->queue.nseg, s->stream),
            "launch period");
    s->launches += 1;
    return RDOS_OK;
}

// Grid of the one-launch path for this simulation, or 0 when it does not
// apply (launch mode 0: work lists of at most kPersistTiles tiles; 1 and 3:
// never; 2: always).  Blocks beyond what a cooperative launch may hold stride over
// the tiles and queue segments.
int32_t persist_grid(rdos_sim *s)
{
    if (s->launch_mode == 1 || s->launch_mode == 3 || (s->launch_mode == 0 && s->n_tiles > kPersistTiles)) return 0;
    if (s->persist_limit < 0) s->persist_limit = persist_grid_limit(s->queue);
    // four blocks per queue segment, so that a segment's tets are shared by
    // 1024 lanes
    const int32_t need = std::max(4 * s->queue.nseg, scan_blocks_for(s->n_tiles));
    return s->persist_limit > 0 ? std::min(need, s->persist_limit) : 0;
}

// The turns of the process's devices.  The books and the words that kernels
// write stay until the process ends (a simulation destroyed at its exit finds
// them); a device's word is made with its first finalized simulation or engine.
namespace {
constexpr int kTurnDevices = 64;
struct Turns {
    LaunchTurn turn[kTurnDevices];
    unsigned long long *ended[kTurnDevices] = {};  // pinned host memory
    const TurnOwner *last[kTurnDevices] = {};      // of the last launch, where others may wait for it
    StreamOwners owners;
};
Turns &turns()  // guarded by device_api_mutex()
{
    alignas(Turns) static unsigned char room[sizeof(Turns)];
    static Turns &t = *new (room) Turns;
    return t;
}
}  // namespace

void prepare_turns(int device)
{
    std::lock_guard<std::mutex> g(device_api_mutex());
    Turns &t = turns();
    if (device < 0 || device >= kTurnDevices || t.ended[device]) return;
    void *p = nullptr;
    if (hipHostMalloc(&p, sizeof(unsigned long long), hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();  // without a word nobody has a turn, and the queue runs the periods
        return;
    }
    t.ended[device] = static_cast<unsigned long long *>(p);
    *t.ended[device] = 0;
}

void join_own_stream(TurnOwner *owner, hipStream_t stream)
{
    std::lock_guard<std::mutex> g(device_api_mutex());
    *owner = TurnOwner{};
    owner->number = turns().owners.own_stream();
    owner->stream = stream;
    if (hipEventCreateWithFlags(&owner->event, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();  // without one, nobody waits for its launches on the device
        owner->event = nullptr;
    }
}

void leave_own_stream(TurnOwner *owner)
{
    std::lock_guard<std::mutex> g(device_api_mutex());
    for (const TurnOwner *&last : turns().last)
        if (last == owner) last = nullptr;
    if (owner->event) (void)hipEventDestroy(owner->event);
    owner->event = nullptr;
}

// The simulation as an owner of turns, when it gets its stream, and before it
// gives the stream up (drained).  The per-thread stream is another one in
// every thread.
static void join_stream(rdos_sim *s)
{
    if (s->own_stream) return join_own_stream(&s->turn, s->stream);
    std::lock_guard<std::mutex> g(device_api_mutex());
    StreamOwners &owners = turns().owners;
    s->turn = TurnOwner{};
    s->turn.number = s->stream == hipStreamPerThread ? owners.own_stream() : owners.join(s->stream);
}
static void leave_stream(rdos_sim *s)
{
    if (!s->stream || s->own_stream) return leave_own_stream(&s->turn);
    if (s->stream == hipStreamPerThread) return;
    std::lock_guard<std::mutex> g(device_api_mutex());
    turns().owners.leave(s->stream);
}

// Runs `launch`, of n_periods periods on the owner's stream, with the
// LaunchEnd of its turn, or behind the last launch where it should wait and
// that one's event can be waited for.
template <class Launch>
static hipError_t launch_in_turn(int device, TurnOwner *owner, bool wait, int32_t n_periods, hipStream_t st,
                                 Launch launch)
{
    std::lock_guard<std::mutex> g(device_api_mutex());
    Turns &t = turns();
    if (device < 0 || device >= kTurnDevices || !t.ended[device]) return hipErrorNotReady;
    LaunchTurn &turn = t.turn[device];
    LaunchEnd end;
    end.word = t.ended[device];
    const uint64_t ended = __atomic_load_n(end.word, __ATOMIC_RELAXED);
    end.number = turn.take(owner->number, ended, n_periods);
    if (end.number == 0) {
        // only streams of the library's own wait, for each other: nothing else can hold them up
        const TurnOwner *last = t.last[device];
        if (!wait || !owner->event || !last || !turn.worth_waiting(ended, owner->last, n_periods))
            return hipErrorNotReady;
        if (hipEventRecord(last->event, last->stream) != hipSuccess ||
            hipStreamWaitEvent(st, last->event, 0) != hipSuccess) {
            (void)hipGetLastError();
            return hipErrorNotReady;
        }
        end.number = turn.take_behind(owner->number, n_periods);
    }
    const hipError_t e = launch(end);
    if (e != hipSuccess) {
        turn.give_back();
        return e;
    }
    owner->last = end.number;
    t.last[device] = owner->event ? owner : nullptr;
    return hipSuccess;
}

hipError_t launch_resident_in_turn(int device, TurnOwner *owner, bool wait, const DevSim *sims,
                                   const ResidentPlan &plan, int64_t iter0, int32_t n_periods, int64_t partial,
                                   double tau_last, uint64_t epoch, hipStream_t st, uint32_t *crowded)
{
    const auto launch = [&](LaunchEnd end) {
        end.crowded = crowded;
        return launch_resident(sims, plan, iter0, n_periods, partial, tau_last, epoch, end, st);
    };
    return plan.max_parts <= 1 ? launch(LaunchEnd{}) : launch_in_turn(device, owner, wait, n_periods, st, launch);
}

// len periods from the current one by the one-launch path over the queue.  A
// captured launch runs when its owner replays it, out of turn.
static hipError_t launch_persist_in_turn(rdos_sim *s, int32_t len, int64_t partial, double tau_last, int32_t grid)
{
    const auto launch = [&](const LaunchEnd &end) {
        return launch_persist(s->d_desc, s->d_tiles, s->step, len, (int32_t)(s->launches & 1), partial, tau_last,
                              s->queue, grid, s->queue.sync, end, s->stream);
    };
    return capturing(s) ? launch(LaunchEnd{}) : launch_in_turn(s->device, &s->turn, true, len, s->stream, launch);
}

// n periods from the current one; the last lasts tau_last when `partial`
// (Algorithm 1, Step 1), all others tau.  Where another's launch has the
// device, this one's waits for it on the device or leaves a few periods to the
// queue and asks again.  That is so for one thread that steps several
// simulations too, since calls return before their periods have run.  Two
// simulations stepped in turn, 100 periods a call, us for a call of each, with
// all of the second's periods over the queue, with both over the queue, and
// so: 2058 tets of three species 11900, 9770 and 4130; 384,000 tets 3560, 3240
// and 2520; the bar of 1080 tets 10500, 12800 and 4490.
constexpr int64_t kBesidePeriods = 8;
rdos_status enqueue_run(rdos_sim *s, int64_t n, bool partial, double tau_last)
{
    if (n <= 0) return RDOS_OK;
    const int64_t partial_index = partial ? s->step + n - 1 : -1;
    const ResidentPlan *plan = resident_for(s, n);
    const int32_t grid = plan ? 0 : persist_grid(s);
    while (n > 0) {
        int64_t over_queue = n;  // by two launches per period (or mode 3's one)
        if (plan || grid > 0) {
            const int32_t len = (int32_t)std::min<int64_t>(n, kPersistPeriods);
            hipError_t e;
            if (plan) {
                e = launch_resident_in_turn(s->device, &s->turn, true, s->d_desc, *plan, s->step, len, partial_index,
                                            tau_last, s->resident_epoch, s->stream, nullptr);
            } else {
                const rdos_status st = ensure_mask(s);
                if (st != RDOS_OK) return st;
                e = launch_persist_in_turn(s, len, partial_index, tau_last, grid);
            }
            if (e == hipSuccess) {
                if (plan) {
                    s->short_run |= !plan->full;
                    s->mask_dirty = false;  // the kernel reads the counts and writes the occupancy bytes
                    s->resident_epoch += len;
                } else {
                    s->launches += len;
                }
                s->step += len;
                n -= len;
                continue;
            }
            if (e != hipErrorNotReady) return hip_fail(s, e, "launch periods");
            over_queue = std::min(n, kBesidePeriods);
        }
        for (; over_queue > 0; --over_queue, --n) {
            const bool last = s->step == partial_index;
            const rdos_status st = enqueue_period(s, s->step, last ? s->step : -1, last ? tau_last : 0.0);
            if (st != RDOS_OK) return st;
            s->step += 1;
        }
    }
    return RDOS_OK;
}

double time_of(const rdos_sim *s, int64_t k)
{
    return s->anchor_t + (double)(k - s->anchor_step) * s->tau;
}

void free_device(rdos_sim *s)
{
    (void)hipSetDevice(s->device);
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    leave_stream(s);
    std::lock_guard<std::mutex> g(device_api_mutex());
    void *ptrs[] = {s->d_mesh,           s->d_state, s->d_desc, s->d_tiles, s->d_allowed, s->resident_one.done,
                    s->resident_many.done};
    for (void *p : ptrs) dev_free(p, s->stream);
    free_queue(&s->queue, s->stream);
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    s->d_mask[0] = s->d_mask[1] = nullptr;
    s->d_mesh = nullptr;
    s->d_state = nullptr;
    s->d_allowed = nullptr;
    s->d_buf[0] = s->d_buf[1] = s->d_flags = nullptr;
    s->d_desc = nullptr;
    s->d_tiles = nullptr;
    s->resident_one = s->resident_many = ResidentPlan{};
    if (s->stream && s->own_stream) (void)hipStreamDestroy(s->stream);
    s->stream = nullptr;
}

}  // namespace rdos

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
#define CHECK_HANDLE(s)                                   \
    do {                                                  \
        if (!(s)) return RDOS_EINVAL;                     \
        if ((s)->engine_owned) return fail(s, RDOS_EBUSY, "simulation is owned by an engine"); \
    } while (0)

extern "C" {

rdos_status rdos_create(rdos_sim **out, int device, uint64_t seed, int32_t n_realizations)
{
    if (!out) return RDOS_EINVAL;
    *out = nullptr;
    if (n_realizations < 1) return RDOS_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return RDOS_EDEVICE;
    rdos_sim *s = new (std::nothrow) rdos_sim();
    if (!s) return RDOS_ENOMEM;
    s->device = device;
    s->seed = seed;
    s->Rz = n_realizations;
    read_buffers().simulation_made();
    *out = s;
    return RDOS_OK;
}

rdos_status rdos_set_mesh(rdos_sim *s, int32_t n_verts, const double *xyz, int32_t n_tets,
                          const int32_t *tet_verts)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Created) return fail(s, RDOS_ESTATE, "set_mesh after the mesh was set");
    if (n_verts < 4 || n_tets < 1 || !xyz || !tet_verts)
        return fail(s, RDOS_EINVAL, "mesh needs >= 4 vertices and >= 1 tetrahedron");
    const int64_t off = first_not_finite(xyz, 3 * (int64_t)n_verts);
    if (off >= 0) return fail(s, RDOS_EINVAL, "vertex coordinate %lld is not finite", (long long)off);
    const int64_t id = first_not_below(tet_verts, 4 * (int64_t)n_tets, n_verts);
    if (id >= 0) return fail(s, RDOS_EINVAL, "vertex id %d out of range at %lld", tet_verts[id], (long long)id);
    s->xyz.assign(xyz, xyz + 3 * (size_t)n_verts);
    s->tet_verts = std::make_shared<const std::vector<int32_t>>(tet_verts, tet_verts + 4 * (size_t)n_tets);
    s->n_verts = n_verts;
    s->T = n_tets;
    s->state = SimState::Meshed;
    return RDOS_OK;
}

rdos_status rdos_set_surface_mesh(rdos_sim *s, int32_t n_verts, const double *xyz, int32_t n_tris,
                                  const int32_t *tri_verts)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Created) return fail(s, RDOS_ESTATE, "set_surface_mesh after the mesh was set");
    if (n_verts < 3 || n_tris < 1 || !xyz || !tri_verts)
        return fail(s, RDOS_EINVAL, "surface needs >= 3 vertices and >= 1 triangle");
    const int64_t off = first_not_finite(xyz, 3 * (int64_t)n_verts);
    if (off >= 0) return fail(s, RDOS_EINVAL, "vertex coordinate %lld is not finite", (long long)off);
    const int64_t id = first_not_below(tri_verts, 3 * (int64_t)n_tris, n_verts);
    if (id >= 0) return fail(s, RDOS_EINVAL, "vertex id %d out of range at %lld", tri_verts[id], (long long)id);
    s->xyz.assign(xyz, xyz + 3 * (size_t)n_verts);
    s->tet_verts = std::make_shared<const std::vector<int32_t>>(tri_verts, tri_verts + 3 * (size_t)n_tris);
    s->cell_verts = 3;
    s->n_verts = n_verts;
    s->T = n_tris;
    s->state = SimState::Meshed;
    return RDOS_OK;
}

rdos_status rdos_add_species(rdos_sim *s, double D, int32_t *out_id)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Meshed) return fail(s, RDOS_ESTATE, "add_species needs a mesh and no finalize yet");
    if (!(D >= 0.0) || !std::isfinite(D)) return fail(s, RDOS_EINVAL, "D must be finite and >= 0");
    if ((int)s->D.size() >= kMaxSpecies) return fail(s, RDOS_EINVAL, "at most %d species", kMaxSpecies);
    s->D.push_back(D);
    if (out_id) *out_id = (int32_t)s->D.size() - 1;
    return RDOS_OK;
}

rdos_status rdos_add_reaction(rdos_sim *s, int32_t n_reac, const int32_t *reac, int32_t n_prod,
                              const int32_t *prod, double k, int32_t *out_id)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Meshed) return fail(s, RDOS_ESTATE, "add_reaction needs a mesh and no finalize yet");
    if (n_reac < 0 || n_reac > 2 || n_prod < 0 || n_prod > 3)
        return fail(s, RDOS_EINVAL, "0..2 reactants and 0..3 products");
    if ((n_reac && !reac) || (n_prod && !prod)) return fail(s, RDOS_EINVAL, "null species list");
    if (!(k >= 0.0) || !std::isfinite(k)) return fail(s, RDOS_EINVAL, "rate constant must be finite and >= 0");
    if ((int)s->rx.size() >= kMaxReactions) return fail(s, RDOS_EINVAL, "at most %d reactions", kMaxReactions);
    Reaction r;
    r.rn = n_reac;
    r.pn = n_prod;
    for (int i = 0; i < n_reac; ++i) {
        if (reac[i] < 0 || reac[i] >= (int32_t)s->D.size()) return fail(s, RDOS_EINVAL, "reactant id out of range");
        r.r[i] = reac[i];
    }
    for (int i = 0; i < n_prod; ++i) {
        if (prod[i] < 0 || prod[i] >= (int32_t)s->D.size()) return fail(s, RDOS_EINVAL, "product id out of range");
        r.p[i] = prod[i];
    }
    r.k = k;
    s->rx.push_back(r);
    if (out_id) *out_id = (int32_t)s->rx.size() - 1;
    return RDOS_OK;
}

rdos_status rdos_set_method(rdos_sim *s, int32_t occupancy_correction, int32_t split_threshold,
                            int32_t tau_outliers)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Meshed) return fail(s, RDOS_ESTATE, "set_method needs a mesh and no finalize yet");
    if (split_threshold < 1 || tau_outliers < 0)
        return fail(s, RDOS_EINVAL, "split_threshold must be >= 1 and tau_outliers >= 0");
    s->first_order = occupancy_correction ? 0 : 1;
    s->split_threshold = split_threshold;
    s->tau_outliers = tau_outliers;
    return RDOS_OK;
}

rdos_status rdos_set_transfer_form(rdos_sim *s, int32_t form)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Meshed)
        return fail(s, RDOS_ESTATE, "set_transfer_form needs a mesh and no finalize yet");
    if (form != 0 && form != 1) return fail(s, RDOS_EINVAL, "transfer form must be 0 or 1");
    s->transfer_form = form;
    return RDOS_OK;
}

rdos_status rdos_set_reaction_region(rdos_sim *s, int32_t reaction, int32_t n_tets, const int32_t *tets)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Meshed)
        return fail(s, RDOS_ESTATE, "set_reaction_region needs a mesh and no finalize yet");
    if (reaction < 0 || reaction >= (int32_t)s->rx.size()) return fail(s, RDOS_EINVAL, "reaction id out of range");
    if (n_tets < 0 || (n_tets > 0 && !tets)) return fail(s, RDOS_EINVAL, "bad tet list");
    std::vector<int32_t> v(tets, tets + n_tets);
    for (int32_t t : v)
        if (t < 0 || t >= s->T) return fail(s, RDOS_EINVAL, "tet id %d out of range", t);
    s->regions[reaction] = std::move(v);
    return RDOS_OK;
}

rdos_status rdos_finalize(rdos_sim *s, double tau_scale, double *out_tau)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Meshed) return fail(s, RDOS_ESTATE, "finalize needs a mesh and must run once");
    if (s->D.empty()) return fail(s, RDOS_EINVAL, "no species");
    if (!(tau_scale > 0.0 && tau_scale <= 1.0)) return fail(s, RDOS_EINVAL, "tau_scale must be in (0, 1]");
    for (const Reaction &r : s->rx)
        for (int i = 0; i < r.pn; ++i)
            if (r.p[i] >= (int32_t)s->D.size()) return fail(s, RDOS_EINVAL, "product id out of range");
    // one realization's counts are addressed with 32-bit byte offsets
    if ((int64_t)s->D.size() * padded_tets(s->T) * 4 > 0x7fffffff)
        return fail(s, RDOS_EINVAL, "tets x species of one realization exceed 2^29");
    // queue entries are int32 (tile * kTetsPerTile + offset): the tiled work
    // list, not only realizations x tets, must stay below 2^31
    if (tiles_of(s) * kTetsPerTile > 0x7fffffff)
        return fail(s, RDOS_EINVAL, "realizations x tiled tets exceed 2^31");
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    if (!s->stream) {
        HIP_TRY(s, hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking), "create stream");
        s->own_stream = true;
        join_stream(s);
    }
    // Face matching (step a0): the cached table of this connectivity, else
    // matching on the device in the set-up buffers below, else on the host.
    const int32_t T = s->T;
    const size_t nbr_n = 4 * (size_t)T;
    uint64_t topo_hash = 0;
    std::shared_ptr<const int32_t> nbr_table = topology_lookup(s, &topo_hash);
    const bool fresh = !nbr_table;
    int32_t bits = 0;
    bool on_device = fresh && device_match_applies(s, &bits);
    rdos_status st = RDOS_OK;
    if (fresh && !on_device) {
        std::vector<int32_t> host;
        st = build_topology_uncached(s, host);
        if (st != RDOS_OK) return st;
        std::shared_ptr<int32_t> t = new_table(nbr_n);
        std::memcpy(t.get(), host.data(), nbr_n * sizeof(int32_t));
        nbr_table = t;
    }
    const int S = (int)s->D.size();
    const int64_t Tp = padded_tets(T);
    const size_t count_bytes = (size_t)s->Rz * S * (size_t)Tp * sizeof(int32_t);
    const size_t mask_bytes = (size_t)s->Rz * S * mask_stride(Tp);

    // temporary set-up buffers, one allocation: each place 256-byte aligned
    char *setup = nullptr;
    size_t setup_bytes = 0;
    const auto place = [&](size_t bytes) {
        const size_t at = setup_bytes;
        setup_bytes += (std::max<size_t>(bytes, 1) + 255) & ~(size_t)255;
        return at;
    };
    const size_t at_xyz = place(s->xyz.size() * sizeof(double)), at_tv = place(s->tet_verts->size() * sizeof(int32_t)),
                 at_nbr = place(nbr_n * sizeof(int32_t)), at_vol = place((size_t)T * sizeof(double)),
                 at_bc = place((size_t)T * 3 * sizeof(double)), at_area = place((size_t)T * 4 * sizeof(double)),
                 at_D = place((size_t)S * sizeof(double)), at_tau = place(sizeof(unsigned long long)),
                 at_err = place(sizeof(int32_t)),
                 at_match = place(on_device ? face_match_scratch_bytes(T, s->cell_verts) : 0);
    std::unique_lock<std::mutex> alloc_lock(device_api_mutex(), std::defer_lock);
    auto cleanup = [&]() {
        if (s->stream) (void)hipStreamSynchronize(s->stream);
        std::unique_lock<std::mutex> g(device_api_mutex(), std::defer_lock);
        if (!alloc_lock.owns_lock()) g.lock();
        dev_free(setup, s->stream);
    };
#define SETUP_TRY(expr, what)                               \
    do {                                                    \
        hipError_t e__ = (expr);                            \
        if (e__ != hipSuccess) {                            \
            if (alloc_lock.owns_lock()) alloc_lock.unlock(); \
            cleanup();                                      \
            free_device(s);                                 \
            return hip_fail(s, e__, what);                  \
        }                                                   \
    } while (0)
    alloc_lock.lock();
    SETUP_TRY(dev_alloc((void **)&s->d_mesh, (size_t)T * sizeof(MeshRec), s->stream), "allocate mesh tables");
    // counts, occupancy maps and flags: one allocation, cleared together
    const size_t count_room = (count_bytes + 255) & ~(size_t)255, mask_room = (mask_bytes + 255) & ~(size_t)255;
    SETUP_TRY(dev_alloc((void **)&s->d_state, 2 * (count_room + mask_room) + 64, s->stream), "allocate counts");
    for (int b = 0; b < 2; ++b) {
        s->d_buf[b] = reinterpret_cast<int32_t *>(s->d_state + b * count_room);
        s->d_mask[b] = reinterpret_cast<uint8_t *>(s->d_state + 2 * count_room + b * mask_room);
    }
    s->d_flags = reinterpret_cast<int32_t *>(s->d_state + 2 * (count_room + mask_room));
    SETUP_TRY(dev_alloc((void **)&s->d_desc, sizeof(DevSim), s->stream), "allocate descriptor");
    SETUP_TRY(dev_alloc((void **)&s->d_tiles, (size_t)tiles_of(s) * sizeof(Tile), s->stream), "allocate work list");
    SETUP_TRY(alloc_queue(&s->queue, tiles_of(s), S, s->stream), "allocate queue");
    s->queue.owned = tiles_of(s) <= kMaxSegments ? 1 : 0;  // a segment and a scan wavefront per tile
    SETUP_TRY(dev_alloc((void **)&setup, setup_bytes, s->stream), "allocate set-up");
    alloc_lock.unlock();
    double *d_xyz = reinterpret_cast<double *>(setup + at_xyz), *d_vol = reinterpret_cast<double *>(setup + at_vol),
           *d_bc = reinterpret_cast<double *>(setup + at_bc), *d_area = reinterpret_cast<double *>(setup + at_area),
           *d_D = reinterpret_cast<double *>(setup + at_D);
    int32_t *d_tv = reinterpret_cast<int32_t *>(setup + at_tv), *d_nbr = reinterpret_cast<int32_t *>(setup + at_nbr),
            *d_match_err = reinterpret_cast<int32_t *>(setup + at_err);
    void *d_match = setup + at_match;
    unsigned long long *d_tau = reinterpret_cast<unsigned long long *>(setup + at_tau);
    SETUP_TRY(hipMemsetAsync(s->d_state, 0, 2 * (count_room + mask_room) + 64, s->stream), "clear counts");
    SETUP_TRY(hipMemsetAsync(d_tau, 0xff, sizeof(unsigned long long), s->stream), "clear tau");
    SETUP_TRY(hipMemcpyAsync(d_xyz, s->xyz.data(), s->xyz.size() * sizeof(double), hipMemcpyHostToDevice, s->stream),
              "upload vertices");
    SETUP_TRY(hipMemcpyAsync(d_tv, s->tet_verts->data(), s->tet_verts->size() * sizeof(int32_t),
                             hipMemcpyHostToDevice, s->stream),
              "upload tetrahedra");
    if (on_device) {
        // keys of each face's sorted vertex ids, a radix sort, pairs of equal keys
        int32_t match_err = 1;
        SETUP_TRY(hipMemsetAsync(d_nbr, 0xff, nbr_n * sizeof(int32_t), s->stream), "face matching");
        SETUP_TRY(hipMemsetAsync(d_match_err, 0, sizeof(int32_t), s->stream), "face matching");
        SETUP_TRY(launch_face_match(d_tv, T, s->cell_verts, bits, d_nbr, d_match, d_match_err, s->stream),
                  "face matching");
        SETUP_TRY(hipMemcpyAsync(&match_err, d_match_err, sizeof(int32_t), hipMemcpyDeviceToHost, s->stream),
                  "face matching");
        SETUP_TRY(hipStreamSynchronize(s->stream), "face matching");
        if (match_err == 0) {
            // the table stays on the device for the geometry pass; a host copy goes to the cache
            std::shared_ptr<int32_t> t = new_table(nbr_n);
            SETUP_TRY(hipMemcpyAsync(t.get(), d_nbr, nbr_n * sizeof(int32_t), hipMemcpyDeviceToHost, s->stream),
                      "read neighbours");
            nbr_table = t;
        } else {
            // a bad face: the host matching names the first one in key order
            std::vector<int32_t> host;
            st = build_topology_uncached(s, host);
            if (st != RDOS_OK) {
                cleanup();
                free_device(s);
                return st;
            }
            std::shared_ptr<int32_t> t = new_table(nbr_n);
            std::memcpy(t.get(), host.data(), nbr_n * sizeof(int32_t));
            nbr_table = t;
            on_device = false;
        }
    }
    if (!on_device)
        SETUP_TRY(hipMemcpyAsync(d_nbr, nbr_table.get(), nbr_n * sizeof(int32_t), hipMemcpyHostToDevice, s->stream),
                  "upload neighbours");
    SETUP_TRY(hipMemcpyAsync(d_D, s->D.data(), (size_t)S * sizeof(double), hipMemcpyHostToDevice, s->stream),
              "upload D");
    if (s->cell_verts == 3)
        SETUP_TRY(launch_geometry_tri(d_xyz, d_tv, d_nbr, T, d_vol, d_bc, d_area, s->d_mesh, s->d_flags + 1,
                                      s->stream),
                  "geometry");
    else
        SETUP_TRY(launch_geometry(d_xyz, d_tv, d_nbr, T, d_vol, d_bc, d_area, s->d_mesh, s->d_flags + 1, s->stream),
                  "geometry");
    if (s->tau_outliers > 0) {
        // Sec. II.A outlier relaxation: the (k+1)-th smallest 1/(D g) sets tau
        void *scratch = nullptr;
        hipError_t e_sel;
        {
            std::lock_guard<std::mutex> g(device_api_mutex());
            e_sel = dev_alloc(&scratch, tau_select_scratch_bytes(T, S), s->stream);
        }
        if (e_sel == hipSuccess) {
            e_sel = launch_tau_select(s->d_mesh, T, d_D, S, s->tau_outliers, scratch, d_tau, s->stream);
            (void)hipStreamSynchronize(s->stream);
            std::lock_guard<std::mutex> g(device_api_mutex());
            dev_free(scratch, s->stream);
        }
        SETUP_TRY(e_sel, "tau selection");
    } else {
        SETUP_TRY(launch_tau_min(s->d_mesh, T, d_D, S, d_tau, s->stream), "tau");
    }
    unsigned long long tau_bits = 0;
    int32_t bad[2] = {0, 0};
    SETUP_TRY(hipMemcpyAsync(&tau_bits, d_tau, sizeof tau_bits, hipMemcpyDeviceToHost, s->stream), "read tau");
    SETUP_TRY(hipMemcpyAsync(bad, s->d_flags, sizeof bad, hipMemcpyDeviceToHost, s->stream), "read flags");
    SETUP_TRY(hipStreamSynchronize(s->stream), "set-up");
    SETUP_TRY(hipMemsetAsync(s->d_flags, 0, 64, s->stream), "clear flags");
    cleanup();
#undef SETUP_TRY
    if (bad[1]) {
        free_device(s);
        return fail(s, RDOS_EINVAL, s->cell_verts == 3 ? "degenerate triangle (zero area)"
                                                       : "degenerate tetrahedron (zero volume)");
    }
    if (tau_bits == ~0ull) {
        free_device(s);
        return fail(s, RDOS_EINVAL, "no diffusing species on a connected cell: tau is undefined");
    }
    double tmin;
    std::memcpy(&tmin, &tau_bits, sizeof tmin);
    s->tau = tau_scale * tmin;

    // kernel-side description
    DevSim &d = s->desc;
    std::memset(&d, 0, sizeof d);
    d.mesh = s->d_mesh;
    d.buf[0] = s->d_buf[0];
    d.buf[1] = s->d_buf[1];
    d.mask[0] = s->d_mask[0];
    d.mask[1] = s->d_mask[1];
    d.flags = s->d_flags;
    d.T = T;
    d.mstride = mask_stride(Tp);
    d.S = S;
    d.R = (int32_t)s->rx.size();
    d.Rz = s->Rz;
    d.key0 = (uint32_t)s->seed;
    d.key1 = (uint32_t)(s->seed >> 32);
    d.tau = s->tau;
    d.step0 = 0;
    d.step_end = std::numeric_limits<int64_t>::max();
    for (int m = 0; m < S; ++m) {
        d.D[m] = s->D[m];
        if (s->D[m] > 0.0) d.diff_mask |= 1u << m;
    }
    d.first_order = s->first_order ? 1u : 0u;
    d.split_threshold = s->split_threshold;
    d.transfer_form = s->transfer_form;
    s->queue.scaled = s->transfer_form == 1 ? 1 : 0;
    if (!s->regions.empty()) {
        std::vector<uint32_t> allowed((size_t)T, 0xFFFFFFFFu);
        for (const auto &kv : s->regions) {
            const uint32_t bit = 1u << kv.first;
            for (uint32_t &a : allowed) a &= ~bit;
            for (int32_t t : kv.second) allowed[t] |= bit;
        }
        hipError_t e_al;
        {
            std::lock_guard<std::mutex> g(device_api_mutex());
            e_al = dev_alloc((void **)&s->d_allowed, allowed.size() * sizeof(uint32_t), s->stream);
        }
        if (e_al == hipSuccess)
            e_al = hipMemcpyAsync(s->d_allowed, allowed.data(), allowed.size() * sizeof(uint32_t),
                                  hipMemcpyHostToDevice, s->stream);
        if (e_al == hipSuccess) e_al = hipStreamSynchronize(s->stream);
        if (e_al != hipSuccess) {
            free_device(s);
            return hip_fail(s, e_al, "upload reaction regions");
        }
        d.allowed = s->d_allowed;
    }
    for (size_t q = 0; q < s->rx.size(); ++q) {
        const Reaction &r = s->rx[q];
        d.rn[q] = r.rn;
        d.pn[q] = r.pn;
        d.r0[q] = r.rn > 0 ? r.r[0] : -1;
        d.r1[q] = r.rn > 1 ? r.r[1] : -1;
        d.p0[q] = r.pn > 0 ? r.p[0] : -1;
        d.p1[q] = r.pn > 1 ? r.p[1] : -1;
        d.p2[q] = r.pn > 2 ? r.p[2] : -1;
        uint32_t inv = 0;
        for (int i = 0; i < r.rn; ++i) inv |= 1u << r.r[i];
        for (int i = 0; i < r.pn; ++i) inv |= 1u << r.p[i];
        d.involved[q] = inv;
        d.k[q] = r.k;
        if (r.rn == 0) d.zeroth = 1;
    }
    // the work list (one tile per 1024 tets of each realization), its header
    // and the descriptor, written by one kernel: nothing to upload and wait for
    s->n_tiles = (int32_t)tiles_of(s);
    st = RDOS_OK;
    hipError_t e = launch_own_work(d, s->d_desc, queue_header(&s->queue, s->n_tiles, 1, 0), s->queue.hdr, s->d_tiles,
                                   s->stream);
    if (e != hipSuccess) st = hip_fail(s, e, "work list");
    prepare_turns(s->device);
    if (st == RDOS_OK) st = plan_resident(s, cut_one(s), &s->resident_one);
    if (st == RDOS_OK) st = plan_resident(s, cut_many(s), &s->resident_many);
    if (st != RDOS_OK) {
        free_device(s);
        return st;
    }
    if (fresh) topology_insert(s, topo_hash, std::move(nbr_table));  // the read-back was waited for above
    s->state = SimState::Ready;
    s->step = 0;
    s->anchor_step = 0;
    s->anchor_t = 0.0;
    s->totals.assign((size_t)s->Rz * S, 0);
    s->species_totals.assign((size_t)S, 0);
    // counts staged before finalize
    for (auto &kv : s->staged) {
        const int32_t r = kv.first / kMaxSpecies, m = kv.first % kMaxSpecies;
        int32_t *dst = s->d_buf[0] + ((int64_t)r * S + m) * Tp;
        HIP_TRY(s, hipMemcpyAsync(dst, kv.second.data(), (size_t)T * sizeof(int32_t), hipMemcpyHostToDevice, s->stream),
                "upload counts");
        for (int32_t c : kv.second) s->totals[(size_t)r * S + m] += c;
        s->species_totals[m] += s->totals[(size_t)r * S + m];
    }
    HIP_TRY(s, hipStreamSynchronize(s->stream), "upload counts");
    s->mask_dirty = true;
    s->staged.clear();
    s->xyz.clear();
    s->xyz.shrink_to_fit();
    if (out_tau) *out_tau = s->tau;
    return RDOS_OK;
}

rdos_status rdos_set_counts(rdos_sim *s, int32_t realization, int32_t species, const int32_t *counts)
{
    CHECK_HANDLE(s);
    if (s->state == SimState::Created) return fail(s, RDOS_ESTATE, "set_counts needs a mesh");
    if (realization < 0 || realization >= s->Rz || species < 0 || species >= (int32_t)s->D.size() || !counts)
        return fail(s, RDOS_EINVAL, "realization or species out of range");
    int64_t negative;
    const int64_t total = sum_counts(counts, s->T, &negative);
    if (negative >= 0) return fail(s, RDOS_EINVAL, "negative count at tet %d", (int32_t)negative);
    if (total > 0x3fffffff) return fail(s, RDOS_EOVERFLOW, "more than 2^30 molecules of one species");
    if ((int64_t)s->Rz * s->T > 0x7fffffff) return fail(s, RDOS_EINVAL, "realizations x tets exceeds 2^31");
    if (s->state == SimState::Meshed) {
        s->staged[realization * kMaxSpecies + species].assign(counts, counts + s->T);
        return RDOS_OK;
    }
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    int32_t *dst = s->d_buf[s->step & 1] + ((int64_t)realization * (int64_t)s->D.size() + species) * padded_tets(s->T);
    HIP_TRY(s, hipMemcpyAsync(dst, counts, (size_t)s->T * sizeof(int32_t), hipMemcpyHostToDevice, s->stream),
            "upload counts");
    if (s->short_run) HIP_TRY(s, launch_clear_flags(s->d_flags, kFlagCrowded, s->stream), "clear flags");
    HIP_TRY(s, hipStreamSynchronize(s->stream), "upload counts");
    s->short_run = s->crowded = s->queue_faster = false;
    s->mask_dirty = true;
    int64_t &last = s->totals[(size_t)realization * s->D.size() + species];
    s->species_totals[species] += total - last;
    last = total;
    return RDOS_OK;
}

rdos_status rdos_get_counts(rdos_sim *s, int32_t realization, int32_t species, int32_t *out)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Ready) return fail(s, RDOS_ESTATE, "get_counts before finalize");
    if (realization < 0 || realization >= s->Rz || species < 0 || species >= (int32_t)s->D.size() || !out)
        return fail(s, RDOS_EINVAL, "realization or species out of range");
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    const int32_t *src =
        s->d_buf[s->step & 1] + ((int64_t)realization * (int64_t)s->D.size() + species) * padded_tets(s->T);
    const size_t bytes = (size_t)s->T * sizeof(int32_t);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    (void)hipStreamIsCapturing(s->stream, &capture);
    if (s->reads <= ReadBuffers::kFirstReads) s->reads += 1;
    void *buffer = s->reads > ReadBuffers::kFirstReads && bytes + sizeof(int32_t) <= ReadBuffers::kReadBytes &&
                           capture == hipStreamCaptureStatusNone
                       ? read_buffers().take()
                       : nullptr;
    if (!buffer) {
        HIP_TRY(s, hipMemcpyAsync(out, src, bytes, hipMemcpyDeviceToHost, s->stream), "download counts");
        return check_flags(s);
    }
    int32_t *staged = static_cast<int32_t *>(buffer);
    hipError_t e = launch_read_counts(src, s->d_flags, staged, s->T, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    int32_t flags = 0;
    if (e == hipSuccess) {
        std::memcpy(out, staged, bytes);
        flags = staged[s->T];
    }
    read_buffers().give(buffer);
    HIP_TRY(s, e, "download counts");
    return flags_status(s, flags);
}

rdos_status rdos_device_counts(rdos_sim *s, int32_t realization, int32_t species, int32_t **out)
{
    CHECK_HANDLE(s);
    if (!out) return fail(s, RDOS_EINVAL, "null output");
    *out = nullptr;
    if (s->state != SimState::Ready) return fail(s, RDOS_ESTATE, "device_counts before finalize");
    if (realization < 0 || realization >= s->Rz || species < 0 || species >= (int32_t)s->D.size())
        return fail(s, RDOS_EINVAL, "realization or species out of range");
    *out = s->d_buf[s->step & 1] + ((int64_t)realization * (int64_t)s->D.size() + species) * padded_tets(s->T);
    s->mask_dirty = true;  // the caller may write through the view
    return RDOS_OK;
}

rdos_status rdos_set_state(rdos_sim *s, int64_t step_index, double t)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Ready) return fail(s, RDOS_ESTATE, "set_state before finalize");
    if (step_index < 0 || !std::isfinite(t)) return fail(s, RDOS_EINVAL, "bad state");
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    HIP_TRY(s, hipStreamSynchronize(s->stream), "set state");
    if ((step_index & 1) != (s->step & 1)) {  // the state moves with k & 1
        std::swap(s->d_buf[0], s->d_buf[1]);
        std::swap(s->d_mask[0], s->d_mask[1]);
    }
    s->step = step_index;
    s->anchor_step = step_index;
    s->anchor_t = t;
    s->mask_dirty = true;  // the occupancy bytes hold tags of the period index
    return match_parity(s);
}

rdos_status rdos_get_time(rdos_sim *s, double *t, int64_t *step_index)
{
    CHECK_HANDLE(s);  // an engine's worker moves the period index of the simulations it owns
    if (t) *t = time_of(s, s->step);
    if (step_index) *step_index = s->step;
    return RDOS_OK;
}

rdos_status rdos_step(rdos_sim *s, int64_t n_steps)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Ready) return fail(s, RDOS_ESTATE, "step before finalize");
    if (n_steps < 0) return fail(s, RDOS_EINVAL, "negative step count");
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    return enqueue_run(s, n_steps, false, 0.0);
}

rdos_status rdos_run_until(rdos_sim *s, double t_end)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Ready) return fail(s, RDOS_ESTATE, "run_until before finalize");
    if (!std::isfinite(t_end)) return fail(s, RDOS_EINVAL, "t_end must be finite");
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    // full periods while one more fits, then (Step 1) a last period shortened
    // to end at t_end
    int64_t k = s->step;
    while (time_of(s, k) < t_end && !(time_of(s, k) + s->tau > t_end)) ++k;
    const bool partial = time_of(s, k) < t_end;
    const double tau_last = partial ? t_end - time_of(s, k) : 0.0;
    rdos_status st = enqueue_run(s, k - s->step + (partial ? 1 : 0), partial, tau_last);
    if (st != RDOS_OK) return st;
    if (partial) {
        s->anchor_step = s->step;
        s->anchor_t = t_end;
    }
    return RDOS_OK;
}

rdos_status rdos_set_launch_mode(rdos_sim *s, int32_t mode)
{
    CHECK_HANDLE(s);
    if (mode < 0 || mode > 3) return fail(s, RDOS_EINVAL, "launch mode must be 0, 1, 2 or 3");
    s->launch_mode = mode;
    return RDOS_OK;
}

rdos_status rdos_synchronize(rdos_sim *s)
{
    CHECK_HANDLE(s);
    if (s->state != SimState::Ready) return RDOS_OK;
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    return check_flags(s);
}

rdos_status rdos_set_stream(rdos_sim *s, void *hip_stream)
{
    CHECK_HANDLE(s);
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    if (s->stream) HIP_TRY(s, hipStreamSynchronize(s->stream), "drain old stream");
    leave_stream(s);
    if (s->stream && s->own_stream) (void)hipStreamDestroy(s->stream);
    s->stream = nullptr;
    if (hip_stream) {
        s->stream = (hipStream_t)hip_stream;
        s->own_stream = false;
        join_stream(s);
    } else if (s->state == SimState::Ready) {
        HIP_TRY(s, hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking), "create stream");
        s->own_stream = true;
        join_stream(s);
    } else {
        s->stream = nullptr;
        s->own_stream = false;
    }
    return RDOS_OK;
}

rdos_status rdos_get_geometry(rdos_sim *s, int32_t *nbr, double *w, double *g, double *nav)
{
    if (!s) return RDOS_EINVAL;
    if (s->state != SimState::Ready) return fail(s, RDOS_ESTATE, "get_geometry before finalize");
    HIP_TRY(s, hipSetDevice(s->device), "set device");
    // The tables of large meshes are laid out apart on the device and copied
    // into the caller's arrays, not copied as records and taken apart on the
    // host.  Small ones are: one copy and a wait against four (750 tets 36 us
    // against 112, 10,368 73 and 119, 20,250 153 and 132; a million 15,900 and
    // 3600).  The first copy into an array is slower, by the pinning of its
    // pages: of 162,000 tets 1310 and 2130 then, and 1110 and 620 into the same
    // arrays again; a million 20,200 and 7200.
    const size_t T = (size_t)s->T;
    const size_t at_w = 16 * T, at_g = at_w + 32 * T, at_nav = at_g + 8 * T;
    char *tables = nullptr;
    if (s->T >= 16384) {
        std::lock_guard<std::mutex> g2(device_api_mutex());
        if (dev_alloc((void **)&tables, at_nav + 8 * T, s->stream) != hipSuccess) {
            (void)hipGetLastError();  // no room beside the simulation
            tables = nullptr;
        }
    }
    if (!tables) {
        std::vector<MeshRec> m(T);
        HIP_TRY(s, hipMemcpyAsync(m.data(), s->d_mesh, T * sizeof(MeshRec), hipMemcpyDeviceToHost, s->stream),
                "download mesh tables");
        HIP_TRY(s, hipStreamSynchronize(s->stream), "download mesh tables");
        for (size_t t = 0; t < T; ++t) {
            for (int f = 0; f < 4; ++f) {
                if (nbr) nbr[4 * t + f] = m[t].nbr[f];
                if (w) w[4 * t + f] = f < 3 ? m[t].w[f] : m[t].w3;
            }
            if (g) g[t] = m[t].g;
            if (nav) nav[t] = m[t].nav;
        }
        return RDOS_OK;
    }
    hipError_t e = launch_unpack_mesh(s->d_mesh, s->T, reinterpret_cast<int32_t *>(tables),
                                      reinterpret_cast<double *>(tables + at_w),
                                      reinterpret_cast<double *>(tables + at_g),
                                      reinterpret_cast<double *>(tables + at_nav), s->stream);
    const auto copy = [&](void *to, size_t at, size_t bytes) {
        if (to && e == hipSuccess) e = hipMemcpyAsync(to, tables + at, bytes, hipMemcpyDeviceToHost, s->stream);
    };
    copy(nbr, 0, 16 * T);
    copy(w, at_w, 32 * T);
    copy(g, at_g, 8 * T);
    copy(nav, at_nav, 8 * T);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    {
        std::lock_guard<std::mutex> g2(device_api_mutex());
        dev_free(tables, s->stream);
    }
    HIP_TRY(s, e, "download mesh tables");
    return RDOS_OK;
}

rdos_status rdos_get_info(rdos_sim *s, int32_t *n_tets, int32_t *n_species, int32_t *n_reactions,
                          int32_t *n_realizations, size_t *device_bytes)
{
    if (!s) return RDOS_EINVAL;
    if (n_tets) *n_tets = s->T;
    if (n_species) *n_species = (int32_t)s->D.size();
    if (n_reactions) *n_reactions = (int32_t)s->rx.size();
    if (n_realizations) *n_realizations = s->Rz;
    if (device_bytes) *device_bytes = state_bytes(s);
    return RDOS_OK;
}

const char *rdos_last_error(const rdos_sim *s) { return s ? s->error.c_str() : "null handle"; }

void rdos_destroy(rdos_sim *s)
{
    if (!s) return;
    free_device(s);
    delete s;
    read_buffers().simulation_gone();
}

}  // extern "C"
