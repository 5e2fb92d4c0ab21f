// gem_plan.hpp -- routes of the fused pass: where each commit's (snapshot,
// moment) chunk comes from and goes to.  Host code only, no HIP dependency
// (the host-logic tests compile it on the CPU).
#pragma once

#include <stdint.h>

namespace gemk {

// Per-commit route of a fused pass (host-planned, uniform across the grid).
// Bits 0-3: where the committing worker's (snapshot, moment) chunk comes from:
// a register slot 0..kHeldSlots-1 or the prefetch ring (memory).  Bits 4-7:
// where it goes: a register slot or memory.  Bit 8: prefetch the rows of
// commit j + depth, which reads them from memory.
constexpr int kHeldSlots = 4;
// How many commits ahead a step prefetches rows: the ring depth.  The deep
// ring is used by the default rule with per-worker moments on generated
// updates, in passes of at least kDeepMinK commits and without diagnostics;
// measured on MI355X it is 2-3% faster there, and 2-3% slower for the
// VALU-bound variants and for short passes, whose occupancy it lowers.
constexpr int kPrefetchShallow = 2;
constexpr int kPrefetchDeep = 4;
constexpr int kDeepMinK = 16;
// A pass of one commit needs no ring beyond that commit's own rows and no
// register slots: its kernel is compiled for exactly one commit (depth 1),
// which needs fewer registers, so more blocks fit a CU at once -- all of a
// 1.2M-parameter vector's blocks, instead of a full round and a tail.
constexpr int kPrefetchNone = 1;
// Blocks (of 256 threads, one wave per SIMD each) a CU holds at once in the
// deep-ring pass: measured on MI355X, its row streams run best with 3 waves
// per SIMD (4 are 1.8% slower, 2 are 7% slower).  The kernel needs few enough
// registers for 4, so an unused LDS reservation sets the cap: with L bytes of
// LDS per CU, a reservation just above L / (kDeepBlocksPerCU + 1) keeps the
// next block out, and stays far enough below L / kDeepBlocksPerCU that the
// allocation granularity does not push out one of the three.
constexpr int kDeepBlocksPerCU = 3;
inline uint32_t deep_lds_bytes(int64_t lds_per_cu)
{
    const int64_t b = (lds_per_cu / (kDeepBlocksPerCU + 1) / 1024 + 1) * 1024;
    const int64_t slack = 4096;   // per block, above any allocation granule
    return (b + slack) * kDeepBlocksPerCU <= lds_per_cu ? static_cast<uint32_t>(b) : 0u;
}

// Blocks of a recording pass over `groups` groups of 1024 elements: 8 a compute
// unit (one per group if their number, cus, is 0: unknown), but as many as
// leave no block more than kRecGroups groups, whose elements a block's 16-bit
// counts hold even when all of a commit's factors fall into one bin.
constexpr int64_t kRecGroups = 63;
inline int32_t rec_blocks(int64_t groups, int cus)
{
    const int64_t least = (groups + kRecGroups - 1) / kRecGroups;
    const int64_t most = cus > 0 ? int64_t{8} * cus : groups;
    const int64_t blocks = most > least ? most : least;
    return static_cast<int32_t>(blocks < groups ? blocks : groups);
}

constexpr uint32_t kRouteSlotMask = 0xFu;
constexpr uint32_t kRouteDstShift = 4;
constexpr uint32_t kFromRing = 0xFu;
constexpr uint32_t kToMemory = 0xFu;
constexpr uint32_t kRoutePrefetch = 1u << 8;
// Longest pass the planner handles (GEM_K_MAX in gem.h).
constexpr int kPlanMaxK = 32;

inline uint32_t make_route(uint32_t src, uint32_t dst, bool prefetch)
{
    return src | (dst << kRouteDstShift) | (prefetch ? kRoutePrefetch : 0u);
}

// Routes of one pass of k <= kPlanMaxK commits for a kernel whose ring
// prefetches depth commits ahead.  A worker's chunk is read from memory at
// its first commit in the pass and written back at its last; in between it
// waits in one of kHeldSlots register slots.  When no slot is free the chunk
// is written back and re-read, which is only valid if the re-read is at least
// depth commits later: the prefetch for commit j + depth is issued right after
// commit j's store.  A nearer repeat that finds no free slot takes the slot of
// the held chunk whose next use is furthest away (Belady's rule), if that
// chunk can go back to memory instead (its re-read at least depth commits
// after its commit).  If none can, the pass has to end after commit j: the
// function then returns j + 1 and the routes are not valid; otherwise it
// returns k.  reads and writes count the row pairs that reach memory.
inline int plan_routes(const int32_t* worker, int k, int depth, uint32_t* routes, int* reads,
                       int* writes)
{
    int next[kPlanMaxK];
    for (int j = 0; j < k; ++j) {
        next[j] = -1;
        for (int q = j + 1; q < k; ++q)
            if (worker[q] == worker[j]) { next[j] = q; break; }
    }
    int held_by[kPlanMaxK];         // slot holding commit j's chunk, or -1
    int holder[kHeldSlots];         // commit whose chunk a slot holds, or -1
    for (int q = 0; q < kHeldSlots; ++q) holder[q] = -1;
    uint32_t src[kPlanMaxK], dst[kPlanMaxK];
    *reads = *writes = 0;
    for (int j = 0; j < k; ++j) {
        held_by[j] = -1;
        int prev = -1;
        for (int q = j - 1; q >= 0 && prev < 0; --q)
            if (worker[q] == worker[j]) prev = q;
        if (prev >= 0 && held_by[prev] >= 0) {
            src[j] = static_cast<uint32_t>(held_by[prev]);
            holder[held_by[prev]] = -1;
        } else {
            src[j] = kFromRing;
            *reads += 1;
        }
        dst[j] = kToMemory;
        if (next[j] >= 0) {
            int slot = -1;
            for (int q = 0; q < kHeldSlots && slot < 0; ++q)
                if (holder[q] < 0) slot = q;
            if (slot < 0 && next[j] - j < depth) {
                // Evict: the held chunk used furthest ahead goes back to memory
                // at its own commit and is read again through the ring.
                for (int q = 0; q < kHeldSlots; ++q) {
                    const int p = holder[q];
                    if (next[p] - p >= depth && (slot < 0 || next[p] > next[holder[slot]]))
                        slot = q;
                }
                if (slot < 0) return j + 1;
                const int p = holder[slot];
                dst[p] = kToMemory;
                held_by[p] = -1;
                *writes += 1;
            }
            if (slot >= 0) {
                holder[slot] = j;
                held_by[j] = slot;
                dst[j] = static_cast<uint32_t>(slot);
            }
        }
        if (dst[j] == kToMemory) *writes += 1;
    }
    for (int j = 0; j < k; ++j) {
        const int jn = j + depth;
        const bool pf = jn < k && src[jn] == kFromRing;
        routes[j] = make_route(src[j], dst[j], pf);
    }
    return k;
}

// The longest prefix of worker[0 .. k) (k <= kPlanMaxK) that plan_routes
// can route, with its routes: a shorter pass holds fewer workers at once, so
// this settles quickly.
inline int plan_pass(const int32_t* worker, int k, int depth, uint32_t* routes, int* reads,
                     int* writes)
{
    for (int fit; (fit = plan_routes(worker, k, depth, routes, reads, writes)) < k;) k = fit;
    return k;
}

// ---- runs: many passes' commits in one launch ---------------------------------
constexpr int kRunDepth = 3;
// One schedule word a commit: bits 0-4 where the committing worker's chunk
// comes from (an LDS slot, or kRunMemory), bits 5-9 where it goes, the worker
// from bit 10 on.
constexpr uint32_t kRunSlotMask = 31u;
constexpr uint32_t kRunMemory = 31u;
constexpr int kRunDstShift = 5;
constexpr int kRunWorkerShift = 10;
constexpr int32_t kRunMaxWorkers = 1 << (32 - kRunWorkerShift);
constexpr int kRunMaxSlots = 31;
// A slot: a block's 1024 elements of a worker's snapshot and moment (of its
// snapshot, half of that, with the default rule's shared moment).
constexpr int kRunSlotBytes = 8192;
constexpr int32_t kRunMinLds = 64 << 10;   // LDS per compute unit the slots are sized for, at least
constexpr int kRunWords = 996;
constexpr int kRunCommits = kRunWords - kRunDepth;
constexpr int kRunTauAt = kRunWords / 2;   // adaptive staleness: where the tau values start

// Routes of one run of k <= kRunCommits commits with `slots` LDS slots, depth
// <= slots: which chunks wait in a slot between two commits of their worker.
// A wait is an interval of commits; at most `slots` may overlap, and the
// most waits are kept by dropping, whenever one too many overlaps, the one
// that ends last.  A wait shorter than depth must be kept (the ring's read for
// its end would be issued before its start is written); fewer than depth such
// waits overlap, so one that may be dropped is always there.  words receives
// the k schedule words and `depth` words that read no memory; last is scratch
// of one int per worker (-1 on entry and on return).  Returns the chunks read from
// memory plus the chunks written to it.
inline int plan_run(const int32_t* worker, int k, int depth, int slots, uint32_t* words, int32_t* last)
{
    int next[kRunCommits], slot[kRunCommits];
    for (int j = k - 1; j >= 0; --j) {
        next[j] = last[worker[j]];
        last[worker[j]] = j;
        slot[j] = -1;
    }
    int holder[kRunMaxSlots];
    for (int q = 0; q < slots; ++q) holder[q] = -1;
    for (int j = 0; j < k; ++j) last[worker[j]] = -1;
    for (int j = 0; j < k; ++j) {
        const int prev = last[worker[j]];
        uint32_t src = kRunMemory;
        if (prev >= 0 && slot[prev] >= 0) {
            src = static_cast<uint32_t>(slot[prev]);
            holder[slot[prev]] = -1;
        }
        last[worker[j]] = j;
        words[j] = (static_cast<uint32_t>(worker[j]) << kRunWorkerShift) | src;
        if (next[j] < 0) continue;
        int free_slot = -1, far = -1;
        for (int q = slots - 1; q >= 0; --q) {
            const int p = holder[q];
            if (p < 0) { free_slot = q; break; }
            if (next[p] - p >= depth && (far < 0 || next[p] > next[holder[far]])) far = q;
        }
        if (free_slot < 0 && far >= 0 && (next[holder[far]] > next[j] || next[j] - j < depth)) {
            slot[holder[far]] = -1;
            free_slot = far;
        }
        if (free_slot >= 0) {
            slot[j] = free_slot;
            holder[free_slot] = j;
        }
    }
    int moved = 0;
    for (int j = 0; j < k; ++j) {
        moved += ((words[j] & kRunSlotMask) == kRunMemory) + (slot[j] < 0);
        words[j] |= (slot[j] >= 0 ? static_cast<uint32_t>(slot[j]) : kRunMemory) << kRunDstShift;
        last[worker[j]] = -1;
    }
    for (int q = 0; q < depth; ++q) words[k + q] = 0u;
    return moved;
}

// ---- runs over short vectors: every worker's rows in LDS ------------------------
constexpr int64_t kShortElems = 64;    // elements of a block
constexpr int kShortPhase = 24;        // commits between two barriers
constexpr int kShortSlots = 128;       // workers of a launch, at most
// 16-bit schedule entries of k commits, with the two read ahead, in whole words.
constexpr int short_sched_pad(int k) { return (k + 3) / 2 * 2; }
// LDS of a block: the slots, two phases' noise, the schedule and the staleness values.
constexpr uint32_t short_run_lds(int slots, int k, bool adaptive)
{
    return static_cast<uint32_t>(slots * kShortElems * 8 + 2 * kShortPhase * kShortElems * 4 +
                                 short_sched_pad(k) * 2 + (adaptive ? k * 4 : 0));
}

// Schedule words of a run of k commits by at most kShortSlots workers: a 16-bit
// slot a commit, two to a word, then each slot's worker, and the number of slots
// (returned) in the last word.  slot_of is scratch of one int per worker (-1 on
// entry and on return).
inline int plan_short_run(const int32_t* worker, int k, uint32_t* words, int32_t* slot_of)
{
    uint32_t* const slot_worker = words + (k + 1) / 2;
    if (k % 2) words[k / 2] = 0;
    int slots = 0;
    for (int j = 0; j < k; ++j) {
        int32_t& slot = slot_of[worker[j]];
        if (slot < 0) {
            slot_worker[slots] = static_cast<uint32_t>(worker[j]);
            slot = slots++;
        }
        if (j % 2) words[j / 2] |= static_cast<uint32_t>(slot) << 16;
        else words[j / 2] = static_cast<uint32_t>(slot);
    }
    for (int j = 0; j < k; ++j) slot_of[worker[j]] = -1;
    words[kRunWords - 1] = static_cast<uint32_t>(slots);
    return slots;
}

// ---- how a run is launched --------------------------------------------------------
struct RunTarget {
    int64_t Pp;       // padded elements of the vector
    int cus;          // compute units (0 if unknown)
    int lds_per_cu;   // LDS of a compute unit, bytes
    int slot_bytes;   // of one of run_kernel's slots
    bool adaptive;    // the launch carries staleness values
};
struct RunLaunch {
    bool is_short;      // short_run_kernel, else run_kernel
    int slots;          // LDS slots of a block
    int64_t distinct;   // distinct workers
    int moved;          // chunks read from memory plus chunks written to it, per block
};

// The most commits of one launch: as many as the argument block takes, and at
// most 2^36 element-commits (a tenth of a second; 32 commits at least), so that a
// launch over a very large vector does not keep the GPU from other streams for long.
inline int run_commits(const RunTarget& to)
{
    const int64_t fit = to.adaptive ? kRunTauAt - kRunDepth : kRunCommits;
    const int64_t cap = (int64_t{1} << 36) / to.Pp;
    const int64_t most = cap > kPlanMaxK ? cap : kPlanMaxK;
    return static_cast<int>(fit < most ? fit : most);
}

// Whether a launch of k commits by `distinct` workers goes to the short-vector
// kernel, which holds all their rows in LDS.  It takes 0.12 us a commit for as
// many blocks as are resident, up to 8 a compute unit with 20 workers and 2 with
// 100; run_kernel takes 0.5 up to 262144 elements.  Past twice the resident blocks
// or 8 a compute unit the latter's fewer instructions per element win.  Measured
// (400 commits and the reads after them, short and run kernel, us): 20 workers,
// 65536 elements 199 and 342, 131072: 257 and 345, 262144: 341 and 351, 524288:
// 522 and 438; 100 workers, 32768: 192 and 343, 65536: 261 and 343, 131072: 386 and
// 347; kappa = 2, 131072: 255 and 421.  With the compute units' number unknown
// run_kernel takes every run.
inline bool short_run(const RunTarget& to, int64_t distinct, int k)
{
    if (distinct > kShortSlots || to.cus < 1) return false;
    const int64_t lds = short_run_lds(static_cast<int>(distinct), k, to.adaptive);
    const int64_t per_cu = (to.Pp / kShortElems + to.cus - 1) / to.cus;
    const int64_t most = 2 * (to.lds_per_cu / lds);
    return per_cu <= (most < 8 ? most : 8);
}

// Whether run_kernel's accesses are non-temporal under GEM_CACHE_AUTO, where the
// state outgrows the Infinity Cache: when few rows are found there again, that is
// beyond 250 workers (12.5M parameters, 988 commits, 300 workers: 26.5 ms, default
// policy 27.2; 200: 24.5, 23.6), or when a worker commits fewer than 1.4 times in
// the launch (25M parameters, 100 workers, 48 commits: 2.59 ms, 2.82; 96 commits:
// 4.91, 4.56).
inline bool stream_run(int64_t distinct, int k) { return distinct > 250 || 10 * k < 14 * distinct; }

// Plans a launch of k commits: the kernel, its slots, its schedule words.
// run_kernel: 160 KiB of LDS per compute unit hold 20 slots (40 with the shared
// moment's half slots), shared by the blocks resident there; measured at 12.5M
// parameters, 988 commits, unless stated:
//   - 4 blocks of 5 (10) slots when that holds every worker: nothing moves, and
//     four waves per SIMD issue best (5 workers: 13.2 ms, 13.8 ms with 3 blocks,
//     16.2 with 2);
//   - 3 blocks of 6 slots while fewer than 0.68 of the commits move their rows (10
//     workers: 15.6, 2 blocks 16.2; 11.7M, 50 workers, 400 commits, 0.61: 6.90, 7.21;
//     25M, 64 workers, 160 commits, 0.67: 6.43, 6.60);
//   - beyond, 2 blocks of 10 slots: fewer rows move, and the rows in flight have
//     larger shares of the Infinity Cache (25M, 100 workers, 160 commits, 0.72:
//     6.93, 3 blocks 7.39; 990 commits, 0.71: 40.3, 41.2; 124M, 64 workers, 160
//     commits of a Pareto schedule, 0.86: 35.0, 38.1; 150 workers: 21.7, 25.2; 300:
//     27.2, 30.0).  The shared moment moves half as much and keeps 3 blocks
//     (300 workers: 17.2, 2 blocks 18.1).  At the line itself the two are within 3%:
//     schedules whose share lies about it (25M, 100 workers: 0.67 to 0.71) may go
//     either way from launch to launch, at no greater difference than that.
// last: scratch of one int per worker (-1 on entry and on return).
inline RunLaunch plan_launch(const RunTarget& to, const int32_t* worker, int k, uint32_t* words,
                             int32_t* last)
{
    RunLaunch p{};
    for (int j = 0; j < k; ++j) {
        p.distinct += last[worker[j]] < 0;
        last[worker[j]] = 0;
    }
    for (int j = 0; j < k; ++j) last[worker[j]] = -1;
    p.is_short = short_run(to, p.distinct, k);
    if (p.is_short) {
        p.slots = plan_short_run(worker, k, words, last);
        p.moved = 2 * p.slots;
        return p;
    }
    constexpr int kLds = 160 << 10;
    const bool shared = to.slot_bytes == kRunSlotBytes / 2;
    const int all = (to.lds_per_cu < kLds ? to.lds_per_cu : kLds) / to.slot_bytes;
    auto plan = [&](int blocks) {
        p.slots = all / blocks;
        if (p.slots < kRunDepth) p.slots = kRunDepth;
        if (p.slots > kRunMaxSlots) p.slots = kRunMaxSlots;
        p.moved = plan_run(worker, k, kRunDepth, p.slots, words, last);
    };
    if (p.distinct <= all / 4) plan(4);
    else {
        plan(3);
        if (100 * p.moved >= 68 * 2 * k && !shared) plan(2);
    }
    return p;
}

}  // namespace gemk
