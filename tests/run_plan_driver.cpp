// Host-logic check of a run's schedule words (plan_run in gem_plan.hpp), on
// the CPU: replays each planned run the way the run kernel moves one thread's
// chunks -- the ring filled depth commits ahead, each step's store before its
// read for commit j + depth, the LDS slots -- with a chunk tracked as (worker,
// version).  Every commit must see its worker's latest version, memory must
// hold every worker's latest version after the run, no step may read a slot
// nobody filled, and no plan with the same slots may hold more waits (the
// greedy optimum, recomputed here by trying every wait in order of its end).
//
// Usage: run_plan_driver [seed] -- prints one summary line and "ok".
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>

#include "../paper_1805_08469_amd/csrc/gem_plan.hpp"

namespace {

int g_fail = 0;

void fail(const char* what, int j, int k, int slots)
{
    if (g_fail++ < 10) std::printf("FAIL: %s (commit %d of %d, %d slots)\n", what, j, k, slots);
}

struct Chunk {
    int worker = -1, version = -1;
};

// The most waits (first, end) that fit `slots` at once: taken by increasing
// end, each into the slot that was freed latest before its start.
int most_waits(const std::vector<int32_t>& w, int slots)
{
    std::vector<std::pair<int, int>> waits;   // (end, start)
    std::vector<int> last;
    for (int j = 0; j < static_cast<int>(w.size()); ++j) {
        if (w[j] >= static_cast<int>(last.size())) last.resize(w[j] + 1, -1);
        if (last[w[j]] >= 0) waits.push_back({j, last[w[j]]});
        last[w[j]] = j;
    }
    std::sort(waits.begin(), waits.end());
    std::vector<int> free_at(slots, -1);
    int n = 0;
    for (const auto& x : waits) {
        int best = -1;
        for (int q = 0; q < slots; ++q)
            if (free_at[q] <= x.second && (best < 0 || free_at[q] > free_at[best])) best = q;
        if (best >= 0) {
            free_at[best] = x.first;
            ++n;
        }
    }
    return n;
}

int replay(const std::vector<int32_t>& w, int n, int depth, int slots)
{
    using namespace gemk;
    const int k = static_cast<int>(w.size());
    std::vector<uint32_t> words(k + depth, 0xFFFFFFFFu);
    std::vector<int32_t> last(n, -1);
    const int planned = plan_run(w.data(), k, depth, slots, words.data(), last.data());
    for (int v : last)
        if (v != -1) fail("scratch not restored", 0, k, slots);
    std::vector<int> mem(n, 0), cur(n, 0);
    std::vector<Chunk> ring(depth), slot(slots);
    auto fetch = [&](int u, uint32_t wd) {
        ring[u] = Chunk{};
        if ((wd & kRunSlotMask) == kRunMemory) {
            const int x = static_cast<int>(wd >> kRunWorkerShift);
            ring[u] = Chunk{x, mem[x]};
        }
    };
    for (int u = 0; u < depth; ++u) fetch(u, words[u]);
    int held = 0;
    for (int j = 0; j < k; ++j) {
        const uint32_t wd = words[j], src = wd & kRunSlotMask, dst = (wd >> kRunDstShift) & kRunSlotMask;
        if (static_cast<int32_t>(wd >> kRunWorkerShift) != w[j]) fail("worker", j, k, slots);
        Chunk c = ring[j % depth];
        if (src != kRunMemory) {
            if (static_cast<int>(src) >= slots) { fail("slot number", j, k, slots); return held; }
            c = slot[src];
            slot[src] = Chunk{};
        }
        if (c.worker != w[j] || c.version != cur[w[j]]) fail("stale chunk", j, k, slots);
        c = Chunk{w[j], ++cur[w[j]]};
        if (dst != kRunMemory) {
            if (static_cast<int>(dst) >= slots) { fail("slot number", j, k, slots); return held; }
            if (slot[dst].worker >= 0) fail("slot overwritten", j, k, slots);
            slot[dst] = c;
            ++held;
        } else {
            mem[w[j]] = c.version;
        }
        fetch(j % depth, words[j + depth]);
    }
    int moved = 0;
    for (int j = 0; j < k; ++j)
        moved += ((words[j] & kRunSlotMask) == kRunMemory) +
                 (((words[j] >> kRunDstShift) & kRunSlotMask) == kRunMemory);
    if (moved != planned) fail("moved chunks", moved, k, slots);
    for (int x = 0; x < n; ++x)
        if (mem[x] != cur[x]) fail("memory behind after the run", x, k, slots);
    return held;
}

// A short vector's words: commit j's slot names commit j's worker, every worker
// has one slot, and nothing past the schedule's parts is written.
void check_short(const std::vector<int32_t>& w, int n)
{
    using namespace gemk;
    const int k = static_cast<int>(w.size());
    std::vector<uint32_t> words(kRunWords, 0xFFFFFFFFu);
    std::vector<int32_t> slot_of(n, -1);
    const int slots = plan_short_run(w.data(), k, words.data(), slot_of.data());
    for (int v : slot_of)
        if (v != -1) fail("short: scratch not restored", 0, k, slots);
    if (words[kRunWords - 1] != static_cast<uint32_t>(slots)) fail("short: slot count", 0, k, slots);
    const uint32_t* slot_worker = words.data() + (k + 1) / 2;
    std::vector<int> seen(n, 0);
    for (int q = 0; q < slots; ++q)
        if (seen[slot_worker[q]]++) fail("short: a worker with two slots", q, k, slots);
    for (int j = 0; j < k; ++j) {
        const uint32_t s = (words[j / 2] >> (16 * (j % 2))) & 0xFFFFu;
        if (static_cast<int>(s) >= slots || static_cast<int32_t>(slot_worker[s]) != w[j])
            fail("short: slot", j, k, slots);
    }
    for (int q = (k + 1) / 2 + slots; q < kRunWords - 1; ++q)
        if (words[q] != 0xFFFFFFFFu) fail("short: word past the end", q, k, slots);
}

// The rules that pick a launch's kernel and slots, on devices with and without
// known figures: the chosen kernel's LDS fits, an unknown number of compute
// units leaves run_kernel, and the words are the plan's.
void check_launch(const std::vector<int32_t>& w, int n)
{
    using namespace gemk;
    const int k = static_cast<int>(w.size());
    for (int cus : {0, 1, 256})
        for (int lds : {kRunMinLds, 160 << 10})
            for (int64_t Pp : {int64_t{64}, int64_t{64} * 8 * 256, int64_t{64} * 8 * 256 + 64, int64_t{1} << 31})
                for (int slot_bytes : {kRunSlotBytes, kRunSlotBytes / 2})
                    for (bool adaptive : {false, true}) {
                        const RunTarget to{Pp, cus, lds, slot_bytes, adaptive};
                        const int most = run_commits(to);
                        if (most < kPlanMaxK || most > kRunCommits || (adaptive && most > kRunTauAt - kRunDepth))
                            fail("commits of a launch", 0, most, lds);
                        if (k > most) continue;
                        std::vector<uint32_t> words(kRunWords, 0xFFFFFFFFu), again(words);
                        std::vector<int32_t> last(n, -1);
                        const RunLaunch p = plan_launch(to, w.data(), k, words.data(), last.data());
                        for (int v : last)
                            if (v != -1) fail("launch: scratch not restored", 0, k, p.slots);
                        if (p.distinct != static_cast<int64_t>(std::set<int32_t>(w.begin(), w.end()).size()))
                            fail("launch: distinct workers", 0, k, p.slots);
                        if (p.is_short) {
                            if (cus == 0 || Pp > int64_t{64} * 8 * cus) fail("launch: short kernel", 0, k, cus);
                            if (static_cast<int64_t>(short_run_lds(p.slots, k, adaptive)) > lds ||
                                p.slots != plan_short_run(w.data(), k, again.data(), last.data()) ||
                                p.moved != 2 * p.slots)
                                fail("launch: short plan", 0, k, p.slots);
                        } else {
                            if (p.slots < kRunDepth || p.slots > kRunMaxSlots || p.slots * slot_bytes > lds ||
                                p.moved != plan_run(w.data(), k, kRunDepth, p.slots, again.data(), last.data()))
                                fail("launch: run plan", 0, k, p.slots);
                        }
                        if (words != again) fail("launch: words", 0, k, p.slots);
                    }
}

}  // namespace

int main(int argc, char** argv)
{
    using namespace gemk;
    std::mt19937 rng(argc > 1 ? std::atoi(argv[1]) : 1);
    int runs = 0;
    for (int rep = 0; rep < 400 && !g_fail; ++rep) {
        const int n = 1 + static_cast<int>(rng() % (rep % 3 == 0 ? 4 : rep % 3 == 1 ? 40 : 300));
        const int k = rep == 0 ? kRunCommits : 1 + static_cast<int>(rng() % (rep % 5 == 0 ? kRunCommits : 120));
        const int depth = 1 + static_cast<int>(rng() % 4);
        const int slots = depth + static_cast<int>(rng() % (kRunMaxSlots - depth + 1));
        const int skew = static_cast<int>(rng() % 4);
        std::vector<int32_t> w(k);
        for (int j = 0; j < k; ++j) {
            switch (skew) {
            case 0: w[j] = static_cast<int32_t>(rng() % n); break;                        // uniform
            case 1: w[j] = static_cast<int32_t>(std::min(rng() % n, rng() % n)); break;   // skewed
            case 2: w[j] = j > 0 && rng() % 2 ? w[j - 1] : static_cast<int32_t>(rng() % n); break;  // repeats
            default: w[j] = j % n; break;                                                 // round robin
            }
        }
        std::vector<int32_t> few(w);
        for (int32_t& x : few) x %= kShortSlots;
        check_short(few, std::min(n, kShortSlots));
        if (rep % 10 == 0) check_launch(w, n);
        const int held = replay(w, n, depth, slots), most = most_waits(w, slots);
        // Waits shorter than depth are kept whatever they push out, so a plan may
        // hold fewer than the optimum only where such waits are.
        bool near = false;
        std::vector<int> at(n, -1);
        for (int j = 0; j < k; ++j) {
            near = near || (at[w[j]] >= 0 && j - at[w[j]] < depth);
            at[w[j]] = j;
        }
        if (held > most || (!near && held < most)) fail("held waits", held, k, slots);
        ++runs;
    }
    std::printf("%d runs replayed\n%s\n", runs, g_fail ? "failed" : "ok");
    return g_fail ? 1 : 0;
}
