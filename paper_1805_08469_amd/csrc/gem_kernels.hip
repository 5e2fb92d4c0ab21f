// gem_kernels.hip -- HIP kernels of the GEM commit pipeline for gfx950.
//
// The work is elementwise and streaming (Philox, Box-Muller, the GEM step): there
// is no contraction, so no MFMA is involved, and the bounds are VALU issue and the
// snapshot and moment rows between the caches and the chip.
//
// Simulated runs of more than one pass go to run_kernel, or over a short vector to
// short_run_kernel: a block takes its elements through up to 993 commits, with rows
// of workers that commit again soon in LDS.  Calls of one pass, caller updates,
// diagnostics and recordings go to pass_kernel: every thread owns four consecutive
// parameters (one 16-byte chunk of every row) and applies the pass's K commits to
// them in clock order.  theta, h and theta* are read once per pass and theta written
// once; a worker's snapshot and moment chunks are read (prefetched two or four
// commits ahead) at its first commit in the pass and written at its last, held in
// registers in between.  In both, rows are read and written as 128-bit accesses,
// consecutive lanes on consecutive chunks, so every wavefront moves 1 KiB contiguous
// per row (the short-vector kernel: 4-byte ones, once a launch).
//
// Also here: the per-segment variant of the scale factor (per commit a streaming
// step kernel and one launch that sums and forms the factors), the stand-alone update
// generator, and small gather, fill, loss and copy kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "gem_device.hpp"
#include "gem_internal.hpp"

// Device scratch of the allocation-free entry point (gem_gather_static): one
// copy per GPU, held until the process ends.  In host code this name is only a
// stand-in for the symbol; the device address of the current GPU's copy comes
// from hipGetSymbolAddress (scratch_address below), and only that address is
// ever passed to kernels or copies.
static __device__ __align__(256) unsigned char scratch[GEM_SCRATCH_BYTES];

namespace gemk {

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};
}  // namespace

hipError_t scratch_address(int device, void** out)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[device]) {
        // once per device, with that device current (the caller's)
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_dev[device] = p;
    }
    *out = g_scratch_dev[device];
    return hipSuccess;
}

namespace {

constexpr int kBlock = 256;

// Segments a block keeps block-local histograms for (per-segment mode);
// elements of further segments count straight into memory.
constexpr int kHistLdsSegs = 8;

// Recording pass (REC): the block keeps one histogram per commit of the pass
// in LDS for the whole pass, two bins per 32-bit word (16-bit counts: the grid
// gives a block at most kRecGroups groups of 1024 elements), cleared once before
// the pass and flushed once after it -- no barrier between commits.
constexpr int kRecWords = (GEM_PI_BINS + 1) / 2;

struct DiagAcc {
    double ek = 0.0, proxy = 0.0, clamped = 0.0, elems = 0.0;
    uint32_t* hist = nullptr;   // block-local histograms of the current commit (LDS)
    int32_t seg_first = 0;      // per-segment mode: the block's first segment
    int32_t lds_rows = 1;       // histograms held in LDS
};

// Histogram bin of an applied scale factor, from its binary32 bits: 0 for
// <= 0 or NaN, 1 below 2^-20, 16 bins per octave over [2^-20, 2^20), and the
// last bin from 2^20 up.
__device__ __forceinline__ int scale_bin(float x)
{
    if (!(x > 0.0f)) return 0;
    const uint32_t b = __float_as_uint(x);
    const int octave = static_cast<int>((b >> 23) & 0xFFu) - 107;
    if (octave < 0) return 1;
    if (octave >= 40) return GEM_PI_BINS - 1;
    return 2 + octave * 16 + static_cast<int>((b >> 19) & 0xFu);
}

// Has x computed here: without it the compiler moves the chain of maxima past
// the branch that follows, where it no longer folds the |.| into them (6
// instructions more).
__device__ __forceinline__ void keep(float& x) { asm volatile("" : "+v"(x)); }

// The least |num|, and the greatest |num| or den, of W quotients.  (Written as
// chains that the three-operand minimum and maximum instructions take.)
template <int W>
__device__ __forceinline__ void magnitudes(const float (&num)[W], const float (&den)[W], float& lo,
                                           float& hi)
{
    if constexpr (W == 1) {
        lo = __builtin_fabsf(num[0]);
        hi = __builtin_fmaxf(lo, den[0]);
        return;
    } else {
        hi = __builtin_fmaxf(__builtin_fabsf(num[0]), __builtin_fabsf(num[1]));
        lo = __builtin_fminf(__builtin_fabsf(num[0]), __builtin_fabsf(num[1]));
#pragma unroll
        for (int k = 2; k < W; k += 2) {
            hi = __builtin_fmaxf(__builtin_fmaxf(hi, __builtin_fabsf(num[k])), __builtin_fabsf(num[k + 1]));
            lo = __builtin_fminf(__builtin_fminf(lo, __builtin_fabsf(num[k])), __builtin_fabsf(num[k + 1]));
        }
#pragma unroll
        for (int k = 0; k < W; k += 2) hi = __builtin_fmaxf(__builtin_fmaxf(hi, den[k]), den[k + 1]);
    }
}

// The default rule's step on a thread's W elements (Fast variants, no
// diagnostics): the same arithmetic as commit_element, with one range check
// for the W quotients.  When all the operand magnitudes lie in
// [2^-60, 2^60], each quotient is div_rn_core -- what div_rn takes for each of
// them; otherwise each goes through div_rn.  A denominator |d| + eps is at
// least eps, so with eps >= 2^-60 (the default is 1e-16) only the numerators
// need the lower check.  fmaxf / fminf skip a NaN operand, which may then reach
// div_rn_core: its quotient is NaN there as in the general division, and the
// clamp makes either pi = 0.
// SMALL_EPS: eps may be below 2^-60 (else the caller has made sure it is not,
// and the step is one straight run of instructions but for the rare fallback).
template <int W, bool SMALL_EPS, typename Args>
__device__ __forceinline__ void commit_fast(const Args& a, const float (&d)[W], const float (&s)[W],
                                            float (&th)[W], float (&m)[W], float* pi_out = nullptr)
{
    float num[W], den[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        m[k] = __builtin_fmaf(a.mu, m[k], d[k]);                    // Alg. 1: m <- mu m + dtheta
        const float drift = th[k] - s[k];                           // theta_t - s_t (eq. 16)
        num[k] = __builtin_fabsf(m[k]) - __builtin_fabsf(drift);
        den[k] = __builtin_fabsf(d[k]) + a.eps;
    }
    float lo, hi;
    magnitudes(num, den, lo, hi);
    if constexpr (SMALL_EPS) {
        keep(hi);
        // (on eps's bits: a scalar comparison; eps is positive)
        if (__float_as_uint(a.eps) < __float_as_uint(0x1p-60f)) {
#pragma unroll
            for (int k = 0; k < W; ++k) lo = __builtin_fminf(lo, den[k]);
        }
    }
    // eq. 18, clamped at +0 (pi = q > 0 ? q : +0).  The median of q, 0 and inf
    // is the clamp in one instruction, a NaN's being 0 (the median instruction
    // takes the minimum of the other two).
    float pi[W];
#pragma unroll
    for (int k = 0; k < W; ++k)
        pi[k] = __builtin_amdgcn_fmed3f(div_rn_core(num[k], den[k]), 0.0f, __builtin_inff());
    if (__builtin_expect(__ballot(!(lo >= 0x1p-60f && hi <= 0x1p60f)) != 0, 0)) {
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const float q = div_rn(num[k], den[k]);
            pi[k] = (q > 0.0f) ? q : 0.0f;
        }
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
        th[k] = __builtin_fmaf(pi[k], d[k], th[k]);                 // eq. 3
        if (pi_out) pi_out[k] = pi[k];
    }
}

template <bool SMALL_EPS, typename Args>
__device__ __forceinline__ void commit4_fast(const Args& a, const float4& d, const float4& s,
                                             float4& th, float4& m, float4& snap,
                                             float* pi_out = nullptr)
{
    const float dv[4] = {d.x, d.y, d.z, d.w}, sv[4] = {s.x, s.y, s.z, s.w};
    float tv[4] = {th.x, th.y, th.z, th.w}, mv[4] = {m.x, m.y, m.z, m.w};
    commit_fast<4, SMALL_EPS>(a, dv, sv, tv, mv, pi_out);
    th = make_float4(tv[0], tv[1], tv[2], tv[3]);
    snap = th;
    m = make_float4(mv[0], mv[1], mv[2], mv[3]);
}

// One element of one commit.  th and m are the element's central value and
// the committing worker's moment (in/out); s is its snapshot; d the update.
// snap receives the value the worker's snapshot takes after this commit.
// FAST: the default rule (GEM, CLAMP0, kappa_eff = 1, post-commit pull) with
// no runtime mode tests; otherwise every mode is read from a.mode.
// hist_row: the histogram row this element's factor counts in, or null.
template <bool FAST, bool DIAG>
__device__ __forceinline__ void commit_element(const PassArgs& a, int tau, float d, float s,
                                               float& th, float& m, float& snap, bool live,
                                               DiagAcc& acc, uint32_t* hist_row)
{
    const float mn = __builtin_fmaf(a.mu, m, d);        // Alg. 1: m <- mu m + dtheta
    const float drift = th - s;                         // theta_t - s_t (eq. 16)
    float th_new;
    float pi_raw = 0.0f;
    float scale;                                        // factor applied to dtheta
    bool gem_rule = true;
    if (FAST) {
        const float num = __builtin_fabsf(mn) - __builtin_fabsf(drift);
        const float den = __builtin_fabsf(d) + a.eps;
        pi_raw = div_rn(num, den);                      // eq. 18 / Alg. 1
        const float pi = (pi_raw > 0.0f) ? pi_raw : 0.0f;
        th_new = __builtin_fmaf(pi, d, th);             // eq. 3
        snap = th_new;
        scale = pi;
    } else {
        if (a.mode & kModeDownpour) {
            gem_rule = false;
            th_new = th + d;                            // eq. 1
            scale = 1.0f;
        } else if (a.mode & kModeAdaptive) {
            gem_rule = false;
            th_new = th + d / static_cast<float>(tau + 1);
            scale = 1.0f / static_cast<float>(tau + 1);
        } else {
            const float km = (a.mode & kModeKappaMul) ? a.k_eff * __builtin_fabsf(mn)
                                                      : __builtin_fabsf(mn);
            const float num = km - __builtin_fabsf(drift);
            const float den = __builtin_fabsf(d) + a.eps;
            pi_raw = div_rn(num, den);
            const float pi = (a.mode & kModeLiteralPi) ? pi_raw
                                                       : ((pi_raw > 0.0f) ? pi_raw : 0.0f);
            th_new = __builtin_fmaf(pi, d, th);
            scale = pi;
        }
        snap = (a.mode & kModePrePull) ? th : th_new;
    }
    if (DIAG && live && hist_row) atomicAdd(&hist_row[scale_bin(scale)], 1u);
    if (DIAG && live) {
        const double e = static_cast<double>(th_new) - static_cast<double>(s);
        const double kmd = static_cast<double>(FAST ? 1.0f : a.k_eff) * static_cast<double>(mn);
        acc.ek += 0.5 * e * e;
        acc.proxy += 0.5 * kmd * kmd;
        if (gem_rule && !(pi_raw >= 0.0f)) acc.clamped += 1.0;
        acc.elems += 1.0;
    }
    th = th_new;
    m = mn;
}

// The simulated worker's updates at W snapshot elements (notation table:
// -eta grad L(s)).
template <int W, bool BF16>
__device__ __forceinline__ void stale_updates(float neg_lr, float sigma, const float* s,
                                              const float* h, const float* ts, const float* z,
                                              float* d)
{
    static_assert(W % 2 == 0, "pairs are rounded together");
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const float nz = sigma * z[k];
        const float g = __builtin_fmaf(h[k], s[k] - ts[k], nz);
        d[k] = neg_lr * g;
    }
    if constexpr (BF16) {
#pragma unroll
        for (int k = 0; k < W; k += 2) round_pair_to_bf16(d[k], d[k + 1]);
    }
}

template <bool BF16>
__device__ __forceinline__ float4 stale_update4(float neg_lr, float sigma, const float4& s,
                                                const float4& h, const float4& ts, const float4& z)
{
    const float sv[4] = {s.x, s.y, s.z, s.w}, hv[4] = {h.x, h.y, h.z, h.w};
    const float tv[4] = {ts.x, ts.y, ts.z, ts.w}, zv[4] = {z.x, z.y, z.z, z.w};
    float d[4];
    stale_updates<4, BF16>(neg_lr, sigma, sv, hv, tv, zv, d);
    return make_float4(d[0], d[1], d[2], d[3]);
}

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b16) { return __uint_as_float(b16 << 16); }

// A caller update for chunk c: four elements, masked past the true length.
template <Source SRC>
__device__ __forceinline__ float4 load_given(const void* base, int64_t c, int64_t P)
{
    const int64_t i0 = c * 4;
    if (SRC == Source::GivenF32) {
        const float* p = static_cast<const float*>(base);
        if (i0 + 4 <= P) return *reinterpret_cast<const float4*>(p + i0);
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i0 + 0 < P) v.x = p[i0 + 0];
        if (i0 + 1 < P) v.y = p[i0 + 1];
        if (i0 + 2 < P) v.z = p[i0 + 2];
        if (i0 + 3 < P) v.w = p[i0 + 3];
        return v;
    } else {
        const uint16_t* p = static_cast<const uint16_t*>(base);
        if (i0 + 4 <= P) {
            const uint2 u = *reinterpret_cast<const uint2*>(p + i0);
            return make_float4(bf16_bits_to_float(u.x & 0xFFFFu), bf16_bits_to_float(u.x >> 16),
                               bf16_bits_to_float(u.y & 0xFFFFu), bf16_bits_to_float(u.y >> 16));
        }
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i0 + 0 < P) v.x = bf16_bits_to_float(p[i0 + 0]);
        if (i0 + 1 < P) v.y = bf16_bits_to_float(p[i0 + 1]);
        if (i0 + 2 < P) v.z = bf16_bits_to_float(p[i0 + 2]);
        if (i0 + 3 < P) v.w = bf16_bits_to_float(p[i0 + 3]);
        return v;
    }
}

struct Rows {
    float4 s, m;
};

// 16-byte loads and stores of the fused pass.  NT marks them non-temporal
// (streaming): each row chunk a pass touches is read once and written once,
// and over a state far larger than the caches the hint lets HBM streams
// bypass the cache residency a reused line would get (measured 7-12% faster
// passes); a state that fits the 256 MiB Infinity Cache keeps the default
// policy, which serves it from there.
typedef float v4f __attribute__((ext_vector_type(4)));

template <bool NT>
__device__ __forceinline__ float4 load4(const float* p)
{
    if constexpr (NT) {
        const v4f v = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
        return make_float4(v.x, v.y, v.z, v.w);
    } else {
        return *reinterpret_cast<const float4*>(p);
    }
}

template <bool NT>
__device__ __forceinline__ void store4(float* p, float4 v)
{
    if constexpr (NT) {
        __builtin_nontemporal_store(v4f{v.x, v.y, v.z, v.w}, reinterpret_cast<v4f*>(p));
    } else {
        *reinterpret_cast<float4*>(p) = v;
    }
}

// The same at a (uniform) base plus a 32-bit byte offset, which the scalar
// base + vector offset addressing takes as is.  FRESH gives each use its own
// copy of the offset (an empty asm), so that the offset's widening to 64 bits
// is not hoisted out of the pass loop: a widened offset no longer fits that
// addressing.
__device__ __forceinline__ uint32_t fresh(uint32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}

template <bool NT, bool FRESH = false>
__device__ __forceinline__ float4 load4_at(const float* base, uint32_t byte_off)
{
    if constexpr (FRESH) byte_off = fresh(byte_off);
    return load4<NT>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + byte_off));
}

template <bool NT, bool FRESH = false>
__device__ __forceinline__ void store4_at(float* base, uint32_t byte_off, float4 v)
{
    if constexpr (FRESH) byte_off = fresh(byte_off);
    store4<NT>(reinterpret_cast<float*>(reinterpret_cast<char*>(base) + byte_off), v);
}


// Per-thread context of a fused pass: the chunk, its central values and the
// problem coefficients, kept in registers for the whole pass.
struct Chunk {
    int64_t c;       // chunk index (= Philox counter q of its four elements)
    int64_t off;     // element offset 4c
    // Addresses as a block-uniform part and a 32-bit lane part: worker w's
    // snapshot chunk is at S + tile + w * 2 * kTileElems plus io bytes (io =
    // 4 * tin + t16), its moment chunk at M + the same; its sink entries at
    // sink_S / sink_M plus so bytes (so = 4 * sink0 + t16); theta, h and
    // theta* at blk0 plus t16 bytes.
    int64_t tile;    // table index of worker 0's snapshot piece of the block's tile
    int64_t tin;     // the block's first element offset inside its tile
    int64_t blk0;    // first element of the block
    int64_t sink0;   // first element of the block's sink entries
    uint32_t io;     // byte offset of the chunk inside its tile's piece
    uint32_t so;     // byte offset of the chunk's entries in the sink buffers
    uint32_t t16;    // 16 * threadIdx.x
    uint32_t q_lo, q_hi;   // words of the chunk index c (the Philox counter)
    bool active;
    bool l0, l1, l2, l3;   // elements below the true length (diagnostics)
    int32_t sg[4];         // per-segment histograms: each element's segment
    float4 th, hh, tt;
    float4 mg;       // the shared moment (global proxy mode)
};

// Register slots holding the (snapshot, moment) chunks of workers that commit
// again later in the same pass.
struct Held {
    Rows h0, h1, h2, h3;
};

__device__ __forceinline__ Rows held_get(const Held& h, uint32_t slot)
{
    switch (slot) {
    case 0: return h.h0;
    case 1: return h.h1;
    case 2: return h.h2;
    default: return h.h3;
    }
}

__device__ __forceinline__ Held held_put(Held h, uint32_t slot, const Rows& r)
{
    switch (slot) {
    case 0: h.h0 = r; break;
    case 1: h.h1 = r; break;
    case 2: h.h2 = r; break;
    default: h.h3 = r; break;
    }
    return h;
}

// One step's row access: worker w's piece of `table` if mem, else the sink.
// The shared-moment variant (VALU-bound) keeps the base block-uniform and
// adds the lane's 16 * threadIdx.x bytes, which saves vector instructions and
// registers (3-4% faster); the per-worker variants (HBM-bound) select a
// per-lane element offset, measured 0.3-4% faster for them.
template <bool UNIFORM, bool NT>
__device__ __forceinline__ float4 row_load(const float* table, const float* sink, bool mem,
                                           int32_t w, const Chunk& ch)
{
    const int64_t wrow = ch.tile + (static_cast<int64_t>(w) << (kTileShift + 1));
    if constexpr (UNIFORM)
        return load4_at<NT, true>(mem ? table + wrow + ch.tin : sink + ch.sink0, ch.t16);
    else
        return load4_at<NT>(mem ? table + wrow : sink, mem ? ch.io : ch.so);
}

template <bool UNIFORM, bool NT>
__device__ __forceinline__ void row_store(float* table, float* sink, bool mem, int32_t w,
                                          const Chunk& ch, float4 v)
{
    const int64_t wrow = ch.tile + (static_cast<int64_t>(w) << (kTileShift + 1));
    if constexpr (UNIFORM)
        store4_at<NT, true>(mem ? table + wrow + ch.tin : sink + ch.sink0, ch.t16, v);
    else
        store4_at<NT>(mem ? table + wrow : sink, mem ? ch.io : ch.so, v);
}

struct StepOut {
    Rows out;    // the worker's (snapshot, moment) chunk after commit j
    Rows next;   // ring entry for commit j + DEPTH
    Held held;
};


// Commit j of a pass.  The committing worker's (snapshot, moment) chunk comes
// from the prefetch ring (loaded DEPTH commits earlier: a first commit in the
// pass, or a worker whose earlier commit in the pass, at least DEPTH commits
// back, wrote its rows back) or from a register slot.  After the commit the
// chunk is written back (the worker's last commit in the pass, or no slot was
// free) or held in a slot; then the rows of commit j + DEPTH are prefetched
// into the ring entry just consumed, if that
// commit reads them from memory.  Every step issues one row-pair store and one
// row-pair load unconditionally -- those a step does not need go to the small
// sink buffer, which stays in cache -- so the wait for a step's rows never
// covers the loads issued after them.
template <Source SRC, Variant V, bool BF16, bool DIAG, int DEPTH, bool NT, bool REC>
__device__ __forceinline__ StepOut pass_step(const PassArgs& a, int j, Chunk& ch, Rows ring,
                                             Held held, DiagAcc& acc, uint32_t* rec_lds)
{
    const uint32_t route = a.routes[j];
    const uint32_t src = route & kRouteSlotMask;
    const uint32_t dst = (route >> kRouteDstShift) & kRouteSlotMask;
    const int w = a.worker[j];
    // (a single-commit pass reads its one commit's rows through the ring)
    Rows rows = (DEPTH == 1 || src == kFromRing) ? ring : held_get(held, src);
    constexpr bool FAST = V != Variant::General;
    const bool global_m = V == Variant::FastGlobal ||
                          (V == Variant::General && (a.mode & kModeGlobalProxy));
    if (global_m) rows.m = ch.mg;   // the shared moment, carried like theta

    float4 d;
    if (SRC == Source::Generated) {
        // The chunk index's high word is the block's (uniform): blocks start at
        // multiples of kBlock chunks, so adding the lane never carries into it.
        const uint64_t q = (static_cast<uint64_t>(ch.q_hi) << 32) | ch.q_lo;
        const float4 z = normals4(q, a.t0 + static_cast<uint32_t>(j),
                                  a.key0, a.key1);
        d = stale_update4<BF16>(a.neg_lr, a.sigma, rows.s, ch.hh, ch.tt, z);
    } else {
        d = ch.active ? load_given<SRC>(a.upd[j], ch.c, a.P) : make_float4(0.f, 0.f, 0.f, 0.f);
    }

    const int tau = a.tau[j];
    // Diagnostic histogram of this commit's scale factors: every thread of
    // the block is at commit j here (the loop is uniform), so the block-local
    // histogram is cleared, filled and flushed between barriers.
    const bool record = DIAG && acc.hist != nullptr && a.hist_first + j < a.hist_cap;
    const int lds_bins = acc.lds_rows * GEM_PI_BINS;
    if (DIAG && acc.hist != nullptr) {
        for (int b = threadIdx.x; b < lds_bins; b += kBlock) acc.hist[b] = 0u;
        __syncthreads();
    }
    // Each element's histogram row: the block-local one of its segment, or
    // (a segment beyond the block's LDS rows) its row of this commit in memory.
    uint32_t* hrow[4] = {nullptr, nullptr, nullptr, nullptr};
    if (DIAG && record) {
        uint32_t* commit_rows = a.pi_hist + (a.hist_first + j) * a.hist_rows * GEM_PI_BINS;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int ls = ch.sg[k] - acc.seg_first;
            hrow[k] = ls < acc.lds_rows ? acc.hist + ls * GEM_PI_BINS
                                        : commit_rows + static_cast<int64_t>(ch.sg[k]) * GEM_PI_BINS;
        }
    }
    StepOut r;
    r.out.m = rows.m;
    if constexpr (FAST && !DIAG) {
        float pis[4];
        commit4_fast<true>(a, d, rows.s, ch.th, r.out.m, r.out.s, REC ? pis : nullptr);
        if constexpr (REC) {
            // this commit's factors into the block's LDS histogram (uniform
            // test: recording stops at the capacity)
            if (ch.active && a.hist_first + j < a.hist_cap) {
                uint32_t* row = rec_lds + j * kRecWords;
                uint32_t* spare = rec_lds + a.K * kRecWords + threadIdx.x;   // this lane's own word
                const bool live[4] = {ch.l0, ch.l1, ch.l2, ch.l3};
                // Clamped factors (+0, bin 0) are often most of a commit's:
                // the wave counts them with ballots and adds them once, while
                // their lanes (and padding elements) add to a word of their
                // own, so no add waits behind one address and no lane
                // branches.  A positive factor's bin is scale_bin's, in
                // integer steps: (bits >> 19) - 1710 clamped to [1, 642].
                uint32_t clamped = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t bits = __float_as_uint(pis[k]);   // +0 or positive
                    const bool counted = live[k] && bits != 0u;
                    clamped += static_cast<uint32_t>(__popcll(__ballot(live[k] && bits == 0u)));
                    const int bin = min(max(static_cast<int>(bits >> 19) - 1710, 1), GEM_PI_BINS - 1);
                    uint32_t* word = counted ? row + (bin >> 1) : spare;
                    atomicAdd(word, 1u << ((bin & 1) << 4));
                }
                const uint64_t lanes = __ballot(1);
                if (clamped != 0u && (threadIdx.x & 63u) == static_cast<uint32_t>(__builtin_ctzll(lanes)))
                    atomicAdd(&row[0], clamped);   // bin 0: the low half of word 0
            }
        }
    } else {
        commit_element<FAST, DIAG>(a, tau, d.x, rows.s.x, ch.th.x, r.out.m.x, r.out.s.x, ch.active && ch.l0, acc, hrow[0]);
        commit_element<FAST, DIAG>(a, tau, d.y, rows.s.y, ch.th.y, r.out.m.y, r.out.s.y, ch.active && ch.l1, acc, hrow[1]);
        commit_element<FAST, DIAG>(a, tau, d.z, rows.s.z, ch.th.z, r.out.m.z, r.out.s.z, ch.active && ch.l2, acc, hrow[2]);
        commit_element<FAST, DIAG>(a, tau, d.w, rows.s.w, ch.th.w, r.out.m.w, r.out.s.w, ch.active && ch.l3, acc, hrow[3]);
    }

    if (DIAG && acc.hist != nullptr) {
        __syncthreads();
        if (record) {
            uint32_t* dst = a.pi_hist +
                            ((a.hist_first + j) * a.hist_rows + acc.seg_first) * GEM_PI_BINS;
            for (int b = threadIdx.x; b < lds_bins; b += kBlock)
                if (acc.hist[b]) atomicAdd(&dst[b], acc.hist[b]);
        }
        __syncthreads();
    }
    if (global_m) ch.mg = r.out.m;
    if (DEPTH > 1 && dst != kToMemory) {
        // The shared-moment variant carries the moment in ch.mg: a held
        // slot keeps only the snapshot (no registers for a moment copy).
        Rows keep = r.out;
        if (V == Variant::FastGlobal) keep.m = make_float4(0.f, 0.f, 0.f, 0.f);
        held = held_put(held, dst, keep);
    }
    r.held = held;
    r.next = ring;
    if (ch.active) {
        // With the shared moment, only snapshot rows move; moment traffic goes
        // to the sink.
        constexpr bool U = V == Variant::FastGlobal;
        const bool st = DEPTH == 1 || dst == kToMemory;
        const bool st_m = st && !global_m;
        row_store<U, NT>(a.S, a.sink_S, st, w, ch, r.out.s);
        row_store<U, NT>(a.M, a.sink_M, st_m, w, ch, r.out.m);
        if constexpr (DEPTH > 1) {
            const bool pf = (route & kRoutePrefetch) != 0;
            const int jn = j + DEPTH < a.K ? j + DEPTH : j;
            const bool pf_m = pf && !global_m;
            r.next.s = row_load<U, NT>(a.S, a.sink_S, pf, a.worker[jn], ch);
            r.next.m = row_load<U, NT>(a.M, a.sink_M, pf_m, a.worker[jn], ch);
        }
    }
    return r;
}

// One pass over the 1024 elements of group grp (the block's 256 chunks).
template <Source SRC, Variant V, bool BF16, bool DIAG, int DEPTH, bool NT, bool REC>
__device__ __forceinline__ void pass_group(const PassArgs& a, int64_t grp, uint32_t* rec_lds)
{
    static_assert(!(REC && DIAG), "recording passes take the fast commit");
    const int64_t nchunk = a.Pp >> 2;
    const int64_t c = grp * kBlock + threadIdx.x;
    Chunk ch;
    ch.active = c < nchunk;
    if (!DIAG && !ch.active) return;   // (the diagnostic variant's barriers need every thread)
    ch.c = ch.active ? c : 0;   // inactive lanes (diagnostic variant) do no memory work
    ch.off = ch.c * 4;
    static_assert((kBlock & (kBlock - 1)) == 0, "block size a power of two");
    ch.q_hi = static_cast<uint32_t>((grp * kBlock) >> 32);
    ch.q_lo = static_cast<uint32_t>(ch.c);
    ch.l0 = ch.off + 0 < a.P;
    ch.l1 = ch.off + 1 < a.P;
    ch.l2 = ch.off + 2 < a.P;
    ch.l3 = ch.off + 3 < a.P;
    ch.th = make_float4(0.f, 0.f, 0.f, 0.f);
    ch.hh = ch.th;
    ch.tt = ch.th;
    ch.mg = ch.th;
    const bool global_m = V == Variant::FastGlobal ||
                          (V == Variant::General && (a.mode & kModeGlobalProxy));
    static_assert(kTileElems % (kBlock * 4) == 0, "a block's chunks lie in one tile");
    static_assert(kSinkChunks % kBlock == 0, "a block's sink entries are contiguous");
    ch.blk0 = grp * (kBlock * 4);
    ch.t16 = threadIdx.x * 16u;
    ch.tile = tile_index(a.nw, 0, ch.blk0 & ~(kTileElems - 1));
    ch.tin = ch.blk0 & (kTileElems - 1);
    ch.sink0 = ((ch.blk0 >> 2) & a.sink_mask) * 4;
    ch.io = static_cast<uint32_t>(ch.tin) * 4u + ch.t16;
    ch.so = static_cast<uint32_t>(ch.c & a.sink_mask) * 16u;   // = 4 * sink0 + t16
    // The shared moment is worker 0's.
    if (global_m && ch.active) ch.mg = load4_at<NT>(a.M + ch.tile, ch.io);
    // A depth-1 kernel runs single-commit passes only (the launch checks it).
    const int K = DEPTH == 1 ? 1 : a.K;
    // Ring of prefetched rows, unrolled DEPTH ways so that every entry
    // is a fixed set of registers: commit j reads ring[j mod depth] and refills
    // it for commit j + depth -- no register copy of an in-flight load.
    Rows ring[DEPTH];
    Held held{};
    if (ch.active) {
        ch.th = a.keep_theta ? load4_at<false>(a.theta + ch.blk0, ch.t16)
                             : load4_at<NT>(a.theta + ch.blk0, ch.t16);
        if (SRC == Source::Generated) {
            if (a.keep_problem) {
                ch.hh = load4_at<false>(a.h + ch.blk0, ch.t16);
                ch.tt = load4_at<false>(a.ts + ch.blk0, ch.t16);
            } else {
                ch.hh = load4_at<NT>(a.h + ch.blk0, ch.t16);
                ch.tt = load4_at<NT>(a.ts + ch.blk0, ch.t16);
            }
        }
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            // Commit u reads memory iff it is the first commit of its worker
            // (u < depth); the others prefetch from the sink.
            // With the shared moment only the snapshot row is read.
            const bool mem = u < K && (a.routes[u] & kRouteSlotMask) == kFromRing;
            const bool mem_m = mem && !global_m;
            constexpr bool U = V == Variant::FastGlobal;
            ring[u].s = row_load<U, NT>(a.S, a.sink_S, mem, a.worker[u], ch);
            ring[u].m = row_load<U, NT>(a.M, a.sink_M, mem_m, a.worker[u], ch);
        }
    } else {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) ring[u] = Rows{};
    }

    DiagAcc acc;
    ch.sg[0] = ch.sg[1] = ch.sg[2] = ch.sg[3] = 0;
    if constexpr (DIAG) {
        __shared__ uint32_t hist_lds[kHistLdsSegs * GEM_PI_BINS];
        if (a.pi_hist) {
            acc.hist = hist_lds;
            if (a.hist_rows > 1) {
                // The block's segments (uniform) and each element's segment.
                const int64_t g_lo = grp * kBlock * 4;
                const int64_t g_last = (g_lo + kBlock * 4 < a.P ? g_lo + kBlock * 4 : a.P) - 1;
                acc.seg_first = a.hseg_grp[grp];
                int32_t seg_last = acc.seg_first;
                while (a.hseg_off[seg_last + 1] <= g_last) ++seg_last;
                const int32_t rows = seg_last - acc.seg_first + 1;
                acc.lds_rows = rows < kHistLdsSegs ? rows : kHistLdsSegs;
                int32_t sg = acc.seg_first;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t i = ch.off + k;
                    if (ch.active && i < a.P)
                        while (a.hseg_off[sg + 1] <= i) ++sg;
                    ch.sg[k] = sg;
                }
            }
        }
    }
    int j = 0;
    for (; j + DEPTH <= K; j += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const StepOut so = pass_step<SRC, V, BF16, DIAG, DEPTH, NT, REC>(a, j + u, ch, ring[u], held,
                                                                            acc, rec_lds);
            ring[u] = so.next;
            held = so.held;
        }
    }
    // At most DEPTH - 1 commits remain.
#pragma unroll
    for (int u = 0; u + 1 < DEPTH; ++u) {
        if (j + u < K) {
            const StepOut so = pass_step<SRC, V, BF16, DIAG, DEPTH, NT, REC>(a, j + u, ch, ring[u], held,
                                                                            acc, rec_lds);
            ring[u] = so.next;
            held = so.held;
        }
    }
    if (ch.active) {
        if (a.keep_theta) store4_at<false>(a.theta + ch.blk0, ch.t16, ch.th);
        else store4_at<NT>(a.theta + ch.blk0, ch.t16, ch.th);
    }
    if (global_m && ch.active) store4_at<NT>(a.M + ch.tile, ch.io, ch.mg);

    if (DIAG && a.diag) {
        __shared__ double red[4][kBlock];
        red[0][threadIdx.x] = acc.ek;
        red[1][threadIdx.x] = acc.proxy;
        red[2][threadIdx.x] = acc.clamped;
        red[3][threadIdx.x] = acc.elems;
        __syncthreads();
        for (int step = kBlock / 2; step > 0; step >>= 1) {
            if (static_cast<int>(threadIdx.x) < step) {
#pragma unroll
                for (int q = 0; q < 4; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + step];
            }
            __syncthreads();
        }
        if (threadIdx.x < 4) atomicAdd(&a.diag[threadIdx.x], red[threadIdx.x][0]);
    }
}

// The fused pass: one group per block; the recording variant (REC) loops its
// blocks over the groups (a grid of a.rec_grid blocks)
// so that each block's per-pass LDS histograms gather many groups before
// their single flush -- one global atomic per nonzero bin and block.
template <Source SRC, Variant V, bool BF16, bool DIAG, int DEPTH, bool NT, bool REC>
__global__ __launch_bounds__(kBlock) void pass_kernel(const PassArgs a)
{
    extern __shared__ uint32_t dyn_lds[];   // REC: K rows of kRecWords, then a word per thread
    if constexpr (REC) {
        for (int w = threadIdx.x; w < a.K * kRecWords; w += kBlock) dyn_lds[w] = 0u;
        __syncthreads();
        const int64_t ngroups = ((a.Pp >> 2) + kBlock - 1) / kBlock;
        for (int64_t grp = blockIdx.x; grp < ngroups; grp += gridDim.x)
            pass_group<SRC, V, BF16, DIAG, DEPTH, NT, REC>(a, grp, dyn_lds);
        // the histograms into the recording, one atomic per nonzero bin
        __syncthreads();
        for (int w = threadIdx.x; w < a.K * kRecWords; w += kBlock) {
            const uint32_t v = dyn_lds[w];
            const int j = w / kRecWords;
            if (v == 0u || a.hist_first + j >= a.hist_cap) continue;
            uint32_t* row = a.pi_hist + (a.hist_first + j) * GEM_PI_BINS;
            const int b = 2 * (w - j * kRecWords);
            if (v & 0xFFFFu) atomicAdd(&row[b], v & 0xFFFFu);
            if (v >> 16) atomicAdd(&row[b + 1], v >> 16);
        }
    } else {
        pass_group<SRC, V, BF16, DIAG, DEPTH, NT, REC>(a, blockIdx.x, dyn_lds);
    }
}

// Mode bits of the General variant's kernels of a run: those of the launch
// (kAnyMode), or one rule's known when compiled (then eps >= 2^-60).  With the
// modes as uniform runtime flags the step is cut by their branches and the noise
// no longer fills its latencies: kappa = 2, 3141593 elements, 30 workers, 500
// commits 2.65 ms, with a kernel of its own 2.47; 65536 elements, 400 commits 236
// and 203 us.
constexpr uint32_t kAnyMode = ~0u;

// The general rule's step on a thread's W elements (run kernels, General
// variant): commit_element's arithmetic, with one range check for the W
// quotients as in commit_fast.
template <int W, uint32_t MODE>
__device__ __forceinline__ void commit_general(const RunArgs& a, int tau, const float (&d)[W],
                                               const float (&s)[W], float (&th)[W], float (&m)[W],
                                               float (&snap)[W])
{
    const uint32_t mode = MODE == kAnyMode ? a.mode : MODE;
    float next[W];
#pragma unroll
    for (int k = 0; k < W; ++k) m[k] = __builtin_fmaf(a.mu, m[k], d[k]);
    if (mode & kModeDownpour) {
#pragma unroll
        for (int k = 0; k < W; ++k) next[k] = th[k] + d[k];         // eq. 1
    } else {
        // num / den: the scale factor (eq. 18), or the damped update itself
        const bool adaptive = (mode & kModeAdaptive) != 0;
        const float k_eff = (mode & kModeKappaMul) ? a.k_eff : 1.0f;
        const float stale = static_cast<float>(tau + 1);
        float num[W], den[W], q[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const float drift = th[k] - s[k];
            num[k] = adaptive ? d[k] : k_eff * __builtin_fabsf(m[k]) - __builtin_fabsf(drift);
            den[k] = adaptive ? stale : __builtin_fabsf(d[k]) + a.eps;
        }
        float lo, hi;
        magnitudes(num, den, lo, hi);
        if constexpr (MODE == kAnyMode) {
            keep(hi);
            if (__float_as_uint(a.eps) < __float_as_uint(0x1p-60f)) {
#pragma unroll
                for (int k = 0; k < W; ++k) lo = __builtin_fminf(lo, den[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < W; ++k) q[k] = div_rn_core(num[k], den[k]);
        if (__builtin_expect(__ballot(!(lo >= 0x1p-60f && hi <= 0x1p60f)) != 0, 0)) {
#pragma unroll
            for (int k = 0; k < W; ++k) q[k] = div_rn(num[k], den[k]);
        }
        if (adaptive) {
#pragma unroll
            for (int k = 0; k < W; ++k) next[k] = th[k] + q[k];
        } else {
            const bool literal = (mode & kModeLiteralPi) != 0;
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const float pi = literal ? q[k] : __builtin_amdgcn_fmed3f(q[k], 0.0f,
                                                                          __builtin_inff());
                next[k] = __builtin_fmaf(pi, d[k], th[k]);          // eq. 3
            }
        }
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
        snap[k] = (mode & kModePrePull) ? th[k] : next[k];
        th[k] = next[k];
    }
}

template <uint32_t MODE>
__device__ __forceinline__ void commit4_general(const RunArgs& a, int tau, const float4& d,
                                                const float4& s, float4& th, float4& m,
                                                float4& snap)
{
    const float dv[4] = {d.x, d.y, d.z, d.w}, sv[4] = {s.x, s.y, s.z, s.w};
    float tv[4] = {th.x, th.y, th.z, th.w}, mv[4] = {m.x, m.y, m.z, m.w}, nv[4];
    commit_general<4, MODE>(a, tau, dv, sv, tv, mv, nv);
    th = make_float4(tv[0], tv[1], tv[2], tv[3]);
    snap = make_float4(nv[0], nv[1], nv[2], nv[3]);
    m = make_float4(mv[0], mv[1], mv[2], mv[3]);
}

// Row accesses of the run kernel: buffer instructions on a descriptor of the
// block's 4 KiB of the row, or of no bytes when the step does not need the
// access: then every lane is out of range, a load gives zeros and a store is
// dropped, without a memory request.  The number of memory instructions a
// step issues is therefore fixed (the compiler's waits count them).
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
constexpr int kBufferFlags = 0x00027000;   // raw 32-bit words, range-checked by bytes

template <bool NT>
__device__ __forceinline__ float4 row_at(float* base, bool mem, uint32_t byte_off)
{
    const __amdgpu_buffer_rsrc_t d =
        __builtin_amdgcn_make_buffer_rsrc(base, 0, mem ? kBlock * 16 : 0, kBufferFlags);
    const v4u v = __builtin_amdgcn_raw_buffer_load_b128(d, byte_off, 0, NT ? 2 : 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                       __uint_as_float(v.w));
}

template <bool NT>
__device__ __forceinline__ void put_row_at(float* base, bool mem, uint32_t byte_off, float4 v)
{
    const __amdgpu_buffer_rsrc_t d =
        __builtin_amdgcn_make_buffer_rsrc(base, 0, mem ? kBlock * 16 : 0, kBufferFlags);
    __builtin_amdgcn_raw_buffer_store_b128(v4u{__float_as_uint(v.x), __float_as_uint(v.y),
                                               __float_as_uint(v.z), __float_as_uint(v.w)},
                                           d, byte_off, 0, NT ? 2 : 0);
}

// A run of up to kRunCommits commits in one launch (generated updates, no
// diagnostics): a block takes its 1024 elements through all of them before the
// next block takes its place.  A pass of 32 commits per launch read and wrote
// each committing worker's rows once a pass, 13.7 bytes per element-commit at
// 100 workers, and waited on that traffic; here
//   - rows of workers that commit again soon wait in LDS slots (plan_run), so
//     a commit moves its worker's rows in 0.7 of the cases with 6 slots and 100
//     workers, 0.63 with 50 (0.84 and 0.78 in passes of 32 with 4 slots);
//   - theta, h and theta* are read once per run instead of once per pass;
//   - the rows a block moves again lie in the Infinity Cache's share of the
//     few hundred blocks in flight, if the workers are not too many.
// What is left is 201 VALU instructions per wave and commit by the counters (209
// with bf16 updates), and the rows' traffic between L2 and the fabric, 10.0 bytes an
// element-commit at 25M parameters and 100 workers, at 6.2-6.4 TB/s, the rate a copy
// reaches.  The step's 192 instructions take 580 cycles of a SIMD: 110 issue every
// two cycles, 74 every four (64-bit multiply-adds, conversions, comparisons, minima
// and maxima, and any that reads a scalar register), 8 every eight.  The counters
// show up to 1.21 of them per SIMD in four cycles.
// Measured at 25M parameters and 100 workers, 1000 commits: 56.4 ms in passes of
// 32, 40.8 ms here; with the shared moment 40.7 and 31.5 (bound by VALU issue).
//
// Two elements a thread, a lane pair sharing a Philox block, would give each
// element twice the slots: 221 instructions, and within 2% at every size.
//
// Rows come DEPTH commits ahead into a register ring; 3 measured best (2 and 4
// are 2% and 1% slower, 6 and 8 more).  Noise is drawn one commit ahead, in
// the same straight run of instructions as the commit's step, so that the two
// chains fill each other's latencies (the kernel runs 3 waves per SIMD: 6%
// faster with all rows in LDS).  Chunks wait in LDS rather than in registers:
// 8 register slots beside 6 in LDS, selected by uniform branches, moved a
// quarter less but ran 2% slower.
template <Variant V, bool BF16, int DEPTH, bool NT, uint32_t MODE>
__global__ __launch_bounds__(kBlock, 4) void run_kernel(const RunArgs a)
{
    extern __shared__ float4 slot_lds[];   // [slots][1 or 2 rows][kBlock]
    constexpr bool SHARED = V == Variant::FastGlobal;       // only snapshots move
    constexpr int kSlotRows = SHARED ? 1 : 2;
    const uint32_t mode = MODE == kAnyMode ? a.mode : MODE;
    const bool global_m = SHARED || (V == Variant::General && (mode & kModeGlobalProxy));
    const int64_t grp = blockIdx.x;
    const int64_t c = grp * kBlock + threadIdx.x;
    if (c >= (a.Pp >> 2)) return;
    const int64_t blk0 = grp * (kBlock * 4);
    const uint32_t t16 = threadIdx.x * 16u;
    const uint32_t q_hi = static_cast<uint32_t>((grp * kBlock) >> 32);
    const uint32_t q_lo = static_cast<uint32_t>(c);
    float* const row0 = a.S + tile_index(a.nw, 0, blk0 & ~(kTileElems - 1)) + (blk0 & (kTileElems - 1));
    float4* const mine = slot_lds + threadIdx.x;

    float4 th = load4_at<false>(a.theta + blk0, t16);
    const float4 hh = load4_at<NT>(a.h + blk0, t16);
    const float4 tt = load4_at<NT>(a.ts + blk0, t16);
    float4 mg = make_float4(0.f, 0.f, 0.f, 0.f);
    if (global_m) mg = load4_at<false>(row0 + kTileElems, t16);

    // Loads of the rows the schedule word wd takes from memory, into r.
    auto fetch = [&](uint32_t wd, Rows& r) __attribute__((always_inline)) {
        const bool mem = (wd & kRunSlotMask) == kRunMemory;
        float* p = row0 + (static_cast<int64_t>(wd >> kRunWorkerShift) << (kTileShift + 1));
        r.s = row_at<NT>(p, mem, t16);
        if constexpr (!SHARED) r.m = row_at<NT>(p + kTileElems, mem, t16);
    };
    Rows ring[DEPTH];
    uint32_t words[DEPTH];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        words[u] = a.sched[u];
        ring[u] = Rows{};
        fetch(words[u], ring[u]);
    }

    auto noise = [&](int j) __attribute__((always_inline)) {
        return normals4((static_cast<uint64_t>(q_hi) << 32) | q_lo,
                        a.t0 + static_cast<uint32_t>(j), a.key0, a.key1);
    };
    float4 z = noise(0);
    auto step = [&](int j, uint32_t& word, Rows& rows) __attribute__((always_inline)) {
        const uint32_t wd = word;
        const uint32_t next = a.sched[j + DEPTH];
        const uint32_t src = wd & kRunSlotMask;
        const uint32_t dst = (wd >> kRunDstShift) & kRunSlotMask;
        if (src != kRunMemory) {
            const float4* p = mine + src * (kSlotRows * kBlock);
            rows.s = p[0];
            if constexpr (!SHARED) rows.m = p[kBlock];
        }
        float4 m = global_m ? mg : rows.m;
        float4 d;
        d = stale_update4<BF16>(a.neg_lr, a.sigma, rows.s, hh, tt, z);
        z = noise(j + 1);
        float4 snap;
        if constexpr (V == Variant::General) {
            const int tau = (mode & kModeAdaptive)
                                ? static_cast<int>(a.sched[kRunTauAt + j]) : 0;
            commit4_general<MODE>(a, tau, d, rows.s, th, m, snap);
        } else {
            commit4_fast<false>(a, d, rows.s, th, m, snap);
        }
        if (global_m) mg = m;
        if (dst != kRunMemory) {
            float4* p = mine + dst * (kSlotRows * kBlock);
            p[0] = snap;
            if constexpr (!SHARED) p[kBlock] = m;
        }
        {
            const bool mem = dst == kRunMemory;
            float* p = row0 + (static_cast<int64_t>(wd >> kRunWorkerShift) << (kTileShift + 1));
            put_row_at<NT>(p, mem, t16, snap);
            if constexpr (!SHARED)
                put_row_at<NT>(p + kTileElems, mem && !(V == Variant::General && global_m), t16, m);
        }
        word = next;
        fetch(next, rows);
    };
    int j = 0;
    for (; j + DEPTH <= a.K; j += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) step(j + u, words[u], ring[u]);
    }
#pragma unroll
    for (int u = 0; u + 1 < DEPTH; ++u)
        if (j + u < a.K) step(j + u, words[u], ring[u]);
    store4_at<false>(a.theta + blk0, t16, th);
    if (global_m) store4_at<false>(row0 + kTileElems, t16, mg);
}

// A run over a vector too short to fill the chip with run_kernel's waves.  There a
// commit takes a wave's 200 instructions one after the other, 0.63 us, however
// few blocks there are; its serial part is only the step itself.  Here a block has
// 64 elements, one a lane of one wave (the consumer), every committing worker's
// pair of rows in LDS, and three waves that draw the noise of the next
// kShortPhase commits while the consumer takes the current ones (two rounds of
// their 192 lanes: 24 commits x 16 Philox blocks).  The consumer's chain is 25
// vector instructions and no memory but LDS, read one commit ahead; a worker that
// commits twice in a row hands its rows over in registers.  The consumer's place
// among the block's waves, which the hardware spreads over the SIMDs, changes every
// 256 blocks, the compute units of this chip: its consumers then share the SIMDs.
// (A tuning constant: another number of units would only spread them less evenly.)
//
// a.sched: the commits' slots, two 16-bit numbers a word; then each slot's worker;
// the staleness values from kRunTauAt on; the number of slots in the last word.
template <Variant V, bool BF16, uint32_t MODE>
__global__ __launch_bounds__(kBlock) void short_run_kernel(const RunArgs a)
{
    extern __shared__ float4 slot_lds[];
    constexpr int kLanes = static_cast<int>(kShortElems);
    constexpr bool FAST = V != Variant::General;
    const uint32_t mode = MODE == kAnyMode ? a.mode : MODE;
    const bool global_m = V == Variant::FastGlobal ||
                          (V == Variant::General && (mode & kModeGlobalProxy));
    const bool adaptive = V == Variant::General && (mode & kModeAdaptive);
    const int slots = static_cast<int>(a.sched[kRunWords - 1]);
    float2* const rows = reinterpret_cast<float2*>(slot_lds);              // [slots][64]: (s, m)
    float* const noise = reinterpret_cast<float*>(rows + slots * kLanes);  // [2][kShortPhase][64]
    uint16_t* const slot_of = reinterpret_cast<uint16_t*>(noise + 2 * kShortPhase * kLanes);
    uint32_t* const tau_of = reinterpret_cast<uint32_t*>(slot_of + short_sched_pad(a.K));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int consumer = (blockIdx.x >> 8) & 3;
    const int64_t blk0 = static_cast<int64_t>(blockIdx.x) * kLanes;        // (Pp: a multiple of 64)
    float* const row0 = a.S + tile_index(a.nw, 0, blk0) + lane;
    const uint32_t* const slot_worker = a.sched + (a.K + 1) / 2;

    for (int j = threadIdx.x; j < a.K + 2; j += kBlock)
        slot_of[j] = j < a.K ? static_cast<uint16_t>(a.sched[j >> 1] >> (16 * (j & 1))) : uint16_t{0};
    if (adaptive)
        for (int j = threadIdx.x; j < a.K; j += kBlock) tau_of[j] = a.sched[kRunTauAt + j];
    for (int k = wave; k < slots; k += 4) {
        const float* p = row0 + (static_cast<int64_t>(slot_worker[k]) << (kTileShift + 1));
        rows[k * kLanes + lane] = make_float2(p[0], global_m ? 0.0f : p[kTileElems]);
    }

    // sigma z of commits j0 .. j0 + kShortPhase - 1, drawn by `threads` threads
    auto draw = [&](int j0, float* out, int id, int threads) __attribute__((always_inline)) {
        for (int k = id; k < kShortPhase * (kLanes / 4); k += threads) {
            const int jj = k / (kLanes / 4);
            const int q = k % (kLanes / 4);
            const float4 z = normals4<false>(static_cast<uint64_t>(blk0 / 4 + q),
                                             a.t0 + static_cast<uint32_t>(j0 + jj), a.key0, a.key1);
            *reinterpret_cast<float4*>(out + jj * kLanes + 4 * q) =
                make_float4(a.sigma * z.x, a.sigma * z.y, a.sigma * z.z, a.sigma * z.w);
        }
    };
    draw(0, noise, threadIdx.x, kBlock);

    float th = 0.0f, hh = 0.0f, tt = 0.0f, mg = 0.0f;
    if (wave == consumer) {
        th = a.theta[blk0 + lane];
        hh = a.h[blk0 + lane];
        tt = a.ts[blk0 + lane];
        if (global_m) mg = row0[kTileElems];
    }
    __syncthreads();

    uint32_t slot = slot_of[0], slot_next = slot_of[1];
    float2 row = rows[slot * kLanes + lane];
    for (int j0 = 0, half = 0; j0 < a.K; j0 += kShortPhase, half ^= 1) {
        if (wave == consumer) {
            const int n = a.K - j0 < kShortPhase ? a.K - j0 : kShortPhase;
            const float* nz = noise + half * (kShortPhase * kLanes) + lane;
            float z = nz[0];
            for (int i = 0; i < n; ++i) {
                // what the next commit reads, before this one's rows are written
                float2 row_next = rows[slot_next * kLanes + lane];
                const uint32_t slot_after = slot_of[j0 + i + 2];
                const float z_next = nz[(i + 1 < kShortPhase ? i + 1 : i) * kLanes];
                const float s[1] = {row.x};
                float d[1] = {a.neg_lr * __builtin_fmaf(hh, s[0] - tt, z)};
                if (BF16) d[0] = __uint_as_float(pack_bf16(d[0], d[0]) << 16);
                float t[1] = {th}, m[1] = {global_m ? mg : row.y}, snap[1];
                if constexpr (FAST) {
                    commit_fast<1, false>(a, d, s, t, m);
                    snap[0] = t[0];
                } else {
                    const int tau = adaptive ? static_cast<int>(tau_of[j0 + i]) : 0;
                    commit_general<1, MODE>(a, tau, d, s, t, m, snap);
                }
                th = t[0];
                if (global_m) mg = m[0];
                rows[slot * kLanes + lane] = make_float2(snap[0], m[0]);
                const bool again = slot_next == slot;
                row.x = again ? snap[0] : row_next.x;
                row.y = again ? m[0] : row_next.y;
                slot = slot_next;
                slot_next = slot_after;
                z = z_next;
            }
        } else if (j0 + kShortPhase < a.K) {
            draw(j0 + kShortPhase, noise + (half ^ 1) * (kShortPhase * kLanes),
                 ((wave - consumer - 1) & 3) * 64 + lane, kBlock - 64);
        }
        __syncthreads();
    }
    for (int k = wave; k < slots; k += 4) {
        float* p = row0 + (static_cast<int64_t>(slot_worker[k]) << (kTileShift + 1));
        const float2 r = rows[k * kLanes + lane];
        p[0] = r.x;
        if (!global_m) p[kTileElems] = r.y;
    }
    if (wave == consumer) {
        a.theta[blk0 + lane] = th;
        if (global_m) row0[kTileElems] = mg;
    }
}

// ---------------------------------------------------------------------------
// Segment-norm scale factors (one pi per segment of the parameter vector).
// A commit's pi needs sums of squares over whole segments, so each commit is
// split in two launches: the step kernel starts commit t (forms d, m and the
// drift, stores m, writes each 1024-index group's tree sums of squares), and
// seg_blocks_kernel adds the group sums of each 2^18-index block by the same
// tree, after which the last block of each segment adds the block sums in
// order and forms the segment's pi.  The next step kernel applies those
// factors (and the pull) before starting the next commit, generating the
// pending update again.
// ---------------------------------------------------------------------------

__device__ __forceinline__ float4 f4(const float* p) { return *reinterpret_cast<const float4*>(p); }
// c ? x : y on values (a conditional on two float4 objects selects between
// their addresses, which keeps them out of registers).
__device__ __forceinline__ float4 pick(bool c, float4 x, float4 y)
{
    return make_float4(c ? x.x : y.x, c ? x.y : y.y, c ? x.z : y.z, c ? x.w : y.w);
}
__device__ __forceinline__ float lane(const float4& v, int k)
{
    return k == 0 ? v.x : k == 1 ? v.y : k == 2 ? v.z : v.w;
}

// Sum of the block's 256 per-thread values by the adjacent-pairs tree: lane
// butterflies (which add pairs 2k, 2k+1, then pairs of pairs, ...) within
// each wave, then (wave 0 + wave 1) + (wave 2 + wave 3).  Thread 0 gets the
// result.  Every thread of the block must call it.
__device__ __forceinline__ double block_tree_sum(double v, double* lds)
{
#pragma unroll
    for (int mask = 1; mask < 64; mask <<= 1) v = v + __shfl_xor(v, mask);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) lds[wave] = v;
    __syncthreads();
    const double r = (lds[0] + lds[1]) + (lds[2] + lds[3]);
    __syncthreads();
    return r;
}

// No occupancy hint: with no barrier in the kernel, the compiler's own
// register budget runs 2.5% faster than a 7-waves-per-SIMD cap.
template <Source SRC, bool BF16, bool DIAG, bool NT>
__global__ __launch_bounds__(kBlock)
void seg_step_kernel(const SegArgs a)
{
    static_assert(kBlock * 4 == kSegGroup, "one block per group of sums");
    __shared__ double lds[3][4];
    const int64_t grp = blockIdx.x;
    const int64_t c = grp * kBlock + threadIdx.x;
    const bool active = c < (a.Pp >> 2);   // the last group may hold fewer chunks
    const int64_t off = c * 4;
    // The block's segments: its first, and whether the whole block lies in it
    // (all but the blocks that hold a segment boundary), in which case every
    // element takes that segment's factor and the block forms one set of
    // sums.  The lookups are issued before the streaming loads, so their
    // latency hides behind those instead of delaying the update.
    const int32_t s_first = a.gseg[grp];
    const int64_t g_lo = grp * kSegGroup;
    const int64_t g_hi = (g_lo + kSegGroup < a.P) ? g_lo + kSegGroup : a.P;
    const int64_t s_lo = a.seg_off[s_first], s_hi = a.seg_off[s_first + 1];
    const bool one_seg = s_hi >= g_hi;
    const float pi_one = a.apply ? a.pi_seg[s_first] : 0.0f;

    const float* th_src = a.theta_row < 0 ? a.theta + off
                                          : a.S + tile_index(a.nw, a.theta_row, off);
    float4 th = active ? load4<NT>(th_src) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 th_old = th;
    float4 hv = make_float4(0.f, 0.f, 0.f, 0.f), tv = hv;
    // h and theta* keep the default cache policy even when everything else
    // streams: every commit reads them, and with the other streams marked
    // non-temporal the Infinity Cache holds them from one launch to the next
    // (measured 10% faster at 25M parameters).
    if (SRC == Source::Generated && active) {
        hv = load4<false>(a.h + off);
        tv = load4<false>(a.ts + off);
    }
    // The rows this commit starts from, loaded with the others so that the
    // thread waits for memory once: the committing worker's snapshot (unused
    // when it is the pending worker, whose pull is stored below) and its
    // moment (no earlier store of this launch touches it).
    // A row that holds theta_t is not read again: the committing worker's
    // snapshot when it is the pending worker (it pulls below) or the worker
    // whose row held theta_t.
    const bool cur_pulls_now = a.apply && a.w_cur == a.w_prev;
    float4 s_cur = make_float4(0.f, 0.f, 0.f, 0.f), m_cur = s_cur;
    if (a.start && active) {
        if (!cur_pulls_now && a.w_cur != a.theta_row)
            s_cur = load4<NT>(a.S + tile_index(a.nw, a.w_cur, off));
        m_cur = load4<NT>(a.M + tile_index(a.nw, a.m_row, off));
    }
    // The pending worker's snapshot, to generate its update again (and for
    // the diagnostics' kinetic energy).
    float* srow = a.S + tile_index(a.nw, a.w_prev, off);
    float4 sp = make_float4(0.f, 0.f, 0.f, 0.f);
    if ((SRC == Source::Generated || DIAG) && a.apply && active)
        sp = a.w_prev == a.theta_row ? th_old : load4<NT>(srow);
    double ek = 0.0, proxy = 0.0;   // diagnostic variant: energies of the pending commit
    if (a.apply && active) {
        // The pending commit's update: the caller's, or generated again at
        // the worker's snapshot, which its pull below replaces.
        float4 d;
        if (SRC == Source::Generated) {
            const float4 z = normals4(static_cast<uint64_t>(c), a.t - 1u, a.key0, a.key1);
            d = stale_update4<BF16>(a.neg_lr, a.sigma, sp, hv, tv, z);
        } else {
            d = load_given<SRC>(a.upd_prev, c, a.P);
        }
        // eq. 3 with the factor of each element's segment (padding stays put)
        if (one_seg) {
            if (off + 0 < a.P) th.x = __builtin_fmaf(pi_one, d.x, th.x);
            if (off + 1 < a.P) th.y = __builtin_fmaf(pi_one, d.y, th.y);
            if (off + 2 < a.P) th.z = __builtin_fmaf(pi_one, d.z, th.z);
            if (off + 3 < a.P) th.w = __builtin_fmaf(pi_one, d.w, th.w);
        } else {
            int32_t seg = s_first;
            auto factor = [&](int64_t i) {
                while (a.seg_off[seg + 1] <= i) ++seg;
                return a.pi_seg[seg];
            };
            if (off + 0 < a.P) th.x = __builtin_fmaf(factor(off + 0), d.x, th.x);
            if (off + 1 < a.P) th.y = __builtin_fmaf(factor(off + 1), d.y, th.y);
            if (off + 2 < a.P) th.z = __builtin_fmaf(factor(off + 2), d.z, th.z);
            if (off + 3 < a.P) th.w = __builtin_fmaf(factor(off + 3), d.w, th.w);
        }
        store4<NT>(srow, pick(a.pre_pull, th_old, th));
        if (DIAG) {
            // E_k against the worker's snapshot (eq. 11) and the proxy energy
            // (eq. 22) of the pending commit, whose moment is already stored.
            const float4 mp = f4(a.M + tile_index(a.nw, a.m_row_prev, off));
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (off + k < a.P) {
                    const double e = static_cast<double>(lane(th, k)) - static_cast<double>(lane(sp, k));
                    const double km = static_cast<double>(a.k_eff) * static_cast<double>(lane(mp, k));
                    ek += 0.5 * e * e;
                    proxy += 0.5 * km * km;
                }
            }
        }
    }
    if (DIAG && a.apply) {   // uniform: every thread of the block takes part
        const double bek = block_tree_sum(ek, lds[0]);
        const double bpr = block_tree_sum(proxy, lds[1]);
        if (threadIdx.x == 0) {
            atomicAdd(&a.diag[0], bek);
            atomicAdd(&a.diag[1], bpr);
        }
    }
    if (!a.start) {
        if (active && a.store_theta) store4<NT>(a.theta + off, th);
        return;
    }

    float4 s, d, mo;
    mo = make_float4(0.f, 0.f, 0.f, 0.f);
    s = mo;
    d = mo;
    if (active) {
        if (cur_pulls_now) s = pick(a.pre_pull, th_old, th);   // just pulled
        else if (a.w_cur == a.theta_row) s = th_old;
        else s = s_cur;
        if (SRC == Source::Generated) {
            const float4 z = normals4(static_cast<uint64_t>(c), a.t, a.key0, a.key1);
            d = stale_update4<BF16>(a.neg_lr, a.sigma, s, hv, tv, z);
        } else {
            d = load_given<SRC>(a.upd_cur, c, a.P);
        }
        float* mrow = a.M + tile_index(a.nw, a.m_row, off);
        mo = m_cur;
        float4 m;
        m.x = __builtin_fmaf(a.mu, mo.x, d.x);     // Alg. 1: m <- mu m + dtheta
        m.y = __builtin_fmaf(a.mu, mo.y, d.y);
        m.z = __builtin_fmaf(a.mu, mo.z, d.z);
        m.w = __builtin_fmaf(a.mu, mo.w, d.w);
        store4<NT>(mrow, m);
        if (a.store_theta) store4<NT>(a.theta + off, th);
        mo = m;
    }
    // Terms of the sums of squares: drift theta_t - s_t (eq. 16), m and d.
    double ta[4], tm[4], td[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double dr = static_cast<double>(lane(th, k) - lane(s, k));
        const double mk = static_cast<double>(lane(mo, k));
        const double dk = static_cast<double>(lane(d, k));
        ta[k] = dr * dr;
        tm[k] = mk * mk;
        td[k] = dk * dk;
    }
    // One set of group sums per segment the group touches (terms outside the
    // segment count as zero); the loop is uniform across the block.
    for (int32_t seg = s_first; seg == s_first || a.seg_off[seg] < g_hi; ++seg) {
        const int64_t lo = seg == s_first ? s_lo : a.seg_off[seg];
        const int64_t hi = seg == s_first ? s_hi : a.seg_off[seg + 1];
        double ca = 0.0, cm = 0.0, cd = 0.0;
        if (one_seg && g_lo + kSegGroup <= a.P) {
            // the whole group inside one segment and below P: no masks
            ca = (ta[0] + ta[1]) + (ta[2] + ta[3]);
            cm = (tm[0] + tm[1]) + (tm[2] + tm[3]);
            cd = (td[0] + td[1]) + (td[2] + td[3]);
        } else if (active) {
            double xa[4], xm[4], xd[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool in = off + k >= lo && off + k < hi;
                xa[k] = in ? ta[k] : 0.0;
                xm[k] = in ? tm[k] : 0.0;
                xd[k] = in ? td[k] : 0.0;
            }
            ca = (xa[0] + xa[1]) + (xa[2] + xa[3]);
            cm = (xm[0] + xm[1]) + (xm[2] + xm[3]);
            cd = (xd[0] + xd[1]) + (xd[2] + xd[3]);
        }
        // The wave's 256-index subtree (lane butterflies add pairs 2k, 2k+1,
        // then pairs of pairs, ...); seg_blocks_kernel adds the group's four
        // wave sums as (w0 + w1) + (w2 + w3), the next level of the same
        // tree.  No barrier: each wave writes its own slot.
#pragma unroll
        for (int mask = 1; mask < 64; mask <<= 1) {
            ca = ca + __shfl_xor(ca, mask);
            cm = cm + __shfl_xor(cm, mask);
            cd = cd + __shfl_xor(cd, mask);
        }
        if ((threadIdx.x & 63) == 0) {
            const int64_t q = (a.part_off[seg] + (grp - (lo / kSegGroup))) * kWavesPerGroup +
                              (threadIdx.x >> 6);
            const int64_t stride = a.npart * kWavesPerGroup;
            a.part[q] = ca;
            a.part[stride + q] = cm;
            a.part[2 * stride + q] = cd;
        }
        if (one_seg) break;
    }
}

// The lanes of one wave see each other's LDS writes made before this point.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The factor of segment seg from its sums of squares of the drift, the moment
// and the update, which lanes 0 to 2 of one whole wave hold as `sum`: the norms
// (binary64 square roots, rounded to binary32), then pi as in the element step
// (eq. 18 with norms).
__device__ void segment_factor(int32_t seg, int64_t size, double sum, const SegFactors& f)
{
    const float norm = static_cast<float>(sqrt(sum));
    const float na = __shfl(norm, 0), nm = __shfl(norm, 1), nd = __shfl(norm, 2);
    if ((threadIdx.x & 63) != 0) return;
    const float num = f.k_eff * nm - na;
    const float den = nd + f.eps;
    const float pi_raw = num / den;
    const float pi = (f.literal || pi_raw > 0.0f) ? pi_raw : 0.0f;
    f.pi_seg[seg] = pi;
    if (f.diag) {   // clamped elements (raw pi negative or NaN) and elements
        if (!(pi_raw >= 0.0f)) atomicAdd(&f.diag[2], static_cast<double>(size));
        atomicAdd(&f.diag[3], static_cast<double>(size));
    }
    // Recording: every element of the segment takes this factor, so its
    // histogram entry is one bin holding the segment's size.
    if (f.hist) {
        uint32_t* row = f.hist + (f.hist_per_seg ? static_cast<int64_t>(seg) * GEM_PI_BINS : 0);
        atomicAdd(&row[scale_bin(pi)], static_cast<uint32_t>(size));
    }
}

// The tree's upper levels and the factors.  A block has TEAMS times 256 threads
// and takes up to TEAMS consecutive index blocks (of kSegBlock indices) of one
// segment: a team of 256 threads adds an index block's 256 group sums -- zero for
// groups outside the segment -- by the same adjacent-pairs tree.  A segment that
// one block covers gets its factor there.  Else the blocks write their index
// blocks' sums, and the last of them to finish (a device-scope counter per
// segment, the sums released and acquired by device fences) adds the segment's
// sums in order and forms the factor; it also resets the counter for the next
// launch.  Which block is last does not change any sum: each is taken in one
// fixed order.
//
// The launch is latency alone (a few hundred kilobytes are read): a chain of
// dependent loads, the tree, the fences and the last block's loads.  With one
// index block a thread block, its metadata found through four arrays and the
// fences on every segment, it took 12.7 us a commit over 62 segments of 11.7M
// parameters (70.3 us a commit in all, now 62.5; 161 segments of 1M: 26.7 and
// 14.6).  So everything a block needs to know is one record (a unit), and four
// index blocks to a thread block spare segments of up to a million indices the
// fences.  Sixteen, four at a time, are slower than the fences (one segment of 3M
// 26.6 us a commit, 23.6).
template <int TEAMS>
__global__ __launch_bounds__(TEAMS* kBlock) void seg_blocks_kernel(const double* __restrict__ part,
                                                                  int64_t npart,
                                                                  const SegUnit* __restrict__ units,
                                                                  double* sup, int64_t nsup,
                                                                  uint32_t* seg_done, SegFactors f)
{
    static_assert(kBlock * kSegGroup == kSegBlock, "256 threads for the groups of an index block");
    static_assert(kWavesPerGroup == 4, "four waves per group");
    __shared__ double lds[3][TEAMS * 4];
    __shared__ double tail[3][64];
    __shared__ int last;
    const SegUnit u = units[blockIdx.x];
    const uint32_t hi = u.lo + (u.size - 1u);                       // the segment's last element
    const uint32_t seg_blk = u.lo / static_cast<uint32_t>(kSegBlock);
    const int sup_count = static_cast<int>(hi / static_cast<uint32_t>(kSegBlock) - seg_blk) + 1;
    const int nblk = sup_count - u.blk < TEAMS ? sup_count - u.blk : TEAMS;
    if (static_cast<int>(threadIdx.x >> 8) < nblk) {
        const uint32_t grp = (seg_blk + u.blk + (threadIdx.x >> 8)) * kBlock + (threadIdx.x & 255);
        const uint32_t g_lo = u.lo / static_cast<uint32_t>(kSegGroup);
        const uint32_t g_hi = hi / static_cast<uint32_t>(kSegGroup);
        double va = 0.0, vm = 0.0, vd = 0.0;
        if (grp >= g_lo && grp <= g_hi) {
            // the group's four wave sums, (w0 + w1) + (w2 + w3)
            const int64_t q = (int64_t{u.part_first} + (grp - g_lo)) * kWavesPerGroup;
            const int64_t stride = npart * kWavesPerGroup;
            const double* pa = part + q;
            const double* pm = part + stride + q;
            const double* pd = part + 2 * stride + q;
            va = (pa[0] + pa[1]) + (pa[2] + pa[3]);
            vm = (pm[0] + pm[1]) + (pm[2] + pm[3]);
            vd = (pd[0] + pd[1]) + (pd[2] + pd[3]);
        }
        // the index block's sums: lane butterflies (which add pairs 2k, 2k+1, then
        // pairs of pairs, ...) within each wave, then (wave 0 + wave 1) + (wave 2 + wave 3)
#pragma unroll
        for (int mask = 1; mask < 64; mask <<= 1) {
            va = va + __shfl_xor(va, mask);
            vm = vm + __shfl_xor(vm, mask);
            vd = vd + __shfl_xor(vd, mask);
        }
        if ((threadIdx.x & 63) == 0) {
            lds[0][threadIdx.x >> 6] = va;
            lds[1][threadIdx.x >> 6] = vm;
            lds[2][threadIdx.x >> 6] = vd;
        }
    }
    __syncthreads();
    const int kind = threadIdx.x < 3 ? static_cast<int>(threadIdx.x) : 0;
    auto pair_sum = [&](int p) {
        const double* l = &lds[kind][4 * p];
        return (l[0] + l[1]) + (l[2] + l[3]);
    };
    if (sup_count <= TEAMS) {
        if (threadIdx.x >= 64) return;
        double sum = 0.0;
        for (int p = 0; p < nblk; ++p) sum = sum + pair_sum(p);
        segment_factor(u.seg, u.size, sum, f);
        return;
    }
    if (threadIdx.x < 64) {
        if (threadIdx.x < 3)
            for (int p = 0; p < nblk; ++p)
                sup[kind * nsup + u.sup_first + u.blk + p] = pair_sum(p);
        if (threadIdx.x == 0) last = 0;
        __threadfence();   // release this block's sums to every XCD
        wave_sync();
        if (threadIdx.x == 0) {
            const uint32_t done = atomicAdd(&seg_done[u.seg], 1u) + 1u;
            last = done == static_cast<uint32_t>((sup_count + TEAMS - 1) / TEAMS);
            if (last) atomicExch(&seg_done[u.seg], 0u);
        }
    }
    __syncthreads();
    if (!last || threadIdx.x >= 64) return;
    __threadfence();       // acquire the other blocks' sums
    double sum = 0.0;
    for (int base = 0; base < sup_count; base += 64) {
        // the lanes load 64 index blocks' sums of each kind at once; lanes 0 to
        // 2 then add a kind each, in order (one wave: its LDS accesses stay in order)
        const int q = base + static_cast<int>(threadIdx.x);
        if (q < sup_count) {
            tail[0][threadIdx.x] = sup[u.sup_first + q];
            tail[1][threadIdx.x] = sup[nsup + u.sup_first + q];
            tail[2][threadIdx.x] = sup[2 * nsup + u.sup_first + q];
        }
        wave_sync();
        const int cnt = sup_count - base < 64 ? sup_count - base : 64;
        for (int k = 0; k < cnt; ++k) sum = sum + tail[kind][k];
        wave_sync();
    }
    segment_factor(u.seg, u.size, sum, f);
}

template <bool BF16>
__global__ __launch_bounds__(kBlock) void generate_kernel(const float* __restrict__ S, int64_t nw,
                                                         int32_t w, const float* __restrict__ h,
                                                         const float* __restrict__ ts, void* out,
                                                         int64_t P, uint32_t t, uint32_t key0,
                                                         uint32_t key1, float neg_lr, float sigma)
{
    const int64_t c = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const int64_t i0 = c * 4;
    if (i0 >= P) return;
    const float4 s = *reinterpret_cast<const float4*>(S + tile_index(nw, w, i0));
    const float4 hv = *reinterpret_cast<const float4*>(h + i0);
    const float4 tv = *reinterpret_cast<const float4*>(ts + i0);
    const float4 z = normals4(static_cast<uint64_t>(c), t, key0, key1);
    const float4 u4 = stale_update4<BF16>(neg_lr, sigma, s, hv, tv, z);
    const float d[4] = {u4.x, u4.y, u4.z, u4.w};
    if (BF16) {
        uint16_t* o = static_cast<uint16_t*>(out);
        if (i0 + 4 <= P) {
            uint2 u;
            u.x = (__float_as_uint(d[0]) >> 16) | (__float_as_uint(d[1]) & 0xFFFF0000u);
            u.y = (__float_as_uint(d[2]) >> 16) | (__float_as_uint(d[3]) & 0xFFFF0000u);
            *reinterpret_cast<uint2*>(o + i0) = u;
        } else {
            for (int k = 0; k < 4; ++k)
                if (i0 + k < P) o[i0 + k] = static_cast<uint16_t>(__float_as_uint(d[k]) >> 16);
        }
    } else {
        float* o = static_cast<float*>(out);
        if (i0 + 4 <= P) {
            *reinterpret_cast<float4*>(o + i0) = make_float4(d[0], d[1], d[2], d[3]);
        } else {
            for (int k = 0; k < 4; ++k)
                if (i0 + k < P) o[i0 + k] = d[k];
        }
    }
}

// Rows w0 .. w0 + rows - 1 of the table pieces at base, over [0, Pp): set to
// row (16-byte aligned), or to zero when row is null.
__global__ __launch_bounds__(kBlock) void fill_rows_kernel(float* base, int64_t nw, int32_t w0,
                                                           int32_t rows, int64_t Pp,
                                                           const float* row)
{
    const int64_t nchunk = Pp >> 2;
    const int64_t c = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (c >= nchunk) return;
    const float4 v = row ? reinterpret_cast<const float4*>(row)[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    for (int32_t r = 0; r < rows; ++r)
        *reinterpret_cast<float4*>(base + tile_index(nw, w0 + r, c * 4)) = v;
}

// out[i] = worker w's element i of the table pieces at base, i < P (out of
// any alignment).  Bound by memory: a thread copies the four elements of one
// 16-byte aligned chunk of out, `lead` being the elements out lies past such an
// address (0 to 3), from a source that need only be 4-byte aligned; chunks
// that reach over out's ends or a tile's edge go element by element.  One
// element per thread (the form without VEC, kept for an out not even aligned
// to 4 bytes) moved 25M elements in 57 us, 3.5 TB/s.
template <bool VEC>
__global__ __launch_bounds__(kBlock) void read_row_kernel(const float* __restrict__ base,
                                                          int64_t nw, int32_t w, int64_t P,
                                                          int32_t lead, float* __restrict__ out)
{
    const int64_t c = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if constexpr (!VEC) {
        if (c < P) out[c] = base[tile_index(nw, w, c)];
    } else {
        const int64_t i = 4 * c - lead;
        if (i >= 0 && i + 4 <= P && (i & (kTileElems - 1)) <= kTileElems - 4) {
            float4 v;
            __builtin_memcpy(&v, base + tile_index(nw, w, i), sizeof(v));
            *reinterpret_cast<float4*>(out + i) = v;
        } else {
            for (int64_t k = i < 0 ? 0 : i; k < i + 4 && k < P; ++k) out[k] = base[tile_index(nw, w, k)];
        }
    }
}

__global__ __launch_bounds__(kBlock) void gather_kernel(const float* __restrict__ src,
                                                        const int64_t* __restrict__ idx,
                                                        int64_t count, float* __restrict__ out)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (k < count) out[k] = src[idx[k]];
}

// out[w * count + k] = worker w's element idx[k] of the table pieces at base,
// for workers w = w0 + blockIdx.y.
__global__ __launch_bounds__(kBlock) void gather_rows_kernel(const float* __restrict__ base,
                                                             int64_t nw, int64_t w0,
                                                             const int64_t* __restrict__ idx,
                                                             int64_t count, float* __restrict__ out)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const int64_t w = w0 + blockIdx.y;
    if (k < count) out[w * count + k] = base[tile_index(nw, w, idx[k])];
}

__global__ __launch_bounds__(kBlock) void loss_kernel(const float* __restrict__ theta,
                                                      const float* __restrict__ h,
                                                      const float* __restrict__ ts, int64_t P,
                                                      double* out)
{
    __shared__ double red[kBlock];
    double acc = 0.0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < P;
         i += static_cast<int64_t>(gridDim.x) * kBlock) {
        const double e = static_cast<double>(theta[i]) - static_cast<double>(ts[i]);
        acc += 0.5 * static_cast<double>(h[i]) * e * e;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int step = kBlock / 2; step > 0; step >>= 1) {
        if (static_cast<int>(threadIdx.x) < step) red[threadIdx.x] += red[threadIdx.x + step];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(out, red[0]);
}

// Plain copy, the bandwidth reference: one 16-byte chunk per thread and
// trip of a grid-stride loop whose grid covers the whole copy up to 4 GiB
// (2^20 blocks), with non-temporal loads and stores.  On MI355X this moves
// 6.5-6.6 TB/s of reads plus writes; default-policy accesses reach 6.2 TB/s,
// and tiles of four chunks per thread 5.6 TB/s.
__global__ __launch_bounds__(kBlock) void copy_kernel(const float* __restrict__ src,
                                                      float* __restrict__ dst, int64_t count)
{
    const int64_t n4 = count / 4;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    for (int64_t k = first; k < n4; k += stride) store4<true>(dst + 4 * k, load4<true>(src + 4 * k));
    if (first < count - n4 * 4) dst[n4 * 4 + first] = src[n4 * 4 + first];
}

inline unsigned blocks_for(int64_t items) {
    return static_cast<unsigned>((items + kBlock - 1) / kBlock);
}

// lds: bytes of dynamic LDS reserved per block (unused by the kernel), which
// caps the blocks a CU holds at once.
template <Source SRC, Variant V, bool BF16, bool DIAG, int DEPTH, bool NT, bool REC = false>
hipError_t launch_one(const PassArgs& a, hipStream_t st, uint32_t lds = 0)
{
    if (REC) {
        // K histograms, then one spare word per thread
        const uint32_t need = (static_cast<uint32_t>(a.K) * kRecWords + kBlock) * 4u;
        lds = lds > need ? lds : need;
    }
    static_assert(DEPTH > 1 || (!REC && !DIAG), "depth 1: the plain single-commit pass");
    if (DEPTH == 1 && a.K != 1) return hipErrorInvalidValue;
    if (REC && a.rec_grid < 1) return hipErrorInvalidValue;
    const unsigned grid = REC ? static_cast<unsigned>(a.rec_grid) : blocks_for(a.Pp >> 2);
    hipLaunchKernelGGL((pass_kernel<SRC, V, BF16, DIAG, DEPTH, NT, REC>), dim3(grid), dim3(kBlock),
                       lds, st, a);
    return hipGetLastError();
}

// Recording passes of the default rule with per-worker moments on generated
// updates (one histogram per commit).
template <bool BF16>
hipError_t launch_rec(const PassArgs& a, int depth, bool stream, uint32_t deep_lds, hipStream_t st)
{
    constexpr Source G = Source::Generated;
    constexpr Variant F = Variant::Fast;
    if (depth == kPrefetchDeep)
        return stream ? launch_one<G, F, BF16, false, kPrefetchDeep, true, true>(a, st, deep_lds)
                      : launch_one<G, F, BF16, false, kPrefetchDeep, false, true>(a, st, deep_lds);
    if (depth != kPrefetchShallow) return hipErrorInvalidValue;
    return stream ? launch_one<G, F, BF16, false, kPrefetchShallow, true, true>(a, st)
                  : launch_one<G, F, BF16, false, kPrefetchShallow, false, true>(a, st);
}

// The diagnostic variant keeps the default cache policy.
template <Source SRC, Variant V, bool BF16>
hipError_t launch_d(const PassArgs& a, bool diag, bool stream, hipStream_t st)
{
    if (diag) return launch_one<SRC, V, BF16, true, kPrefetchShallow, false>(a, st);
    return stream ? launch_one<SRC, V, BF16, false, kPrefetchShallow, true>(a, st)
                  : launch_one<SRC, V, BF16, false, kPrefetchShallow, false>(a, st);
}

template <Source SRC, bool BF16>
hipError_t launch_fd(const PassArgs& a, Variant v, bool diag, int depth, bool stream,
                     uint32_t deep_lds, hipStream_t st)
{
    if (depth == kPrefetchDeep) {
        if constexpr (SRC == Source::Generated) {
            if (v == Variant::Fast && !diag)
                return stream ? launch_one<SRC, Variant::Fast, BF16, false, kPrefetchDeep, true>(
                                    a, st, deep_lds)
                              : launch_one<SRC, Variant::Fast, BF16, false, kPrefetchDeep, false>(
                                    a, st, deep_lds);
        }
        return hipErrorInvalidValue;
    }
    if (depth == kPrefetchNone && !diag) {
        switch (v) {
        case Variant::Fast:
            return stream ? launch_one<SRC, Variant::Fast, BF16, false, kPrefetchNone, true>(a, st)
                          : launch_one<SRC, Variant::Fast, BF16, false, kPrefetchNone, false>(a, st);
        case Variant::FastGlobal:
            return stream
                       ? launch_one<SRC, Variant::FastGlobal, BF16, false, kPrefetchNone, true>(a, st)
                       : launch_one<SRC, Variant::FastGlobal, BF16, false, kPrefetchNone, false>(a, st);
        case Variant::General: break;
        }
        return stream ? launch_one<SRC, Variant::General, BF16, false, kPrefetchNone, true>(a, st)
                      : launch_one<SRC, Variant::General, BF16, false, kPrefetchNone, false>(a, st);
    }
    if (depth != kPrefetchShallow && depth != kPrefetchNone) return hipErrorInvalidValue;
    switch (v) {
    case Variant::Fast: return launch_d<SRC, Variant::Fast, BF16>(a, diag, stream, st);
    case Variant::FastGlobal: return launch_d<SRC, Variant::FastGlobal, BF16>(a, diag, stream, st);
    case Variant::General: break;
    }
    return launch_d<SRC, Variant::General, BF16>(a, diag, stream, st);
}

}  // namespace

hipError_t launch_pass(const PassArgs& a, Source src, Variant v, bool bf16_out, bool diag,
                       bool rec, int depth, bool stream_rows, uint32_t deep_lds,
                       hipStream_t stream)
{
    if (rec) {
        if (src != Source::Generated || v != Variant::Fast || diag) return hipErrorInvalidValue;
        return bf16_out ? launch_rec<true>(a, depth, stream_rows, deep_lds, stream)
                        : launch_rec<false>(a, depth, stream_rows, deep_lds, stream);
    }
    switch (src) {
    case Source::Generated:
        return bf16_out ? launch_fd<Source::Generated, true>(a, v, diag, depth, stream_rows,
                                                             deep_lds, stream)
                        : launch_fd<Source::Generated, false>(a, v, diag, depth, stream_rows,
                                                              deep_lds, stream);
    case Source::GivenF32:
        return launch_fd<Source::GivenF32, false>(a, v, diag, depth, stream_rows, deep_lds, stream);
    case Source::GivenBF16:
        return launch_fd<Source::GivenBF16, false>(a, v, diag, depth, stream_rows, deep_lds,
                                                   stream);
    }
    return hipErrorInvalidValue;
}

namespace {

// Calls f(V, MODE) (as integral constants) with a run's specialisation: the
// default rule's variants, and of the general ones those whose single mode has
// its own kernel (kappa, the pre-commit pull, adaptive staleness, each with
// per-worker moments).
template <typename F>
hipError_t with_run_rule(const RunArgs& a, Variant v, F f)
{
    using AnyMode = std::integral_constant<uint32_t, kAnyMode>;
    using General = std::integral_constant<Variant, Variant::General>;
    switch (v) {
    case Variant::Fast: return f(std::integral_constant<Variant, Variant::Fast>{}, AnyMode{});
    case Variant::FastGlobal: return f(std::integral_constant<Variant, Variant::FastGlobal>{}, AnyMode{});
    case Variant::General: break;
    }
    if (a.eps >= 0x1p-60f) {
        switch (a.mode) {
        case kModeKappaMul: return f(General{}, std::integral_constant<uint32_t, kModeKappaMul>{});
        case kModePrePull: return f(General{}, std::integral_constant<uint32_t, kModePrePull>{});
        case kModeAdaptive: return f(General{}, std::integral_constant<uint32_t, kModeAdaptive>{});
        default: break;
        }
    }
    return f(General{}, AnyMode{});
}

}  // namespace

hipError_t launch_run(const RunArgs& a, Variant v, bool bf16_out, bool stream_rows,
                      uint32_t lds_bytes, hipStream_t stream)
{
    if (a.K < 1 || a.K > kRunCommits) return hipErrorInvalidValue;
    const dim3 grid(blocks_for(a.Pp >> 2)), block(kBlock);
    return with_run_rule(a, v, [&](auto rule, auto rule_mode) {
        constexpr Variant V = decltype(rule)::value;
        constexpr uint32_t MODE = decltype(rule_mode)::value;
        if (bf16_out && stream_rows)
            hipLaunchKernelGGL((run_kernel<V, true, kRunDepth, true, MODE>), grid, block, lds_bytes, stream, a);
        else if (bf16_out)
            hipLaunchKernelGGL((run_kernel<V, true, kRunDepth, false, MODE>), grid, block, lds_bytes, stream, a);
        else if (stream_rows)
            hipLaunchKernelGGL((run_kernel<V, false, kRunDepth, true, MODE>), grid, block, lds_bytes, stream, a);
        else
            hipLaunchKernelGGL((run_kernel<V, false, kRunDepth, false, MODE>), grid, block, lds_bytes, stream, a);
        return hipGetLastError();
    });
}

hipError_t launch_short_run(const RunArgs& a, Variant v, bool bf16_out, hipStream_t stream)
{
    const uint32_t slots = a.sched[kRunWords - 1];
    const bool adaptive = v == Variant::General && (a.mode & kModeAdaptive);
    if (a.K < 1 || slots < 1 || slots > static_cast<uint32_t>(kShortSlots) || a.Pp % kShortElems != 0 ||
        (a.K + 1) / 2 + static_cast<int>(slots) > (adaptive ? kRunTauAt : kRunWords - 1) ||
        (adaptive && kRunTauAt + a.K > kRunWords - 1))
        return hipErrorInvalidValue;
    const uint32_t lds = short_run_lds(static_cast<int>(slots), a.K, adaptive);
    const dim3 grid(static_cast<unsigned>(a.Pp / kShortElems)), block(kBlock);
    return with_run_rule(a, v, [&](auto rule, auto rule_mode) {
        constexpr Variant V = decltype(rule)::value;
        constexpr uint32_t MODE = decltype(rule_mode)::value;
        if (bf16_out) hipLaunchKernelGGL((short_run_kernel<V, true, MODE>), grid, block, lds, stream, a);
        else hipLaunchKernelGGL((short_run_kernel<V, false, MODE>), grid, block, lds, stream, a);
        return hipGetLastError();
    });
}

template <bool DIAG, bool NT>
void launch_seg_step_d(const SegArgs& a, Source src, bool bf16_out, hipStream_t stream)
{
    const unsigned grid = blocks_for(a.Pp >> 2);
    switch (src) {
    case Source::Generated:
        if (bf16_out)
            hipLaunchKernelGGL((seg_step_kernel<Source::Generated, true, DIAG, NT>), dim3(grid),
                               dim3(kBlock), 0, stream, a);
        else
            hipLaunchKernelGGL((seg_step_kernel<Source::Generated, false, DIAG, NT>), dim3(grid),
                               dim3(kBlock), 0, stream, a);
        break;
    case Source::GivenF32:
        hipLaunchKernelGGL((seg_step_kernel<Source::GivenF32, false, DIAG, NT>), dim3(grid),
                           dim3(kBlock), 0, stream, a);
        break;
    case Source::GivenBF16:
        hipLaunchKernelGGL((seg_step_kernel<Source::GivenBF16, false, DIAG, NT>), dim3(grid),
                           dim3(kBlock), 0, stream, a);
        break;
    }
}

hipError_t launch_seg_step(const SegArgs& a, Source src, bool bf16_out, bool stream_rows,
                           hipStream_t stream)
{
    // The diagnostic variant keeps the default cache policy (one instance).
    if (a.diag) launch_seg_step_d<true, false>(a, src, bf16_out, stream);
    else if (stream_rows) launch_seg_step_d<false, true>(a, src, bf16_out, stream);
    else launch_seg_step_d<false, false>(a, src, bf16_out, stream);
    return hipGetLastError();
}

hipError_t launch_seg_blocks(const double* part, int64_t npart, const SegUnit* units,
                            int64_t nunits, int teams, double* sup, int64_t nsup,
                            uint32_t* seg_done, const SegFactors& f, hipStream_t stream)
{
    if (nunits <= 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(nunits));
    if (teams == kSegTeams)
        hipLaunchKernelGGL(seg_blocks_kernel<kSegTeams>, grid, dim3(kSegTeams * kBlock), 0, stream, part,
                           npart, units, sup, nsup, seg_done, f);
    else if (teams == 1)
        hipLaunchKernelGGL(seg_blocks_kernel<1>, grid, dim3(kBlock), 0, stream, part, npart, units, sup,
                           nsup, seg_done, f);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_generate(const float* S, int64_t nw, int32_t w, const float* h,
                           const float* ts, void* out, bool bf16, int64_t P, uint32_t t,
                           uint32_t key0, uint32_t key1, float neg_lr, float sigma,
                           hipStream_t stream)
{
    const unsigned grid = blocks_for((P + 3) / 4);
    if (bf16)
        hipLaunchKernelGGL(generate_kernel<true>, dim3(grid), dim3(kBlock), 0, stream, S, nw, w, h,
                           ts, out, P, t, key0, key1, neg_lr, sigma);
    else
        hipLaunchKernelGGL(generate_kernel<false>, dim3(grid), dim3(kBlock), 0, stream, S, nw, w, h,
                           ts, out, P, t, key0, key1, neg_lr, sigma);
    return hipGetLastError();
}

hipError_t launch_fill_rows(float* base, int64_t nw, int32_t w0, int32_t rows, int64_t Pp,
                            const float* row, hipStream_t stream)
{
    if (rows <= 0 || Pp <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_rows_kernel, dim3(blocks_for(Pp >> 2)), dim3(kBlock), 0, stream, base,
                       nw, w0, rows, Pp, row);
    return hipGetLastError();
}

hipError_t launch_read_row(const float* base, int64_t nw, int32_t w, int64_t P, float* out,
                           hipStream_t stream)
{
    if (P <= 0) return hipSuccess;
    const auto at = reinterpret_cast<uintptr_t>(out);
    if (at % 4 != 0) {
        hipLaunchKernelGGL(read_row_kernel<false>, dim3(blocks_for(P)), dim3(kBlock), 0, stream, base,
                           nw, w, P, 0, out);
    } else {
        const int32_t lead = static_cast<int32_t>(at / 4 % 4);
        hipLaunchKernelGGL(read_row_kernel<true>, dim3(blocks_for((P + lead + 3) / 4)), dim3(kBlock), 0,
                           stream, base, nw, w, P, lead, out);
    }
    return hipGetLastError();
}

hipError_t launch_gather(const float* src, const int64_t* idx, int64_t count, float* out,
                         hipStream_t stream)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_kernel, dim3(blocks_for(count)), dim3(kBlock), 0, stream, src, idx,
                       count, out);
    return hipGetLastError();
}

hipError_t launch_gather_rows(const float* base, int64_t nw, const int64_t* idx, int64_t count,
                              float* out, hipStream_t stream)
{
    if (count <= 0 || nw <= 0) return hipSuccess;
    constexpr int64_t kMaxY = 65535;   // grid y limit
    for (int64_t w0 = 0; w0 < nw; w0 += kMaxY) {
        const int64_t rows = nw - w0 < kMaxY ? nw - w0 : kMaxY;
        hipLaunchKernelGGL(gather_rows_kernel, dim3(blocks_for(count), static_cast<unsigned>(rows)),
                           dim3(kBlock), 0, stream, base, nw, w0, idx, count, out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_loss(const float* theta, const float* h, const float* ts, int64_t P, double* out,
                       hipStream_t stream)
{
    const int64_t want = blocks_for(P);
    const unsigned grid = static_cast<unsigned>(want < 4096 ? (want > 0 ? want : 1) : 4096);
    hipLaunchKernelGGL(loss_kernel, dim3(grid), dim3(kBlock), 0, stream, theta, h, ts, P, out);
    return hipGetLastError();
}

hipError_t launch_copy(const float* src, float* dst, int64_t count, hipStream_t stream)
{
    if (count <= 0) return hipSuccess;
    const int64_t want = (count / 4 + kBlock - 1) / kBlock;
    const int64_t cap = int64_t{1} << 20;
    const unsigned grid = static_cast<unsigned>(want < 1 ? 1 : want < cap ? want : cap);
    hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(kBlock), 0, stream, src, dst, count);
    return hipGetLastError();
}

}  // namespace gemk
