// gem_selftest.hip -- device self-tests of the library's numerics, and the launches
// that a run is planned as (built as libgem_selftest.so; not part of the commit
// path).
//
// The commit kernels use range-specialised forms of correctly rounded
// division and square root (gem_device.hpp).  These kernels compare them, on
// the device and bit for bit, with hipcc's general IEEE operations:
//   - the logarithm's (f - 1) / (f + 1) (ln_quotient, and the general core
//     div_rn_core on the same operands) for every binary32 f the logarithm
//     can see (the 2^23 values in (sqrt(1/2), sqrt(2)]);
//   - the Box-Muller radius sqrt(-2 ln u) for every u = k 2^-24, k in
//     [1, 2^24]: the radicand against the logarithm's defined steps, the root
//     against the IEEE square root;
//   - r cos(phi), r sin(phi) for all 2^24 angles and both signs of r against
//     the defined steps of sin and cos;
//   - the core quotient div_rn_core on every pair of significands;
//   - the rounding to bfloat16 of every binary32 value, and the noise's Philox
//     words against the generator's plain rounds;
//   - the guarded quotient div_rn on Philox-random operand pairs spread over
//     the whole binary32 range (zeros, subnormals, infinities and NaNs
//     included), and on every significand of the denominator against a set
//     of numerators.
// Each entry point returns GEM_OK and the number of mismatching results, or a
// GEM_E* code (bad argument, allocation or HIP failure).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "../../include/gem.h"
#include "gem_device.hpp"
#include "gem_plan.hpp"

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ bool same_bits(float x, float y)
{
    const bool both_nan = (x != x) && (y != y);
    return both_nan || __float_as_uint(x) == __float_as_uint(y);
}

// f in (sqrt(1/2), sqrt(2)]: index j < 2^23 takes 1.m with m = j (up to the
// sqrt(2) cut), j >= 2^23 takes 0.5 * 1.m; out-of-domain indices are skipped.
__global__ __launch_bounds__(kThreads) void ln_div_kernel(unsigned long long* bad)
{
    const uint32_t j = blockIdx.x * kThreads + threadIdx.x;   // grid covers 2^24 exactly
    const uint32_t mant = j & 0x007FFFFFu;
    const bool upper = j >= (1u << 23);
    if (upper != (mant > 0x003504F3u)) return;   // the logarithm picks the branch by mant
    const float f = __uint_as_float(mant | (upper ? 0x3F000000u : 0x3F800000u));
    const float a = f - 1.0f, b = f + 1.0f;
    const float want = a / b;
    // the two forms the library uses for this quotient
    if (!same_bits(gemk::ln_quotient(a, b), want)) atomicAdd(bad, 1ull);
    if (!same_bits(gemk::div_rn_core(a, b), want)) atomicAdd(bad, 1ull);
}

// The defined steps of ln u, u = k 2^-24 in (0, 1], and of sin and cos of
// 2 pi k / 2^24, written out plainly with the general IEEE operations.
__device__ float defined_ln(float u)
{
    const uint32_t bits = __float_as_uint(u);
    int e = static_cast<int>(bits >> 23) - 127;
    const uint32_t mant = bits & 0x007FFFFFu;
    float f = __uint_as_float(mant | 0x3F800000u);
    if (mant > 0x003504F3u) {
        f = 0.5f * f;
        e += 1;
    }
    const float s = (f - 1.0f) / (f + 1.0f);
    const float z = s * s;
    float p = 1.0f / 9.0f;
    p = __builtin_fmaf(p, z, 1.0f / 7.0f);
    p = __builtin_fmaf(p, z, 1.0f / 5.0f);
    p = __builtin_fmaf(p, z, 1.0f / 3.0f);
    p = p * z;
    const float s2 = s + s;
    float r = __builtin_fmaf(static_cast<float>(e), 0x1.7f7d1cp-20f, __builtin_fmaf(s2, p, s2));
    return __builtin_fmaf(static_cast<float>(e), 0x1.62e4p-1f, r);
}

__device__ void defined_sincos(uint32_t k, float& sn, float& cs)
{
    const uint32_t j = (k + (1u << 21)) >> 22;
    const int rem = static_cast<int>(k) - static_cast<int>(j << 22);
    const float x = static_cast<float>(rem) * (6.28318530717958647692f * 0x1p-24f);
    const float x2 = x * x;
    float ps = 1.0f / 362880.0f;
    ps = __builtin_fmaf(ps, x2, -1.0f / 5040.0f);
    ps = __builtin_fmaf(ps, x2, 1.0f / 120.0f);
    ps = __builtin_fmaf(ps, x2, -1.0f / 6.0f);
    ps = ps * x2;
    const float sx = __builtin_fmaf(x, ps, x);
    float pc = -1.0f / 3628800.0f;
    pc = __builtin_fmaf(pc, x2, 1.0f / 40320.0f);
    pc = __builtin_fmaf(pc, x2, -1.0f / 720.0f);
    pc = __builtin_fmaf(pc, x2, 1.0f / 24.0f);
    pc = __builtin_fmaf(pc, x2, -0.5f);
    const float cx = __builtin_fmaf(pc, x2, 1.0f);
    switch (j & 3u) {
    case 0: sn = sx; cs = cx; break;
    case 1: sn = cx; cs = -sx; break;
    case 2: sn = -sx; cs = -cx; break;
    default: sn = -cx; cs = sx; break;
    }
}

__global__ __launch_bounds__(kThreads) void radius_kernel(unsigned long long* bad)
{
    const uint32_t k = blockIdx.x * kThreads + threadIdx.x + 1u;   // 1 .. 2^24
    const float want = -2.0f * defined_ln(static_cast<float>(k) * 0x1p-24f);
    const float x = gemk::neg_radicand_of_k24(k);
    if (!same_bits(-x, want)) atomicAdd(bad, 1ull);
    if (!same_bits(-gemk::neg_radius(x), __builtin_sqrtf(want))) atomicAdd(bad, 1ull);
}

__global__ __launch_bounds__(kThreads) void turn_kernel(float r, unsigned long long* bad)
{
    const uint32_t k = blockIdx.x * kThreads + threadIdx.x;        // 0 .. 2^24 - 1
    float sn, cs, zc, zs;
    defined_sincos(k, sn, cs);
    // (the word's low 8 bits do not enter)
    gemk::turn_times(-r, (k << 8) | ((k * 37u) & 255u), zc, zs);
    if (!same_bits(zc, r * cs)) atomicAdd(bad, 1ull);
    if (!same_bits(zs, r * sn)) atomicAdd(bad, 1ull);
}

// A binary32 value from 32 random bits, with the exponent field drawn over
// its whole range (so every binade, subnormals, zeros, infinities and NaNs
// occur), or from a narrower window around 1.
__device__ __forceinline__ float spread(uint32_t x, uint32_t y, bool narrow)
{
    const uint32_t sign = x & 0x80000000u;
    const uint32_t mant = x & 0x007FFFFFu;
    uint32_t ex = narrow ? 127u - 70u + (y % 141u) : (y % 256u);
    return __uint_as_float(sign | (ex << 23) | mant);
}

__global__ __launch_bounds__(kThreads) void div_random_kernel(uint64_t seed, int64_t count,
                                                              unsigned long long* bad)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (i >= count) return;
    const gemk::Words4 w = gemk::philox10(static_cast<uint32_t>(i), static_cast<uint32_t>(i >> 32),
                                          0x5e1f7e57u, 0u, static_cast<uint32_t>(seed),
                                          static_cast<uint32_t>(seed >> 32));
    const bool narrow = (w.x2 & 3u) != 0;   // three in four pairs near the core range
    const float num = spread(w.x0, w.x2 >> 2, narrow);
    const float den = spread(w.x1, w.x3, narrow);
    if (!same_bits(gemk::div_rn(num, den), num / den)) atomicAdd(bad, 1ull);
}

// Every significand of a denominator in [1, 2) scaled by 2^e_den, against
// numerators num[r].
__global__ __launch_bounds__(kThreads) void div_grid_kernel(const float* nums, int32_t nnum,
                                                            int32_t e_den, unsigned long long* bad)
{
    const uint32_t m = blockIdx.x * kThreads + threadIdx.x;   // grid covers 2^23 exactly
    const float den = __uint_as_float(((127u + static_cast<uint32_t>(e_den)) << 23) | m);
    uint32_t miss = 0;
    for (int32_t r = 0; r < nnum; ++r) {
        const float num = nums[r];
        miss += same_bits(gemk::div_rn(num, den), num / den) ? 0u : 1u;
    }
    if (miss) atomicAdd(bad, static_cast<unsigned long long>(miss));
}

// div_rn_core of every pair of numerator significand a0 + r, r < count, and
// denominator significand (a thread each): the residual num - den q is exact, and
// q is the correctly rounded quotient iff it lies within half a unit of q's last
// place times den (2^-24 den for q in [1, 2), 2^-25 den below 1; ties do not occur).
__global__ __launch_bounds__(kThreads) void div_core_kernel(uint32_t a0, uint32_t count,
                                                            unsigned long long* bad)
{
    const uint32_t m = blockIdx.x * kThreads + threadIdx.x;   // grid covers 2^23 exactly
    const float den = __uint_as_float(0x3F800000u | m);
    uint32_t miss = 0;
    for (uint32_t r = 0; r < count; ++r) {
        const float num = __uint_as_float(0x3F800000u | (a0 + r));
        const float half = (a0 + r >= m ? 0x1p-24f : 0x1p-25f) * den;
        const float res = __builtin_fmaf(-den, gemk::div_rn_core(num, den), num);
        miss += __builtin_fabsf(res) < half ? 0u : 1u;
    }
    if (miss) atomicAdd(bad, static_cast<unsigned long long>(miss));
}

// binary32 -> bfloat16 -> binary32, nearest-even; NaN stays a (quiet) NaN: the
// defined steps, on the integer.
__device__ float defined_bf16(float x)
{
    uint32_t b = __float_as_uint(x);
    if ((b & 0x7FFFFFFFu) > 0x7F800000u) b = (b | 0x00400000u) & 0xFFFF0000u;
    else b = (b + 0x7FFFu + ((b >> 16) & 1u)) & 0xFFFF0000u;
    return __uint_as_float(b);
}

__global__ __launch_bounds__(kThreads) void bf16_kernel(unsigned long long* bad)
{
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x;   // grid covers 2^24 exactly
    uint32_t miss = 0;
    for (uint32_t hi = 0; hi < 256; ++hi) {
        const float x = __uint_as_float((hi << 24) | i), y = __uint_as_float(((hi << 24) | i) * 2654435761u);
        float a = x, b = y;
        gemk::round_pair_to_bf16(a, b);
        miss += __float_as_uint(a) != __float_as_uint(defined_bf16(x));
        miss += __float_as_uint(b) != __float_as_uint(defined_bf16(y));
    }
    if (miss) atomicAdd(bad, static_cast<unsigned long long>(miss));
}

// The noise's words of counters (i, q_hi, t, 0), t uniform and per lane.
__global__ __launch_bounds__(kThreads) void noise_words_kernel(uint32_t q_hi, uint32_t t, uint32_t k0,
                                                               uint32_t k1, unsigned long long* bad)
{
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
    const uint32_t tl = t + (threadIdx.x & 1u);
    const gemk::Words4 a = gemk::philox10(i, q_hi, t, 0u, k0, k1);
    const gemk::Words4 b = gemk::philox10_noise<true>(i, q_hi, t, k0, k1);
    const gemk::Words4 c = gemk::philox10(i, q_hi, tl, 0u, k0, k1);
    const gemk::Words4 d = gemk::philox10_noise<false>(i, q_hi, tl, k0, k1);
    const bool ok = a.x0 == b.x0 && a.x1 == b.x1 && a.x2 == b.x2 && a.x3 == b.x3 &&
                    c.x0 == d.x0 && c.x1 == d.x1 && c.x2 == d.x2 && c.x3 == d.x3;
    if (!ok) atomicAdd(bad, 1ull);
}

template <typename Launch>
int run_counting(Launch launch, uint64_t* mismatches)
{
    unsigned long long* d_bad = nullptr;
    if (hipMalloc(&d_bad, sizeof(*d_bad)) != hipSuccess) return GEM_ENOMEM;
    int rc = GEM_OK;
    unsigned long long host = 0;
    if (hipMemset(d_bad, 0, sizeof(*d_bad)) != hipSuccess) rc = GEM_EHIP;
    if (!rc) {
        launch(d_bad);
        if (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess) rc = GEM_EHIP;
    }
    if (!rc && hipMemcpy(&host, d_bad, sizeof(host), hipMemcpyDeviceToHost) != hipSuccess)
        rc = GEM_EHIP;
    (void)hipFree(d_bad);
    if (!rc) *mismatches = host;
    return rc;
}

}  // namespace

extern "C" {

int gem_selftest_ln_div(uint64_t* mismatches)
{
    if (!mismatches) return GEM_EINVAL;
    return run_counting([](unsigned long long* bad) {
        hipLaunchKernelGGL(ln_div_kernel, dim3((1u << 24) / kThreads), dim3(kThreads), 0, 0, bad);
    }, mismatches);
}

int gem_selftest_radius(uint64_t* mismatches)
{
    if (!mismatches) return GEM_EINVAL;
    return run_counting([](unsigned long long* bad) {
        hipLaunchKernelGGL(radius_kernel, dim3((1u << 24) / kThreads), dim3(kThreads), 0, 0, bad);
    }, mismatches);
}

int gem_selftest_turn(float r, uint64_t* mismatches)
{
    if (!mismatches) return GEM_EINVAL;
    return run_counting([&](unsigned long long* bad) {
        hipLaunchKernelGGL(turn_kernel, dim3((1u << 24) / kThreads), dim3(kThreads), 0, 0, r, bad);
    }, mismatches);
}

// Numerator significands [a0, a0 + count), a0 + count <= 2^23, against all denominators'.
int gem_selftest_div_core(uint32_t a0, uint32_t count, uint64_t* mismatches)
{
    if (!mismatches || count > (1u << 23) || a0 > (1u << 23) - count) return GEM_EINVAL;
    return run_counting([&](unsigned long long* bad) {
        // launches of a fraction of a second each
        for (uint32_t done = 0; done < count;) {
            const uint32_t part = count - done < (1u << 14) ? count - done : 1u << 14;
            hipLaunchKernelGGL(div_core_kernel, dim3((1u << 23) / kThreads), dim3(kThreads), 0, 0,
                               a0 + done, part, bad);
            done += part;
        }
    }, mismatches);
}

int gem_selftest_bf16(uint64_t* mismatches)
{
    if (!mismatches) return GEM_EINVAL;
    return run_counting([](unsigned long long* bad) {
        hipLaunchKernelGGL(bf16_kernel, dim3((1u << 24) / kThreads), dim3(kThreads), 0, 0, bad);
    }, mismatches);
}

int gem_selftest_noise_words(uint32_t q_hi, uint32_t t, uint64_t seed, uint64_t* mismatches)
{
    if (!mismatches) return GEM_EINVAL;
    return run_counting([&](unsigned long long* bad) {
        hipLaunchKernelGGL(noise_words_kernel, dim3(1u << 12), dim3(kThreads), 0, 0, q_hi, t,
                           static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32), bad);
    }, mismatches);
}

int gem_selftest_div_random(uint64_t seed, int64_t count, uint64_t* mismatches)
{
    if (!mismatches || count < 0 || count > (int64_t{1} << 34)) return GEM_EINVAL;
    if (count == 0) {
        *mismatches = 0;
        return GEM_OK;
    }
    const unsigned grid = static_cast<unsigned>((count + kThreads - 1) / kThreads);
    return run_counting([&](unsigned long long* bad) {
        hipLaunchKernelGGL(div_random_kernel, dim3(grid), dim3(kThreads), 0, 0, seed, count, bad);
    }, mismatches);
}

// nums: host array of nnum numerators (1 <= nnum <= 4096); e_den in [-126, 127].
int gem_selftest_div_grid(const float* nums, int32_t nnum, int32_t e_den, uint64_t* mismatches)
{
    if (!mismatches || !nums || nnum < 1 || nnum > 4096 || e_den < -126 || e_den > 127)
        return GEM_EINVAL;
    float* d_nums = nullptr;
    if (hipMalloc(&d_nums, sizeof(float) * static_cast<size_t>(nnum)) != hipSuccess) return GEM_ENOMEM;
    int rc = GEM_OK;
    if (hipMemcpy(d_nums, nums, sizeof(float) * static_cast<size_t>(nnum), hipMemcpyHostToDevice) !=
        hipSuccess)
        rc = GEM_EHIP;
    if (!rc)
        rc = run_counting([&](unsigned long long* bad) {
            hipLaunchKernelGGL(div_grid_kernel, dim3((1u << 23) / kThreads), dim3(kThreads), 0, 0,
                               d_nums, nnum, e_den, bad);
        }, mismatches);
    (void)hipFree(d_nums);
    return rc;
}

// The launches that gem_sim_run takes T commits in (T > K, eps >= 2^-60, no
// diagnostics or recording), for the benchmark's labels and byte counts: out[0]
// launches, out[1] of them of short_run_kernel, out[2] of run_kernel with
// non-temporal accesses where the state outgrows the Infinity Cache, and out[3] the
// row pieces (a worker's snapshot and moment; with `shared` its snapshot) read from
// memory plus those written to it, in rows.  shared: the default rule with the
// shared moment.  cus and lds (bytes a compute unit): 0 for the current device's.
// Host only.
int gem_selftest_run_plan(int64_t P, int32_t n, int32_t shared, int32_t adaptive,
                          const int32_t* worker, int64_t T, int32_t cus, int32_t lds, int64_t* out)
{
    if (P < 1 || n < 1 || T < 0 || (T > 0 && !worker) || !out) return GEM_EINVAL;
    for (int64_t j = 0; j < T; ++j)
        if (worker[j] < 0 || worker[j] >= n) return GEM_EWORKER;
    int device = 0;
    if ((cus < 1 || lds < 1) &&
        (hipGetDevice(&device) != hipSuccess ||
         hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
         hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, device) !=
             hipSuccess))
        return GEM_EHIP;
    const gemk::RunTarget to{(P + 63) / 64 * 64, cus, lds,
                             shared ? gemk::kRunSlotBytes / 2 : gemk::kRunSlotBytes, adaptive != 0};
    const int64_t most = gemk::run_commits(to), launches = (T + most - 1) / most;
    std::vector<int32_t> last(static_cast<size_t>(n), -1);
    std::vector<uint32_t> words(gemk::kRunWords);
    out[0] = launches;
    out[1] = out[2] = out[3] = 0;
    for (int64_t l = 0, j0 = 0; l < launches; ++l) {
        const int k = static_cast<int>((T - j0) / (launches - l));
        const gemk::RunLaunch p = gemk::plan_launch(to, worker + j0, k, words.data(), last.data());
        out[1] += p.is_short;
        out[2] += !p.is_short && gemk::stream_run(p.distinct, k);
        out[3] += p.moved;
        j0 += k;
    }
    return GEM_OK;
}

}  // extern "C"
