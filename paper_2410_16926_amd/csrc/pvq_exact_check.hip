// The short quotients and roots of pvq_exact_dev.h against the operations that serve every argument, on the machine whose
// v_rcp_f32 and v_rsq_f32 they start from: points, amplitude codes and corrected weights are the same bits only if these are.
#include <hip/hip_runtime.h>

#include "pvq.h"
#include "pvq_diagnostics.h"
#include "pvq_exact_dev.h"

namespace {

using namespace pvq_exact_dev;

constexpr uint32_t kFrom = (127u - 100u) << 23, kTo = (127u + 100u) << 23;   // bits of 2^-100 and 2^100

__device__ inline bool same(float a, float b) { return __float_as_uint(a) == __float_as_uint(b); }

// 64 bits that look random for every (seed, i) (Steele, Lea and Flood, Fast splittable pseudorandom number generators, 2014)
__device__ inline uint64_t mixed(uint64_t seed, uint64_t i)
{
    uint64_t z = seed * 0xD1B54A32D192ED03ull + i * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ inline float with_exponent(int e, uint32_t significand) { return __uint_as_float((uint32_t)(e + 127) << 23 | (significand & 0x7FFFFFu)); }

// Sample i of `divide`: divisors of either sign over all their exponents (every second one the root of an integer), dividends
// that are arbitrary, or next to a multiple of the divisor, or next to one and a half, where quotients are nearest to what
// rounds the other way; exponents up to the ends of what the header allows.
__device__ inline bool divide_sample(uint64_t seed, uint64_t i)
{
    const uint64_t h = mixed(seed, 2 * i), g = mixed(seed, 2 * i + 1);
    divisor d;
    if (i & 1) {
        const float n = (float)(1 + (uint32_t)(h & 0xFFFF));
        d = root_divisor(n);
    } else {
        uint32_t significand = (uint32_t)h;
        if ((h >> 60) == 0) significand = (h >> 32 & 1) ? 0x7FFFFFu - (significand & 15) : significand & 15;
        float b = with_exponent((int)((h >> 33) % 120) - 60, significand);
        if (h >> 59 & 1) b = -b;
        d = divisor_of(b, reciprocal(b));
    }
    // q between the exponents -99 and 98, a = q b between -89 and 88 (a product's exponent is the sum of both or one more)
    const int eb = (int)(__float_as_uint(d.b) >> 23 & 0xFF) - 127;
    const int low = max(-99, -89 - eb), high = min(98, 87 - eb);
    const int eq = low + (int)((g >> 40) % (uint32_t)(high - low + 1));
    const float q = with_exponent(eq, (uint32_t)g);
    const int mode = (int)(g >> 24 & 3);
    float a;
    if (mode == 0) a = with_exponent(eq + eb, (uint32_t)(g >> 26));
    else a = (float)((mode == 2 ? (double)q + (double)with_exponent(eq - 24, 0u) : (double)q) * (double)fabsf(d.b));
    if (mode == 3) a = __uint_as_float(__float_as_uint(a) + (g >> 63 ? 1u : ~0u));
    if (h >> 58 & 1) a = -a;
    if (mode == 0 && (g & 0xFFF) == 0 && d.b > 0.0f) a = 0.0f;
    return same(divide(a, d), a / d.b);
}

__global__ __launch_bounds__(256) void exact_check_kernel(int what, uint32_t k, uint64_t first, uint64_t count, unsigned long long *mismatches)
{
    unsigned long long bad = 0;
    const uint64_t lanes = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += lanes) {
        const float x = __uint_as_float((uint32_t)(first + i));
        bool right = true;
        switch (what) {
        case PVQ_EXACT_RECIPROCAL: right = same(reciprocal(x), 1.0f / x); break;
        case PVQ_EXACT_ROOT: right = same(root_of(x), sqrtf(x)); break;
        case PVQ_EXACT_SMALL_OVER: right = same(small_over((float)k, x), (float)k / x); break;
        case PVQ_EXACT_INTEGER_OVER: right = same(integer_over((float)k, x), (float)k / x); break;
        case PVQ_EXACT_ROOT_DIVISOR: {
            const float n = (float)(first + i), root = sqrtf(n);
            const divisor d = root_divisor(n);
            right = same(d.b, root) && same(d.y, 1.0f / root);
            break;
        }
        default: right = divide_sample(k, first + i); break;
        }
        bad += right ? 0 : 1;
    }
    if (bad) atomicAdd(mismatches, bad);
}

}  // namespace

extern "C" int pvq_exact_selftest(int what, uint32_t k, uint64_t first, uint64_t count, uint64_t *mismatches, void *stream)
{
    if (!mismatches || what < PVQ_EXACT_RECIPROCAL || what > PVQ_EXACT_DIVIDE) return PVQ_E_INVALID_ARG;
    const uint64_t low = what == PVQ_EXACT_ROOT_DIVISOR ? 1 : what == PVQ_EXACT_DIVIDE ? 0 : kFrom;
    const uint64_t high = what == PVQ_EXACT_ROOT_DIVISOR ? 65537 : what == PVQ_EXACT_DIVIDE ? (uint64_t)1 << 40 : kTo;
    if (first < low || first > high || count > high - first) return PVQ_E_INVALID_ARG;
    if (what == PVQ_EXACT_SMALL_OVER && (k < 1 || k > 255)) return PVQ_E_INVALID_ARG;
    if (what == PVQ_EXACT_INTEGER_OVER && (k < 1 || k > 1023)) return PVQ_E_INVALID_ARG;
    if (count == 0) return PVQ_OK;
    const unsigned grid = (unsigned)((count + 255) / 256 < 4096 ? (count + 255) / 256 : 4096);
    hipLaunchKernelGGL(exact_check_kernel, dim3(grid), dim3(256), 0, reinterpret_cast<hipStream_t>(stream), what, k, first, count,
                       reinterpret_cast<unsigned long long *>(mismatches));
    return hipGetLastError() == hipSuccess ? PVQ_OK : PVQ_E_HIP;
}
