// The device's half-normal text on the host, where the same correctly rounded
// operations give the same bits: HALF_NORMAL_TEXT as it stands, and
// DEFINED_TEXT with the definition's reciprocal square root (six Newton steps
// from a line); and the oracle's C functions, which are the definition itself.
#include <atomic>
#include <cstdint>
#include <cstring>
#include <thread>
#include <vector>

extern "C" double oracle_radius(uint32_t w_radius);
extern "C" double oracle_angle(uint32_t w_angle);

#define __device__
#define __forceinline__ inline __attribute__((always_inline))
#define __constant__ static const

static inline long long __double_as_longlong(double x) {
    long long b;
    std::memcpy(&b, &x, 8);
    return b;
}
static inline double __longlong_as_double(long long b) {
    double x;
    std::memcpy(&x, &b, 8);
    return x;
}
static inline double series_step(double c, double x, double k) { return __builtin_fma(c, x, k); }
// x 2^k, exact
static inline double scaled(double x, int k) {
    return x * __longlong_as_double((long long)(1023 + k) << 52);
}
#define __builtin_ldexp(x, k) scaled(x, k)

namespace device {
#include HALF_NORMAL_TEXT
}
namespace defined {
#include DEFINED_TEXT
}

// what: 0 the radius against DEFINED_TEXT, 1 against the oracle, 2 the angle
// against the oracle.  Blocks of kBlock words `stride` blocks apart.
constexpr uint32_t kBlock = 256;
static uint32_t block_differs(int what, uint32_t w0) {
    double a[kBlock], b[kBlock];
    if (what == 2) {
        for (uint32_t i = 0; i < kBlock; ++i) {
            const uint32_t w = w0 + i;
            a[i] = w >= 0x80000000u ? device::half_normal_angle<true>(device::kHalfNormalSeries, w)
                                    : device::half_normal_angle<false>(device::kHalfNormalSeries, w);
            b[i] = oracle_angle(w);
        }
    } else {
        for (uint32_t i = 0; i < kBlock; ++i)
            a[i] = device::half_normal_radius(device::kHalfNormalSeries, w0 + i);
        if (what == 0)
            for (uint32_t i = 0; i < kBlock; ++i)
                b[i] = defined::half_normal_radius(defined::kHalfNormalSeries, w0 + i);
        else
            for (uint32_t i = 0; i < kBlock; ++i) b[i] = oracle_radius(w0 + i);
    }
    uint32_t n = 0;
    for (uint32_t i = 0; i < kBlock; ++i) n += a[i] != b[i];
    return n;
}

extern "C" uint64_t differing(int what, uint32_t stride, uint32_t threads) {
    std::atomic<uint64_t> count{0};
    std::vector<std::thread> pool;
    constexpr uint32_t blocks = (uint32_t)((1ull << 32) / kBlock);
    for (uint32_t t = 0; t < threads; ++t)
        pool.emplace_back([&, t] {
            uint64_t n = 0;
            for (uint64_t k = t; k * stride < blocks; k += threads)
                n += block_differs(what, (uint32_t)(k * stride) * kBlock);
            n += t == 0 ? block_differs(what, 0u - kBlock) : 0u;
            count += n;
        });
    for (auto& p : pool) p.join();
    return count;
}
