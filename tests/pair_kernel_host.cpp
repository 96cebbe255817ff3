// The table kernel of the MRCA pairs (mrca_general_pairs_kernel) run on the
// host: its source text, PAIR_KERNEL_TEXT, with one thread per lane of a
// workgroup and a barrier for __syncthreads, workgroup after workgroup.
#include <barrier>
#include <cstddef>
#include <cstdint>
#include <thread>
#include <vector>

struct Index {
    uint32_t x, y;
};
static thread_local Index threadIdx;
static Index blockIdx;
static std::barrier<>* g_barrier;

struct alignas(16) uint4 {
    uint32_t x, y, z, w;
};
static inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
    return {x, y, z, w};
}
static inline uint32_t min(uint32_t a, uint32_t b) { return a < b ? a : b; }

#define __global__ static
#define __device__ static
#define __forceinline__ inline
#define __launch_bounds__(threads)
#define __shared__ static
#define __align__(bytes) __attribute__((aligned(bytes)))
#define __syncthreads() g_barrier->arrive_and_wait()

constexpr uint32_t kEmpty = 0xffffffffu, kWsStatus = 0, kWsStatusMixed = 1;

#include PAIR_KERNEL_TEXT

extern "C" void pairs(uint32_t S, uint32_t diff_log2, uint32_t n, const uint32_t* counter,
                      const uint32_t* surf, const uint32_t* times, const uint8_t* sites,
                      uint32_t* lb, uint32_t* ub) {
    const uint32_t ws[1] = {kWsStatusMixed};
    constexpr uint32_t cols = kPairTileCols * kPairColTiles;
    std::barrier<> barrier(kPairTileCols);
    g_barrier = &barrier;
    const uint32_t gx = (n + cols - 1) / cols, gy = (n + kPairTileRows - 1) / kPairTileRows;
    std::vector<std::thread> lanes;
    for (uint32_t t = 0; t < kPairTileCols; ++t)
        lanes.emplace_back([=] {
            threadIdx = {t, 0};
            for (uint32_t b = 0; b < gx * gy; ++b) {
                if (t == 0) blockIdx = {b % gx, b / gx};
                g_barrier->arrive_and_wait();
                mrca_general_pairs_kernel(S, diff_log2, n, counter, surf, times, sites, ws, lb,
                                          ub);
                g_barrier->arrive_and_wait();
            }
        });
    for (auto& lane : lanes) lane.join();
}
