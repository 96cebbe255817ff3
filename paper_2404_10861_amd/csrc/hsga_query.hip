// hsga_query.hip -- gfx950 kernels of the end-of-run queries and their
// launchers: the stratified sample, the MRCA-generation bounds of all pairs,
// and trie reconstruction (tree metrics and the tree itself).
#include <mutex>

#include "hsga_device.hpp"
#include "hsga_internal.hpp"
#include "hsga_layout.hpp"

namespace hsga {

// ---------------------------------------------------------------------------
// Stratified end-of-run sample (Results, On-hardware Trial): agent k is
// drawn uniformly from the k-th of n equal strata; every agent when A <= n.
// counter == nullptr: a synchronous run, whose every counter is T.
__global__ __launch_bounds__(256) void sample_kernel(const uint32_t* __restrict__ counter,
                                                    const uint32_t* __restrict__ surf, uint32_t A,
                                                    uint32_t SW, uint32_t n, uint32_t T,
                                                    uint32_t k0, uint32_t k1,
                                                    uint32_t* __restrict__ idx_out,
                                                    uint32_t* __restrict__ counter_out,
                                                    uint32_t* __restrict__ surf_out) {
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t taken = A <= n ? A : n;
    if (k >= taken) return;
    uint32_t a = k;
    if (A > n) {
        const uint32_t lo = (uint32_t)((uint64_t)k * A / n);
        const uint32_t hi = (uint32_t)((uint64_t)(k + 1) * A / n);
        const uint4 w = philox4x32_10(make_uint4(k, 0u, T, kSample), k0, k1);
        a = lo + word_below(w.x, hi - lo);
    }
    idx_out[k] = a;
    counter_out[k] = counter ? counter[a] : T;
    for (uint32_t w = 0; w < SW; ++w) surf_out[(size_t)k * SW + w] = surf[(size_t)w * A + a];
}

// The whole population as its sample, four agents per thread: plain copies,
// transposed where a surface has two words, so bound by memory; 16-byte
// accesses move every line once, where one agent per thread wrote the two
// words of a surface in two strided passes.
template <int SW, bool COUNTER>
__global__ __launch_bounds__(256) void sample_all_kernel(const uint4* __restrict__ counter,
                                                        const uint32_t* __restrict__ surf,
                                                        uint32_t A, uint32_t T,
                                                        uint4* __restrict__ idx_out,
                                                        uint4* __restrict__ counter_out,
                                                        uint4* __restrict__ surf_out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A / 4u) return;
    const uint4 lo = reinterpret_cast<const uint4*>(surf)[i];
    uint4 hi = lo, c = make_uint4(T, T, T, T);
    if constexpr (SW > 1) hi = reinterpret_cast<const uint4*>(surf + A)[i];
    if constexpr (COUNTER) c = counter[i];
    idx_out[i] = make_uint4(4u * i, 4u * i + 1u, 4u * i + 2u, 4u * i + 3u);
    counter_out[i] = c;
    if constexpr (SW > 1) {
        surf_out[2 * (size_t)i] = make_uint4(lo.x, hi.x, lo.y, hi.y);
        surf_out[2 * (size_t)i + 1] = make_uint4(lo.z, hi.z, lo.w, hi.w);
    } else {
        surf_out[i] = lo;
    }
}

template <int SW>
static void launch_sample_all(const uint32_t* counter, const uint32_t* surf, uint32_t A,
                              uint32_t T, uint32_t* idx_out, uint32_t* counter_out,
                              uint32_t* surf_out, hipStream_t stream) {
    const dim3 blocks((A / 4 + 255) / 256);
    auto* c = reinterpret_cast<const uint4*>(counter);
    auto* io = reinterpret_cast<uint4*>(idx_out);
    auto* co = reinterpret_cast<uint4*>(counter_out);
    auto* so = reinterpret_cast<uint4*>(surf_out);
    if (counter)
        hipLaunchKernelGGL((sample_all_kernel<SW, true>), blocks, dim3(256), 0, stream, c, surf, A,
                           T, io, co, so);
    else
        hipLaunchKernelGGL((sample_all_kernel<SW, false>), blocks, dim3(256), 0, stream, c, surf,
                           A, T, io, co, so);
}

hipError_t launch_sample(const uint32_t* counter, const uint32_t* surf, uint32_t A, uint32_t SW,
                         uint32_t n, uint32_t T, uint32_t k0, uint32_t k1, uint32_t* idx_out,
                         uint32_t* counter_out, uint32_t* surf_out, hipStream_t stream) {
    // whole words of four agents where planes and buffers allow it (the
    // planes' own starts are 256-byte aligned, the second word's is A words on)
    const uintptr_t at = (uintptr_t)idx_out | (uintptr_t)counter_out | (uintptr_t)surf_out |
                         (uintptr_t)surf | (uintptr_t)counter;
    if (A <= n && A % 4 == 0 && at % 16 == 0) {
        if (SW == 1)
            launch_sample_all<1>(counter, surf, A, T, idx_out, counter_out, surf_out, stream);
        else
            launch_sample_all<2>(counter, surf, A, T, idx_out, counter_out, surf_out, stream);
        return hipGetLastError();
    }
    const uint32_t taken = A <= n ? A : n;
    const uint32_t blocks = (taken + 255) / 256;
    hipLaunchKernelGGL(sample_kernel, dim3(blocks ? blocks : 1), dim3(256), 0, stream, counter,
                       surf, A, SW, n, T, k0, k1, idx_out, counter_out, surf_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// MRCA-generation bounds (Distributed Phylogenetic Tracking: mismatching
// differentiae delimit common ancestry).
//
// Workspace header words.
constexpr uint32_t kWsStatus = 0;  // 0 all counters equal, 1 mixed, 2 past horizon
constexpr uint32_t kWsT = 1;
constexpr uint32_t kWsF = 2;
constexpr uint32_t kWsPerm = 64;    // site of each time rank (ascending time)
constexpr uint32_t kWsTimes = 128;  // deposit time of each rank
constexpr uint32_t kWsLbTab = 192;  // 65 entries: lb when the first mismatch is rank r (64: none)
constexpr uint32_t kWsUbTab = 320;  // 65 entries: ub likewise
constexpr uint32_t kWsStatusMixed = 1, kWsStatusHorizon = 2;

// Rank of this lane's time among the S lanes (ascending; empty sites last,
// ties by lane).  All 64 lanes call it.
__device__ __forceinline__ uint32_t time_rank(uint32_t held, uint32_t lane, uint32_t S) {
    uint32_t rank = 0;
    for (uint32_t q = 0; q < S; ++q) {
        const uint32_t tq = lane_value(held, q);
        rank += (tq < held || (tq == held && q < lane)) ? 1u : 0u;
    }
    return rank;
}

// Layout after T ingests, replayed in the wavefront (lane = site).
__device__ __forceinline__ uint32_t replay_layout(uint32_t kind, uint32_t S, uint32_t T,
                                                  uint32_t lane) {
    uint32_t held = kEmpty, leave = 0;
    place_items(kind, S, 0, T, held, leave, lane, [](uint32_t, int) {});
    return held;
}

// The item lane's site holds after T ingests: from the rule's tables when
// the query has them (constant time per site), else by the replay.
__device__ __forceinline__ uint32_t layout_lane(const RuleTable* rules, uint32_t kind, uint32_t S,
                                                uint32_t T, uint32_t lane) {
    if (rules) return scheme_layout_wave(rules, kind, S, T);
    return replay_layout(kind, S, T, lane);
}

// Classify the counters (four wavefronts); when all are equal, wavefront 0
// lays out the shared layout once (in ingest units: from the rule's tables,
// or by replaying the placements when the caller has none), orders its
// sites by deposit time and tabulates the bounds, in generations, for every
// possible first-mismatch rank.  A run's own layout (hint, S words in
// ingest units, the layout after the ingests of generation count hint_T) is
// used as it stands when every counter is hint_T: the layout is a function
// of the scheme and the count alone, so all three give the same words.
constexpr uint32_t kPrepareThreads = 256;   // 4 wavefronts classify; wave 0 does the rest
__global__ __launch_bounds__(kPrepareThreads) void mrca_prepare_kernel(
    Scheme sc, uint32_t n, const uint32_t* __restrict__ counter, uint32_t* __restrict__ ws,
    const uint32_t* __restrict__ hint, uint32_t hint_T, const RuleTable* __restrict__ rules) {
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t S = sc.S;
    const uint32_t T0 = counter[0];
    const uint64_t hz = horizon_of(sc.kind, S);
    // past_hz: an item past the site rule's horizon; long: more ingests
    // than a replay may take (no limit when the run's layout is used)
    bool same = true, past_hz = false, long_replay = false;
    // 16 loads in flight per thread before any is used
    constexpr uint32_t kBatch = 16;
    for (uint32_t k0 = tid; k0 < n; k0 += kPrepareThreads * kBatch) {
        uint32_t c[kBatch];
#pragma unroll
        for (uint32_t j = 0; j < kBatch; ++j) {
            const uint32_t k = k0 + kPrepareThreads * j;
            c[j] = k < n ? counter[k] : T0;
        }
#pragma unroll
        for (uint32_t j = 0; j < kBatch; ++j) {
            const uint32_t ing = ingests_of(c[j], sc.interval);
            same = same && c[j] == T0;
            past_hz = past_hz || (ing > 0 && (uint64_t)(ing - 1) > hz);
            long_replay = long_replay || ing > kMaxReplayGenerations;
        }
    }
    // the four wavefronts' findings, combined through LDS
    __shared__ uint32_t flags[kPrepareThreads / 64];
    const uint32_t f_wave = (__ballot(!same) != 0 ? 1u : 0u) | (__ballot(past_hz) != 0 ? 2u : 0u) |
                            (__ballot(long_replay) != 0 ? 4u : 0u);
    if (lane == 0) flags[tid >> 6] = f_wave;
    __syncthreads();
    uint32_t f = 0;
#pragma unroll
    for (uint32_t w = 0; w < kPrepareThreads / 64; ++w) f |= flags[w];
    const bool all_same = (f & 1u) == 0;
    const bool hinted = all_same && hint && T0 == hint_T;
    const bool any_past = (f & 2u) != 0 || (!hinted && !rules && (f & 4u) != 0);
    if (any_past || !all_same) {                 // the same decision in every thread
        if (tid == 0) {
            ws[kWsStatus] = any_past ? kWsStatusHorizon : kWsStatusMixed;
            ws[kWsT] = T0;
        }
        return;
    }
    __shared__ uint32_t times[64];
    uint32_t F = 0;
    if (tid < 64) {                              // wavefront 0: lane = site
        const uint32_t held = hinted ? (lane < S ? hint[lane] : kEmpty)
                                     : layout_lane(rules, sc.kind, S,
                                                   ingests_of(T0, sc.interval), lane);
        const uint32_t rank = time_rank(held, lane, S);
        F = (uint32_t)__popcll(__ballot(lane < S && held != kEmpty));
        if (lane < S) {
            const uint32_t gen = held == kEmpty ? kEmpty : held * sc.interval;   // deposit generation
            times[rank] = gen;
            ws[kWsPerm + rank] = lane;
            ws[kWsTimes + rank] = gen;
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    // first mismatch at rank r: ub = times[r], lb = times[r-1] + 1 (0 if r = 0);
    // no mismatch (entry 64): ub = T, lb = times[F-1] + 1 (0 if F = 0)
    ws[kWsLbTab + lane] = lane == 0 ? 0u : (lane < S ? times[lane - 1] + 1u : 0u);
    ws[kWsUbTab + lane] = lane < S ? times[lane] : 0u;
    if (lane == 0) {
        ws[kWsLbTab + 64] = F > 0 ? times[F - 1] + 1u : 0u;
        ws[kWsUbTab + 64] = T0;
        ws[kWsT] = T0;
        ws[kWsF] = F;
        ws[kWsStatus] = 0;
    }
}

// The annotation's surface words as one 64-bit value.
__device__ __forceinline__ uint64_t surface64(const uint32_t* __restrict__ surf, uint32_t SW,
                                              uint32_t a) {
    return SW == 2 ? ((uint64_t)surf[(size_t)a * 2 + 1] << 32) | surf[(size_t)a * 2]
                   : (uint64_t)surf[a];
}

// Fast route: each annotation's differentiae in ascending-time order, packed
// in 64 bits (rank r at bit r for one-bit differentiae, at byte r for bytes).
__device__ __forceinline__ void rank_annotations(uint32_t S, uint32_t diff_log2, uint32_t n,
                                                 const uint32_t* __restrict__ surf,
                                                 const uint32_t* __restrict__ ws,
                                                 uint64_t* __restrict__ ranked) {
    __shared__ uint32_t perm[64];
    if (threadIdx.x < 64) perm[threadIdx.x] = ws[kWsPerm + threadIdx.x];
    __syncthreads();
    const uint32_t a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= n) return;
    const uint32_t F = ws[kWsF];
    const uint64_t s = surface64(surf, (S << diff_log2) >> 5, a);
    const uint64_t mask = diff_log2 ? 0xffull : 1ull;
    uint64_t packed = 0;
    for (uint32_t r = 0; r < F; ++r)
        packed |= ((s >> (perm[r] << diff_log2)) & mask) << (r << diff_log2);
    ranked[a] = packed;
}

__global__ __launch_bounds__(256) void mrca_rank_kernel(uint32_t S, uint32_t diff_log2,
                                                       uint32_t n,
                                                       const uint32_t* __restrict__ surf,
                                                       const uint32_t* __restrict__ ws,
                                                       uint64_t* __restrict__ ranked) {
    if (ws[kWsStatus] != 0) return;
    rank_annotations(S, diff_log2, n, surf, ws, ranked);
}

// Fast route, all ordered pairs: x = P_a xor P_b; the first set bit gives
// the rank of the first mismatch (its bit index, or its byte index).  Each thread owns 4 adjacent columns of 4
// rows, so stores are 16-byte and a wavefront writes 1 KiB contiguously.
constexpr uint32_t kPairRows = 4;
__global__ __launch_bounds__(256) void mrca_allpairs_kernel(uint32_t n, uint32_t diff_log2,
                                                           const uint64_t* __restrict__ ranked,
                                                           const uint32_t* __restrict__ ws,
                                                           uint32_t* __restrict__ lb,
                                                           uint32_t* __restrict__ ub) {
    const uint32_t status = ws[kWsStatus];
    if (status == kWsStatusHorizon) {
        // a counter past the horizon: every bound reads 0xFFFFFFFF, a value
        // no valid bound takes (bounds are at most 2^32 - 2)
        const uint32_t c0 = (blockIdx.x * blockDim.x + threadIdx.x) * 4u;
        for (uint32_t rr = 0; rr < kPairRows; ++rr) {
            const uint32_t a = blockIdx.y * kPairRows + rr;
            for (uint32_t q = 0; q < 4; ++q) {
                if (a < n && c0 + q < n) {
                    lb[(size_t)a * n + c0 + q] = kEmpty;
                    ub[(size_t)a * n + c0 + q] = kEmpty;
                }
            }
        }
        return;
    }
    if (status != 0) return;
    __shared__ uint32_t lbt[65], ubt[65];
    if (threadIdx.x < 65) {
        lbt[threadIdx.x] = ws[kWsLbTab + threadIdx.x];
        ubt[threadIdx.x] = ws[kWsUbTab + threadIdx.x];
    }
    __syncthreads();
    const uint32_t c0 = (blockIdx.x * blockDim.x + threadIdx.x) * 4u;
    if (c0 >= n) return;
    const uint32_t a0 = blockIdx.y * kPairRows;
    uint64_t pb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) pb[q] = c0 + q < n ? ranked[c0 + q] : 0ull;
    const bool vec = (n & 3u) == 0;
    for (uint32_t rr = 0; rr < kPairRows; ++rr) {
        const uint32_t a = a0 + rr;
        if (a >= n) break;
        const uint64_t pa = ranked[a];
        uint32_t l[4], u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint64_t x = pa ^ pb[q];
            const uint32_t idx =
                x ? ((uint32_t)(__ffsll((long long)x) - 1) >> diff_log2) : 64u;
            l[q] = lbt[idx];
            u[q] = ubt[idx];
        }
        const size_t off = (size_t)a * n + c0;
        if (vec) {
            *reinterpret_cast<uint4*>(lb + off) = make_uint4(l[0], l[1], l[2], l[3]);
            *reinterpret_cast<uint4*>(ub + off) = make_uint4(u[0], u[1], u[2], u[3]);
        } else {
            for (uint32_t q = 0; q < 4 && c0 + q < n; ++q) {
                lb[off + q] = l[q];
                ub[off + q] = u[q];
            }
        }
    }
}

// General route (counters differ): one wavefront per annotation lays out
// its own layout (from the rule's tables, else by replay) and stores its
// retained deposit generations in ascending order with their sites.
// One launch for either kind of query: annotations that share a counter are
// put in time-rank order, one per thread of the first workgroups; those of
// different ages are laid out, one per wavefront.
__global__ __launch_bounds__(256) void mrca_annotations_kernel(
    Scheme sc, uint32_t diff_log2, uint32_t n, const uint32_t* __restrict__ counter,
    const uint32_t* __restrict__ surf, const uint32_t* __restrict__ ws,
    uint64_t* __restrict__ ranked, uint32_t* __restrict__ times, uint8_t* __restrict__ sites,
    const RuleTable* __restrict__ rules) {
    const uint32_t status = ws[kWsStatus];
    if (status == 0) {
        if (blockIdx.x * blockDim.x < n) rank_annotations(sc.S, diff_log2, n, surf, ws, ranked);
        return;
    }
    const uint32_t a = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (status != kWsStatusMixed || a >= n) return;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t S = sc.S;
    const uint32_t held = layout_lane(rules, sc.kind, S, ingests_of(counter[a], sc.interval), lane);
    const uint32_t rank = time_rank(held, lane, S);
    if (lane < S) {
        times[(size_t)a * S + rank] = held == kEmpty ? kEmpty : held * sc.interval;
        sites[(size_t)a * S + rank] = (uint8_t)lane;
    }
}

// General route, all ordered pairs.  An item keeps its site until it is
// overwritten, and every annotation's items come from one history, so of a
// pair with counters Ta >= Tb the retained items common to both are exactly
// a's items older than Tb: a prefix of a's time order, at the same sites in
// both.  The first mismatch is then the lowest time rank (in a's order)
// among the differing sites, counted only if its time is below Tb, and the
// item before it in a's order is the last agreeing one.
//
// The lowest rank among the set bits of a word is the least of eight table
// entries, one per byte; the 2 KB of tables of a row serve all its columns.
// A workgroup takes kPairTileRows rows and kPairTileCols columns (one per
// thread) kPairColTiles times, and writes a pair into both its rows: the
// row of the later annotation directly, the other one transposed through
// LDS so that 16 lanes write 64 contiguous bytes (pairs of equal counters
// are worked out once from each side).  Bound by LDS reads (ten a pair) and
// the stores.  A merge of the two time lists, up to 128 dependent steps a
// pair over global memory, took 1,148 us for 4,096 annotations of a hybrid
// 64-site surface, this form 81 us.
constexpr uint32_t kPairTileRows = 16, kPairTileCols = 256, kPairColTiles = 4;
constexpr uint32_t kNoRank = 64;
// words between columns of the transposed tile: 16 rows, then padding that
// keeps the 16-byte alignment and spreads the banks
constexpr uint32_t kPairStage = 20;

__global__ __launch_bounds__(kPairTileCols) void mrca_general_pairs_kernel(
    uint32_t S, uint32_t diff_log2, uint32_t n, const uint32_t* __restrict__ counter,
    const uint32_t* __restrict__ surf, const uint32_t* __restrict__ times,
    const uint8_t* __restrict__ sites, const uint32_t* __restrict__ ws, uint32_t* __restrict__ lb,
    uint32_t* __restrict__ ub) {
    if (ws[kWsStatus] != kWsStatusMixed) return;
    constexpr uint32_t R = kPairTileRows;
    __shared__ __align__(16) uint8_t first[R][8][256];       // lowest rank of a byte's bits
    __shared__ uint32_t t_of[R][64];                         // time of each rank
    __shared__ uint64_t s_row[R];
    __shared__ uint32_t T_row[R], T_col[kPairTileCols];
    __shared__ __align__(16) uint32_t stage[2][kPairTileCols * kPairStage];
    const uint32_t tid = threadIdx.x;
    const uint32_t row0 = blockIdx.y * R;
    const uint32_t SW = (S << diff_log2) >> 5;

    // the rows' tables, by way of rank by site and rank by nibble (in the
    // memory of the stage, which is not in use yet)
    uint8_t* rank_of = reinterpret_cast<uint8_t*>(stage[0]);            // [R][64]
    uint8_t* nibble = rank_of + R * 64;                                  // [R][16][16]
    for (uint32_t i = tid; i < R * 64; i += kPairTileCols) {
        const uint32_t row = i >> 6, r = i & 63u, a = row0 + row;
        uint32_t t = kEmpty;
        if (r < S && a < n) {
            t = times[(size_t)a * S + r];
            rank_of[row * 64 + sites[(size_t)a * S + r]] = (uint8_t)r;
        }
        t_of[row][r] = t;
    }
    if (tid < R) {
        const uint32_t a = row0 + tid;
        s_row[tid] = a < n ? surface64(surf, SW, a) : 0ull;
        T_row[tid] = a < n ? counter[a] : 0u;
    }
    __syncthreads();
    {
        const uint32_t row = tid >> 4, nib = tid & 15u;
        uint32_t rk[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t site = (nib * 4 + k) >> diff_log2;
            rk[k] = site < S && row0 + row < n ? rank_of[row * 64 + site] : kNoRank;
        }
        uint32_t val[16];
        val[0] = kNoRank;
#pragma unroll
        for (uint32_t v = 1; v < 16; ++v) val[v] = min(val[v & (v - 1)], rk[__builtin_ctz(v)]);
#pragma unroll
        for (uint32_t v = 0; v < 16; ++v) nibble[tid * 16 + v] = (uint8_t)val[v];
    }
    __syncthreads();
    for (uint32_t i = tid; i < R * 8 * 64; i += kPairTileCols) {
        const uint32_t row = i >> 9, byte = (i >> 6) & 7u, q = i & 63u;   // values 4q .. 4q + 3
        const uint8_t* lo = nibble + (row * 16 + byte * 2) * 16 + (q & 3u) * 4;
        const uint32_t hi = nibble[(row * 16 + byte * 2 + 1) * 16 + (q >> 2)];
        uint32_t w = 0;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) w |= min((uint32_t)lo[k], hi) << (8 * k);
        reinterpret_cast<uint32_t*>(first)[i] = w;
    }

    for (uint32_t ct = 0; ct < kPairColTiles; ++ct) {
        const uint32_t b0 = (blockIdx.x * kPairColTiles + ct) * kPairTileCols;
        if (b0 >= n) break;
        const uint32_t b = b0 + tid;
        const uint64_t sb = b < n ? surface64(surf, SW, b) : 0ull;
        // (a column past n takes no part: it is not stored directly, and no
        // row is above its counter in the transposed stores; a row may be
        // equal to it, since 2^32 - 1 is a counter too)
        const uint32_t Tb = b < n ? counter[b] : kEmpty;
        __syncthreads();          // tables built; the last tile's stage read
        T_col[tid] = Tb;
#pragma unroll
        for (uint32_t g = 0; g < R; g += 4) {
            uint32_t l4[4], u4[4];
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t row = g + q;
                const uint64_t y = s_row[row] ^ sb;
                const uint32_t y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32);
                uint32_t r = kNoRank;
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    r = min(r, (uint32_t)first[row][k][(y0 >> (8 * k)) & 0xffu]);
                if (SW > 1) {
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k)
                        r = min(r, (uint32_t)first[row][4 + k][(y1 >> (8 * k)) & 0xffu]);
                }
                u4[q] = r < kNoRank ? t_of[row][r] : kEmpty;
                l4[q] = r - 1u < kNoRank - 1u ? t_of[row][r - 1u] + 1u : 0u;
                const bool later = b < n && Tb <= T_row[row];
                if (later && u4[q] >= Tb) {
                    // no mismatch: the last of a's items older than Tb
                    uint32_t f = 0;
#pragma unroll
                    for (uint32_t step = 32; step; step >>= 1)
                        if (t_of[row][f + step - 1] < Tb) f += step;
                    if (t_of[row][f] < Tb) ++f;
                    u4[q] = Tb;
                    l4[q] = f ? t_of[row][f - 1] + 1u : 0u;
                }
                if (later && row0 + row < n) {
                    const size_t off = (size_t)(row0 + row) * n + b;
                    lb[off] = l4[q];
                    ub[off] = u4[q];
                }
            }
            *reinterpret_cast<uint4*>(&stage[0][tid * kPairStage + g]) =
                make_uint4(l4[0], l4[1], l4[2], l4[3]);
            *reinterpret_cast<uint4*>(&stage[1][tid * kPairStage + g]) =
                make_uint4(u4[0], u4[1], u4[2], u4[3]);
        }
        __syncthreads();
        const uint32_t row = tid & (R - 1u), a = row0 + row;
        for (uint32_t c = tid / R; c < kPairTileCols; c += kPairTileCols / R) {
            if (a < n && T_col[c] < T_row[row]) {
                const size_t off = (size_t)(b0 + c) * n + a;
                lb[off] = stage[0][c * kPairStage + row];
                ub[off] = stage[1][c * kPairStage + row];
            }
        }
    }
}

// ... where few sites or few annotations leave the tables above little to
// serve: the two sorted time lists of a pair are merged as they stand, at
// most 2 S steps, one thread per pair and nothing to prepare.  A whole query,
// merged and by tables: 4 sites 33.6 and 50.7 us for 1,919 annotations, 150
// and 179 for 6,000; 8 sites 40.9 and 50.6, but 111 and 93 for 4,096; 32
// sites 46.6 and 49.3 for 64, 53.3 and 61.0 for 513, 59.4 and 66.0 for 600,
// equal at 768 (where the tables' workgroups take a fourth tile of columns), 87
// and 73 for 900; 64 sites 41.0 and 30.5 for 100.
inline bool merge_pairs(uint32_t S, uint32_t n) {
    return S <= 4 || (S <= 8 && n < 3072) || (S <= 32 && n < 768);
}
constexpr uint32_t kMergePairRows = 512;     // grid rows
__global__ __launch_bounds__(256) void mrca_merge_pairs_kernel(
    uint32_t S, uint32_t diff_log2, uint32_t n, const uint32_t* __restrict__ counter,
    const uint32_t* __restrict__ surf, const uint32_t* __restrict__ times,
    const uint8_t* __restrict__ sites, const uint32_t* __restrict__ ws, uint32_t* __restrict__ lb,
    uint32_t* __restrict__ ub) {
    if (ws[kWsStatus] != kWsStatusMixed) return;
    const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n) return;
    const uint32_t SW = (S << diff_log2) >> 5;
    const uint64_t sb = surface64(surf, SW, b);
    const uint64_t mask = diff_log2 ? 0xffull : 1ull;
    const uint32_t* tb = times + (size_t)b * S;
    const uint8_t* kb = sites + (size_t)b * S;
    const uint32_t Tb = counter[b];
    // rows a = blockIdx.y, blockIdx.y + gridDim.y, ...: a small grid, so that
    // the shared-counter route, which skips this kernel, pays little for it
    for (uint32_t a = blockIdx.y; a < n; a += gridDim.y) {
        const uint64_t sa = surface64(surf, SW, a);
        const uint32_t* ta = times + (size_t)a * S;
        const uint8_t* ka = sites + (size_t)a * S;
        uint32_t i = 0, k = 0;
        bool have_last = false, mismatch = false;
        uint32_t last = 0, tstar = 0;
        while (i < S && k < S) {
            const uint32_t x = ta[i], y = tb[k];
            if (x == kEmpty || y == kEmpty) break;
            if (x == y) {
                if (((sa >> ((uint32_t)ka[i] << diff_log2)) & mask) !=
                    ((sb >> ((uint32_t)kb[k] << diff_log2)) & mask)) {
                    mismatch = true;
                    tstar = x;
                    break;
                }
                have_last = true;
                last = x;
                ++i;
                ++k;
            } else if (x < y) {
                ++i;
            } else {
                ++k;
            }
        }
        const uint32_t Ta = counter[a];
        const size_t off = (size_t)a * n + b;
        ub[off] = mismatch ? tstar : (Ta < Tb ? Ta : Tb);
        lb[off] = have_last ? last + 1u : 0u;
    }
}

// ---------------------------------------------------------------------------
// Trie reconstruction and phylometrics of annotations sharing a counter
// (Distributed Phylogenetic Tracking: reconstruction is a trie over the
// record of differentiae; Results, On-hardware Trial: sum branch length and
// mean evolutionary distinctiveness).  Annotations read as their
// differentiae in ascending deposit time are sorted lexicographically;
// neighbours in that order share a prefix of d_i = LCP(i, i+1) retained
// items, and the trie's branching nodes are exactly these boundaries.  A
// node at depth d sits at time tau(d) = t_d (the MRCA upper bound of the
// pairs it separates), tau(F) = T (identical annotations).
//   boundaries of one node: equal depth d with nothing shallower between
//     (a many-way split, or a run of identical annotations); the node
//     starts at the boundary whose nearest not-deeper left neighbour is
//     strictly shallower;
//   leaf i hangs from the deeper of boundaries i-1, i;
//   a node hangs from the deeper of its nearest strictly shallower
//   boundaries on either side (none: the root);
//   pairs (a, b) meet at the shallowest boundary between them, so the sum
//   over pairs of T - tau(MRCA) is a sum over all boundary ranges of their
//   minimum, counted by nearest-smaller spans.
// Six result words: sum of branch lengths, pair sum, root time, internal
// nodes, status, n.

// Sort keys: rank 0 most significant (bit-reversed for one-bit
// differentiae, byte-reversed for bytes).
__global__ __launch_bounds__(256) void phylo_keys_kernel(uint32_t n, uint32_t npad,
                                                        uint32_t diff_log2,
                                                        const uint64_t* __restrict__ ranked,
                                                        const uint32_t* __restrict__ ws,
                                                        uint64_t* __restrict__ keys,
                                                        uint32_t* __restrict__ idx) {
    if (ws[kWsStatus] != 0) return;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= npad) return;
    uint64_t key = ~0ull;
    if (i < n) key = diff_log2 ? __builtin_bswap64(ranked[i]) : __brevll(ranked[i]);
    keys[i] = key;
    idx[i] = i < n ? i : 0xffffffffu;
}

// Sort of (key, index), ascending by key then index.  Chunks of kSortChunk
// entries are sorted in LDS by a bitonic network (for k = 2, 4, .., chunk
// and j = k/2, .., 1, entries i and i + j, i with bit j clear, are ordered
// ascending where bit k of i is clear and descending where it is set), then
// merged in one launch: an entry's place is its place in its own chunk plus
// the number of entries before it in each other one, a binary search each.
// A chain of 11 loads per search (several searches side by side) replaces
// the network's passes over the whole array, one launch per stride: the
// 10,000-annotation tree took nine launches after the chunks' sort.
constexpr uint32_t kSortChunk = 2048;

__device__ __forceinline__ void sort_exchange(uint64_t& ka, uint32_t& ia, uint64_t& kb,
                                              uint32_t& ib, bool up) {
    const bool greater = ka > kb || (ka == kb && ia > ib);
    if (greater == up) {
        const uint64_t tk = ka;
        ka = kb;
        kb = tk;
        const uint32_t ti = ia;
        ia = ib;
        ib = ti;
    }
}

// One chunk of `chunk` entries (a power of two, at most kSortChunk) per
// workgroup of chunk / 2 threads.
__global__ __launch_bounds__(kSortChunk / 2) void phylo_sort_local_kernel(
    uint32_t chunk, const uint32_t* __restrict__ ws, uint64_t* __restrict__ keys,
    uint32_t* __restrict__ idx) {
    if (ws[kWsStatus] != 0) return;
    __shared__ uint64_t sk[kSortChunk];
    __shared__ uint32_t si[kSortChunk];
    const uint32_t base = blockIdx.x * chunk;
    const uint32_t t = threadIdx.x;
    sk[t] = keys[base + t];
    si[t] = idx[base + t];
    sk[t + chunk / 2] = keys[base + t + chunk / 2];
    si[t + chunk / 2] = idx[base + t + chunk / 2];
    __syncthreads();
    for (uint32_t k = 2; k <= chunk; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            const uint32_t i = (t / j) * 2 * j + (t % j);
            sort_exchange(sk[i], si[i], sk[i + j], si[i + j], (i & k) == 0);
            __syncthreads();
        }
    }
    keys[base + t] = sk[t];
    idx[base + t] = si[t];
    keys[base + t + chunk / 2] = sk[t + chunk / 2];
    idx[base + t + chunk / 2] = si[t + chunk / 2];
}

// The sorted chunks (kSortChunk entries each) merged into the first n places
// of keys_out and idx_out; the padding, greater than every annotation's
// entry, is left out.
__global__ __launch_bounds__(256) void phylo_merge_kernel(uint32_t n, uint32_t chunks,
                                                         const uint32_t* __restrict__ ws,
                                                         const uint64_t* __restrict__ keys,
                                                         const uint32_t* __restrict__ idx,
                                                         uint64_t* __restrict__ keys_out,
                                                         uint32_t* __restrict__ idx_out) {
    if (ws[kWsStatus] != 0) return;
    const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= chunks * kSortChunk) return;
    const uint64_t key = keys[e];
    const uint32_t id = idx[e];
    const uint32_t mine = e / kSortChunk;
    uint32_t place = e % kSortChunk;
    auto before = [&](uint32_t at) {
        const uint64_t k = keys[at];
        return k < key || (k == key && idx[at] < id);
    };
#pragma unroll 4
    for (uint32_t c = 0; c < chunks; ++c) {
        const uint32_t base = c * kSortChunk;
        uint32_t lo = 0;                       // entries known to come before
        for (uint32_t step = kSortChunk / 2; step > 0; step >>= 1)
            if (before(base + lo + step - 1)) lo += step;
        if (before(base + lo)) ++lo;
        place += c == mine ? 0u : lo;
    }
    if (place < n) {
        keys_out[place] = key;
        idx_out[place] = id;
    }
}

// Boundary depths and the tree, in parallel.  tab[k][i] = the minimum depth
// over boundaries [i, i + 2^k) (a sparse table); the nearest boundary to the
// left or right of b shallower than a depth is found by binary lifting over
// it, one thread per boundary.  Sums go to 64-bit accumulators.
constexpr uint32_t kPhyloMaxLevels = 17;   // 2^16 > 65534 boundaries
constexpr uint32_t kNoBoundary = 0xffffffffu;

struct PhyloAcc {
    unsigned long long sbl, pairs, internal, dmin;
};

__device__ __forceinline__ uint64_t phylo_tau(const uint32_t* ws, uint32_t d) {
    const uint32_t F = ws[kWsF];
    return d < F ? (uint64_t)ws[kWsTimes + d] : (uint64_t)ws[kWsT];
}

// The boundaries' depths (level 0) and the table's levels up to
// kTileLevels, a tile of 2^kTileLevels boundaries per workgroup: its depths
// and those of the next tile are enough, and stay in LDS from level to
// level, where each level was a launch of its own.
constexpr uint32_t kTileLevels = 10;
constexpr uint32_t kTableTile = 1u << kTileLevels;
__global__ __launch_bounds__(256) void phylo_depth_kernel(uint32_t n, uint32_t diff_log2,
                                                         uint32_t levels,
                                                         const uint32_t* __restrict__ ws,
                                                         const uint64_t* __restrict__ keys,
                                                         uint8_t* __restrict__ tab,
                                                         PhyloAcc* __restrict__ acc) {
    if (ws[kWsStatus] != 0) return;
    constexpr uint32_t PER = 2 * kTableTile / 256;
    __shared__ uint8_t low[2 * kTableTile];
    const uint32_t t = threadIdx.x, first = blockIdx.x * kTableTile;
    const uint32_t F = ws[kWsF], m = n - 1;
    if (first + t == 0) {
        acc->sbl = 0;
        acc->pairs = 0;
        acc->internal = 0;
        acc->dmin = F;
    }
    uint8_t v[PER];
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const uint32_t i = t + 256u * q, b = first + i;
        v[q] = 0xff;
        if (b < m) {
            const uint64_t x = keys[b] ^ keys[b + 1];
            const uint32_t d = x ? ((uint32_t)__clzll((long long)x) >> diff_log2) : 64u;
            v[q] = (uint8_t)(d < F ? d : F);
            if (i < kTableTile) tab[b] = v[q];
        }
        low[i] = v[q];
    }
    for (uint32_t k = 1; k < levels && k <= kTileLevels; ++k) {
        const uint32_t half = 1u << (k - 1);
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint32_t i = t + 256u * q + half;
            const uint8_t o = i < 2 * kTableTile ? low[i] : (uint8_t)0xff;
            v[q] = o < v[q] ? o : v[q];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint32_t i = t + 256u * q, b = first + i;
            low[i] = v[q];
            if (i < kTableTile && b + 2 * half <= m) tab[(size_t)k * m + b] = v[q];
        }
    }
}

// The levels above: minima of level kTileLevels at strides of its span.
__global__ __launch_bounds__(256) void phylo_table_kernel(uint32_t m, uint32_t levels,
                                                         const uint32_t* __restrict__ ws,
                                                         uint8_t* __restrict__ tab) {
    if (ws[kWsStatus] != 0) return;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i + 2 * kTableTile > m) return;
    const uint8_t* span = tab + (size_t)kTileLevels * m + i;
    uint8_t v = span[0];
    for (uint32_t k = kTileLevels + 1, j = 1; k < levels && i + (1u << k) <= m; ++k) {
        for (; j < 1u << (k - kTileLevels); ++j) {
            const uint8_t o = span[j * kTableTile];
            v = o < v ? o : v;
        }
        tab[(size_t)k * m + i] = v;
    }
}

// Nearest boundary i < b with depth[i] < d.
__device__ __forceinline__ uint32_t phylo_left_below(const uint8_t* tab, uint32_t m,
                                                     uint32_t levels, uint32_t b, uint32_t d) {
    uint32_t pos = b;   // every boundary in [pos, b) is at depth >= d
    for (uint32_t k = levels; k-- > 0;) {
        const uint32_t len = 1u << k;
        if (pos >= len && tab[(size_t)k * m + pos - len] >= d) pos -= len;
    }
    return pos == 0 ? kNoBoundary : pos - 1;
}

// Nearest boundary i > b with depth[i] < d.
__device__ __forceinline__ uint32_t phylo_right_below(const uint8_t* tab, uint32_t m,
                                                      uint32_t levels, uint32_t b, uint32_t d) {
    uint32_t pos = b + 1;   // every boundary in (b, pos) is at depth >= d
    for (uint32_t k = levels; k-- > 0;) {
        const uint32_t len = 1u << k;
        if (pos + len <= m && tab[(size_t)k * m + pos] >= d) pos += len;
    }
    return pos >= m ? kNoBoundary : pos;
}

__device__ __forceinline__ void phylo_add(PhyloAcc* acc, uint64_t sbl, uint64_t pairs,
                                          uint64_t internal, uint32_t dmin) {
    __shared__ unsigned long long s_sbl, s_pairs, s_internal;
    __shared__ uint32_t s_dmin;
    if (threadIdx.x == 0) {
        s_sbl = 0;
        s_pairs = 0;
        s_internal = 0;
        s_dmin = 0xffffffffu;
    }
    __syncthreads();
    if (sbl) atomicAdd(&s_sbl, (unsigned long long)sbl);
    if (pairs) atomicAdd(&s_pairs, (unsigned long long)pairs);
    if (internal) atomicAdd(&s_internal, (unsigned long long)internal);
    if (dmin != 0xffffffffu) atomicMin(&s_dmin, dmin);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_sbl) atomicAdd(&acc->sbl, s_sbl);
        if (s_pairs) atomicAdd(&acc->pairs, s_pairs);
        if (s_internal) atomicAdd(&acc->internal, s_internal);
        if (s_dmin != 0xffffffffu) atomicMin(&acc->dmin, (unsigned long long)s_dmin);
    }
}

// One thread per boundary b (depth d):
//   pairs meeting at b (b the rightmost shallowest boundary between them):
//     (b - L) (Rq - b), L = nearest left shallower (-1 if none), Rq =
//     nearest right not deeper (m if none), each adding T - tau(d);
//   a tree node starts at b unless the nearest not-deeper boundary on its
//   left has the same depth (one many-way node, or a run of identical
//   annotations); the node hangs from the deeper of its nearest shallower
//   boundaries (none on either side: the root).
__global__ __launch_bounds__(256) void phylo_boundary_kernel(uint32_t m, uint32_t levels,
                                                            const uint32_t* __restrict__ ws,
                                                            const uint8_t* __restrict__ tab,
                                                            PhyloAcc* __restrict__ acc) {
    if (ws[kWsStatus] != 0) return;
    const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t sbl = 0, pairs = 0, internal = 0;
    uint32_t dmin = 0xffffffffu;
    if (b < m) {
        const uint8_t* depth = tab;
        const uint32_t d = depth[b];
        const uint64_t T = ws[kWsT];
        const uint32_t L = phylo_left_below(tab, m, levels, b, d);
        const uint32_t Lq = phylo_left_below(tab, m, levels, b, d + 1);
        const uint32_t R = phylo_right_below(tab, m, levels, b, d);
        const uint32_t Rq = phylo_right_below(tab, m, levels, b, d + 1);
        const uint64_t nl = (uint64_t)b - (L == kNoBoundary ? (uint64_t)-1 : L);
        const uint64_t nr = (uint64_t)(Rq == kNoBoundary ? m : Rq) - b;
        pairs = (T - phylo_tau(ws, d)) * nl * nr;
        dmin = d;
        if (Lq == kNoBoundary || depth[Lq] < d) {
            internal = 1;
            if (L != kNoBoundary || R != kNoBoundary) {
                uint32_t pd;
                if (L == kNoBoundary) pd = depth[R];
                else if (R == kNoBoundary) pd = depth[L];
                else pd = depth[L] > depth[R] ? depth[L] : depth[R];
                sbl = phylo_tau(ws, d) - phylo_tau(ws, pd);
            }
        }
    }
    phylo_add(acc, sbl, pairs, internal, dmin);
}

// One thread per leaf: its edge from the deeper adjacent boundary to T.
__global__ __launch_bounds__(256) void phylo_leaf_kernel(uint32_t n,
                                                        const uint32_t* __restrict__ ws,
                                                        const uint8_t* __restrict__ depth,
                                                        PhyloAcc* __restrict__ acc) {
    if (ws[kWsStatus] != 0) return;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t sbl = 0;
    if (i < n && n > 1) {
        const uint32_t m = n - 1;
        uint32_t pd = i > 0 ? depth[i - 1] : 0u;
        if (i < m && (i == 0 || depth[i] > pd)) pd = depth[i];
        sbl = (uint64_t)ws[kWsT] - phylo_tau(ws, pd);
    }
    phylo_add(acc, sbl, 0, 0, 0xffffffffu);
}

__global__ __launch_bounds__(64) void phylo_finish_kernel(uint32_t n,
                                                         const uint32_t* __restrict__ ws,
                                                         const PhyloAcc* __restrict__ acc,
                                                         uint64_t* __restrict__ out) {
    if (threadIdx.x != 0) return;
    const uint32_t status = ws[kWsStatus];
    if (status != 0) {
        out[0] = out[1] = out[2] = out[3] = out[6] = out[7] = 0;
    } else {
        out[0] = acc->sbl;
        out[1] = acc->pairs;
        out[2] = n > 1 ? phylo_tau(ws, (uint32_t)acc->dmin) : ws[kWsT];
        out[3] = acc->internal;
        // the means, as binary64: mean evolutionary distinctiveness under
        // fair proportion (each edge shared equally by the leaves below it)
        // is the sum of branch lengths over n; the mean pairwise distance
        // is twice the pair sum over the n(n-1)/2 pairs (a path runs from
        // each leaf up to their MRCA)
        const double pairs = (double)n * (double)(n - 1) * 0.5;
        const double ed = (double)acc->sbl / (double)n;
        const double mpd = n > 1 ? 2.0 * (double)acc->pairs / pairs : 0.0;
        out[6] = (uint64_t)__double_as_longlong(ed);
        out[7] = (uint64_t)__double_as_longlong(mpd);
    }
    out[4] = status;
    out[5] = n;
}

// The tree itself.  A node is named by the first boundary of its run (the
// first boundary after its nearest shallower left boundary L that is not
// deeper than it).
constexpr uint32_t kPhyloRoot = 0xffffffffu, kPhyloNotNode = 0xfffffffeu;

__device__ __forceinline__ uint32_t phylo_node_of(const uint8_t* tab, uint32_t m,
                                                  uint32_t levels, uint32_t b) {
    const uint32_t d = tab[b];
    const uint32_t L = phylo_left_below(tab, m, levels, b, d);
    if (L == kNoBoundary) return tab[0] <= d ? 0u : phylo_right_below(tab, m, levels, 0, d + 1);
    return phylo_right_below(tab, m, levels, L, d + 1);
}

// One thread per boundary: node_parent[b] = the parent node (kPhyloRoot for
// the root) when b starts a node, kPhyloNotNode otherwise; node_time[b] =
// the time of b's node.
__global__ __launch_bounds__(256) void phylo_tree_kernel(uint32_t m, uint32_t levels,
                                                        const uint32_t* __restrict__ ws,
                                                        const uint8_t* __restrict__ tab,
                                                        uint32_t* __restrict__ node_parent,
                                                        uint32_t* __restrict__ node_time) {
    if (ws[kWsStatus] != 0) return;
    const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= m) return;
    const uint32_t d = tab[b];
    node_time[b] = (uint32_t)phylo_tau(ws, d);
    const uint32_t Lq = phylo_left_below(tab, m, levels, b, d + 1);
    if (Lq != kNoBoundary && tab[Lq] == d) {
        node_parent[b] = kPhyloNotNode;
        return;
    }
    const uint32_t L = phylo_left_below(tab, m, levels, b, d);
    const uint32_t R = phylo_right_below(tab, m, levels, b, d);
    if (L == kNoBoundary && R == kNoBoundary) {
        node_parent[b] = kPhyloRoot;
        return;
    }
    uint32_t p;
    if (L == kNoBoundary) p = R;
    else if (R == kNoBoundary) p = L;
    else p = tab[L] >= tab[R] ? L : R;
    node_parent[b] = phylo_node_of(tab, m, levels, p);
}

// One thread per sorted position i: the annotation idx[i] hangs from the
// node of the deeper adjacent boundary.
__global__ __launch_bounds__(256) void phylo_tree_leaf_kernel(uint32_t n, uint32_t levels,
                                                             const uint32_t* __restrict__ ws,
                                                             const uint8_t* __restrict__ tab,
                                                             const uint32_t* __restrict__ idx,
                                                             uint32_t* __restrict__ leaf_parent) {
    if (ws[kWsStatus] != 0) return;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (n == 1) {
        leaf_parent[idx[i]] = kPhyloRoot;
        return;
    }
    const uint32_t m = n - 1;
    uint32_t pb;
    if (i == 0) pb = 0;
    else if (i == m) pb = m - 1;
    else pb = tab[i] > tab[i - 1] ? i : i - 1;
    leaf_parent[idx[i]] = phylo_node_of(tab, m, levels, pb);
}

size_t phylo_workspace_bytes(uint32_t S, uint32_t n) {
    size_t npad = 1;
    while (npad < n) npad <<= 1;
    const size_t a = (MrcaWorkspace::bytes(S, n) + 255) & ~(size_t)255;
    return a + npad * 8 + npad * 4 + 256 + (size_t)kPhyloMaxLevels * n + 1024;
}

hipError_t launch_phylo(const Scheme& scm, uint32_t n, const uint32_t* counter,
                        const uint32_t* surf, uint64_t* out, void* workspace,
                        hipStream_t stream, uint32_t* leaf_parent, uint32_t* node_parent,
                        uint32_t* node_time, LayoutHint hint) {
    const uint32_t diff_log2 = scm.bits == 8 ? 3u : 0u;
    uint8_t* base = static_cast<uint8_t*>(workspace);
    uint32_t* ws = reinterpret_cast<uint32_t*>(base);
    uint64_t* ranked = reinterpret_cast<uint64_t*>(base + MrcaWorkspace::kHeader);
    size_t npad = 1;
    while (npad < n) npad <<= 1;
    size_t off = (MrcaWorkspace::bytes(scm.S, n) + 255) & ~(size_t)255;
    uint64_t* keys = reinterpret_cast<uint64_t*>(base + off);   off += npad * 8;
    uint32_t* idx = reinterpret_cast<uint32_t*>(base + off);    off += npad * 4;
    off = (off + 255) & ~(size_t)255;
    PhyloAcc* acc = reinterpret_cast<PhyloAcc*>(base + off);    off += 256;
    uint8_t* tab = base + off;                                  // levels x m bytes
    const uint32_t m = n - 1;
    uint32_t levels = 1;
    while (levels < kPhyloMaxLevels && (2u << (levels - 1)) <= m) ++levels;
    const uint32_t gn = (n + 255) / 256;
    hipLaunchKernelGGL(mrca_prepare_kernel, dim3(1), dim3(kPrepareThreads), 0, stream, scm, n,
                       counter, ws, hint.layout, hint.T, hint.rules);
    hipLaunchKernelGGL(mrca_rank_kernel, dim3(gn), dim3(256), 0, stream, scm.S, diff_log2, n,
                       surf, ws, ranked);
    hipLaunchKernelGGL(phylo_keys_kernel, dim3((uint32_t)((npad + 255) / 256)), dim3(256), 0,
                       stream, n, (uint32_t)npad, diff_log2, ranked, ws, keys, idx);
    if (npad > 1) {
        const uint32_t chunk = npad < kSortChunk ? (uint32_t)npad : kSortChunk;
        const uint32_t chunks = (n + chunk - 1) / chunk;
        hipLaunchKernelGGL(phylo_sort_local_kernel, dim3(chunks), dim3(chunk / 2), 0, stream,
                           chunk, ws, keys, idx);
        if (chunks > 1) {
            // into the workspace's layouts, which this query does not use
            // (12 bytes per annotation of at least 20)
            uint8_t* to = base + MrcaWorkspace::kHeader + (((size_t)n * 8 + 255) & ~(size_t)255);
            uint64_t* keys_out = reinterpret_cast<uint64_t*>(to);
            uint32_t* idx_out = reinterpret_cast<uint32_t*>(to + (size_t)n * 8);
            hipLaunchKernelGGL(phylo_merge_kernel, dim3(chunks * kSortChunk / 256), dim3(256), 0,
                               stream, n, chunks, ws, keys, idx, keys_out, idx_out);
            keys = keys_out;
            idx = idx_out;
        }
    }
    const uint32_t tiles = m ? (m + kTableTile - 1) / kTableTile : 1u;
    hipLaunchKernelGGL(phylo_depth_kernel, dim3(tiles), dim3(256), 0, stream, n, diff_log2, levels,
                       ws, keys, tab, acc);
    if (levels > kTileLevels + 1)
        hipLaunchKernelGGL(phylo_table_kernel, dim3(gn), dim3(256), 0, stream, m, levels, ws, tab);
    if (m > 0)
        hipLaunchKernelGGL(phylo_boundary_kernel, dim3((m + 255) / 256), dim3(256), 0, stream, m,
                           levels, ws, tab, acc);
    hipLaunchKernelGGL(phylo_leaf_kernel, dim3(gn), dim3(256), 0, stream, n, ws, tab, acc);
    hipLaunchKernelGGL(phylo_finish_kernel, dim3(1), dim3(64), 0, stream, n, ws, acc, out);
    if (leaf_parent) {
        if (m > 0)
            hipLaunchKernelGGL(phylo_tree_kernel, dim3((m + 255) / 256), dim3(256), 0, stream, m,
                               levels, ws, tab, node_parent, node_time);
        hipLaunchKernelGGL(phylo_tree_leaf_kernel, dim3(gn), dim3(256), 0, stream, n, levels, ws,
                           tab, idx, leaf_parent);
    }
    return hipGetLastError();
}

hipError_t launch_mrca(const Scheme& scm, uint32_t n, const uint32_t* counter,
                       const uint32_t* surf, uint32_t* lb, uint32_t* ub, void* workspace,
                       hipStream_t stream, LayoutHint hint) {
    const uint32_t S = scm.S;
    const uint32_t diff_log2 = scm.bits == 8 ? 3u : 0u;
    uint8_t* base = static_cast<uint8_t*>(workspace);
    uint32_t* ws = reinterpret_cast<uint32_t*>(base);
    uint64_t* ranked = reinterpret_cast<uint64_t*>(base + MrcaWorkspace::kHeader);
    const size_t ranked_bytes = ((size_t)n * 8 + 255) & ~(size_t)255;
    uint32_t* times = reinterpret_cast<uint32_t*>(base + MrcaWorkspace::kHeader + ranked_bytes);
    const size_t times_bytes = ((size_t)n * S * 4 + 255) & ~(size_t)255;
    uint8_t* sites = base + MrcaWorkspace::kHeader + ranked_bytes + times_bytes;

    hipLaunchKernelGGL(mrca_prepare_kernel, dim3(1), dim3(kPrepareThreads), 0, stream, scm, n,
                       counter, ws, hint.layout, hint.T, hint.rules);
    hipLaunchKernelGGL(mrca_annotations_kernel, dim3((n + 3) / 4), dim3(256), 0, stream, scm,
                       diff_log2, n, counter, surf, ws, ranked, times, sites, hint.rules);
    hipLaunchKernelGGL(mrca_allpairs_kernel, dim3((n + 1023) / 1024, (n + kPairRows - 1) / kPairRows),
                       dim3(256), 0, stream, n, diff_log2, ranked, ws, lb, ub);
    if (merge_pairs(S, n)) {
        const uint32_t rows = n < kMergePairRows ? n : kMergePairRows;
        hipLaunchKernelGGL(mrca_merge_pairs_kernel, dim3((n + 255) / 256, rows), dim3(256), 0,
                           stream, S, diff_log2, n, counter, surf, times, sites, ws, lb, ub);
        return hipGetLastError();
    }
    constexpr uint32_t cols = kPairTileCols * kPairColTiles;
    hipLaunchKernelGGL(mrca_general_pairs_kernel,
                       dim3((n + cols - 1) / cols, (n + kPairTileRows - 1) / kPairTileRows),
                       dim3(kPairTileCols), 0, stream, S, diff_log2, n, counter, surf, times, sites, ws, lb, ub);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Allocation-free MRCA bounds: the workspace is a static device array that
// the library holds, one copy per device (the array's name is a host-side
// stand-in, so kernels take its device address, looked up once per device
// with that device current).  Every call on a device shares its copy: calls
// that overlap on one device race.  Nothing in the workspace needs clearing
// first: the prepare kernel writes every word the later kernels read.
static __device__ __align__(256) uint8_t scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t launch_mrca_noalloc(const Scheme& scm, uint32_t n, const uint32_t* counter,
                               const uint32_t* surf, uint32_t* lb, uint32_t* ub,
                               hipStream_t stream) {
    if (n == 0 || n > kNoAllocMaxN || scm.S > 64) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            e = hipGetSymbolAddress(&g_scratch_ptr[dev], HIP_SYMBOL(scratch));
            if (e != hipSuccess) {
                g_scratch_ptr[dev] = nullptr;
                return e;
            }
        }
        ptr = g_scratch_ptr[dev];
    }
    return launch_mrca(scm, n, counter, surf, lb, ub, ptr, stream);
}

}  // namespace hsga
