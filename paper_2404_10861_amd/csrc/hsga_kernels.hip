// hsga_kernels.hip -- gfx950 kernels of the island-model GA with
// hereditary-stratigraphy surface annotations (founders, site schedule, the
// generation step, its batched form), and their launchers.  The end-of-run
// queries live in hsga_query.hip.
//
// Device state is structure-of-arrays: trait[A], the S/32 surface word
// planes [S/32][A] and, for asynchronous runs only, counter[A] (in a
// synchronous run every counter is the generation number), agent a =
// island * N + slot.  Consecutive
// lanes own consecutive agents, so every population read and write is a
// contiguous 256-byte wavefront access per plane.
#include <type_traits>

#include "hsga_device.hpp"
#include "hsga_internal.hpp"
#include "hsga_layout.hpp"

namespace hsga {

// ---------------------------------------------------------------------------
// Founders (Genome Model; Distributed Phylogenetic Tracking): trait 0,
// counter 0 (written only when the run keeps a counter plane), every site
// 0, and an empty layout.  Founders carry no
// differentia; item g is deposited by generation g's births.  With founder
// tags (Results, Clade Reconstruction Trial) the trait word is instead a
// random 16-bit identifier: the low half of the first word of Philox block
// (a, 0, 0, founder).
__global__ __launch_bounds__(256) void founders_kernel(uint32_t* __restrict__ trait,
                                                      uint32_t* __restrict__ counter,
                                                      uint32_t* __restrict__ surf, uint32_t A,
                                                      uint32_t SW, uint32_t* __restrict__ layout,
                                                      uint32_t S, uint32_t tags, uint32_t k0,
                                                      uint32_t k1) {
    const uint32_t stride = gridDim.x * blockDim.x;
    const uint32_t first = blockIdx.x * blockDim.x + threadIdx.x;
    for (uint32_t a = first; a < A; a += stride) {
        trait[a] = tags ? philox4x32_10(make_uint4(a, 0u, 0u, kFounder), k0, k1).x & 0xffffu : 0u;
        if (counter) counter[a] = 0u;
        for (uint32_t w = 0; w < SW; ++w) surf[(size_t)w * A + a] = 0u;
    }
    if (first < S) layout[first] = kEmpty;
}

hipError_t launch_founders(uint32_t* trait, uint32_t* counter, uint32_t* surf, uint32_t A,
                           uint32_t SW, uint32_t* layout, uint32_t S, bool tags, uint32_t k0,
                           uint32_t k1, hipStream_t stream) {
    uint32_t blocks = (A + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks == 0) blocks = 1;
    hipLaunchKernelGGL(founders_kernel, dim3(blocks), dim3(256), 0, stream, trait, counter, surf,
                       A, SW, layout, S, tags ? 1u : 0u, k0, k1);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Site schedule.  In a synchronous run every parent of generation T carries
// counter T, so the surface site is the same for the whole population and
// is computed once per generation (Results, Surface Algorithm Benchmark:
// synchronous simulations can cache placements for a whole
// subpopulation).  The sites of a launch batch's ingests come from the
// rule's constant-time tables, one thread per ingest, and the first
// wavefront writes the run's layout after them (lane = site, S <= 64), for
// the run-bound queries and the read calls.
__device__ __forceinline__ void run_sites(const RuleTable* rules, uint32_t kind, uint32_t S,
                                          uint32_t* sites, uint32_t* layout, uint32_t tau0,
                                          uint32_t count, uint32_t k) {
    if (k < count) sites[k] = scheme_site(rules, kind, S, tau0 + k);
    if (k < 64) {
        const uint32_t item = scheme_layout_wave(rules, kind, S, (uint64_t)tau0 + count);
        if (k < S) layout[k] = item;
    }
}

__global__ __launch_bounds__(256) void run_sites_kernel(const RuleTable* __restrict__ rules,
                                                       uint32_t kind, uint32_t S,
                                                       uint32_t* __restrict__ sites,
                                                       uint32_t* __restrict__ layout,
                                                       uint32_t tau0, uint32_t count) {
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    run_sites(rules, kind, S, sites, layout, tau0, count, k);
}

hipError_t launch_run_sites(const RuleTable* rules, uint32_t kind, uint32_t S, uint32_t* sites,
                            uint32_t* layout, uint32_t tau0, uint32_t count,
                            hipStream_t stream) {
    if (S > 64) return hipErrorInvalidValue;
    const uint32_t blocks = count > 256 ? (count + 255) / 256 : 1u;
    hipLaunchKernelGGL(run_sites_kernel, dim3(blocks), dim3(256), 0, stream, rules, kind, S,
                       sites, layout, tau0, count);
    return hipGetLastError();
}

// Sites of ingests tau0 .. tau0 + count - 1 into an asynchronous run's
// ring, one thread per ingest, from the rule's constant-time tables.
__global__ __launch_bounds__(256) void fill_site_ring_kernel(const RuleTable* __restrict__ rules,
                                                            uint32_t kind, uint32_t S,
                                                            uint32_t* __restrict__ ring,
                                                            uint32_t tau0, uint32_t count) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const uint32_t tau = tau0 + i;
    ring[tau & (kSiteRing - 1u)] = scheme_site(rules, kind, S, tau);
}

hipError_t launch_fill_site_ring(const RuleTable* rules, uint32_t kind, uint32_t S,
                                 uint32_t* ring, uint32_t tau0, uint32_t count,
                                 hipStream_t stream) {
    if (count == 0) return hipSuccess;
    if (count > kSiteRing) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fill_site_ring_kernel, dim3((count + 255) / 256), dim3(256), 0, stream,
                       rules, kind, S, ring, tau0, count);
    return hipGetLastError();
}

// A run's layout set from the host through the kernel's arguments (so no
// host buffer has to outlive the call).
struct LayoutWords {
    uint32_t w[64];
};

__global__ __launch_bounds__(64) void set_layout_kernel(uint32_t* __restrict__ layout,
                                                        LayoutWords words, uint32_t S) {
    if (threadIdx.x < S) layout[threadIdx.x] = words.w[threadIdx.x];
}

hipError_t launch_set_layout(uint32_t* layout, const uint32_t* words, uint32_t S,
                             hipStream_t stream) {
    if (S > 64) return hipErrorInvalidValue;
    LayoutWords lw{};
    for (uint32_t k = 0; k < S; ++k) lw.w[k] = words[k];
    hipLaunchKernelGGL(set_layout_kernel, dim3(1), dim3(64), 0, stream, layout, lw, S);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Generations of the step, (P_g, O_g) -> (P_{g+K}, O_{g+K}) (Methods,
// Asynchronous Island-model Genetic Algorithm), K = p.gens in one launch.
//
// One workgroup per tile of tile_w x tile_h whole islands; the tile's
// population is staged in LDS as structure-of-arrays planes and stays there
// for the launch's K generations.  A generation needs nothing of the
// neighbouring islands but the emigrants that they posted in the generation
// before, so a second generation needs, of each island around the tile, one
// birth: the emigrant's.  Only the islands whose emigrant comes the tile's
// way (a quarter of them) work it out, from P_g and O_g in memory; the
// same draws give the same child in the island's own tile.  Planes and
// outboxes are then read and written once for two generations, where one
// generation per launch was bound by that traffic.  Paper-scale run (16.8 M
// agents, two-word surfaces): 70.5 us per generation with one a launch (5.9
// TB/s, 415 VALU instructions per wavefront), 45.8 us with two (357 per
// generation, 80 % of VALU issue).  Float births with migration, and integer
// runs whose islands around a tile are many for its agents, take step_line.
//  1. Each thread issues one 16-byte (APT = 4) non-temporal load per plane
//     for its APT consecutive agents: traits and surface words, counters
//     only for asynchronous ticks (in a synchronous run every counter is the
//     generation number).  In the same round the threads issue the loads of
//     the outbox entries of the tile's islands and of those around it, the
//     islands' draws for two generations are made, one lane per draw, the
//     emigrants of the islands around are worked out, and each thread draws
//     the Philox blocks of its births.
//  2. Records and entries go to LDS; after a barrier, the thread of each
//     island copies the neighbours' emigrants addressed to it over the
//     drawn slots, north, south, west, east (a later one wins).
//  3. Each thread gives birth to its APT agents: a tournament of two over
//     the island's LDS traits, the parent record copied from LDS, trait
//     mutation, counter + 1 and the differentia bit written at this
//     generation's site.  The children replace the staged records and the
//     thread holding the island's emigrant posts its copy in LDS, or, after
//     the last generation, the children leave with one 16-byte store per
//     plane and the emigrant goes to the outbox.
// Immigration word: bits 6d .. 6d+5 = slot for direction d.  Emigration
// word: bits 0..7 = slot, 8..10 = direction (4: none, an idle island).
template <int APT>
struct Lanes {
    uint32_t v[APT];
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Population planes stream through once per launch: global accesses
// carry the non-temporal hint.  LDS accesses are APT-word aligned.
// at: the first agent (a plane's byte offsets fit 32 bits).
template <int APT>
__device__ __forceinline__ Lanes<APT> load_lanes(const uint32_t* __restrict__ plane, uint32_t at) {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(
        reinterpret_cast<const char*>(plane) + (uint32_t)(at * 4u));
    Lanes<APT> r;
    if constexpr (APT == 4) {
        const u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src));
        r.v[0] = x.x; r.v[1] = x.y; r.v[2] = x.z; r.v[3] = x.w;
    } else if constexpr (APT == 2) {
        const u32x2 x = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(src));
        r.v[0] = x.x; r.v[1] = x.y;
    } else {
        r.v[0] = __builtin_nontemporal_load(src);
    }
    return r;
}

template <int APT>
__device__ __forceinline__ void store_lanes(uint32_t* __restrict__ plane, uint32_t at,
                                            const Lanes<APT>& r) {
    uint32_t* dst = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(plane) +
                                                (uint32_t)(at * 4u));
    if constexpr (APT == 4) {
        u32x4 x = {r.v[0], r.v[1], r.v[2], r.v[3]};
        __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(dst));
    } else if constexpr (APT == 2) {
        u32x2 x = {r.v[0], r.v[1]};
        __builtin_nontemporal_store(x, reinterpret_cast<u32x2*>(dst));
    } else {
        __builtin_nontemporal_store(r.v[0], dst);
    }
}

template <int APT>
__device__ __forceinline__ void lds_store_lanes(uint32_t* dst, const Lanes<APT>& r) {
    if constexpr (APT == 4) {
        *reinterpret_cast<u32x4*>(__builtin_assume_aligned(dst, 16)) =
            u32x4{r.v[0], r.v[1], r.v[2], r.v[3]};
    } else if constexpr (APT == 2) {
        *reinterpret_cast<u32x2*>(__builtin_assume_aligned(dst, 8)) = u32x2{r.v[0], r.v[1]};
    } else {
        *dst = r.v[0];
    }
}

// n / d by d's multiplier (column_magic).
__device__ __forceinline__ uint32_t quotient_of(uint32_t n, uint32_t magic, uint32_t shift) {
    const uint32_t t = __umulhi(n, magic);
    return (t + ((n - t) >> (shift & 0xffu))) >> (shift >> 8);
}

// Island index of a neighbour: 0 north, 1 south, 2 west, 3 east (torus).
__device__ __forceinline__ uint32_t neighbour_of(uint32_t isl, uint32_t x, uint32_t d, uint32_t W,
                                                 uint32_t I) {
    if (d == 0) return isl >= W ? isl - W : isl + I - W;
    if (d == 1) return isl + W < I ? isl + W : isl + W - I;
    if (d == 2) return x > 0 ? isl - 1 : isl + W - 1;
    return x + 1 < W ? isl + 1 : isl + 1 - W;
}

// base + the set bits of a wave mask on lanes below this one.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m, uint32_t base = 0u) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
}

// This wavefront's LDS accesses so far come before its later ones.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

extern __shared__ __attribute__((aligned(16))) uint32_t g_step_lds[];

// The LDS of a tile of RI islands, in words: trait, counter (asynchronous
// ticks) and surface planes of TA words, the outbox entries of two
// generations (NE each: the tile's islands and the ring around them, or a
// whole torus), the islands' draws of `draws` generations (the
// emigration words in 16 bits), then the float births' draw queues.
struct TileLds {
    uint32_t TA, NE, obw, entries, imm, act, emig, queue;
};

__host__ __device__ inline TileLds tile_lds(uint32_t RI, uint32_t NE, uint32_t N, uint32_t SW,
                                            bool async, uint32_t draws) {
    TileLds l;
    l.TA = (RI * N + 3u) & ~3u;
    l.NE = NE;
    l.obw = async ? kOutboxWords : kSyncOutboxWords;
    l.entries = (1u + SW + (async ? 1u : 0u)) * l.TA;
    l.imm = l.entries + 2u * NE * l.obw;
    l.act = l.imm + draws * RI;
    l.emig = l.act + (async ? draws * RI : 0u);
    l.queue = (l.emig + (draws * RI + 1u) / 2u + 3u) & ~3u;
    return l;
}

// The run's key, opaque in tiles: a generation's draws then work out its
// schedule themselves (kept for all of a launch's draws it would take 20
// scalar registers; a resident run's loop keeps it).
template <bool OPAQUE>
__device__ __forceinline__ uint2 run_key(const StepParams& p) {
    uint2 k = make_uint2(p.k0, p.k1);
    if (OPAQUE) asm volatile("" : "+s"(k.x), "+s"(k.y));
    return k;
}

// The Philox blocks of K births from slot j on (and the second blocks of
// float births), computed as interleaved chains.  Their counter words
// (slot, island, generation, purpose) need no population data.
template <uint32_t BM, int K>
struct BirthDraws {
    static constexpr int NB = BM == kBirthFloat ? 2 * K : K;
    uint4 blk[NB];
    __device__ __forceinline__ void compute(uint2 key, uint32_t j, uint32_t isl, uint32_t g) {
#pragma unroll
        for (int q = 0; q < K; ++q) {
            blk[q] = make_uint4(j + q, isl, g, kBirth);
            if constexpr (BM == kBirthFloat) blk[K + q] = make_uint4(j + q, isl, g, kBirthB);
        }
        philox4x32_10_multi<NB>(blk, key.x, key.y);
    }
};

// A slot draw onto [0, N): a shift when N is a power of two above 1
// (n_shift = 32 - log2 N), which mulhi(w, N) then equals.
template <bool POW2>
__device__ __forceinline__ uint32_t pick_slot(uint32_t w, uint32_t N, uint32_t n_shift) {
    if constexpr (POW2) return w >> n_shift;
    else return word_below(w, N);
}

// Where a birth deposits: the bits of the two surface words that its
// differentia replaces (none between ingests) and their offset.
struct Deposit {
    uint32_t mask[2], shift;
};

__device__ __forceinline__ Deposit deposit_at(uint32_t site, uint32_t diff_log2) {
    const uint32_t shift = (site << diff_log2) & 31u;
    const uint32_t m = (diff_log2 ? 0xffu : 1u) << shift;
    const bool second = (site >> (5u - diff_log2)) != 0u;
    return {{second ? 0u : m, second ? m : 0u}, shift};
}

// ... of an asynchronous birth: the parent's own counter T picks the item
// and, in constant time through the rule's tables, its site.
__device__ __forceinline__ Deposit deposit_of(const StepParams& p, uint32_t T) {
    const uint32_t tau = p.interval == 1u ? T : T / p.interval;
    if (tau * p.interval != T) return {{0u, 0u}, 0u};
    return deposit_at(tau >= p.ring_lo ? p.ring[tau & (kSiteRing - 1u)]
                                       : scheme_site(p.rules, p.kind, p.S, tau),
                      p.diff_log2);
}

// Surface word w with the differentia's low bits deposited (one v_bfi_b32
// after the shift).
__device__ __forceinline__ uint32_t deposited(uint32_t word, int w, const Deposit& d,
                                              uint32_t bits) {
    return (word & ~d.mask[w]) | ((bits << d.shift) & d.mask[w]);
}

// ... of generation g of a synchronous run, whose parents all carry
// counter g: the batch's schedule.
template <class Word>
__device__ __forceinline__ Deposit scheduled_deposit(const StepParams& p, uint32_t g,
                                                     Word* sites) {
    const uint32_t tau = p.interval == 1u ? g : g / p.interval;
    if (tau * p.interval != g) return {{0u, 0u}, 0u};
    return deposit_at(sites[tau - p.tau0], p.diff_log2);
}

__device__ __forceinline__ Deposit scheduled_deposit(const StepParams& p, uint32_t g) {
    return scheduled_deposit(p, g, p.sites);
}

__device__ __forceinline__ uint32_t int_mutation(const StepParams& p, uint32_t test,
                                                 uint32_t amount) {
    return test < p.mut_thr ? (uint32_t)((int32_t)word_below(amount, p.mut_span) + p.mut_lo) : 0u;
}

// A mutating float birth: deleterious below del_thr, beneficial in the top
// ben_thr words.
__device__ __forceinline__ bool float_mutates(const StepParams& p, uint32_t class_word) {
    return class_word < p.del_thr || (p.ben_thr != 0u && class_word >= 0u - p.ben_thr);
}

// An outbox entry: direction (4: none), trait, counter (asynchronous
// ticks), surface words.
struct Emigrant {
    uint32_t dir, trait, counter, s0, s1;
};

template <bool ASYNC>
__device__ __forceinline__ void post_entry(uint32_t* o, const Emigrant& e) {
    if constexpr (!ASYNC) {
        // synchronous: always a direction below 4, counter implied
        *reinterpret_cast<uint4*>(o) = make_uint4(e.dir, e.trait, e.s0, e.s1);
    } else if (e.dir < 4u) {
        *reinterpret_cast<uint4*>(o) = make_uint4(e.dir, e.trait, e.counter, e.s0);
        *reinterpret_cast<uint4*>(o + 4) = make_uint4(e.s1, 0u, 0u, 0u);
    } else {
        *reinterpret_cast<uint4*>(o) = make_uint4(e.dir, 0u, 0u, 0u);
        *reinterpret_cast<uint4*>(o + 4) = make_uint4(0u, 0u, 0u, 0u);
    }
}

// The emigrant that an island around a tile posts in generation p.g, its
// slot and direction drawn already: that slot's (integer) birth, from P_g
// and O_g in memory.  A drawn candidate is an immigrant where the last
// arrival written to its slot says so.  load() issues everything the birth
// may need at once, so that the few lanes that work one out wait once, and
// that behind the loads of the tile and the birth draws; child() is the
// birth.
template <int SW, uint32_t BM, bool ASYNC>
struct RingBirth {
    static constexpr uint32_t OBW = ASYNC ? kOutboxWords : kSyncOutboxWords;
    static constexpr int NC = BM == kBirthIntTournament ? 2 : 1;
    uint4 en[4];                          // the neighbours' entries (SW > 1 ticks: and hi)
    uint32_t hi[4];
    uint32_t tr[NC], cn[NC], sf[NC][SW];  // the candidates' records
    uint32_t match;                       // bit 4c + d: direction d's immigrant has c's slot
    uint32_t w0, w1;                      // the birth's words r.z, r.w

    __device__ __forceinline__ void load(const StepParams& p, uint32_t isl, uint32_t x,
                                         uint32_t slot) {
        const uint32_t N = p.N;
#pragma unroll
        for (uint32_t d = 0; d < 4; ++d) {
            const uint32_t* o = p.ob_in + (size_t)neighbour_of(isl, x, d, p.W, p.I) * OBW;
            en[d] = *reinterpret_cast<const uint4*>(o);
            if (ASYNC && SW > 1) hi[d] = o[4];
        }
        uint4 b[2] = {make_uint4(slot, isl, p.g, kBirth), make_uint4(0u, isl, p.g, kImmigrate)};
        const uint2 key = run_key<true>(p);
        philox4x32_10_multi<2>(b, key.x, key.y);
        const uint32_t words[2] = {b[0].x, b[0].y};
        const uint32_t imm[4] = {word_below(b[1].x, N), word_below(b[1].y, N),
                                 word_below(b[1].z, N), word_below(b[1].w, N)};
        const size_t a0 = (size_t)isl * N;
        match = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t cand = word_below(words[c], N);
            tr[c] = p.in_trait[a0 + cand];
            if constexpr (ASYNC) cn[c] = p.in_counter[a0 + cand];
#pragma unroll
            for (int w = 0; w < SW; ++w) sf[c][w] = p.in_surf[(size_t)w * p.A + a0 + cand];
#pragma unroll
            for (uint32_t d = 0; d < 4; ++d) match |= (imm[d] == cand ? 1u : 0u) << (4 * c + d);
        }
        // before the first generation no entry was posted
        if (!p.has_inbox) match = 0;
        w0 = b[0].z;
        w1 = b[0].w;
    }

    __device__ __forceinline__ Emigrant child(const StepParams& p, uint32_t dir, Deposit dep) {
        // a neighbour delivers when its emigrant was sent our way
        uint32_t sent = 0;
#pragma unroll
        for (uint32_t d = 0; d < 4; ++d) sent |= (en[d].x == (d ^ 1u) ? 1u : 0u) << d;
        uint32_t best = 0, src = 0, T = p.g, s[SW] = {};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            // the directions whose immigrant candidate c is; the last one wins
            const uint32_t arr = (match >> (4 * c)) & sent;
            uint32_t t = tr[c];
#pragma unroll
            for (uint32_t d = 0; d < 4; ++d) {
                const uint32_t y = en[d].y;
                t = (arr >> d) & 1u ? y : t;
            }
            const bool win = c == 0 || (int32_t)t > (int32_t)best;
            best = win ? t : best;
            src = win ? arr : src;
            if constexpr (ASYNC) {
                const uint32_t n = cn[c];
                T = win ? n : T;
            }
#pragma unroll
            for (int w = 0; w < SW; ++w) {
                const uint32_t f = sf[c][w], o = s[w];
                s[w] = win ? f : o;
            }
        }
#pragma unroll
        for (uint32_t d = 0; d < 4; ++d) {
            const bool it = (src >> d) & 1u;
            const uint4 e = en[d];
            const uint32_t h = hi[d], f0 = s[0], f1 = s[SW - 1];
            if constexpr (ASYNC) T = it ? e.z : T;
            const uint32_t e0 = ASYNC ? e.w : e.z, e1 = ASYNC ? h : e.w;
            s[0] = it ? e0 : f0;
            if (SW > 1) s[SW - 1] = it ? e1 : f1;
        }
        best += int_mutation(p, w0, w1);
        if constexpr (ASYNC) dep = deposit_of(p, T);
        return {dir, best, T + 1u, deposited(s[0], 0, dep, w1),
                SW > 1 ? deposited(s[SW - 1], 1, dep, w1) : 0u};
    }
};

// The children of a thread's APT births.
template <int SW, int APT>
struct Children {
    Lanes<APT> tr, cn, sf[SW];
};

// An idle island of an asynchronous tick: the same individuals on the next.
template <int SW, int APT>
__device__ __forceinline__ void keep_agents(const uint32_t* lds, uint32_t TA, uint32_t la0,
                                            Children<SW, APT>& kid) {
#pragma unroll
    for (int q = 0; q < APT; ++q) {
        kid.tr.v[q] = lds[la0 + q];
#pragma unroll
        for (int w = 0; w < SW; ++w) kid.sf[w].v[q] = lds[(1 + w) * TA + la0 + q];
        kid.cn.v[q] = lds[(1 + SW) * TA + la0 + q];
    }
}

// The island's emigrant (its emigration word), if it is one of the thread's
// agents (slots j0 on; mine: it has any), to the entry o.  (The test of mine
// stands here: a branch around the call has cost small resident runs 5 %.)
template <int SW, int APT, bool ASYNC>
__device__ __forceinline__ void post_emigrant(uint32_t* o, bool mine, uint32_t emig, uint32_t j0,
                                              const Children<SW, APT>& kid) {
    const uint32_t qe = (emig & 0xffu) - j0;            // >= APT: another thread's
    if (!mine || qe >= (uint32_t)APT) return;
    Emigrant out{emig >> 8, kid.tr.v[0], ASYNC ? kid.cn.v[0] : 0u, kid.sf[0].v[0],
                 SW > 1 ? kid.sf[SW - 1].v[0] : 0u};
#pragma unroll
    for (int q = 1; q < APT; ++q) {
        const bool it = qe == (uint32_t)q;
        const uint32_t a = kid.tr.v[q], b = kid.sf[0].v[q], c = kid.sf[SW - 1].v[q];
        out.trait = it ? a : out.trait;
        if constexpr (ASYNC) {
            const uint32_t d = kid.cn.v[q];
            out.counter = it ? d : out.counter;
        }
        out.s0 = it ? b : out.s0;
        if (SW > 1) out.s1 = it ? c : out.s1;
    }
    post_entry<ASYNC>(o, out);
}

// The children into the planes, from agent ga on.
template <int SW, int APT, bool ASYNC>
__device__ __forceinline__ void store_children(const StepParams& p, uint32_t ga,
                                               const Children<SW, APT>& kid) {
    store_lanes<APT>(p.out_trait, ga, kid.tr);
    // a synchronous run keeps no counter plane: every counter is the generation
    if constexpr (ASYNC) store_lanes<APT>(p.out_counter, ga, kid.cn);
#pragma unroll
    for (int w = 0; w < SW; ++w) store_lanes<APT>(p.out_surf + (size_t)w * p.A, ga, kid.sf[w]);
}

// The rest of a birth once its parent (LDS agent par) is chosen: its
// surface with the differentia (the low bits of `bits`) deposited and, in
// asynchronous ticks, its counter.  Synchronous generations: every member's
// counter is the generation and dep its deposit.
template <int SW, int APT, bool ASYNC>
__device__ __forceinline__ void inherit(const StepParams& p, const uint32_t* lds, uint32_t TA,
                                        uint32_t par, uint32_t bits, Deposit dep, int q,
                                        Children<SW, APT>& kid) {
    if constexpr (ASYNC) {
        const uint32_t T = lds[(1 + SW) * TA + par];
        kid.cn.v[q] = T + 1u;
        dep = deposit_of(p, T);
    }
#pragma unroll
    for (int w = 0; w < SW; ++w)
        kid.sf[w].v[q] = deposited(lds[(1 + w) * TA + par], w, dep, bits);
}

// Integer births of this thread's APT agents.  APT divides N, so they share
// one island, whose agents start at LDS agent base.
template <int SW, uint32_t BM, int APT, bool ASYNC, bool POW2>
__device__ __forceinline__ void step_births(const StepParams& p, const uint32_t* lds, uint32_t TA,
                                            uint32_t base, const BirthDraws<BM, APT>& draws,
                                            const Deposit& dep, uint32_t n_shift,
                                            Children<SW, APT>& kid) {
    const uint32_t* l_trait = lds;
#pragma unroll
    for (int q = 0; q < APT; ++q) {
        const uint4 r = draws.blk[q];
        uint32_t par = base + pick_slot<POW2>(r.x, p.N, n_shift);
        uint32_t ptrait = l_trait[par];
        if constexpr (BM == kBirthIntTournament) {
            const uint32_t pb = base + pick_slot<POW2>(r.y, p.N, n_shift);
            const uint32_t tb = l_trait[pb];
            if ((int32_t)tb > (int32_t)ptrait) {
                par = pb;
                ptrait = tb;
            }
        }
        kid.tr.v[q] = ptrait + int_mutation(p, r.z, r.w);
        inherit<SW, APT, ASYNC>(p, lds, TA, par, r.w, dep, q, kid);
    }
}

// Float births of this thread's APT agents (slots j0 on of island isl),
// drawn and chosen two at a time: four chains are enough to overlap, and
// the blocks of all four births at once would take the registers of two
// wavefronts per SIMD.  The half-normal draws of the mutating births are
// queued in the wave's LDS area wq (64 APT entries: cosine cases from the
// front, sine cases from the back) and evaluated after all births in rounds
// of the wave's lanes, so the draw runs once per mutating birth rather than
// once per birth for the whole wave, and no round mixes the two series.
template <int SW, int APT, bool ASYNC, bool POW2, bool WHOLE, bool DRAWN = false>
__device__ __forceinline__ void step_float_births(const StepParams& p, const uint32_t* lds,
                                                  uint32_t TA, uint32_t base, uint32_t j0,
                                                  uint32_t isl, uint32_t g, const Deposit& dep,
                                                  uint32_t n_shift, uint2* wq,
                                                  Children<SW, APT>& kid,
                                                  const BirthDraws<kBirthFloat, APT>* drawn) {
    constexpr int K = DRAWN ? APT : (APT < 2 ? APT : 2);
    constexpr uint32_t QC = 64u * APT;
    const uint32_t* l_trait = lds;
    uint32_t fslot = 0, ncos = 0, nsin = 0;
    bool mutates[APT], worse[APT];
    auto enqueue = [&](int q, const uint4& v) __attribute__((always_inline)) {
        mutates[q] = float_mutates(p, v.y);
        worse[q] = v.y < p.del_thr;
        const bool sn = v.w >= 0x80000000u;              // the draw's sine case
        const uint64_t mc = __ballot(mutates[q] && !sn);
        const uint64_t ms = __ballot(mutates[q] && sn);
        if (mutates[q]) {
            const uint32_t slot = sn ? QC - 1u - lanes_below(ms, nsin) : lanes_below(mc, ncos);
            wq[slot] = make_uint2(v.z, v.w);
            fslot |= slot << (8 * q);
        }
        ncos += (uint32_t)__popcll(mc);
        nsin += (uint32_t)__popcll(ms);
    };
    const uint2 key = run_key<!WHOLE>(p);
#pragma unroll
    for (int q0 = 0; q0 < APT; q0 += K) {
        BirthDraws<kBirthFloat, K> draws;
        if constexpr (!DRAWN) draws.compute(key, j0 + q0, isl, g);
#pragma unroll
        for (int i = 0; i < K; ++i) {
            // tournament of p.tour draws (words r.x, r.y, r.z, r.w, v.x),
            // the first of maximal fitness winning; mutation class from
            // v.y, |Z| from v.z and v.w, differentia the low bits of v.w
            const int q = q0 + i;
            const uint4 r = DRAWN ? drawn->blk[q] : draws.blk[i];
            const uint4 v = DRAWN ? drawn->blk[APT + q] : draws.blk[K + i];
            uint32_t par = base + pick_slot<POW2>(r.x, p.N, n_shift);
            float best = __uint_as_float(l_trait[par]);
            const uint32_t words[4] = {r.y, r.z, r.w, v.x};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if ((uint32_t)c + 1u < p.tour) {
                    const uint32_t cb = base + pick_slot<POW2>(words[c], p.N, n_shift);
                    const float fc = __uint_as_float(l_trait[cb]);
                    if (fc > best) {
                        best = fc;
                        par = cb;
                    }
                }
            }
            kid.tr.v[q] = __float_as_uint(best);         // the draw is applied below
            inherit<SW, APT, ASYNC>(p, lds, TA, par, v.w, dep, q, kid);
            if constexpr (!DRAWN) enqueue(q, v);
        }
    }
    // (all four births' reads before the queue's first write, which would
    // hold up those after it)
    if constexpr (DRAWN) {
#pragma unroll
        for (int q = 0; q < APT; ++q) enqueue(q, drawn->blk[APT + q]);
    }
    // the queued draws in rounds of the active lanes (one wavefront: its
    // LDS writes land before its later reads), then each birth's fitness
    const uint64_t ex = __ballot(true);
    const uint32_t me = lanes_below(ex), na = (uint32_t)__popcll(ex);
    // (a resident run loads the coefficients once a generation, a draw of a
    // synchronous line tile the radius's all at once: taken as the steps come
    // to them they would be waited for four times instead of twice.  Ticks,
    // short of scalar registers, take them so)
    constexpr bool HELD = DRAWN && !ASYNC;
    const HalfNormalCoefficients kept = half_normal_coefficients();
    auto evaluate = [&](uint32_t n, auto sine) __attribute__((always_inline)) {
        constexpr bool SIN = decltype(sine)::value;
        for (uint32_t b0 = 0; b0 < n; b0 += na) {
            if (b0 + me < n) {
                const uint32_t i = SIN ? QC - 1u - (b0 + me) : b0 + me;
                const uint2 e = wq[i];
                const HalfNormalCoefficients K = WHOLE ? kept : half_normal_coefficients();
                double z;
                if constexpr (HELD) {
                    RadiusRegisters radius;
                    radius.load(K);
                    z = half_normal_radius(radius, e.x);
                }
                else z = half_normal_radius(K, e.x);
                z *= half_normal_angle<SIN>(K, e.y);
                const uint64_t zb = (uint64_t)__double_as_longlong(z);
                wq[i] = make_uint2((uint32_t)zb, (uint32_t)(zb >> 32));
            }
        }
    };
    evaluate(ncos, std::false_type{});
    evaluate(nsin, std::true_type{});
#pragma unroll
    for (int q = 0; q < APT; ++q) {
        if (mutates[q]) {
            const uint2 e = wq[(fslot >> (8 * q)) & 0xffu];
            const double z = __longlong_as_double((long long)(((uint64_t)e.y << 32) | e.x));
            kid.tr.v[q] = __float_as_uint(apply_half_normal(
                __uint_as_float(kid.tr.v[q]), worse[q] ? p.del_scale : p.ben_scale, z));
        }
    }
}

// One tile of one run.  Shared by the plain kernel (one run per launch),
// the batched kernel (many runs per launch) and the resident kernel (WHOLE:
// the tile is the whole torus, so its islands' neighbours are its own and
// any number of generations follow one another in LDS).
template <int SW, uint32_t BM, bool MIGR, int APT, bool ASYNC, bool WHOLE>
__device__ __forceinline__ void step_tile(const StepParams& p, uint32_t tile) {
    constexpr uint32_t OBW = ASYNC ? kOutboxWords : kSyncOutboxWords;
    uint32_t* lds = g_step_lds;
    const uint32_t N = p.N, W = p.W, H = p.H;
    const uint32_t TW = p.tile.w, RI = p.tile.w * p.tile.h;   // WHOLE: W and I
    const uint32_t PW = WHOLE ? W : TW + 2u;                  // entries per row
    const TileLds L = tile_lds(RI, WHOLE ? RI : PW * (p.tile.h + 2u), N, SW, ASYNC,
                              WHOLE ? p.tile.draws : kTileGens);
    const uint32_t TA = L.TA;
    uint32_t* l_trait = lds;
    uint32_t* l_surf = lds + TA;                       // SW planes of TA words
    uint32_t* l_count = lds + (1 + SW) * TA;           // asynchronous ticks only
    uint32_t* l_imm = lds + L.imm;                     // [draws][RI]
    uint32_t* l_act = lds + L.act;                     // the same, asynchronous ticks only
    uint16_t* l_emig = reinterpret_cast<uint16_t*>(lds + L.emig);   // the same
    const size_t A = p.A;
    const uint32_t t = threadIdx.x;
    const uint32_t la0 = t * APT;

    // the tile's islands: columns x0 .. x0 + vw - 1, rows y0 .. y0 + vh - 1
    uint32_t x0 = 0, y0 = 0, vw = W, vh = H;
    if constexpr (!WHOLE) {
        const uint32_t ty = quotient_of(tile, p.tile.cols_magic, p.tile.cols_shift);
        x0 = (tile - ty * p.tile.cols) * TW;
        y0 = ty * p.tile.h;
        vw = min(TW, W - x0);
        vh = min(p.tile.h, H - y0);
    }
    // this thread's island (il of the tile, isl of the run, its entry at
    // eidx) and first slot (one division: la0 < 4096)
    const uint32_t il = (la0 * p.tile.n_magic) >> 20;
    const uint32_t j0 = la0 - il * N;
    bool mine = il < RI;
    uint32_t isl = il, eidx = il;
    if constexpr (!WHOLE) {
        const uint32_t ly = (il * p.tile.w_magic) >> 20, lx = il - ly * TW;
        mine = mine && lx < vw && ly < vh;
        isl = (y0 + ly) * W + x0 + lx;
        eidx = (ly + 1u) * PW + lx + 1u;
    }
    const uint32_t ga = isl * N + j0;

    // A wave issues its loads at the highest priority and then drops back:
    // when a fresh wave arrives, its loads go out ahead of the arithmetic of
    // waves already holding data, which keeps more bytes in flight.
    __builtin_amdgcn_s_setprio(3);
    // 1. this thread's agents, every plane
    Lanes<APT> tr, ct, sf[SW];
    if (mine) {
        tr = load_lanes<APT>(p.in_trait, ga);
        // only asynchronous runs keep a counter plane: in synchronous
        // generations every agent's counter is the generation number
        // (founders 0, each birth one above a parent of the same
        // generation)
        if (ASYNC) ct = load_lanes<APT>(p.in_counter, ga);
#pragma unroll
        for (int w = 0; w < SW; ++w) sf[w] = load_lanes<APT>(p.in_surf + w * A, ga);
    }
    // Entry e of the tile's entries: the outbox of its island (the ring's
    // corners and what a ragged tile leaves out read entry 0, unused).  The
    // first round's loads are issued outside any branch (before the first
    // generation the entries are read but not used) so that nothing waits
    // for them before the birth draws.
    auto outbox_at = [&](uint32_t e) -> size_t {
        if constexpr (WHOLE) return e < RI ? (size_t)e * OBW : 0;
        const uint32_t py = quotient_of(e, p.tile.pw_magic, p.tile.pw_shift), px = e - py * PW;
        if (px > vw + 1u || py > vh + 1u) return 0;
        // the ring wraps round the torus (vw <= W: at most twice)
        uint32_t x = x0 + W - 1u + px, y = y0 + H - 1u + py;
        x -= x >= W ? W : 0u;
        x -= x >= W ? W : 0u;
        y -= y >= H ? H : 0u;
        y -= y >= H ? H : 0u;
        return ((size_t)y * W + x) * OBW;
    };
    uint4 in_lo, in_hi;
    if constexpr (MIGR) {
        // (a wave-uniform test: most wavefronts of a large tile load none)
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)t) < L.NE) {
            const uint32_t* o = p.ob_in + (t < L.NE ? outbox_at(t) : 0);
            in_lo = *reinterpret_cast<const uint4*>(o);
            if (ASYNC && SW > 1) in_hi = *reinterpret_cast<const uint4*>(o + 4);
        }
    }
    __builtin_amdgcn_s_setprio(0);

    const uint32_t n_shift = (N > 1u && (N & (N - 1u)) == 0u) ? 32u - __builtin_ctz(N) : 0u;
    // islands per wavefront, where every island's agents belong to one: its
    // LDS accesses are in order, so only the entries need a workgroup barrier
    // (a resident run, whose generations are a chain of latencies; 0: the
    // tile's last wavefronts take all its islands' immigrants, which is the
    // least work)
    const uint32_t own = WHOLE && 64u * APT % N == 0u ? 64u * APT / N : 0u;
    const bool ring = MIGR && !WHOLE && p.gens > 1u;   // the emigrants of the islands around
    BirthDraws<BM, APT> draws;
    // The islands' draws, one lane each: immigration, emigration and
    // (asynchronous ticks) activity, of two generations at once for a
    // tile's launch of two -- and, with them, the emigration draws of
    // the islands around: 44 lanes of one evaluation for a tile of 4 x 2
    // islands.  A resident run draws as many generations' at once as its
    // threads hold, after the births that read the last of those before.
    constexpr uint32_t KINDS = (MIGR ? 2u : 0u) + (ASYNC ? 1u : 0u);
    uint32_t r_isl = 0, r_x = 0, r_pos = 0, r_draw = kEmpty;   // an island around
    auto draw_islands = [&](uint32_t k) {
        const uint32_t g = p.g + k;
        const uint32_t inner = KINDS * (WHOLE ? p.tile.draws : p.gens) * RI;
        const uint32_t all = inner + (ring ? 2u * (vw + vh) : 0u);
        for (uint32_t j = t; j < all; j += blockDim.x) {
            uint32_t at = 0, gen = g, purpose, di, need = 4u;
            bool around = false;
            if (!ring || j < inner) {
                const uint32_t q = WHOLE ? quotient_of(j, p.tile.cols_magic, p.tile.cols_shift)
                                         : (j * p.tile.isl_magic) >> 20;
                const uint32_t li = j - q * RI;
                const uint32_t half = q / (KINDS ? KINDS : 1u);
                uint32_t kind = q - half * KINDS;
                gen += half;
                at = half * RI + li;
                di = li;
                if constexpr (!WHOLE) {
                    const uint32_t ly = (li * p.tile.w_magic) >> 20;
                    di = (y0 + ly) * W + x0 + li - ly * TW;
                }
                if (!MIGR) kind = 2u;
                purpose = kind == 0u ? kImmigrate : (kind == 1u ? kEmigrate : kActivity);
            } else {
                // north, south, west, east sides; an emigrant comes in
                // when it was sent the opposite way
                around = true;
                uint32_t h = j - inner, px, py;
                if (h < 2u * vw) {
                    const bool s = h >= vw;
                    px = 1u + h - (s ? vw : 0u);
                    py = s ? vh + 1u : 0u;
                    need = s ? 0u : 1u;
                } else {
                    h -= 2u * vw;
                    const bool e = h >= vh;
                    py = 1u + h - (e ? vh : 0u);
                    px = e ? vw + 1u : 0u;
                    need = e ? 2u : 3u;
                }
                uint32_t x = x0 + W - 1u + px, y = y0 + H - 1u + py;
                x -= x >= W ? W : 0u;
                x -= x >= W ? W : 0u;
                y -= y >= H ? H : 0u;
                y -= y >= H ? H : 0u;
                di = y * W + x;
                r_isl = di;
                r_x = x;
                r_pos = py * PW + px;
                purpose = kEmigrate;
            }
            const uint2 key = run_key<!WHOLE>(p);
            const uint4 w4 = philox4x32_10(make_uint4(0u, di, gen, purpose), key.x, key.y);
            const uint32_t emig = word_below(w4.x, N) | ((w4.y >> 30) << 8);
            if (around) {
                r_draw = (emig >> 8) == need ? emig : 4u << 8;
            } else if (purpose == kImmigrate) {
                l_imm[at] = word_below(w4.x, N) | (word_below(w4.y, N) << 6) |
                            (word_below(w4.z, N) << 12) | (word_below(w4.w, N) << 18);
            } else if (purpose == kEmigrate) {
                l_emig[at] = (uint16_t)emig;
            } else {
                // asynchronous ticks: an island runs a generation iff its
                // activity draw is below the threshold; an idle island
                // takes no immigrants and posts no emigrant
                l_act[at] = w4.x < p.async_thr ? 1u : 0u;
            }
        }
    };
    if constexpr (KINDS != 0) draw_islands(0);
    // the first generation's deposit
    Deposit dep{{0u, 0u}, 0u};
    if constexpr (!ASYNC) dep = scheduled_deposit(p, p.g);
    // 2. stage the tile and its entries in LDS
    if (mine) {
        lds_store_lanes<APT>(l_trait + la0, tr);
        if (ASYNC) lds_store_lanes<APT>(l_count + la0, ct);
#pragma unroll
        for (int w = 0; w < SW; ++w) lds_store_lanes<APT>(l_surf + w * TA + la0, sf[w]);
    }
    if constexpr (MIGR) {
        for (uint32_t e = t; e < L.NE; e += blockDim.x) {
            if (e != t) {
                const uint32_t* o = p.ob_in + outbox_at(e);
                in_lo = *reinterpret_cast<const uint4*>(o);
                if (ASYNC && SW > 1) in_hi = *reinterpret_cast<const uint4*>(o + 4);
            }
            uint32_t* o = lds + L.entries + e * OBW;
            *reinterpret_cast<uint4*>(o) = in_lo;
            if (ASYNC && SW > 1) *reinterpret_cast<uint4*>(o + 4) = in_hi;
        }
    }
    // the emigrants that come in from the islands around (an idle island
    // of an asynchronous tick sends none)
    RingBirth<SW, BM, ASYNC> rb;
    uint32_t r_dir = r_draw >> 8;
    if constexpr (MIGR && !WHOLE) {
        if (r_dir < 4u) {
            if constexpr (ASYNC)
                if (philox4x32_10(make_uint4(0u, r_isl, p.g, kActivity), p.k0, p.k1).x >=
                    p.async_thr)
                    r_dir = 4u;
            rb.load(p, r_isl, r_x, r_draw & 0xffu);
        }
    }
    if constexpr (MIGR && !WHOLE) {
        if (r_draw != kEmpty) {
            uint32_t* o = lds + L.entries + (L.NE + r_pos) * OBW;
            if (r_dir < 4u) post_entry<ASYNC>(o, rb.child(p, r_dir, dep));
            else o[0] = 4u;
        }
    }
    // the first generation's birth draws (float births' two blocks per agent
    // would cost a wave per SIMD here: they are drawn after the barrier)
    if constexpr (BM != kBirthFloat)
        if (mine) draws.compute(run_key<!WHOLE>(p), j0, isl, p.g);
    Children<SW, APT> kid;
    uint32_t emig = 0;
    auto advance = [&](uint32_t k) __attribute__((always_inline)) {
        const uint32_t g = p.g + k;
        __syncthreads();
        const uint32_t half = (WHOLE ? k % p.tile.draws : k) * RI;
        if constexpr (MIGR) {
            // immigrants over the drawn slots (north, south, west, east: a
            // later direction overwrites an earlier one)
            if (k > 0 || p.has_inbox) {
                // island ii is thread blockDim - 1 - ii's: a tile's last
                // wavefronts, the first ones have made the islands' draws
                // (worked out anew each generation: kept across the loop,
                // the indices would cost a wave per SIMD)
                const uint32_t wave0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
                uint32_t ii = blockDim.x - 1u - t;
                bool take = false, some = blockDim.x - 64u - wave0 < RI;
                if (own) {
                    // the islands of this wavefront's agents
                    ii = own * (wave0 >> 6) + (t & 63u);
                    some = own * (wave0 >> 6) < RI;
                }
                asm volatile("" : "+v"(ii));
                uint32_t iy = 0, ix = 0;
                if (some) {
                    iy = (ii * p.tile.w_magic) >> 20;
                    ix = ii - iy * TW;
                    take = ii < RI && ix < vw && iy < vh;
                    if (own) take = take && (t & 63u) < own;
                    if (ASYNC && take) take = l_act[half + ii] != 0u;
                }
                if (take) {
                    const uint32_t* ent = lds + L.entries + ((k & 1u) ? L.NE * OBW : 0u);
                    uint32_t n[4];
                    if constexpr (WHOLE) {
#pragma unroll
                        for (uint32_t d = 0; d < 4; ++d) n[d] = neighbour_of(ii, ix, d, W, RI);
                    } else {
                        const uint32_t c = (iy + 1u) * PW + ix + 1u;
                        n[0] = c - PW;
                        n[1] = c + PW;
                        n[2] = c - 1u;
                        n[3] = c + 1u;
                    }
                    const uint32_t slots = l_imm[half + ii];
                    // all four entries at once: read one by one, each
                    // would wait for the write before it
                    uint4 o[4];
                    uint32_t hi[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (uint32_t d = 0; d < 4; ++d) {
                        o[d] = *reinterpret_cast<const uint4*>(ent + n[d] * OBW);
                        if (ASYNC && SW > 1) hi[d] = ent[n[d] * OBW + 4u];
                    }
#pragma unroll
                    for (uint32_t d = 0; d < 4; ++d) {
                        // a neighbour delivers when its emigrant was sent our way
                        if (o[d].x == (d ^ 1u)) {
                            const uint32_t la = ii * N + ((slots >> (6u * d)) & 63u);
                            l_trait[la] = o[d].y;
                            if constexpr (ASYNC) l_count[la] = o[d].z;
                            l_surf[la] = ASYNC ? o[d].w : o[d].z;
                            if (SW > 1) l_surf[TA + la] = ASYNC ? hi[d] : o[d].w;
                        }
                    }
                }
                if (own) wave_order();
                else __syncthreads();
            }
        }

        // 3. births
        if (mine) {
            bool act = true;
            if constexpr (ASYNC) {
                act = l_act[half + il] != 0u;
                if (!act) keep_agents<SW, APT>(lds, TA, la0, kid);
            }
            if (act) {
                const uint32_t base = il * N;
                // a wave-uniform choice between two copies of the births
                if constexpr (BM == kBirthFloat) {
                    uint2* wq = reinterpret_cast<uint2*>(lds + L.queue) + (t >> 6) * (64u * APT);
                    if (n_shift)
                        step_float_births<SW, APT, ASYNC, true, WHOLE>(p, lds, TA, base, j0, isl, g, dep,
                                                                n_shift, wq, kid, nullptr);
                    else
                        step_float_births<SW, APT, ASYNC, false, WHOLE>(p, lds, TA, base, j0, isl, g, dep,
                                                                 n_shift, wq, kid, nullptr);
                } else if (n_shift) {
                    step_births<SW, BM, APT, ASYNC, true>(p, lds, TA, base, draws, dep, n_shift,
                                                          kid);
                } else {
                    step_births<SW, BM, APT, ASYNC, false>(p, lds, TA, base, draws, dep, n_shift,
                                                           kid);
                }
            }
            if constexpr (MIGR) {
                emig = l_emig[half + il];
                if (ASYNC && !act) emig = (emig & 0xffu) | (4u << 8);
            }
        }
    };
    // the children of generation k are the next one's parents (every parent
    // has been read), and the next generation's draws and deposit
    auto succeed = [&](uint32_t k) __attribute__((always_inline)) {
        if (own) wave_order();
        else __syncthreads();
        if constexpr (MIGR)
            post_emigrant<SW, APT, ASYNC>(lds + L.entries + (((k & 1u) ? 0u : L.NE) + eidx) * OBW,
                                          mine, emig, j0, kid);
        if (mine) {
            lds_store_lanes<APT>(l_trait + la0, kid.tr);
            if constexpr (ASYNC) lds_store_lanes<APT>(l_count + la0, kid.cn);
#pragma unroll
            for (int w = 0; w < SW; ++w) lds_store_lanes<APT>(l_surf + w * TA + la0, kid.sf[w]);
        }
        if constexpr (WHOLE && KINDS != 0) {
            if ((k + 1u) % p.tile.draws == 0u) {
                // over draws that other wavefronts' births may still read
                if (own) __syncthreads();
                draw_islands(k + 1u);
            }
        }
        if constexpr (!ASYNC) dep = scheduled_deposit(p, p.g + k + 1u);
        if constexpr (BM != kBirthFloat) {
            // (the slots' share of the first two rounds is worked out again:
            // kept from the generation before, it would cost registers)
            uint32_t j = j0;
            asm volatile("" : "+v"(j));
            if (mine) draws.compute(run_key<!WHOLE>(p), j, isl, p.g + k + 1u);
        }
    };
    if constexpr (WHOLE || KINDS == 0) {
        for (uint32_t k = 0;; ++k) {
            advance(k);
            if (k + 1u == p.gens) break;
            succeed(k);
        }
    } else {
        advance(0);
        if (p.gens > 1u) {
            succeed(0);
            advance(1u);
        }
    }
    if constexpr (MIGR)
        post_emigrant<SW, APT, ASYNC>(p.ob_out + (size_t)isl * OBW, mine, emig, j0, kid);
    if (mine) store_children<SW, APT, ASYNC>(p, ga, kid);
}

// The LDS of a line tile, in words: trait, surface and (asynchronous ticks)
// counter planes of TA words, an emigration word per island, then the draw
// queues.
struct LineLds {
    uint32_t TA, emig, queue;
};

__host__ __device__ inline LineLds line_lds(uint32_t islands, uint32_t N, uint32_t SW,
                                            bool async) {
    LineLds l;
    l.TA = (islands * N + 3u) & ~3u;
    l.emig = (1u + SW + (async ? 1u : 0u)) * l.TA;
    l.queue = (l.emig + islands + 3u) & ~3u;
    return l;
}

// A line tile: one generation, with migration, of p.tile.w islands in a row
// of the population (they may run over several of the torus).  An island's
// four entries go from memory to the lane that draws its slots, which writes
// the immigrants after the staging.
//
// The form of float births, whose launch is bound by VALU issue: the planes'
// second trip through memory hides behind the births, while a second
// generation's emigrants from around the tile, few lanes of a wave with a
// half-normal each, make 958 VALU instructions per wavefront and generation
// of 828 (18 M agents, tournament of five: 112.4 us per generation in
// launches of two, 105.2 here, or 112.9 and 111.9 on a card that holds a lower
// clock under this load; one-word surfaces 107.3 and 97.2; ticks of
// 8.4 M agents 71.6 and 68.4).  A run below half a million agents is bound
// by its chain of latencies instead: the arguments' cache lines are asked for
// at once, the coefficients' while the planes are on their way, and the
// schedule's word by a scalar load (96 k agents 6.28 us in launches of two,
// 5.88 here; 6.2 without those three).
template <int SW, uint32_t BM, int APT, bool ASYNC>
__device__ __forceinline__ void step_line(const StepParams& p, uint32_t tile) {
    constexpr uint32_t OBW = ASYNC ? kOutboxWords : kSyncOutboxWords;
    uint32_t* lds = g_step_lds;
    const uint32_t N = p.N, W = p.W;
    const LineLds L = line_lds(p.tile.w, N, SW, ASYNC);
    const uint32_t TA = L.TA;
    uint32_t* l_trait = lds;
    uint32_t* l_surf = lds + TA;                       // SW planes of TA words
    uint32_t* l_count = lds + (1 + SW) * TA;           // asynchronous ticks only
    uint32_t* l_emig = lds + L.emig;
    const size_t A = p.A;
    const uint32_t t = threadIdx.x;
    const uint32_t la0 = t * APT;
    const uint32_t first = tile * p.tile.w;            // the tile's islands
    const uint32_t nisl = min((uint32_t)p.tile.w, p.I - first);
    const bool mine = la0 < nisl * N;
    const uint32_t ga = first * N + la0;

    // 1. the loads, all issued before anything waits for one (as in step_tile)
    __builtin_amdgcn_s_setprio(3);
    Lanes<APT> tr, ct, sf[SW];
    if (mine) {
        tr = load_lanes<APT>(p.in_trait, ga);
        if (ASYNC) ct = load_lanes<APT>(p.in_counter, ga);
#pragma unroll
        for (int w = 0; w < SW; ++w) sf[w] = load_lanes<APT>(p.in_surf + w * A, ga);
    }
    // thread t takes island t's immigrants; lanes without one read entry 0,
    // outside any branch (before the first generation the entries are read
    // but not used).  Only wavefronts that hold an island work out indices.
    size_t e[4] = {0, 0, 0, 0};
    if ((uint32_t)__builtin_amdgcn_readfirstlane((int)t) < nisl) {
        const bool lane_isl = t < nisl;
        const uint32_t isl = first + (lane_isl ? t : 0u);
        const uint32_t x = isl - quotient_of(isl, p.tile.cols_magic, p.tile.cols_shift) * W;
#pragma unroll
        for (uint32_t d = 0; d < 4; ++d)
            e[d] = lane_isl ? (size_t)neighbour_of(isl, x, d, W, p.I) * OBW : 0;
    }
    uint4 in_lo[4];
    uint32_t in_hi[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        in_lo[d] = *reinterpret_cast<const uint4*>(p.ob_in + e[d]);
        if (ASYNC && SW > 1) in_hi[d] = p.ob_in[e[d] + 4];
    }
    __builtin_amdgcn_s_setprio(0);
    // the islands' draws, one lane each: immigration by the lane that holds
    // the island's entries, emigration by the lanes after (or, where the
    // islands take more than half of them, by the same ones)
    uint32_t imm_slots = 0;
    bool imm_take = false;
    const uint2 key = run_key<true>(p);
    auto active = [&](uint32_t isl) {
        // asynchronous ticks: an idle island takes no immigrants and posts
        // no emigrant
        if constexpr (ASYNC)
            return philox4x32_10(make_uint4(0u, isl, p.g, kActivity), key.x, key.y).x <
                   p.async_thr;
        return true;
    };
    // the half-normal's coefficients, a word of each of their cache lines,
    // while the planes are on their way: the births load them when they need them
    if constexpr (BM == kBirthFloat) {
        const HalfNormalCoefficients K = half_normal_coefficients();
        asm volatile("" ::"s"(K[0]), "s"(K[8]), "s"(K[16]), "s"(K[24]), "s"(K[30]));
    }
    auto draw_island = [&](uint32_t il, bool imm) {
        const uint32_t isl = first + il;
        const bool act = active(isl);
        const uint4 w4 = philox4x32_10(make_uint4(0u, isl, p.g, imm ? kImmigrate : kEmigrate),
                                       key.x, key.y);
        if (!imm) {
            l_emig[il] = word_below(w4.x, N) | ((act ? w4.y >> 30 : 4u) << 8);
        } else if (p.has_inbox && act) {
            imm_slots = word_below(w4.x, N) | (word_below(w4.y, N) << 6) |
                        (word_below(w4.z, N) << 12) | (word_below(w4.w, N) << 18);
            imm_take = true;
        }
    };
    // (the schedule is of an earlier launch, so a scalar load: a vector load
    // here would be waited for with the planes)
    typedef const __attribute__((address_space(4))) uint32_t Scheduled;
    Deposit dep{{0u, 0u}, 0u};
    if constexpr (!ASYNC) dep = scheduled_deposit(p, p.g, (Scheduled*)p.sites);
    if (2u * nisl <= blockDim.x) {
        if (t < 2u * nisl) draw_island(t < nisl ? t : t - nisl, t < nisl);
    } else if (t < nisl) {
        draw_island(t, true);
        draw_island(t, false);
    }
    // this thread's island and first slot (one division: la0 < 4096), and its
    // birth draws while the loads are in flight (a float birth's two blocks
    // an agent would cost a wave per SIMD here)
    auto place = [&](uint32_t la, uint32_t& il, uint32_t& j) {
        il = (la * p.tile.n_magic) >> 20;
        j = la - il * N;
    };
    uint32_t lil, j0;
    place(la0, lil, j0);
    BirthDraws<BM, APT> draws;
    if constexpr (BM != kBirthFloat)
        if (mine) draws.compute(key, j0, first + lil, p.g);
    // 2. stage the tile, then the immigrants over the drawn slots (north,
    // south, west, east: a later direction overwrites an earlier one)
    if (mine) {
        lds_store_lanes<APT>(l_trait + la0, tr);
        if (ASYNC) lds_store_lanes<APT>(l_count + la0, ct);
#pragma unroll
        for (int w = 0; w < SW; ++w) lds_store_lanes<APT>(l_surf + w * TA + la0, sf[w]);
    }
    __syncthreads();
    if (imm_take) {
#pragma unroll
        for (uint32_t d = 0; d < 4; ++d) {
            // a neighbour delivers when its emigrant was sent our way
            if (in_lo[d].x == (d ^ 1u)) {
                const uint32_t la = t * N + ((imm_slots >> (6u * d)) & 63u);
                l_trait[la] = in_lo[d].y;
                if constexpr (ASYNC) l_count[la] = in_lo[d].z;
                l_surf[la] = ASYNC ? in_lo[d].w : in_lo[d].z;
                if (SW > 1) l_surf[TA + la] = ASYNC ? in_hi[d] : in_lo[d].w;
            }
        }
    }
    __syncthreads();
    // 3. births
    if (!mine) return;
    // (the thread's place is worked out again: kept across the barriers it would
    // cost tournaments on two-word surfaces the eighth wave per SIMD, and runs
    // of 2^21 agents, just eight waves on every SIMD, a second round: 14.4 ->
    // 12.5 us per generation at four agents to an island)
    uint32_t la = la0;
    asm volatile("" : "+v"(la));
    place(la, lil, j0);
    const uint32_t isl = first + lil;
    const uint32_t emig = l_emig[lil], base = lil * N;
    Children<SW, APT> kid;
    if (ASYNC && (emig >> 8) == 4u) {
        keep_agents<SW, APT>(lds, TA, la0, kid);
    } else {
        if constexpr (BM == kBirthFloat) draws.compute(key, j0, isl, p.g);
        const uint32_t n_shift = (N > 1u && (N & (N - 1u)) == 0u) ? 32u - __builtin_ctz(N) : 0u;
        // a wave-uniform choice between two copies of the births
        if constexpr (BM == kBirthFloat) {
            uint2* wq = reinterpret_cast<uint2*>(lds + L.queue) + (t >> 6) * (64u * APT);
            if (n_shift)
                step_float_births<SW, APT, ASYNC, true, false, true>(
                    p, lds, TA, base, j0, isl, p.g, dep, n_shift, wq, kid, &draws);
            else
                step_float_births<SW, APT, ASYNC, false, false, true>(
                    p, lds, TA, base, j0, isl, p.g, dep, n_shift, wq, kid, &draws);
        } else if (n_shift) {
            step_births<SW, BM, APT, ASYNC, true>(p, lds, TA, base, draws, dep, n_shift, kid);
        } else {
            step_births<SW, BM, APT, ASYNC, false>(p, lds, TA, base, draws, dep, n_shift, kid);
        }
    }
    post_emigrant<SW, APT, ASYNC>(p.ob_out + (size_t)isl * OBW, true, emig, j0, kid);
    store_children<SW, APT, ASYNC>(p, ga, kid);
}

template <int SW, uint32_t BM, int APT, bool ASYNC>
__global__ __launch_bounds__(1024) void line_kernel(const StepParams p) {
    // a word of each cache line of the arguments, all on their way at once
    asm volatile("" ::"s"(p.in_trait), "s"(p.sites), "s"(p.tile.n_magic), "s"(p.interval));
    step_line<SW, BM, APT, ASYNC>(p, xcd_local_block(blockIdx.x, gridDim.x));
}

template <int SW, uint32_t BM, bool MIGR, int APT, bool ASYNC>
__global__ __launch_bounds__(1024) void step_kernel(const StepParams p) {
    step_tile<SW, BM, MIGR, APT, ASYNC, false>(p, xcd_local_block(blockIdx.x, gridDim.x));
}

// The resident form of a small synchronous run: its whole torus is one
// tile, and one workgroup takes it through all p.gens generations of a
// launch batch in LDS, with a workgroup barrier between generations where
// the plain form has a kernel boundary.
template <int SW, uint32_t BM, bool MIGR, int APT>
__global__ __launch_bounds__(1024) void resident_step_kernel(const StepParams p) {
    step_tile<SW, BM, MIGR, APT, false, true>(p, 0u);
}

size_t step_lds_bytes(const TileGeom& tg, uint32_t N, uint32_t SW, bool async,
                      bool float_births, uint32_t apt) {
    if (tg.line)
        return 4 * (size_t)line_lds(tg.w, N, SW, async).queue +
               (float_births ? 8 * (size_t)tg.threads * apt : 0);
    const bool whole = tg.whole != 0;
    const uint32_t RI = tg.w * tg.h;
    const TileLds l = tile_lds(RI, whole ? RI : (tg.w + 2u) * (tg.h + 2u), N, SW, async,
                               tg.draws);
    return 4 * (size_t)l.queue + (float_births ? 8 * (size_t)tg.threads * apt : 0);
}

template <int SW, uint32_t BM, bool MIGR, int APT, bool ASYNC>
static hipError_t launch_step_t(const StepParams& p, hipStream_t stream) {
    const TileGeom& tg = p.tile;
    if (p.gens == 0 || tg.w * tg.h * p.N > tg.threads * APT || tg.threads > 1024)
        return hipErrorInvalidValue;
    const size_t lds = step_lds_bytes(tg, p.N, SW, ASYNC, BM == kBirthFloat, APT);
    if (tg.whole) {
        if constexpr (ASYNC) {
            return hipErrorInvalidValue;
        } else {
            if (tg.w != p.W || tg.h != p.H) return hipErrorInvalidValue;
            hipLaunchKernelGGL((resident_step_kernel<SW, BM, MIGR, APT>), dim3(1),
                               dim3(tg.threads), lds, stream, p);
        }
    } else if (tg.line) {
        if constexpr (MIGR) {
            if (p.gens != 1 || tg.w > tg.threads) return hipErrorInvalidValue;
            hipLaunchKernelGGL((line_kernel<SW, BM, APT, ASYNC>), dim3(tile_count(tg, p.W, p.H)),
                               dim3(tg.threads), lds, stream, p);
        } else {
            return hipErrorInvalidValue;
        }
    } else if constexpr (line_only(BM, MIGR)) {
        return hipErrorInvalidValue;
    } else {
        // more generations than the emigrants around a tile reach
        if (p.gens > kTileGens && (MIGR || ASYNC)) return hipErrorInvalidValue;
        if (2u * (tg.w + tg.h) > tg.threads) return hipErrorInvalidValue;
        hipLaunchKernelGGL((step_kernel<SW, BM, MIGR, APT, ASYNC>), dim3(tile_count(tg, p.W, p.H)),
                           dim3(tg.threads), lds, stream, p);
    }
    return hipGetLastError();
}

template <int SW, uint32_t BM, bool MIGR, bool ASYNC>
static hipError_t launch_step_apt(const StepParams& p, uint32_t apt, hipStream_t stream) {
    if (apt == 4) return launch_step_t<SW, BM, MIGR, 4, ASYNC>(p, stream);
    if (apt == 2) return launch_step_t<SW, BM, MIGR, 2, ASYNC>(p, stream);
    return launch_step_t<SW, BM, MIGR, 1, ASYNC>(p, stream);
}

template <int SW, uint32_t BM, bool ASYNC>
static hipError_t launch_step_mig(const StepParams& p, bool migration, uint32_t apt,
                                  hipStream_t stream) {
    return migration ? launch_step_apt<SW, BM, true, ASYNC>(p, apt, stream)
                     : launch_step_apt<SW, BM, false, ASYNC>(p, apt, stream);
}

template <int SW, bool ASYNC>
static hipError_t launch_step_model(const StepParams& p, uint32_t birth_model, bool migration,
                                    uint32_t apt, hipStream_t stream) {
    if (birth_model == kBirthFloat)
        return launch_step_mig<SW, kBirthFloat, ASYNC>(p, migration, apt, stream);
    if (birth_model == kBirthIntTournament)
        return launch_step_mig<SW, kBirthIntTournament, ASYNC>(p, migration, apt, stream);
    return launch_step_mig<SW, kBirthIntNeutral, ASYNC>(p, migration, apt, stream);
}

template <bool ASYNC>
static hipError_t launch_step_sw(const StepParams& p, uint32_t SW, uint32_t birth_model,
                                 bool migration, uint32_t apt, hipStream_t stream) {
    if (SW == 1) return launch_step_model<1, ASYNC>(p, birth_model, migration, apt, stream);
    return launch_step_model<2, ASYNC>(p, birth_model, migration, apt, stream);
}

hipError_t launch_step(const StepParams& p, uint32_t SW, uint32_t birth_model, bool migration,
                       uint32_t agents_per_thread, hipStream_t stream) {
    if (p.async_thr)
        return launch_step_sw<true>(p, SW, birth_model, migration, agents_per_thread, stream);
    return launch_step_sw<false>(p, SW, birth_model, migration, agents_per_thread, stream);
}

// ---------------------------------------------------------------------------
// Batched forms: many runs of different sizes, surfaces, treatments and
// agents per thread in one launch, each run stepping its own tiles'
// generations of it, sharing step_tile, step_line and run_sites with the
// plain forms.
__global__ __launch_bounds__(256) void batch_sites_kernel(const BatchRun* __restrict__ runs) {
    const BatchRun& R = runs[blockIdx.y];
    const uint32_t tau0 = ingests_of(R.T0, R.interval);
    const uint32_t count = ingests_of(R.T0 + R.gens, R.interval) - tau0;
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    run_sites(R.rules, R.kind, R.S, R.sites, R.layout, tau0, count, k);
}

hipError_t launch_batch_sites(const BatchRun* runs, uint32_t nruns, uint32_t max_gens,
                              hipStream_t stream) {
    if (nruns == 0) return hipSuccess;
    const uint32_t blocks = max_gens > 256 ? (max_gens + 255) / 256 : 1u;
    hipLaunchKernelGGL(batch_sites_kernel, dim3(blocks, nruns), dim3(256), 0, stream, runs);
    return hipGetLastError();
}

template <int SW, uint32_t BM, bool MIGR, int APT, bool LINES>
__device__ __forceinline__ void step_batched(const StepParams& p, uint32_t tile) {
    if constexpr (LINES || line_only(BM, MIGR)) step_line<SW, BM, APT, false>(p, tile);
    else step_tile<SW, BM, MIGR, APT, false, false>(p, tile);
}

template <int SW, uint32_t BM, bool MIGR, bool LINES>
__device__ __forceinline__ void step_tile_apt(const StepParams& p, uint32_t tile, uint32_t apt_log2) {
    if (apt_log2 == 2) step_batched<SW, BM, MIGR, 4, LINES>(p, tile);
    else if (apt_log2 == 1) step_batched<SW, BM, MIGR, 2, LINES>(p, tile);
    else step_batched<SW, BM, MIGR, 1, LINES>(p, tile);
}

template <uint32_t BM, bool LINES>
__device__ __forceinline__ void step_tile_variant(const StepParams& p, uint32_t tile,
                                                  uint32_t variant) {
    const uint32_t apt_log2 = (variant >> 4) & 3u;
    const bool mig = LINES || ((variant >> 3) & 1u);
    if (variant & 1u) {
        if (mig) step_tile_apt<2, BM, true, LINES>(p, tile, apt_log2);
        else if constexpr (!LINES) step_tile_apt<2, BM, false, LINES>(p, tile, apt_log2);
    } else {
        if (mig) step_tile_apt<1, BM, true, LINES>(p, tile, apt_log2);
        else if constexpr (!LINES) step_tile_apt<1, BM, false, LINES>(p, tile, apt_log2);
    }
}

// WITH_FLOAT: the batch may hold float-treatment runs.  Integer-only
// batches use the instantiation without them, which needs fewer registers.
// LINES: every run steps over line tiles, one generation (a kernel of its
// own: both forms' integer births in one made 64 batched runs 7 % slower).
template <bool WITH_FLOAT, bool LINES>
__global__ __launch_bounds__(1024) void batch_step_kernel(const BatchRun* __restrict__ runs,
                                                         const uint32_t* __restrict__ xcd_tab,
                                                         uint32_t nruns, uint32_t k) {
    // Workgroup b runs on XCD x = b mod 8 as the XCD's j-th workgroup, j =
    // b / 8 (the dispatcher deals workgroups to the XCDs in turn).  Every
    // run's tiles are cut into 8 contiguous chunks, one per XCD, so
    // each XCD gets an equal share of every run: a launch of runs of
    // unequal cost per tile then finishes on all XCDs together, while torus
    // neighbours within a chunk still share an L2.  xcd_tab holds, per
    // XCD, the ascending offsets of the runs' chunks among its workgroups
    // (nruns words), then per XCD the first tile of each run's chunk.
    const uint32_t x = blockIdx.x % kXcds, j = blockIdx.x / kXcds;
    const uint32_t* __restrict__ pre = xcd_tab + x * nruns;
    // the run owning this workgroup: the number of runs whose chunk starts
    // at or before j, less one (a run with an empty chunk shares its
    // offset with the next and is passed over) -- one load per lane and a
    // ballot per 64 runs in every wavefront, with no LDS round trip or
    // barrier before the run's parameters can be fetched
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t before = 0;
    for (uint32_t b0 = 0; b0 < nruns; b0 += 64) {
        const uint32_t i = b0 + lane;
        const bool le = i < nruns && pre[i] <= j;
        before += (uint32_t)__popcll(__ballot(le));
    }
    const uint32_t lo = before - 1u;       // pre[0] = 0: at least one run
    const BatchRun& R = runs[lo];
    const uint32_t t = xcd_tab[(kXcds + x) * nruns + lo] + (j - pre[lo]);
    // (a constant where no run steps otherwise: read from the table it would
    // be one more wait before the tile's loads, 2 % of 64 batched runs)
    const uint32_t per = LINES ? 1u : WITH_FLOAT ? R.tile.draws : kTileGens;
    if (k * per >= R.gens) return;
    const uint32_t g = R.T0 + k * per;
    const uint32_t src = k & 1u, dst = src ^ 1u;
    StepParams p;
    p.in_trait = R.trait[src];
    p.in_counter = nullptr;    // batched runs are synchronous
    p.in_surf = R.surf[src];
    p.out_trait = R.trait[dst];
    p.out_counter = nullptr;
    p.out_surf = R.surf[dst];
    p.ob_in = R.outbox[src];
    p.ob_out = R.outbox[dst];
    p.sites = R.sites;
    p.tau0 = ingests_of(R.T0, R.interval);
    p.diff_log2 = R.diff_log2;
    p.W = R.W; p.H = R.H; p.N = R.N;
    p.I = R.W * R.H;
    p.A = p.I * R.N;
    p.g = g;
    p.gens = min(per, R.gens - k * per);
    p.k0 = R.k0; p.k1 = R.k1;
    p.mut_thr = R.mut_thr; p.mut_lo = R.mut_lo; p.mut_span = R.mut_span;
    const bool mig = (R.variant >> 3) & 1u;
    p.has_inbox = (mig && g > 0) ? 1u : 0u;
    p.tile = R.tile;
    p.async_thr = 0u;
    p.rules = nullptr;
    p.ring = nullptr;
    p.ring_lo = 0u;
    p.kind = R.kind;
    p.S = R.S;
    p.interval = R.interval;
    p.tour = R.tour;
    p.del_thr = R.del_thr; p.ben_thr = R.ben_thr;
    p.del_scale = -(double)R.del_sigma; p.ben_scale = R.ben_sigma;
    const uint32_t model = (R.variant >> 1) & 3u;
    if (model == kBirthIntTournament)
        step_tile_variant<kBirthIntTournament, LINES>(p, t, R.variant);
    else if (WITH_FLOAT && model == kBirthFloat)
        step_tile_variant<kBirthFloat, LINES>(p, t, R.variant);
    else
        step_tile_variant<kBirthIntNeutral, LINES>(p, t, R.variant);
}

hipError_t launch_batch_step(const BatchRun* runs, const uint32_t* xcd_tab, uint32_t nruns,
                             uint32_t total_tiles, uint32_t k, uint32_t block_threads,
                             size_t lds_bytes, bool with_float, bool lines,
                             hipStream_t stream) {
    if (nruns == 0 || total_tiles == 0) return hipSuccess;
    const auto kernel = lines        ? &batch_step_kernel<true, true>
                        : with_float ? &batch_step_kernel<true, false>
                                     : &batch_step_kernel<false, false>;
    hipLaunchKernelGGL(kernel, dim3(total_tiles), dim3(block_threads), lds_bytes, stream, runs,
                       xcd_tab, nruns, k);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Plain streaming copy (instrumentation): one 16-byte non-temporal load
// and store per thread over a grid that covers the buffer (the fastest of
// the simple copy forms on this chip, so the attainable-bandwidth figure
// is not understated).
__global__ __launch_bounds__(256) void probe_copy_kernel(const u32x4* __restrict__ src,
                                                        u32x4* __restrict__ dst, size_t n16) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n16) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

hipError_t launch_probe_copy(const void* src, void* dst, size_t bytes, hipStream_t stream) {
    const size_t n16 = bytes / 16;
    const size_t blocks = (n16 + 255) / 256;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0xffffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(probe_copy_kernel, dim3((uint32_t)blocks), dim3(256), 0, stream,
                       static_cast<const u32x4*>(src), static_cast<u32x4*>(dst), n16);
    return hipGetLastError();
}

}  // namespace hsga
