// Device side of libbyzshield (gfx950): majority vote over the r copies of each file (Eq. 3 of
// the ByzShield paper; exact and tolerant), coordinate-wise median over the f winners (Sec. 2,
// Sec. 6.1), the fused single-pass vote+median, the trimmed mean and the second phase of
// Bulyan, plus the C-ABI entry points that launch them.
//
// Work decomposition shared by all streaming kernels: one thread owns V consecutive
// coordinates (4 in the vote; in the single pass 4, or 2 or 1 for the largest networks and short
// rows; 1 in most kernels with one slot per file) and walks over all files, so every global
// load of a wave is one contiguous segment of one row (1 KiB with 16-byte loads; gfx950 global
// loads only need dword alignment).  Threads past the end of the grid redo the last vector, so
// loads and wave ballots sit in straight-line code; trailing words are done by a few threads
// of the last block or by letting the last vector overlap its neighbour.
// Per-file "copies differ" bits are reduced inside a wave with ballots (scalar registers),
// parked in lane j mod 64 for file j (one word per 64 files), and merged across waves with one
// atomicOr per file and wave that is skipped when the bits are already set.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <new>
#include <type_traits>

#include "byz_internal.h"
#include "byzshield.h"
#include "byzshield_bench.h"

// The build compiles this file once per BYZ_PART, in parallel, because the kernels are large: part
// 0 holds every entry point, the vote and the smaller Bulyan kernels, parts 1..4, 7, 14, 15 and 18 one
// group of single-pass instantiations each (byz_internal_launch_single_pass_<n>), parts 5 and 6
// the median and trimmed-mean kernels up to 81 wires (and the 121-wire median), parts 8..11,
// 14, 15 and 19..23 the larger ones, parts 12 and 13 the second phase of Bulyan on 57 to 81 and on 97
// to 137 wires, parts 16 and 17 the two-wave median and trimmed-mean kernels for f > 169, 24 and 25 the pass over their files.
// Without BYZ_PART the whole library is this one translation unit.
#ifndef BYZ_PART
#define BYZ_PART -1
#endif
#define BYZ_IN_PART(p) (BYZ_PART == -1 || BYZ_PART == (p))

namespace {

#define BYZ_HIP(call)                                \
    do {                                             \
        hipError_t e_ = (call);                      \
        if (e_ != hipSuccess) {                      \
            byz_internal_set_hip_error((int)e_);     \
            return BYZ_EDEVICE;                      \
        }                                            \
    } while (0)

#if BYZ_IN_PART(0)
thread_local int g_last_hip_error = 0;

// Optional timing of the dominant kernel: event pairs recorded around it by byz_aggregate.
struct ProfileState {
    int capacity = 0;
    int count = 0;
    hipEvent_t *start = nullptr;
    hipEvent_t *stop = nullptr;
    const char *kernel = "";  // the one the last pair stands around
};
thread_local ProfileState g_prof;
#endif

// Files a kernel of several words per thread prefetches ahead of the one it consumes, from the number
// of 16-byte loads per thread it should keep in flight.  Measured on MI355X: about 6 for f = 25
// (3-4 waves per SIMD), about 12 for f = 49 (2 waves per SIMD); more is slower.  f = 121 runs
// one word per thread (4-byte loads); f = 81 (two words per thread, 253 registers) has no room for
// more than 5.  The kernels with one slot per file run one word per thread, twenty files ahead.
constexpr int prefetch_depth(int f, int slots) {
    if (f > 81) return 5;
    const int target = f >= 49 ? 12 : 6;
    const int a = (target + slots - 1) / slots - 1;
    return a < 1 ? 1 : (a > 5 ? 5 : a);
}
// f with a generated streamed network (gen_selnet.py STREAMED_SIZES): the paper's file counts
// l^2 (MOLS, Ramanujan Case 1; 81, 121, 169 for l = 9, 11, 13) and m*s (Ramanujan Case 2)
constexpr bool has_streamed_network(int f) {
    return f == 9 || f == 15 || f == 21 || f == 25 || f == 31 || f == 35 || f == 41 || f == 49 ||
           f == 57 || f == 63 || f == 65 || f == 73 || f == 81 || f == 97 || f == 109 || f == 121 ||
           f == 137 || f == 153 || f == 169;
}
// Fewest rows the n-wire network is launched with: one more than the next smaller size holds.  Only
// the wires from there on can be spare, so only they are looked at (a test on every wire cost 4 %).
constexpr int least_rows(int n) {
    int below = n - 1;
    while (below > 0 && !has_streamed_network(below)) --below;
    return below + 1;
}
// Words per thread of the single pass: fewer for the large networks, whose keys fill the register
// file.  The kernels with one slot per file run one word per thread at every size: the sorting
// ones by far (fewer registers, more waves; 2.9 M coordinates, four words / one, us: f = 49 108 /
// 96, f = 35 75 / 67), the medians by 1-3 % (f = 49 92.4 / 89.7, f = 9 17.9 / 17.1).
constexpr int vec_for(int f) { return f <= 49 ? 4 : (f <= 81 ? 2 : 1); }
// With five or seven copies of a file in flight two words per thread
// (more waves per SIMD, 8-byte loads) measured 1-2 % faster than four (r = 7 would not fit
// the registers with four; long rows of five copies: four_words_of_five); with three copies four words are faster, but for a sort of 49 keys
// (four: 269 registers, one wave per SIMD, 409 us for 4 M coordinates; two: 377)
constexpr int vec_for_pass(int f, int r, bool trim) {
    return ((r >= 5 || (trim && f > 35)) && f <= 49) ? 2 : vec_for(f);
}
// Rows up to which the single pass runs one word per thread whatever the network, with more files
// in flight (8 ahead for three copies, 5 for five or seven) where launch_short has no room for it or
// early-majority mode rules it out: with fewer threads than fill the chip
// the walk over the files is bound by the latency of its loads.  us a call, four or two words and
// one: (25,3) d = 100003 21.6 / 18.4, 262000 23.5 / 28.0; (49,3) 131072 32.4 / 27.8; (49,7) 131072
// 51.2 / 46.0; (25,5) 20000 25.8 / 23.5, 131072 25.5 / 26.6.  Depths, us of GPU time, 4 and 3 ahead / 5 and
// 2 / 8 and 5 / 20 and 8: (25,3) d = 100003 16.6 / 16.3 / 16.1 / 15.2, (49,3) 27.1 / 26.9 / 26.7 / 25.9, (49,5)
// 34.1 / 34.4 / 34.1 / 34.2, (49,7) 42.4 / 42.6 / 42.7 / 43.2 (20 for three copies would be the better one).
// Rows that one block holds with the wider form, but not with one word per thread, keep the wider form:
// a block merges its bits with no other ((25,3) d = 1003, us of GPU time, median 14.4, one word 15.2,
// early-majority 16.0 and 18.3; (25,5) 500 17.4 and 20.5).
// Rows of five copies from which four words per thread are the faster form after all: always up to 25 files, and
// off the cache lines up to 49, where two words a thread leave more lines shared by two blocks.  us a call, two
// words / four: (25,5) 1 M 91.6 / 92.0 off lines, 1.05 M 122 / 100 off and 118 / 94 on, 2.1 M 212 / 183 and 194 / 172,
// 4 M 383 / 338 and 346 / 320; (35,5) off lines 0.7 M 84 / 90, 1.05 M 161 / 132, 2.1 M 277 / 239, 4 M 503 / 435, 6 M on
// lines 637 / 641; (49,5) off lines 1.05 M 189 / 183, 4 M 661 / 618, trimmed mean 1.1 M 197 / 208, 1.2 M 217 / 211, 4 M 663 /
// 640, 6 M on lines 876 / 887.  Early-majority mode, where three copies are read: off lines (25,5) 2.1 M 123 / 112,
// (35,5) 161 / 159, (49,5) 1.1 M 127 / 134, 2.1 M 224 / 218, 4 M 412 / 396.  But its trimmed mean keeps two words:
// (49,5) 1.1 M 129 / 148, 4 M 416 / 428, (35,5) 2.1 M 168 / 168, (25,5) 1.7 M 98 / 103, on lines 97 / 103.
[[maybe_unused]] constexpr bool four_words_of_five(int f, int64_t d, bool lines, bool early_trim) {
    return !early_trim && d >= (int64_t)15 << 16 && (f <= 25 || (f <= 49 && !lines));
}
[[maybe_unused]] constexpr int64_t short_row(int f, int r) { return f <= 25 && r == 5 ? 65536 : 131072; }
// Files ahead of the one in use in the first kernel of short calls: the depths measured above, as far as
// registers allow.
constexpr int short_pass_ahead(int f, int r) { return r == 3 ? (f <= 81 ? 20 : 8) : 5; }
constexpr int kProbe = 256;  // sampled coordinates of the probe (512: 2x slower)
constexpr int kProbeSplit = 4;  // the files are dealt out to this many groups of kProbe threads
constexpr int kProbeThreads = kProbe * kProbeSplit;
constexpr int kBlock = 256;  // threads per block of the streaming kernels (128/512/1024: slower)
constexpr int kWide = BYZ_MAX_F_WIDE;  // largest f of the vote, the median (255) and the trimmed mean
static_assert(kWide <= kBlock, "one thread per file in the deciding block");
// Which kernels of one slot per file pin their schedule (selnet_pin_on.inc).  Trimmed mean, 4 M
// coordinates, left alone / pinned: f = 49 143 / 198 us, 57 157 / 148, 81 226 / 206, 97 310 / 291,
// 137 500 / 475, 169 the same.  Median: f = 97 236 / 238, 109 266 / 268, 121 307 / 300, 137 370 / 355,
// 153 392 / 428, 169 507 / 472.
constexpr bool pins_trimmed_mean(int f) { return f >= 57; }
constexpr bool pins_median(int f) { return f >= 121 && f != 153; }
constexpr int kRowStride = 8;  // slots per file in the permuted row table (>= BYZ_MAX_R)

// ----------------------------------------------------------------------------- helpers

template <int V> struct VecT;
template <> struct VecT<1> { typedef uint32_t type; };
// Vector types that only promise dword alignment: global memory accesses of gfx950 need no
// more, so rows whose pitch is not a multiple of four words still get 16-byte loads.
template <> struct VecT<2> {
    typedef uint32_t type __attribute__((ext_vector_type(2), aligned(4)));
};
template <> struct VecT<4> {
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4)));
};

// Streaming load of V words (each input word is used exactly once: non-temporal hint).
template <int V>
__device__ __forceinline__ void load_vec(const uint32_t *p, uint32_t (&x)[V]) {
    typedef typename VecT<V>::type T;
    const T t = __builtin_nontemporal_load(reinterpret_cast<const T *>(p));
    if constexpr (V == 1) {
        x[0] = t;
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v) x[v] = t[v];
    }
}

template <int V>
__device__ __forceinline__ void store_vec(uint32_t *p, const uint32_t (&x)[V]) {
    typedef typename VecT<V>::type T;
    T t;
    if constexpr (V == 1) {
        t = x[0];
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v) t[v] = x[v];
    }
    __builtin_nontemporal_store(t, reinterpret_cast<T *>(p));
}

// OR over the V words of (a xor b): nonzero iff the two copies differ somewhere in the chunk
template <int V>
__device__ __forceinline__ uint32_t differ(const uint32_t (&a)[V], const uint32_t (&b)[V]) {
    uint32_t acc = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) acc |= a[v] ^ b[v];
    return acc;
}

// 1 iff the two chunks differ in any active lane of the wave (wave-uniform result).  One ballot
// per word, merged as scalars: each is a single vector compare that writes its lane mask.
template <int V>
__device__ __forceinline__ uint32_t wave_differ(const uint32_t (&a)[V], const uint32_t (&b)[V]) {
    uint64_t m = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) m |= __builtin_amdgcn_ballot_w64(a[v] != b[v]);
    return m != 0 ? 1u : 0u;
}

// 1 iff any active lane of the wave has a nonzero x (wave-uniform result)
__device__ __forceinline__ uint32_t wave_any(uint32_t x) {
    return __builtin_amdgcn_ballot_w64(x != 0) != 0 ? 1u : 0u;
}

// Total order on fp32 bit patterns as unsigned keys:
//   -NaN < -inf < ... < -0 < +0 < ... < +inf < +NaN
__device__ __forceinline__ uint32_t to_key(uint32_t u) {
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ uint32_t from_key(uint32_t k) {
    return k ^ ((uint32_t)((int32_t)(~k) >> 31) | 0x80000000u);
}

__device__ __forceinline__ uint32_t min3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_min3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ uint32_t max3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_max3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Bit of pair (a, b), a < b, in lexicographic numbering (0,1),(0,2),..,(1,2),..
__device__ __host__ __forceinline__ constexpr int pair_bit(int r, int a, int b) {
    return a * r - a * (a + 1) / 2 + (b - a - 1);
}

__device__ __forceinline__ bool copies_equal(uint32_t neq, int r, int a, int b) {
    if (a == b) return true;
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    return ((neq >> pair_bit(r, lo, hi)) & 1u) == 0;
}

// Eq. 3 with the implementation note of Sec. 2: the copy that appears most often; among
// equally frequent values the one held by the lowest replica index.
__device__ __forceinline__ int decide_winner(uint32_t neq, int r) {
    int best = -1, arg = 0;
    for (int a = 0; a < r; ++a) {
        int cnt = 0;
        for (int b = 0; b < r; ++b) cnt += copies_equal(neq, r, a, b) ? 1 : 0;
        if (cnt > best) { best = cnt; arg = a; }
    }
    return arg;
}

// All pair bits that involve slot a, of n slots.
__device__ __host__ __forceinline__ constexpr uint32_t pairs_of_slot(int n, int a) {
    uint32_t m = 0;
    for (int b = 0; b < n; ++b)
        if (b != a) m |= 1u << pair_bit(n, a < b ? a : b, a < b ? b : a);
    return m;
}

// Which of a file's NS slots feeds the median network on one wave's coordinates, from the pair
// bits wb the wave found there (all wave-uniform): the first slot of the largest class of slots
// that are identical on these coordinates.  Being identical on a fixed set of coordinates is an
// equivalence, so a class that holds a strict majority of the copies over all of d is inside the
// largest class here, and the chosen slot then carries the majority's values on this wave's
// coordinates whether or not it belongs to the majority elsewhere.  differs gets bit b set iff
// slot b differs from the chosen one here.
// Packed as pick | differs << 3.
__device__ __host__ __forceinline__ constexpr uint32_t local_choice_packed(int ns, uint32_t wb) {
    int pick = 0, fewest = ns;
    for (int a = 0; a < ns; ++a) {
        int n = 0;
        for (int b = 0; b < ns; ++b)
            if (b != a) n += (int)((wb >> pair_bit(ns, a < b ? a : b, a < b ? b : a)) & 1u);
        if (n < fewest) { fewest = n; pick = a; }
    }
    uint32_t differs = 0;
    for (int b = 0; b < ns; ++b)
        if (b != pick)
            differs |= ((wb >> pair_bit(ns, pick < b ? pick : b, pick < b ? b : pick)) & 1u) << b;
    return (uint32_t)pick | differs << 3;
}
static_assert(local_choice_packed(3, 0b110u) == (0u | 0b100u << 3), "{0,1},{2}: slot 0 feeds, 2 differs");
static_assert(local_choice_packed(3, 0b011u) == (1u | 0b001u << 3), "{0},{1,2}: slot 1 feeds, 0 differs");
static_assert(local_choice_packed(3, 0b111u) == (0u | 0b110u << 3), "three singletons: slot 0 feeds");
static_assert(local_choice_packed(5, 0u) == 0u, "all alike");
// The eight cases of three slots as one constant, a byte each: pick in bits 0..1, above it what
// the wave adds to the file's word in the workspace (its pair bits, then the differs bits).
__device__ __host__ __forceinline__ constexpr uint64_t local_choice_table3() {
    uint64_t t = 0;
    for (uint32_t wb = 0; wb < 8; ++wb) {
        const uint32_t p = local_choice_packed(3, wb);
        t |= (uint64_t)((p & 3u) | (wb | (p >> 3) << 3) << 2) << (8 * wb);
    }
    return t;
}
// -> the slot that feeds; word = what the wave adds to the file's word in the workspace.
template <int NS>
__device__ __forceinline__ int local_choice(uint32_t wb, uint32_t &word) {
    if constexpr (NS == 2) {
        word = wb | wb << 2;  // two unequal slots: the first feeds, the second differs from it
        return 0;
    } else if constexpr (NS == 3) {
        constexpr uint64_t kTable = local_choice_table3();
        const uint32_t e = (uint32_t)(kTable >> (8 * wb)) & 255u;
        word = e >> 2;
        return (int)(e & 3u);
    } else {
        word = wb;
        if (wb == 0) return 0;
        int pick = 0, fewest = NS;
#pragma unroll
        for (int a = 0; a < NS; ++a) {
            const int n = __builtin_popcount(wb & pairs_of_slot(NS, a));
            if (n < fewest) { fewest = n; pick = a; }
        }
        uint32_t differs = 0;
#pragma unroll
        for (int a = 0; a < NS; ++a)
            if (pick == a) {
#pragma unroll
                for (int b = 0; b < NS; ++b)
                    if (b != a) differs |= ((wb >> pair_bit(NS, a < b ? a : b, a < b ? b : a)) & 1u) << b;
            }
        word |= differs << (NS * (NS - 1) / 2);
        return pick;
    }
}

__device__ __forceinline__ uint32_t load_shared_word(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave-uniform: is any of words[0..n-1] nonzero?  Used by the gated kernels behind the single
// pass to return at once when the decision kernel did not ask for them.
__device__ __forceinline__ bool any_word_set(const uint32_t *__restrict__ words, int n) {
    const int lane = threadIdx.x & 63;
    bool any = false;
    for (int n0 = 0; n0 < n; n0 += 64) {
        const uint32_t v = n0 + lane < n ? words[n0 + lane] : 0u;
        any = any || __builtin_amdgcn_ballot_w64(v != 0) != 0;
    }
    return any;
}

// Merge a wave's per-file bits (lane j = file j) into global words, skipping the atomic when
// nothing new would be set.  A stale read only costs a redundant atomic.
__device__ __forceinline__ void merge_flags(uint32_t *words, int f, int lane, uint32_t flags) {
    if (lane < f && flags != 0) {
        const uint32_t cur = load_shared_word(&words[lane]);
        if ((cur & flags) != flags) atomicOr(&words[lane], flags);
    }
}

// ------------------------------------------------------------------- selection networks

#define BYZ_CE(i, j)                                   \
    {                                                  \
        const uint32_t a_ = k[i], b_ = k[j];           \
        k[i] = a_ < b_ ? a_ : b_;                      \
        k[j] = a_ < b_ ? b_ : a_;                      \
    }
#define BYZ_CE_LO(i, j) { k[i] = k[i] < k[j] ? k[i] : k[j]; }
#define BYZ_CE_HI(i, j) { k[j] = k[i] < k[j] ? k[j] : k[i]; }
#define BYZ_MEDIAN_WIRE(w) result = k[w];

template <int F> struct SelNet;
template <> struct SelNet<1> {
    static __device__ __forceinline__ uint32_t median(uint32_t (&k)[1]) { return k[0]; }
};
template <> struct SelNet<3> {
    static __device__ __forceinline__ uint32_t median(uint32_t (&k)[3]) {
        uint32_t result;
#include "generated/selnet_3.inc"
        return result;
    }
};
template <> struct SelNet<5> {
    static __device__ __forceinline__ uint32_t median(uint32_t (&k)[5]) {
        uint32_t result;
#include "generated/selnet_5.inc"
        return result;
    }
};
template <> struct SelNet<7> {
    static __device__ __forceinline__ uint32_t median(uint32_t (&k)[7]) {
        uint32_t result;
#include "generated/selnet_7.inc"
        return result;
    }
};

// --------------------------------------------------------------------- device workspace

struct AggWorkspace {
    // single pass: bit pair_bit(NS, p, q) set iff the copies in slots p < q of the file's
    // permuted row list differ anywhere in [0, d) (NS = slots the pass read: r, or r' when every
    // file ran in early-majority mode); above them, bit NS(NS-1)/2 + p set iff some wave fed the
    // network from a slot that differed from slot p on that wave's coordinates
    uint32_t pneq[kWide];
    uint32_t pair_neq[kWide];        // two-step path and re-vote: all pair bits, replica numbering
    // byte offsets row*ld*4 of a file's rows, probable winner's class first; in a call on short rows the
    // blocks' slots instead (short_pass_kernel)
    uint64_t perm_off[kWide * kRowStride];
    // bits 3p..3p+2: replica in slot p; bits 24..27: slots of the file that hold a copy of their
    // own (r, or r' for a file read in early-majority mode; the other slots repeat slot 0)
    uint32_t perm[kWide];
    int32_t winner_row[kWide];       // rows of the true winners (decided after the pass)
    uint32_t revote_file[kWide];     // early-majority mode: 1 for the files whose r' copies differed
    uint32_t need_median;            // 1: some file's slot 0 was not its winner -> median redone
    uint32_t need_revote;            // 1: early-majority mode met a file whose r' copies differ
    uint32_t path;                   // byz_path of the call, for byz_aggregate_path
    uint32_t slots_per_file;         // slots of every file the single pass reads: r or r'
    uint32_t pad[60];
};
static_assert(sizeof(AggWorkspace) % 256 == 0, "whole 256-byte lines");

// ------------------------------------------------------------------------------ kernels

// Clears the accumulators of one two-step aggregation (no hipMemset: callers may capture).
__global__ void reset_workspace_kernel(AggWorkspace *ws, uint32_t path) {
    const int i = threadIdx.x;
    if (i < kWide) {
        ws->pneq[i] = 0;
        ws->pair_neq[i] = 0;
    }
    if (i == 0) {
        ws->need_median = 0;
        ws->need_revote = 0;
        ws->path = path;
    }
}

// Plain copy with the same load/store flavour as the streaming kernels (16-byte non-temporal):
// a reference of known traffic for reading hardware HBM counters.
__global__ __launch_bounds__(kBlock) void calibration_copy_kernel(const uint32_t *__restrict__ src,
                                                                  uint32_t *__restrict__ dst,
                                                                  int64_t n_vec) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_vec) return;
    uint32_t x[4];
    load_vec<4>(src + i * 4, x);
    store_vec<4>(dst + i * 4, x);
}

// The single pass's memory access pattern and nothing else: every thread reads 16 bytes of
// each of n_rows rows (non-temporal loads, six in flight), XORs them, and -- if do_store --
// writes its 16 bytes (non-temporal).  Timed with and without the store it tells what a kernel
// of this shape can reach and what the output costs.
__global__ __launch_bounds__(kBlock) void calibration_read_rows_kernel(
    const uint32_t *__restrict__ X, int64_t n_vec, int64_t ld, int n_rows,
    uint32_t *__restrict__ out, int do_store) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_vec) return;
    constexpr int kRing = 6;
    const uint32_t *p = X + i * 4;
    uint32_t st[kRing][4];
#pragma unroll
    for (int u = 0; u < kRing; ++u) load_vec<4>(p + (int64_t)(u < n_rows ? u : 0) * ld, st[u]);
    uint32_t acc[4] = {0, 0, 0, 0};
    for (int k0 = 0; k0 < n_rows; k0 += kRing) {
#pragma unroll
        for (int u = 0; u < kRing; ++u) {
            const int k = k0 + u;  // the same for every thread
            if (k < n_rows) {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] ^= st[u][e];
                if (k + kRing < n_rows) load_vec<4>(p + (int64_t)(k + kRing) * ld, st[u]);
            }
        }
    }
    if (do_store != 0) {
        store_vec<4>(out + i * 4, acc);
    } else if (acc[0] == 0x5EEDu && acc[1] == 0xC0FFEEu && acc[2] == 0x12345u) {
        out[0] = acc[3];  // practically never: keeps the loads alive without a store
    }
}

__global__ void fill_u32_kernel(uint32_t *p, int n, uint32_t value) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

// Vote, decision: winners from the pair bits (thread j = file j).
__device__ __forceinline__ void decide_files(const uint32_t *pair_neq,
                                             const int32_t *__restrict__ file_rows, int f, int r,
                                             int32_t *winner_replica, int32_t *winner_row) {
    const int j = threadIdx.x;
    if (j >= f) return;
    const int a = decide_winner(load_shared_word(&pair_neq[j]), r);
    if (winner_replica != nullptr) winner_replica[j] = a;
    if (winner_row != nullptr) winner_row[j] = file_rows[j * r + a];
}

__global__ void vote_decide_kernel(const uint32_t *pair_neq, const int32_t *__restrict__ file_rows,
                                   int f, int r, int32_t *winner_replica, int32_t *winner_row) {
    decide_files(pair_neq, file_rows, f, r, winner_replica, winner_row);
}

// Replica held by slot p of a file's permuted row list (AggWorkspace::perm).
__device__ __forceinline__ int perm_slot(uint32_t packed, int p) { return (int)((packed >> (3 * p)) & 7u); }

// Bit of a file's word in AggWorkspace::pneq that says: on some wave's coordinates, the slot that
// fed the network there differed from slot p (ns = slots the pass numbered its bits by).
__device__ __forceinline__ uint32_t fed_differs_bit(int ns, int p) { return 1u << (ns * (ns - 1) / 2 + p); }

// The decision behind the single pass (one block, thread j = file j).  The pass compared every
// pair of the slots it read over all d coordinates, so its bits are the vote's pair bits up to
// the slot numbering: the true winner of every file follows by Eq. 3, whatever order the
// slots are in.  The pass's output stands iff, for every file, no wave fed the network from a slot
// that differed from the winner's on that wave's coordinates; otherwise need_median makes the
// gated median kernel redo the output from the true winners (the inputs are not compared again).
// A file read in early-majority mode has only r' slots of its own: if they are identical they
// are the majority (Sec. 2) and any of them is the winner; if not, nothing is known about the
// copies that were skipped and need_revote sends the call through the gated vote kernel.
// two_step: the call counts as a two-step one (BYZ_PATH_TWO_STEP is set as well).
__global__ void single_pass_decide_kernel(AggWorkspace *ws, const int32_t *__restrict__ file_rows,
                                          int f, int r, int32_t *winner_replica, int two_step) {
    __shared__ uint32_t s_median, s_revote;
    if (threadIdx.x == 0) { s_median = 0; s_revote = 0; }
    __syncthreads();
    const int j = threadIdx.x;
    if (j < f) {
        const uint32_t pn = load_shared_word(&ws->pneq[j]);
        const uint32_t packed = ws->perm[j];
        const int own = (int)(packed >> 24);       // slots with a copy of their own
        const int ns = (int)ws->slots_per_file;    // slots the pass read and numbered its bits by
        if (own == r) {
            uint32_t neq = 0;
            for (int p = 0; p < r; ++p)
                for (int q = p + 1; q < r; ++q)
                    if ((pn >> pair_bit(ns, p, q)) & 1u) {
                        const int a = perm_slot(packed, p), b = perm_slot(packed, q);
                        neq |= 1u << pair_bit(r, a < b ? a : b, a < b ? b : a);
                    }
            const int w = decide_winner(neq, r);
            if (winner_replica != nullptr) winner_replica[j] = w;
            ws->winner_row[j] = file_rows[j * r + w];
            for (int p = 0; p < r; ++p)
                if (perm_slot(packed, p) == w && (pn & fed_differs_bit(ns, p)) != 0) s_median = 1;
        } else {
            uint32_t differ_bits = 0;
            for (int p = 0; p < own; ++p)
                for (int q = p + 1; q < own; ++q) differ_bits |= (pn >> pair_bit(ns, p, q)) & 1u;
            const int w = perm_slot(packed, 0);
            if (winner_replica != nullptr) winner_replica[j] = w;
            ws->winner_row[j] = file_rows[j * r + w];
            if (differ_bits != 0) s_revote = 1;
            ws->revote_file[j] = differ_bits;
        }
        if (own == r) ws->revote_file[j] = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        ws->need_median = s_median;
        ws->need_revote = s_revote;
        ws->path = (two_step != 0 ? (uint32_t)BYZ_PATH_TWO_STEP : 0u) |
                   (s_median != 0 ? (uint32_t)BYZ_PATH_MEDIAN_REDONE : 0u) |
                   (s_revote != 0 ? (uint32_t)BYZ_PATH_REVOTED : 0u);
    }
}

// Early-majority mode only, after the gated vote kernel: if the decision above asked for a
// re-vote, the winners of the files it named come from the pair bits that kernel collected
// for them, and the median is redone unless, for each of those files, the winner's copy was
// among the slots the pass read and no wave fed the network from a slot that differed from it.
__global__ void revote_decide_kernel(AggWorkspace *ws, const int32_t *__restrict__ file_rows, int f,
                                     int r, int32_t *winner_replica) {
    if (ws->need_revote == 0) return;
    __shared__ uint32_t s_median;
    if (threadIdx.x == 0) s_median = 0;
    __syncthreads();
    const int j = threadIdx.x;
    if (j < f && ws->revote_file[j] != 0) {  // the other files keep the winners decided above
        const uint32_t neq = load_shared_word(&ws->pair_neq[j]);
        const int a = decide_winner(neq, r);
        if (winner_replica != nullptr) winner_replica[j] = a;
        ws->winner_row[j] = file_rows[j * r + a];
        const uint32_t pn = load_shared_word(&ws->pneq[j]);
        const uint32_t packed = ws->perm[j];
        const int own = (int)(packed >> 24), ns = (int)ws->slots_per_file;
        bool stands = false;
        for (int p = 0; p < own; ++p)
            if (perm_slot(packed, p) == a && (pn & fed_differs_bit(ns, p)) == 0) stands = true;
        if (!stands) s_median = 1;
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_median != 0) {
        ws->need_median = 1;
        ws->path = (uint32_t)BYZ_PATH_REVOTED | (uint32_t)BYZ_PATH_MEDIAN_REDONE;
    }
}

// Vote, comparison: for every file, which pairs of copies differ anywhere in [0, d).  Threads own
// vectors of V words; the d % V trailing words go to the first threads of the last block.
// If `gate` is given, the kernel only runs when one of gate[0..gate_n-1] is nonzero; if
// `only_files` is given, only the files j with only_files[j] != 0 are read and compared.
template <int R, int V>
__global__ __launch_bounds__(kBlock) void vote_pairs_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ file_rows,
    int f, int files_per_block, uint32_t *pair_neq, const uint32_t *__restrict__ gate, int gate_n,
    const uint32_t *__restrict__ only_files) {
    if (gate != nullptr && !any_word_set(gate, gate_n)) return;
    const int lane = threadIdx.x & 63;
    const int64_t n_vec = d / V;
    const int64_t gt = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int j_begin = blockIdx.y * files_per_block;
    const int j_end = j_begin + files_per_block < f ? j_begin + files_per_block : f;
    if (n_vec > 0) {
        // threads past the end redo the last vector: no branches around loads and ballots
        const uint32_t *base = X + (gt < n_vec ? gt : n_vec - 1) * V;
        // files in groups of 64: lane j - j0 collects the bits of file j
        for (int j0 = j_begin; j0 < j_end; j0 += 64) {
            const int j1 = j0 + 64 < j_end ? j0 + 64 : j_end;
            uint32_t flags = 0;
            for (int j = j0; j < j1; ++j) {
                if (only_files != nullptr && only_files[j] == 0) continue;  // the same for every thread
                uint32_t x[R][V];
#pragma unroll
                for (int k = 0; k < R; ++k)
                    load_vec<V>(base + (int64_t)file_rows[j * R + k] * ld, x[k]);
                uint32_t wb = 0;
#pragma unroll
                for (int a = 0; a < R; ++a)
#pragma unroll
                    for (int b = a + 1; b < R; ++b)
                        wb |= wave_any(differ<V>(x[a], x[b])) << pair_bit(R, a, b);
                if (lane == j - j0) flags |= wb;
            }
            merge_flags(pair_neq + j0, j1 - j0, lane, flags);
        }
    }
    const int tail = (int)(d - n_vec * V);
    if (blockIdx.x == gridDim.x - 1 && (int)threadIdx.x < tail) {
        const int64_t c = n_vec * V + threadIdx.x;
        for (int j = j_begin; j < j_end; ++j) {
            if (only_files != nullptr && only_files[j] == 0) continue;
            uint32_t x[R];
#pragma unroll
            for (int k = 0; k < R; ++k) x[k] = X[(int64_t)file_rows[j * R + k] * ld + c];
            uint32_t bits = 0;
#pragma unroll
            for (int a = 0; a < R; ++a)
#pragma unroll
                for (int b = a + 1; b < R; ++b)
                    bits |= (x[a] != x[b] ? 1u : 0u) << pair_bit(R, a, b);
            if (bits != 0) atomicOr(&pair_neq[j], bits);
        }
    }
}

// Nonzero iff some word of the two chunks is not close: bit patterns differ and
// |a - b| > atol + rtol * max(|a|, |b|) (or the test involves a NaN).  Every operation is
// rounded to fp32 on its own (no fused multiply-add), as the CPU reference does.
template <int V>
__device__ __forceinline__ uint32_t far_apart(const uint32_t (&a)[V], const uint32_t (&b)[V],
                                              float atol, float rtol) {
    uint32_t acc = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const float x = __uint_as_float(a[v]), y = __uint_as_float(b[v]);
        const float diff = fabsf(__fsub_rn(x, y));
        const float bound = __fadd_rn(atol, __fmul_rn(rtol, fmaxf(fabsf(x), fabsf(y))));
        acc |= (a[v] != b[v] && !(diff <= bound)) ? 1u : 0u;
    }
    return acc;
}

// The same for a whole wave, all lanes active: is some word of some lane far apart?  The five operations of the
// bound are all a pair of close chunks takes: bit patterns are looked at only where a bound was missed (they
// excuse only copies that are both infinite or NaN).
template <int V>
__device__ __forceinline__ uint32_t wave_far_apart(const uint32_t (&a)[V], const uint32_t (&b)[V], float atol,
                                                   float rtol) {
    uint64_t missed[V], any = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const float x = __uint_as_float(a[v]), y = __uint_as_float(b[v]);
        const float diff = fabsf(__fsub_rn(x, y));
        const float bound = __fadd_rn(atol, __fmul_rn(rtol, fmaxf(fabsf(x), fabsf(y))));
        missed[v] = __builtin_amdgcn_ballot_w64(!(diff <= bound));
        any |= missed[v];
    }
    if (any == 0) return 0;
    any = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) any |= missed[v] & __builtin_amdgcn_ballot_w64(a[v] != b[v]);
    return any != 0 ? 1u : 0u;
}

// Tolerant variant of the vote's comparison (Sec. 2: rounding differences between honest copies can be
// handled by clustering the copies): for every file, which pairs of copies are not close
// somewhere in [0, d).  Same decomposition as vote_pairs_kernel.
template <int R, int V>
__global__ __launch_bounds__(kBlock) void vote_pairs_tolerant_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ file_rows,
    int f, int files_per_block, float atol, float rtol, uint32_t *pair_far) {
    const int lane = threadIdx.x & 63;
    const int64_t n_vec = d / V;
    const int64_t gt = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int j_begin = blockIdx.y * files_per_block;
    const int j_end = j_begin + files_per_block < f ? j_begin + files_per_block : f;
    if (n_vec > 0) {
        const uint32_t *base = X + (gt < n_vec ? gt : n_vec - 1) * V;
        for (int j0 = j_begin; j0 < j_end; j0 += 64) {
            const int j1 = j0 + 64 < j_end ? j0 + 64 : j_end;
            uint32_t flags = 0;
            for (int j = j0; j < j1; ++j) {
                uint32_t x[R][V];
#pragma unroll
                for (int k = 0; k < R; ++k)
                    load_vec<V>(base + (int64_t)file_rows[j * R + k] * ld, x[k]);
                uint32_t wb = 0;
#pragma unroll
                for (int a = 0; a < R; ++a)
#pragma unroll
                    for (int b = a + 1; b < R; ++b)
                        wb |= wave_far_apart<V>(x[a], x[b], atol, rtol) << pair_bit(R, a, b);
                if (lane == j - j0) flags |= wb;
            }
            merge_flags(pair_far + j0, j1 - j0, lane, flags);
        }
    }
    const int tail = (int)(d - n_vec * V);
    if (blockIdx.x == gridDim.x - 1 && (int)threadIdx.x < tail) {
        const int64_t c = n_vec * V + threadIdx.x;
        for (int j = j_begin; j < j_end; ++j) {
            uint32_t x[R][1];
#pragma unroll
            for (int k = 0; k < R; ++k) x[k][0] = X[(int64_t)file_rows[j * R + k] * ld + c];
            uint32_t bits = 0;
#pragma unroll
            for (int a = 0; a < R; ++a)
#pragma unroll
                for (int b = a + 1; b < R; ++b)
                    bits |= far_apart<1>(x[a], x[b], atol, rtol) << pair_bit(R, a, b);
            if (bits != 0) atomicOr(&pair_far[j], bits);
        }
    }
}

// Steps of the generated streamed programs (selnet_stream_<f>.inc), written against local names
// of the kernel that includes them: NS slots per file, V words per thread, kAhead, stage, key,
// o, lane, flags (one word per 64 files), and BYZ_S_ROW_ADDR(j, k) = address of this thread's vector in
// slot k of file j.
// Hook a kernel may redefine around the include: BYZ_S_KEY(j, x) = key of word x of file j.
// BYZ_S_STEP(j) opens file j's share of the program and BYZ_S_PIN(w) follows the comparators of
// a share for every wire they changed; both do nothing unless a kernel redefines them.
#define BYZ_S_KEY(j, x) to_key(x)
#define BYZ_S_STEP(j)
#define BYZ_S_PIN(w)
// An empty statement the compiler may not execute speculatively: keeps the one-lane update of a
// file's pair bits a real branch, and with it the file boundaries of the program (left as one
// straight-line block, the compiler keeps every ballot alive to the end and runs out of
// registers).
#define BYZ_S_KEEP_BRANCH asm volatile("" ::: "memory");
#define BYZ_S_LOAD_(j)                                                                        \
    _Pragma("unroll") for (int k_ = 0; k_ < NS; ++k_)                                         \
        load_vec<V>(reinterpret_cast<const uint32_t *>(BYZ_S_ROW_ADDR(j, k_)),                \
                    stage[(j) % (kAhead + 1)][k_]);
#define BYZ_S_LOAD1(j) if constexpr (kAhead == 1) { BYZ_S_LOAD_(j) }
#define BYZ_S_LOAD2(j) if constexpr (kAhead == 2) { BYZ_S_LOAD_(j) }
#define BYZ_S_LOAD3(j) if constexpr (kAhead == 3) { BYZ_S_LOAD_(j) }
#define BYZ_S_LOAD4(j) if constexpr (kAhead == 4) { BYZ_S_LOAD_(j) }
#define BYZ_S_LOAD5(j) if constexpr (kAhead == 5) { BYZ_S_LOAD_(j) }
#define BYZ_S_LOAD8(j) if constexpr (kAhead == 8) { BYZ_S_LOAD_(j) }
#define BYZ_S_LOAD20(j) if constexpr (kAhead == 20) { BYZ_S_LOAD_(j) }
#define BYZ_S_USE(j)                                                                          \
    {                                                                                         \
        [[maybe_unused]] int pick_ = 0;                                                       \
        if constexpr (NS > 1) {                                                               \
        uint32_t wb_ = 0, word_ = 0;                                                          \
        _Pragma("unroll") for (int a_ = 0; a_ < NS; ++a_)                                     \
        _Pragma("unroll") for (int b_ = a_ + 1; b_ < NS; ++b_)                                \
            wb_ |= wave_differ<V>(stage[(j) % (kAhead + 1)][a_],                              \
                                  stage[(j) % (kAhead + 1)][b_]) << pair_bit(NS, a_, b_);     \
        pick_ = local_choice<NS>(wb_, word_);                                                 \
        if (lane == ((j) & 63)) {                                                             \
            flags[(j) >> 6] |= word_;                                                         \
            BYZ_S_KEEP_BRANCH                                                                 \
        }                                                                                     \
        }                                                                                     \
        _Pragma("unroll") for (int v_ = 0; v_ < V; ++v_)                                      \
            key[v_][j] = BYZ_S_KEY(j, stage[(j) % (kAhead + 1)][0][v_]);                      \
        if constexpr (NS > 1) {                                                               \
        /* wave-uniform and rare: slot 0 is outside the largest class of this wave */         \
        if (__builtin_expect(pick_ != 0, 0)) {                                                \
            _Pragma("unroll") for (int v_ = 0; v_ < V; ++v_) {                                \
                uint32_t x_ = stage[(j) % (kAhead + 1)][1][v_];                               \
                _Pragma("unroll") for (int k_ = 2; k_ < NS; ++k_)                             \
                    x_ = pick_ == k_ ? stage[(j) % (kAhead + 1)][k_][v_] : x_;                \
                key[v_][j] = BYZ_S_KEY(j, x_);                                                \
            }                                                                                 \
            BYZ_S_KEEP_BRANCH                                                                 \
        }                                                                                     \
        }                                                                                     \
    }
#define BYZ_S_CE(i, j)                                                                        \
    _Pragma("unroll") for (int v_ = 0; v_ < V; ++v_) {                                        \
        const uint32_t a_ = key[v_][i], b_ = key[v_][j];                                      \
        key[v_][i] = a_ < b_ ? a_ : b_;                                                       \
        key[v_][j] = a_ < b_ ? b_ : a_;                                                       \
    }
#define BYZ_S_CE_LO(i, j)                                                                     \
    _Pragma("unroll") for (int v_ = 0; v_ < V; ++v_)                                          \
        key[v_][i] = key[v_][i] < key[v_][j] ? key[v_][i] : key[v_][j];
#define BYZ_S_CE_HI(i, j)                                                                     \
    _Pragma("unroll") for (int v_ = 0; v_ < V; ++v_)                                          \
        key[v_][j] = key[v_][i] < key[v_][j] ? key[v_][j] : key[v_][i];
// Three wires in order with the three-operand instructions, only the outputs that are needed (the
// compiler finds v_med3 and v_min3 in nested minima only where no intermediate value is shared)
#define BYZ_S_SORT3(i, j, k, lo, mid, hi)                                                     \
    _Pragma("unroll") for (int v_ = 0; v_ < V; ++v_) {                                        \
        const uint32_t a_ = key[v_][i], b_ = key[v_][j], c_ = key[v_][k];                     \
        if constexpr (lo) key[v_][i] = min3_u32(a_, b_, c_);                                  \
        if constexpr (mid) key[v_][j] = med3_u32(a_, b_, c_);                                 \
        if constexpr (hi) key[v_][k] = max3_u32(a_, b_, c_);                                  \
    }
#define BYZ_S_SORTED(n)  // wires 0..n-1 now hold the keys in ascending order
#define BYZ_S_MEDIAN(w)                                                                       \
    _Pragma("unroll") for (int v_ = 0; v_ < V; ++v_) o[v_] = from_key(key[v_][w]);

// Order of the blocks for rows that do not start on cache lines: neighbouring blocks share a line of
// every row, and blocks go to the eight XCDs round-robin, so each XCD gets `group` neighbours at a
// time.
__device__ __forceinline__ unsigned neighbours_together(unsigned b, unsigned n_blocks, unsigned group) {
    const unsigned r = b % (8 * group);
    return b - r + 8 * group <= n_blocks ? b - r + (r % 8) * group + r / 8 : b;
}

// Coordinate-wise median of F rows (fewer than the streamed networks start at) by a register
// selection network, V words per thread.
template <int F, int V>
__global__ __launch_bounds__(kBlock) void median_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ row_index,
    uint32_t *__restrict__ out, const uint32_t *__restrict__ gate, int gate_n) {
    if (gate != nullptr && !any_word_set(gate, gate_n)) return;
    const int64_t n_vec = d / V;
    const int64_t gt = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (gt < n_vec) {
        uint32_t key[V][F];
        uint32_t o[V];
        const uint32_t *base = X + gt * V;
#pragma unroll
        for (int j = 0; j < F; ++j) {
            uint32_t x[V];
            load_vec<V>(base + (int64_t)row_index[j] * ld, x);
#pragma unroll
            for (int v = 0; v < V; ++v) key[v][j] = to_key(x[v]);
        }
#pragma unroll
        for (int v = 0; v < V; ++v) o[v] = from_key(SelNet<F>::median(key[v]));
        store_vec<V>(out + gt * V, o);
    }
    const int tail = (int)(d - n_vec * V);
    if (blockIdx.x == gridDim.x - 1 && (int)threadIdx.x < tail) {
        const int64_t c = n_vec * V + threadIdx.x;
        uint32_t key[F];
#pragma unroll
        for (int j = 0; j < F; ++j) key[j] = to_key(X[(int64_t)row_index[j] * ld + c]);
        out[c] = from_key(SelNet<F>::median(key));
    }
}

// Coordinate-wise median by the streamed program of the generated network on F wires, one word per
// thread: exactly F rows or, with PAD, any odd least_rows(F) <= f <= F --
// the F - f spare wires reload row_index[0] and are tied half to the smallest and half to the
// largest key, which leaves the median where it was.  Within 4 % of the time its bytes take up to
// F = 153 (4 M coordinates at 6.5 TB/s and measured, us: f = 81 202 and 196, 109 271 and 266, 137 340 and
// 355, 153 379 and 392), bound by min/max issue at 169 (419 and 472; with two-wire comparators and
// fewer sizes 153 took 655 and 169 577).
// (V = 4: thread t owns the words from min(4t, d - 4), the last vector overlaps its neighbour; d >= 4)
// group: see neighbours_together; 0 = plain order.
template <int F, int V, bool PAD>
__global__ __launch_bounds__(kBlock) void median_large_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ row_index,
    int f, unsigned group, uint32_t *__restrict__ out, const uint32_t *__restrict__ gate, int gate_n) {
    if (gate != nullptr && !any_word_set(gate, gate_n)) return;
    const int pad_low_end = f + (F - f) / 2;  // wires [f, pad_low_end) smallest key, rest largest
    (void)pad_low_end;
    const unsigned tile = group != 0 ? neighbours_together(blockIdx.x, gridDim.x, group) : blockIdx.x;
    const int64_t gt = (int64_t)tile * kBlock + threadIdx.x;
    if (gt >= (d + V - 1) / V) return;
    const int64_t c0 = gt * V + V <= d ? gt * V : d - V;
    // one word per thread: twenty files ahead (as measured best at F = 121)
    constexpr int NS = 1, kAhead = V == 1 ? 20 : prefetch_depth(F, NS);
    uint32_t key[V][F];
    uint32_t o[V];
    const uint32_t voff = (uint32_t)(c0 * 4);
    const char *Xb = reinterpret_cast<const char *>(X);
    uint32_t stage[kAhead + 1][NS][V];
    const int lane = 0;
    uint32_t flags[(F + 63) / 64] = {};
    (void)lane; (void)flags;
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) \
    (!PAD || (j) < least_rows(F) || (j) < f ? to_key(x) : ((j) < pad_low_end ? 0u : 0xFFFFFFFFu))
#define BYZ_S_ROW_ADDR(j, k) \
    (Xb + (uint64_t)(uint32_t)row_index[!PAD || (j) < least_rows(F) || (j) < f ? (j) : 0] * (uint64_t)ld * 4u + voff)
    if constexpr (pins_median(F)) {
#include "selnet_pin_on.inc"
#include "generated/selnet_stream_dispatch.inc"
#include "selnet_pin_off.inc"
    } else {
#include "generated/selnet_stream_dispatch.inc"
    }
#undef BYZ_S_ROW_ADDR
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) to_key(x)
    store_vec<V>(out + c0, o);
}

// The median of two sorted halves of F keys, the wave of wires 0..F-1 and that of F..2F-1 (see
// median_halves_kernel): out[c] of lane ln.
template <int F>
__device__ __forceinline__ void median_of_halves(const uint32_t (&k)[F], uint32_t *s_half, int first, int ln,
                                                 int64_t c, int64_t d, uint32_t *__restrict__ out) {
    if (first != 0) {
#pragma unroll
        for (int m = 0; m < F; ++m) s_half[m * 64 + ln] = k[m];
    }
    __syncthreads();
    if (first == 0) {
        uint32_t best = k[F - 1] < s_half[(F - 1) * 64 + ln] ? k[F - 1] : s_half[(F - 1) * 64 + ln];
#pragma unroll
        for (int m = 0; m < F - 1; ++m) {
            const uint32_t b = s_half[(F - 2 - m) * 64 + ln];
            const uint32_t t = k[m] > b ? k[m] : b;
            best = best < t ? best : t;
        }
        if (c < d) out[c] = from_key(best);
    }
}

// Coordinate-wise median of H < f <= 2H - 1 rows (H = 96, 112, 128: up to 255 rows), two waves per
// 64 coordinates: wave h of a block sorts wires [hH, hH + H) of its coordinates in registers
// (H-wire sorting network, one word per thread), wave 1 hands its sorted keys over through LDS,
// and wave 0 takes rank H - 1 of the union of the two sorted halves A and B as
//     min( B[H-1], A[H-1], min over m = 0..H-2 of max(A[m], B[H-2-m]) )
// (the H smallest of the union are the i smallest of A and the H - i smallest of B for some i;
// the largest of those is max(A[i-1], B[H-1-i]), and the right i minimises it).  The 2H - f
// spare wires sit at the end of half B, H - 1 - (f-1)/2 of them with the smallest key and the
// rest with the largest, which puts the median of the f values at rank H - 1.  Half the
// registers of one network over all rows, so two or three waves per SIMD instead of one and no
// spills; the schedule is not pinned (pinned as in the single pass it was 14 % slower).
// The waves-per-SIMD attribute states what the registers allow anyway; without it the compiler
// schedules the H = 128 kernel half as fast (4.7 instead of 3.0 ms on 11.2 M coordinates).
// GROUP: see neighbours_together; 0 = plain order (a constant: as an argument it costs 7-16 % on the lines).
template <int F, unsigned GROUP>  // F = H
__global__ __launch_bounds__(128)
__attribute__((amdgpu_waves_per_eu(F <= 96 ? 3 : 2, F <= 96 ? 3 : 2)))
void median_halves_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ row_index,
    int f, uint32_t *__restrict__ out, const uint32_t *__restrict__ gate, int gate_n) {
    if (gate != nullptr && !any_word_set(gate, gate_n)) return;
    __shared__ uint32_t s_half[F * 64];
    const int ln = threadIdx.x & 63;
    const int first = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * F;  // first wire of this wave
    int64_t c;
    if constexpr (GROUP != 0)
        c = (int64_t)neighbours_together(blockIdx.x, gridDim.x, GROUP) * 64 + ln;
    else
        c = (int64_t)blockIdx.x * 64 + ln;
    const int64_t cc = c < d ? c : d - 1;  // lanes past the end redo the last coordinate
    const int pad_low_end = f + (F - 1 - (f - 1) / 2);
    constexpr int V = 1, NS = 1, kAhead = 20;
    uint32_t key[V][F];
    const uint32_t voff = (uint32_t)(cc * 4);
    const char *Xb = reinterpret_cast<const char *>(X);
    uint32_t stage[kAhead + 1][NS][V];
    const int lane = 0;
    uint32_t flags[(F + 63) / 64] = {};
    (void)lane; (void)flags;
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) \
    (first + (j) < f ? to_key(x) : (first + (j) < pad_low_end ? 0u : 0xFFFFFFFFu))
#define BYZ_S_ROW_ADDR(j, k) \
    (Xb + (uint64_t)(uint32_t)row_index[first + (j) < f ? first + (j) : 0] * (uint64_t)ld * 4u + voff)
#include "generated/selnet_sort_stream_dispatch.inc"
#undef BYZ_S_ROW_ADDR
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) to_key(x)
    median_of_halves<F>(key[0], s_half, first, ln, c, d, out);
}

// Rounding contract of the trimmed mean: fp32, the kept values (ranks b .. F-b-1 of the sorted
// keys) are added one by one in ascending order starting from +0, then one IEEE division.
template <int F, int V, bool RUNS = false>
__device__ __forceinline__ void trimmed_mean_of_sorted(const uint32_t (&key)[V][F], int f, int b,
                                                       uint32_t (&o)[V]) {
    // wires 0..f-1 hold the f values in ascending order (f = F unless the network is padded)
    const float denom = (float)(f - 2 * b);
    if constexpr (RUNS) {
        // b and f are wave-uniform: runs of eight ranks that lie wholly inside [b, f - b) are
        // added without a test, runs wholly outside are skipped (for the kernels whose
        // schedule is pinned; the others lose registers to it)
        float acc[V];
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = 0.0f;
#pragma unroll
        for (int i0 = 0; i0 < F; i0 += 8) {
            const int lo = i0, hi = (i0 + 8 < F ? i0 + 8 : F) - 1;
            if (lo >= b && hi < f - b) {
#pragma unroll
                for (int i = i0; i < i0 + 8; ++i)
                    if (i < F) {
#pragma unroll
                        for (int v = 0; v < V; ++v)
                            acc[v] += __uint_as_float(from_key(key[v][i < F ? i : 0]));
                    }
            } else if (hi >= b && lo < f - b) {
#pragma unroll
                for (int i = i0; i < i0 + 8; ++i)
                    if (i < F && i >= b && i < f - b) {
#pragma unroll
                        for (int v = 0; v < V; ++v)
                            acc[v] += __uint_as_float(from_key(key[v][i < F ? i : 0]));
                    }
            }
        }
#pragma unroll
        for (int v = 0; v < V; ++v) o[v] = __float_as_uint(acc[v] / denom);
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            float acc = 0.0f;
#pragma unroll
            for (int i = 0; i < F; ++i)
                if (i >= b && i < f - b) acc += __uint_as_float(from_key(key[v][i]));
            o[v] = __float_as_uint(acc / denom);
        }
    }
}

// Coordinate-wise trimmed mean of F rows: the F values of a coordinate are sorted (total order
// of the keys), the b smallest and the b largest are dropped and the remaining F - 2b are
// averaged.  Rounding contract: fp32, the kept values are added one by one in ascending order
// starting from +0, then divided by float(F - 2b) (IEEE division).  One word per thread: f = 81
// takes 0.57 ms for 11.2 M coordinates, 1.01 of the time its bytes take at 6.5 TB/s (0.78 with
// two-wire comparators), f = 121 0.41 ms for 4 M (0.30 by bytes; 0.45 before): min/max issue.
template <int F, int V, bool PAD>
__global__ __launch_bounds__(kBlock) void trimmed_mean_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ row_index,
    int f, int b, unsigned group, uint32_t *__restrict__ out, const uint32_t *__restrict__ gate, int gate_n) {
    if (gate != nullptr && !any_word_set(gate, gate_n)) return;
    // (only the one-word form is launched in groups; without the test for it the gated form took 0.2-0.4 us longer)
    const unsigned tile = V == 1 && group != 0 ? neighbours_together(blockIdx.x, gridDim.x, group) : blockIdx.x;
    const int64_t gt = (int64_t)tile * kBlock + threadIdx.x;
    if (gt >= (d + V - 1) / V) return;
    const int64_t c0 = gt * V + V <= d ? gt * V : d - V;
    constexpr int NS = 1, kAhead = V == 1 ? 20 : prefetch_depth(F, NS);  // as the median kernels
    uint32_t key[V][F];
    const uint32_t voff = (uint32_t)(c0 * 4);
    const char *Xb = reinterpret_cast<const char *>(X);
    uint32_t stage[kAhead + 1][NS][V];
    const int lane = 0;
    uint32_t flags[(F + 63) / 64] = {};
    (void)lane; (void)flags;
    // PAD: f < F rows on the next generated size; the spare wires reload row_index[0] and carry
    // the largest key, so wires 0..f-1 end up holding the f values in ascending order
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) (!PAD || (j) < least_rows(F) || (j) < f ? to_key(x) : 0xFFFFFFFFu)
#define BYZ_S_ROW_ADDR(j, k) \
    (Xb + (uint64_t)(uint32_t)row_index[!PAD || (j) < least_rows(F) || (j) < f ? (j) : 0] * (uint64_t)ld * 4u + voff)
    if constexpr (pins_trimmed_mean(F)) {
#include "selnet_pin_on.inc"
#include "generated/selnet_sort_stream_dispatch.inc"
#include "selnet_pin_off.inc"
    } else {
#include "generated/selnet_sort_stream_dispatch.inc"
    }
#undef BYZ_S_ROW_ADDR
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) to_key(x)
    uint32_t o[V];
    trimmed_mean_of_sorted<F, V, pins_trimmed_mean(F)>(key, PAD ? f : F, b, o);
    store_vec<V>(out + c0, o);
}

// Sorts a bitonic sequence of F keys ascending with the log2(P) rounds of comparators P/2, P/4,
// ..., 1 apart of the P-wire bitonic merger, P the power of two at or above F.  The P - F spare
// wires carry the smallest key in front of a sequence that rises and then falls (LOW), the
// largest key behind one that falls and then rises (!LOW), which keeps either bitonic;
// comparators that only see spare wires fold away at compile time.
template <int F, int P, bool LOW>
__device__ __forceinline__ void sort_bitonic(uint32_t (&keys)[F]) {
    static_assert((P & (P - 1)) == 0 && P >= F && P < 2 * F, "P = power of two at or above F");
    if constexpr (P == F) {
        uint32_t(&k)[F] = keys;
#pragma unroll
        for (int apart = P / 2; apart >= 1; apart /= 2)
#pragma unroll
            for (int i = 0; i < P; ++i)
                if ((i & apart) == 0) BYZ_CE(i, i + apart)
    } else {
        uint32_t k[P];
#pragma unroll
        for (int i = 0; i < P; ++i)
            k[i] = LOW ? (i < P - F ? 0u : keys[i - (P - F) < 0 ? 0 : i - (P - F)])
                       : (i < F ? keys[i < F ? i : 0] : 0xFFFFFFFFu);
#pragma unroll
        for (int apart = P / 2; apart >= 1; apart /= 2)
#pragma unroll
            for (int i = 0; i < P; ++i)
                if ((i & apart) == 0) BYZ_CE(i, i + apart)
#pragma unroll
        for (int i = 0; i < F; ++i) keys[i] = k[LOW ? P - F + i : i];
    }
}

// acc += the keys' values whose ranks rank0 + i lie in [b, f - b), in ascending order.  b and f are
// wave-uniform: runs of eight ranks that lie wholly inside are added without a test, runs
// wholly outside are skipped.
template <int F>
__device__ __forceinline__ float add_kept_ranks(const uint32_t (&k)[F], int rank0, int b, int f,
                                                float acc) {
    static_assert(F % 8 == 0, "runs of eight");
#pragma unroll
    for (int i0 = 0; i0 < F; i0 += 8) {
        const int lo = rank0 + i0, hi = lo + 7;
        if (lo >= b && hi < f - b) {
#pragma unroll
            for (int i = i0; i < i0 + 8; ++i) acc += __uint_as_float(from_key(k[i]));
        } else if (hi >= b && lo < f - b) {
#pragma unroll
            for (int i = i0; i < i0 + 8; ++i)
                if (rank0 + i >= b && rank0 + i < f - b) acc += __uint_as_float(from_key(k[i]));
        }
    }
    return acc;
}

// The trimmed mean of two sorted halves (see trimmed_halves_kernel): out[c] of lane ln.
template <int F>
__device__ __forceinline__ void trimmed_mean_of_halves(uint32_t (&k)[F], uint32_t *s_half, float *s_sum,
                                                       int first, int ln, int64_t c, int64_t d, int f, int b,
                                                       uint32_t *__restrict__ out) {
    if (first != 0) {
#pragma unroll
        for (int m = 0; m < F; ++m) s_half[m * 64 + ln] = k[m];
    }
    __syncthreads();
    if (first == 0) {
#pragma unroll
        for (int m = 0; m < F; ++m) {
            const uint32_t a_ = k[m], b_ = s_half[(F - 1 - m) * 64 + ln];
            k[m] = a_ < b_ ? a_ : b_;
            s_half[(F - 1 - m) * 64 + ln] = a_ < b_ ? b_ : a_;
        }
    }
    __syncthreads();
    // ranks first .. first + F - 1, ascending; wave 0 adds its kept ranks first
    float acc = 0.0f;
    constexpr int P = 128;  // wires of the bitonic merger
    if constexpr (F == P) {
        if (first != 0) {
#pragma unroll
            for (int m = 0; m < F; ++m) k[m] = s_half[m * 64 + ln];
        }
        sort_bitonic<F, P, true>(k);  // no spare wires: one code path for both waves
    }
    if (first == 0) {
        if constexpr (F != P) sort_bitonic<F, P, true>(k);
        acc = add_kept_ranks<F>(k, 0, b, f, acc);
        s_sum[ln] = acc;
    }
    __syncthreads();
    if (first != 0) {
        if constexpr (F != P) {
#pragma unroll
            for (int m = 0; m < F; ++m) k[m] = s_half[m * 64 + ln];
            sort_bitonic<F, P, false>(k);
        }
        acc = add_kept_ranks<F>(k, F, b, f, s_sum[ln]);
        if (c < d) out[c] = __float_as_uint(acc / (float)(f - 2 * b));
    }
}

// Coordinate-wise trimmed mean of F < f <= 2F rows (F = 96, 112, 128), two waves per 64 coordinates, same
// rounding contract as trimmed_mean_kernel.  Wave h sorts wires [hF, hF + F) of its coordinates
// in registers (the 2F - f spare wires at the end carry the largest key).  With A and B the two
// sorted halves, min(A[m], B[F-1-m]) over m holds the F smallest of the union and max(...) the
// F largest, each as a bitonic sequence: wave 1 passes B through LDS, wave 0 keeps the minima
// and passes the maxima back through the same words, and each wave sorts its bitonic half
// (sort_bitonic).  Wave 0 then holds ranks 0..F-1 and
// wave 1 ranks F..2F-1; the kept ranks are added in ascending order, wave 0's partial sum
// going to wave 1 through LDS.  Half the registers of one 256-wire network per thread.
template <int F>
__global__ __launch_bounds__(128)
__attribute__((amdgpu_waves_per_eu(2, 2)))
void trimmed_halves_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ row_index,
    int f, int b, uint32_t *__restrict__ out, const uint32_t *__restrict__ gate, int gate_n) {
    if (gate != nullptr && !any_word_set(gate, gate_n)) return;
    __shared__ uint32_t s_half[F * 64];
    __shared__ float s_sum[64];
    const int ln = threadIdx.x & 63;
    const int first = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * F;  // first wire of this wave
    const int64_t c = (int64_t)blockIdx.x * 64 + ln;
    const int64_t cc = c < d ? c : d - 1;  // lanes past the end redo the last coordinate
    constexpr int V = 1, NS = 1, kAhead = 20;
    uint32_t key[V][F];
    const uint32_t voff = (uint32_t)(cc * 4);
    const char *Xb = reinterpret_cast<const char *>(X);
    uint32_t stage[kAhead + 1][NS][V];
    const int lane = 0;
    uint32_t flags[(F + 63) / 64] = {};
    (void)lane; (void)flags;
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) (first + (j) < f ? to_key(x) : 0xFFFFFFFFu)
#define BYZ_S_ROW_ADDR(j, k) \
    (Xb + (uint64_t)(uint32_t)row_index[first + (j) < f ? first + (j) : 0] * (uint64_t)ld * 4u + voff)
#include "generated/selnet_sort_stream_dispatch.inc"
#undef BYZ_S_ROW_ADDR
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) to_key(x)
    trimmed_mean_of_halves<F>(key[0], s_half, s_sum, first, ln, c, d, f, b, out);
}

// Mean around the median (second phase of Bulyan) for one coordinate whose theta values sit
// in ascending order in col[0], col[stride], ..: the beta values closest to the middle one
// (the median), added in ascending order from +0 in fp32 and divided by float(beta).
// Growing the window from the median one neighbour at a time -- the lower one when
// (median - lower) <= (upper - median) in fp32, or when no upper one is left -- ends, for
// finite values, at the window that starts at the first position s (from max(0, h-beta+1) to
// h, h the median's position) whose value is taken before the one beta places above it:
// s + beta beyond the end, or (median - col[s]) <= (col[s+beta] - median).  That test is
// false up to s and true from s on (rounded differences stay monotone, infinite ones too), so the start is found by
// halving the candidates: a test is two LDS reads and five instructions, and 3 to 6 tests do for 15 to 127 values where
// testing every candidate took as many as there are.  The additions read at fixed distances from the start, eight, then
// four, two and one, without a test per value.  us a call, before (every candidate, eight at a time) / with both:
// 4 M coordinates, 25 values beta = 7 66.5 / 65.1, 33 and 17 107.8 / 98.1, 49 and 33 170 / 149; 2 M, 121 and 60 372 / 290;
// 1 M, 127 and 127 267 / 202, 127 and 20 208 / 194; Bulyan 49 x 11.2 M 724 / 702.
// A column with a NaN or an infinite median has differences that are NaN, and no order: there every
// candidate is tested and the failed tests are counted (the same number where there is an order; with a NaN in every
// column 121 and 60 371 / 305, 49 and 33 167 / 143).
__device__ __forceinline__ float mean_around_median(const float *col, int stride, int theta,
                                                    int beta) {
    const int h = (theta - 1) / 2;
    const float med = col[h * stride], least = col[0], most = col[(theta - 1) * stride];
    const int s_min = h - beta + 1 > 0 ? h - beta + 1 : 0;
    const int last = h < theta - beta ? h : theta - beta;  // from here on a candidate is taken untested
    const float *at = col + s_min * stride;
    auto fails = [&](const float *c) { return !((med - c[0]) <= (c[beta * stride] - med)); };
    const bool ordered = least == least && most == most && __builtin_fabsf(med) < __builtin_inff();
    if (__builtin_amdgcn_ballot_w64(!ordered) == 0) {
        for (int n = last - s_min; n > 0; n /= 2) {  // the start is among the n candidates from `at` on, or behind them
            const int half = (n + 1) / 2;
            if (fails(at + (half - 1) * stride)) at += half * stride;
        }
    } else {
        int count = 0;
        for (int s = 0; s < last - s_min; ++s) count += fails(at + s * stride) ? 1 : 0;
        at += count * stride;
    }
    float acc = 0.0f;
    int t = 0;
    auto add = [&](auto number) {
        constexpr int N = decltype(number)::value;
        float x[N];
#pragma unroll
        for (int u = 0; u < N; ++u) x[u] = at[u * stride];
#pragma unroll
        for (int u = 0; u < N; ++u) acc += x[u];
        at += N * stride;
        t += N;
    };
    while (t + 8 <= beta) add(std::integral_constant<int, 8>());
    if (beta - t >= 4) add(std::integral_constant<int, 4>());
    if (beta - t >= 2) add(std::integral_constant<int, 2>());
    if (beta - t >= 1) add(std::integral_constant<int, 1>());
    return acc / (float)beta;
}

// Second phase of Bulyan: the theta rows selected_rows[0..theta-1] are sorted per coordinate
// by the streamed full-sort network on N >= theta wires (N the next generated size); the
// N - theta spare wires reload the first row and are tied to the largest key, so wires
// 0..theta-1 end up holding the chosen values in ascending order.  They go to an LDS column of the
// thread (word i*BLOCK + thread: conflict-free), where the window around the median is found with
// run-time indices.  One word per thread.
// Dynamic LDS: N*BLOCK*4 bytes; the widest networks run one wave a block, so that several
// blocks' columns fit a CU and the number of waves is again what the registers allow.
template <int F, int BLOCK>
__global__ __launch_bounds__(BLOCK) void bulyan_mean_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld,
    const int32_t *__restrict__ selected_rows, int theta, int beta, unsigned group, uint32_t *__restrict__ out) {
    extern __shared__ float s_bulyan_col[];
    const unsigned tile = group != 0 ? neighbours_together(blockIdx.x, gridDim.x, group) : blockIdx.x;
    const int64_t c0 = (int64_t)tile * BLOCK + threadIdx.x;
    if (c0 >= d) return;
    constexpr int V = 1, NS = 1, kAhead = 20;
    uint32_t key[V][F];
    const uint32_t voff = (uint32_t)(c0 * 4);
    const char *Xb = reinterpret_cast<const char *>(X);
    uint32_t stage[kAhead + 1][NS][V];
    const int lane = 0;
    uint32_t flags[(F + 63) / 64] = {};
    (void)lane; (void)flags;
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) ((j) < least_rows(F) || (j) < theta ? to_key(x) : 0xFFFFFFFFu)
#define BYZ_S_ROW_ADDR(j, k) \
    (Xb + (uint64_t)(uint32_t)selected_rows[(j) < least_rows(F) || (j) < theta ? (j) : 0] * (uint64_t)ld * 4u + voff)
    if constexpr (pins_trimmed_mean(F)) {
#include "selnet_pin_on.inc"
#include "generated/selnet_sort_stream_dispatch.inc"
#include "selnet_pin_off.inc"
    } else {
#include "generated/selnet_sort_stream_dispatch.inc"
    }
#undef BYZ_S_ROW_ADDR
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) to_key(x)
    float *col = s_bulyan_col + threadIdx.x;
#pragma unroll
    for (int i = 0; i < F; ++i) col[i * BLOCK] = __uint_as_float(from_key(key[0][i]));
    const uint32_t o[1] = {__float_as_uint(mean_around_median(col, BLOCK, theta, beta))};
    store_vec<1>(out + c0, o);
}

// First kernel of a single-pass call: clears the state the later kernels accumulate into and
// lays out the rows of each file for the pass.  When every copy is read, that is the replica
// order as it stands: each wave chooses for itself which copy feeds the median.
// In early-majority mode the kernel is a probe: it compares the copies of every file on a
// sample of <= kProbe coordinates (kProbe/16 runs of 16 consecutive words spread over [0, d); all
// of [0, d) when d <= kProbe), derives the probable equality classes, and puts the probable
// winner's class first (the copies that mode reads) and equal-looking copies adjacent.  Only
// the speed of the call depends on this guess.
// One block of kProbeThreads threads: thread group q = tid / kProbe takes the files
// q, q + kProbeSplit, ..., every group on the same kProbe sample coordinates, so a thread waits
// for F*R / kProbeSplit loads.
template <int F, int R>
__global__ __launch_bounds__(kProbeThreads) void probe_kernel(const uint32_t *__restrict__ X,
                                                           int64_t d, int64_t ld,
                                                           const int32_t *__restrict__ file_rows,
                                                           AggWorkspace *ws, int probe_opts) {
    const int early_majority = probe_opts & 1;        // bit 0: early-majority mode
    const uint32_t shift = (uint32_t)probe_opts >> 16;  // bits 16..31: moves the sample
    __shared__ uint32_t s_neq[kWide];
    __shared__ uint32_t s_all_majority;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    static_assert(kProbe >= kWide, "one probe thread per file");
    if (tid < kWide) {
        s_neq[tid] = 0;
        ws->pneq[tid] = 0;
        ws->pair_neq[tid] = 0;
    }
    if (tid == 0) {
        s_all_majority = 1;
        ws->need_median = 0;
        ws->need_revote = 0;
        ws->path = 0;
    }
    __syncthreads();
    if (early_majority == 0) {
        if (tid < F) {
            uint32_t packed = (uint32_t)R << 24;
            for (int p = 0; p < R; ++p) {
                ws->perm_off[tid * kRowStride + p] = (uint64_t)file_rows[tid * R + p] * (uint64_t)ld * 4u;
                packed |= (uint32_t)p << (3 * p);
            }
            ws->perm[tid] = packed;
        }
        if (tid == 0) ws->slots_per_file = R;
        return;
    }

    // threads without a sample coordinate of their own redo coordinate 0
    const int ct = tid % kProbe;  // which sample coordinate
    const int q = tid / kProbe;   // which share of the files (wave-uniform: kProbe % 64 == 0)
    int64_t c = 0;
    if (d <= kProbe) {
        if (ct < d) c = ct;
    } else {
        // runs start (d - 16) / 15 apart from a point the caller's shift picks, wrapping
        // around so that a run stays inside [0, d)
        const int64_t run = ct >> 4, off = ct & 15;
        const uint64_t start = ((uint64_t)shift * 2654435761ull) % (uint64_t)(d - 15);
        c = (int64_t)(((uint64_t)(run * ((d - 16) / (kProbe / 16 - 1))) + start) % (uint64_t)(d - 15)) + off;
    }
    // this group's files in batches of G: all loads of a batch are issued before the first
    // ballot waits; the bits of file j are parked in lane j % 64, word j / 64
    constexpr int kMine = (F + kProbeSplit - 1) / kProbeSplit;  // files per group, at most
    constexpr int G = (kMine * R <= 96) ? kMine : 96 / R;
    uint32_t flags[(F + 63) / 64] = {};
#pragma unroll
    for (int t0 = 0; t0 < kMine; t0 += G) {
        uint32_t x[G][R];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int j = q + kProbeSplit * (t0 + g);
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (t0 + g < kMine && j < F) x[g][k] = X[(int64_t)file_rows[j * R + k] * ld + c];
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int j = q + kProbeSplit * (t0 + g);
            if (t0 + g >= kMine || j >= F) continue;
            uint32_t wb = 0;
#pragma unroll
            for (int a = 0; a < R; ++a)
#pragma unroll
                for (int b = a + 1; b < R; ++b)
                    wb |= wave_any(x[g][a] ^ x[g][b]) << pair_bit(R, a, b);
#pragma unroll
            for (int w = 0; w < (F + 63) / 64; ++w)
                if (lane == (j & 63) && (j >> 6) == w) flags[w] |= wb;
        }
    }
#pragma unroll
    for (int w = 0; w < (F + 63) / 64; ++w)
        if (64 * w + lane < F && flags[w] != 0) atomicOr(&s_neq[64 * w + lane], flags[w]);
    __syncthreads();

    if (tid < F) {
        const int j = tid;
        const uint32_t neq = s_neq[j];
        const int w = decide_winner(neq, R);
        // label[k] = lowest replica that looked equal to k on the sample
        int label[R];
        for (int k = 0; k < R; ++k) {
            label[k] = k;
            for (int a = 0; a < k; ++a)
                if (copies_equal(neq, R, a, k)) { label[k] = a; break; }
        }
        // order: the winner's class, then the other classes by lowest member; members ascending
        int perm[R];
        int n = 0;
        for (int k = 0; k < R; ++k)
            if (label[k] == label[w]) perm[n++] = k;
        for (int c0 = 0; c0 < R; ++c0) {
            if (label[c0] != c0 || c0 == label[w]) continue;
            for (int k = 0; k < R; ++k)
                if (label[k] == c0) perm[n++] = k;
        }
        // Early-majority mode: once r' = (R+1)/2 copies are known to be identical they are the
        // majority whatever the other copies hold (Sec. 2), so when the probable winner's class
        // has at least r' members only its first r' are read and verified; the remaining slots
        // repeat slot 0 (served from cache) and carry no assumption.
        int members = 0;
        for (int k = 0; k < R; ++k) members += label[k] == label[w] ? 1 : 0;
        const int need = (R + 1) / 2;
        const int slots = (early_majority != 0 && members >= need) ? need : R;
        uint32_t packed = (uint32_t)slots << 24;
        for (int p = 0; p < R; ++p) {
            const int k = perm[p < slots ? p : 0];
            ws->perm_off[j * kRowStride + p] = (uint64_t)file_rows[j * R + k] * (uint64_t)ld * 4u;
            packed |= (uint32_t)k << (3 * p);
        }
        ws->perm[j] = packed;
        if (slots != need) s_all_majority = 0;
    }
    __syncthreads();
    // if every file gets by with r' slots, the single pass loads only those
    if (tid == 0) ws->slots_per_file = (early_majority != 0 && s_all_majority != 0) ? (R + 1) / 2 : R;
}

// Which tile of kBlock threads a block works on.  Blocks go to the eight XCDs round-robin
// (block b runs on XCD b mod 8).  A launch that is over after a round or two of resident blocks
// is dominated by its start: there every XCD gets one contiguous eighth of the tiles, so that
// its L2 and address translation see one range of every row instead of all of it (d = 2^20,
// 75 rows: 56 -> 52.5 us).  In long launches that costs 1-3 %; there each XCD gets GROUP neighbours at a time,
// which share the cache lines where rows don't start on one.  us a call, plain order / 16 / 64 neighbours, 6 M
// coordinates off lines: (25,3) 302 / 292 / 290, (49,3) 589 / 569 / 566, (49,7) 1377 / 1329 / 1332, (81,3) 962 /
// 924 / 928; on lines 291 / 292 / 289, 556 / 548 / 544, 1233 / 1212 / 1218, 893 / 872 / 878.  One word a thread, 2.5 M:
// (121,3) 668 / 639 / 637 off lines, 562 / 571 / 556 on, (169,3) 922 / 870 / 864 and 792 / 787 / 785.
// Up to 15 files of which every copy is read that pays later: us a call, plain / 64 neighbours, (9,3) 2.2 M 70.0 / 74.2 on
// the lines, 74.3 / 78.8 off, 3.5 M 89.2 / 96.5 and 96.7 / 104.2, 6 M the same, 11.2 M 242.7 / 236.4 and 263.3 /
// 256.3; (15,3) 3.5 M 117.7 / 122.3 and 127.1 / 133.3, 6 M 194.7 / 194.6 and 208.3 / 211.3, 11.2 M the same.  (21,3)
// 3.5 M 147.8 / 149.6, trimmed mean off the lines 156.5 / 152.5; early-majority (9,3) 2.5 M 43.6 / 43.0 and 44.6 / 43.3.
constexpr unsigned kShortLaunchBlocks = 2048;
constexpr unsigned block_group(int v) { return v == 2 ? 16 : 64; }
// Longest launch in plain order, of those that are not short.
constexpr unsigned plain_launch_blocks(int f, bool all_copies) {
    return f <= 15 && all_copies ? 4 * kShortLaunchBlocks : kShortLaunchBlocks;
}
template <unsigned GROUP, unsigned PLAIN = kShortLaunchBlocks>
__device__ __forceinline__ unsigned tile_of_block(unsigned b, unsigned n_blocks) {
    if (n_blocks > PLAIN) return neighbours_together(b, n_blocks, GROUP);
    if (PLAIN > kShortLaunchBlocks && n_blocks > kShortLaunchBlocks) return b;
    const unsigned q = n_blocks / 8, rem = n_blocks % 8, x = b % 8, i = b / 8;
    return x * q + (x < rem ? x : rem) + i;  // XCD x owns q tiles, one more if x < rem
}

// Vote and median in one pass: streams the first NS slots of every file's permuted row list once (NS = R:
// every copy; NS = r' = (R+1)/2 in early-majority mode when every file has a probable
// majority).  Every pair of slots is compared over all coordinates (ws->pneq), which is the whole
// of the vote's comparison, and each wave feeds the median network from the slot that
// local_choice picks by what it has just compared: where a file has a strict majority over all
// of d, that slot holds the majority's values on the wave's coordinates, so a copy that was
// tampered with somewhere else costs nothing.  The decision kernel behind this one knows the
// true winners and, from the bits that say which slots the fed ones differed from, whether
// every wave fed the winner's values.
template <int F, int R, int NS, bool TRIM, int V>
__device__ __forceinline__ void fused_body(const uint32_t *__restrict__ X, int64_t d, int64_t ld,
                                           const uint64_t *__restrict__ perm_off,
                                           AggWorkspace *ws, int trim_b,
                                           uint32_t *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    // Thread t owns the V words starting at min(V*t, d - V): the last vector of a row overlaps
    // its neighbour instead of a scalar tail, and threads past the end redo it, so there are
    // no branches around loads and ballots (d >= V is the launcher's business).
    const int64_t n_thr = (d + V - 1) / V;
    constexpr unsigned kPlain = plain_launch_blocks(F, NS == R);
    const int64_t gt = (int64_t)tile_of_block<block_group(V), kPlain>(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    const int64_t c0 = (gt + 1) * V <= d ? gt * V : d - V;
    uint32_t flags[(F + 63) / 64] = {};  // lane j%64 collects the pair bits of file j
    // What other waves have published so far, read now so that the wait is over long before the
    // end: a wave whose bits were all there when it started (all but the first waves of a
    // launch) ends without touching the shared words at all.
    uint32_t seen[(F + 63) / 64];
#pragma unroll
    for (int w = 0; w < (F + 63) / 64; ++w)
        seen[w] = 64 * w + lane < F ? load_shared_word(&ws->pneq[64 * w + lane]) : 0u;
    const uint32_t voff = (uint32_t)(c0 * 4);
    const char *Xb = reinterpret_cast<const char *>(X);
    uint32_t key[V][F];       // wire j of the network = file j
    // files prefetched ahead of the one being consumed
    constexpr int kAhead = V < vec_for_pass(F, R, TRIM) ? (NS <= 3 ? 8 : 5) : prefetch_depth(F, NS);
    uint32_t stage[kAhead + 1][NS][V];  // copies of the file in use and of those in flight
    uint32_t o[V];
    // The generated program walks the files in order: the loads of file j+kAhead are issued
    // before file j is consumed (compares, key), followed by every comparator of the median
    // (or, for the trimmed mean, sorting) network whose inputs are complete by then.
#define BYZ_S_ROW_ADDR(j, k) (Xb + perm_off[(j) * kRowStride + (k)] + voff)
    if constexpr (!TRIM) {
        // median: every comparator is made to run in the share of the file that completes its
        // inputs, so that a wave has loads in flight while it works through the network instead
        // of running the whole network at the end
#include "selnet_pin_on.inc"
#include "generated/selnet_stream_dispatch.inc"
#include "selnet_pin_off.inc"
    } else {
#include "selnet_pin_on.inc"
#include "generated/selnet_sort_stream_dispatch.inc"
#include "selnet_pin_off.inc"
        trimmed_mean_of_sorted<F, V, true>(key, F, trim_b, o);
    }
#undef BYZ_S_ROW_ADDR
    if (gt < n_thr) store_vec<V>(out + c0, o);
#pragma unroll
    for (int w = 0; w < (F + 63) / 64; ++w)
        merge_flags(ws->pneq + 64 * w, F - 64 * w < 64 ? F - 64 * w : 64, lane,
                    flags[w] & ~seen[w]);
}

template <int F, int R, bool TRIM, int V>
__global__ __launch_bounds__(kBlock) void fused_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const uint64_t *__restrict__ perm_off,
    const uint32_t *__restrict__ slots_per_file, AggWorkspace *ws, int trim_b,
    uint32_t *__restrict__ out) {
    // wave-uniform choice written by the probe (four_words_of_five: no early-majority trimmed mean)
    constexpr bool kEarly = !(TRIM && R == 5 && V == 4);
    if constexpr (kEarly) {
        if (*slots_per_file == (R + 1) / 2) {
            fused_body<F, R, (R + 1) / 2, TRIM, V>(X, d, ld, perm_off, ws, trim_b, out);
            return;
        }
    }
    fused_body<F, R, R, TRIM, V>(X, d, ld, perm_off, ws, trim_b, out);
}

// First kernel of a call on more than 169 files: clears the state the later kernels accumulate into and
// lays out the rows of each file in replica order, spare wires repeating file 0.
__global__ __launch_bounds__(kWide) void lay_out_rows_kernel(const int32_t *__restrict__ file_rows, int f, int r,
                                                             int64_t ld, AggWorkspace *ws) {
    const int j = threadIdx.x;
    ws->pneq[j] = 0;
    uint32_t packed = (uint32_t)r << 24;
    for (int p = 0; p < r; ++p) {
        ws->perm_off[j * kRowStride + p] = (uint64_t)file_rows[(j < f ? j : 0) * r + p] * (uint64_t)ld * 4u;
        packed |= (uint32_t)p << (3 * p);
    }
    ws->perm[j] = packed;
    if (j == 0) {
        ws->need_median = 0;
        ws->need_revote = 0;
        ws->slots_per_file = (uint32_t)r;
    }
}

// Vote and median or trimmed mean of F < f <= 2F - 1 files of three copies in one pass, the files split over two
// waves per 64 coordinates as the rows are in median_halves_kernel: each wave streams the copies of its F
// files, compares them and chooses what it feeds as in fused_body.  Within 1.12 of the time its bytes take at
// 6.5 TB/s at f = 255 (1 M coordinates 554 us a call, vote and median one after the other 709; 2 M 992 and 1374;
// trimmed mean 647 and 833): two waves per SIMD, HBM and min/max issue together.  F = 96 leaves room for a
// third wave (171 files, 1 M: 383 -> 338; 112 would spill).  20 files ahead: 2 % slower than 5.
// A block's 64 words off the cache lines are three lines for two: there neighbours go to one XCD (f = 255, 1 M
// 705 us in plain order, 597; 2 M 1379, 1149; on lines 188.7 and 192 for 300 k, the same for 2 M).
template <int F, bool TRIM>
__global__ __launch_bounds__(128)
__attribute__((amdgpu_waves_per_eu(!TRIM && F <= 96 ? 3 : 2, !TRIM && F <= 96 ? 3 : 2)))
void fused_halves_kernel(const uint32_t *__restrict__ X, int64_t d, const uint64_t *__restrict__ perm_off,
                         AggWorkspace *ws, int f, int trim_b, unsigned group, uint32_t *__restrict__ out) {
    __shared__ uint32_t s_half[F * 64];
    __shared__ float s_sum[64];
    const int lane = threadIdx.x & 63;
    const int first = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * F;  // first file of this wave
    const int64_t c = (int64_t)(group != 0 ? neighbours_together(blockIdx.x, gridDim.x, group) : blockIdx.x) * 64 + lane;
    const int64_t cc = c < d ? c : d - 1;  // lanes past the end redo the last coordinate
    const int pad_low_end = TRIM ? f : f + (F - 1 - (f - 1) / 2);
    constexpr int V = 1, NS = 3, kAhead = 5;
    uint32_t flags[(F + 63) / 64] = {}, seen[(F + 63) / 64];
#pragma unroll
    for (int w = 0; w < (F + 63) / 64; ++w)
        seen[w] = 64 * w + lane < F && first + 64 * w + lane < f ? load_shared_word(&ws->pneq[first + 64 * w + lane]) : 0u;
    const uint32_t voff = (uint32_t)(cc * 4);
    const char *Xb = reinterpret_cast<const char *>(X);
    uint32_t key[V][F];
    uint32_t stage[kAhead + 1][NS][V];
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) \
    (first + (j) < f ? to_key(x) : (first + (j) < pad_low_end ? 0u : 0xFFFFFFFFu))
#define BYZ_S_ROW_ADDR(j, k) (Xb + perm_off[(first + (j)) * kRowStride + (k)] + voff)
#include "selnet_pin_on.inc"
#include "generated/selnet_sort_stream_dispatch.inc"
#include "selnet_pin_off.inc"
#undef BYZ_S_ROW_ADDR
#undef BYZ_S_KEY
#define BYZ_S_KEY(j, x) to_key(x)
#pragma unroll
    for (int w = 0; w < (F + 63) / 64; ++w) {
        const int here = F - 64 * w < 64 ? F - 64 * w : 64, files = f - first - 64 * w;
        merge_flags(ws->pneq + first + 64 * w, files < here ? files : here, lane, flags[w] & ~seen[w]);
    }
    if constexpr (TRIM)
        trimmed_mean_of_halves<F>(key[0], s_half, s_sum, first, lane, c, d, f, trim_b, out);
    else
        median_of_halves<F>(key[0], s_half, first, lane, c, d, out);
}

// The call on short rows in two kernels that need nothing cleared before them: instead of merging their bits
// into shared words by atomics, the blocks of the first write them to a slot each, and every block of the
// second adds the slots up and decides for itself.  Four kernels one after the other (clear and lay
// out, pass, decide, gated median) cost 14 us of launches and waits whatever d is; the figures of both
// forms stand at launch_short.
// Slots sit where the long form keeps its row offsets: one to four bytes per file, whole 16-byte pieces.
constexpr int slot_bits(int r) { return r == 3 ? 8 : (r == 5 ? 16 : 32); }  // of the r(r-1)/2 + r used
constexpr int slot_words(int f, int r) { return (f * slot_bits(r) + 127) / 128 * 4; }
constexpr int most_slots(int f, int r) {
    return (int)(sizeof(AggWorkspace::perm_off) / 4) / slot_words(f, r);
}

// First kernel.
template <int F, int R, bool TRIM, int V, int BLOCK>
__global__ __launch_bounds__(BLOCK) void short_pass_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ file_rows,
    uint32_t *__restrict__ slots, int trim_b, uint32_t *__restrict__ out) {
    const int64_t gt = (int64_t)tile_of_block<block_group(V)>(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
#include "short_pass.inc"
    __syncthreads();
    for (int t = threadIdx.x; t < kWords; t += BLOCK) slots[(int64_t)blockIdx.x * kWords + t] = s_bits[t];
}

// The decision of single_pass_decide_kernel on a call that read every copy, in every block: findings_of(j) = the bits
// of file j, complete behind a barrier.  Then, where it asks for it, the median or trimmed mean of the winners' rows
// again by thread gt.  Block 0 writes what the caller gets.
template <int F, int R, bool TRIM, int V, typename Findings>
__device__ __forceinline__ void decide_and_redo(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ file_rows, AggWorkspace *ws,
    int64_t gt, int trim_b, int32_t *winner_replica, uint32_t *__restrict__ out, Findings findings_of) {
    __shared__ uint32_t s_redo;
    __shared__ int32_t s_row[F];
    if (threadIdx.x == 0) s_redo = 0;
    __syncthreads();  // the findings are complete, too
    if (const int j = threadIdx.x; j < F) {
        const uint32_t field = findings_of(j);
        const int w = decide_winner(field, R);
        if ((field & fed_differs_bit(R, w)) != 0) s_redo = 1;
        s_row[j] = file_rows[j * R + w];
        if (blockIdx.x == 0) {
            if (winner_replica != nullptr) winner_replica[j] = w;
            ws->winner_row[j] = s_row[j];
        }
    }
    __syncthreads();
    const bool redo = s_redo != 0;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        ws->path = redo ? (uint32_t)BYZ_PATH_MEDIAN_REDONE : (uint32_t)BYZ_PATH_SINGLE_PASS;
    if (!redo) return;
    if (gt >= (d + V - 1) / V) return;
    const int64_t c0 = gt * V + V <= d ? gt * V : d - V;
    constexpr int NS = 1, kAhead = V == 1 ? 20 : prefetch_depth(F, NS);
    uint32_t key[V][F];
    uint32_t o[V];
    const uint32_t voff = (uint32_t)(c0 * 4);
    const char *Xb = reinterpret_cast<const char *>(X);
    uint32_t stage[kAhead + 1][NS][V];
    const int lane = 0;
    uint32_t flags[(F + 63) / 64] = {};
    (void)lane; (void)flags;
    // (the winners' rows from LDS as scalars)
#define BYZ_S_ROW_ADDR(j, k) \
    (Xb + (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(s_row[j]) * (uint64_t)ld * 4u + voff)
    if constexpr (!TRIM) {
        if constexpr (pins_median(F)) {
#include "selnet_pin_on.inc"
#include "generated/selnet_stream_dispatch.inc"
#include "selnet_pin_off.inc"
        } else {
#include "generated/selnet_stream_dispatch.inc"
        }
    } else {
        if constexpr (pins_trimmed_mean(F)) {
#include "selnet_pin_on.inc"
#include "generated/selnet_sort_stream_dispatch.inc"
#include "selnet_pin_off.inc"
        } else {
#include "generated/selnet_sort_stream_dispatch.inc"
        }
        trimmed_mean_of_sorted<F, V, pins_trimmed_mean(F)>(key, F, trim_b, o);
    }
#undef BYZ_S_ROW_ADDR
    store_vec<V>(out + c0, o);
}

// The bits of file j in a block's slot.
template <int R>
__device__ __forceinline__ uint32_t slot_findings(const uint32_t *s_bits, int j) {
    constexpr int kBits = slot_bits(R);
    return s_bits[j * kBits / 32] >> (j * kBits % 32);
}

// Second kernel, and the last one of a call that reads every copy and has no slots (SLOTS false: the findings are in
// ws->pneq; decides_in_median).
template <int F, int R, bool TRIM, int V, bool SLOTS>
__global__ __launch_bounds__(kBlock) void decide_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ file_rows,
    AggWorkspace *ws, int n_slots, int trim_b, int32_t *winner_replica, uint32_t *__restrict__ out) {
    constexpr int kBits = slot_bits(R), kWords = slot_words(F, R), kPieces = kWords / 4;
    static_assert(R * (R - 1) / 2 + R <= kBits && kPieces <= kBlock && F <= kBlock, "a file's bits, a thread a piece and a file");
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __shared__ uint32_t s_bits[kWords];
    if constexpr (SLOTS) {
        for (int t = threadIdx.x; t < kWords; t += kBlock) s_bits[t] = 0;
        const u32x4 *pieces = reinterpret_cast<const u32x4 *>(ws->perm_off);
        constexpr int kStride = kBlock / kPieces * kPieces;  // a thread's pieces are the same files' every time
        u32x4 mine = {0, 0, 0, 0};
        if ((int)threadIdx.x < kStride) {
#pragma unroll 4
            for (int t = threadIdx.x; t < n_slots * kPieces; t += kStride) mine |= pieces[t];
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (mine[e] != 0) atomicOr(&s_bits[(int)threadIdx.x % kPieces * 4 + e], mine[e]);
    }
    decide_and_redo<F, R, TRIM, V>(X, d, ld, file_rows, ws, (int64_t)blockIdx.x * kBlock + threadIdx.x, trim_b,
                                   winner_replica, out, [&](int j) {
                                       if constexpr (SLOTS) return slot_findings<R>(s_bits, j);
                                       else return load_shared_word(&ws->pneq[j]);
                                   });
}

// Both in one, for rows that one block holds, a word per thread (64 threads or more: the loops over s_bits and files).
constexpr int kOneBlock = 1024;
template <int F, int R, bool TRIM>
__global__ __launch_bounds__(kOneBlock) void one_block_kernel(
    const uint32_t *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ file_rows,
    AggWorkspace *ws, int trim_b, int32_t *winner_replica, uint32_t *__restrict__ out) {
    static_assert(F <= 64 && slot_words(F, R) <= 64, "a wave covers the files and the words of their bits");
    constexpr int V = 1, BLOCK = kOneBlock;
    const int64_t gt = threadIdx.x;
#include "short_pass.inc"
    decide_and_redo<F, R, TRIM, 1>(X, d, ld, file_rows, ws, threadIdx.x, trim_b, winner_replica, out,
                                   [&](int j) { return slot_findings<R>(s_bits, j); });
}

// ---------------------------------------------------------------------------- launchers

[[maybe_unused]] constexpr int kVec = 4;  // words per thread and load; rows only need dword alignment

// blocks for n_vec vector-owning threads; at least one so the trailing words get a block
inline unsigned blocks_for(int64_t n_vec) {
    const int64_t b = (n_vec + kBlock - 1) / kBlock;
    return (unsigned)(b > 0 ? b : 1);
}

// Behind the single pass and its decision the median or trimmed-mean kernel nearly always returns at once, and its
// cost is that of launching its blocks (1800 a microsecond: 24 us of a 540 us call with one word
// per thread at d = 11.2 M).  There, on rows longer than this, the networks of up to 49 wires run
// four words per thread.
[[maybe_unused]] constexpr int64_t kManyBlocks = 131072;
constexpr int gated_vec(int f) { return f <= 49 ? 4 : 1; }

// Rows that do not start on cache lines: with one word per thread a block of the median reads nine
// lines for eight of every row (f = 49, 2 M coordinates: 77 us, 68 with four words; on lines 63
// and 67).  So networks that HBM bounds alone run four words per thread there, up to 35 wires
// from kManyBlocks coordinates on (f = 25, 0.4 / 2 M: 7.7 / 34.4 us, one word 8.5 / 38.2), up to 49 from
// 1 M on (f = 49, 0.7 M: 27.4, one word 25.6), and otherwise up to 81 wires neighbouring blocks go
// to one XCD, sixteen at a time (f = 65, 2 M: 99.9 -> 95.4; above 81 wires nothing is gained).
[[maybe_unused]] inline bool rows_on_lines(const void *X, int64_t ld) {
    return ((uintptr_t)X & 127u) == 0 && ld % 32 == 0;
}
// Neighbouring blocks an XCD takes at a time in the two-wave kernels off the lines (64 words a block).
[[maybe_unused]] constexpr unsigned kHalvesGroup = 64;
[[maybe_unused]] constexpr int64_t four_words_from(int f) { return f <= 35 ? kManyBlocks : (int64_t)1 << 20; }

[[maybe_unused]] constexpr int64_t kMaxCoords = (int64_t)1 << 30;  // byte offsets inside a row fit 32 bits

#if BYZ_IN_PART(0)
// Blocks of a vote: every block walks over its files one after the other, so where the rows alone
// do not give 1024 blocks the files are dealt out too, two or more to a block ((255,3) whole call,
// d = 1003 206 -> 23 us, 100000 234 -> 89, 500000 381 -> 345; 512 or 2048 blocks: up to 20 % slower).
// `even`: nearly two blocks a CU are left as they are, which suits the exact vote of five or seven copies
// (rows of 500032 words: (49,5) 77.5 -> 72.7 us, (49,7) 113 -> 102; of 400001 dealt out 70.6 and 104,
// left 80.3 and 116) and neither three copies (500032: 45.7 dealt out, 50.0 left) nor the tolerant vote.
inline dim3 vote_grid(int64_t d, int f, bool even) {
    const unsigned x = blocks_for(d / kVec);
    const unsigned want = even && x > 450 ? 1 : 1024u / x, most = ((unsigned)f + 1) / 2;
    const unsigned y = want < 1 ? 1 : (want < most ? want : most);
    const unsigned per = ((unsigned)f + y - 1) / y;
    return dim3(x, ((unsigned)f + per - 1) / per);
}

template <int R>
int launch_vote_pairs(const uint32_t *X, int64_t d, int64_t ld, const int32_t *rows, int f,
                      uint32_t *neq, const uint32_t *gate, int gate_n, const uint32_t *only_files,
                      hipStream_t s) {
    const dim3 grid = vote_grid(d, f, R >= 5);
    vote_pairs_kernel<R, kVec><<<grid, kBlock, 0, s>>>(X, d, ld, rows, f, (f + grid.y - 1) / grid.y, neq,
                                                       gate, gate_n, only_files);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

int launch_vote_pairs_r(int r, const uint32_t *X, int64_t d, int64_t ld, const int32_t *rows,
                        int f, uint32_t *neq, const uint32_t *gate, int gate_n,
                        const uint32_t *only_files, hipStream_t s) {
    switch (r) {
        case 3: return launch_vote_pairs<3>(X, d, ld, rows, f, neq, gate, gate_n, only_files, s);
        case 5: return launch_vote_pairs<5>(X, d, ld, rows, f, neq, gate, gate_n, only_files, s);
        case 7: return launch_vote_pairs<7>(X, d, ld, rows, f, neq, gate, gate_n, only_files, s);
        default: return BYZ_EINVAL;
    }
}

int launch_vote_pairs_tolerant(int r, const uint32_t *X, int64_t d, int64_t ld,
                               const int32_t *rows, int f, float atol, float rtol, uint32_t *far,
                               hipStream_t s) {
    const dim3 g = vote_grid(d, f, false);
    const int per = (f + (int)g.y - 1) / (int)g.y;
    switch (r) {
        case 3:
            vote_pairs_tolerant_kernel<3, kVec><<<g, kBlock, 0, s>>>(X, d, ld, rows, f, per, atol, rtol, far);
            break;
        case 5:
            vote_pairs_tolerant_kernel<5, kVec><<<g, kBlock, 0, s>>>(X, d, ld, rows, f, per, atol, rtol, far);
            break;
        case 7:
            vote_pairs_tolerant_kernel<7, kVec><<<g, kBlock, 0, s>>>(X, d, ld, rows, f, per, atol, rtol, far);
            break;
        default: return BYZ_EINVAL;
    }
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

#endif  // part 0

#if BYZ_IN_PART(5)
template <int F>
int launch_median_net(const uint32_t *X, int64_t d, int64_t ld, const int32_t *row_index,
                      uint32_t *out, const uint32_t *gate, int gate_n, hipStream_t s) {
    median_kernel<F, kVec><<<blocks_for(d / kVec), kBlock, 0, s>>>(X, d, ld, row_index, out, gate,
                                                                  gate_n);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

#endif  // part 5

#if BYZ_IN_PART(5) || BYZ_IN_PART(9) || BYZ_IN_PART(11) || BYZ_IN_PART(19) || BYZ_IN_PART(20)
template <int F, bool PAD>
int launch_median_large(const uint32_t *X, int64_t d, int64_t ld, const int32_t *row_index, int f,
                        uint32_t *out, const uint32_t *gate, int gate_n, hipStream_t s) {
    const bool lines = rows_on_lines(X, ld);
    if constexpr (gated_vec(F) > 1) {
        if ((gate != nullptr && d > kManyBlocks) || (!lines && d > four_words_from(F))) {
            constexpr int V = gated_vec(F);
            median_large_kernel<F, V, PAD><<<blocks_for((d + V - 1) / V), kBlock, 0, s>>>(
                X, d, ld, row_index, f, 0, out, gate, gate_n);
            BYZ_HIP(hipGetLastError());
            return BYZ_OK;
        }
    }
    const unsigned group = !lines && F <= 81 && d > kManyBlocks ? 16 : 0;
    median_large_kernel<F, 1, PAD><<<blocks_for(d), kBlock, 0, s>>>(X, d, ld, row_index, f, group, out,
                                                                    gate, gate_n);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

#endif  // parts 5, 9, 11, 19, 20

#if BYZ_IN_PART(5)
int launch_median(const uint32_t *X, int64_t d, int64_t ld, const int32_t *row_index, int f,
                  uint32_t *out, const uint32_t *gate, int gate_n, hipStream_t s) {
    if (d == 0) return BYZ_OK;
    switch (f) {
        case 1: return launch_median_net<1>(X, d, ld, row_index, out, gate, gate_n, s);
        case 3: return launch_median_net<3>(X, d, ld, row_index, out, gate, gate_n, s);
        case 5: return launch_median_net<5>(X, d, ld, row_index, out, gate, gate_n, s);
        case 7: return launch_median_net<7>(X, d, ld, row_index, out, gate, gate_n, s);
        default: break;
    }
    // the paper's file counts exactly, any other odd f on the next generated size with spare wires
    if (f == 9) return launch_median_large<9, false>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f == 15) return launch_median_large<15, false>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f == 21) return launch_median_large<21, false>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f == 25) return launch_median_large<25, false>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f == 35) return launch_median_large<35, false>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f == 49) return launch_median_large<49, false>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 15) return launch_median_large<15, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 21) return launch_median_large<21, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 25) return launch_median_large<25, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 31) return launch_median_large<31, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 35) return launch_median_large<35, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 41) return launch_median_large<41, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 49) return launch_median_large<49, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 57) return launch_median_large<57, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 63) return launch_median_large<63, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 65) return launch_median_large<65, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 73) return launch_median_large<73, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f == 81) return launch_median_large<81, false>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 81) return launch_median_large<81, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 97) return byz_internal_launch_median_97(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 109) return byz_internal_launch_median_109(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f == 121) return launch_median_large<121, false>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 121) return launch_median_large<121, true>(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 137) return byz_internal_launch_median_137(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 153) return byz_internal_launch_median_153(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f == 169) return byz_internal_launch_median_169(X, d, ld, row_index, f, out, gate, gate_n, s);
    if (f <= 169) return byz_internal_launch_median_169_padded(X, d, ld, row_index, f, out, gate, gate_n, s);
    return byz_internal_launch_median_255_padded(X, d, ld, row_index, f, out, gate, gate_n, s);
}

#endif  // part 5

// Redone one word per thread up to kManyBlocks coordinates.
template <int F, int R, bool TRIM, int V, bool SLOTS>
void launch_decide(const uint32_t *X, int64_t d, int64_t ld, const int32_t *rows, AggWorkspace *ws, int n_slots,
                   int trim_b, int32_t *winner_replica, uint32_t *out, hipStream_t s) {
    if (V == 1 || d <= kManyBlocks)
        decide_kernel<F, R, TRIM, 1, SLOTS><<<blocks_for(d), kBlock, 0, s>>>(X, d, ld, rows, ws, n_slots, trim_b,
                                                                             winner_replica, out);
    else
        decide_kernel<F, R, TRIM, V, SLOTS><<<blocks_for((d + V - 1) / V), kBlock, 0, s>>>(
            X, d, ld, rows, ws, n_slots, trim_b, winner_replica, out);
}

// Calls without slots that decide in the blocks of the median, one launch for two; beyond, their many blocks would each
// decide for themselves in turn, and a fixed number of blocks that redo the output in rounds is slower at it than a block
// per tile ((25,3) 11.2 M 722 us a call that redoes its output, 702 in kernels of their own; (49,3) trimmed mean 4 M
// 576 and 515; 1 to 4 us less for calls that don't).  us a call, kernels of their own / this, in brackets redone: (9,3) 1 M 23.5 / 21.0
// (32.4 / 30.6), (25,3) 2 M 97.7 / 95.3 (133 / 131), (25,5) 0.6 M 56.0 / 52.7 (90.5 / 88.8), (49,7) 0.2 M 52.1 / 47.0 (65.5 / 59.0), (81,3)
// 0.5 M 85.0 / 81.4 (113 / 110); (121,3) 150000 57.5 / 54.5 (75.3 / 73.1), (169,3) 101.3 / 99.1 (129.5 / 130.7), but 300000 86.2 / 92.1
// and (121,3) 0.5 M 127 / 131 (172 / 179).  The trimmed mean of 49 files takes all registers with four words a thread ((49,3)
// 2 M redone 277 and 313), and decides here with one.
constexpr int decide_vec(int f, bool trim) { return f == 49 && trim ? 1 : gated_vec(f); }
constexpr bool decides_in_median(int f, bool trim, int64_t d) {
    if (decide_vec(f, trim) != gated_vec(f)) return d <= kManyBlocks;
    return d <= (int64_t)(f <= 81 ? 2048 : 768) * kBlock * gated_vec(f);
}

// The two kernels of a short call; *done stays false where the blocks have no room for their slots.
template <int F, int R, bool TRIM, int V, int BLOCK, int DV>
int launch_short_pair(const uint32_t *X, int64_t d, int64_t ld, const int32_t *rows, AggWorkspace *ws,
                      uint32_t *out, int trim_b, int32_t *winner_replica, bool *done, hipStream_t s) {
    const int64_t blocks = (d + (int64_t)V * BLOCK - 1) / ((int64_t)V * BLOCK);
    if (blocks > most_slots(F, R)) return BYZ_OK;
    int rc = byz_internal_profile_mark(0, s, "short_pass_kernel");
    if (rc != BYZ_OK) return rc;
    short_pass_kernel<F, R, TRIM, V, BLOCK><<<(unsigned)blocks, BLOCK, 0, s>>>(
        X, d, ld, rows, reinterpret_cast<uint32_t *>(ws->perm_off), trim_b, out);
    BYZ_HIP(hipGetLastError());
    rc = byz_internal_profile_mark(1, s);
    if (rc != BYZ_OK) return rc;
    // redone one word per thread up to kManyBlocks coordinates, where the wider form leaves CUs idle (as the gated
    // kernels of long calls).  us a call that redoes its output, four words / one: (49,7) d = 60001 median 50.9 /
    // 46.5, trimmed mean 57.4 / 49.9, (49,5) 100003 38.6 / 34.9 and 44.8 / 38.5, (35,5) 125003 34.6 / 32.8 and 39.4 / 35.7
    launch_decide<F, R, TRIM, DV, true>(X, d, ld, rows, ws, (int)blocks, trim_b, winner_replica, out, s);
    BYZ_HIP(hipGetLastError());
    *done = true;
    return BYZ_OK;
}

// Which block of the first kernel: the smallest whose slots fit, one word per thread while that is the faster
// form.  us a call, four kernels / two: 256 threads (25,3) d = 1003 15.3 / 9.1, 100003 18.3 / 12.1, (49,5) 20000
// 37.1 / 23.2, (169,3) 20000 65.8 / 37.1; 512 threads (49,3) 100000 24.7 / 16.8, (81,3) 86000 40.8 / 22.3, (49,7)
// 30000 45.1 / 38.5, (169,3) 46000 64.0 / 40.7.  Then up to 49 files: the long form's words per thread and 512
// threads for five and seven copies ((49,5) 145000 40.2 / 33.4, (25,5) 260000 33.7 / 24.5) and for the median of up
// to 25 files of three (1 M 55.9 / 50.8, 400000 25.9 / 22.7), two words for their trimmed mean (500000 31.1 /
// 27.5; four 41.0), 1024 threads of one word for 49 files of three (250000 37.4 / 29.0; 512 of two 50.4).  More
// files and two words per thread: (81,3) 140000 44.4 / 65.6, (63,7) 50000 54.2 / 56.8.  Fewer than 21 files of
// longer rows keep the four kernels: (15,3) 500000 20.7 / 39.3, (9,3) 17.6 / 22.9.  So do medians of (25,3) whose
// blocks are a little more than one a CU: 524288 coordinates 32.0 / 28.3, 525001 34.3 / 35.1 (off the cache lines
// 35.9 / 37.4), 600000 37.0 / 37.6 (38.0 / 39.6), 700001 39.7 / 39.8 (39.9 / 40.8), 786432 44.5 / 41.5 (44.7 / 42.4); on
// the far side of 2^20 there are no slots (1048581 63.5, with two kernels' 1048576 53.4).
constexpr int64_t kOneBlockPerCu = 256;
// Rows that one block holds take one kernel, where its CU can read them in about the time of a second launch: us a call,
// two kernels / one, among others: (25,3) d = 64 9.1 / 6.3, 512 8.8 / 6.3, 1024 8.7 to 10.0 / 8.5 (alone 21.6 / 22.3), trimmed mean
// 1003 8.9 / 9.5; (25,3) where the output is redone 500 9.6 / 7.6, 1003 9.8 / 10.6; (9,3) 1003 8.9 / 6.3; (21,3) trimmed mean 1000 8.9 / 8.3; (25,5) 500 12.6 / 12.5, 1003 12.3 / 17.0.  Up to 25
// files: more, a word per thread, take all registers 16 waves have, and are past the line from 300 coordinates on.
constexpr int64_t one_block_words(int r, bool trim) { return r == 3 && !trim ? 5 << 14 : 3 << 14; }
template <int F, int R, bool TRIM>
int launch_short(const uint32_t *X, int64_t d, int64_t ld, const int32_t *rows, AggWorkspace *ws,
                 uint32_t *out, int trim_b, int32_t *winner_replica, bool *done, hipStream_t s) {
    if (F < 21 && d > kManyBlocks) return BYZ_OK;
    if constexpr (F <= 25) {
        if (d <= kOneBlock && d * F * R <= one_block_words(R, TRIM)) {
            int rc = byz_internal_profile_mark(0, s, "one_block_kernel");
            if (rc != BYZ_OK) return rc;
            one_block_kernel<F, R, TRIM><<<1, (unsigned)((d + 63) / 64 * 64), 0, s>>>(X, d, ld, rows, ws, trim_b,
                                                                                      winner_replica, out);
            BYZ_HIP(hipGetLastError());
            *done = true;
            return byz_internal_profile_mark(1, s);
        }
    }
    int rc = launch_short_pair<F, R, TRIM, 1, kBlock, 1>(X, d, ld, rows, ws, out, trim_b, winner_replica, done, s);
    if (rc != BYZ_OK || *done) return rc;
    rc = launch_short_pair<F, R, TRIM, 1, 512, 1>(X, d, ld, rows, ws, out, trim_b, winner_replica, done, s);
    if (rc != BYZ_OK || *done) return rc;
    if constexpr (F >= 21 && F <= 49) {
        constexpr bool one_word = R == 3 && F > 25;
        constexpr int V = one_word ? 1 : (R == 3 && TRIM ? 2 : vec_for_pass(F, R, TRIM));
        if (F > 21 && V == 4 && d > kOneBlockPerCu * 512 * V && d <= kOneBlockPerCu * 4 / 3 * 512 * V) return BYZ_OK;
        rc = launch_short_pair<F, R, TRIM, V, one_word ? 1024 : 512, gated_vec(F)>(
            X, d, ld, rows, ws, out, trim_b, winner_replica, done, s);
    }
    return rc;
}

// Probe and single pass of a long call (WITH_TRIM, WITH_MEDIAN: see launch_fused).
template <int F, int R, bool WITH_TRIM, bool WITH_MEDIAN>
int launch_long_pass(const uint32_t *X, int64_t d, int64_t ld, const int32_t *rows, AggWorkspace *ws,
                     uint32_t *out, int probe_opts, int trim_b, hipStream_t s) {
    probe_kernel<F, R><<<1, kProbeThreads, 0, s>>>(X, d, ld, rows, ws, probe_opts);
    BYZ_HIP(hipGetLastError());
    int rc = byz_internal_profile_mark(0, s, "fused_kernel");
    if (rc != BYZ_OK) return rc;
    constexpr bool kShortToo = vec_for_pass(F, R, false) > 1;  // or the only width is one word already
    const int64_t one_block = (int64_t)kBlock * vec_for_pass(F, R, trim_b >= 0);
    [[maybe_unused]] const bool four =
        four_words_of_five(F, d, rows_on_lines(X, ld), (probe_opts & 1) != 0 && trim_b >= 0);
    if (kShortToo && d <= short_row(F, R) && (d <= kBlock || d > one_block)) {
        if constexpr (kShortToo) {
            if (trim_b < 0)
                fused_kernel<F, R, false, 1><<<blocks_for(d), kBlock, 0, s>>>(
                    X, d, ld, ws->perm_off, &ws->slots_per_file, ws, 0, out);
            else
                fused_kernel<F, R, true, 1><<<blocks_for(d), kBlock, 0, s>>>(
                    X, d, ld, ws->perm_off, &ws->slots_per_file, ws, trim_b, out);
        }
    } else if (trim_b < 0) {
        if constexpr (WITH_MEDIAN) {
            constexpr int V = vec_for_pass(F, R, false);
            if constexpr (R == 5 && F <= 49) {
                if (four) {
                    fused_kernel<F, R, false, 4><<<blocks_for((d + 3) / 4), kBlock, 0, s>>>(
                        X, d, ld, ws->perm_off, &ws->slots_per_file, ws, 0, out);
                    BYZ_HIP(hipGetLastError());
                    return byz_internal_profile_mark(1, s);
                }
            }
            fused_kernel<F, R, false, V><<<blocks_for((d + V - 1) / V), kBlock, 0, s>>>(
                X, d, ld, ws->perm_off, &ws->slots_per_file, ws, 0, out);
        }
    } else if constexpr (WITH_TRIM) {
        constexpr int V = vec_for_pass(F, R, true);
        if constexpr (R == 5 && F <= 49) {
            if (four) {
                fused_kernel<F, R, true, 4><<<blocks_for((d + 3) / 4), kBlock, 0, s>>>(
                    X, d, ld, ws->perm_off, &ws->slots_per_file, ws, trim_b, out);
                BYZ_HIP(hipGetLastError());
                return byz_internal_profile_mark(1, s);
            }
        }
        fused_kernel<F, R, true, V><<<blocks_for((d + V - 1) / V), kBlock, 0, s>>>(
            X, d, ld, ws->perm_off, &ws->slots_per_file, ws, trim_b, out);
    }
    BYZ_HIP(hipGetLastError());
    return byz_internal_profile_mark(1, s);
}

// WITH_TRIM = false / WITH_MEDIAN = false leave that variant of the kernel out (a shape whose two
// variants are compiled in different build parts)
template <int F, int R, bool WITH_TRIM = true, bool WITH_MEDIAN = true>
int launch_fused(const uint32_t *X, int64_t d, int64_t ld, const int32_t *rows, AggWorkspace *ws,
                 uint32_t *out, int probe_opts, int trim_b, int32_t *winner_replica, bool *done,
                 hipStream_t s) {
    if ((!WITH_TRIM && trim_b >= 0) || (!WITH_MEDIAN && trim_b < 0)) return BYZ_EINTERNAL;
    if ((probe_opts & 1) == 0) {
        int rc = BYZ_EINTERNAL;
        if (trim_b < 0) {
            if constexpr (WITH_MEDIAN) rc = launch_short<F, R, false>(X, d, ld, rows, ws, out, 0, winner_replica, done, s);
        } else if constexpr (WITH_TRIM) {
            rc = launch_short<F, R, true>(X, d, ld, rows, ws, out, trim_b, winner_replica, done, s);
        }
        if (rc != BYZ_OK || *done) return rc;
    }
    int rc = launch_long_pass<F, R, WITH_TRIM, WITH_MEDIAN>(X, d, ld, rows, ws, out, probe_opts, trim_b, s);
    // early-majority mode and longer rows decide in kernels of their own
    if (rc != BYZ_OK || (probe_opts & 1) != 0 || !decides_in_median(F, trim_b >= 0, d)) return rc;
    if (trim_b < 0) {
        if constexpr (WITH_MEDIAN && decides_in_median(F, false, 0))
            launch_decide<F, R, false, decide_vec(F, false), false>(X, d, ld, rows, ws, 0, 0, winner_replica, out, s);
    } else if constexpr (WITH_TRIM && decides_in_median(F, true, 0)) {
        launch_decide<F, R, true, decide_vec(F, true), false>(X, d, ld, rows, ws, 0, trim_b, winner_replica, out, s);
    }
    BYZ_HIP(hipGetLastError());
    *done = true;
    return BYZ_OK;
}

#if BYZ_IN_PART(6) || BYZ_IN_PART(8) || BYZ_IN_PART(10) || BYZ_IN_PART(14) || BYZ_IN_PART(15) || \
    BYZ_IN_PART(21) || BYZ_IN_PART(22) || BYZ_IN_PART(23)
template <int F, bool PAD>
int launch_trimmed_net(const uint32_t *X, int64_t d, int64_t ld, const int32_t *row_index, int f,
                       int b, uint32_t *O, const uint32_t *gate, int gate_n, hipStream_t s) {
    // fewer than nine rows are bound by the launch of their blocks too (f = 3, 0.4 / 2 M coordinates: 3.7 /
    // 9.6 us, one word per thread 4.2 / 12.0; f = 7, 131073: 3.5 and 2.8)
    constexpr bool few_rows = F == 9 && PAD;
    if constexpr (gated_vec(F) > 1 && (few_rows || !PAD)) {
        if (few_rows ? d > 2 * kManyBlocks : gate != nullptr && d > kManyBlocks) {
            constexpr int V = gated_vec(F);
            trimmed_mean_kernel<F, V, PAD><<<blocks_for((d + V - 1) / V), kBlock, 0, s>>>(
                X, d, ld, row_index, f, b, 0, O, gate, gate_n);
            BYZ_HIP(hipGetLastError());
            return BYZ_OK;
        }
    }
    // off the cache lines, as the median (4 M coordinates, us: f = 25 76.5 -> 72.3, 49 157 -> 152, 81 239 -> 232; above
    // 81 wires nothing is gained)
    const unsigned group = F <= 81 && d > kManyBlocks && !rows_on_lines(X, ld) ? 16 : 0;
    trimmed_mean_kernel<F, 1, PAD><<<blocks_for(d), kBlock, 0, s>>>(X, d, ld, row_index, f, b, group, O,
                                                                    gate, gate_n);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

#endif  // parts 6, 8, 10, 14, 15, 21..23

#if BYZ_IN_PART(6)
int launch_trimmed_mean(const uint32_t *X, int64_t d, int64_t ld, const int32_t *row_index, int f,
                        int b, uint32_t *O, const uint32_t *gate, int gate_n, hipStream_t s) {
    if (d == 0) return BYZ_OK;
    // the generated full-sort network of size f, else the next size with spare wires
    switch (f) {
        case 9: return launch_trimmed_net<9, false>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
        case 15: return launch_trimmed_net<15, false>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
        case 21: return launch_trimmed_net<21, false>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
        case 25: return launch_trimmed_net<25, false>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
        case 35: return launch_trimmed_net<35, false>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
        case 49: return launch_trimmed_net<49, false>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
        default: break;
    }
    if (f <= 9) return launch_trimmed_net<9, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 15) return launch_trimmed_net<15, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 21) return launch_trimmed_net<21, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 25) return launch_trimmed_net<25, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 31) return launch_trimmed_net<31, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 35) return launch_trimmed_net<35, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 41) return launch_trimmed_net<41, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 49) return launch_trimmed_net<49, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 57) return launch_trimmed_net<57, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 63) return byz_internal_launch_trimmed_mean_63(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 65) return byz_internal_launch_trimmed_mean_65(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 73) return launch_trimmed_net<73, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f == 81) return launch_trimmed_net<81, false>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 81) return launch_trimmed_net<81, true>(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 97) return byz_internal_launch_trimmed_mean_97(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 109) return byz_internal_launch_trimmed_mean_109(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 121) return byz_internal_launch_trimmed_mean_121(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 137) return byz_internal_launch_trimmed_mean_137(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 153) return byz_internal_launch_trimmed_mean_153(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f == 169) return byz_internal_launch_trimmed_mean_169(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    if (f <= 169)
        return byz_internal_launch_trimmed_mean_169_padded(X, d, ld, row_index, f, b, O, gate, gate_n, s);
    return byz_internal_launch_trimmed_mean_256_padded(X, d, ld, row_index, f, b, O, gate, gate_n, s);
}

#endif  // part 6

#if BYZ_IN_PART(0) || BYZ_IN_PART(12) || BYZ_IN_PART(13)
template <int F>
int launch_bulyan_net(const uint32_t *X, int64_t d, int64_t ld, const int32_t *selected_rows,
                      int theta, int beta, uint32_t *O, hipStream_t s) {
    constexpr int BLOCK = F > 49 ? 64 : kBlock;
    constexpr size_t lds = (size_t)F * BLOCK * 4;
    static_assert(lds <= 64 * 1024, "more than a kernel may use without asking");
    // off the cache lines (us, plain / in groups: f = 15 0.5 M 8.7 / 8.4, 3 M 36.1 / 34.9, 49 0.5 M 26.9 / 26.3, 1 M 47.1 / 46.4,
    // 65 1 M 77.8 / 73.7, 97 148 / 145, 127 269 / 264; but up to nine wires 3 M 22.4 / 24.3, 1 M 9.2 / 9.9)
    const unsigned group = F > 9 && d > kManyBlocks && !rows_on_lines(X, ld) ? (BLOCK == 64 ? kHalvesGroup : 16) : 0;
    bulyan_mean_kernel<F, BLOCK><<<(unsigned)((d + BLOCK - 1) / BLOCK), BLOCK, lds, s>>>(
        X, d, ld, selected_rows, theta, beta, group, O);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}
#endif

#if BYZ_IN_PART(0)

// (f, r) with a compiled single-pass kernel: MOLS / Ramanujan Case 1 (f = l^2: 9, 25, 49) with
// r = 3, 5 (and 7 for f = 49, which is also Ramanujan Case 2 with m = s = 7), the Ramanujan Case 2
// shapes f = m*s with r = s: (15,3), (21,3), (35,5), (65,5), (63,7), and MOLS over F_9, F_11 and
// F_13 with r = 3: (81,3), (121,3), (169,3)
bool has_fused(int f, int r) {
    return (f == 9 && r == 3) || (f == 25 && (r == 3 || r == 5)) ||
           (f == 49 && (r == 3 || r == 5 || r == 7)) || ((f == 15 || f == 21) && r == 3) ||
           (f == 35 && r == 5) || (f == 65 && r == 5) || (f == 63 && r == 7) ||
           ((f == 81 || f == 121 || f == 169) && r == 3);
}
// ... whose trimmed-mean variant is compiled as well: all of them
bool has_fused_trim(int f, int r) { return has_fused(f, r); }

// More than 169 files of three copies, rows of four rounds of resident blocks or more: one pass with the files
// split over two waves.  Shorter rows are voted on faster with the files dealt out to more blocks (f = 255,
// us a call, vote and median / one pass: d = 10000 34 / 54, 100000 89 / 91, 140000 114 / 121, 200000 151 / 150,
// 262145 218 / 172; f = 195 200000 121 / 129, 262145 167 / 150; f = 171 200000 100 / 101, 262145 141 / 117).
// A file without a majority that makes the pass feed a loser's values costs the median on top: f = 171 262200
// coordinates 125 (vote and median) / 159, trimmed mean 158 / 224, 1 M 482 / 509 and 606 / 740, 2.5 M 1176 / 1149 and 1454 / 1684;
// f = 255 188 / 245, 219 / 303, 749 / 797, 868 / 997.  As everywhere, who does that gives up the vote in those files.
bool takes_halves_pass(int f, int r, int64_t d) {
    return f > 169 && f <= 255 && r == 3 && d >= ((int64_t)1 << 18);
}

int check_common(const void *copies, int64_t d, int64_t ld, const void *rows, int f, int r) {
    if (copies == nullptr || rows == nullptr) return BYZ_EINVAL;
    if (d < 0 || ld < d || d > kMaxCoords) return BYZ_EINVAL;
    if (f < 1 || f > kWide) return BYZ_EINVAL;
    if (r < 3 || r > BYZ_MAX_R || (r % 2) == 0) return BYZ_EINVAL;
    return BYZ_OK;
}

#endif  // part 0

}  // namespace

// --------------------------------------- median and trimmed-mean launchers, a part each

#if BYZ_IN_PART(5)
int byz_internal_launch_median(const void *X, long long d, long long ld, const int *row_index,
                               int f, void *out, const void *gate, int gate_n, void *stream) {
    return launch_median(static_cast<const uint32_t *>(X), d, ld, row_index, f,
                         static_cast<uint32_t *>(out), static_cast<const uint32_t *>(gate), gate_n,
                         (hipStream_t)stream);
}
#endif

// second phase of Bulyan on the larger networks: 49 < theta <= 81 and 81 < theta <= 128
#if BYZ_IN_PART(12)
int byz_internal_launch_bulyan_mean_81(const void *X, long long d, long long ld,
                                       const int *selected_rows, int theta, int beta, void *out,
                                       void *stream) {
    const uint32_t *x = static_cast<const uint32_t *>(X);
    uint32_t *o = static_cast<uint32_t *>(out);
    hipStream_t s = (hipStream_t)stream;
    if (theta <= 57) return launch_bulyan_net<57>(x, d, ld, selected_rows, theta, beta, o, s);
    if (theta <= 63) return launch_bulyan_net<63>(x, d, ld, selected_rows, theta, beta, o, s);
    if (theta <= 65) return launch_bulyan_net<65>(x, d, ld, selected_rows, theta, beta, o, s);
    if (theta <= 73) return launch_bulyan_net<73>(x, d, ld, selected_rows, theta, beta, o, s);
    return launch_bulyan_net<81>(x, d, ld, selected_rows, theta, beta, o, s);
}
#endif
#if BYZ_IN_PART(13)
int byz_internal_launch_bulyan_mean_137(const void *X, long long d, long long ld,
                                        const int *selected_rows, int theta, int beta, void *out,
                                        void *stream) {
    const uint32_t *x = static_cast<const uint32_t *>(X);
    uint32_t *o = static_cast<uint32_t *>(out);
    hipStream_t s = (hipStream_t)stream;
    if (theta <= 97) return launch_bulyan_net<97>(x, d, ld, selected_rows, theta, beta, o, s);
    if (theta <= 109) return launch_bulyan_net<109>(x, d, ld, selected_rows, theta, beta, o, s);
    if (theta <= 121) return launch_bulyan_net<121>(x, d, ld, selected_rows, theta, beta, o, s);
    return launch_bulyan_net<137>(x, d, ld, selected_rows, theta, beta, o, s);
}
#endif

// the larger networks, one or two to a build part: byz_internal_launch_median_<n> and
// byz_internal_launch_trimmed_mean_<n> run the n-wire network on n rows or, padded, on fewer
#define BYZ_DEFINE_MEDIAN(name, wires, pad)                                                      \
    int byz_internal_launch_median_##name(const void *X, long long d, long long ld,              \
                                          const int *row_index, int f, void *out,                \
                                          const void *gate, int gate_n, void *stream) {          \
        return launch_median_large<wires, pad>(static_cast<const uint32_t *>(X), d, ld,          \
                                               row_index, f, static_cast<uint32_t *>(out),       \
                                               static_cast<const uint32_t *>(gate), gate_n,      \
                                               (hipStream_t)stream);                             \
    }
#define BYZ_DEFINE_TRIMMED_MEAN(name, wires, pad)                                                \
    int byz_internal_launch_trimmed_mean_##name(const void *X, long long d, long long ld,        \
                                                const int *row_index, int f, int b, void *out,   \
                                                const void *gate, int gate_n, void *stream) {    \
        return launch_trimmed_net<wires, pad>(static_cast<const uint32_t *>(X), d, ld,           \
                                              row_index, f, b, static_cast<uint32_t *>(out),     \
                                              static_cast<const uint32_t *>(gate), gate_n,       \
                                              (hipStream_t)stream);                              \
    }
#if BYZ_IN_PART(8)
BYZ_DEFINE_TRIMMED_MEAN(169, 169, false)
#endif
#if BYZ_IN_PART(9)
BYZ_DEFINE_MEDIAN(169, 169, false)
#endif
#if BYZ_IN_PART(10)
BYZ_DEFINE_TRIMMED_MEAN(169_padded, 169, true)
#endif
#if BYZ_IN_PART(11)
BYZ_DEFINE_MEDIAN(169_padded, 169, true)
#endif
#if BYZ_IN_PART(14)
BYZ_DEFINE_TRIMMED_MEAN(63, 63, true)
#endif
#if BYZ_IN_PART(15)
BYZ_DEFINE_TRIMMED_MEAN(65, 65, true)
#endif
#if BYZ_IN_PART(19)
BYZ_DEFINE_MEDIAN(97, 97, true)
BYZ_DEFINE_MEDIAN(109, 109, true)
#endif
#if BYZ_IN_PART(20)
BYZ_DEFINE_MEDIAN(137, 137, true)
BYZ_DEFINE_MEDIAN(153, 153, true)
#endif
#if BYZ_IN_PART(21)
BYZ_DEFINE_TRIMMED_MEAN(97, 97, true)
BYZ_DEFINE_TRIMMED_MEAN(109, 109, true)
#endif
#if BYZ_IN_PART(22)
BYZ_DEFINE_TRIMMED_MEAN(121, 121, true)
BYZ_DEFINE_TRIMMED_MEAN(137, 137, true)
#endif
#if BYZ_IN_PART(23)
BYZ_DEFINE_TRIMMED_MEAN(153, 153, true)
#endif

// more than 169 rows: the two-wave kernels, median for 169 < f <= 255, trimmed mean for
// 169 < f <= 256 (it also takes even f); a build part each
#if BYZ_IN_PART(16)
int byz_internal_launch_median_255_padded(const void *X, long long d, long long ld,
                                          const int *row_index, int f, void *out, const void *gate,
                                          int gate_n, void *stream) {
    if (d <= 0) return BYZ_OK;
    if (f <= 128 || f > 255) return BYZ_EINTERNAL;
    const unsigned g = (unsigned)((d + 63) / 64);
    const uint32_t *x = static_cast<const uint32_t *>(X), *gt = static_cast<const uint32_t *>(gate);
    uint32_t *o = static_cast<uint32_t *>(out);
    hipStream_t s = (hipStream_t)stream;
    // the smallest pair of halves that holds f rows; off the lines neighbours go to one XCD (1 M coordinates, us:
    // f = 171 161 -> 136, 191 178 -> 144, 223 217 -> 190, 255 252 -> 223)
    const bool together = d > kManyBlocks && !rows_on_lines(X, ld);
#define BYZ_LAUNCH_HALVES(H)                                                                          \
    do {                                                                                              \
        if (together)                                                                                 \
            median_halves_kernel<H, kHalvesGroup><<<g, 128, 0, s>>>(x, d, ld, row_index, f, o, gt, gate_n); \
        else                                                                                          \
            median_halves_kernel<H, 0><<<g, 128, 0, s>>>(x, d, ld, row_index, f, o, gt, gate_n);      \
    } while (0)
    if (f <= 2 * 96 - 1)
        BYZ_LAUNCH_HALVES(96);
    else if (f <= 2 * 112 - 1)
        BYZ_LAUNCH_HALVES(112);
    else
        BYZ_LAUNCH_HALVES(128);
#undef BYZ_LAUNCH_HALVES
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}
#endif
#if BYZ_IN_PART(17)
int byz_internal_launch_trimmed_mean_256_padded(const void *X, long long d, long long ld,
                                                const int *row_index, int f, int b, void *out,
                                                const void *gate, int gate_n, void *stream) {
    if (d <= 0) return BYZ_OK;
    if (f <= 128 || f > 256) return BYZ_EINTERNAL;
    const unsigned g = (unsigned)((d + 63) / 64);
    const uint32_t *x = static_cast<const uint32_t *>(X), *gt = static_cast<const uint32_t *>(gate);
    uint32_t *o = static_cast<uint32_t *>(out);
    hipStream_t s = (hipStream_t)stream;
    // the smallest pair of halves that holds f rows
    if (f <= 2 * 96)
        trimmed_halves_kernel<96><<<g, 128, 0, s>>>(x, d, ld, row_index, f, b, o, gt, gate_n);
    else if (f <= 2 * 112)
        trimmed_halves_kernel<112><<<g, 128, 0, s>>>(x, d, ld, row_index, f, b, o, gt, gate_n);
    else
        trimmed_halves_kernel<128><<<g, 128, 0, s>>>(x, d, ld, row_index, f, b, o, gt, gate_n);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}
#endif

#if BYZ_IN_PART(24) || BYZ_IN_PART(25)
namespace {
template <bool TRIM>
int launch_halves_pass(const uint32_t *X, int64_t d, int64_t ld, const int32_t *rows, int f, AggWorkspace *ws,
                       uint32_t *out, int trim_b, hipStream_t s) {
    lay_out_rows_kernel<<<1, kWide, 0, s>>>(rows, f, 3, ld, ws);
    BYZ_HIP(hipGetLastError());
    int rc = byz_internal_profile_mark(0, s, "fused_halves_kernel");
    if (rc != BYZ_OK) return rc;
    const unsigned g = (unsigned)((d + 63) / 64);
    const unsigned group = rows_on_lines(X, ld) ? 0 : kHalvesGroup;
    if (f <= 2 * 96 - 1)
        fused_halves_kernel<96, TRIM><<<g, 128, 0, s>>>(X, d, ws->perm_off, ws, f, trim_b, group, out);
    else if (f <= 2 * 112 - 1)
        fused_halves_kernel<112, TRIM><<<g, 128, 0, s>>>(X, d, ws->perm_off, ws, f, trim_b, group, out);
    else
        fused_halves_kernel<128, TRIM><<<g, 128, 0, s>>>(X, d, ws->perm_off, ws, f, trim_b, group, out);
    BYZ_HIP(hipGetLastError());
    return byz_internal_profile_mark(1, s);
}
}  // namespace
#define BYZ_DEFINE_HALVES_PASS(name, trim)                                                        \
    int byz_internal_launch_##name##_halves_pass(const void *X, long long d, long long ld,        \
                                                 const int *rows, int f, void *ws, void *out,     \
                                                 int trim_b, void *stream) {                      \
        return launch_halves_pass<trim>(static_cast<const uint32_t *>(X), d, ld, rows, f,         \
                                        static_cast<AggWorkspace *>(ws),                          \
                                        static_cast<uint32_t *>(out), trim_b, (hipStream_t)stream); \
    }
#if BYZ_IN_PART(24)
BYZ_DEFINE_HALVES_PASS(median, false)
#endif
#if BYZ_IN_PART(25)
BYZ_DEFINE_HALVES_PASS(trimmed, true)
#endif
#endif

#if BYZ_IN_PART(6)
int byz_internal_launch_trimmed_mean(const void *X, long long d, long long ld,
                                     const int *row_index, int f, int b, void *out,
                                     const void *gate, int gate_n, void *stream) {
    return launch_trimmed_mean(static_cast<const uint32_t *>(X), d, ld, row_index, f, b,
                               static_cast<uint32_t *>(out), static_cast<const uint32_t *>(gate),
                               gate_n, (hipStream_t)stream);
}
#endif

// ------------------------------------------------- single-pass launchers, one group per part

#if BYZ_IN_PART(1)
int byz_internal_launch_single_pass_1(int f, int r, const void *X, long long d, long long ld,
                                      const int *rows, void *ws, void *out, int probe_opts, int trim_b,
                                      int *winner_replica, bool *done, void *stream) {
    const uint32_t *x = static_cast<const uint32_t *>(X);
    AggWorkspace *w = static_cast<AggWorkspace *>(ws);
    uint32_t *o = static_cast<uint32_t *>(out);
    hipStream_t s = (hipStream_t)stream;
    if (f == 9 && r == 3) return launch_fused<9, 3>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    if (f == 15 && r == 3) return launch_fused<15, 3>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    if (f == 21 && r == 3) return launch_fused<21, 3>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    if (f == 25 && r == 3) return launch_fused<25, 3>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    if (f == 25 && r == 5) return launch_fused<25, 5>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    if (f == 35 && r == 5) return launch_fused<35, 5>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    return BYZ_EINTERNAL;
}
#endif

#if BYZ_IN_PART(2)
int byz_internal_launch_single_pass_2(int f, int r, const void *X, long long d, long long ld,
                                      const int *rows, void *ws, void *out, int probe_opts, int trim_b,
                                      int *winner_replica, bool *done, void *stream) {
    const uint32_t *x = static_cast<const uint32_t *>(X);
    AggWorkspace *w = static_cast<AggWorkspace *>(ws);
    uint32_t *o = static_cast<uint32_t *>(out);
    hipStream_t s = (hipStream_t)stream;
    if (f == 49 && r == 3) return launch_fused<49, 3>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    if (f == 49 && r == 5) return launch_fused<49, 5>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    if (f == 49 && r == 7) return launch_fused<49, 7>(x, d, ld, rows, w, o, probe_opts, trim_b, winner_replica, done, s);
    return BYZ_EINTERNAL;
}
#endif

#if BYZ_IN_PART(3)
int byz_internal_launch_single_pass_3(int f, int r, const void *X, long long d, long long ld,
                                      const int *rows, void *ws, void *out, int probe_opts, int trim_b,
                                      int *winner_replica, bool *done, void *stream) {
    if (f == 81 && r == 3)
        return launch_fused<81, 3>(static_cast<const uint32_t *>(X), d, ld, rows,
                                   static_cast<AggWorkspace *>(ws), static_cast<uint32_t *>(out),
                                   probe_opts, trim_b, winner_replica, done, (hipStream_t)stream);
    return BYZ_EINTERNAL;
}
#endif

#if BYZ_IN_PART(4)
int byz_internal_launch_single_pass_4(int f, int r, const void *X, long long d, long long ld,
                                      const int *rows, void *ws, void *out, int probe_opts, int trim_b,
                                      int *winner_replica, bool *done, void *stream) {
    if (f == 121 && r == 3)
        return launch_fused<121, 3>(static_cast<const uint32_t *>(X), d, ld, rows,
                                    static_cast<AggWorkspace *>(ws), static_cast<uint32_t *>(out),
                                    probe_opts, trim_b, winner_replica, done, (hipStream_t)stream);
    return BYZ_EINTERNAL;
}
#endif

#if BYZ_IN_PART(7)
int byz_internal_launch_single_pass_5(int f, int r, const void *X, long long d, long long ld,
                                      const int *rows, void *ws, void *out, int probe_opts, int trim_b,
                                      int *winner_replica, bool *done, void *stream) {
    if (f == 169 && r == 3)
        return launch_fused<169, 3, false>(static_cast<const uint32_t *>(X), d, ld, rows,
                                    static_cast<AggWorkspace *>(ws), static_cast<uint32_t *>(out),
                                    probe_opts, trim_b, winner_replica, done, (hipStream_t)stream);
    return BYZ_EINTERNAL;
}
#endif

#if BYZ_IN_PART(18)
// (169, 3) with the trimmed mean: the widest sorting network in the single pass, a part of its own
int byz_internal_launch_single_pass_8(int f, int r, const void *X, long long d, long long ld,
                                      const int *rows, void *ws, void *out, int probe_opts, int trim_b,
                                      int *winner_replica, bool *done, void *stream) {
    if (f == 169 && r == 3)
        return launch_fused<169, 3, true, false>(static_cast<const uint32_t *>(X), d, ld, rows,
                                    static_cast<AggWorkspace *>(ws), static_cast<uint32_t *>(out),
                                    probe_opts, trim_b, winner_replica, done, (hipStream_t)stream);
    return BYZ_EINTERNAL;
}
#endif

#if BYZ_IN_PART(14)
int byz_internal_launch_single_pass_6(int f, int r, const void *X, long long d, long long ld,
                                      const int *rows, void *ws, void *out, int probe_opts, int trim_b,
                                      int *winner_replica, bool *done, void *stream) {
    if (f == 63 && r == 7)
        return launch_fused<63, 7>(static_cast<const uint32_t *>(X), d, ld, rows,
                                    static_cast<AggWorkspace *>(ws), static_cast<uint32_t *>(out),
                                    probe_opts, trim_b, winner_replica, done, (hipStream_t)stream);
    return BYZ_EINTERNAL;
}
#endif

#if BYZ_IN_PART(15)
int byz_internal_launch_single_pass_7(int f, int r, const void *X, long long d, long long ld,
                                      const int *rows, void *ws, void *out, int probe_opts, int trim_b,
                                      int *winner_replica, bool *done, void *stream) {
    if (f == 65 && r == 5)
        return launch_fused<65, 5>(static_cast<const uint32_t *>(X), d, ld, rows,
                                    static_cast<AggWorkspace *>(ws), static_cast<uint32_t *>(out),
                                    probe_opts, trim_b, winner_replica, done, (hipStream_t)stream);
    return BYZ_EINTERNAL;
}
#endif

#if BYZ_IN_PART(0)

// ---------------------------------------------------------------------------- C-ABI

// which: 0 = before (kernel: its name), 1 = after the dominant kernel of an aggregation on `stream`
int byz_internal_profile_mark(int which, void *stream, const char *kernel) {
    if (g_prof.count >= g_prof.capacity) return BYZ_OK;
    if (which == 0) {
        g_prof.kernel = kernel;
        BYZ_HIP(hipEventRecord(g_prof.start[g_prof.count], (hipStream_t)stream));
    } else {
        BYZ_HIP(hipEventRecord(g_prof.stop[g_prof.count], (hipStream_t)stream));
        ++g_prof.count;
    }
    return BYZ_OK;
}

int byz_internal_launch_bulyan_mean(const float *rows_base, long long d, long long ld,
                                    const int *selected_rows_dev, int f, int theta, int beta,
                                    float *out, void *stream) {
    if (d == 0) return BYZ_OK;
    if (f < 1 || f > BYZ_MAX_F_KRUM || theta < 1 || theta > f || (theta % 2) == 0 || beta < 1 ||
        beta > theta)
        return BYZ_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const uint32_t *X = reinterpret_cast<const uint32_t *>(rows_base);
    uint32_t *O = reinterpret_cast<uint32_t *>(out);
    // the smallest generated network that holds the theta chosen rows
    if (theta <= 9) return launch_bulyan_net<9>(X, d, ld, selected_rows_dev, theta, beta, O, s);
    if (theta <= 15) return launch_bulyan_net<15>(X, d, ld, selected_rows_dev, theta, beta, O, s);
    if (theta <= 21) return launch_bulyan_net<21>(X, d, ld, selected_rows_dev, theta, beta, O, s);
    if (theta <= 25) return launch_bulyan_net<25>(X, d, ld, selected_rows_dev, theta, beta, O, s);
    if (theta <= 31) return launch_bulyan_net<31>(X, d, ld, selected_rows_dev, theta, beta, O, s);
    if (theta <= 35) return launch_bulyan_net<35>(X, d, ld, selected_rows_dev, theta, beta, O, s);
    if (theta <= 41) return launch_bulyan_net<41>(X, d, ld, selected_rows_dev, theta, beta, O, s);
    if (theta <= 49) return launch_bulyan_net<49>(X, d, ld, selected_rows_dev, theta, beta, O, s);
    if (theta <= 81)
        return byz_internal_launch_bulyan_mean_81(X, d, ld, selected_rows_dev, theta, beta, O, s);
    return byz_internal_launch_bulyan_mean_137(X, d, ld, selected_rows_dev, theta, beta, O, s);
}

extern "C" int byz_last_hip_error(void) { return g_last_hip_error; }

void byz_internal_set_hip_error(int code) { g_last_hip_error = code; }

extern "C" int byz_vote(const float *copies, int64_t d, int64_t ld, const int32_t *file_rows_dev,
                        int f, int r, int32_t *winner_replica, int32_t *winner_row,
                        uint32_t *pair_neq, void *stream) {
    int rc = check_common(copies, d, ld, file_rows_dev, f, r);
    if (rc != BYZ_OK) return rc;
    if (winner_replica == nullptr || winner_row == nullptr || pair_neq == nullptr)
        return BYZ_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const uint32_t *X = reinterpret_cast<const uint32_t *>(copies);
    fill_u32_kernel<<<1, kWide, 0, s>>>(pair_neq, f, 0u);
    BYZ_HIP(hipGetLastError());
    if (d > 0) {
        rc = launch_vote_pairs_r(r, X, d, ld, file_rows_dev, f, pair_neq, nullptr, 0, nullptr, s);
        if (rc != BYZ_OK) return rc;
    }
    vote_decide_kernel<<<1, kWide, 0, s>>>(pair_neq, file_rows_dev, f, r, winner_replica,
                                               winner_row);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

extern "C" int byz_vote_tolerant(const float *copies, int64_t d, int64_t ld,
                                 const int32_t *file_rows_dev, int f, int r, float atol, float rtol,
                                 int32_t *winner_replica, int32_t *winner_row, uint32_t *pair_far,
                                 void *stream) {
    int rc = check_common(copies, d, ld, file_rows_dev, f, r);
    if (rc != BYZ_OK) return rc;
    if (winner_replica == nullptr || winner_row == nullptr || pair_far == nullptr)
        return BYZ_EINVAL;
    if (!(atol >= 0.0f) || !(rtol >= 0.0f)) return BYZ_EINVAL;  // also rejects NaN
    hipStream_t s = (hipStream_t)stream;
    const uint32_t *X = reinterpret_cast<const uint32_t *>(copies);
    fill_u32_kernel<<<1, kWide, 0, s>>>(pair_far, f, 0u);
    BYZ_HIP(hipGetLastError());
    if (d > 0) {
        rc = launch_vote_pairs_tolerant(r, X, d, ld, file_rows_dev, f, atol, rtol, pair_far, s);
        if (rc != BYZ_OK) return rc;
    }
    vote_decide_kernel<<<1, kWide, 0, s>>>(pair_far, file_rows_dev, f, r, winner_replica,
                                           winner_row);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

extern "C" int byz_median(const float *rows_base, int64_t d, int64_t ld,
                          const int32_t *row_index_dev, int f, float *out, void *stream) {
    if (rows_base == nullptr || row_index_dev == nullptr || (out == nullptr && d > 0))
        return BYZ_EINVAL;
    if (d < 0 || ld < d || d > kMaxCoords) return BYZ_EINVAL;
    if (f < 1 || f > kWide) return BYZ_EINVAL;
    if ((f % 2) == 0) return BYZ_EUNSUPPORTED;
    return byz_internal_launch_median(rows_base, d, ld, row_index_dev, f, out, nullptr, 0, stream);
}

extern "C" int byz_trimmed_mean(const float *rows_base, int64_t d, int64_t ld,
                                const int32_t *row_index_dev, int f, int b, float *out,
                                void *stream) {
    if (rows_base == nullptr || row_index_dev == nullptr || (out == nullptr && d > 0))
        return BYZ_EINVAL;
    if (d < 0 || ld < d || d > kMaxCoords) return BYZ_EINVAL;
    if (f < 1 || f > kWide || b < 0 || 2 * b >= f) return BYZ_EINVAL;
    if (d == 0) return BYZ_OK;
    return byz_internal_launch_trimmed_mean(rows_base, d, ld, row_index_dev, f, b, out, nullptr, 0,
                                            stream);
}

extern "C" size_t byz_aggregate_workspace_bytes(int f, int r) {
    if (f < 1 || f > kWide || r < 3 || r > BYZ_MAX_R || (r % 2) == 0) return 0;
    return sizeof(AggWorkspace);
}

extern "C" int byz_aggregate_has_single_pass(int f, int r) { return has_fused(f, r) ? 1 : 0; }

// byz_aggregate_opts after its workspace has been settled: validates the rest and enqueues
// the launches.  ws is device memory of sizeof(AggWorkspace) bytes, 256-byte aligned.
static int aggregate_on_workspace(const float *copies, int64_t d, int64_t ld,
                                  const int32_t *file_rows_dev, int f, int r, float *out,
                                  int32_t *winner_replica, AggWorkspace *ws, unsigned flags,
                                  void *stream) {
    if ((flags & ~(unsigned)(BYZ_AGG_EARLY_MAJORITY | BYZ_AGG_TRIMMED_MEAN | 0xFFFFFF00u)) != 0)
        return BYZ_EINVAL;
    // what the probe needs to know: bit 0 early-majority mode, bits 16..31 the sample shift
    const int probe_opts = (int)((flags & BYZ_AGG_EARLY_MAJORITY) | (flags & 0xFFFF0000u));
    // trim_b < 0: median; otherwise trimmed mean dropping trim_b values at each end
    const int trim_b = (flags & BYZ_AGG_TRIMMED_MEAN) != 0 ? (int)((flags >> 8) & 0xFFu) : -1;
    if (trim_b < 0 && (flags & 0xFF00u) != 0) return BYZ_EINVAL;
    if (trim_b >= 0 && 2 * trim_b >= f) return BYZ_EINVAL;
    int rc = check_common(copies, d, ld, file_rows_dev, f, r);
    if (rc != BYZ_OK) return rc;
    if ((out == nullptr && d > 0) || ws == nullptr) return BYZ_EINVAL;
    if ((f % 2) == 0) return BYZ_EUNSUPPORTED;
    hipStream_t s = (hipStream_t)stream;
    const uint32_t *X = reinterpret_cast<const uint32_t *>(copies);
    uint32_t *O = reinterpret_cast<uint32_t *>(out);

    if (takes_halves_pass(f, r, d)) {
        rc = trim_b >= 0
                 ? byz_internal_launch_trimmed_halves_pass(X, d, ld, file_rows_dev, f, ws, O, trim_b, s)
                 : byz_internal_launch_median_halves_pass(X, d, ld, file_rows_dev, f, ws, O, trim_b, s);
        if (rc != BYZ_OK) return rc;
        single_pass_decide_kernel<<<1, kWide, 0, s>>>(ws, file_rows_dev, f, r, winner_replica, 1);
        BYZ_HIP(hipGetLastError());
        if (trim_b >= 0)
            return byz_internal_launch_trimmed_mean(X, d, ld, ws->winner_row, f, trim_b, O,
                                                    &ws->need_median, 1, s);
        return byz_internal_launch_median(X, d, ld, ws->winner_row, f, O, &ws->need_median, 1, s);
    }
    if (!has_fused(f, r) || d < kVec || (trim_b >= 0 && !has_fused_trim(f, r))) {
        // two-step path, unconditionally: vote, then median over the winners
        reset_workspace_kernel<<<1, kWide, 0, s>>>(ws, (uint32_t)BYZ_PATH_TWO_STEP);
        BYZ_HIP(hipGetLastError());
        if (d > 0) {
            rc = byz_internal_profile_mark(0, s, "vote_pairs_kernel");
            if (rc != BYZ_OK) return rc;
            rc = launch_vote_pairs_r(r, X, d, ld, file_rows_dev, f, ws->pair_neq, nullptr, 0, nullptr, s);
            if (rc != BYZ_OK) return rc;
            rc = byz_internal_profile_mark(1, s);
            if (rc != BYZ_OK) return rc;
        }
        vote_decide_kernel<<<1, kWide, 0, s>>>(ws->pair_neq, file_rows_dev, f, r, winner_replica,
                                               ws->winner_row);
        BYZ_HIP(hipGetLastError());
        if (trim_b >= 0)
            return byz_internal_launch_trimmed_mean(X, d, ld, ws->winner_row, f, trim_b, O, nullptr,
                                                    0, s);
        return byz_internal_launch_median(X, d, ld, ws->winner_row, f, O, nullptr, 0, s);
    }

    // probe -> single pass -> decision (one block) -> median, which returns at once unless the
    // decision found a file of which some wave fed a copy that is not the winner's.  Early-majority mode adds the
    // gated vote kernel and its decision between the two, for the files whose r' copies differ.
    // Where the blocks of the median are few they decide for themselves (decides_in_median); short rows
    // take two kernels instead of all that, rows that one block holds one.
    bool done = false;
    if (f == 169 && trim_b >= 0)
        rc = byz_internal_launch_single_pass_8(f, r, X, d, ld, file_rows_dev, ws, O, probe_opts, trim_b,
                                                 winner_replica, &done, s);
    else if (f == 169)
        rc = byz_internal_launch_single_pass_5(f, r, X, d, ld, file_rows_dev, ws, O, probe_opts, trim_b,
                                                 winner_replica, &done, s);
    else if (f == 121)
        rc = byz_internal_launch_single_pass_4(f, r, X, d, ld, file_rows_dev, ws, O, probe_opts, trim_b,
                                                 winner_replica, &done, s);
    else if (f == 81)
        rc = byz_internal_launch_single_pass_3(f, r, X, d, ld, file_rows_dev, ws, O, probe_opts, trim_b,
                                                 winner_replica, &done, s);
    else if (f == 63)
        rc = byz_internal_launch_single_pass_6(f, r, X, d, ld, file_rows_dev, ws, O, probe_opts, trim_b,
                                                 winner_replica, &done, s);
    else if (f == 65)
        rc = byz_internal_launch_single_pass_7(f, r, X, d, ld, file_rows_dev, ws, O, probe_opts, trim_b,
                                                 winner_replica, &done, s);
    else if (f == 49)
        rc = byz_internal_launch_single_pass_2(f, r, X, d, ld, file_rows_dev, ws, O, probe_opts, trim_b,
                                                 winner_replica, &done, s);
    else
        rc = byz_internal_launch_single_pass_1(f, r, X, d, ld, file_rows_dev, ws, O, probe_opts, trim_b,
                                                 winner_replica, &done, s);
    if (rc != BYZ_OK || done) return rc;
    single_pass_decide_kernel<<<1, kWide, 0, s>>>(ws, file_rows_dev, f, r, winner_replica, 0);
    BYZ_HIP(hipGetLastError());
    if ((flags & BYZ_AGG_EARLY_MAJORITY) != 0) {
        rc = launch_vote_pairs_r(r, X, d, ld, file_rows_dev, f, ws->pair_neq, &ws->need_revote, 1,
                                 ws->revote_file, s);
        if (rc != BYZ_OK) return rc;
        revote_decide_kernel<<<1, kWide, 0, s>>>(ws, file_rows_dev, f, r, winner_replica);
        BYZ_HIP(hipGetLastError());
    }
    if (trim_b >= 0)
        return byz_internal_launch_trimmed_mean(X, d, ld, ws->winner_row, f, trim_b, O,
                                                &ws->need_median, 1, s);
    return byz_internal_launch_median(X, d, ld, ws->winner_row, f, O, &ws->need_median, 1, s);
}

extern "C" int byz_aggregate_opts(const float *copies, int64_t d, int64_t ld,
                                  const int32_t *file_rows_dev, int f, int r, float *out,
                                  int32_t *winner_replica, void *workspace, size_t workspace_bytes,
                                  unsigned flags, void *stream) {
    if (workspace == nullptr || ((uintptr_t)workspace & 255u) != 0) return BYZ_EINVAL;
    // the reasons that come before "workspace too small" keep their codes
    const int rc = check_common(copies, d, ld, file_rows_dev, f, r);
    if (rc != BYZ_OK) return rc;
    if (workspace_bytes < sizeof(AggWorkspace)) return BYZ_ENOMEM;
    return aggregate_on_workspace(copies, d, ld, file_rows_dev, f, r, out, winner_replica,
                                  reinterpret_cast<AggWorkspace *>(workspace), flags, stream);
}

extern "C" int byz_aggregate(const float *copies, int64_t d, int64_t ld,
                             const int32_t *file_rows_dev, int f, int r, float *out,
                             int32_t *winner_replica, void *workspace, size_t workspace_bytes,
                             void *stream) {
    return byz_aggregate_opts(copies, d, ld, file_rows_dev, f, r, out, winner_replica, workspace,
                              workspace_bytes, 0u, stream);
}

// Scratch of byz_aggregate_static: one AggWorkspace per GPU, part of the loaded code object
// (so it is there without any allocation) and held until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress; what the kernels get is the device
// address that call returns, looked up once per device.
constexpr size_t kStaticScratchBytes = 24 * 1024;
static_assert(sizeof(AggWorkspace) <= kStaticScratchBytes, "byz_aggregate_static's scratch");
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static std::atomic<void *> g_scratch_ptr[kMaxDevices];

extern "C" int byz_aggregate_static(const float *copies, int64_t d, int64_t ld,
                                    const int32_t *file_rows_dev, int f, int r, float *out,
                                    int32_t *winner_replica, unsigned flags, void *stream) {
    // sizes first: what the fixed scratch cannot hold is refused before anything else happens
    if (f > kWide || r > BYZ_MAX_R) return BYZ_ENOMEM;
    int dev = -1;
    BYZ_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return BYZ_EUNSUPPORTED;
    void *ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (ptr == nullptr) {
        // first call on this device (which is current): every GPU has its own copy of the array
        BYZ_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (ptr == nullptr || ((uintptr_t)ptr & 255u) != 0) return BYZ_EINTERNAL;
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    }
    return aggregate_on_workspace(copies, d, ld, file_rows_dev, f, r, out, winner_replica,
                                  static_cast<AggWorkspace *>(ptr), flags, stream);
}

extern "C" int byz_calibration_copy(const void *src, void *dst, size_t bytes, void *stream) {
    if (src == nullptr || dst == nullptr || bytes == 0 || (bytes % 16) != 0) return BYZ_EINVAL;
    if ((((uintptr_t)src | (uintptr_t)dst) & 3u) != 0 || bytes > ((size_t)1 << 40)) return BYZ_EINVAL;
    const int64_t n_vec = (int64_t)(bytes / 16);
    calibration_copy_kernel<<<blocks_for(n_vec), kBlock, 0, (hipStream_t)stream>>>(
        reinterpret_cast<const uint32_t *>(src), reinterpret_cast<uint32_t *>(dst), n_vec);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

extern "C" int byz_calibration_read_rows(const void *rows_base, int64_t d, int64_t ld, int n_rows,
                                         void *out, int store, void *stream) {
    if (rows_base == nullptr || out == nullptr || d < 4 || ld < d || d > kMaxCoords) return BYZ_EINVAL;
    if (n_rows < 1 || n_rows > kWide * BYZ_MAX_R) return BYZ_EINVAL;
    if ((((uintptr_t)rows_base | (uintptr_t)out) & 3u) != 0) return BYZ_EINVAL;
    const int64_t n_vec = d / 4;
    calibration_read_rows_kernel<<<blocks_for(n_vec), kBlock, 0, (hipStream_t)stream>>>(
        reinterpret_cast<const uint32_t *>(rows_base), n_vec, ld, n_rows,
        reinterpret_cast<uint32_t *>(out), store);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

extern "C" int byz_profile_enable(int max_calls) {
    for (int i = 0; i < g_prof.capacity; ++i) {
        (void)hipEventDestroy(g_prof.start[i]);
        (void)hipEventDestroy(g_prof.stop[i]);
    }
    delete[] g_prof.start;
    delete[] g_prof.stop;
    g_prof = ProfileState();
    if (max_calls < 0 || max_calls > 100000) return BYZ_EINVAL;
    if (max_calls == 0) return BYZ_OK;
    g_prof.start = new (std::nothrow) hipEvent_t[max_calls];
    g_prof.stop = new (std::nothrow) hipEvent_t[max_calls];
    if (g_prof.start == nullptr || g_prof.stop == nullptr) {
        delete[] g_prof.start;
        delete[] g_prof.stop;
        g_prof = ProfileState();
        return BYZ_ENOMEM;
    }
    for (int i = 0; i < max_calls; ++i) {
        hipError_t e = hipEventCreate(&g_prof.start[i]);
        if (e == hipSuccess) {
            e = hipEventCreate(&g_prof.stop[i]);
            if (e != hipSuccess) (void)hipEventDestroy(g_prof.start[i]);
        }
        if (e != hipSuccess) {
            g_last_hip_error = (int)e;
            g_prof.capacity = i;
            (void)byz_profile_enable(0);
            return BYZ_EDEVICE;
        }
        g_prof.capacity = i + 1;
    }
    return BYZ_OK;
}

extern "C" int byz_profile_collect(float *ms_out, int capacity, int *n_out) {
    if (n_out == nullptr || capacity < 0 || (ms_out == nullptr && capacity > 0)) return BYZ_EINVAL;
    const int n = g_prof.count < capacity ? g_prof.count : capacity;
    for (int i = 0; i < n; ++i) {
        BYZ_HIP(hipEventSynchronize(g_prof.stop[i]));
        BYZ_HIP(hipEventElapsedTime(&ms_out[i], g_prof.start[i], g_prof.stop[i]));
    }
    *n_out = n;
    g_prof.count = 0;
    return BYZ_OK;
}

extern "C" const char *byz_profile_kernel(void) { return g_prof.kernel; }

extern "C" int byz_aggregate_path(const void *workspace, int *path, void *stream) {
    if (workspace == nullptr || path == nullptr) return BYZ_EINVAL;
    const AggWorkspace *ws = reinterpret_cast<const AggWorkspace *>(workspace);
    uint32_t v = 0;
    hipStream_t s = (hipStream_t)stream;
    BYZ_HIP(hipMemcpyAsync(&v, &ws->path, sizeof(v), hipMemcpyDeviceToHost, s));
    BYZ_HIP(hipStreamSynchronize(s));
    *path = (int)v;
    return BYZ_OK;
}

#endif  // part 0
