// Multi-Krum on the vote winners (gfx950).  The ByzShield paper pairs its vote with the
// coordinate-wise median and names Multi-Krum and Bulyan as aggregators that can take the
// median's place (Sec. 6.1, Sec. 7); it defines neither, so this file follows the published
// rule: with f vectors of which c may be Byzantine (f >= 2c + 3, the requirement quoted in
// Sec. 6.1), the score of vector i is the sum of its f - c - 2 smallest squared distances to
// other vectors; the m vectors of lowest score are averaged.
//
// The pairwise squared distances come from the Gram matrix G = W W^T of the f x d matrix of
// winners: the one dense contraction of the whole path, done with fp32 MFMA tiles
// (v_mfma_f32_16x16x4f32), only those on and above the diagonal of the symmetric matrix (f = 25
// costs 3 tiles of 16x16 instead of one padded 32x32), and v_mfma_f32_4x4x1f32 for a few rows behind
// the last full tile.  On long rows the choice is guessed from a sample first and the mean of the guessed vectors is
// taken in the same pass; the choice from the whole matrix decides whether it stands or is taken again.  The waves walk the coordinates
// grid-stride.  Per-block partial tiles are added in fp64 in block order, so the result does not
// depend on scheduling.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <type_traits>

#include "byz_internal.h"
#include "byzshield.h"

namespace {

#define BYZ_HIP(call)                              \
    do {                                           \
        hipError_t e_ = (call);                    \
        if (e_ != hipSuccess) {                    \
            byz_internal_set_hip_error((int)e_);   \
            return BYZ_EDEVICE;                    \
        }                                          \
    } while (0)

constexpr int kBlock = 256;            // 4 waves
constexpr int kGramBlocks = 512;       // partial Gram tiles (2 blocks per CU; 1024: 4 % faster, reduction 3 us slower)
constexpr int kTile = 16 * 16;         // outputs of one MFMA tile
constexpr int kMaxKrum = BYZ_MAX_F_KRUM;  // most vectors Multi-Krum takes (Bulyan: BYZ_MAX_F)
constexpr int kMaxNT = kMaxKrum / 16;  // row tiles of the largest matrix
constexpr int kMaxPairs = kMaxNT * (kMaxNT + 1) / 2;  // tiles on and above the diagonal

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// How the Gram matrix of f vectors is cut: nt row tiles of 16, of which the 16x16 tiles on and above
// the diagonal are computed, and `groups` groups of four rows behind them.  A group is multiplied with
// all rows by 4x4x1 matrix instructions, four rows against 64 a time, a quarter of the cycles of a tile
// for one coordinate of four: it costs one tile up to 64 rows and two above, a row tile with a few rows
// in it costs nt + 1.  Two tiles saved or more pay; with seven row tiles (f = 105..108) one does, as the
// kernel of seven spills.  Five and two groups (f = 85..88) would leave one wave per SIMD, up to 32 rows HBM
// bounds the kernel.  Calls of Multi-Krum on 3 M coordinates, us, without / with groups: f = 33 131 / 112,
// 49 190 / 165, 53 196 / 182, 65 275 / 245, 81 384 / 343, 97 494 / 431, 108 511 / 495, 113 659 / 537,
// 120 259 / 220 (1 M); of 140 k, f = 49 34.6 / 32.2, 97 76.5 / 71.6.  (40 rows, two groups for three tiles: 60.3 /
// 62.2 on 1 M; 60 rows, three for four: 208.6 / 203.7, short rows the same.)  The vector ALU instead of the
// small matrix instructions costs the same a row and more from two rows on: the two do not overlap.
__host__ __device__ constexpr int row_groups(int f) {
    const int nt = f / 16, groups = (f % 16 + 3) / 4, saved = nt + 1 - groups * (f <= 64 ? 1 : 2);
    return nt >= 2 && groups <= 3 && (saved >= 2 || (nt == 6 && saved >= 1)) && !(nt == 5 && groups == 2)
               ? groups : 0;
}
__host__ __device__ constexpr int row_tiles(int f) { return row_groups(f) != 0 ? f / 16 : (f + 15) / 16; }
// stored tiles of 256 values: the 16x16 ones, then every group's 4x64 ones
__host__ __device__ constexpr int stored_tiles(int nt, int groups) {
    return nt * (nt + 1) / 2 + groups * (nt < 4 ? 1 : 2);
}
__host__ __device__ constexpr int stored_tiles(int f) { return stored_tiles(row_tiles(f), row_groups(f)); }

// Tile (ti, tj), ti <= tj < nt, of the upper triangle, numbered row by row.
__host__ __device__ constexpr int tile_pair(int nt, int ti, int tj) {
    return ti * nt - ti * (ti - 1) / 2 + (tj - ti);
}

// The 16x16 MFMA result: accumulator register v of lane l holds row 4*(l/16) + v, column l%16
// (gram_at below inverts this).

// Waves per block, for sf steps of 32 coordinates a wave has in flight: enough waves to keep about
// 100 KB per CU in flight as far as registers allow (f = 16 on 4 M coordinates: 16 waves x 2 steps
// 139 us a call, 4 x 8 145; f = 25 on 11.2 M: 4 x 2 279, 8 x 1 282; f = 49: 4 x 1 629, 8 x 1 664,
// 4 x 2 644).  Short rows of up to 16 vectors: 8 waves (f = 16, d = 20011 16.8, 16 waves 17.7, 4 17.7).
constexpr int gram_waves(int nt, int sf) {
    return sf == 1 ? (nt <= 2 ? 8 : 4) : (nt <= 1 ? 16 : 4);
}
constexpr int kStep = 32;  // coordinates a wave multiplies between two visits to its stage

// Rows that do not start on cache lines (LINES false): the pieces of two neighbouring waves share a
// line.  Ordinary loads leave it in the L2, and groups of eight blocks' neighbours go to one of the
// eight L2s (blocks go to the XCDs round-robin), 4 KB of a row together.  us a call, non-temporal
// loads in plain order / this: 25 x 3 M 108 / 92, 48 x 3 M 195 / 166, 64 x 3 M 277 / 231; on cache
// lines ordinary loads are slower (48 x 3 M 151 / 160).
__device__ __forceinline__ unsigned neighbours_together(unsigned b, unsigned n_blocks, unsigned group) {
    const unsigned r = b % (8 * group);
    return b - r + 8 * group <= n_blocks ? b - r + (r % 8) * group + r / 8 : b;
}

// Compile-time fence: what the wave's lanes have written to LDS is read by other lanes of the same
// wave (LDS serves a wave's accesses in order, so the hardware needs no wait).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Rows of a wave's stage: whole loads of 64 pieces of 16 bytes.
__host__ __device__ constexpr int staged_rows(int nt, int groups, int sf) {
    const int per_load = 64 / (kStep * sf / 4);
    return (16 * nt + 4 * groups + per_load - 1) / per_load * per_load;
}

// Element e of the sixteen coordinates in y, quarter q: run[g * kParts + c] (four rows of group g against the rows
// 64c + lane) takes its product, one rounding; the caller goes through the quarters in ascending order.
template <int NT, int NG, int kParts, int N>
__device__ __forceinline__ void group_products(const f32x4 (&y)[kParts > 0 ? kParts : 1][4], int q, int e, bool fresh,
                                               f32x4 (&run)[N]) {
    constexpr f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    // (cbsz 4 and abid name the block of four lanes that is A for all sixteen blocks; constants)
#define BYZ_GROUP(g)                                                                                  \
    if constexpr (NG > (g))                                                                           \
        _Pragma("unroll") for (int c = 0; c < kParts; ++c)                                            \
            run[(g) * kParts + c] = __builtin_amdgcn_mfma_f32_4x4x1f32(                               \
                y[kParts - 1][q][e], y[c][q][e], fresh && q == 0 ? zero : run[(g) * kParts + c], 4,   \
                (4 * NT + (g)) % 16, 0);
    BYZ_GROUP(0)
    BYZ_GROUP(1)
    BYZ_GROUP(2)
#undef BYZ_GROUP
}

// Sample for a guess at Multi-Krum's choice among up to kMaxGuess vectors: stretches of 32 coordinates, one at a
// random place of every 1/kSampleSpans of the row (pitch: a whole number of stretches, so that rows on cache lines
// are sampled in whole lines).  The even blocks' partial matrices are one half of the sample, the odd blocks' the other:
// what the scores on the halves differ by tells how far the scores on the sample may be off.
constexpr int kMaxGuess = 64;
constexpr int kSampleSpans = 4096;
constexpr int kSampleBlocks = 256, kSampleWaves = 8;  // two stretches a wave: 5 to 8 us, 64 blocks with eight a wave 8 to 17
__device__ __forceinline__ int64_t sample_start(int64_t at, int64_t pitch) {
    const uint32_t hash = (uint32_t)at * 2654435761u;
    return at * pitch + (int64_t)(((uint64_t)hash * (uint64_t)(pitch / kStep)) >> 32) * kStep;
}

// Multi-Krum's choice, thread i = vector i with the score `mine` (the first kMaxKrum threads of a block): the m lowest
// scores, the lower index first among equal scores.  Returns i's place in that order, chosen if below m;
// *before = chosen vectors with a lower index, *total = how many there are.  All threads of the block call it.
__device__ __forceinline__ int choose_vector(double mine, int f, int m, double *s_score, uint64_t *s_chosen, int *before,
                                             int *total) {
    const int i = threadIdx.x;
    if (i < kMaxKrum) s_score[i] = mine;
    __syncthreads();
    int rank = 0;
#pragma unroll 8
    for (int k = 0; k < f; ++k) {
        const double other = s_score[k];
        rank += (other < mine || (other == mine && k < i)) ? 1 : 0;
    }
    if (i >= f) rank = kMaxKrum;
    const uint64_t mask = __builtin_amdgcn_ballot_w64(rank < m);
    if (i < kMaxKrum && (i & 63) == 0) s_chosen[i >> 6] = mask;
    __syncthreads();
    *before = __builtin_popcountll(mask & ((1ull << (i & 63)) - 1ull));
    *total = 0;
#pragma unroll
    for (int w = 0; w < kMaxKrum / 64; ++w) {
        const int n = __builtin_popcountll(s_chosen[w]);
        if (w < (i >> 6)) *before += n;
        *total += n;
    }
    return rank;
}

// Scores on the sample: of vector i on all of it, and the first half's less the second's.
struct SampleScores {
    double score[kMaxGuess], apart[kMaxGuess];
};

// The guess, by every block of the Gram pass for itself from the scores on the sample; all its threads call it.
// None where it may be wrong: where the last vector chosen and the first one not are closer than kSure standard deviations
// of such a distance, taken from what neighbours in the order of the scores, up to kNeighbours on each side of that place,
// differ by between the halves (relative to their scores: what makes all scores larger or smaller alike does not
// count).  Right / none / wrong of 40 calls each on 2 M coordinates, a tenth of the vectors reversed, each vector with a
// scale of its own, by this rule and by a fixed margin of 0.2 % of the score: f = 25 m = 20 37 / 3 / 0 and 37 / 2 / 1, with a
// log-normal scale (sigma 1) per coordinate besides 23 / 16 / 1 and 28 / 1 / 11, per sixtieth of the row 28 / 10 / 2 and 36 / 1 /
// 3, sigma 2 per coordinate 0 / 39 / 1 and 1 / 2 / 37; f = 49 m = 40 36 / 4 / 0, 10 / 29 / 1, 22 / 17 / 1, 0 / 40 / 0 and 37 / 3 / 0, 17 / 5 / 18,
// 32 / 2 / 6, 1 / 2 / 37.  Two deviations halve the right ones of the last three and save no more than one wrong one.
// Nor where the output overlaps a row, which the guessed mean would overwrite before the row's last reader.
// (The sample's places are the same in every call on rows of a length, so a sender who knows them can look different
// there: that makes the guess wrong and the call slower, figures at guess_pays; the words are the same.)
constexpr double kSure = 1.0;
constexpr int kNeighbours = 8;
__device__ __forceinline__ uint64_t guess_vectors(const SampleScores *__restrict__ sample, int f, int m,
                                                  const float *rows_base, int64_t d, int64_t ld,
                                                  const int32_t *__restrict__ row_index, const float *out, double *s_room) {
    double *s_order = s_room + kMaxKrum, *s_off = s_order + kMaxGuess;  // by place: scores, relative differences
    uint64_t *s_chosen = reinterpret_cast<uint64_t *>(s_off + kMaxGuess), *s_guess = s_chosen + kMaxKrum / 64;
    const int i = threadIdx.x;
    if (i < kMaxGuess) s_order[i] = s_off[i] = 0.0;
    const double mine = i < f ? sample->score[i] : 0.0, apart = i < f ? sample->apart[i] : 0.0;
    bool overlap = false;
    if (i < f) {
        const uintptr_t row = (uintptr_t)(rows_base + (int64_t)row_index[i] * ld), o = (uintptr_t)out;
        const uintptr_t bytes = (uintptr_t)d * sizeof(float);
        overlap = o < row + bytes && row < o + bytes;
    }
    int before, total;
    const int rank = choose_vector(mine, f, m, s_room, s_chosen, &before, &total);
    if (i < f) {
        s_order[rank] = mine;
        s_off[rank] = apart / mine;
    }
    __syncthreads();
    if (i < 64) {
        const int place = m - kNeighbours + i;  // between the vectors of places place - 1 and place
        const bool used = i < 2 * kNeighbours && place >= 1 && place < f;
        const double off = used ? s_off[place] - s_off[place - 1] : 0.0;
        double square = off * off;
#pragma unroll
        for (int k = 1; k < 2 * kNeighbours; k <<= 1) square += __shfl_xor(square, k, 64);
        const int count = __builtin_popcountll(__builtin_amdgcn_ballot_w64(used));
        const bool clash = __builtin_amdgcn_ballot_w64(overlap) != 0;
        if (i == 0) {
            const double last = s_order[m - 1], gap = m < f ? s_order[m] - last : 0.0;
            const bool sure = m == f || gap * gap * count > kSure * kSure * square * last * last;
            *s_guess = sure && !clash ? s_chosen[0] : 0ull;
        }
    }
    __syncthreads();
    const uint64_t chosen = *s_guess;
    __syncthreads();  // the room is used for other things
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(chosen >> 32)) << 32 |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)chosen);
}

// What a Gram pass that takes a mean on the way is given: scores on the sample, how many vectors to choose, where the
// mean goes and where the guess is left for chosen_mean_kernel.
struct GuessedPass {
    const SampleScores *scores;
    int m;
    float *out;
    uint64_t *chosen;
};

// Mean of the guessed vectors over the stretch a wave has in its stage, lane = coordinate: the additions and the
// division of chosen_mean_kernel, so that the words are the same.  A vector that is not guessed adds +0, which leaves
// every partial sum as it is (sums from +0 are never -0).  It adds 25 us to the 176 us of the Gram pass of 25 x 11.2 M
// (6 of them the output) and saves the 152 us of a second pass; with 49 vectors 80 us.  Eight waves a block, one
// multiply-add by 1 or 0 for mask and addition, or the place behind the matrix instructions: the same or slower.
constexpr int kMeanRows = 16;  // a step, whose reads of LDS are under way together
struct GuessedMean {
    uint64_t chosen;  // bit i = vector i; none: no mean is taken
    float count;
    float *out;
    template <int ROWS, int SPAN>
    __device__ __forceinline__ void add(const float *stage, int64_t c0, int64_t d) const {
        if (count == 0.0f) return;
        const int lane = threadIdx.x & 63, at = lane % SPAN;
        float a = 0.0f;
#pragma unroll
        for (int r0 = 0; r0 < ROWS; r0 += kMeanRows) {
            uint32_t bits = (uint32_t)(chosen >> r0) & ((1u << kMeanRows) - 1u);
            if (bits == 0) continue;
            asm volatile("" : "+s"(bits));  // or a mask per vector is kept over all stretches, and spilled
            uint32_t v[kMeanRows];
#pragma unroll
            for (int u = 0; u < kMeanRows; ++u)
                if (r0 + u < ROWS)
                    v[u] = __float_as_uint(stage[(r0 + u) * SPAN + ((at / 4) ^ (u & 7)) * 4 + at % 4]);
#pragma unroll
            for (int u = 0; u < kMeanRows; ++u)
                if (r0 + u < ROWS) a += __uint_as_float(v[u] & (uint32_t)__builtin_amdgcn_sbfe((int)bits, u, 1));
        }
        const float mean = a / count;
        if (lane < SPAN && c0 + at < d) __builtin_nontemporal_store(mean, out + c0 + at);
    }
};

// What a Gram kernel reads: long rows, short rows, a sample of long ones, long ones whose mean is taken on the way.  (The
// sample as a run-time case of the short rows' kernel cost that one up to 16 registers: us a call, with / without, 40 x 250000
// 31.0 / 30.2, 49 x 100000 27.0 / 26.6, 97 x 250000 83.8 / 82.8.)
enum class Gram { kLong, kShort, kSample, kMean };
constexpr int gram_waves(int nt, int sf, Gram kind) { return kind == Gram::kSample ? kSampleWaves : gram_waves(nt, sf); }

// Accumulates the Gram tiles of all f rows over this wave's coordinates, NT = row tiles of 16, NG =
// groups of four rows behind them (row_groups).
// A wave takes whole stretches of 32*SF coordinates of every row, so every word is loaded once
// and no barrier stands between the loads and the matrix instructions.  Consecutive lanes load
// consecutive words of a row; a pass through the wave's own
// piece of LDS gives lane l four coordinates of row l%16 at a time, the k of its quarter of the
// wave for four instructions (16-byte pieces, piece p of row r in place p ^ (r%8): neither side
// has bank conflicts).  Products are the fp32 instruction's, rounded once each into their sum; G(i, j)
// and G(j, i) are the same bits, and equal rows tie exactly.
// A long running sum is off by its roundings and, one-sidedly, by about 1.3e-11 of itself per
// product (25 x 11.2 M, 5456 products: 2e-7 of the norms).  So a run ends after three steps of 32
// coordinates (two of 64) and is added to the totals by the vector ALU; SHORT, one to four steps a
// wave, ends it after 16 coordinates, where the sums are few.  Distances' error over G_ii + G_jj,
// rms, 1e-9, f = 49, d = 2048 / 20011 / 140001 / 1.1 M: 5.0 / 2.5 / 1.1 / 1.7; one running sum 8.7 / 3.4 / 2.3 /
// 8.9; bf16 matrix units on rows split in three parts 7.9 / 2.9 / 2.1 / 2.0.
// Calls of Multi-Krum with rows on cache lines, us, in brackets with one running sum, a tile in LDS
// shared by the block, two barriers a chunk and row tiles rounded up to 6 or 8 above 64 rows: 49 x
// 11.2 M 660 (705; with a group instead of a row tile 577), 80 x 3 M 308 (442), 128 x 3 M 697 (843); to
// f = 32, HBM-bound, the same (32 x 11.2 M 355 and 352).  From f = 49 up matrix instructions and what little
// the vector ALU does bound it together, as they share one datapath (six tiles and a group at f = 49: the
// kernel takes 390 us, 344 with its loads left out, 322 with its products left out; more waves, longer
// stretches or loads two steps ahead changed nothing); the runs cost 3 % there (15 % with eight row
// tiles, where the sums fill the registers).
template <int NT, int NG, int SF, bool LINES, Gram KIND>
__device__ __forceinline__ void gram_accumulate(const float *__restrict__ X, int64_t d, int64_t ld,
                                                const int32_t *__restrict__ row_index, int f, int64_t pitch,
                                                const GuessedMean &guessed, float *stage, f32x4 (&acc)[stored_tiles(NT, NG)]) {
    constexpr bool SHORT = KIND == Gram::kShort || KIND == Gram::kSample, MEAN = KIND == Gram::kMean;
    constexpr int NP = NT * (NT + 1) / 2, NALL = stored_tiles(NT, NG), kSpan = kStep * SF;
    constexpr int kPieces = kSpan / 4, kRows = 64 / kPieces, kLoads = staged_rows(NT, NG, SF) / kRows;
    constexpr int kParts = NG == 0 ? 0 : (NALL - NP) / NG;  // stretches of 64 rows a group meets
    const int lane = threadIdx.x & 63;
    const int64_t n_spans = KIND == Gram::kSample ? kSampleSpans : (d + kSpan - 1) / kSpan;
    constexpr int kWaves = gram_waves(NT, SF, KIND);
    const int64_t stride = (int64_t)gridDim.x * kWaves;
    constexpr unsigned kGroup = NT <= 1 ? 1 : (NT == 2 ? 4 : 8);
    const unsigned block = LINES ? blockIdx.x : neighbours_together(blockIdx.x, gridDim.x, kGroup);
    int64_t span = (int64_t)block * kWaves + (threadIdx.x >> 6);
    // load n: rows n*kRows .. + kRows - 1, one after the other; rows past f in a load that has others
    // repeat row f-1 (nothing reads their results), loads without a row are left out
    auto row_of = [&](int n) { return n * kRows + lane / kPieces; };
    auto piece_of = [&](int n) { return (lane % kPieces) ^ (row_of(n) & 7); };
    auto used = [&](int n) { return NG > 0 || n * kRows <= 16 * (NT - 1) || n * kRows < f; };
    const float *rowp[kLoads];
#pragma unroll
    for (int n = 0; n < kLoads; ++n)
        rowp[n] = X + (int64_t)row_index[row_of(n) < f ? row_of(n) : f - 1] * ld + 4 * piece_of(n);
    f32x4 *slots = reinterpret_cast<f32x4 *>(stage);  // [16*NT rows][kPieces]
#pragma unroll
    for (int n = 0; n < kLoads; ++n)
        if (!used(n)) slots[64 * n + lane] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 raw[kLoads];
    auto fetch = [&](int64_t at) {
        const int64_t c0 = KIND == Gram::kSample ? sample_start(at, pitch) : at * kSpan;
        if (c0 + kSpan <= d) {
#pragma unroll
            for (int n = 0; n < kLoads; ++n)
                if (used(n)) {
                    const f32x4u *p = reinterpret_cast<const f32x4u *>(rowp[n] + c0);
                    raw[n] = LINES ? __builtin_nontemporal_load(p) : *p;
                }
        } else {  // the ragged end: missing coordinates count as zero
#pragma unroll
            for (int n = 0; n < kLoads; ++n)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    raw[n][e] = c0 + 4 * piece_of(n) + e < d ? rowp[n][c0 + e] : 0.0f;
        }
    };
    constexpr f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int kRun = SHORT ? 1 : (SF == 1 ? 3 : 2);  // stretches of a run (SHORT: each adds its own)
    constexpr int kRuns = SHORT ? (NP < 6 ? NP : 6) : NP;  // tiles whose runs are open at a time
    constexpr int kGroupRuns = NG > 0 ? NALL - NP : 1;
    // The first stretch of a run in a body of its own, whose first products take an inline zero instead of cleared
    // registers; with the groups' chains between the tiles, us a call: Multi-Krum 49 x 3 M 158 -> 155, 81 x 3 M 342 -> 327,
    // 96 x 2 M 272 -> 262, 101 x 3 M 514 -> 493, 112 x 2 M 339 -> 318, Bulyan 49 x 11.2 M 694 -> 687.  Slower without groups
    // at 64 and 80 x 3 M (177 / 179, 297 / 307), twice as slow at 128 (spills), the same with the mean; and with four tiles and a
    // group (65 x 11 M off the cache lines 723 / 751) and seven and three (spills: 121 x 11 M 1915 / 2816, 0.3 M 103 / 124).
    constexpr bool kPeel =
        SHORT || (NG > 0 ? !MEAN && NT != 4 && !(NT == 7 && NG == 3) : NT == 6 || NT == 7);
    f32x4 run[kRuns], grun[kGroupRuns];
#pragma unroll
    for (int p = 0; p < NALL; ++p) acc[p] = zero;
    const int row = lane & 15;
    // one stretch; `first` of a run: its sums start from zero
    auto step = [&](auto first) {
        constexpr bool kFirst = decltype(first)::value;
        wave_fence();
#pragma unroll
        for (int n = 0; n < kLoads; ++n)
            if (used(n)) slots[64 * n + lane] = raw[n];
        wave_fence();
        if (span + stride < n_spans) fetch(span + stride);
        if constexpr (MEAN) guessed.template add<16 * NT + 4 * NG, kSpan>(stage, span * kSpan, d);
#pragma unroll
        for (int h = 0; h < 2 * SF; ++h) {  // 16 coordinates
            const int piece = 8 * (h / 2) + 2 * (lane >> 4) + h % 2;
            f32x4 x[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t)
                x[t] = slots[(16 * t + row) * kPieces + (piece ^ (row & 7))];
            // the groups' operand, both sides of it: lane l holds row l (and 64 + l); the
            // instruction takes the four lanes of one group as A and all as B.  The order of
            // the products is that of the 16x16 instruction, which multiplies the four
            // quarters of the wave one after the other.
            f32x4 y[NG > 0 ? kParts : 1][4];
            if constexpr (NG > 0)
#pragma unroll
                for (int c = 0; c < kParts; ++c)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int r = 64 * c + lane < 16 * NT + 4 * NG ? 64 * c + lane : 16 * NT;
                        y[c][q] = slots[r * kPieces + ((8 * (h / 2) + 2 * q + h % 2) ^ (r & 7))];
                    }
            // lane l holds A[row = l%16][k = l/16], which is also B[k][col = l%16] of the
            // transposed operand; tiles p0 .. p0 + kRuns - 1
#pragma unroll
            for (int p0 = 0; p0 < NP; p0 += kRuns) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool fresh = e == 0 && (SHORT || (kFirst && h == 0));
#pragma unroll
                    for (int ti = 0; ti < NT; ++ti)
#pragma unroll
                        for (int tj = ti; tj < NT; ++tj) {
                            const int p = tile_pair(NT, ti, tj) - p0;
                            if (p < 0 || p >= kRuns) continue;
                            // the groups' chains of four between the tiles, whose instructions they would
                            // otherwise wait in front of
                            if constexpr (NG > 0)
                                if (p0 == 0 && p < 4) group_products<NT, NG, kParts>(y, p, e, fresh, grun);
                            run[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                x[ti][e], x[tj][e], fresh ? zero : run[p], 0, 0, 0);
                        }
                    if constexpr (NG > 0)
                        if (p0 == 0)
#pragma unroll
                            for (int q = kRuns < 4 ? kRuns : 4; q < 4; ++q)
                                group_products<NT, NG, kParts>(y, q, e, fresh, grun);
                }
                if constexpr (SHORT)
#pragma unroll
                    for (int p = 0; p < kRuns && p0 + p < NP; ++p) acc[p0 + p] += run[p];
            }
            if constexpr (SHORT)
#pragma unroll
                for (int p = NP; p < NALL; ++p) acc[p] += grun[p - NP];
        }
        span += stride;
    };
    if (span < n_spans) fetch(span);
    while (span < n_spans) {
        if constexpr (kPeel) {
            step(std::true_type());
        } else {
#pragma unroll
            for (int p = 0; p < NP; ++p) run[p] = zero;
#pragma unroll
            for (int p = 0; p < kGroupRuns; ++p) grun[p] = zero;
        }
        for (int k = kPeel ? 1 : 0; k < kRun && span < n_spans; ++k) step(std::false_type());
        if constexpr (!SHORT) {
#pragma unroll
            for (int p = 0; p < NP; ++p) acc[p] += run[p];
#pragma unroll
            for (int p = NP; p < NALL; ++p) acc[p] += grun[p - NP];
        }
    }
}

// Partial Gram tiles of the rows row_index[0..f-1] over this block's coordinates.  partial:
// [gridDim.x][tiles][256] values, position v*64 + lane, tiles = stored_tiles(NT, NG), fp32 or, where a few
// blocks would leave their last roundings visible, fp64 (d = 2048: 8.9e-9 -> 4.9e-9 at f = 100).
template <int NT, int NG, int SF, bool LINES, Gram KIND>
__global__ __launch_bounds__(64 * gram_waves(NT, SF, KIND))
// (2: accumulators in ordinary registers; more row tiles would spill: 96 x 11.2 M 1502 us, 1362 with 1,
// 80 x 11.2 M 998 and 1060; the same with groups, (5, 1) on long rows 41 registers)
__attribute__((amdgpu_waves_per_eu(NG > 0 ? (NT <= 4 || (NT == 5 && KIND == Gram::kShort) ? 2 : 1) : (NT <= 5 || (NT == 6 && KIND == Gram::kShort) ? 2 : 1))))
void gram_partial_kernel(
    const float *__restrict__ X, int64_t d, int64_t ld, const int32_t *__restrict__ row_index, int f,
    float *__restrict__ partial, int in_fp64, int64_t pitch, GuessedPass guess) {
    constexpr int NP = stored_tiles(NT, NG), kWaves = gram_waves(NT, SF, KIND);
    constexpr int kStage = staged_rows(NT, NG, SF) * kStep * SF;  // floats of one wave's stage
    constexpr int kRoom = 16 * 1024 / (kWaves * kTile);  // tiles of every wave that 64 KB hold
    constexpr int kAtOnce = NP < kRoom ? NP : kRoom;
    constexpr int kRed = kWaves * kAtOnce * kTile;
    __shared__ __align__(16) float lds[kRed > kWaves * kStage ? kRed : kWaves * kStage];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    f32x4 acc[NP];
    GuessedMean guessed = {0, 0.0f, nullptr};
    if constexpr (KIND == Gram::kMean) {
        guessed.chosen = guess_vectors(guess.scores, f, guess.m, X, d, ld, row_index, guess.out,
                                       reinterpret_cast<double *>(lds));
        guessed.count = (float)__builtin_popcountll(guessed.chosen);
        guessed.out = guess.out;
        if (blockIdx.x == 0 && tid == 0) *guess.chosen = guessed.chosen;
    }
    gram_accumulate<NT, NG, SF, LINES, KIND>(X, d, ld, row_index, f, pitch, guessed, lds + wave * kStage, acc);
    // the waves' tiles are added in wave order in fp64, as many tiles at a time as fit
#pragma unroll
    for (int p0 = 0; p0 < NP; p0 += kAtOnce) {
        __syncthreads();  // the stages, or the tiles before these, are read before these replace them
#pragma unroll
        for (int p = p0; p < p0 + kAtOnce && p < NP; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                lds[(wave * kAtOnce + p - p0) * kTile + v * 64 + lane] = acc[p][v];
        __syncthreads();
        const int count = (NP - p0 < kAtOnce ? NP - p0 : kAtOnce) * kTile;
        for (int i = tid; i < count; i += 64 * kWaves) {
            double total = lds[i];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) total += (double)lds[w * kAtOnce * kTile + i];
            const int64_t at = ((int64_t)blockIdx.x * NP + p0) * kTile + i;
            if (in_fp64 != 0)
                reinterpret_cast<double *>(partial)[at] = total;
            else
                partial[at] = (float)total;
        }
    }
}

// gram[t][pos] = sum over blocks of partial[block][t][pos] in fp64, in a fixed order: thread
// (pos, g) adds the blocks g, g+8, g+16, ... one by one, then the eight group sums are added
// in order.  Block = 32 positions x 8 groups.  HALVES: the even blocks' sums, and the odd blocks' behind the
// matrix.
template <typename T, bool HALVES>
__global__ __launch_bounds__(kBlock) void gram_reduce_kernel(const T *__restrict__ partial,
                                                             int n_partial, int ntiles,
                                                             double *__restrict__ gram) {
    __shared__ double s_sum[8][32];
    const int lp = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int i = blockIdx.x * 32 + lp;  // ntiles * 256 is a multiple of 32
    double acc = 0.0;
#pragma unroll 8
    for (int p = g; p < n_partial; p += 8) acc += (double)partial[(int64_t)p * ntiles * kTile + i];
    s_sum[g][lp] = acc;
    __syncthreads();
    if (HALVES ? g < 2 : g == 0) {
        double total = s_sum[g][lp];
        for (int k = HALVES ? g + 2 : 1; k < 8; k += HALVES ? 2 : 1) total += s_sum[k][lp];
        gram[(HALVES ? g * ntiles * kTile : 0) + i] = total;
    }
}

__device__ inline double gram_at(const double *gram, int f, int i, int j) {
    // entry (i, j) of the symmetric matrix from the stored upper-triangle tiles
    if (i > j) { const int t = i; i = j; j = t; }
    const int nt = row_tiles(f), g = (j - 16 * nt) / 4;
    if (j >= 16 * nt)  // row j of group g, column i
        return gram[(nt * (nt + 1) / 2 + g * (nt < 4 ? 1 : 2) + i / 64) * kTile + j % 4 * 64 + i % 64];
    const int r = i % 16, c = j % 16;
    // row r = 4*(l/16) + v, column c = l%16  =>
    const int v = r % 4, l = c + 16 * (r / 4);
    return gram[tile_pair(nt, i / 16, j / 16) * kTile + v * 64 + l];
}

// The value lane `from` (the same for the whole wave) holds.
__device__ __forceinline__ double lane_value(double v, int from) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), from);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), from);
    return __hiloint2double(hi, lo);
}

// (key, tag) pairs of the row sort: spare keys (tag >= 256) last, else by value, then by tag.
__device__ __forceinline__ bool key_before(double a_v, int a_t, double b_v, int b_t) {
    const bool a_spare = a_t >= 256, b_spare = b_t >= 256;
    return a_spare != b_spare ? b_spare : (a_v < b_v || (a_v == b_v && a_t < b_t));
}

// Set-up of the selections, one wave per vector i (4 per block), for f <= 64*PER: the lane
// computes the squared distances d(i,j) = G_ii + G_jj - 2 G_ij (clamped at 0, exactly 0 on the
// diagonal) for j = lane and, with PER = 2, j = lane + 64, and writes them to dist_out; a
// bitonic network over the 64*PER keys of the wave then sorts the distances to the other
// vectors in ascending order (value, then index), the keys of j = i and j >= f sorting behind
// every distance.  The t-th nearest of vector i goes to sorted_dist[t*kRowStride + i] and
// sorted_nbr[t*kRowStride + i] (t < f-1; the other entries are not written).  With
// n_terms >= 0 the wave also adds the n_terms smallest distances one by one in ascending
// order from +0: the Krum score, into scores and scores_out.  (Sort and sum as functions of their own, with the arrays
// handed over, take 1.2 to 1.6 us more for 65 vectors and more: Multi-Krum 65 x 2000 29.5 / 31.7, 128 x 100000 74.1 / 76.4.)
constexpr int kRowStride = kMaxKrum;

template <int PER>
__global__ __launch_bounds__(kBlock) void distance_rows_kernel(const double *__restrict__ gram, int f,
                                                               int n_terms, double *dist_out,
                                                               double *__restrict__ sorted_dist,
                                                               uint8_t *__restrict__ sorted_nbr,
                                                               double *__restrict__ scores,
                                                               double *scores_out) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (i >= f) return;  // whole wave
    double v[PER];
    int tag[PER];
    const double g_ii = gram_at(gram, f, i, i);
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int j = lane + 64 * e;
        v[e] = 0.0;
        if (j < f) {
            const double dij = g_ii + gram_at(gram, f, j, j) - 2.0 * gram_at(gram, f, i, j);
            if (!(dij < 0.0) && j != i) v[e] = dij;
            if (dist_out != nullptr) dist_out[i * f + j] = v[e];
        }
        tag[e] = j | ((j >= f || j == i) ? 256 : 0);  // every key distinct
    }
#pragma unroll
    for (int k = 2; k <= 64 * PER; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j == 64) {
                // partner in the same lane; k = 128 here, so the order is ascending
                if constexpr (PER == 2) {
                    if (!key_before(v[0], tag[0], v[1], tag[1])) {
                        const double tv = v[0];
                        const int tt = tag[0];
                        v[0] = v[1];
                        tag[0] = tag[1];
                        v[1] = tv;
                        tag[1] = tt;
                    }
                }
            } else {
                const bool lower = (lane & j) == 0;
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                    const double ov = __shfl_xor(v[e], j, 64);
                    const int otag = __shfl_xor(tag[e], j, 64);
                    // both lanes of a pair evaluate the same comparison (lower lane's key
                    // first), so the exchange is a permutation whatever the values are
                    const bool lo_first = lower ? key_before(v[e], tag[e], ov, otag)
                                                : key_before(ov, otag, v[e], tag[e]);
                    const bool ascending = ((lane + 64 * e) & k) == 0;
                    if (lo_first != ascending) {
                        v[e] = ov;
                        tag[e] = otag;
                    }
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int t = lane + 64 * e;
        if (t < f - 1) {
            sorted_dist[t * kRowStride + i] = v[e];
            sorted_nbr[t * kRowStride + i] = (uint8_t)tag[e];
        }
    }
    if (n_terms >= 0) {
        double score = 0.0;
        for (int t = 0; t < n_terms && t < 64; ++t) score += lane_value(v[0], t);
        if constexpr (PER == 2)
            for (int t = 64; t < n_terms; ++t) score += lane_value(v[1], t - 64);
        if (lane == 0) {
            scores[i] = score;
            if (scores_out != nullptr) scores_out[i] = score;
        }
    }
}

// Scores of the f <= kMaxGuess vectors on the sample, a wave per vector, lane = the other one: the n_terms smallest
// distances on the whole sample, and the same ones on either half.  The n_terms-th smallest is found bit by bit; as many of
// several equal to it count as are missing.
__global__ __launch_bounds__(64) void sample_scores_kernel(const double *__restrict__ halves, int f, int n_terms,
                                                           SampleScores *__restrict__ sample) {
    const int i = blockIdx.x, lane = threadIdx.x, j = lane < f ? lane : i;
    auto apart = [&](const double *g) {
        return fmax(gram_at(g, f, i, i) + gram_at(g, f, j, j) - 2.0 * gram_at(g, f, i, j), 0.0);
    };
    const double a = apart(halves), b = apart(halves + stored_tiles(f) * kTile);
    const uint32_t key = j != i ? __float_as_uint((float)(a + b)) : ~0u;
    uint32_t nth = 0;
#pragma unroll
    for (int bit = 31; bit >= 0; --bit)
        if (__builtin_popcountll(__builtin_amdgcn_ballot_w64(key < (nth | 1u << bit))) < n_terms) nth |= 1u << bit;
    const int below = __builtin_popcountll(__builtin_amdgcn_ballot_w64(key < nth));
    const int equal = __builtin_popcountll(__builtin_amdgcn_ballot_w64(key == nth));
    const double weight = key < nth ? 1.0 : (key == nth ? (double)(n_terms - below) / (double)equal : 0.0);
    double sum_a = weight != 0.0 ? weight * a : 0.0, sum_b = weight != 0.0 ? weight * b : 0.0;
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
        sum_a += __shfl_xor(sum_a, k, 64);
        sum_b += __shfl_xor(sum_b, k, 64);
    }
    if (lane == 0) {
        sample->score[i] = sum_a + sum_b;
        sample->apart[i] = sum_a - sum_b;
    }
}

// quad_perm [1,0,3,2]: lane ^ 1; quad_perm [2,3,0,1]: lane ^ 2; row_half_mirror: the other quad of the
// 8; row_mirror: the other half of the 16
constexpr int kDppPairs[4] = {0xB1, 0x4E, 0x141, 0x140};

// The smallest of the wave's 64 values, in every lane.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
    auto lower = [](uint32_t a, int b) { return a < (uint32_t)b ? a : (uint32_t)b; };
    v = lower(v, __builtin_amdgcn_update_dpp(0, (int)v, kDppPairs[0], 0xF, 0xF, false));
    v = lower(v, __builtin_amdgcn_update_dpp(0, (int)v, kDppPairs[1], 0xF, 0xF, false));
    v = lower(v, __builtin_amdgcn_update_dpp(0, (int)v, kDppPairs[2], 0xF, 0xF, false));
    v = lower(v, __builtin_amdgcn_update_dpp(0, (int)v, kDppPairs[3], 0xF, 0xF, false));
    uint32_t least = (uint32_t)__builtin_amdgcn_readlane((int)v, 0);
#pragma unroll
    for (int row = 1; row < 4; ++row) least = lower(least, __builtin_amdgcn_readlane((int)v, 16 * row));
    return least;
}

// What a vector's score is ordered by.  Scores are sums of distances from +0, never negative, so their bit
// patterns are in the order of the values, NaNs behind infinity; a vector that is not left comes behind any score.
__device__ __forceinline__ uint64_t score_key(double score, bool left) {
    return left ? (uint64_t)__double_as_longlong(score) : ~0ull;
}

// Lowest (key, lane) of the wave: the lowest upper half, the lowest lower half that comes with it, the first
// lane that has both.
__device__ __forceinline__ void wave_argmin(uint64_t key, int i, uint64_t &w_key, int &w_best) {
    const uint32_t hi = (uint32_t)(key >> 32), lo = (uint32_t)key;
    const uint32_t least_hi = wave_min(hi);
    const uint32_t least_lo = wave_min(hi == least_hi ? lo : 0xFFFFFFFFu);
    const uint64_t here = __builtin_amdgcn_ballot_w64(hi == least_hi && lo == least_lo);
    w_key = (uint64_t)least_hi << 32 | least_lo;
    w_best = __builtin_amdgcn_readfirstlane(i) + (int)__builtin_ctzll(here);
}

// First phase of Bulyan: Krum applied again and again to the vectors not yet chosen, until
// theta = f - 2c are chosen.  Round with n' vectors left: score(i) = the n' - c - 2 smallest
// distances from i to the other vectors left, added one by one in ascending order (no terms
// when that count is <= 0); lowest score wins, lowest index among equal scores.
// One thread per vector, WAVES = 1 up to 64 vectors and 2 up to 128, on the sorted rows
// distance_rows_kernel left.  A vector left has n' - 1 others left and takes n' - c - 2 of them, so its
// terms are the others left without the c + 1 farthest; choosing a vector removes it from every row:
// where it was a term the row loses it, elsewhere it was one of the c + 1 farthest and the farthest
// term takes its place there.  So only the first f - c - 2 of a row are ever terms.  They sit in LDS, a
// column per vector, and a term that goes is overwritten with zero: a score is a walk of plain
// additions over the column, as x + 0 is x, with no test per position.  Which positions are still
// terms is a mask of 64 * WAVES bits, for the farthest one and for the end of the walk.
// Bound by latencies: per round the walk's chain of additions, the search, and the look where the
// chosen vector stands in each row.  Calls of Bulyan on 10 k coordinates,
// us, with a test per position on rows in registers (f <= 64) or in LDS / this: f = 25 42.7 / 30.8, 49 67.8 /
// 46.9, 63 87 / 60, 65 175 / 78, 101 327 / 119, 127 503 / 164.
// The other waves of the block only help to fill LDS.
// Dynamic LDS: select_terms(f, c) * 64 * WAVES doubles, pairs of positions next to each other, then f * 64 *
// WAVES bytes.
constexpr int kSelectThreads = 512;
__host__ __device__ constexpr int select_terms(int f, int c) { return (f - c - 2 + 15) / 16 * 16; }

template <int WAVES>
__global__ __launch_bounds__(kSelectThreads) void bulyan_select_kernel(
    const double *__restrict__ sorted_dist, const uint8_t *__restrict__ sorted_nbr, int f, int c,
    int32_t *selected_out, int32_t *order_out, int32_t *selected_list, int32_t *n_selected,
    const int32_t *__restrict__ row_index, int32_t *selected_rows) {
    constexpr int S = 64 * WAVES, kFillers = kSelectThreads / S;
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) double s_rows[];
    __shared__ uint64_t s_wave_key[2][WAVES];
    __shared__ int s_wave_best[2][WAVES];
    __shared__ int32_t s_row_of[S];
    const int i = threadIdx.x % S, filler = threadIdx.x / S;
    const int theta = f - 2 * c, n_terms = f - c - 2, walk = select_terms(f, c);
    uint8_t *s_pos = reinterpret_cast<uint8_t *>(s_rows + walk * S);  // [j*S + i]: where vector j stands in i's row
    auto place = [&](int t) { return (t / 2 * S + i) * 2 + t % 2; };
#pragma unroll 8
    for (int t = filler; t < walk; t += kFillers)
        s_rows[place(t)] = t < n_terms && i < f ? sorted_dist[t * kRowStride + i] : 0.0;
#pragma unroll 8
    for (int t = filler; t < f - 1; t += kFillers)
        if (i < f) s_pos[sorted_nbr[t * kRowStride + i] * S + i] = (uint8_t)t;
    if (filler == 0) {
        s_row_of[i] = row_index[i < f ? i : 0];
        if (i < f) selected_out[i] = 0;
    }
    __syncthreads();
    if (filler != 0) return;  // whole waves
    bool left = i < f;  // not chosen yet
    uint64_t lo = !left ? 0ull : (n_terms >= 64 ? ~0ull : (1ull << n_terms) - 1ull);  // positions 0..63
    uint64_t hi = !left || n_terms <= 64 ? 0ull : (1ull << (n_terms - 64)) - 1ull;    // 64..
    int32_t first_row = 0;
    const f64x2 *column = reinterpret_cast<const f64x2 *>(s_rows) + i;
    for (int round = 0; round < theta; ++round) {
        double score = 0.0;
        f64x2 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = column[u * S];
        for (int t0 = 0;; t0 += 16) {
            // has any vector of this wave terms further on?
            const int on = t0 + 16;
            const uint64_t rest = on < 64 ? ((lo >> on) | hi) : (on < 128 ? hi >> (on - 64) : 0ull);
            const bool more = __builtin_amdgcn_ballot_w64(rest != 0) != 0;
            f64x2 y[8];
            if (more) {
#pragma unroll
                for (int u = 0; u < 8; ++u) y[u] = column[(on / 2 + u) * S];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                score += x[u][0];
                score += x[u][1];
            }
            if (!more) break;
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = y[u];
        }
        uint64_t w_key;
        int best;
        wave_argmin(score_key(score, left), i, w_key, best);
        if constexpr (WAVES > 1) {
            const int side = round & 1;  // a round's winners are read while the next one's are written
            if ((i & 63) == 0) {
                s_wave_key[side][i >> 6] = w_key;
                s_wave_best[side][i >> 6] = best;
            }
            __syncthreads();
            uint64_t b_key = s_wave_key[side][0];
            best = s_wave_best[side][0];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) {
                const uint64_t o_key = s_wave_key[side][w];
                const int o_best = s_wave_best[side][w];
                if (o_key < b_key || (o_key == b_key && o_best < best)) {
                    b_key = o_key;
                    best = o_best;
                }
            }
        }
        const int p = s_pos[best * S + i];
        const int32_t best_row = s_row_of[best];
        if (round == 0) first_row = best_row;
        if (i == 0) {
            selected_list[round] = best;
            selected_rows[round] = best_row;
            selected_out[best] = 1;
            if (order_out != nullptr) order_out[round] = best;
        }
        if (i == best) {
            left = false;
            lo = 0;
            hi = 0;
        } else if (left && (lo | hi) != 0) {
            const bool is_term = ((p < 64 ? lo >> p : hi >> (p - 64)) & 1ull) != 0;
            const int gone = is_term ? p : (hi != 0 ? 127 - __builtin_clzll(hi) : 63 - __builtin_clzll(lo));
            const uint64_t bit = 1ull << (gone & 63);
            lo &= gone < 64 ? ~bit : ~0ull;
            hi &= gone < 64 ? ~0ull : ~bit;
            s_rows[place(gone)] = 0.0;
        }
    }
    // rows of the chosen vectors for the second phase; the spare entries of the whole table
    // (the second phase's network may have more wires than there are vectors) repeat the first one
    for (int e = i; e < kMaxKrum; e += S)
        if (e >= theta) selected_rows[e] = first_row;
    if (i == 0) *n_selected = theta;
}

// Whether the m guessed vectors are Multi-Krum's choice, found by every wave for itself (lane = vector) from the upper
// words of the scores; where those tie or are NaN the answer is no.
__device__ __forceinline__ bool guess_holds(uint64_t guess, double score, int f, int m) {
    if (__builtin_popcountll(guess) != m) return false;
    const int i = threadIdx.x & 63;
    if (__builtin_amdgcn_ballot_w64(i < f && !(score >= 0.0)) != 0) return false;
    const uint32_t word = (uint32_t)__double2hiint(score);
    const bool in = ((guess >> i) & 1ull) != 0;
    return ~wave_min(in ? ~word : ~0u) < wave_min(in || i >= f ? ~0u : word);
}

// Choice and mean: every block chooses for itself (block 0 writes the choice; a kernel of its own for the choice
// took 5 us more: f = 25, 1 M 47.1 -> 45.7), then out[c] = mean of the chosen
// rows: fp32, added one by one in ascending file index starting from +0, one IEEE division by the count.  Thread t
// of the grid owns the words from min(4t, d-4) (d >= 4).  With a guess (f <= kMaxGuess) whose mean the Gram pass has
// written the blocks return when it was right.  A block per 4 * kBlock words: 2048
// blocks with a stride are idle for two thirds of the sixth round of 11.2 M coordinates (1819 with even rounds walk in step
// and are slower still).  us a call that takes its mean here, with a stride / now: 25 x 11.2 M 357.6 / 350.4, 49 x 11.2 M 709 /
// 692, 9 x 23 M 282 / 269; where the guess held 238.2 / 240.6 (245 with the full choice in front of the return).
__global__ __launch_bounds__(kBlock) void chosen_mean_kernel(const float *__restrict__ X, int64_t d, int64_t ld,
                                                             const int32_t *__restrict__ row_index,
                                                             const double *__restrict__ scores, int f, int m,
                                                             const uint64_t *__restrict__ guess,
                                                             int32_t *selected_out, float *__restrict__ out) {
    static_assert(kBlock >= kMaxKrum, "a thread per vector");
    __shared__ double s_score[kMaxKrum];
    __shared__ uint64_t s_chosen[kMaxKrum / 64];
    __shared__ int32_t s_row[kMaxKrum];
    const int i = threadIdx.x, own = guess != nullptr ? i & 63 : i;
    const double mine = own < f ? scores[own] : 0.0;
    if (guess != nullptr) {
        const uint64_t guessed = *guess;
        if (guess_holds(guessed, mine, f, m)) {
            if (blockIdx.x == 0 && i < f) selected_out[i] = (int32_t)((guessed >> i) & 1ull);
            return;
        }
    }
    int before, n;
    const bool chosen = choose_vector(mine, f, m, s_score, s_chosen, &before, &n) < m;
    n = __builtin_amdgcn_readfirstlane(n);
    if (blockIdx.x == 0 && i < f) selected_out[i] = chosen ? 1 : 0;
    if (guess != nullptr) {
        if (*guess == s_chosen[0]) return;
    }
    if (chosen) s_row[before] = row_index[i];
    __syncthreads();
    const int64_t gt = (int64_t)blockIdx.x * kBlock + i;
    if (gt >= (d + 3) / 4) return;
    const float dn = (float)n;
    const int64_t c0 = (gt + 1) * 4 <= d ? gt * 4 : d - 4;
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
    auto load = [&](int t) {
        const float *p = X + (int64_t)__builtin_amdgcn_readfirstlane(s_row[t]) * ld + c0;
        return __builtin_nontemporal_load(reinterpret_cast<const f32x4u *>(p));
    };
    auto add = [&](const f32x4u &v) { a0 += v[0]; a1 += v[1]; a2 += v[2]; a3 += v[3]; };
    int t = 0;
    for (; t + 4 <= n; t += 4) {
        f32x4u v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = load(t + u);
#pragma unroll
        for (int u = 0; u < 4; ++u) add(v[u]);
    }
    for (; t < n; ++t) add(load(t));
    f32x4u o;
    o[0] = a0 / dn; o[1] = a1 / dn; o[2] = a2 / dn; o[3] = a3 / dn;
    __builtin_nontemporal_store(o, reinterpret_cast<f32x4u *>(out + c0));
}

// Both on short rows, where a launch and the chain of loads count and not HBM: every block chooses for itself
// (block 0 writes the choice) and takes one word per thread, kAheadRows rows in flight; the additions are those
// of chosen_mean_kernel.  Figures at short_mean.
constexpr int kAheadRows = 32;
__global__ __launch_bounds__(kBlock) void choose_and_mean_kernel(const float *__restrict__ X, int64_t d, int64_t ld,
                                                                 const int32_t *__restrict__ row_index,
                                                                 const double *__restrict__ scores, int f, int m,
                                                                 int32_t *selected_out, float *__restrict__ out) {
    static_assert(kBlock >= kMaxKrum, "a thread per vector");
    __shared__ double s_score[kMaxKrum];
    __shared__ uint64_t s_chosen[kMaxKrum / 64];
    __shared__ int64_t s_first[kMaxKrum];  // first words of the chosen rows
    const int i = threadIdx.x;
    int before, n;
    const bool chosen = choose_vector(i < f ? scores[i] : 0.0, f, m, s_score, s_chosen, &before, &n) < m;
    if (blockIdx.x == 0 && i < f) selected_out[i] = chosen ? 1 : 0;
    if (chosen) s_first[before] = (int64_t)row_index[i] * ld;
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * kBlock + i;
    if (c >= d) return;
    float a = 0.0f;
    for (int t = 0; t < n; t += kAheadRows) {
        float v[kAheadRows];
#pragma unroll
        for (int u = 0; u < kAheadRows; ++u) v[u] = t + u < n ? X[s_first[t + u] + c] : 0.0f;
#pragma unroll
        for (int u = 0; u < kAheadRows; ++u) a = t + u < n ? a + v[u] : a;
    }
    out[c] = a / (float)n;
}

struct KrumWorkspace {
    double gram[kMaxPairs * kTile];
    double sorted_dist[kMaxKrum * kRowStride];  // [t*kRowStride + i]: i's t-th smallest distance
    union {
        double scores[kMaxKrum];
        SampleScores sample;
    };
    uint8_t sorted_nbr[kMaxKrum * kRowStride];  // and the vector it leads to
    int32_t selected_list[kMaxKrum];
    int32_t selected_rows[kMaxKrum];  // Bulyan: rows of the chosen vectors, spare entries valid
    int32_t n_selected;
    int32_t pad[61];
    uint64_t guess;  // Multi-Krum: the vectors the Gram pass has averaged, bit i = vector i
    float partial[1];  // [kGramBlocks][tiles of f][256], sized by krum_workspace_bytes
};
static_assert(offsetof(KrumWorkspace, partial) % sizeof(double) == 0, "partial tiles may be fp64");
static_assert(2 * stored_tiles(kMaxGuess) <= kMaxPairs && kSampleBlocks % 8 == 0, "room for both halves' matrices");

// Blocks up to which partial tiles are fp64: a quarter of the grid they have room for in fp32.
inline bool partials_in_fp64(int grid) { return grid <= kGramBlocks / 4; }

inline size_t krum_workspace_bytes(int f) {
    // (callers know this size: beyond 64 vectors it has room for 6 or 8 row tiles, whatever is used)
    const int nt = f <= 64 ? (f + 15) / 16 : (f <= 96 ? 6 : 8);
    return offsetof(KrumWorkspace, partial) +
           sizeof(float) * (size_t)kGramBlocks * (nt * (nt + 1) / 2) * kTile;
}

// What a Gram pass is for: the whole matrix, the matrix of a sample, or the whole with a guessed mean (guess.out set).
struct GramPass {
    bool sample;
    GuessedPass guess;
};
constexpr GramPass kWholeMatrix = {false, {nullptr, 0, nullptr, nullptr}}, kSampleMatrix = {true, kWholeMatrix.guess};

template <int NT, int NG, int SF, bool LINES, bool MEAN>
void launch_gram_spans(const float *rows_base, int64_t d, int64_t ld, const int32_t *row_index_dev,
                       int f, float *partial, int *grid, GramPass pass, hipStream_t s) {
    constexpr int kWaves = gram_waves(NT, SF);
    constexpr int64_t kSpan = kStep * SF * kWaves;  // coordinates a block takes at a time
    // up to a block per CU each takes one step, then up to the full grid each takes two: a block more is
    // a partial matrix more to write and add (128 x 50001 62.9 us, one step each 73.9; 96 x 50001 48.7
    // and 51.3)
    const int64_t steps = (d + kSpan - 1) / kSpan;
    int64_t n = steps;
    if (n > kGramBlocks / 2) n = n > kGramBlocks ? (n + 1) / 2 : kGramBlocks / 2;
    *grid = n < 1 ? 1 : (n < kGramBlocks ? (int)n : kGramBlocks);  // d == 0: one block writes zero tiles
    const int in_fp64 = partials_in_fp64(*grid) ? 1 : 0;
    // up to four steps a wave; two steps of 32 at a time are taken on longer rows only
    if (!MEAN && SF == 1 && steps <= 4 * (int64_t)*grid)
        gram_partial_kernel<NT, NG, 1, LINES, SF == 1 ? Gram::kShort : Gram::kLong><<<*grid, 64 * gram_waves(NT, 1), 0, s>>>(
            rows_base, d, ld, row_index_dev, f, partial, in_fp64, 0, pass.guess);
    else
        gram_partial_kernel<NT, NG, SF, LINES, MEAN ? Gram::kMean : Gram::kLong><<<*grid, 64 * kWaves, 0, s>>>(
            rows_base, d, ld, row_index_dev, f, partial, in_fp64, 0, pass.guess);
}

template <int NT, int NG, bool LINES>
void launch_gram_rows(const float *rows_base, int64_t d, int64_t ld, const int32_t *row_index_dev,
                      int f, float *partial, int *grid, GramPass pass, hipStream_t s) {
    // Long rows: two steps at a time up to 32 vectors (four steps per wave or fewer: one at a time
    // spreads them over more waves and partial sums).  Above, more registers and fewer waves cost more
    // than longer pieces of a row give, but for rows off the cache lines that are far larger than the
    // last-level cache (48 x 11.2 M 596 -> 584 us, 64 x 11.2 M 857 -> 804; 64 x 3 M 231 -> 232).
    constexpr int SF = NT <= 2 || (NT + (NG > 0 ? 1 : 0) <= 4 && !LINES) ? 2 : 1;
    const int64_t one_at_a_time = (int64_t)1 << (NT <= 1 ? 20 : (NT <= 2 ? 19 : 22));
    const bool two_steps = SF > 1 && d > one_at_a_time;  // whatever the pass is for: the order of the additions
    if constexpr (16 * NT + 4 * NG <= kMaxGuess) {
        if (pass.sample) {
            *grid = kSampleBlocks;
            gram_partial_kernel<NT, NG, 1, LINES, Gram::kSample><<<kSampleBlocks, 64 * kSampleWaves, 0, s>>>(
                rows_base, d, ld, row_index_dev, f, partial, 0, d / kSampleSpans / kStep * kStep, pass.guess);
            return;
        }
        if (pass.guess.out != nullptr) {
            if constexpr (NT <= 2)  // such rows are long enough for two steps at a time (guess_pays)
                launch_gram_spans<NT, NG, SF, LINES, true>(rows_base, d, ld, row_index_dev, f, partial, grid, pass, s);
            else if (two_steps)
                launch_gram_spans<NT, NG, SF, LINES, true>(rows_base, d, ld, row_index_dev, f, partial, grid, pass, s);
            else
                launch_gram_spans<NT, NG, 1, LINES, true>(rows_base, d, ld, row_index_dev, f, partial, grid, pass, s);
            return;
        }
    }
    if (two_steps)
        launch_gram_spans<NT, NG, SF, LINES, false>(rows_base, d, ld, row_index_dev, f, partial, grid, pass, s);
    else
        launch_gram_spans<NT, NG, 1, LINES, false>(rows_base, d, ld, row_index_dev, f, partial, grid, pass, s);
}

inline bool rows_on_lines(const float *rows_base, int64_t ld) {
    return ((uintptr_t)rows_base & 127u) == 0 && ld % 32 == 0;
}

template <int NT, int NG>
int launch_gram_shape(const float *rows_base, int64_t d, int64_t ld, const int32_t *row_index_dev,
                      int f, float *partial, int *grid, GramPass pass, hipStream_t s) {
    if (rows_on_lines(rows_base, ld))
        launch_gram_rows<NT, NG, true>(rows_base, d, ld, row_index_dev, f, partial, grid, pass, s);
    else
        launch_gram_rows<NT, NG, false>(rows_base, d, ld, row_index_dev, f, partial, grid, pass, s);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

// Gram matrix of the f rows into ws->gram (partial tiles, then the fp64 reduction; of a sample its two halves').
int launch_gram(const float *rows_base, int64_t d, int64_t ld, const int32_t *row_index_dev, int f,
                KrumWorkspace *ws, GramPass pass, hipStream_t s) {
    int rc, grid = 0;
    switch (4 * row_tiles(f) + row_groups(f)) {
#define BYZ_GRAM_SHAPE(nt, ng)                                                                           \
    case 4 * (nt) + (ng):                                                                                \
        rc = launch_gram_shape<nt, ng>(rows_base, d, ld, row_index_dev, f, ws->partial, &grid, pass, s); \
        break;
        BYZ_GRAM_SHAPE(1, 0) BYZ_GRAM_SHAPE(2, 0) BYZ_GRAM_SHAPE(3, 0) BYZ_GRAM_SHAPE(4, 0)
        BYZ_GRAM_SHAPE(5, 0) BYZ_GRAM_SHAPE(6, 0) BYZ_GRAM_SHAPE(7, 0) BYZ_GRAM_SHAPE(8, 0)
        BYZ_GRAM_SHAPE(2, 1) BYZ_GRAM_SHAPE(3, 1) BYZ_GRAM_SHAPE(3, 2) BYZ_GRAM_SHAPE(4, 1) BYZ_GRAM_SHAPE(5, 1)
        BYZ_GRAM_SHAPE(6, 1) BYZ_GRAM_SHAPE(6, 2) BYZ_GRAM_SHAPE(6, 3)
        BYZ_GRAM_SHAPE(7, 1) BYZ_GRAM_SHAPE(7, 2) BYZ_GRAM_SHAPE(7, 3)
#undef BYZ_GRAM_SHAPE
        default: return BYZ_EINTERNAL;
    }
    if (rc != BYZ_OK) return rc;
    const int ntiles = stored_tiles(f);
    if (pass.sample)
        gram_reduce_kernel<float, true><<<ntiles * kTile / 32, kBlock, 0, s>>>(ws->partial, grid, ntiles, ws->gram);
    else if (partials_in_fp64(grid))
        gram_reduce_kernel<double, false><<<ntiles * kTile / 32, kBlock, 0, s>>>(
            reinterpret_cast<const double *>(ws->partial), grid, ntiles, ws->gram);
    else
        gram_reduce_kernel<float, false><<<ntiles * kTile / 32, kBlock, 0, s>>>(ws->partial, grid, ntiles, ws->gram);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

// Sorted distance rows (and Krum scores when n_terms >= 0) from ws->gram.
int launch_distance_rows(int f, int n_terms, double *dist_out, double *scores_out, KrumWorkspace *ws,
                         hipStream_t s) {
    const int row_blocks = (f + kBlock / 64 - 1) / (kBlock / 64);
    if (f <= 64)
        distance_rows_kernel<1><<<row_blocks, kBlock, 0, s>>>(ws->gram, f, n_terms, dist_out,
                                                              ws->sorted_dist, ws->sorted_nbr,
                                                              ws->scores, scores_out);
    else
        distance_rows_kernel<2><<<row_blocks, kBlock, 0, s>>>(ws->gram, f, n_terms, dist_out,
                                                              ws->sorted_dist, ws->sorted_nbr,
                                                              ws->scores, scores_out);
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

}  // namespace

extern "C" size_t byz_multi_krum_workspace_bytes(int f) {
    if (f < 1 || f > kMaxKrum) return 0;
    return krum_workspace_bytes(f);
}

// Rows up to which the choice is made in the blocks of the mean; its narrow loads cost more where rows are not on cache
// lines.  us a call, two kernels / one: f = 25 d = 1003 21.3 / 18.6, 131072 23.9 / 21.0, 393216 31.5 / 31.5 off the lines and
// 35.3 / 31.2 on them, 700000 37.4 / 38.9; f = 31 300001 31.2 / 30.6 and 33.4 / 31.3, 360001 32.5 / 33.3 and 34.9 / 33.5;
// f = 33 327680 34.5 / 33.3 off; f = 60 262144 47.3 / 48.0 and 50.5 / 47.5, 300001 50.6 / 52.0 and 52.7 / 51.0, 393216 57.1 / 59.3 and 57.8 / 58.0; f = 127 1003
// 45.2 / 41.8, 100003 87.2 / 75.0, 262144 119 / 121 and 127 / 122, 327680 143 / 146 and 136 / 137, 393216 157 / 162 and 147 / 152.
constexpr int64_t short_mean(int f, bool lines) {
    if (lines) return f <= 96 ? 3 << 17 : 5 << 16;
    return f <= 25 ? 3 << 17 : (f <= 40 ? 5 << 16 : 1 << 18);
}

// Where the mean is taken on the way: m rows fewer to read against the sample with its reduction and scores (16 us up
// to 32 vectors, 20 above), the additions (about what a quarter of the rows takes to read: vector and matrix
// instructions share one datapath) and the output written meanwhile.  More than 64 vectors leave no registers.  Where no
// guess is made, as on rows of one distribution, the sample is lost, so the two passes have to be 1.4 GB or more.
// us a call, in two passes / right / none / wrong: f = 25 m = 20 11.2 M 331 / 238 / 347 / 387, off the lines 354 / 257 / 367,
// 7.9 M 241 / 176 / 255 / 283 (the line; 5.6 M 175 / 131 / 188 / 207); f = 9 m = 7 23 M 267 / 192 / 266 / 304; f = 16 m = 14 11.8 M 242 / 166 /
// 254 / 280; f = 33 m = 28 5.8 M 244 / 176 / 259 / 278; f = 49 m = 40 11.2 M 698 / 520 / 702 / 797, 4 M 260 / 205 / 274 / 310; f = 64
// m = 54 3 M 259 / 204 / 277 / 308.
constexpr bool guess_pays(int f, int m, int64_t d) {
    return f <= kMaxGuess && (int64_t)(f + m) * d >= 350000000 &&
           (int64_t)(m - 2 - f / 4) * d >= (f <= 32 ? (int64_t)1 << 26 : (int64_t)3 << 25);
}

extern "C" int byz_multi_krum(const float *rows_base, int64_t d, int64_t ld,
                              const int32_t *row_index_dev, int f, int c, int m, float *out,
                              int32_t *selected_out, double *scores_out, double *dist_out,
                              void *workspace, size_t workspace_bytes, void *stream) {
    if (rows_base == nullptr || row_index_dev == nullptr || selected_out == nullptr ||
        workspace == nullptr || (out == nullptr && d > 0))
        return BYZ_EINVAL;
    if (d < 0 || ld < d || d > ((int64_t)1 << 30)) return BYZ_EINVAL;
    if (f < 3 || f > kMaxKrum || c < 0 || f < 2 * c + 3) return BYZ_EINVAL;  // Sec. 6.1
    if (m < 1 || m > f - c) return BYZ_EINVAL;
    if (((uintptr_t)workspace & 255u) != 0) return BYZ_EINVAL;
    if (workspace_bytes < krum_workspace_bytes(f)) return BYZ_ENOMEM;
    hipStream_t s = (hipStream_t)stream;
    KrumWorkspace *ws = reinterpret_cast<KrumWorkspace *>(workspace);
    int rc;
    const bool guess = guess_pays(f, m, d);
    if (guess) {
        rc = launch_gram(rows_base, d, ld, row_index_dev, f, ws, kSampleMatrix, s);
        if (rc != BYZ_OK) return rc;
        sample_scores_kernel<<<f, 64, 0, s>>>(ws->gram, f, f - c - 2, &ws->sample);
        BYZ_HIP(hipGetLastError());
    }
    rc = launch_gram(rows_base, d, ld, row_index_dev, f, ws,
                     guess ? GramPass{false, {&ws->sample, m, out, &ws->guess}} : kWholeMatrix, s);
    if (rc != BYZ_OK) return rc;
    rc = launch_distance_rows(f, f - c - 2, dist_out, scores_out, ws, s);
    if (rc != BYZ_OK) return rc;
    if (d <= short_mean(f, rows_on_lines(rows_base, ld))) {
        const int64_t blocks = d > 0 ? (d + kBlock - 1) / kBlock : 1;  // d == 0: the choice alone
        choose_and_mean_kernel<<<(unsigned)blocks, kBlock, 0, s>>>(
            rows_base, d, ld, row_index_dev, ws->scores, f, m, selected_out, out);
    } else {
        chosen_mean_kernel<<<(unsigned)(((d + 3) / 4 + kBlock - 1) / kBlock), kBlock, 0, s>>>(
            rows_base, d, ld, row_index_dev, ws->scores, f, m, guess ? &ws->guess : nullptr, selected_out, out);
    }
    BYZ_HIP(hipGetLastError());
    return BYZ_OK;
}

extern "C" size_t byz_bulyan_workspace_bytes(int f) { return byz_multi_krum_workspace_bytes(f); }

extern "C" int byz_bulyan(const float *rows_base, int64_t d, int64_t ld,
                          const int32_t *row_index_dev, int f, int c, float *out,
                          int32_t *selected_out, int32_t *order_out, double *dist_out,
                          void *workspace, size_t workspace_bytes, void *stream) {
    if (rows_base == nullptr || row_index_dev == nullptr || selected_out == nullptr ||
        workspace == nullptr || (out == nullptr && d > 0))
        return BYZ_EINVAL;
    if (d < 0 || ld < d || d > ((int64_t)1 << 30)) return BYZ_EINVAL;
    if (f < 3 || f > kMaxKrum || c < 0 || f < 4 * c + 3) return BYZ_EINVAL;  // Sec. 6.1
    if ((f % 2) == 0) return BYZ_EUNSUPPORTED;  // the median of the f - 2c chosen values must be one of them
    if (((uintptr_t)workspace & 255u) != 0) return BYZ_EINVAL;
    if (workspace_bytes < krum_workspace_bytes(f)) return BYZ_ENOMEM;
    hipStream_t s = (hipStream_t)stream;
    KrumWorkspace *ws = reinterpret_cast<KrumWorkspace *>(workspace);
    int rc = launch_gram(rows_base, d, ld, row_index_dev, f, ws, kWholeMatrix, s);
    if (rc != BYZ_OK) return rc;
    rc = launch_distance_rows(f, -1, dist_out, nullptr, ws, s);
    if (rc != BYZ_OK) return rc;
    if (f <= BYZ_MAX_F) {
        const size_t lds = (size_t)select_terms(f, c) * 64 * sizeof(double) + (size_t)f * 64;
        bulyan_select_kernel<1><<<1, kSelectThreads, lds, s>>>(
            ws->sorted_dist, ws->sorted_nbr, f, c, selected_out, order_out, ws->selected_list,
            &ws->n_selected, row_index_dev, ws->selected_rows);
    } else {
        const size_t lds = (size_t)select_terms(f, c) * 128 * sizeof(double) + (size_t)f * 128;
        BYZ_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&bulyan_select_kernel<2>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        bulyan_select_kernel<2><<<1, kSelectThreads, lds, s>>>(
            ws->sorted_dist, ws->sorted_nbr, f, c, selected_out, order_out, ws->selected_list,
            &ws->n_selected, row_index_dev, ws->selected_rows);
    }
    BYZ_HIP(hipGetLastError());
    const int theta = f - 2 * c;
    return byz_internal_launch_bulyan_mean(rows_base, d, ld, ws->selected_rows, f, theta,
                                           theta - 2 * c, out, stream);
}

extern "C" int byz_mean_around_median(const float *rows_base, int64_t d, int64_t ld,
                                      const int32_t *row_index_dev, int f, int beta, float *out,
                                      void *stream) {
    if (rows_base == nullptr || row_index_dev == nullptr || (out == nullptr && d > 0))
        return BYZ_EINVAL;
    if (d < 0 || ld < d || d > ((int64_t)1 << 30)) return BYZ_EINVAL;
    if (f < 1 || f > kMaxKrum || beta < 1 || beta > f) return BYZ_EINVAL;
    if ((f % 2) == 0) return BYZ_EUNSUPPORTED;  // the median must be one of the values
    return byz_internal_launch_bulyan_mean(rows_base, d, ld, row_index_dev, f, f, beta, out, stream);
}
