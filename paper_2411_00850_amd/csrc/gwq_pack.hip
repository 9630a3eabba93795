// gwq_pack on gfx950: outlier selection (Sec. 3.2, Eq. 8) by the bit patterns of |score|, from a sampled band of them or by a
// radix select over all, CSR build in flat-index order, then per (row, group of 16 to 128) the scale,
// zero point and codes of Eq. 6, 7 and 9 and the word layout documented in gwq.h.
//
// Everything is integer work or arithmetic whose result is that of exact arithmetic rounded once (see the encoder),
// so the output is a function of the inputs alone.  Integer atomics are used for the
// histograms (order-independent); there are no floating-point atomics.
#include <algorithm>
#include <type_traits>

#include "gwq_internal.h"

#pragma clang fp contract(off)

namespace gwq {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kElemsPerThread = 8;
constexpr int kElemsPerIter = kThreads * kElemsPerThread;   // 2048 = 16 groups

// Ranking key: bit pattern of |score| as binary32 (monotone in the magnitude, NaN on top).
__device__ inline uint32_t key_from_f32(uint32_t bits) { return bits & 0x7FFFFFFFu; }

__device__ inline uint32_t key_from_f16(uint16_t h)
{
    const uint32_t e = (h >> 10) & 0x1F, f = h & 0x3FF;
    if (e == 31) return 0x7F800000u | (f << 13);                 // inf / NaN keep their payload
    const float v = (float)__builtin_bit_cast(_Float16, (uint16_t)(h & 0x7FFF));  // exact widening
    return __builtin_bit_cast(uint32_t, v);
}

// Digit of a key in pass 0, 1, 2 (11 + 11 + 9 bits of the 31-bit key) and the bits above it.
template <int PASS> __device__ inline uint32_t digit_of(uint32_t key)
{
    return PASS == 0 ? key >> 20 : PASS == 1 ? (key >> 9) & 0x7FFu : key & 0x1FFu;
}
template <int PASS> __device__ inline bool prefix_matches(uint32_t key, uint32_t prefix)
{
    return PASS == 0 ? true : PASS == 1 ? (key >> 20) == (prefix >> 20) : (key >> 9) == (prefix >> 9);
}

template <bool F16> __device__ inline void load_keys8(const void *score, size_t idx, uint32_t key[8])
{
    if (F16) {
        const uint4 v = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(score) + idx);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            key[2 * i] = key_from_f16((uint16_t)(w[i] & 0xFFFF));
            key[2 * i + 1] = key_from_f16((uint16_t)(w[i] >> 16));
        }
    } else {
        const uint4 *p = reinterpret_cast<const uint4 *>(static_cast<const uint32_t *>(score) + idx);
        const uint4 a = p[0], b = p[1];
        key[0] = key_from_f32(a.x); key[1] = key_from_f32(a.y);
        key[2] = key_from_f32(a.z); key[3] = key_from_f32(a.w);
        key[4] = key_from_f32(b.x); key[5] = key_from_f32(b.y);
        key[6] = key_from_f32(b.z); key[7] = key_from_f32(b.w);
    }
}

__device__ inline uint32_t wave_inclusive_scan(uint32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(v, d);
        if (lane >= d) v += t;
    }
    return v;
}

// Exclusive scan of one value per thread over the block, plus the block total.
template <int WAVES> __device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t *smem, uint32_t &total)
{
    const uint32_t inc = wave_inclusive_scan(v);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 63) smem[w] = inc;
    __syncthreads();
    uint32_t base = 0, sum = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        const uint32_t s = smem[i];
        if (i < w) base += s;
        sum += s;
    }
    total = sum;
    return base + inc - v;
}

// ---- the selection ---------------------------------------------------------------------------------
//
// Up to kScoresUpTo scores: a radix select over all of them in digits of 11, 11 and 9 bits (FP16 scores: two digits).  Beyond:
// a sample of 32768 keys gives a band of keys that holds the threshold (five standard deviations of the rank on either
// side: 0.6 % of the keys at 1 % outliers).  One pass over the scores then counts per row the keys above the band and
// collects those inside it - the candidates - and what is left works on that short list: the threshold's offset in the band
// by digits from its top bit down, and the per-row counts.  A band of a single key (scores of few distinct values) needs no
// list: its keys are counted.  Where the counts say that the threshold lies outside the band, or a row has more candidates
// than its part of the list holds, the same launches do the radix select over all scores instead; which of the two, every
// block works out for itself from the same counts, so the choice costs no host synchronisation, and both give the same bytes.
//
// What bounds it: the one pass (180 MB of FP32 scores, 11008 x 4096: 36 us, 5.0 TB/s), then launches, 4.5 us each beside it,
// so a kernel picks the digit that its predecessor has counted (every block does, from 8 KB).  It was a pass over all scores
// for the first digit, 40 us, and one that collected the keys of the threshold's first digit and added each to a histogram in
// global memory by itself: 29 us where those are 0.2 % of all, 250 for uniform scores, 16 ms where all are equal.
//
// The line: sample, band and candidates are three launches and 20 us (a block for the band alone takes 10), which a pass over
// all scores takes less than from the caches up to about nine million of them.  us of a whole gwq_pack replayed from a graph,
// 4 bits, 1 % outliers: the histograms in global memory / by list / by scores, * the one taken ("few rows": all outliers
// in 2 % of the rows, which by list ends by scores), with an encoder that took 1 to 4 us
// more and the launch of row_scan_kernel on all sides:
//     scores                  512 x 512        1000 x 2048        1024 x 4096        1024 x 8192       11008 x 1024        4096 x 4096
//     normal, FP32        35 / 39 / 29*      46 / 40 / 36*      54 / 44 / 44*      70 / 56 / 56*      86 / 70* / 79      94 / 70* / 89
//     normal, FP16        30 / 33 / 26*      41 / 37 / 34*      49 / 42 / 40*      65 / 54 / 54*      77 / 67* / 68      90 / 66* / 73
//     uniform, FP32       38 / 37 / 29*      67 / 40 / 41*      87 / 45 / 47*     122 / 56 / 57*     149 / 70* / 80     187 / 70* / 90
//     in order            35 / 41 / 28*      49 / 49 / 33*      63 / 60 / 40*      99 / 76 / 50*     125 / 99* / 74    161 / 115* / 87
//     few rows            36 / 42 / 29*      46 / 49 / 35*      56 / 60 / 42*      78 / 76 / 53*      92 / 97* / 75    108 / 108* / 87
//     51 values           95 / 37 / 29*     344 / 54 / 39*     656 / 63 / 45*    1270 / 77 / 55*   1689 / 106* / 78   2485 / 116* / 89
//     all equal          226 / 59 / 29*    791 / 143 / 38*   1576 / 146 / 46*   3115 / 155 / 57*   4165 / 167* / 76   6179 / 172* / 89
// Larger, normal scores: 11008 x 4096 193 / 124*, 8192 x 28672 895 / 592*.
constexpr size_t kScoresUpTo = (size_t)8 << 20;
enum Way { kByList = 1, kByScores = 2, kSingleKey = 3 };        // what the launches found, in the workspace

// Where a row's outliers start is the count of what the rows before it keep.  Up to kSummedRows rows each wave of the encoder
// adds that up for itself (rows_before), from the rows of its own block of rows and the sums of the blocks before it, which
// rows_kernel has made, and writes row_ptr; beyond, one block of threads does it for all rows (row_scan_kernel), a launch that
// waits for the one before and takes 4.0 us up to 4096 rows, 8.2 at 11008.  The sums are added up with atomics, and those on one
// line are served one after another, 15 ns each: a line for each sum, several rows to an atomic, and up to 1024 rows are a
// single block, which needs none.  The line: a wave reads a line for every 256 rows before its own.  us of a whole gwq_pack replayed
// from a graph, 4 bits, with the launch / without:
//     scores         64 x 512      1024 x 4096    4096 x 4096    11008 x 4096     28672 x 1024     65536 x 128      65536 x 1024     131072 x 1024
//     FP32        26.8 / 23.8*    43.0 / 40.3*   67.0 / 63.8*   118.7 / 111.4*   115.2 / 98.7*   154.2 / 128.5*   241.0 / 234.0*   450.1* / 487.2
//     FP16        24.1 / 21.0*    38.6 / 36.7*   62.6 / 59.9*   104.8 / 97.7*    108.2 / 95.0*   164.0 / 132.8*   203.6 / 194.5*   399.7* / 437.3
constexpr int kSummedRows = 65536, kSumStride = 32;     // words from one block's sums to the next
__host__ __device__ constexpr int block_rows_log2(int N) { return N <= 1024 ? 10 : 8; }
__device__ inline uint32_t *block_sums(uint32_t *ws, int N) { return ws + kWsRows + 2 * (size_t)N; }
// Adds to the sums of row n's block: keys above the threshold and equal to it.  The last block's nobody reads.
__device__ inline void add_to_block(uint32_t *ws, int N, int n, uint32_t gt, uint32_t eq)
{
    const int b = n >> block_rows_log2(N);
    if (N > kSummedRows || b >= (N - 1) >> block_rows_log2(N)) return;
    uint32_t *s = block_sums(ws, N) + (size_t)b * kSumStride;
    if (gt) atomicAdd(&s[0], gt);
    if (eq) atomicAdd(&s[1], eq);
}

// The sample: pieces of 16 bytes, one at a pseudo-random place of each of as many equal parts of the scores - one of 32 there
// are, 8192 (FP16 scores: 4096) at most; as keys into the part of the workspace where the candidates come later, which holds
// total / 32 words.  Many blocks: 8192 lines are a megabyte, and one compute unit that reads it takes 15 us.  Clears the
// counters on the way; parts = 0: that alone, and the selection goes by scores.
constexpr uint32_t kSampleKeys = 32768;
struct __attribute__((packed, aligned(4))) Keys4 { uint32_t k[4]; };     // the workspace is aligned to four bytes only
inline uint32_t sample_keys(size_t total) { return total / 32 < kSampleKeys ? (uint32_t)(total / 256 * 8) : kSampleKeys; }
template <bool F16>
__global__ __launch_bounds__(kThreads) void sample_kernel(const void *__restrict__ score, uint64_t total, uint32_t *ws, int N, uint32_t parts,
                                                          uint32_t k_out)
{
    constexpr int kKeys = F16 ? 8 : 4;
    const uint32_t j = blockIdx.x * kThreads + threadIdx.x, threads = gridDim.x * kThreads;
    for (uint32_t i = j; i < kWsRows; i += threads) ws[i] = i == kWsWanted ? k_out : i == kWsCandOverflow ? parts == 0 : 0u;
    for (uint32_t i = j; i < 3 * kSpread; i += threads) ws[kWsRows + 3 * N + i] = 0;
    if (N <= kSummedRows)
        for (uint32_t i = j; i < 2u * (uint32_t)((N - 1) >> block_rows_log2(N)); i += threads) block_sums(ws, N)[i / 2 * kSumStride + i % 2] = 0;
    if (j >= parts) return;
    const uint64_t pieces = total / kKeys;              // total is a multiple of 128
    const uint64_t lo = j * pieces / parts, hi = (j + 1) * pieces / parts;
    const uint64_t at = lo + (((uint64_t)(j * 2654435761u) * (hi - lo)) >> 32);
    const uint4 raw = static_cast<const uint4 *>(score)[at];
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
    uint32_t key[kKeys];
#pragma unroll
    for (int i = 0; i < kKeys; ++i) key[i] = F16 ? key_from_f16((uint16_t)(w[i / 2 % 4] >> (16 * (i & 1)))) : key_from_f32(w[i % 4]);
    Keys4 *out = reinterpret_cast<Keys4 *>(ws + pack_keys_at(N) + (size_t)j * kKeys);
#pragma unroll
    for (int i = 0; i < kKeys / 4; ++i) out[i] = Keys4{{key[4 * i], key[4 * i + 1], key[4 * i + 2], key[4 * i + 3]}};
}

// The band, by one block.  Its ends are exact keys where both share 22 bits (then they may be the same key), otherwise the ends
// of their ranges of 512 keys.  The first digit's few bins take most of the keys: eight copies of it, one per lane of eight,
// each on banks of its own.
constexpr int kBandThreads = 1024, kCopies = 8, kCopyStride = kSelBins + 8;
__global__ __launch_bounds__(kBandThreads) void band_kernel(uint32_t *ws, int N, uint32_t sampled, float share)
{
    constexpr int kRounds = kSampleKeys / 4 / kBandThreads;
    __shared__ uint32_t h[kCopies * kCopyStride], smem[kBandThreads / 64];
    __shared__ uint32_t found_digit[2], found_rest[2];
    const int tid = threadIdx.x;
    const Keys4 *sample = reinterpret_cast<const Keys4 *>(ws + pack_keys_at(N));
    uint32_t key[kRounds][4];
#pragma unroll
    for (int q = 0; q < kRounds; ++q) {
        const uint32_t at = tid + q * kBandThreads;
        Keys4 v = {{~0u, ~0u, ~0u, ~0u}};
        if (4 * at < sampled) v = sample[at];
#pragma unroll
        for (int i = 0; i < 4; ++i) key[q][i] = v.k[i];
    }

    // Ranks from the top: of the band's lower end and of its upper end.  0: the band is open at that end.
    const float r = share * (float)sampled, m = 5.f * __builtin_sqrtf(r) + 8.f;
    uint32_t rank[2] = {r + m < (float)sampled ? (uint32_t)(r + m) : 0u, r - m >= 1.f ? (uint32_t)(r - m) : 0u};
    uint32_t prefix[2] = {0u, 0u};
    const bool open_lo = rank[0] == 0, open_hi = rank[1] == 0;
    auto pass = [&](auto which) {
        constexpr int PASS = decltype(which)::value;
        for (int i = tid; i < (PASS == 0 ? kCopies * kCopyStride : 2 * kSelBins); i += kBandThreads) h[i] = 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kRounds; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t x = key[q][i];
                if (PASS == 0) {
                    if (!(x >> 31)) atomicAdd(&h[(tid & (kCopies - 1)) * kCopyStride + digit_of<PASS>(x)], 1u);
                } else {
                    if (prefix_matches<PASS>(x, prefix[0])) atomicAdd(&h[digit_of<PASS>(x)], 1u);
                    if (prefix_matches<PASS>(x, prefix[1])) atomicAdd(&h[kSelBins + digit_of<PASS>(x)], 1u);
                }
            }
        __syncthreads();
        // Keys of digits 2 tid and 2 tid + 1, for the lower end and, in the high halves, for the upper: 32768 at most.
        uint32_t b0 = 0, b1 = 0, sum;
        if (PASS == 0) {
#pragma unroll
            for (int i = 0; i < kCopies; ++i) b0 += h[i * kCopyStride + 2 * tid], b1 += h[i * kCopyStride + 2 * tid + 1];
            b0 |= b0 << 16;
            b1 |= b1 << 16;
        } else {
            b0 = h[2 * tid] | h[kSelBins + 2 * tid] << 16;
            b1 = h[2 * tid + 1] | h[kSelBins + 2 * tid + 1] << 16;
        }
        const uint32_t below = block_exclusive_scan<kBandThreads / 64>(b0 + b1, smem, sum);
        const uint32_t above = sum - below - b0 - b1;                    // (no borrow between the halves: sum of parts each)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t gt1 = above >> 16 * t & 0xFFFFu, gt0 = gt1 + (b1 >> 16 * t & 0xFFFFu), ge0 = gt0 + (b0 >> 16 * t & 0xFFFFu);
            if (rank[t] > gt1 && rank[t] <= gt0) found_digit[t] = 2 * tid + 1, found_rest[t] = rank[t] - gt1;
            if (rank[t] > gt0 && rank[t] <= ge0) found_digit[t] = 2 * tid, found_rest[t] = rank[t] - gt0;
        }
        __syncthreads();
        constexpr int shift = PASS == 0 ? 20 : PASS == 1 ? 9 : 0;
        for (int t = 0; t < 2; ++t)
            if (rank[t]) prefix[t] |= found_digit[t] << shift, rank[t] = found_rest[t];
    };
    pass(std::integral_constant<int, 0>{});
    pass(std::integral_constant<int, 1>{});
    if (open_lo || open_hi || prefix[0] != prefix[1]) {
        prefix[1] |= 0x1FFu;
    } else {
        __syncthreads();                                // `found` is read
        pass(std::integral_constant<int, 2>{});
    }
    if (tid == 0) {
        ws[kWsBandLo] = open_lo ? 0u : prefix[0];
        ws[kWsBandHi] = open_hi ? 0x7FFFFFFFu : prefix[1];
    }
}

// Nothing to select: the threshold sits above every key, no row keeps anything.
__global__ void nothing_kernel(uint32_t *ws, int N)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kWsRows + 3 * N; i += gridDim.x * blockDim.x)
        ws[i] = i == kWsPrefix ? 0xFFFFFFFFu : 0u;
}

// By list: the bits of an offset into the band that lie below its digit 0, 1 or 2 (9, 11 and 11 bits at most; the low 13 bits
// of FP16 scores' keys are all zero).  The first digit is the one that all candidates are counted for: few bins to add up.
template <bool F16> __device__ inline int bits_below(int digit, uint32_t lo, uint32_t hi)
{
    const int least = F16 ? 13 : 0, below = 32 - __builtin_clz((hi - lo) | 1u) - 9 - 11 * digit;
    return below > least ? below : least;
}
template <bool F16> __device__ inline bool is_last(int below) { return below == (F16 ? 13 : 0); }

// The pass over the scores: a block per row.
template <bool F16>
__global__ __launch_bounds__(kThreads) void candidates_kernel(const void *score, int K, uint32_t *ws, int N, int per_row)
{
    __shared__ uint32_t red[2][kWaves];
    __shared__ uint32_t count_s;
    const int n = blockIdx.x;
    if (threadIdx.x == 0) count_s = 0;
    __syncthreads();
    const uint32_t lo = ws[kWsBandLo], hi = ws[kWsBandHi], width = hi - lo;
    const bool single = width == 0;
    uint32_t *sums = ws + kWsRows + 3 * N, *counts = ws + pack_keys_at(N) - N, *keys = counts + N + (size_t)n * per_row;
    uint32_t gt = 0, eq = 0;
    uint32_t key[8], next[8];
    const size_t row = (size_t)n * K;
    if ((int)threadIdx.x * 8 < K) load_keys8<F16>(score, row + threadIdx.x * 8, next);
    for (int k = threadIdx.x * 8; k < K; k += kElemsPerIter) {
#pragma unroll
        for (int i = 0; i < 8; ++i) key[i] = next[i];
        if (k + kElemsPerIter < K) load_keys8<F16>(score, row + k + kElemsPerIter, next);
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            gt += key[i] > hi;
            mine += key[i] - lo <= width;
        }
        if (single) {
            eq += mine;
        } else if (mine) {
            uint32_t slot = atomicAdd(&count_s, mine);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (key[i] - lo <= width) {
                    if (slot < (uint32_t)per_row) keys[slot] = key[i];
                    ++slot;
                }
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) { gt += __shfl_xor(gt, d); eq += __shfl_xor(eq, d); }
    if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = gt; red[1][threadIdx.x >> 6] = eq; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t found = count_s;
        uint32_t a = 0, b = 0;
        for (int i = 0; i < kWaves; ++i) { a += red[0][i]; b += red[1][i]; }
        ws[kWsRows + n] = a;                            // rows_kernel adds the candidates above the threshold (or counts anew)
        ws[kWsRows + N + n] = b;
        counts[n] = found < (uint32_t)per_row ? found : (uint32_t)per_row;
        // The totals, over many addresses: one would serialise the rows.
        if (a) atomicAdd(&sums[n % kSpread], a);
        if (b) atomicAdd(&sums[kSpread + n % kSpread], b);
        if (found) atomicAdd(&sums[2 * kSpread + n % kSpread], found);
        if (found > (uint32_t)per_row) ws[kWsCandOverflow] = 1u;
    }
}

// The digit d of a histogram with (#keys with digit > d) < wanted <= (#keys with digit >= d), and wanted less the former;
// by every block for itself.
template <int THREADS>
__device__ inline void pick_digit(const uint32_t *hist, uint32_t wanted, uint32_t *smem, uint32_t &digit, uint32_t &rest)
{
    constexpr int PER = kSelBins / THREADS;
    __shared__ uint32_t found[2];
    uint32_t bin[PER], sum = 0, total;
#pragma unroll
    for (int i = 0; i < PER; ++i) { bin[i] = hist[PER * threadIdx.x + i]; sum += bin[i]; }
    if (threadIdx.x == 0) found[0] = 0, found[1] = wanted;
    uint32_t gt = block_exclusive_scan<THREADS / 64>(sum, smem, total);  // (its barriers also order the line above)
    gt = total - gt - sum;
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
        if (wanted > gt && wanted <= gt + bin[i]) found[0] = PER * threadIdx.x + i, found[1] = wanted - gt;
        gt += bin[i];
    }
    __syncthreads();
    digit = found[0];
    rest = found[1];
    __syncthreads();
}

// A block ends with atomics on the bins it has counted in, and those of all blocks on one line are served one after another:
// few large blocks, one for each CU over the scores and half as many over the list (11008 x 4096, 26 candidates a row, STEP 0:
// 344 blocks of 256 threads 14.4 us, 688 17.1, 128 of 1024 7.6).
constexpr int kDigitThreads = 1024, kScoreBlocks = 256, kListBlocks = 128;

// One digit of all scores into LDS, then to `g`.
template <int PASS, bool F16> __device__ inline void count_scores(const void *score, size_t total, uint32_t prefix, uint32_t *h, uint32_t *g)
{
    constexpr int shift = PASS == 0 ? 20 : PASS == 1 ? 9 : 0;
    const size_t stride = (size_t)gridDim.x * kDigitThreads * 8;
    for (size_t idx = ((size_t)blockIdx.x * kDigitThreads + threadIdx.x) * 8; idx < total; idx += stride) {
        uint32_t key[8];
        load_keys8<F16>(score, idx, key);
        uint32_t apart = 0;
#pragma unroll
        for (int i = 1; i < 8; ++i) apart |= key[i] ^ key[0];
        if (apart >> shift == 0) {                      // scores in order, or alike, would meet in one bin eight times
            if (prefix_matches<PASS>(key[0], prefix)) atomicAdd(&h[digit_of<PASS>(key[0])], 8u);
            continue;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (prefix_matches<PASS>(key[i], prefix)) atomicAdd(&h[digit_of<PASS>(key[i])], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kSelBins; i += kDigitThreads)
        if (h[i]) atomicAdd(&g[i], h[i]);
}

// Every candidate of every row: four rows to a wave, sixteen lanes each.  visit(key) once per candidate; row_done(n) by every
// lane of a row when it has seen its own.  A row's part holds 32 keys at least: those are loaded before the count is known.
template <int WAVES, typename Visit, typename RowDone>
__device__ inline void for_candidates(const uint32_t *ws, int N, int per_row, int blocks, Visit visit, RowDone row_done)
{
    const uint32_t *counts = ws + pack_keys_at(N) - N, *keys = counts + N;
    const int lane = threadIdx.x & 63, wave = blockIdx.x * WAVES + (threadIdx.x >> 6);
    for (int n0 = 4 * wave; n0 < N; n0 += 4 * WAVES * blocks) {
        const int n = n0 + (lane >> 4);
        const uint32_t *k = keys + (size_t)(n < N ? n : 0) * per_row + (lane & 15);
        const uint32_t k0 = k[0], k1 = k[16], count = n < N ? counts[n] : 0u, i0 = lane & 15;
        if (i0 < count) visit(k0);
        if (i0 + 16 < count) visit(k1);
#pragma unroll 4
        for (uint32_t i = i0 + 32; i < count; i += 16) visit(k[i - i0]);
        row_done(n);
    }
}

// Counts digit STEP, having picked the one before.  STEP 0 also decides the way.
template <int STEP, bool F16>
__global__ __launch_bounds__(kDigitThreads) void digit_kernel(const void *score, size_t total, uint32_t *ws, int N, int per_row)
{
    __shared__ uint32_t h[kSelBins], smem[kDigitThreads / 64];
    const uint32_t lo = ws[kWsBandLo], hi = ws[kWsBandHi], k_out = ws[kWsWanted];
    uint32_t way = ws[kWsWay], base = 0, wanted = k_out;
    if (STEP == 0) {
        const uint32_t *sums = ws + kWsRows + 3 * N;
        uint32_t sum[3];                                // above the band, of a single key, candidates
        static_assert(kSpread <= kDigitThreads, "a word a thread");
#pragma unroll
        for (int t = 0; t < 3; ++t)
            block_exclusive_scan<kDigitThreads / 64>(threadIdx.x < kSpread ? sums[t * kSpread + threadIdx.x] : 0u, smem, sum[t]);
        const uint32_t above = sum[0];
        const bool in = above < k_out && k_out - above <= (lo == hi ? sum[1] : sum[2]) && ws[kWsCandOverflow] == 0;
        way = !in ? kByScores : lo == hi ? kSingleKey : kByList;
        if (way != kByScores) base = lo, wanted = k_out - above;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            ws[kWsWay] = way;
            ws[kWsStep] = base;
            ws[kWsStep + 1] = wanted;
            if (way == kSingleKey) ws[kWsPrefix] = base, ws[kWsRemaining] = wanted;
        }
    }
    if (way == kSingleKey || (way == kByList && blockIdx.x >= kListBlocks)) return;
    if (STEP > 0) {
        base = ws[kWsStep + 2 * (STEP - 1)];
        wanted = ws[kWsStep + 2 * (STEP - 1) + 1];
        const int below = way == kByList ? bits_below<F16>(STEP - 1, lo, hi) : STEP == 1 ? 20 : 9;
        if (way == kByList && STEP == 2 && is_last<F16>(bits_below<F16>(0, lo, hi))) return;      // rows_kernel picks it
        if (way == kByList && is_last<F16>(below)) return;
        uint32_t digit;
        pick_digit<kDigitThreads>(ws + (STEP - 1) * kSelBins, wanted, smem, digit, wanted);
        base += digit << below;
        if (blockIdx.x == 0 && threadIdx.x == 0) ws[kWsStep + 2 * STEP] = base, ws[kWsStep + 2 * STEP + 1] = wanted;
    }
    for (int i = threadIdx.x; i < kSelBins; i += kDigitThreads) h[i] = 0;
    __syncthreads();
    uint32_t *g = ws + STEP * kSelBins;
    if (way == kByScores) {
        count_scores<STEP, F16>(score, total, base, h, g);
        return;
    }
    const int below = bits_below<F16>(STEP, lo, hi);
    const uint32_t last = STEP == 0 ? hi - lo : (1u << bits_below<F16>(STEP - 1, lo, hi)) - 1u;   // largest offset still open
    for_candidates<kDigitThreads / 64>(ws, N, per_row, min((int)gridDim.x, kListBlocks), [&](uint32_t key) {
        if (key - base <= last) atomicAdd(&h[(key - base) >> below], 1u);
    }, [](int) {});
    __syncthreads();
    for (int i = threadIdx.x; i < kSelBins; i += kDigitThreads)
        if (h[i]) atomicAdd(&g[i], h[i]);
}

// Picks the last digit, and per row: how many keys are above the threshold and how many are equal to it; and the sums of both
// over blocks of rows.
template <bool F16>
__global__ __launch_bounds__(kThreads) void rows_kernel(const void *score, int K, uint32_t *ws, int N, int per_row)
{
    __shared__ uint32_t red[2][kWaves], smem[kWaves];
    const uint32_t way = ws[kWsWay];
    if (way == kSingleKey) {                            // both are known
        if (N > kSummedRows) return;
        const int wave = blockIdx.x * kWaves + (threadIdx.x >> 6), lane = threadIdx.x & 63;
        for (int n0 = 64 * wave; n0 < N; n0 += 64 * kWaves * (int)gridDim.x) {
            uint32_t gt = 0, eq = 0;
            if (n0 + lane < N) gt = ws[kWsRows + n0 + lane], eq = ws[kWsRows + N + n0 + lane];
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) { gt += __shfl_xor(gt, d); eq += __shfl_xor(eq, d); }
            if (lane == 0) add_to_block(ws, N, n0, gt, eq);
        }
        return;
    }
    int last = F16 ? 1 : 2, below = 0;                  // the last digit counted
    if (way == kByList) {
        const uint32_t lo = ws[kWsBandLo], hi = ws[kWsBandHi];
        for (last = 0; !is_last<F16>(below = bits_below<F16>(last, lo, hi));) ++last;
    } else if (F16) {                                   // (the low 13 bits of every key are zero: two digits are all)
        below = 9;
    }
    uint32_t thr = ws[kWsStep + 2 * last], wanted = ws[kWsStep + 2 * last + 1], digit;
    pick_digit<kThreads>(ws + last * kSelBins, wanted, smem, digit, wanted);
    thr += digit << below;
    if (blockIdx.x == 0 && threadIdx.x == 0) ws[kWsPrefix] = thr, ws[kWsRemaining] = wanted;
    if (way == kByList) {
        uint32_t gt = 0, eq = 0;
        for_candidates<kWaves>(ws, N, per_row, (int)gridDim.x, [&](uint32_t key) {
            gt += key > thr;
            eq += key == thr;
        }, [&](int n) {
#pragma unroll
            for (int d = 8; d > 0; d >>= 1) { gt += __shfl_xor(gt, d); eq += __shfl_xor(eq, d); }
            if ((threadIdx.x & 15) == 0 && n < N) {
                gt += ws[kWsRows + n];
                ws[kWsRows + n] = gt;
                ws[kWsRows + N + n] = eq;
            } else {
                gt = eq = 0;
            }
            gt += __shfl_xor(gt, 16);                   // lane 0: the wave's four rows
            eq += __shfl_xor(eq, 16);
            gt += __shfl_xor(gt, 32);
            eq += __shfl_xor(eq, 32);
            if ((threadIdx.x & 63) == 0) add_to_block(ws, N, n, gt, eq);
            gt = eq = 0;
        });
        return;
    }
    // Neighbouring rows to a block of threads: one atomic for those of one block of rows.
    const int rows = (N + (int)gridDim.x - 1) / (int)gridDim.x, n_begin = (int)blockIdx.x * rows, n_end = min(n_begin + rows, N);
    uint32_t sum_gt = 0, sum_eq = 0;
    for (int n = n_begin; n < n_end; ++n) {
        uint32_t gt = 0, eq = 0;
        for (int k = threadIdx.x * 8; k < K; k += kElemsPerIter) {
            uint32_t key[8];
            load_keys8<F16>(score, (size_t)n * K + k, key);
#pragma unroll
            for (int i = 0; i < 8; ++i) { gt += key[i] > thr; eq += key[i] == thr; }
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) { gt += __shfl_xor(gt, d); eq += __shfl_xor(eq, d); }
        __syncthreads();                                // the row before is done with `red`
        if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = gt; red[1][threadIdx.x >> 6] = eq; }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t a = 0, b = 0;
            for (int i = 0; i < kWaves; ++i) { a += red[0][i]; b += red[1][i]; }
            ws[kWsRows + n] = a;
            ws[kWsRows + N + n] = b;
            sum_gt += a;
            sum_eq += b;
            if (n + 1 == n_end || (n + 1) >> block_rows_log2(N) != n >> block_rows_log2(N)) {
                add_to_block(ws, N, n, sum_gt, sum_eq);
                sum_gt = sum_eq = 0;
            }
        }
    }
}

// More than kSummedRows rows: the kept ties of every row and row_ptr.
// Ties at the threshold are kept in flat-index order until `remaining` of them are taken;
// row_ptr is the running count of kept entries.  One block, since every row needs the sum of those before it; a chain of
// two block scans and their barriers per round bounds it, so a round takes many rows (4096: four consecutive rows for each
// of the 1024 threads that a block can have) and the next round's counts are requested before this round's scans.
// 4.0 us at 4096 rows, one round, and 8.2 at 11008 (256 threads, rounds of 2048 rows, no early requests: 8.6 and 22.8).  The
// counts go through LDS: read from memory with consecutive threads on consecutive rows, handed to the thread that owns them.
constexpr int kScanThreads = 1024;
constexpr int kRowsPerThread = 4;
__global__ __launch_bounds__(kScanThreads) void row_scan_kernel(uint32_t *ws, int N, int32_t *row_ptr)
{
    constexpr int kRound = kScanThreads * kRowsPerThread;
    __shared__ uint32_t smem[kScanThreads / 64];
    __shared__ uint32_t s_gt[kRound], s_eq[kRound];
    const uint32_t need = ws[kWsRemaining];
    uint32_t eq_before = 0, kept_before = 0;
    uint32_t next_gt[kRowsPerThread], next_eq[kRowsPerThread];
    auto request = [&](int n0) {
#pragma unroll
        for (int i = 0; i < kRowsPerThread; ++i) {
            const int n = n0 + i * kScanThreads + (int)threadIdx.x;
            next_gt[i] = n < N ? ws[kWsRows + n] : 0u;
            next_eq[i] = n < N ? ws[kWsRows + N + n] : 0u;
        }
    };
    request(0);
    for (int n0 = 0; n0 < N; n0 += kRound) {
        __syncthreads();                                // the round before is done with the LDS arrays
#pragma unroll
        for (int i = 0; i < kRowsPerThread; ++i) {
            const int l = i * kScanThreads + threadIdx.x;
            s_gt[l] = next_gt[i];
            s_eq[l] = next_eq[i];
        }
        request(n0 + kRound);
        __syncthreads();
        const int local = threadIdx.x * kRowsPerThread;
        uint32_t gt[kRowsPerThread], eq[kRowsPerThread], eq_sum = 0;
#pragma unroll
        for (int i = 0; i < kRowsPerThread; ++i) {
            gt[i] = s_gt[local + i];
            eq[i] = s_eq[local + i];
            eq_sum += eq[i];
        }
        uint32_t eq_total, kept_total;
        uint32_t eq_rank = eq_before + block_exclusive_scan<kScanThreads / 64>(eq_sum, smem, eq_total);
        uint32_t take[kRowsPerThread], kept_sum = 0;
#pragma unroll
        for (int i = 0; i < kRowsPerThread; ++i) {
            take[i] = eq_rank >= need ? 0u : (need - eq_rank < eq[i] ? need - eq_rank : eq[i]);
            eq_rank += eq[i];
            kept_sum += gt[i] + take[i];
        }
        uint32_t pos = kept_before + block_exclusive_scan<kScanThreads / 64>(kept_sum, smem, kept_total);
        // results back through LDS, written out with consecutive threads on consecutive rows
#pragma unroll
        for (int i = 0; i < kRowsPerThread; ++i) {
            s_gt[local + i] = take[i];
            s_eq[local + i] = pos;
            pos += gt[i] + take[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kRowsPerThread; ++i) {
            const int l = i * kScanThreads + threadIdx.x, n = n0 + l;
            if (n < N) { ws[kWsRows + 2 * N + n] = s_gt[l]; row_ptr[n] = (int32_t)s_eq[l]; }
        }
        eq_before += eq_total;
        kept_before += kept_total;
    }
    if (threadIdx.x == 0) row_ptr[N] = (int32_t)kept_before;
}

// ---- the encoder ---------------------------------------------------------------------------------
//
// One wave walks a row (or, where there are few rows, one of four consecutive parts of it) in flat-index order, 512
// weights per trip, eight per lane: it marks the kept entries, appends them to the CSR arrays, and quantises and packs the
// rest.  The trips need no barrier and no LDS: positions are a sum over the lanes by DPP (compare masks only rank ties), a
// group's 2 to 16 lanes meet by DPP, the 3-bit words are put together across a quad of lanes.  (The four waves of a shared row exchange
// once, before their trips, what each part keeps.)  Two trips' weights and scores are on their way while one is worked on.
//
// Bound by HBM (6.56 bytes per weight at FP32 scores), which needs the instruction stream short: about 180 vector
// instructions per trip and wave.  A kept weight is replaced by 0: a group's range always contains 0 and 0 gets the code
// z, so masking it once serves the range and the code.  The quotient w / s is one reciprocal per group and three
// instructions per weight (see quotient).
//
// Measured, 11008 x 4096, 4 bits, with the layer's index, medians of a kernel trace (in brackets, on the same machine, with 300
// instructions a trip: ranges as numbers, a branch per kept weight, register sets copied): FP32 scores 48.9 us = 6.0 TB/s
// (52.7), FP16 41.3 (48.0), 3 bits in groups of 16 53.1 (57.1).  (A block of four waves per row with a barrier per 2048
// weights, IEEE divisions and fp64 scales took 88 .. 92 us, and 7 .. 12 us more for a kernel that wrote the index.)

// w / s for an FP16 number w and the FP16 scale s (r: its reciprocal to 1 ulp), by one step of Markstein's correction with
// fused multiply-adds: the product with r is within 2^-22 of the quotient, its residual w - t s has at most 13 significant bits and is exact, and the correction leaves an error below
// 2^-44 before the last rounding.  What follows rounds to an integer, half to even: a quotient that is exactly a
// half-integer is representable and comes out exactly; any other (mw 2^a / ms 2^b with 11-bit mw, ms) is at least
// 1 / (4 ms) >= 2^-13 away from one while below 2^6 in magnitude, and larger ones are clamped to the same end whatever
// their rounding.  So the code is the one that exact arithmetic gives.
__device__ inline float quotient(float w, float s, float r)
{
    const float t = w * r;
    return __builtin_fmaf(__builtin_fmaf(-t, s, w), r, t);
}

__device__ inline float half_bits_to_float(uint32_t h) { return (float)__builtin_bit_cast(_Float16, (uint16_t)h); }

// Eq. 6 / Eq. 7 for one group from its masked min and max (both already widened to contain 0): the smallest FP16 s with
// s * maxq >= mx - mn, and z = clamp(rint(-mn / s), 0, maxq).  The range is held exactly as d + err (Knuth's two-sum), products
// s * maxq are exact in FP32, so comparing them is exact.  The guess RN(d / maxq) is the wanted s or its neighbour.
template <int BITS> __device__ inline void scale_and_zero(float mn, float mx, uint32_t &s_bits, float &s, float &r, float &z)
{
    constexpr float maxq = (float)((1 << BITS) - 1);
    const float d = mx - mn, bb = d - mx, err = (mx - (d - bb)) + (-mn - bb);
    // s * maxq >= d + err: as s * maxq and d are either equal or further apart than |err|, the sign of their difference less
    // err (which a rounding does not change) decides; an infinite d is never covered.
    auto covers = [&](uint32_t sb) { return __builtin_fmaf(half_bits_to_float(sb), maxq, -d) >= err; };
    uint32_t sb = __builtin_bit_cast(uint16_t, (_Float16)(d * (1.f / maxq)));
    sb = sb == 0 ? 1 : sb;
    sb += (uint32_t)(sb < 0x7BFFu) & (uint32_t)!covers(sb);
    sb -= (uint32_t)(sb > 1) & (uint32_t)covers(sb - 1);
    if (d == 0.f) sb = 0x3C00u;                         // an empty range: s = 1 and, as -mn / 1 = 0, z = 0
    s_bits = sb;
    s = half_bits_to_float(sb);
    r = __builtin_amdgcn_rcpf(s);
    z = rintf(__builtin_amdgcn_fmed3f(quotient(-mn, s, r), 0.f, maxq));     // (a NaN gives the lower end)
}

template <int CTRL> __device__ inline uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
// DPP controls: lanes exchange within pairs, within quads, halves of eight and of sixteen are mirrored, a row rotates.
constexpr int kDppPair = 0xB1, kDppQuad = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140, kDppRor4 = 0x124, kDppRor8 = 0x128;

// Range of the 2^STEPS lanes that share a group, from each lane's own.  Both bounds contain 0, so as bit patterns the upper one
// orders like a signed integer and the lower one, downwards, like an unsigned one: one instruction a step, where the
// floating-point minimum also quiets its operand first.
template <int STEPS> __device__ inline void group_range(float &mn, float &mx)
{
    uint32_t lo = __builtin_bit_cast(uint32_t, mn);
    int32_t hi = __builtin_bit_cast(int32_t, mx);
    auto meet = [&](auto ctrl) {
        const uint32_t l = dpp_u32<decltype(ctrl)::value>(lo);
        const int32_t h = (int32_t)dpp_u32<decltype(ctrl)::value>((uint32_t)hi);
        lo = l > lo ? l : lo;
        hi = h > hi ? h : hi;
    };
    meet(std::integral_constant<int, kDppPair>{});
    if constexpr (STEPS > 1) meet(std::integral_constant<int, kDppQuad>{});
    if constexpr (STEPS > 2) meet(std::integral_constant<int, kDppHalfMirror>{});
    if constexpr (STEPS > 3) meet(std::integral_constant<int, kDppMirror>{});
    mn = __builtin_bit_cast(float, lo);
    mx = __builtin_bit_cast(float, hi);
}

// Sum over the lanes up to and including this one.
__device__ inline uint32_t wave_sum_to_here(uint32_t v)
{
    auto add = [&](auto ctrl, auto rows) { v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xF, false); };
    add(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});       // row_shr 1, 2, 4, 8: within rows of 16
    add(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});
    add(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});
    add(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});
    add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});       // row_bcast 15: to rows 1 and 3
    add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});       // row_bcast 31: to rows 2 and 3
    return v;
}

// Lanes below this one whose bit is set, added to `base`.
__device__ inline uint32_t count_below(uint64_t mask, uint32_t base)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, base));
}

// What a lane holds of one trip: eight weights and their scores as they lie in memory.
template <bool F16> struct EncodeRegs {
    uint4 w, s[F16 ? 1 : 2];
    __device__ inline void load(const uint16_t *W, const char *score, uint32_t k)    // of a row, from column k
    {
        w = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(W) + 2 * k);
        if (F16) {
            s[0] = *reinterpret_cast<const uint4 *>(score + 2 * k);
        } else {
            const uint4 *p = reinterpret_cast<const uint4 *>(score + 4 * k);
            s[0] = p[0];
            s[F16 ? 0 : 1] = p[1];
        }
    }
    __device__ inline void keys(uint32_t key[8]) const
    {
        if (F16) {
            const uint32_t v[4] = {s[0].x, s[0].y, s[0].z, s[0].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                key[2 * i] = key_from_f16((uint16_t)(v[i] & 0xFFFF));
                key[2 * i + 1] = key_from_f16((uint16_t)(v[i] >> 16));
            }
        } else {
            const uint4 &b = s[F16 ? 0 : 1];
            key[0] = key_from_f32(s[0].x); key[1] = key_from_f32(s[0].y); key[2] = key_from_f32(s[0].z); key[3] = key_from_f32(s[0].w);
            key[4] = key_from_f32(b.x); key[5] = key_from_f32(b.y); key[6] = key_from_f32(b.z); key[7] = key_from_f32(b.w);
        }
    }
};

constexpr int kTrip = 512;                              // weights per wave and trip

// What the rows before row n keep, by a wave: `start`; of row n's keys equal to the threshold the first `take` are kept;
// `end`: start and what row n keeps.  Of the ties in the rows before, in flat-index order, the first `need` are kept.
struct RowRange { uint32_t start, take, end; };
__device__ inline RowRange rows_before(const uint32_t *ws, int N, int n)
{
    const int lane = threadIdx.x & 63, log2 = block_rows_log2(N), block = n >> log2;
    const uint32_t *gt_of = ws + kWsRows, *eq_of = gt_of + N, *sums = eq_of + N;
    uint32_t gt = 0, eq = 0;
    // The block's rows, four to a lane.  (What lies behind the counts of equal keys is the block sums, at 4 bytes' alignment.)
    for (int r0 = block << log2; r0 < n; r0 += 256) {
        const int r = r0 + 4 * lane;
        if (r < n) {
            const Keys4 g = *reinterpret_cast<const Keys4 *>(gt_of + r), e = *reinterpret_cast<const Keys4 *>(eq_of + r);
#pragma unroll
            for (int i = 0; i < 4; ++i) { gt += r + i < n ? g.k[i] : 0u; eq += r + i < n ? e.k[i] : 0u; }
        }
    }
    for (int b = lane; b < block; b += 64) { gt += sums[b * kSumStride]; eq += sums[b * kSumStride + 1]; }
    const uint32_t need = ws[kWsRemaining], mine = gt_of[n], ties = eq_of[n];
    gt = (uint32_t)__builtin_amdgcn_readlane((int)wave_sum_to_here(gt), 63);
    eq = (uint32_t)__builtin_amdgcn_readlane((int)wave_sum_to_here(eq), 63);
    const uint32_t taken = eq < need ? eq : need, left = need - taken, take = ties < left ? ties : left;
    return {gt + taken, take, gt + taken + mine + take};
}

// STEPS: log2 of the lanes that share a group (group = 16, 32, 64, 128: 1 to 4).  parts: waves per row, 1 or 4.
// rec, fine: the layer's index (gwq_internal.h), or NULL.
template <int BITS, bool F16, int STEPS>
__global__ __launch_bounds__(kThreads) void encode_kernel(const uint16_t *__restrict__ W, const void *__restrict__ score, int N, int K,
                                                          int parts, const uint32_t *__restrict__ ws,
                                                          int32_t *__restrict__ row_ptr, uint32_t *__restrict__ qweight,
                                                          uint16_t *__restrict__ scales, uint8_t *__restrict__ zeros,
                                                          uint16_t *__restrict__ col_idx, uint16_t *__restrict__ out_val,
                                                          GroupRecord *__restrict__ rec, uint32_t *__restrict__ fine)
{
    constexpr int group = 8 << STEPS;
    constexpr int wpg = words_per_group(BITS);
    constexpr float maxq = (float)((1 << BITS) - 1);
    constexpr uint32_t cap = index_scale_cap(BITS);
    __shared__ uint32_t part_gt[kWaves], part_eq[kWaves];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = parts == 1 ? (int)blockIdx.x * kWaves + wave : (int)blockIdx.x;
    if (n >= N) return;                                 // whole waves, and only where nobody waits for them (parts = 1)
    const int trips = (K + kTrip - 1) / kTrip, per_part = (trips + parts - 1) / parts;
    const int t_begin = parts == 1 ? 0 : wave * per_part;
    const int t_end = t_begin + per_part < trips ? t_begin + per_part : trips;
    const uint32_t thr = ws[kWsPrefix];
    const int gpr = K / kGroup, spr = K / group;
    RowRange row;
    if (N <= kSummedRows) {
        row = rows_before(ws, N, n);
        if (lane == 0 && t_begin == 0) {
            row_ptr[n] = (int32_t)row.start;
            if (n == N - 1) row_ptr[N] = (int32_t)row.end;
        }
    } else {
        row = {(uint32_t)row_ptr[n], ws[kWsRows + 2 * N + n], (uint32_t)row_ptr[n + 1]};
    }
    const uint32_t take = row.take;                     // of the row's keys equal to the threshold the first `take` are kept
    const uint32_t row_start = row.start;
    // The row's part of each array: uniform, so that a lane's place is a 32-bit offset.
    W += (size_t)n * K;
    const char *const row_score = static_cast<const char *>(score) + (size_t)n * K * (F16 ? 2 : 4);
    qweight += (size_t)n * gpr * wpg;
    scales += (size_t)n * spr;
    zeros += (size_t)n * spr;
    col_idx += row_start;
    out_val += row_start;
    uint32_t pos = 0, ties_seen = 0;                    // kept and equal to the threshold in the row so far
    if (rec) {
        rec += (size_t)n * (gpr + 1);
        fine += (size_t)n * (K / 16);
        if (lane == 0 && t_begin == 0) rec[gpr] = GroupRecord{(int32_t)row.end, 0u};
    }

    // Lanes beyond the end of the row (whole groups of lanes) repeat its last weights and keep nothing.
    auto column = [&](int t) { return (uint32_t)(t * kTrip + lane * 8); };
    auto request = [&](int t, EncodeRegs<F16> &R) {
        const uint32_t k = column(t < t_end ? t : t_end - 1);
        R.load(W, row_score, k < (uint32_t)K ? k : (uint32_t)K - 8);
    };
    EncodeRegs<F16> even, odd;
    if (t_begin < t_end) {
        request(t_begin, even);
        request(t_begin + 1, odd);
    }

    if (parts > 1) {                                    // what the parts before this one keep
        uint32_t gt = 0, eq = 0;
        for (int t = t_begin; t < t_end; ++t) {
            EncodeRegs<F16> R;
            request(t, R);
            uint32_t key[8];
            R.keys(key);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                gt += column(t) < (uint32_t)K && key[i] > thr;
                eq += column(t) < (uint32_t)K && key[i] == thr;
            }
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) { gt += __shfl_xor(gt, d); eq += __shfl_xor(eq, d); }
        if (lane == 0) { part_gt[wave] = gt; part_eq[wave] = eq; }
        __syncthreads();
        for (int w = 0; w < wave; ++w) { pos += part_gt[w]; ties_seen += part_eq[w]; }
        pos += ties_seen < take ? ties_seen : take;
    }

    // One trip; TIES: the row keeps some of its keys that equal the threshold.
    auto trip = [&](int t, const EncodeRegs<F16> &R, auto TIES) {
        const uint32_t k = column(t);
        const bool active = k < (uint32_t)K;
        const uint32_t vw[4] = {R.w.x, R.w.y, R.w.z, R.w.w};
        float w[8];
        uint32_t kept = 0;                              // bit i: weight i is an outlier
        {
            uint32_t key[8];
            R.keys(key);
            const uint32_t above = active ? thr : ~0u;  // no key is larger than that, or equal to it
            bool keep[8];
            if constexpr (!decltype(TIES)::value) {
#pragma unroll
                for (int i = 0; i < 8; ++i) keep[i] = key[i] > above;
            } else {
                uint32_t rank = ties_seen;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint64_t m = __ballot(key[i] == above);
                    rank = count_below(m, rank);
                    ties_seen += (uint32_t)__builtin_popcountll(m);
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const bool tie = key[i] == above;
                    keep[i] = key[i] > above || (tie && rank < take);
                    rank += tie;
                }
            }
#pragma unroll
            for (int i = 7; i >= 0; --i) {
                kept = 2 * kept + keep[i];
                w[i] = keep[i] ? 0.f : half_bits_to_float(i & 1 ? vw[i >> 1] >> 16 : vw[i >> 1] & 0xFFFFu);
            }
        }
        const uint32_t count = (uint32_t)__builtin_popcount(kept), to_here = wave_sum_to_here(count);
        const uint32_t first = pos + to_here - count;   // of the row's outliers, this lane's first
        pos += (uint32_t)__builtin_amdgcn_readlane((int)to_here, 63);
        // A lane has more than one of its eight to store once in a few hundred lanes, so the wave goes round once, or twice.
        for (uint32_t at = first; kept; ++at) {
            const uint32_t i = (uint32_t)__builtin_ctz(kept);
            kept &= kept - 1;
            const uint32_t pair = i & 4 ? (i & 2 ? vw[3] : vw[2]) : (i & 2 ? vw[1] : vw[0]);
            col_idx[at] = (uint16_t)(k + i);
            out_val[at] = (uint16_t)(pair >> (16 * (i & 1)));
        }

        float mn = 0.f, mx = 0.f;
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            mn = __builtin_fminf(__builtin_fminf(w[i], w[i + 1]), mn);      // a NaN loses against a number
            mx = __builtin_fmaxf(__builtin_fmaxf(w[i], w[i + 1]), mx);
        }
        group_range<STEPS>(mn, mx);
        uint32_t s_bits;
        float s, r, zf;
        scale_and_zero<BITS>(mn, mx, s_bits, s, r, zf);
        const uint32_t z = (uint32_t)(int)zf;

        // Eq. 9: rint(w / s) by adding 1.5 * 2^23 (an even number: halves go to even); its low bits, shifted to their
        // places and summed, carry a known multiple of that number's pattern, taken off with z added for all eight at once.
        // Even positions in the low half-word, odd ones in the high half-word, `BITS` bits apiece.
        constexpr uint32_t ones = BITS == 4 ? 0x11111111u : 0x02490249u;
        const float lo = -zf, hi = maxq - zf;
        uint32_t codes = 0u - (0x4B400000u - z) * ones;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float q = __builtin_amdgcn_fmed3f(quotient(w[i], s, r), lo, hi) + 12582912.f;
            codes += __builtin_bit_cast(uint32_t, q) << (16 * (i & 1) + BITS * (i >> 1));
        }

        if (BITS == 4) {
            if (active) qweight[k >> 3] = codes;
        } else {
            // A quad of lanes holds a slot: 16 codes of the even and 16 of the odd positions, 48 bits each.  Lane q < 3 of the
            // quad makes word q of the slot (15 bits of each), lane 3 the slot's two codes of the tail word.
            const uint32_t p0 = dpp_u32<0x00>(codes), p1 = dpp_u32<0x55>(codes), p2 = dpp_u32<0xAA>(codes), p3 = dpp_u32<0xFF>(codes);
            auto stream = [&](int sh) {
                return (uint64_t)((p0 >> sh & 0xFFFu) | (p1 >> sh & 0xFFFu) << 12) | (uint64_t)((p2 >> sh & 0xFFFu) | (p3 >> sh & 0xFFFu) << 12) << 24;
            };
            const int q = lane & 3, b = (lane >> 2) & 3;
            const uint32_t even_codes = (uint32_t)(stream(0) >> (15 * q)) & 0x7FFFu, odd_codes = (uint32_t)(stream(16) >> (15 * q)) & 0x7FFFu;
            uint32_t tail = q == 3 ? (even_codes & 7u) << (3 * b) | (odd_codes & 7u) << (16 + 3 * b) : 0u;
            tail |= dpp_u32<kDppRor4>(tail);
            tail |= dpp_u32<kDppRor8>(tail);
            if (active && (q < 3 || b == 3)) qweight[(k >> 7) * wpg + 3 * b + q] = q < 3 ? even_codes | odd_codes << 16 : tail;
        }
        if (active && (lane & ((1 << STEPS) - 1)) == 0) {
            scales[k / group] = (uint16_t)s_bits;
            zeros[k / group] = (uint8_t)z;
        }
        if (rec && active) {
            const uint32_t pair = (s_bits < cap ? s_bits : cap) | z << 16;
            if ((lane & 15) == 0) rec[k >> 7] = GroupRecord{(int32_t)(row_start + first), STEPS == 4 ? pair : 0u};
            if (STEPS < 4 && (lane & 1) == 0) fine[k >> 4] = pair;
        }
    };
    // Two trips' weights and scores are on their way.
    auto walk = [&](auto TIES) {
        int t = t_begin;
        for (; t + 2 <= t_end; t += 2) {
            trip(t, even, TIES);
            request(t + 2, even);
            trip(t + 1, odd, TIES);
            request(t + 3, odd);
        }
        if (t < t_end) trip(t, even, TIES);
    };
    if (take == 0) walk(std::false_type{});             // uniform over the wave; nearly every row
    else walk(std::true_type{});
}

template <bool F16>
hipError_t run_select(const void *score, int N, int K, uint32_t *ws, int32_t *row_ptr, uint32_t k_out, PackWay way, hipStream_t st)
{
    const size_t total = (size_t)N * K;
    const int per_row = pack_candidates_per_row(K);
    if (k_out) {
        const int blocks = (int)std::min<size_t>((total / 8 + kDigitThreads - 1) / kDigitThreads, kScoreBlocks);
        const uint32_t sampled = way == PackWay::list || (way == PackWay::by_size && total > kScoresUpTo) ? sample_keys(total) : 0;
        sample_kernel<F16><<<32, kThreads, 0, st>>>(score, total, ws, N, sampled / (F16 ? 8 : 4), k_out);
        if (sampled) {
            band_kernel<<<1, kBandThreads, 0, st>>>(ws, N, sampled, (float)k_out / (float)total);
            candidates_kernel<F16><<<N, kThreads, 0, st>>>(score, K, ws, N, per_row);
        }
        digit_kernel<0, F16><<<blocks, kDigitThreads, 0, st>>>(score, total, ws, N, per_row);
        digit_kernel<1, F16><<<blocks, kDigitThreads, 0, st>>>(score, total, ws, N, per_row);
        if (!F16) digit_kernel<2, F16><<<blocks, kDigitThreads, 0, st>>>(score, total, ws, N, per_row);
        rows_kernel<F16><<<std::min(N, 1024), kThreads, 0, st>>>(score, K, ws, N, per_row);
    } else {
        nothing_kernel<<<8, kThreads, 0, st>>>(ws, N);
    }
    if (N > kSummedRows) row_scan_kernel<<<1, kScanThreads, 0, st>>>(ws, N, row_ptr);
    return hipGetLastError();
}

template <int BITS, bool F16, int STEPS>
hipError_t run_encode(const void *W, const void *score, const gwq_packed &P, const uint32_t *ws, hipStream_t st)
{
    // Few rows: one wave for each leaves the chip waiting for its trips, so four share a row, at the price of reading the
    // scores once more to count what the parts before keep.  Where that stops to pay (us that
    // four waves save over one; FP32 scores 1024 x 8192 10, 1300 x 65536 3, 1500 x 65536 -16, 1900 x 8192 -3; FP16 scores, half
    // the bytes, 1500 x 28672 37, 2047 x 8192 4, 2047 x 2048 -0.2).
    const int parts = P.N < (F16 ? 2048 : 1300) ? kWaves : 1;
    const int blocks = parts == 1 ? (P.N + kWaves - 1) / kWaves : P.N;
    GroupRecord *rec = static_cast<GroupRecord *>(P.index);
    uint32_t *fine = rec ? reinterpret_cast<uint32_t *>(static_cast<char *>(P.index) + index_record_bytes(P.N, P.K)) : nullptr;
    encode_kernel<BITS, F16, STEPS><<<blocks, kThreads, 0, st>>>(static_cast<const uint16_t *>(W), score, P.N, P.K, parts, ws, P.row_ptr,
                                                                P.qweight, P.scales, P.zeros, P.col_idx, P.out_val, rec, fine);
    return hipGetLastError();
}
template <int BITS, bool F16>
hipError_t run_encode(const void *W, const void *score, const gwq_packed &P, const uint32_t *ws, hipStream_t st)
{
    switch (P.group) {
    case 16: return run_encode<BITS, F16, 1>(W, score, P, ws, st);
    case 32: return run_encode<BITS, F16, 2>(W, score, P, ws, st);
    case 64: return run_encode<BITS, F16, 3>(W, score, P, ws, st);
    default: return run_encode<BITS, F16, 4>(W, score, P, ws, st);
    }
}

}  // namespace

hipError_t launch_pack(const void *W, const void *score, int score_is_f16, const gwq_packed &P,
                       uint32_t *ws, PackWay way, hipStream_t st)
{
    const hipError_t e = score_is_f16 ? run_select<true>(score, P.N, P.K, ws, P.row_ptr, (uint32_t)P.n_outliers, way, st)
                                      : run_select<false>(score, P.N, P.K, ws, P.row_ptr, (uint32_t)P.n_outliers, way, st);
    if (e != hipSuccess) return e;
    if (P.bits == 4)
        return score_is_f16 ? run_encode<4, true>(W, score, P, ws, st) : run_encode<4, false>(W, score, P, ws, st);
    return score_is_f16 ? run_encode<3, true>(W, score, P, ws, st) : run_encode<3, false>(W, score, P, ws, st);
}

}  // namespace gwq
