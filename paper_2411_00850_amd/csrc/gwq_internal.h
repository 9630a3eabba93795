// Internal declarations shared by the HIP translation units of libgwq (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "gwq.h"

namespace gwq {

constexpr int kGroup = 128;        // codes per quantisation group along K
constexpr int kSelBins = 2048;     // bins of one radix-select pass
constexpr int kMaxBatch = GWQ_MAX_BATCH;   // layers per grouped decode launch

__host__ __device__ constexpr int words_per_group(int bits) { return bits == 4 ? 16 : 13; }

// What lanes of a wave wrote to the LDS before this, its other lanes read after it.  A wave's LDS accesses are carried out in
// order, so nothing is waited for; the fences hold the compiler to the order of the source, which the barrier alone does not.
__device__ inline void wave_meet()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Compute units of the current device, asked once per device (256 on MI355X; 256 if the query fails).
int device_cus();

// Lets `kernel` use up to `bytes` of dynamic LDS on the current device.  `done` is the caller's per-kernel
// record (bit d: done on device d); the HIP call is idempotent, so a race between threads is harmless.
hipError_t allow_dynamic_lds(const void *kernel, int bytes, std::atomic<uint32_t> &done);

// ---- The layer's index (gwq_packed.index) -----------------------------------------------------
// One record per (channel, block of 128 codes) for the GEMM's producers - the CSR index of the block's first outlier, and
// the block's scale and zero point, so that one 8-byte load fetches everything a block needs besides its codes - and one
// more per channel that holds the channel's end.  For groups below 128 the records carry no scale, and behind them (at
// index_record_bytes) lie eight words scale bits | zero point << 16 per channel and block, one per 16 columns.
struct GroupRecord {
    int32_t first;
    uint32_t scale_zero;                                // scale bits | zero point << 16
};
inline size_t index_record_bytes(int64_t N, int64_t K) { return ((size_t)(N * (K / kGroup + 1)) * sizeof(GroupRecord) + 255) / 256 * 256; }
// The GEMM multiplies FP16 operands s * (q - z): in the index a scale is capped at the largest FP16 value whose product
// with 2^bits - 1 is still finite (4364 * 15 = 65460, 9352 * 7 = 65464; only ranges beyond 65460 reach it; positive FP16
// patterns order like integers).
__host__ __device__ constexpr uint32_t index_scale_cap(int bits) { return bits == 4 ? 0x6C43u : 0x7091u; }

// ---- gwq_pack workspace: uint32 words -------------------------------------------------------
// [0, 3*kSelBins)        histograms of the selection's later digits (gwq_pack.hip)
// kWsPrefix              the threshold: key of the smallest kept entry
// kWsRemaining           how many of the keys equal to it are kept
// kWsCandOverflow        nonzero when there is no list, or some row had more candidates than its share of it holds
// kWsBandLo, kWsBandHi   the band of keys that the sample puts the threshold in, both ends included
// kWsWanted, kWsWay      entries to select; by list, by scores or a single key
// kWsStep + 2 i, + 1     after digit i: what is known of the threshold, and how many entries are still wanted from there
// kWsRows + 0*N ..       per row: count of keys above the threshold
// kWsRows + 1*N ..       per row: count of keys equal to the threshold
// kWsRows + 2*N ..       per row: how many of its threshold ties are kept; up to kSummedRows rows: the first two of the counts
//                        above, summed over blocks of rows, each in a line of its own
// kWsRows + 3*N ..       kSelBins words: three times kSpread whose sums are the keys above the band, where it is a single key
//                        the keys equal to it, and the candidates
// then                   per row: number of candidates; then the candidates' keys, [N][pack_candidates_per_row(K)]
// Every row has its own part of the list (no counter shared between blocks).
constexpr int kWsPrefix = 3 * kSelBins;
constexpr int kWsRemaining = kWsPrefix + 1;
constexpr int kWsCandOverflow = kWsPrefix + 3;
constexpr int kWsBandLo = kWsPrefix + 4, kWsBandHi = kWsPrefix + 5, kWsWanted = kWsPrefix + 6, kWsWay = kWsPrefix + 7;
constexpr int kWsStep = kWsPrefix + 8;                 // three pairs
constexpr int kWsRows = kWsPrefix + 16;
constexpr int kSpread = 512;
static_assert(3 * kSpread <= kSelBins, "the place of one histogram");

inline int pack_candidates_per_row(int64_t K) { return K / 32 < 32 ? 32 : (int)(K / 32); }
__host__ __device__ constexpr int64_t pack_keys_at(int64_t N) { return kWsRows + 3 * N + kSelBins + N; }   // a multiple of four
inline size_t pack_workspace_bytes(int64_t N, int64_t K)
{
    return (size_t)(pack_keys_at(N) + N * pack_candidates_per_row(K)) * 4 + 256;
}

// Launchers (defined in the .hip files).  Each enqueues on `stream` and returns the last HIP error.
// way: how gwq_pack finds the threshold - by the number of scores, or (measurement and test hook) always by passes over all
// of them, or always by the list of candidates, where it fits.
enum class PackWay { by_size = 0, scores = 1, list = 2 };
hipError_t launch_pack(const void *W, const void *score, int score_is_f16, const gwq_packed &P,
                       uint32_t *ws, PackWay way, hipStream_t stream);
// Measurement overrides of the decode launch (0 = built-in choice): waves per block of the lean kernel;
// streaming kernel 1 = never, 2 = for every M <= 16 it can take; its tiles per block.
struct DecodeTuning {
    int waves, stream, tiles;
    int lean_rows = 0;          // largest M the kernel with X[M][K] in LDS takes (0 = built-in choice, at most 8)
    int pairs = 0;              // that kernel with two tiles per block for 5 <= M <= 8: 0 = built-in choice, 1 = never, 2 = wherever it fits
    bool gated_pairs = false;   // layers (2i, 2i+1) are gate and up of a gated pair: one launch writes silu(gate) * up into Y[2i+1]
    bool bf16 = false;          // X and Y are bfloat16 (groups of 128 only; the kernel for any M <= 16 takes these)
};
// With `describe` set a launcher only writes there which kernel, template arguments and launch shape it
// would use for these arguments, and launches nothing.
struct PlanText {
    char text[192];
};
hipError_t launch_decode(int count, const gwq_packed *const *P, const void *const *X, int M, void *const *Y,
                         const DecodeTuning &tune, hipStream_t stream, PlanText *describe = nullptr);
// Measurement overrides of the GEMM launch (0 = built-in choice): rows of Y per block; X through the LDS (1: always, 2: never
// where the scratch allows it).
struct GemmTuning {
    int rows, staged;
};
// index: gemm_index_bytes(N, K, group) bytes, 16-byte aligned (one record per channel and block of 128 codes:
// index of the block's first outlier, scale, zero point; for groups below 128 also a scale / zero-point pair
// per 16 columns; a multiple of 256 bytes).  scratch: gemm_scratch_bytes(N, M_max)
// bytes for the partial sums of launches that also split K and, where it fits, a copy of X (may be NULL: then neither).
size_t gemm_index_bytes(int64_t N, int64_t K, int group);
size_t gemm_scratch_bytes(int64_t N, int64_t M_max);
hipError_t launch_gemm_index(const gwq_packed &P, void *index, hipStream_t stream);        // fills the records
// The GEMM whose X operands come from memory in fragment order (gwq_gemm_frag.hip): frag = frag_bytes(M, K) bytes for that
// copy of X, 16-byte aligned; rows = 32, 64, 96, 128, 160, 192 or 256 rows of Y per block; partial for splits > 1.
size_t frag_bytes(int64_t M, int64_t K);
hipError_t launch_gemm_frag(const gwq_packed &P, const void *X, int M, void *Y, const void *index, void *frag, float *partial,
                            int rows, int splits, int split_groups, hipStream_t stream, PlanText *describe, bool bf16);
hipError_t launch_gemm(const gwq_packed &P, const void *X, int M, void *Y, const void *index, void *scratch,
                       size_t scratch_bytes, const GemmTuning &tune, hipStream_t stream,
                       PlanText *describe = nullptr, bool bf16 = false);                   // reads them; bf16: X, Y bfloat16

// workspace: quality_workspace_bytes(N) bytes, 8-byte aligned (one partial result per channel); out: 3 doubles.
size_t quality_workspace_bytes(int64_t N);
hipError_t launch_quality(const gwq_packed &P, const void *W, const void *score, int score_is_f16, void *workspace,
                          double *out, hipStream_t stream);

// Measurement probes (gwq_probe.hip): one plain streaming read of `bytes` (a multiple of 16); `blocks` blocks of
// four waves that issue 8 * iters 32x32x16 FP16 MFMAs each out of registers.  sink: 4 bytes, practically never written.
hipError_t launch_probe_stream(const void *src, size_t bytes, void *sink, hipStream_t stream);
hipError_t launch_probe_mfma(int blocks, int iters, void *sink, hipStream_t stream);

// H = silu(G) * U elementwise over `count` FP16 values (the unfused form of the gated pair).
hipError_t launch_silu_mul(const void *G, const void *U, void *H, size_t count, hipStream_t stream);

// score = beta * score + alpha * dY^T X (dY [M][N], X [M][K] FP16; score [N][K] FP32); K a multiple of 128.
hipError_t launch_score(const void *dY, const void *X, int M, int N, int K, float alpha, float beta, float *score,
                        hipStream_t stream);

}  // namespace gwq
