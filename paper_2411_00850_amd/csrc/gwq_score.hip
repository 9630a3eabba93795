// gwq_score on gfx950: the score that gwq_pack ranks, produced on the device for one linear layer.
// The score is the gradient of the loss with respect to the weights (Sec. 3.1, Eq. 2); for Y = X W^T
// without bias the chain rule gives, from the gradient dY of the loss with respect to Y,
//   g[n][k] = sum_m dY[m][n] * X[m][k]
// and the entry point writes score = beta * score + alpha * g, so that the mean over calibration
// samples (Sec. 4.3, ablation on the number of calibration samples) is a sequence of calls with alpha = 1 / samples.
//
// A dense contraction over the samples m with both operands stored m-major, bound by MFMA.  Two kernels: this one for
// outputs too small to fill the chip with larger tiles, and score_big_kernel below.  A block of
// four waves owns a 128 (n) x 128 (k) tile of the score and walks m in steps of 64; a wave owns 64 x 64
// of it as 2 x 2 tiles of v_mfma_f32_32x32x16_f16 (FP32 accumulators, exact FP16 products).  The MFMA
// wants, per lane, eight consecutive m of one n (or k), while memory has eight consecutive n of one m:
// a thread loads 16 bytes of four consecutive rows m, regroups them in registers into eight 8-byte
// pieces "four m of one n" and stores those, so the LDS copy is transposed, [n][m] and [k][m], 128
// bytes per row, and fragment reads are plain 16-byte reads.  The eight 16-byte units of a row are
// XOR-permuted by row so that both the fragment reads (16 consecutive rows x one unit) and the
// transposing stores (rows 8 apart) are free of bank conflicts.  Two LDS buffers, one block barrier
// per step; global loads run a step ahead in two register sets; the stores of the next step are
// spread behind the MFMA batches of the current one.
#include <type_traits>

#include "gwq_internal.h"

namespace gwq {
namespace {

typedef _Float16 half8s __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int kTile = 128;         // tile edge along n and along k
constexpr int kStepM = 64;         // samples per step
constexpr int kScoreThreads = 256;
constexpr int kUnitsPerBuf = kTile * 8;                 // 16-byte units of one operand's tile (128 rows x 64 halves)
constexpr size_t kScoreLds = (size_t)2 * 2 * kUnitsPerBuf * 16;   // two buffers x two operands = 64 KB

// 16-byte unit c of row `row` of a tile in LDS (rows of 128 bytes: two rows span the 64 banks).  The XOR
// term has bit 0 = row bit 3 and bits 2..1 = row bits 2..1 ^ row bits 5..4: the 16 consecutive rows of a
// fragment read meet 16 different (row parity, unit) pairs, and so do the 16 rows, 8 apart and of both
// parities, that the lanes of a transposing store write.
__device__ inline int unit_of(int row, int c)
{
    return row * 8 + (c ^ (((((row >> 1) ^ (row >> 4)) & 3) << 1) | ((row >> 3) & 1)));
}

struct RowSet {
    uint4 a[4], b[4];             // 8 halves of dY and of X from four consecutive rows m
};

template <bool N8>
__global__ __launch_bounds__(kScoreThreads, N8 ? 2 : 1) void score_kernel(const _Float16 *__restrict__ dY,
                                                              const _Float16 *__restrict__ X, int M, int N, int K,
                                                              int tiles_n, int tiles_k, float alpha, float beta,
                                                              float *__restrict__ score)
{
    extern __shared__ uint4 lds[];                      // [buffer][operand][unit]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Workgroups go round-robin to the 8 XCDs, each with an L2 of its own: XCD x takes the x-th eighth of
    // the tiles, in an order that walks k inside bands of 8 tile rows, so that the blocks an XCD runs at
    // one time form a patch of about 8 x 8 tiles and share their operands' tiles in its L2.
    const int per_xcd = (tiles_n * tiles_k + 7) >> 3;
    const int lin = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (lin >= tiles_n * tiles_k) return;               // whole block, before any barrier
    const int band = lin / (8 * tiles_k), in_band = lin - band * 8 * tiles_k;
    const int band_rows = tiles_n - 8 * band < 8 ? tiles_n - 8 * band : 8;
    const int n0 = (8 * band + in_band % band_rows) * kTile, k0 = (in_band / band_rows) * kTile;
    // Staging: a thread takes columns 8 * chunk .. + 7 of rows 4 * quad .. + 3.  Lanes 16 apart and lanes 32
    // apart both differ in the 8-byte half of a unit they store to, and a lane with chunk >= 8 stores the
    // odd column while the others store the even one: whichever lanes the LDS serves together, their
    // stores fall into different banks.
    const int chunk = lane & 15, quad = 4 * wave + 2 * (lane >> 5) + (((lane >> 4) ^ (lane >> 5)) & 1);
    const int flip = chunk >> 3;
    const int wn = wave >> 1, wk = wave & 1;
    const int steps = (M + kStepM - 1) / kStepM;

    // Requests for step t.  Rows beyond M and columns beyond N read a valid address.  Columns beyond N
    // only reach rows of the tile that are never stored; rows beyond M are zeroed in both operands when the
    // set is staged (touching a loaded value here would wait for it here): next to a zero in one of them
    // alone, an infinity in the row that was read in their place would make a NaN.
    auto fetch = [&](int t, RowSet &r) {
        const int nn = n0 + 8 * chunk, kk = k0 + 8 * chunk;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = t * kStepM + 4 * quad + i;
            const size_t mrow = m < M ? m : 0;
            r.b[i] = *reinterpret_cast<const uint4 *>(X + mrow * K + kk);
            if (N8) {                                   // N is a multiple of 8: a chunk is inside or outside
                r.a[i] = *reinterpret_cast<const uint4 *>(dY + mrow * N + (nn < N ? nn : 0));
            } else {                                    // rows of dY are not 16-byte aligned: element by element
                uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    w[j >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, dY[mrow * N + (nn + j < N ? nn + j : 0)]) << (16 * (j & 1));
                r.a[i] = uint4{w[0], w[1], w[2], w[3]};
            }
        }
    };
    // Transposing store of the register set of step t into buffer `buf`: for each of the thread's eight
    // columns the four rows' halves as one 8-byte piece at [column][4 * quad .. + 3].  Done in four parts
    // (columns 2 * part and 2 * part + 1 of both operands), one behind each batch of MFMAs, whose shadow
    // hides them.
    auto stage_part = [&](int buf, int t, const RowSet &r, int part) {
        char *a_base = reinterpret_cast<char *>(lds + (size_t)(2 * buf) * kUnitsPerBuf);
        char *b_base = reinterpret_cast<char *>(lds + (size_t)(2 * buf + 1) * kUnitsPerBuf);
        const int m = t * kStepM + 4 * quad;
        const uint32_t rows01 = (m < M ? 0xFFFFu : 0u) | (m + 1 < M ? 0xFFFF0000u : 0u);
        const uint32_t rows23 = (m + 2 < M ? 0xFFFFu : 0u) | (m + 3 < M ? 0xFFFF0000u : 0u);
        auto put = [&](char *base, const uint4 *v) {
            const uint32_t w[4][4] = {{v[0].x, v[0].y, v[0].z, v[0].w}, {v[1].x, v[1].y, v[1].z, v[1].w},
                                      {v[2].x, v[2].y, v[2].z, v[2].w}, {v[3].x, v[3].y, v[3].z, v[3].w}};
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int j = 2 * part + jj;            // column j ^ flip: the same word of the loaded 16 bytes
                // the same half of two words; a selector byte of 0x0C gives zero
                const uint32_t sel = ((j & 1) ^ flip) ? 0x07060302u : 0x05040100u;
                uint2 piece;
                piece.x = __builtin_amdgcn_perm(w[1][j >> 1], w[0][j >> 1], (sel & rows01) | (0x0C0C0C0Cu & ~rows01));
                piece.y = __builtin_amdgcn_perm(w[3][j >> 1], w[2][j >> 1], (sel & rows23) | (0x0C0C0C0Cu & ~rows23));
                const int row = 8 * chunk + (j ^ flip);
                *reinterpret_cast<uint2 *>(base + (size_t)unit_of(row, quad >> 1) * 16 + 8 * (quad & 1)) = piece;
            }
        };
        put(a_base, r.a);
        put(b_base, r.b);
    };

    float16v acc[2][2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[s][t][v] = 0.f;

    // One step: the MFMAs of buffer `buf` and the staging of step `next`, held in `r`, into the other
    // buffer.  Behind the last step this stages a repeat of it that nobody reads: no branch.
    auto step = [&](int buf, int next, const RowSet &r) {
        const uint4 *a_base = lds + (size_t)(2 * buf) * kUnitsPerBuf;
        const uint4 *b_base = lds + (size_t)(2 * buf + 1) * kUnitsPerBuf;
#pragma unroll
        for (int kb = 0; kb < kStepM / 16; ++kb) {
            const int c = 2 * kb + (lane >> 5);         // the lane's eight samples: 16 * kb + 8 * (lane / 32) ..
            uint4 fa[2], fb[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                fa[s] = a_base[unit_of(wn * 64 + s * 32 + (lane & 31), c)];
                fb[s] = b_base[unit_of(wk * 64 + s * 32 + (lane & 31), c)];
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[s][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8s, fa[s]),
                                                                       __builtin_bit_cast(half8s, fb[t]), acc[s][t], 0, 0, 0);
            stage_part(buf ^ 1, next, r, kb);
        }
    };

    // Set (t & 1) holds step t until it is staged.  Requests past the last step repeat the last one
    // (in bounds): no load sits inside a branch, so none is waited for early.
    RowSet set0, set1;
    const int last = steps - 1;
    fetch(0, set0);
    fetch(last < 1 ? last : 1, set1);
#pragma unroll
    for (int part = 0; part < 4; ++part) stage_part(0, 0, set0, part);
    fetch(last < 2 ? last : 2, set0);
    __syncthreads();
    for (int t = 0; t < steps; t += 2) {
        step(0, t + 1, set1);
        fetch(last < t + 3 ? last : t + 3, set1);
        __syncthreads();
        if (t + 1 >= steps) break;
        step(1, t + 2, set0);
        fetch(last < t + 4 ? last : t + 4, set0);
        __syncthreads();
    }

    // D layout of a 32x32 tile: column (k) = lane % 32, row (n) = 8 * (v / 4) + 4 * (lane / 32) + v % 4.
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int k = k0 + wk * 64 + t * 32 + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int n = n0 + wn * 64 + s * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (n < N) {
                    float *p = score + (size_t)n * K + k;
                    float g = alpha * acc[s][t][v];
                    if (beta != 0.f) g += beta * *p;
                    *p = g;
                }
            }
        }
}

// ---- 256 x 256 tiles ------------------------------------------------------------------------------
//
// A 128 x 128 tile reads 512 bytes of operands per sample for 128 x 128 products: at the matrix cores' rate 64 bytes per
// clock and CU, twice what the L2 delivers when all CUs ask.  This kernel's tile needs half of that.  Eight waves, two per
// SIMD, own 128 (n) x 64 (k) each: 4 x 2 tiles of v_mfma_f32_32x32x16_f16.  Steps of 32 samples pass through a ring of four
// LDS buffers, [operand][32 samples][256 columns] as the rows lie in memory, which loads with an LDS destination fill three
// steps ahead, and the transposition the MFMA operands need is done by the LDS reads (ds_read_b64_tr_b16: of the sixteen
// lanes of a group, lanes 4 j .. 4 j + 3 address sixteen columns of sample j, and lane i receives column i of samples
// 0 .. 3), so the multiplying waves issue nothing but reads, MFMAs and a few requests.  The 16-byte units of a sample's row
// are permuted by sample (unit u of sample m at u ^ 4 (m % 4)): the four samples of a read fall into different banks.
// One barrier per step, in its middle: behind it the next step is staged and this one's operands are in registers.
//
// Measured at M = 2048 (128 x 128 tiles in brackets), calls replayed from a graph on normally distributed inputs:
// 4096 x 4096, one round of tiles, 73.7 us = 932 TFLOP/s (104.9); 4096 x 11008 192 us (262), accumulating 210 us (318);
// unaligned 3333 x 4096 75 us (336), 9001 x 4096 193 us (753).  That was with all reads of a batch before its MFMAs; with two
// behind each MFMA (interleave), on another machine, both in turn: 4096 x 4096 71.7 -> 68.9 us (1.0 PFLOP/s), 11008 x 4096
// 196 -> 185, two samples into one score 4096 x 11008 410 -> 397, unaligned 9001 x 4096 406 -> 394.  On zeros 158 -> 147 where
// normal inputs take 196 -> 185: the difference is power.  The matrix cores work 53 to 55 % of the time (48 to 50 before), the LDS sees
// no bank conflict.  What is left at 4096 x 11008: 688 tiles on 256 CUs are three rounds at 2.69 rounds' work, and 180 MB
// of FP32 scores (36 us at HBM speed) are written at the rounds' ends.  Four waves of 128 x 128 (a third less LDS traffic,
// one wave per SIMD): 10 % slower, and slower with the reads so placed too; nontemporal stores: 10 % slower; the old score
// requested a tile ahead: no difference.
//
// N8 = false: rows of dY are not 16-byte aligned.  Their pieces come through registers (loads at 2-byte alignment, requested
// at the start of a step and stored at its end); only the piece that would reach beyond the end of dY is read from 16 bytes before
// the end and shifted (N >= 8).
constexpr int kBig = 256, kBigStep = 32, kBigThreads = 512, kBigStages = 4;
constexpr uint32_t kBigRow = kBig * 2, kBigOperand = kBigStep * kBigRow, kBigStage = 2 * kBigOperand;    // bytes
constexpr size_t kBigLds = (size_t)kBigStages * kBigStage;                                               // 128 KB

typedef short short4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4s __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2), may_alias));     // 16 bytes at 2-byte alignment
typedef __attribute__((address_space(3))) unsigned char lds_byte;

template <int N> __device__ inline void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

template <bool N8>
__global__ __launch_bounds__(kBigThreads) void score_big_kernel(const _Float16 *__restrict__ dY, const _Float16 *__restrict__ X,
                                                                int M, int N, int K, int tiles_n, int tiles_k, float alpha, float beta,
                                                                float *__restrict__ score)
{
    extern __shared__ unsigned char big_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // XCD x takes the x-th eighth of the tiles, in bands of four tile rows (see above).
    const int per_xcd = (tiles_n * tiles_k + 7) >> 3;
    const int lin = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (lin >= tiles_n * tiles_k) return;               // whole block, before any barrier
    const int band = lin / (4 * tiles_k), in_band = lin - band * 4 * tiles_k;
    const int band_rows = tiles_n - 4 * band < 4 ? tiles_n - 4 * band : 4;
    const int n0 = (4 * band + in_band % band_rows) * kBig, k0 = (in_band / band_rows) * kBig;
    const int wn = wave >> 2, wk = wave & 3;
    const int steps = (M + kBigStep - 1) / kBigStep;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)big_lds;

    // Staging: wave w brings samples 4 w .. 4 w + 3 of a step, two per 1 KB request; lane l takes the unit that belongs
    // at position l % 32 of its row.  Columns beyond N or K read column 0 (their results are not stored), samples
    // beyond M the last one (zeroed once they are in LDS).  A request's address is the step's first sample (scalar) plus a
    // lane offset that changes in the last step alone.
    const int row_in = 4 * wave + (lane >> 5);          // + 2 i: this lane's sample of the step
    uint32_t col_a[2], col_b[2];                        // first column of the lane's unit, per request
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int u = (lane & 31) ^ (4 * ((2 * i + (lane >> 5)) & 3));
        col_a[i] = n0 + 8 * u < N ? n0 + 8 * u : 0;
        col_b[i] = k0 + 8 * u < K ? k0 + 8 * u : 0;
    }
    auto sample = [&](int t, int i) {                   // within the step
        const int m = row_in + 2 * i, rest = M - 1 - t * kBigStep;
        return m < rest ? m : rest;
    };
    uint32_t off_a[2], off_b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        off_a[i] = ((uint32_t)(row_in + 2 * i) * N + col_a[i]) * 2;
        off_b[i] = ((uint32_t)(row_in + 2 * i) * K + col_b[i]) * 2;
    }
    // (m0 holds the LDS address; nothing else in this kernel uses it, and the compiler takes it in no clobber list.)
    auto load_lds = [&](uint32_t dst, uint32_t off, const _Float16 *base) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(base) : "memory");
    };
    auto slot = [&](int t, int i) { return (uint32_t)(t & (kBigStages - 1)) * kBigStage + (uint32_t)(4 * wave + 2 * i) * kBigRow; };
    auto cut = [&](int t) { return t * kBigStep + kBigStep > M; };         // the step ends beyond M
    auto request_a = [&](int t) {
        const _Float16 *base = dY + (size_t)t * kBigStep * N;
#pragma unroll
        for (int i = 0; i < 2; ++i) load_lds(lds0 + slot(t, i), cut(t) ? ((uint32_t)sample(t, i) * N + col_a[i]) * 2 : off_a[i], base);
    };
    auto request_b = [&](int t) {
        const _Float16 *base = X + (size_t)t * kBigStep * K;
#pragma unroll
        for (int i = 0; i < 2; ++i) load_lds(lds0 + slot(t, i) + kBigOperand, cut(t) ? ((uint32_t)sample(t, i) * K + col_b[i]) * 2 : off_b[i], base);
    };
    // N8 = false: the same pieces of dY in registers, by ordinary loads: the compiler knows that they are in flight and waits
    // before it touches the registers, whatever it does with them.
    auto piece_back = [&](int t, int i) {               // columns by which the piece would pass the end of dY
        const int past = (int)col_a[i] + 8 - N;
        return t * kBigStep + sample(t, i) == M - 1 && past > 0 ? past : 0;
    };
    auto request_piece = [&](int t, u32x4s piece[2]) {
        const _Float16 *base = dY + (size_t)t * kBigStep * N;
        const bool last = t == steps - 1;               // uniform
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t off = last ? ((uint32_t)sample(t, i) * N + col_a[i] - piece_back(t, i)) * 2 : off_a[i];
            piece[i] = *reinterpret_cast<const u32x4u *>(reinterpret_cast<const char *>(base) + off);
        }
    };
    auto store_piece = [&](int t, u32x4s piece[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (t == steps - 1) {                       // nonzero at most for the last columns of the last sample
                int back = piece_back(t, i);
                u32x4s &v = piece[i];
                for (; back >= 2; back -= 2) v = u32x4s{v.y, v.z, v.w, 0u};
                if (back) v = u32x4s{v.x >> 16 | v.y << 16, v.y >> 16 | v.z << 16, v.z >> 16 | v.w << 16, v.w >> 16};
            }
            *reinterpret_cast<u32x4s *>(big_lds + slot(t, i) + 16 * lane) = piece[i];
        }
    };
    // Samples beyond M of step t, which this wave brought, become zeros in both operands.
    auto zero_tail = [&](int t) {
        if (!cut(t)) return;                            // uniform: the last step alone
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (t * kBigStep + row_in + 2 * i >= M) {
                *reinterpret_cast<u32x4s *>(big_lds + slot(t, i) + 16 * lane) = u32x4s{0u, 0u, 0u, 0u};
                *reinterpret_cast<u32x4s *>(big_lds + slot(t, i) + kBigOperand + 16 * lane) = u32x4s{0u, 0u, 0u, 0u};
            }
    };

    // Operands: lane l holds column l % 32 of a 32-column tile and samples 8 (l / 32) .. + 7 of a batch of 16, read as two
    // times four samples.
    const int j = (lane >> 2) & 3, c = lane & 3, half = (lane >> 4) & 1;
    const uint32_t lane_at = (uint32_t)(8 * (lane >> 5) + j) * kBigRow + 16u * (2 * half + (c >> 1)) + 8u * (c & 1);
    uint32_t at_a[4], at_b[2];
#pragma unroll
    for (int s = 0; s < 4; ++s) at_a[s] = lane_at + 16u * (uint32_t)((16 * wn + 4 * s) ^ (4 * j));
#pragma unroll
    for (int s = 0; s < 2; ++s) at_b[s] = kBigOperand + lane_at + 16u * (uint32_t)((8 * wk + 4 * s) ^ (4 * j));
    half8s fa[2][4], fb[2][2];
    auto read_tile = [&](uint32_t at) {
        typedef __attribute__((address_space(3))) short4v lds_short4;
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(lds_byte *)(big_lds + at));
        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(lds_byte *)(big_lds + at + 4 * kBigRow));
        return __builtin_bit_cast(half8s, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_batch = [&](int t, int batch, int set) {
        const uint32_t base = (uint32_t)(t & (kBigStages - 1)) * kBigStage + (uint32_t)batch * 16 * kBigRow;
#pragma unroll
        for (int s = 0; s < 4; ++s) fa[set][s] = read_tile(base + at_a[s]);
#pragma unroll
        for (int s = 0; s < 2; ++s) fb[set][s] = read_tile(base + at_b[s]);
    };
    float16v acc[4][2];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[s][u][v] = 0.f;
    auto multiply = [&](int set) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[s][u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[set][s], fb[set][u], acc[s][u], 0, 0, 0);
    };

    // The twelve reads of the next batch go between the eight MFMAs of this one, two behind each.
    auto interleave = [] {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);          // an MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);          // LDS reads
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    // Steps 0, 1, 2 requested (unaligned: dY of steps 0 and 1); all of that staged.
    u32x4s first[2], second[2];
    if constexpr (!N8) {
        request_piece(0, first);
        if (steps > 1) request_piece(1, second);
    }
    for (int t = 0; t < 3 && t < steps; ++t) {
        if constexpr (N8) request_a(t);
        request_b(t);
    }
    if constexpr (!N8) {
        store_piece(0, first);
        if (steps > 1) store_piece(1, second);
    }
    wait_loads<0>();
    for (int t = 0; t < 3 && t < steps; ++t) zero_tail(t);
    __syncthreads();
    read_batch(0, 0, 0);
    for (int t = 0; t < steps; ++t) {
        u32x4s piece[2];
        const bool more = t + 3 < steps;                // uniform
        if constexpr (N8) {
            if (more) { request_a(t + 3); request_b(t + 3); }
        } else {
            if (more) request_b(t + 3);
            if (t + 2 < steps) request_piece(t + 2, piece);
        }
        __builtin_amdgcn_sched_barrier(0);
        read_batch(t, 1, 1);
        multiply(0);
        interleave();
        if constexpr (N8) {
            // Step t + 1 has landed, the two behind it may be on their way.
            if (more) wait_loads<8>();
            else wait_loads<0>();
            if (t + 1 < steps) zero_tail(t + 1);
        }
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        read_batch(t + 1, 0, 0);                        // past the last step: stale bytes, not used
        multiply(1);
        interleave();
        if constexpr (!N8) {
            // Step t + 2 is staged a barrier before it is read: its pieces have had this whole step to arrive, and X of the
            // steps up to t + 3 arrives with them.
            if (t + 2 < steps) {
                wait_loads<0>();
                store_piece(t + 2, piece);
                zero_tail(t + 2);
            }
        }
    }

    // D layout of a 32x32 tile: column (k) = lane % 32, row (n) = 8 * (v / 4) + 4 * (lane / 32) + v % 4.
    if (k0 + wk * 64 >= K) return;                      // K is a multiple of 128
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = k0 + wk * 64 + u * 32 + (lane & 31);
            const int nb = n0 + wn * 128 + s * 32 + 4 * (lane >> 5);
            float *p = score + (size_t)nb * K + k;
            // Rows v0 .. v1 of the sixteen; whole: none of them lies beyond N.
            auto finish = [&](auto whole, int v0, int v1) {
                float old[16];
                if (beta != 0.f)
#pragma unroll
                    for (int v = v0; v < v1; ++v) {
                        const int dn = 8 * (v >> 2) + (v & 3);
                        old[v] = decltype(whole)::value || nb + dn < N ? p[(size_t)dn * K] : 0.f;
                    }
#pragma unroll
                for (int v = v0; v < v1; ++v) {
                    const int dn = 8 * (v >> 2) + (v & 3);
                    float g = alpha * acc[s][u][v];
                    if (beta != 0.f) g += beta * old[v];
                    if (decltype(whole)::value || nb + dn < N) p[(size_t)dn * K] = g;
                }
            };
            if (n0 + wn * 128 + 128 <= N) { finish(std::true_type{}, 0, 16); continue; }
            // A tile cut by N: eight rows (four of each half of the wave) at a time, of which at most one lot is cut itself.
            // (A guard on every store is code enough to be fetched at 5 us a block: 100 x 1024, M = 33, 16.0 -> 10.7 us.)
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                const int rows = N - (n0 + wn * 128 + s * 32 + 2 * v);
                if (rows >= 8) finish(std::true_type{}, v, v + 4);
                else if (!N8 && rows > 0) finish(std::false_type{}, v, v + 4);
            }
        }
}

}  // namespace

hipError_t launch_score(const void *dY, const void *X, int M, int N, int K, float alpha, float beta, float *score,
                        hipStream_t st)
{
    const _Float16 *d = static_cast<const _Float16 *>(dY), *x = static_cast<const _Float16 *>(X);
    const bool n8 = N % 8 == 0;
    const int cus = device_cus();
    static std::atomic<uint32_t> lds_allowed[4];        // per kernel
    // Which tile.  A round of 256 x 256 tiles over the chip does twice the work of a round of 128 x 128 ones (two blocks per
    // CU), so it is taken where it needs at most half the rounds (us at M = 33 and 2048, 128 against 256: one round
    // against one, 2048 x 4096 13.2 and 56.8 against 13.5 and 57.8; two against one, 4096 x 4096 20.7 and 104.9 against 17.6
    // and 73.7; six against three, 4096 x 11008 44.9 and 262 against 37.8 and 192).  In between (three against two,
    // 6144 x 4096 27.2 and 148 against 24.9 and 120) the large tiles win as well, which this rule forgoes.
    // Rows of dY that are not 16-byte aligned take the large tiles from 12 channels on: the other kernel reads them element
    // by element, which is the faster way only while nearly all lanes of a load share one column (us at M = 33 and 2048,
    // 128 against 256: 9 x 4096 8.9 and 46.9 against 9.5 and 54.4; 12 x 1024 9.8 and 54.1 against 9.3 and 54.1;
    // 100 x 1024 13.3 and 82.8 against 10.8 and 55.4; 9001 x 4096 97 and 753 against 36 and 193).
    const int big_k = (K + kBig - 1) / kBig, big_n = (N + kBig - 1) / kBig;
    const int tiles_k = K / kTile, tiles_n = (N + kTile - 1) / kTile;
    const int64_t rounds_big = ((int64_t)big_k * big_n + cus - 1) / cus, rounds_small = ((int64_t)tiles_k * tiles_n + 2 * cus - 1) / (2 * cus);
    if (n8 ? rounds_small >= 2 * rounds_big : N >= 12) {
        const void *kernel = n8 ? reinterpret_cast<const void *>(&score_big_kernel<true>) : reinterpret_cast<const void *>(&score_big_kernel<false>);
        hipError_t e = allow_dynamic_lds(kernel, (int)kBigLds, lds_allowed[n8 ? 2 : 3]);
        if (e != hipSuccess) return e;
        const int blocks = (big_k * big_n + 7) / 8 * 8;
        if (n8) score_big_kernel<true><<<blocks, kBigThreads, kBigLds, st>>>(d, x, M, N, K, big_n, big_k, alpha, beta, score);
        else score_big_kernel<false><<<blocks, kBigThreads, kBigLds, st>>>(d, x, M, N, K, big_n, big_k, alpha, beta, score);
        return hipGetLastError();
    }
    {
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(&score_kernel<true>), (int)kScoreLds, lds_allowed[0]);
        if (e == hipSuccess)
            e = allow_dynamic_lds(reinterpret_cast<const void *>(&score_kernel<false>), (int)kScoreLds, lds_allowed[1]);
        if (e != hipSuccess) return e;
    }
    const int blocks = (tiles_n * tiles_k + 7) / 8 * 8;
    if (n8)
        score_kernel<true><<<blocks, kScoreThreads, kScoreLds, st>>>(d, x, M, N, K, tiles_n, tiles_k, alpha, beta, score);
    else
        score_kernel<false><<<blocks, kScoreThreads, kScoreLds, st>>>(d, x, M, N, K, tiles_n, tiles_k, alpha, beta, score);
    return hipGetLastError();
}

}  // namespace gwq
