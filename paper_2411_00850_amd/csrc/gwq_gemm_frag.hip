// gwq_linear for M > 16 on gfx950 where the caller's scratch has room for a copy of X: an MFMA GEMM whose X operands come
// straight from memory into registers.
//
//   Y[m][n] = sum_k X[m][k] * What[n][k],  What = s*(q - z) (Sec. 3.2, Eq. 10) with the FP16 outliers in their places
//
// In gwq_gemm.hip both operands pass the LDS and X is copied there with every step.  Here X does not: arrange_kernel copies
// it once into fragment order - the 1 KB that one v_mfma_f32_16x16x32 takes of 16 rows and 32 columns, lane by lane - so
// that a wave fetches an operand with one coalesced 16-byte load per lane, requested a whole group of 128 columns ahead.
// Only the weights, which must meet their outliers at addresses known at run time, pass through the LDS, read by as few waves
// as can be.  The copy is a launch of 2 us and 0.6 us per million entries.
//
// A block owns a tile of Y, 256 x 128 or 32 J x 128, and walks K group by group (128 columns).  Four consumer waves, one
// per SIMD, multiply; four or eight producer waves turn the next group's codes into FP16 (exact q - z, one multiply by the
// scale) and store them to one of two LDS buffers, then the group's outliers over their zeros.  One barrier per group.
//
// What bounds it: a group takes a producer wave 500 to 900 clocks per run of 16 channels beside its neighbours (95 vector
// instructions, two producers a SIMD one after the other) and 400 for its stores, which is longer than the MFMAs of a tile of
// 128 rows or less; hence eight producers where the registers allow them (28672 x 8192, M = 64: 83 us with four, 61 with eight;
// M = 301, tiles of 160: 191 and 166).  With the producers' loop unrolled over a window of eight groups, so that nothing but
// vector instructions is left of the bookkeeping and no wait drains the loads in flight: M = 64 60 -> 56 us, M = 2048 799 -> 765
// (1.26 PFLOP/s), 11008 x 4096 172 -> 166.  With 256 rows it is power that bounds it: on another machine the same instructions took
// 752 us on normal numbers and 552 on zeros for X and the weights (28672 x 8192, M = 2048).
#include <stdio.h>

#include <type_traits>

#include "gwq_gemm_parts.h"

namespace gwq {
namespace {

typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kDump = 512;              // bytes behind the two buffers, where absent outliers are written
constexpr int kFragBytes = 1024;        // one operand: 16 rows x 32 columns
constexpr int kRun = 16 * 80;           // bytes of a run's side data: 64 per channel, 80 apart for the LDS banks
// LDS of a tile of BN channels: two buffers of weights (256 bytes per channel and group, 16-byte chunks permuted), the dump,
// records and outliers of eight groups at a time (see the producers).
constexpr int weight_bytes(int BN) { return BN * kGroup * 2; }
constexpr size_t lds_bytes(int BN) { return 2 * weight_bytes(BN) + kDump + (BN / 16) * (3 + 4) * kRun; }

// Where chunk c (columns 8c .. 8c+7) of a channel lies in its row of an LDS buffer.  A fragment read takes the same chunk
// of 16 channels (or neighbouring chunks of two sets of eight, as the hardware groups the lanes), a store the chunks
// 4 apart of two channels: each meets all banks once.
__device__ inline uint32_t chunk_place(uint32_t c, uint32_t channel) { return c ^ (c >> 3 << 1) ^ (channel & 15); }

// X [M][K] -> fragment order [ceil(M/16)][K/32][64 lanes][8]: lane l holds columns 8*(l/16) .. +7 of the 32, of row l%16.
// Rows beyond M are zeros.  One wave per 16 rows and 128 columns.
__global__ __launch_bounds__(256) void arrange_kernel(const uint16_t *__restrict__ X, uint16_t *__restrict__ F, int M, int K)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int pieces = (K / kGroup + 3) / 4;
    const int m16 = blockIdx.x / pieces, g = blockIdx.x % pieces * 4 + wave;
    if (g >= K / kGroup) return;
    const int m = m16 * 16 + (lane & 15);
    const uint16_t *src = X + (size_t)(m < M ? m : M - 1) * K + g * kGroup + 8 * (lane >> 4);
    uint16_t *dst = F + ((size_t)m16 * (K / 32) + 4 * g) * (kFragBytes / 2) + 8 * lane;
    u32x4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const u32x4 *>(src + 32 * i);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        *reinterpret_cast<u32x4 *>(dst + i * (kFragBytes / 2)) = m < M ? v[i] : u32x4{0, 0, 0, 0};
}

// Sixteen bytes at 2-byte alignment: eight CSR entries (gfx950 global memory takes unaligned vector loads).
struct __attribute__((packed, aligned(2))) U128a2 { uint32_t x, y, z, w; };

struct FragArgs {
    const uint32_t *qweight;
    const uint16_t *col_idx, *out_val;
    const GroupRecord *rec;
    const uint32_t *fine;
    const char *xf;
    void *y;
    float *partial;                     // FP32 sums of a K-split launch, [split][M][N]; else NULL
    int split_groups, N, K, M, tiles_m, tiles_n, last_entry;
};

// J: 16-row pieces of X per consumer wave; WM x WN: consumer waves along m and n; P: producer waves; D: groups a producer
// has in flight.  FINE, BF16 as in gwq_gemm.hip.
template <int BITS, int BN, int J, int WM, int WN, int P, int D, bool FINE, bool BF16>
__device__ inline void frag_tile(const FragArgs &a, char *lds)
{
    static_assert(WM * WN == 4, "one consumer wave per SIMD");
    constexpr int BM = 16 * J * WM;
    constexpr int NB = BN / 16 / WN;                    // 16-channel pieces per consumer wave
    constexpr int wpg = words_per_group(BITS);
    const int N = a.N, K = a.K, M = a.M;

    // Tile order: bands of two m-tiles, n fastest inside a band; when the tile count divides by 8 every XCD (blocks go
    // round-robin over the 8 XCDs) gets one contiguous run of that order.
    const int total = a.tiles_m * a.tiles_n;
    const int split = blockIdx.x / total;
    int id = blockIdx.x % total;
    if (total % 8 == 0) id = (id % 8) * (total / 8) + id / 8;
    const int band_m = a.tiles_m >= 2 ? 2 : 1;
    const int per_band = band_m * a.tiles_n;
    const int band = id / per_band, in_band = id % per_band;
    const int rows_here = (band + 1) * band_m <= a.tiles_m ? band_m : a.tiles_m - band * band_m;
    const int nt = in_band / rows_here, mt = band * band_m + in_band % rows_here;
    const int n0 = nt * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gpr = K / kGroup;
    const int g_first = split * a.split_groups;         // this block's groups: g_first .. g_first + gl - 1
    const int gl = gpr - g_first < a.split_groups ? gpr - g_first : a.split_groups;

    // Every wave passes 1 + gl barriers.  Barrier 0: group 0 is staged.  Barrier t + 1: group t + 1 is staged, and group t
    // has been read (its last fragments are in registers).
    if (wave >= 4) {
        // ======================================= producers =====================================
        // Wave (wave - 4) owns I runs of 16 channels, four lanes each; lane l has channel l/4 of a run and slot l%4 of
        // every group: 64 bytes of codes per channel and load.  A load that touches 16 rows costs the CU's address unit
        // several times what a contiguous one does, and three more of them per group (columns and values of the
        // outliers, record) cost as much as the MFMAs of a third of the tile (28672 x 8192, M = 1024: 460 us with them,
        // 373 without).  So these come a window of eight groups at a time: one load per wave and trip, in turn a run's
        // records, its columns and its values, 64 bytes per channel, into the wave's own part of the LDS.
        //
        // A trip is bound by one wave's own instructions (nothing else on its SIMD hides them but MFMAs), so the loop is
        // unrolled over a window: which side load a trip makes and which buffer it fills are known when compiling, and what a
        // trip needs of the side data is read from the LDS a trip ahead.
        constexpr int RUNS = BN / 16, I = RUNS / P;     // runs of the tile, runs per wave
        static_assert((D == 2 && I <= 2) || (D == 4 && I == 1), "a window's entries must be in the LDS before its first group");
        const int slot = lane & 3, ch16 = lane >> 2;
        const DecodeConsts dc(BITS);
        const char *q_tile = reinterpret_cast<const char *>(a.qweight + ((size_t)n0 * gpr + g_first) * wpg);
        const char *r_tile = reinterpret_cast<const char *>(a.rec + (size_t)n0 * (gpr + 1) + g_first);
        const char *f_tile = reinterpret_cast<const char *>(a.fine + ((size_t)n0 * gpr + g_first) * 8);
        // Side data: records [3][RUNS][16][8], entries [2][RUNS]{columns, values}[16][32]; channels 80 bytes apart.
        char *const dump = lds + 2 * weight_bytes(BN) + 8 * lane;
        char *const side = lds + 2 * weight_bytes(BN) + kDump + (wave - 4) * kRun + 80 * ch16;
        constexpr uint32_t kRecWindow = RUNS * kRun, kCsrWindow = 2 * RUNS * kRun, kCsr = 3 * kRecWindow;
        uint32_t rec_window[3] = {0, kRecWindow, 2 * kRecWindow};          // of windows w, w + 1, w + 2
        uint32_t csr_window[2] = {kCsr + (wave - 4) * kRun, kCsr + kCsrWindow + (wave - 4) * kRun};     // of windows w, w + 1
        uint32_t q_off[I], r_off[I], f_off[I];          // bytes
        uint32_t dst[I];                                // LDS bytes of the channel's row; its chunks as this lane stores them
        uint32_t chunk[4];
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const int ch = 16 * (wave - 4 + P * i) + ch16;
            const int c = n0 + ch < N ? ch : N - 1 - n0;                // clamped: loads stay in bounds, the tile's rows are unused
            q_off[i] = (uint32_t)c * (uint32_t)gpr * (4 * wpg) + 4 * (BITS == 4 ? 4 : 3) * slot;
            r_off[i] = (uint32_t)c * (uint32_t)(gpr + 1) * 8;
            f_off[i] = (uint32_t)c * (uint32_t)gpr * 32 + 8 * slot;
            dst[i] = (uint32_t)ch * (2 * kGroup);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) chunk[j] = 16 * chunk_place(4 * slot + j, ch16);
        // Lane s of a channel fetches records g = 8w + 2s and g + 1, or gl - 1 and gl (the row's end) where g would pass that.
        auto rec_offset = [&](int g0, int i) {
            const int g = g0 + 2 * slot;
            return r_off[i] + 8u * (uint32_t)(g < gl - 1 ? g : gl - 1);
        };
        // Record g0 + k of the window that starts at group g0 (a multiple of 8); record gl beyond that.
        auto read_rec = [&](uint32_t window, int g0, int k, int i) {
            const uint32_t second = k & 1 ? 8u : g0 + k >= gl ? 8u : 0u;
            return *reinterpret_cast<const uint2 *>(side + window + P * i * kRun + k / 2 * 16 + second);
        };
        auto csr_offset = [&](uint32_t first) {         // bytes; the arrays carry 16 spare bytes
            const int j = (int)first + 8 * slot;
            return 2u * (uint32_t)(j < a.last_entry ? j : a.last_entry);
        };
        auto load16 = [](const void *base, uint32_t offset) { return *reinterpret_cast<const U128a2 *>(static_cast<const char *>(base) + offset); };
        auto store16 = [&](uint32_t at, const U128a2 &v) { *reinterpret_cast<u32x4 *>(side + at + 16 * slot) = u32x4{v.x, v.y, v.z, v.w}; };

        SlotRegs<BITS> codes[D][I];
        uint2 sub[D][I];                                // FINE: scale | zero << 16 of the slot's halves
        U128a2 side_regs[D];
        uint2 now[I], next[I], after[I];                // records of groups t, t + 1 and, read during trip t, t + 2
        uint32_t window_first[I];
        uint32_t cols[I], vals[I];                      // entries 2 slot and 2 slot + 1 of group t
        struct Entries { uint32_t c[2], v[2], shift; } ahead[I];           // the words that hold those of group t + 1
        auto issue_codes = [&](int g, int r) {
            g = g < gl ? g : gl - 1;                    // past the end: the last group again, unused
            const char *q = q_tile + (uint32_t)g * (4 * wpg), *f = f_tile + (uint32_t)g * 32;
#pragma unroll
            for (int i = 0; i < I; ++i) {
                load_slot<BITS>(codes[r][i], reinterpret_cast<const uint32_t *>(q + q_off[i]), 0);
                if constexpr (FINE) sub[r][i] = *reinterpret_cast<const uint2 *>(f + f_off[i]);
            }
        };
        // Trips 0 .. I-1 of window w ask for the records of window w + 2, trips 2 .. 2I+1 for columns and values of window
        // w + 1; D trips later, in the same window, they go to the LDS.
        auto asks_records = [](int k) { return k >= 0 && k < I; };
        auto asks_entries = [](int k) { return k >= 2 && k < 2 + 2 * I; };
        auto side_run = [](int k) { return I == 2 && (k == 1 || k >= 4) ? I - 1 : 0; };
        auto keep_side = [&](int k, int r) {            // what trip k asked for
            if (asks_records(k)) store16(rec_window[2] + P * side_run(k) * kRun, side_regs[r]);
            else if (asks_entries(k)) store16(csr_window[1] + (2 * P * side_run(k) + (k & 1)) * kRun, side_regs[r]);
        };
        // A group's entries, from its window's in the LDS, its record, and the entry at which the window starts.
        auto read_entries = [&](uint32_t window, uint32_t first, uint32_t start, int i) {
            const uint32_t e = first - start + 2 * slot, o = e < 31 ? e : 31;
            const uint32_t *run = reinterpret_cast<const uint32_t *>(side + window + 2 * P * i * kRun) + (o >> 1);
            ahead[i] = Entries{{run[0], run[1]}, {run[kRun / 4], run[kRun / 4 + 1]}, 16 * (o & 1)};
        };
        auto take_entries = [&](int i) {
            cols[i] = __builtin_amdgcn_alignbit(ahead[i].c[1], ahead[i].c[0], ahead[i].shift);
            vals[i] = __builtin_amdgcn_alignbit(ahead[i].v[1], ahead[i].v[0], ahead[i].shift);
        };
        auto column_place = [&](uint32_t c) { return (2 * c) ^ (c >> 6 << 5) ^ (16u * ch16); };   // chunk_place of column c, in bytes
        auto stage = [&](int t, int k, int r) {
            const uint32_t k_lo = (uint32_t)(g_first + t) * kGroup;
            uint64_t more = 0;
#pragma unroll
            for (int i = 0; i < I; ++i) {
                const SlotRegs<BITS> &q = codes[r][i];
                char *row = lds + (k & 1) * weight_bytes(BN) + dst[i];
                const uint32_t sz = now[i].y, z = sz >> 16, s2 = (sz & 0xFFFFu) * 0x10001u;
                u32x4 f[4];
                uint32_t tail = 0;
                if constexpr (BITS == 3)                // the block's tail word is the fourth word of slot 3: quad_perm 3,3,3,3
                    tail = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)q.fourth, 0xFF, 0xF, 0xF, false) >> (3 * slot);
                if constexpr (FINE) {
                    const uint32_t lo = sub[r][i].x, hi = sub[r][i].y;
                    if constexpr (BITS == 4) decode_slot4_halves(q.w, lo >> 16, hi >> 16, dc, f);
                    else decode_slot3_halves(q.w, tail, lo >> 16, hi >> 16, dc, f);
                    scale_halves(f, (lo & 0xFFFFu) * 0x10001u, (hi & 0xFFFFu) * 0x10001u);
                } else {
                    if constexpr (BITS == 4) decode_slot4(q.w, z, dc, f);
                    else decode_slot3(q.w, tail, z, dc, f);
                    if constexpr (BF16) {
                        const float sf = (float)__builtin_bit_cast(_Float16, (uint16_t)(sz & 0xFFFFu));
#pragma unroll
                        for (int j = 0; j < 4; ++j) f[j] = scale_frag_bf16(f[j], sf);
                    } else {
                        scale_halves(f, s2, s2);
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4 *>(row + chunk[j]) = f[j];
                // The group's first eight outliers, two per lane, over their decoded zeros (stored before by this wave,
                // whose LDS accesses are in order); absent entries go to the dump, without a branch.
                const int cnt = (int)(next[i].x - now[i].x), room = 32 - (int)(now[i].x - window_first[i]);
                const int near = cnt < room ? cnt : room;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const uint32_t c = ((cols[i] >> (16 * e)) & 0xFFFFu) - k_lo;
                    const uint32_t v = (vals[i] >> (16 * e)) & 0xFFFFu;
                    char *at = 2 * slot + e < near && c < (uint32_t)kGroup ? row + column_place(c) : dump;
                    *reinterpret_cast<uint16_t *>(at) = BF16 ? half_bits_to_bf16_bits(v) : (uint16_t)v;
                }
                more |= __builtin_amdgcn_ballot_w64(cnt > (room < 8 ? room : 8));
            }
            if (more) {                                 // rare: more than eight outliers in this group, or than 32 in its window so far
#pragma unroll
                for (int i = 0; i < I; ++i) {
                    const int cnt = (int)(next[i].x - now[i].x), room = 32 - (int)(now[i].x - window_first[i]);
                    if (slot == 0)
                        for (int e = room < 0 ? 0 : room < 8 ? room : 8; e < cnt; ++e) {
                            const uint32_t c = load_u16_now(a.col_idx + now[i].x + e) - k_lo;
                            if (c < (uint32_t)kGroup) {
                                const uint32_t v = load_u16_now(a.out_val + now[i].x + e);
                                *reinterpret_cast<uint16_t *>(lds + (k & 1) * weight_bytes(BN) + dst[i] + column_place(c)) =
                                    BF16 ? half_bits_to_bf16_bits(v) : (uint16_t)v;
                            }
                        }
                }
            }
        };
        // Trip t = g0 + k of the window at g0 stages group t and refills its registers with group t + D.
        auto trip = [&](int g0, int k) {
            const int t = g0 + k, r = k % D;
            if (k == 0) {
#pragma unroll
                for (int i = 0; i < I; ++i) window_first[i] = now[i].x;
            }
            keep_side(k - D, r);
            if (k == 7) wave_meet();                    // the next window's entries, stored up to now, are read in this trip
            uint32_t side_first = 0;
            if (asks_entries(k)) side_first = read_rec(rec_window[1], g0 + 8, 0, side_run(k)).x;
#pragma unroll
            for (int i = 0; i < I; ++i) {
                after[i] = k < 6 ? read_rec(rec_window[0], g0, k + 2, i) : read_rec(rec_window[1], g0 + 8, k - 6, i);
                if (k < 7) read_entries(csr_window[0], next[i].x, window_first[i], i);
                else read_entries(csr_window[1], next[i].x, next[i].x, i);
            }
            __builtin_amdgcn_sched_barrier(0);
            stage(t, k, r);
            __builtin_amdgcn_sched_barrier(0);
            issue_codes(t + D, r);
            if (asks_records(k)) side_regs[r] = load16(r_tile, rec_offset(g0 + 16, side_run(k)));
            else if (asks_entries(k)) side_regs[r] = load16(k & 1 ? a.out_val : a.col_idx, csr_offset(side_first));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < I; ++i) {
                take_entries(i);
                now[i] = next[i];
                next[i] = after[i];
            }
            __syncthreads();
        };
        {
            U128a2 v0[I], v1[I];
#pragma unroll
            for (int i = 0; i < I; ++i) v0[i] = load16(r_tile, rec_offset(0, i)), v1[i] = load16(r_tile, rec_offset(8, i));
#pragma unroll
            for (int r = 0; r < D; ++r) issue_codes(r, r);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < I; ++i) {
                store16(rec_window[0] + P * i * kRun, v0[i]);
                store16(rec_window[1] + P * i * kRun, v1[i]);
            }
            wave_meet();
#pragma unroll
            for (int i = 0; i < I; ++i) {
                now[i] = read_rec(rec_window[0], 0, 0, i);
                next[i] = read_rec(rec_window[0], 0, 1, i);
                v0[i] = load16(a.col_idx, csr_offset(now[i].x));
                v1[i] = load16(a.out_val, csr_offset(now[i].x));
            }
#pragma unroll
            for (int i = 0; i < I; ++i) {
                store16(csr_window[0] + 2 * P * i * kRun, v0[i]);
                store16(csr_window[0] + (2 * P * i + 1) * kRun, v1[i]);
            }
            wave_meet();
#pragma unroll
            for (int i = 0; i < I; ++i) {
                read_entries(csr_window[0], now[i].x, now[i].x, i);
                take_entries(i);
            }
        }
        // Whole windows, then the rest, each trip inside the branch of the one before: a way out of the loop's middle, or past
        // a trip, would join paths with other loads in flight, and the compiler would wait there for all of them.
        int g0 = 0;
        for (; g0 + 8 <= gl; g0 += 8) {
#pragma unroll
            for (int k = 0; k < 8; ++k) trip(g0, k);
            const uint32_t oldest = rec_window[0], csr = csr_window[0];
            rec_window[0] = rec_window[1], rec_window[1] = rec_window[2], rec_window[2] = oldest;
            csr_window[0] = csr_window[1], csr_window[1] = csr;
        }
        auto rest = [&](auto self, auto k) {
            if constexpr (k < 7)
                if (g0 + k < gl) {
                    trip(g0, k);
                    self(self, std::integral_constant<int, k + 1>{});
                }
        };
        rest(rest, std::integral_constant<int, 0>{});
        __syncthreads();
        return;
    }

    // ========================================= consumers =======================================
    // MFMAs of 16 x 16 x 32: lane l of an operand holds row (or channel) l % 16, columns 8*(l/16) .. +7 of the 32.  (With
    // 32 x 32 x 16 a tile of 8192 x 8192, M = 1024, took 8 % fewer clocks and 3 % more time.)
    const int wm = wave / WN, wn = wave % WN;
    const int row = lane & 15, b = lane >> 4;
    const int kb_row = K / 32, m16_last = (M + 15) / 16 - 1;
    const char *xa[J];                                  // wave-uniform
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int m16 = mt * (BM / 16) + wm * J + j;
        xa[j] = a.xf + ((size_t)(m16 < m16_last ? m16 : m16_last) * kb_row + 4 * g_first) * kFragBytes;
    }
    float4v acc[J][NB];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[j][n] = float4v{0.f, 0.f, 0.f, 0.f};

    // A batch: the J MFMAs of one weight fragment.  Weight fragments are requested R - 1 batches ahead.
    constexpr int S = 4 * NB;                           // batches per group
    constexpr int R = NB == 8 || J > 3 || (J == 3 && P == 8) ? 8 : 16;      // register sets for the weights
    static_assert(S % R == 0, "a batch's register set does not depend on the group");
    constexpr int Q = R - 1;
    constexpr int XS = P == 8 && J > 4 ? 2 : 4;         // register sets for X: requested XS fragments ahead
    u32x4 fa[XS][J], fb[R];
    // chunk_place of fragment kb: what the lane adds to the chunk's number only flips address bits below a row.
    const uint32_t w0 = (uint32_t)(wn * (16 * NB) + row) * (2 * kGroup) + 16 * chunk_place(b, row);
    auto read_x = [&](int g, int kb) {                  // fragment kb of group g (of the next group for kb >= 4)
        g += kb / 4;
        const uint32_t off = (uint32_t)(g < gl ? g : gl - 1) * (4 * kFragBytes) + 16 * lane;
#pragma unroll
        for (int j = 0; j < J; ++j) fa[kb % XS][j] = *reinterpret_cast<const u32x4 *>(xa[j] + off + kb % 4 * kFragBytes);
    };
    auto read_w = [&](int g, int s) {                   // batch s of group g (of the next group for s >= S)
        const uint32_t at = w0 ^ (16 * chunk_place(4 * (s % S / NB), 0));
        fb[s % R] = *reinterpret_cast<const u32x4 *>(lds + ((g + s / S) & 1) * weight_bytes(BN) + at + (s % NB) * (32 * kGroup));
    };
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
#pragma unroll
    for (int kb = 0; kb < XS; ++kb) {
        read_x(0, kb);
        fence();                                        // in the order of the loop, whose waits count on it
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < Q; ++s) read_w(0, s);
    for (int g = 0; g < gl; ++g) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (s == S - Q) __syncthreads();            // the next group is staged; this one's fragments are all in registers
            read_w(g, s + Q);
            fence();
#pragma unroll
            for (int j = 0; j < J; ++j) {
                float4v &c = acc[j][s % NB];
                const u32x4 w = fb[s % R], x = fa[s / NB % XS][j];
                if constexpr (BF16) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
                else c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, w), __builtin_bit_cast(half8, x), c, 0, 0, 0);
            }
            fence();
            if ((s + 1) % NB == 0) read_x(g, s / NB + XS);
            fence();
        }
    }

    // Lane l of an MFMA's result holds row l % 16 of the tile and channels 4*(l/16) .. +3.  Rows are stored at whatever
    // alignment N and Y give them (global memory takes unaligned vector stores).
    typedef std::conditional_t<BF16, __bf16, _Float16> act_t;
    const int m_wave = mt * BM + wm * (16 * J), n_wave = n0 + wn * (16 * NB);
    if (a.partial) {
        struct __attribute__((packed, aligned(4))) Four { float e[4]; };
        float *y = a.partial + (size_t)split * M * N;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int m = m_wave + 16 * j + row;
            if (m >= M) continue;
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                const int ch = n_wave + 16 * n + 4 * b;
                float *p = y + (size_t)m * N + ch;
                if (ch + 3 < N) {
                    *reinterpret_cast<Four *>(p) = Four{acc[j][n][0], acc[j][n][1], acc[j][n][2], acc[j][n][3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (ch + e < N) p[e] = acc[j][n][e];
                }
            }
        }
        return;
    }
    // 16-bit results go through the LDS (free since the last barrier) and out in whole runs of a row: stored from the
    // MFMA's layout, 32 bytes of 16 rows each, a 256 x 128 tile took 3 us longer.
    struct __attribute__((packed, aligned(2))) Eight { u32x4 v; };
    typedef act_t act4 __attribute__((ext_vector_type(4)));
    constexpr int kOut = 32 * NB + 16, kLanes = 2 * NB; // bytes of a row in LDS; lanes that store a row
    char *const out = lds + wave * (16 * J * kOut);
    static_assert(4 * 16 * J * kOut <= (int)lds_bytes(BN), "the tile fits");
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int n = 0; n < NB; ++n)
            *reinterpret_cast<act4 *>(out + (16 * j + row) * kOut + 32 * n + 8 * b) =
                act4{(act_t)acc[j][n][0], (act_t)acc[j][n][1], (act_t)acc[j][n][2], (act_t)acc[j][n][3]};
    wave_meet();
    const int ch = n_wave + 8 * (lane % kLanes);
#pragma unroll
    for (int i = 0; i < 16 * J * kLanes / 64; ++i) {
        const int r = i * (64 / kLanes) + lane / kLanes;
        const u32x4 v = *reinterpret_cast<const u32x4 *>(out + r * kOut + 16 * (lane % kLanes));
        if (m_wave + r >= M) continue;
        act_t *p = static_cast<act_t *>(a.y) + (size_t)(m_wave + r) * N + ch;
        if (ch + 7 < N) {
            reinterpret_cast<Eight *>(p)->v = v;
        } else {
            const uint16_t *h = reinterpret_cast<const uint16_t *>(out + r * kOut + 16 * (lane % kLanes));
            for (int e = 0; ch + e < N; ++e) reinterpret_cast<uint16_t *>(p)[e] = h[e];
        }
    }
}

// Tiles of WM * 32 MS rows, consumer waves one above the other (32 MS rows x 64 NS channels each): 256 x 128 as <.., 2, 2, 4, ..>.
template <int BITS, int MS, int NS, int WM, bool FINE, bool BF16>
__global__ __launch_bounds__(512) void gemm_kernel(const FragArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    frag_tile<BITS, 64 * NS, 2 * MS, WM, 1, 4, 2, FINE, BF16>(a, lds);
}
// Tiles of 32 J rows x 128 channels, consumer waves 2 x 2 (16 J rows x 64 channels each).
constexpr int row_producers(int rows) { return rows <= 160 ? 8 : 4; }
template <int BITS, int J, bool FINE, bool BF16>
__global__ __launch_bounds__(64 * (4 + row_producers(32 * J))) void gemm_kernel_rows(const FragArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr int P = row_producers(32 * J);
    frag_tile<BITS, 128, J, 2, 2, P, P == 8 ? 4 : 2, FINE, BF16>(a, lds);
}

template <int BITS, bool FINE, bool BF16>
hipError_t launch_tile(int rows, const FragArgs &args, int blocks, hipStream_t st)
{
    const size_t lds = lds_bytes(128);
    static std::atomic<uint32_t> allowed[8];            // per instantiation; zero-initialised
#define GWQ_FRAG(IDX, KERNEL)                                                                                  \
    {                                                                                                          \
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(&KERNEL), (int)lds, allowed[IDX]);     \
        if (e != hipSuccess) return e;                                                                         \
        KERNEL<<<blocks, 64 * (4 + row_producers(rows)), lds, st>>>(args);                                                                \
        return hipGetLastError();                                                                              \
    }
    switch (rows) {
    case 32: GWQ_FRAG(0, (gemm_kernel_rows<BITS, 1, FINE, BF16>))
    case 64: GWQ_FRAG(1, (gemm_kernel_rows<BITS, 2, FINE, BF16>))
    case 96: GWQ_FRAG(2, (gemm_kernel_rows<BITS, 3, FINE, BF16>))
    case 128: GWQ_FRAG(3, (gemm_kernel_rows<BITS, 4, FINE, BF16>))
    case 160: GWQ_FRAG(4, (gemm_kernel_rows<BITS, 5, FINE, BF16>))
    case 192: GWQ_FRAG(5, (gemm_kernel_rows<BITS, 6, FINE, BF16>))
    default: GWQ_FRAG(6, (gemm_kernel<BITS, 2, 2, 4, FINE, BF16>))
    }
#undef GWQ_FRAG
}

}  // namespace

size_t frag_bytes(int64_t M, int64_t K) { return (size_t)((M + 15) / 16) * (size_t)(K / 32) * kFragBytes; }

hipError_t launch_gemm_frag(const gwq_packed &P, const void *X, int M, void *Y, const void *index, void *frag, float *partial,
                            int rows, int splits, int split_groups, hipStream_t st, PlanText *describe, bool bf16)
{
    const int tiles_m = (M + rows - 1) / rows, bn = 128, tiles_n = (int)((P.N + bn - 1) / bn);
    const bool fine = P.group != kGroup;
    if (describe) {
        char name[64];
        const char *f = fine ? "true" : "false", *h = bf16 ? "true" : "false";
        if (rows == 256) snprintf(name, sizeof(name), "gemm_kernel<%d,2,2,4,%s,%s>", P.bits, f, h);
        else snprintf(name, sizeof(name), "gemm_kernel_rows<%d,%d,%s,%s>", P.bits, rows / 32, f, h);
        snprintf(describe->text, sizeof(describe->text), "%s tile %dx%d grid %d block %d lds %zu k_splits %d", name, rows, bn,
                 tiles_m * tiles_n * splits, 64 * (4 + row_producers(rows)), lds_bytes(bn), splits);
        return hipSuccess;
    }
    const int pieces = (P.K / kGroup + 3) / 4;
    arrange_kernel<<<(M + 15) / 16 * pieces, 256, 0, st>>>(static_cast<const uint16_t *>(X), static_cast<uint16_t *>(frag), M, P.K);
    FragArgs a;
    a.qweight = P.qweight; a.col_idx = P.col_idx; a.out_val = P.out_val;
    a.rec = static_cast<const GroupRecord *>(index);
    a.fine = reinterpret_cast<const uint32_t *>(static_cast<const char *>(index) + index_record_bytes(P.N, P.K));
    a.xf = static_cast<const char *>(frag);
    a.y = Y;
    a.partial = splits > 1 ? partial : nullptr;
    a.split_groups = split_groups;
    a.N = P.N; a.K = P.K; a.M = M;
    a.tiles_m = tiles_m; a.tiles_n = tiles_n;
    a.last_entry = P.n_outliers > 0 ? (int)P.n_outliers - 1 : 0;
    const int blocks = tiles_m * tiles_n * splits;
    if (bf16) return P.bits == 4 ? launch_tile<4, false, true>(rows, a, blocks, st) : launch_tile<3, false, true>(rows, a, blocks, st);
    if (fine) return P.bits == 4 ? launch_tile<4, true, false>(rows, a, blocks, st) : launch_tile<3, true, false>(rows, a, blocks, st);
    return P.bits == 4 ? launch_tile<4, false, false>(rows, a, blocks, st) : launch_tile<3, false, false>(rows, a, blocks, st);
}

}  // namespace gwq
