// What the matrix-core kernels share (device side): MFMA types, the order of the output tiles, LDS use and code of the
// epilogue that scatters a tile's stored neurons to their columns of y.
#pragma once
#include "srigl_internal.h"

namespace srigl {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kXcds = 8;                  // dies with an L2 of their own; workgroup id % 8 selects the die
#ifndef SRIGL_PANEL_N
#define SRIGL_PANEL_N 8
#endif
constexpr int kPanelN = SRIGL_PANEL_N;    // tile columns per panel of the tile order

static __device__ const uint4 g_zero16 = {0u, 0u, 0u, 0u};   // source of the pieces past the end of a row

// s_waitcnt immediate that waits for the vector-memory counter only (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

constexpr int kLgkm0 = 0xc07f;   // ... for the LDS counter only

// waits until at most N of this wavefront's vector-memory loads are in flight; nothing moves across it
template <int N> __device__ __forceinline__ void wait_loads() {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(N));
    asm volatile("" ::: "memory");
}

// A workgroup barrier that waits for this wavefront's LDS requests only (__syncthreads() also waits for every vector-memory
// load in flight, the stages requested ahead included).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

using gptr_t = const __attribute__((address_space(1))) void*;
using lptr_t = __attribute__((address_space(3))) void*;

// Workgroup -> tile.  Consecutive workgroup ids go round-robin to the 8 XCDs, each with its own L2.  The tiles are put
// in an order in which neighbours share operands (panels of kPanelN tile columns, row by row inside a panel), that order
// is cut into 8 equal runs, and XCD c walks run c: the 32 tiles it holds at a time cover about 4 x 8 tiles, which
// share their rows of x and of the weights through that L2, and every XCD gets the same number of tiles.
// false: padding of the last run.
__device__ __forceinline__ bool tile_of_workgroup(int id, int tiles_m, int tiles_n, int* tile_m, int* tile_n) {
    const int total = tiles_m * tiles_n;
    const int per_xcd = (total + kXcds - 1) / kXcds;
    const int q = (id % kXcds) * per_xcd + id / kXcds;
    if (id / kXcds >= per_xcd || q >= total) return false;
    const int full_panel = tiles_m * kPanelN;
    const int panel = q / full_panel, r = q - panel * full_panel;
    const int width = min(kPanelN, tiles_n - panel * kPanelN);
    *tile_m = r / width;
    *tile_n = panel * kPanelN + r - *tile_m * width;
    return true;
}

// ---- epilogue: a tile's sums to their columns of y ----
// The columns of y that the tile at stored neuron n0 writes: its stored neurons and the ablated ones in front of them (behind the
// last one too in the last tile) are one contiguous range.
struct TileColumns { int lo, hi, stored, base; };   // base: where the windows begin
// A tile's first column lies anywhere with ablated neurons.  The windows begin at its 128-byte line of y where y is large (line_run), all rows of y have lines there and the tile's
// rows take no more runs of `run` columns (a wavefront's stores of a row; 0: never) for it: 124 -> 6696 at batch 1270, whose rows begin anywhere, 20.9 us from the column and 22.2 from
// the line; 384 -> 5120 with 3072 stored at batch 288 in 64 x 64 tiles, whose runs are two lines long, 8.0 and 8.4.
__device__ __forceinline__ TileColumns tile_columns(int n0, int bn, const int32_t* active, int n_active, int d_out, int run) {
    const int cnt = min(bn, n_active - n0);
    if (!active) return {n0, n0 + cnt - 1, cnt, n0};   // (tiles are multiples of 32 columns)
    const int lo = max((n0 > 0) ? active[n0 - 1] + 1 : 0, 0), hi = min((n0 + cnt == n_active) ? d_out - 1 : active[n0 + cnt - 1], d_out - 1), line = lo & ~31;
    return {lo, hi, cnt, run && d_out % 32 == 0 && (hi - line) / run == (hi - lo) / run ? line : lo};
}

// `run` for tile_columns, of a launch that writes y and reads `inputs` bytes.  Windows from the line cost a tile's wavefronts the single stores of a first piece beside those of the
// last one, 1 us in tiles 128 to 192 wide and 2 in 256 wide ones whatever the size; from the column on, a line of y is written in two parts, which costs nothing
// while the caches hold it until both are there, and 1 to 8 us on larger results.  The line is taken from where it lost 2 % at most on 354 bf16 products and 300 condensed
// calls (y 8 to 112 MB, in one buffer or in six by turns): y and half of the inputs (of as much as y of them) 31.5 MB in products in tiles up to 192 wide and 52 in 256 wide ones, 46.5 and 77 in the condensed
// form.  The way taken is behind the better one by 0.3 % on average, always the line 3.1 %, never 4.  40 -> 10304 with 7463 stored at batch 1027 (42 MB) 17.8 us from the
// column, 20.1 from the line; 144 -> 13216 with 12680 at 1232 (65 MB) 29.0 and 23.8; 896 -> 12576, K = 179, with 8598 at 1763 (89 MB) 52.1 and 43.9.
__device__ __forceinline__ int line_run(int B, int d_out, long long inputs, int run, float from_mb) {
    const long long y = 4ll * B * d_out;
    return y + min(inputs, y) / 2 >= (long long)(from_mb * 1e6f) ? run : 0;
}

// LDS of the epilogue: one 32-row part of each wavefront row's tile at a time, at the rows' final columns (a window of COLS of them;
// most ranges fit one), and the tables: the stored neurons' places in the range, for the window's columns which neuron
// they are (-1: ablated) and their bias.
template <int BN, int WGM>
struct EpiLayout {
    static constexpr int COLS = BN >= 256 ? 512 : 256, ROWS = 32 * WGM, PITCH = COLS + 4;
    static constexpr int LINE_RUN = BN >= 256 ? 256 : (BN >= 128 ? 128 : 0);   // for line_run
    static constexpr size_t TILE_BYTES = (size_t)ROWS * PITCH * 4, TABLE_BYTES = (size_t)BN * 4 + (size_t)COLS * 8;
    static constexpr size_t BYTES = TILE_BYTES + TABLE_BYTES;
};

// Fills the tables for the window from column cc on (the places only with the first window).  No barrier: a stored neuron's thread
// marks the gap in front of it too.
template <int BN, int WGM, int NT>
__device__ __forceinline__ void fill_table(unsigned char* at, int cc, const TileColumns& c, int n0, const int32_t* active, const float* bias) {
    constexpr int COLS = EpiLayout<BN, WGM>::COLS;
    int* const place = reinterpret_cast<int*>(at);
    int* const table = place + BN;
    float* const tbias = reinterpret_cast<float*>(table + COLS);
    const int tid = threadIdx.x, wc = min(COLS, c.hi - cc + 1);
    for (int k = tid; k < wc; k += NT) tbias[k] = bias ? bias[cc + k] : 0.0f;
    for (int s = tid; s < BN; s += NT) {
        if (s >= c.stored) {
            place[s] = -1;
            continue;
        }
        const int col = active ? active[n0 + s] : n0 + s;
        const int prev = s == 0 ? c.lo - 1 : (active ? active[n0 + s - 1] : n0 + s - 1);
        place[s] = col >= c.lo && col <= c.hi ? col - c.base : -1;
        for (int k = max(prev + 1 - cc, 0); k < min(col - cc, wc); ++k) table[k] = -1;
        if (col >= cc && col - cc < wc) table[col - cc] = s;
        if (s == c.stored - 1)
            for (int k = max(col + 1 - cc, 0); k < wc; ++k) table[k] = -1;
    }
}

// Epilogue of a BM x BN tile at batch row m0, stored neuron n0, held as 32x32 blocks (accumulator register e of lane l is row
// 8*(e/4) + 4*(l/32) + e%4, column l%32).  Every wavefront puts 32 of its rows at a time into LDS, sums plus bias at their final columns,
// and the rows are then read and written 4 columns per lane and 4 rows at a time, ablated columns from registers.  No column
// of y is touched twice and none is left out.  (A 256 x 256 tile's epilogue took 28 us with one value at a time, each behind a read of
// a column table and one of the tile, and 10 with 4-way bank conflicts of lanes that gathered four columns each.)
// The LDS must be free (the caller has waited for its own loads into it and passed a barrier); have_table: the first window's tables
// stand at table_at already.  act: the activation applied to every value, written once, as a loop over values in LDS: inlined for each of
// a lane's 16 values it made the epilogue kilobytes of code that every workgroup fetched anew.
// With that and the float4 rows a 768 -> 3072 layer in 256 x 256 tiles went from 36.4 to 32.3 us, 4096 -> 16384 at batch 2048 from 297 to
// 279 in 128 x 128 tiles.  Narrow tiles put 2 or 4 rows into one LDS request (16 or 32 lanes each): with 64 lanes on a row 64 x 64
// tiles took 11.5 us instead of 9.4 on 768 -> 3072 at batch 128.
// The windows begin at a 128-byte line of y where that is of use (tile_columns, line_run; columns in front of the tile's own are left out): from a column inside of a
// line on every store of a kilobyte then began and ended in part of a line, which streaming stores do not put together: 4096 -> 16384 with
// 13108 stored at batch 2048 207 -> 201 us (condensed form 212 -> 208), 1024 -> 16384 with 8192 stored 73 -> 64.  (Plain stores: the first two 203 and 218.)
// SPOILED: the tile's rows with a sum that is not finite get their bits set in `spoiled` (BM of them, in LDS); what has been written for
// them is up to the caller to mend.
template <int BM, int BN, int WGM, int WGN, bool SPOILED, int TM, int TN>
__device__ __forceinline__ void store_tile(unsigned char* smem, unsigned char* table_at, bool have_table, const f32x16_t (&acc)[TM][TN],
                                           const TileColumns& cols, int m0, int n0, int B, const int32_t* active, const float* bias,
                                           int d_out, float* y, int act, uint32_t* spoiled) {
    using EL = EpiLayout<BN, WGM>;
    constexpr int NWAVES = WGM * WGN, WTM = BM / WGM, WTN = BN / WGN, PITCH = EL::PITCH;
    // lanes that share a row (four columns each), rows per LDS request, runs of columns of a window
    constexpr int LR = BN >= 256 ? 64 : (BN >= 128 ? 32 : 16), RPI = 64 / LR, RUN = 4 * LR, RUNS = EL::COLS / RUN;
    typedef float float4_t __attribute__((ext_vector_type(4)));
    typedef float float4_at4_t __attribute__((ext_vector_type(4), aligned(4)));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv / WGN, wn = wv % WGN;
    float* const tile = reinterpret_cast<float*>(smem);
    const int* const place = reinterpret_cast<const int*>(table_at);
    const int* const table = place + BN;
    float* const tbias = reinterpret_cast<float*>(table_at + (size_t)(BN + EL::COLS) * 4);
    if (!have_table) {
        fill_table<BN, WGM, NWAVES * 64>(table_at, cols.base, cols, n0, active, bias);
        __syncthreads();
    }
    for (int cc = cols.base; cc <= cols.hi; cc += EL::COLS) {
        const int wc = min(EL::COLS, cols.hi - cc + 1);
        const int head = max(cols.lo - cc, 0);   // columns of the first line that are the tile's before
        if (cc != cols.base) {
            __syncthreads();   // the previous window is done with the tables
            fill_table<BN, WGM, NWAVES * 64>(table_at, cc, cols, n0, active, bias);
            __syncthreads();
        }
        if (act != SRIGL_ACT_NONE) {
            __syncthreads();
            for (int k = tid; k < wc; k += NWAVES * 64)
                if (k >= head && table[k] < 0) tbias[k] = apply_act(tbias[k], act);
            __syncthreads();
        }
        int at[TN];        // this lane's columns in the window
        float badd[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int q = place[wn * WTN + j * 32 + (lane & 31)];
            at[j] = q < 0 ? -1 : q - (cc - cols.base);
            if (at[j] >= wc) at[j] = -1;
            badd[j] = tbias[max(at[j], 0)];
        }
        float flat[RUNS][4];
        int gaps = 0;      // bit 4 run + j: an ablated column, or none of the window
#pragma unroll
        for (int run = 0; run < RUNS; ++run)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = RUN * run + 4 * (lane % LR) + j, in = min(k, wc - 1);
                flat[run][j] = tbias[in];
                if (k < head || k >= wc || table[in] < 0) gaps |= 1 << (4 * run + j);
            }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (i > 0 || cc != cols.base) __syncthreads();   // the rows before have been read
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (at[j] >= 0) {
                    float* const t = tile + (wm * 32 + 4 * (lane >> 5)) * PITCH + at[j];
#pragma unroll
                    for (int e = 0; e < 16; ++e) t[(8 * (e >> 2) + (e & 3)) * PITCH] = acc[i][j][e] + badd[j];
                }
            }
            __syncthreads();
            for (int r0 = 4 * RPI * wv; r0 < EL::ROWS; r0 += 4 * RPI * NWAVES) {   // 4 RPI rows of one wavefront row
                const int row = r0 + lane / LR, m = m0 + (r0 >> 5) * WTM + i * 32 + (row & 31);   // this lane's rows: every RPI-th from here
                if (m - lane / LR >= B) continue;
#pragma unroll
                for (int run = 0; run < RUNS; ++run) {
                    if (RUN * run >= wc) break;
                    const int k0 = RUN * run + 4 * (lane % LR);
                    float* const t0 = tile + row * PITCH + k0;
                    float4_t v[4];
                    bool finite = true;
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4_t*>(t0 + u * RPI * PITCH);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            if ((gaps >> (4 * run + j)) & 1) v[u][j] = 0.0f;
                            else if (SPOILED) finite = finite && fabsf(v[u][j]) <= 3.4028234e38f;
                        }
                    if (SPOILED && __any(!finite)) {
#pragma unroll 1
                        for (int q = 0; q < 16; ++q) {
                            const int k = k0 + (q & 3), mq = m + (q >> 2) * RPI, r = mq - m0;
                            if (k >= head && k < wc && table[k] >= 0 && mq < B && !(fabsf(t0[(q >> 2) * RPI * PITCH + (q & 3)]) <= 3.4028234e38f))
                                atomicOr(&spoiled[r >> 5], 1u << (r & 31));
                        }
                    }
                    if (act != SRIGL_ACT_NONE) {
#pragma unroll 1
                        for (int q = 0; q < 16; ++q) {
                            const int k = k0 + (q & 3), mq = m + (q >> 2) * RPI;
                            float* const at_q = t0 + (q >> 2) * RPI * PITCH + (q & 3);
                            if (k >= head && k < wc && table[k] >= 0 && mq < B) *at_q = apply_act(*at_q, act);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4_t*>(t0 + u * RPI * PITCH);
                    }
                    float* const yr = y + (size_t)m * d_out + cc + k0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) v[u][j] = (gaps >> (4 * run + j)) & 1 ? flat[run][j] : v[u][j];
                        float* const yu = yr + (size_t)(u * RPI) * d_out;
                        if (m + u * RPI < B) {
                            if (k0 >= head && k0 + 4 <= wc) {
                                __builtin_nontemporal_store(v[u], reinterpret_cast<float4_at4_t*>(yu));
                            } else {
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    if (k0 + j >= head && k0 + j < wc) yu[j] = v[u][j];
                            }
                        }
                    }
                }
            }
        }
    }
}

}  // namespace srigl
