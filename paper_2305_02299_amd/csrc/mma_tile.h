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

// LDS use of the epilogue: an fp32 tile (pitch BN + 4) of all BM rows when that fits, else of the rows of one wavefront row at
// a time, and the column table with its bias values.
constexpr int kTableCols = 1024;   // columns of y per pass over the tile
constexpr size_t kTableBytes = (size_t)kTableCols * 8;
template <int BM, int BN, int WGM>
struct EpiLayout {
    static constexpr int PITCH = BN + 4;
    static constexpr int PHASES = ((size_t)BM * PITCH * 4 + kTableBytes <= kLdsMax) ? 1 : WGM;
    static constexpr size_t TILE_BYTES = (size_t)(BM / PHASES) * PITCH * 4;
    static constexpr size_t BYTES = TILE_BYTES + kTableBytes;
};

// The columns of y that the tile at stored neuron n0 writes: its stored neurons and the ablated ones in front of them (behind the
// last one too in the last tile) are one contiguous range.
struct TileColumns { int lo, hi, stored; };
__device__ __forceinline__ TileColumns tile_columns(int n0, int bn, const int32_t* active, int n_active, int d_out) {
    const int cnt = min(bn, n_active - n0);
    if (!active) return {n0, n0 + cnt - 1, cnt};
    return {max((n0 > 0) ? active[n0 - 1] + 1 : 0, 0), min((n0 + cnt == n_active) ? d_out - 1 : active[n0 + cnt - 1], d_out - 1), cnt};
}

// The table of columns cc .. cc + kTableCols - 1 of that range: table[k] = the stored neuron of the tile that column cc + k is, or -1
// (the column is its bias); bias values behind it.  A stored neuron's thread marks the gap in front of it too.  No barrier.
template <int NT>
__device__ __forceinline__ void fill_table(unsigned char* at, int cc, const TileColumns& c, int n0, const int32_t* active, const float* bias) {
    int* table = reinterpret_cast<int*>(at);
    float* tbias = reinterpret_cast<float*>(at + kTableCols * 4);
    const int tid = threadIdx.x, wc = min(kTableCols, c.hi - cc + 1);
    for (int k = tid; k < wc; k += NT) tbias[k] = bias ? bias[cc + k] : 0.0f;
    for (int s = tid; s < c.stored; s += NT) {
        const int col = active ? active[n0 + s] : n0 + s;
        const int prev = s == 0 ? c.lo - 1 : (active ? active[n0 + s - 1] : n0 + s - 1);
        for (int k = max(prev + 1 - cc, 0); k < min(col - cc, wc); ++k) table[k] = -1;
        if (col >= cc && col - cc < wc) table[col - cc] = s;
        if (s == c.stored - 1)
            for (int k = max(col + 1 - cc, 0); k < wc; ++k) table[k] = -1;
    }
}

// Epilogue of a BM x BN tile at batch row m0, stored neuron n0, held as 32x32 blocks (accumulator register e of lane l is row
// 8*(e/4) + 4*(l/32) + e%4, column l%32).  The tile's columns of y are written row by row with neighbouring lanes on neighbouring
// columns: the table says which stored neuron of the tile a column is, and the accumulators pass through an LDS tile at smem.
// No column of y is touched twice and none is left out.  The LDS must be free (the caller has waited for its own loads into it and
// passed a barrier); have_table: the first columns' table stands there already.
// finish.stored(sum, bias) and finish.ablated(bias) give the values to write; finish.repaired(m, s) the sum to use where one is not
// finite (Finish::kRepairs).
template <int BM, int BN, int WGM, int WGN, int TM, int TN, typename Finish>
__device__ __forceinline__ void store_tile(unsigned char* smem, unsigned char* table_at, bool have_table, const f32x16_t (&acc)[TM][TN],
                                           const TileColumns& cols, int m0, int n0, int B, const int32_t* active, const float* bias,
                                           int d_out, float* y, const Finish& finish) {
    using EL = EpiLayout<BM, BN, WGM>;
    constexpr int NWAVES = WGM * WGN, NT = NWAVES * 64, WTM = BM / WGM, WTN = BN / WGN;
    constexpr int PITCH = EL::PITCH, EPH = EL::PHASES, PROWS = BM / EPH, WPP = WGM / EPH;
    // A lane keeps NJ neighbouring columns of a run of 64 NJ in registers and takes NI rows at a time: 16 outputs' LDS reads in
    // flight, then NI stores of NJ values.  (One value at a time, each behind a read of the table and then one of the tile, a
    // 256 x 256 tile's epilogue took 28 us; with 4-byte stores 12.)
    constexpr int NJ = BN >= 256 ? 4 : BN / 64, NI = 16 / NJ;
    typedef float Run __attribute__((ext_vector_type(NJ == 1 ? 2 : NJ), aligned(4)));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv / WGN, wn = wv % WGN;
    float* tile = reinterpret_cast<float*>(smem);                         // [PROWS][PITCH]
    const int* table = reinterpret_cast<const int*>(table_at);
    const float* tbias = reinterpret_cast<const float*>(table_at + kTableCols * 4);
    for (int cc = cols.lo; cc <= cols.hi; cc += kTableCols) {
        const int wc = min(kTableCols, cols.hi - cc + 1);
        if (cc != cols.lo) __syncthreads();   // the previous pass is done with the table
        if (cc != cols.lo || !have_table) fill_table<NT>(table_at, cc, cols, n0, active, bias);
#pragma unroll
        for (int ph = 0; ph < EPH; ++ph) {
            if (ph > 0) __syncthreads();   // tile free again
            if (wm / WPP == ph) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            tile[((wm % WPP) * WTM + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * PITCH + wn * WTN + j * 32 + (lane & 31)] =
                                acc[i][j][e];
            }
            __syncthreads();   // tile, table and bias values complete
            const int rows = min(PROWS, B - (m0 + ph * PROWS));
            for (int kb = 0; kb < wc; kb += 64 * NJ) {
                const int k0 = kb + NJ * lane;   // this lane's first column
                int tix[NJ];
                float bv[NJ], flat[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int k = min(k0 + j, wc - 1);
                    tix[j] = table[k];
                    bv[j] = tbias[k];
                    flat[j] = finish.ablated(bv[j]);
                }
                for (int r = NI * wv; r < rows; r += NI * NWAVES) {
                    float v[NI][NJ];
                    bool finite = true;
#pragma unroll
                    for (int i = 0; i < NI; ++i)
#pragma unroll
                        for (int j = 0; j < NJ; ++j) {
                            v[i][j] = tile[min(r + i, PROWS - 1) * PITCH + max(tix[j], 0)];
                            if (Finish::kRepairs) finite = finite && fabsf(v[i][j]) <= 3.4028234e38f;
                        }
                    if (Finish::kRepairs && __any(!finite)) {
#pragma unroll 1
                        for (int e = 0; e < NI * NJ; ++e) {
                            const int row = r + e / NJ, t = table[min(k0 + e % NJ, wc - 1)];
                            if (t >= 0 && row < rows && !(fabsf(tile[row * PITCH + t]) <= 3.4028234e38f))
                                tile[row * PITCH + t] = finish.repaired(m0 + ph * PROWS + row, n0 + t);
                        }
#pragma unroll
                        for (int i = 0; i < NI; ++i)
#pragma unroll
                            for (int j = 0; j < NJ; ++j) v[i][j] = tile[min(r + i, PROWS - 1) * PITCH + max(tix[j], 0)];
                    }
                    float* yr = y + (size_t)(m0 + ph * PROWS + r) * d_out + cc + k0;
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        if (r + i >= rows) break;
                        Run run;
#pragma unroll
                        for (int j = 0; j < NJ; ++j) run[j] = tix[j] >= 0 ? finish.stored(v[i][j], bv[j]) : flat[j];
                        if (k0 + NJ <= wc) {
                            if constexpr (NJ == 1) __builtin_nontemporal_store(run[0], yr + (size_t)i * d_out);
                            else __builtin_nontemporal_store(run, reinterpret_cast<Run*>(yr + (size_t)i * d_out));
                        } else {
#pragma unroll
                            for (int j = 0; j + 1 < NJ; ++j)
                                if (k0 + j < wc) yr[(size_t)i * d_out + j] = run[j];
                        }
                    }
                }
            }
        }
    }
}

}  // namespace srigl
