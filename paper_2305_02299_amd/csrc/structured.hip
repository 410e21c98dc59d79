// Structured-only representation (gfx950): the stored neurons of a layer trained with SRigL keep dense rows
// (ablated neurons removed, fine-grained sparsity not exploited; Sec. 4.4, Fig. 4 and App. H of arXiv
// 2305.02299), and the forward pass is a dense product on the matrix cores,
//     y[b][active[s]] = bias[active[s]] + sum_j Wd[s][j] * x[b][j].
//
// The product is an "NT" GEMM: both operands are K-contiguous (x[b][:], Wd[s][:]).  A workgroup owns a BM x BN
// output tile and walks d_in in stages of SLAB = 128 or 64 bytes per row.  Stages travel from global memory straight
// into a ring of NS LDS stages (global_load_lds_dwordx4: every lane brings 16 bytes, a wavefront fills 1 KB = 1024 / SLAB
// rows of the stage), up to NS - 1 stages ahead of the one being multiplied; one barrier per stage.
// LDS layout of a stage: row r at r * SLAB bytes; its 16-byte piece q sits in slot q ^ ((r >> 1) & 7) for SLAB = 128 and
// q ^ ((r >> 2) & 3) for SLAB = 64: rows that share their banks get different slots, so the 16-byte reads of consecutive
// rows at one q spread over all banks (measured: same rate as a padded pitch, which a direct load cannot produce).  The
// swizzle is applied on the global side: the lane that fills slot s of row r fetches piece s ^ swizzle(r).
// A wavefront owns a (BM/WGM) x (BN/WGN) part of the tile as 32x32 MFMA blocks:
//   bf16: v_mfma_f32_32x32x16_bf16, lane l holds row l%32 and the 8 consecutive k of piece l/32 of the 32-byte step;
//   fp32: v_mfma_f32_32x32x2_f32, lane l holds row l%32, k = l/32; the lane's 16-byte piece carries 4 k, used by 4
//         successive MFMAs (both operands use the same k-to-slot map, so the sum runs over matching k).
// Result block layout: accumulator register e of lane l is row 8*(e/4) + 4*(l/32) + e%4, column l%32.
#include "mma_tile.h"
#include <algorithm>
#include <cmath>

namespace srigl {

constexpr int kSlabBytes = 128;   // bytes of K per row and slab = LDS row pitch

// zero fill, then scatter: two launches so that no ordering inside a wavefront is relied on
__global__ __launch_bounds__(256) void k_fill_zero16(uint4* __restrict__ p, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const uint4 z = {0u, 0u, 0u, 0u};
    for (; i < n16; i += stride) p[i] = z;
}
__global__ __launch_bounds__(256) void k_fill_zero_bytes(unsigned char* __restrict__ p, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0;
}
template <typename T>
__global__ __launch_bounds__(256) void k_scatter_rows(const T* __restrict__ W_c, const int32_t* __restrict__ idx, long long n_terms,
                                                      int K, int d_in, T* __restrict__ Wd) {
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (; t < n_terms; t += stride) {
        const long long s = t / K;
        const int j = idx[t];
        if (j >= 0 && j < d_in) Wd[s * d_in + j] = W_c[t];
    }
}

// Columns that are not stored get their bias (used when no neuron is stored at all; otherwise the product kernel's epilogue
// writes them).  A workgroup takes 256 consecutive columns and kFillRows rows: every thread
// looks its column up in the ascending active list, the ablated ones are gathered into a list in LDS, and the threads then
// walk (row, listed column) pairs so that neighbouring lanes write neighbouring ablated columns of one row.
constexpr int kFillRows = 128;
__global__ __launch_bounds__(256) void k_fill_ablated(const int32_t* __restrict__ active, int n_active, const float* __restrict__ bias,
                                                      int B, int d_out, float* __restrict__ y) {
    __shared__ int list[256];
    __shared__ float list_bias[256];
    __shared__ int wave_count[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int c = blockIdx.x * 256 + tid;
    bool ablated = c < d_out;
    if (ablated && n_active > 0) {
        int lo = 0, hi = n_active;   // first position whose entry is >= c
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (active[mid] < c) lo = mid + 1; else hi = mid;
        }
        ablated = !(lo < n_active && active[lo] == c);
    }
    const unsigned long long vote = __ballot(ablated);
    const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(vote >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)vote, 0));
    if (lane == 0) wave_count[wv] = __popcll(vote);
    __syncthreads();
    int base = 0, n_list = 0;
    for (int w = 0; w < 4; ++w) {
        if (w < wv) base += wave_count[w];
        n_list += wave_count[w];
    }
    if (ablated) {
        list[base + before] = c;
        list_bias[base + before] = bias ? bias[c] : 0.0f;
    }
    __syncthreads();
    if (n_list == 0) return;
    const int r0 = blockIdx.y * kFillRows;
    const int rows = min(kFillRows, B - r0);
    for (int idx = tid; idx < rows * n_list; idx += 256) {
        const int r = idx / n_list, k = idx - r * n_list;
        y[(size_t)(r0 + r) * d_out + list[k]] = list_bias[k];
    }
}

// y[r][c] = bias[c] + sum over the parts z (ascending) of part[z][r][s] when column c is stored neuron s, else bias[c].
// One thread per (row r, slot s <= n_active): slot s writes its neuron's column and the ablated columns between the previous
// stored neuron and its own; slot n_active writes the ablated columns after the last stored neuron.  The parts' values are
// requested together (up to kMaxSplits independent loads), so a thread waits for memory twice: the list, then the values.
constexpr int kMaxSplits = 16;
__global__ __launch_bounds__(256) void k_sum_parts(const float* __restrict__ part, int splits, int B, int n_active,
                                                   const int32_t* __restrict__ active, const float* __restrict__ bias, int d_out,
                                                   float* __restrict__ y) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (s > n_active) return;
    float v[kMaxSplits];
    const size_t plane = (size_t)B * n_active;
    const float* p = part + (size_t)r * n_active + (s < n_active ? s : 0);
#pragma unroll
    for (int z = 0; z < kMaxSplits; ++z) v[z] = (z < splits && s < n_active) ? p[z * plane] : 0.0f;
    int lo, hi;   // ablated columns lo .. hi - 1, then the stored neuron's column hi (none for the last slot)
    if (active == nullptr) {
        lo = hi = s;   // every neuron stored: n_active == d_out
    } else {
        lo = s > 0 ? active[s - 1] + 1 : 0;
        hi = s < n_active ? active[s] : d_out;
    }
    float* yr = y + (size_t)r * d_out;
    for (int c = lo; c < hi; ++c) __builtin_nontemporal_store(bias ? bias[c] : 0.0f, &yr[c]);
    if (s < n_active) {
        float sum = 0.0f;
#pragma unroll
        for (int z = 0; z < kMaxSplits; ++z) sum += v[z];   // parts past `splits` hold zeros
        __builtin_nontemporal_store(sum + (bias ? bias[hi] : 0.0f), &yr[hi]);
    }
}

template <typename T> struct Frag;
template <> struct Frag<uint16_t> { using type = bf16x8_t; };
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <> struct Frag<float> { using type = f32x4_t; };

__device__ __forceinline__ void mma_block(f32x16_t& acc, const bf16x8_t& a, const bf16x8_t& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma_block(f32x16_t& acc, const f32x4_t& a, const f32x4_t& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
}

// BM x BN output tile per workgroup of WGM x WGN wavefronts; NS >= 2 LDS stages of SLAB (128 or 64) bytes of K per row.
//
// Schedule of one stage h (KSTEPS = SLAB / 32 MFMA steps): the fragments of step kk + 1 are requested between the MFMAs of
// step kk, the first ones before the first of them; before the last step the wavefront waits until its own loads of stage h + 1 have
// landed and its own reads of stage h have returned, meets the others at the barrier (after which stage h + 1 is complete and the slot of
// stage h is free), and requests the first fragments of stage h + 1 and, between the MFMAs of this step and of the next stage's first
// one, the pieces of stage h + NS.  The MFMAs right after the barrier have their operands in registers already, so the matrix pipe does
// not drain at the barrier.
// What bounds it: the matrix units' rate at the clock that the card holds (4096 -> 16384 at batch 2048: 1.4 PFLOP/s, 1.2 to 1.75 for a
// library product on the same cards) and the fp32 result.  Everything of a step in one block, and loaded where the
// compiler wanted it, just before its use: the matrix pipe was busy 42 % of the time, and in 256 x 256 tiles two stages of 128 bytes took
// longer than five of 64.  Before -> now (bf16, us): 16384 stored at batch 2048, d_in 4096, 240 -> 215; 5023 at 1696, 1136, 53 -> 36; 13569 at
// 1816, 1040, 128 -> 78; fp32 538 at 256, 3072, in one part 86 -> 59; 64 x 64 tiles on small products 5.9 -> 5.8.
template <typename T, int BM, int BN, int WGM, int WGN, int NS, int SLAB, bool RAGGED>
__global__ __launch_bounds__(WGM * WGN * 64) void k_structured_gemm(const T* __restrict__ x, int B, int d_in, const T* __restrict__ Wd,
                                                                   const int32_t* __restrict__ active, int n_active,
                                                                   const float* __restrict__ bias, int d_out, float* __restrict__ y,
                                                                   int splits, float* __restrict__ part) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];   // [NS][BM + BN rows][SLAB bytes]
    using F = typename Frag<T>::type;
    constexpr int NWAVES = WGM * WGN;
    constexpr int EPS = SLAB / (int)sizeof(T);         // elements of K per stage
    constexpr int EPP = 16 / (int)sizeof(T);           // elements per 16-byte piece
    constexpr int PIECES = SLAB / 16;                  // pieces per row and stage (8 or 4)
    constexpr int KSTEPS = SLAB / 32;                  // MFMA steps per stage (two pieces each)
    constexpr int RPL = 1024 / SLAB;                   // rows one wavefront-wide direct load fills (8 or 16)
    constexpr int SWZ_SHIFT = (SLAB == 128) ? 1 : 2;   // rows 2^shift apart share their banks
    constexpr int WTM = BM / WGM, WTN = BN / WGN;      // wavefront tile
    constexpr int TM = WTM / 32, TN = WTN / 32;
    constexpr int ROWS = BM + BN;
    constexpr int STAGE = ROWS * SLAB;
    constexpr int PASSES = ROWS / RPL / NWAVES;        // 1 KB direct loads per wavefront and stage
    static_assert(SLAB == 128 || SLAB == 64, "stage width");
    static_assert(ROWS % (RPL * NWAVES) == 0 && WTM % 32 == 0 && WTN % 32 == 0 && NS >= 2, "tile shape");
    static_assert((NS - 1) * PASSES <= 63, "vmcnt range");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront index as a scalar
    const int wm = wv / WGN, wn = wv % WGN;
    int tile_m, tile_n;
    if (!tile_of_workgroup(blockIdx.x, (B + BM - 1) / BM, (n_active + BN - 1) / BN, &tile_m, &tile_n)) return;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    // loader: pass p of wavefront wv fills rows RPL * (p * NWAVES + wv) .. + RPL - 1; lane -> (row + lane / PIECES, slot lane % PIECES).
    // The first XP passes are rows of x, the others rows of Wd; a lane keeps one 32-bit byte offset per pass from the tile's
    // first row, the stage advance is scalar.  Rows past the matrix re-read its last row (their results are never stored).
    constexpr int XP = BM / RPL / NWAVES;
    static_assert((BM / RPL) % NWAVES == 0, "a pass is all x rows or all Wd rows");
    uint32_t voff[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int row = RPL * (p * NWAVES + wv) + lane / PIECES;
        const int piece = (lane % PIECES) ^ ((row >> SWZ_SHIFT) & (PIECES - 1));
        const int r = (p < XP) ? min(row, B - 1 - m0) : min(row - BM, n_active - 1 - n0);
        voff[p] = (uint32_t)r * (uint32_t)(d_in * (int)sizeof(T)) + piece * 16;
    }
    const unsigned char* xbase = reinterpret_cast<const unsigned char*>(x + (size_t)m0 * d_in);
    const unsigned char* wbase = reinterpret_cast<const unsigned char*>(Wd + (size_t)n0 * d_in);
    // Part blockIdx.y of d_in (splits parts of whole stages, sizes one stage apart at most): stages h_first .. h_first + n_st - 1
    // of the row.  With one part the tile's sums are complete and go to y; with several they go to part[blockIdx.y][B][n_active].
    const int n_st_row = (d_in + EPS - 1) / EPS;
    // (32 bits hold it: at most kMaxSplits parts of 2^26 stages; 64-bit divisions were a third of the instructions before the first request)
    const unsigned n_parts = (unsigned)splits, part_no = blockIdx.y;
    const int h_first = n_parts == 1 ? 0 : (int)(part_no * (unsigned)n_st_row / n_parts);
    const int n_st = n_parts == 1 ? n_st_row : (int)((part_no + 1) * (unsigned)n_st_row / n_parts) - h_first;
    // RAGGED: d_in is not a multiple of EPS; the pieces of the last stage that lie past the end of the rows come from zeros.
    // A stage index past the end re-issues the last stage (into a slot nobody reads again): the loop body has no branches
    // and the number of loads in flight at each wait is fixed.
    auto issue_piece = [&](int p, int h_unclamped, int slot) {   // slot: byte offset of the stage's place in the ring
        const int h = h_first + min(h_unclamped, n_st - 1);
        const unsigned char* const rows = ((p < XP) ? xbase : wbase) + (size_t)h * SLAB;
        uint32_t off = voff[p];
        asm("" : "+v"(off));   // (a lane offset from a scalar base: seen to be 32 bits only next to the load)
        const unsigned char* g = rows + off;
        if (RAGGED) {
            const int row = RPL * (p * NWAVES + wv) + lane / PIECES;
            const int piece = (lane % PIECES) ^ ((row >> SWZ_SHIFT) & (PIECES - 1));
            if (h * EPS + piece * EPP >= d_in) g = reinterpret_cast<const unsigned char*>(&g_zero16);   // a piece is whole or absent
        }
        __builtin_amdgcn_global_load_lds((gptr_t)g, (lptr_t)(smem + slot + 1024 * wv + 1024 * NWAVES * p), 16, 0, 0);
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    constexpr int EARLY = TM * TN == 1 ? PASSES : PASSES / 2;   // pieces of a stage that are requested right behind the barrier, the others a step later
    if (n_st > 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int p = 0; p < (s < NS - 1 ? PASSES : EARLY); ++p) issue_piece(p, s, s * STAGE);
    }

    // reader: row l%32 of a block, piece 2*kk + l/32; the swizzle term only depends on the lane (block rows start at multiples of 32)
    const int swz = ((lane & 31) >> SWZ_SHIFT) & (PIECES - 1);
    int frag_off[KSTEPS];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) frag_off[kk] = (lane & 31) * SLAB + (((2 * kk + (lane >> 5)) ^ swz) * 16);

    F a[2][TM], b[2][TN];
    // fragment f of a step, in the order the products take them: a[0], the b's, the other a's
    auto read_frag = [&](int f, int slot, int kk, int set) {
        const unsigned char* buf = smem + slot + frag_off[kk];
        if (f >= 1 && f <= TN) b[set][f - 1] = *reinterpret_cast<const F*>(buf + (BM + wn * WTN + (f - 1) * 32) * SLAB);
        else a[set][f ? f - TN : 0] = *reinterpret_cast<const F*>(buf + (wm * WTM + (f ? f - TN : 0) * 32) * SLAB);
    };

    if (n_st > 0) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * PASSES + EARLY));
        __syncthreads();
#pragma unroll
        for (int f = 0; f < TM + TN; ++f) read_frag(f, 0, 0, 0);
        // (opaque: a value that is a load here and in the loop is loaded where it is used, behind everything that was to hide it)
#pragma unroll
        for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(a[0][i]));
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(b[0][j]));
    }
    int slot = 0, before = (NS - 1) * STAGE;   // of stage h and of the one before it
    for (int h = 0; h < n_st; ++h) {
        const int after = slot == (NS - 1) * STAGE ? 0 : slot + STAGE;
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            constexpr int N_MMA = TM * TN, N_FRAG = TM + TN, N_READ = N_MMA > N_FRAG ? N_FRAG : (N_MMA + 1) / 2;
            const bool last = kk + 1 == KSTEPS;
            if (last) {
                __builtin_amdgcn_s_waitcnt(kLgkm0);
                // stages up to h + NS - 1 are on their way; stage h + 1 must have landed.  Every fragment of stage h is in
                // registers by now, so its slot is refilled right away.
                __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * PASSES));
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            // The next step's fragments and this step's share of the stage requested ahead go out between the multiplications
#pragma unroll
            for (int m = 0; m < N_MMA; ++m) {
#pragma unroll
                for (int f = m * N_FRAG / N_READ; f < (m + 1) * N_FRAG / N_READ && f < N_FRAG; ++f)
                    read_frag(f, last ? after : slot, last ? 0 : kk + 1, (kk + 1) & 1);
                if (N_MMA > 1) mma_block(acc[m / TN][m % TN], a[kk & 1][m / TN], b[kk & 1][m % TN]);
                if (last) {
#pragma unroll
                    for (int p = m * EARLY / N_MMA; p < (m + 1) * EARLY / N_MMA; ++p) issue_piece(p, h + NS, slot);
                }
                if (kk == 0) {
#pragma unroll
                    for (int p = EARLY + m * (PASSES - EARLY) / N_MMA; p < EARLY + (m + 1) * (PASSES - EARLY) / N_MMA; ++p) issue_piece(p, h + NS - 1, before);
                }
                if (N_MMA == 1) mma_block(acc[0][0], a[kk & 1][0], b[kk & 1][0]);   // (it waits for the one before: requests first)
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        before = slot;
        slot = after;
    }

    // One part of several: the partial sums of the tile, stored neuron s in column s of this part's [B][n_active] array
    // (bias, ablated columns and the sum over the parts belong to k_sum_parts).
    if (part != nullptr) {
        float* pz = part + (size_t)blockIdx.y * B * n_active;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + wn * WTN + j * 32 + (lane & 31);
            if (col >= n_active) continue;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = m0 + wm * WTM + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                    if (m < B) pz[(size_t)m * n_active + col] = acc[i][j][e];
                }
            }
        }
        return;
    }

    // Epilogue of 64 x 64 tiles without an active list: stored neuron s is column s; every lane writes its accumulators where they belong
    // (32 neighbouring lanes cover 128 contiguous bytes of a row).  Larger tiles go through the LDS below here too, which writes whole
    // rows of the tile: 13108 columns at batch 2048, d_in 4096, in 256 x 256 tiles 221 us -> 180, 9000 at 1024, d_in 2048, 55 -> 47, 3000 at
    // 2048, d_in 1024, in 256 x 128 tiles 24 -> 20; in 64 x 64 tiles 28 -> 29.
    if (TM * TN == 1 && active == nullptr) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + wn * WTN + j * 32 + (lane & 31);
            if (col >= n_active) continue;
            const float bv = bias ? bias[col] : 0.0f;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = m0 + wm * WTM + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                    if (m < B) __builtin_nontemporal_store(acc[i][j][e] + bv, &y[(size_t)m * d_out + col]);   // y is not read again here
                }
            }
        }
        return;
    }

    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // the re-issued last stages may still be landing in the ring
    __syncthreads();
    const int run = line_run(B, d_out, ((long long)B + n_active) * d_in * (int)sizeof(T), EpiLayout<BN, WGM>::LINE_RUN, BN >= 256 ? 52.0f : 31.5f);
    store_tile<BM, BN, WGM, WGN, false>(smem, smem + EpiLayout<BN, WGM>::TILE_BYTES, false, acc, tile_columns(n0, BN, active, n_active, d_out, run), m0, n0, B,
                                    active, bias, d_out, y, SRIGL_ACT_NONE, nullptr);
}

template <typename T, int BM, int BN, int WGM, int WGN, int NS, int SLAB, bool RAGGED>
static srigl_status launch_gemm_r(const void* x, int B, int d_in, const void* Wd, const int32_t* active, int n_active, const float* bias,
                                int d_out, float* y, int splits, float* part, hipStream_t st) {
    auto kern = k_structured_gemm<T, BM, BN, WGM, WGN, NS, SLAB, RAGGED>;
    constexpr size_t ring = (size_t)NS * (BM + BN) * SLAB, epi = EpiLayout<BN, WGM>::BYTES;
    constexpr size_t lds = ring > epi ? ring : epi;
    static_assert(lds <= kLdsMax, "LDS");
    static LdsLimit lds_limit;
    if (lds_limit.ensure(kern, lds) != SRIGL_OK) return SRIGL_ERR_HIP;
    const long long tiles_m = (B + BM - 1) / BM, tiles_n = (n_active + BN - 1) / BN;
    const long long n_wg = ((tiles_m * tiles_n + kXcds - 1) / kXcds) * kXcds;   // 8 equal runs of tiles, one per XCD
    if (n_wg > 0x7fffffffLL) return SRIGL_ERR_UNSUPPORTED;
    // every part holds at least one stage
    if (splits < 1 || splits > kMaxSplits || (splits > 1 && (part == nullptr || splits > (d_in * (int)sizeof(T) + SLAB - 1) / SLAB)))
        return SRIGL_ERR_INVALID_ARG;
    if (splits > 1 && B > 65535) return SRIGL_ERR_UNSUPPORTED;   // the sum's grid has one row of workgroups per batch row
    const dim3 grid((unsigned)n_wg, (unsigned)splits);
    // a lane addresses its rows with 32-bit byte offsets from the tile's first row
    if ((long long)(BM > BN ? BM : BN) * d_in * (long long)sizeof(T) >= (1ll << 31)) return SRIGL_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kern, grid, dim3(WGM * WGN * 64), lds, st, (const T*)x, B, d_in, (const T*)Wd, active, n_active, bias, d_out, y,
                       splits, splits > 1 ? part : nullptr);
    if (splits > 1) {
        hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)(n_active / 256 + 1), (unsigned)B), dim3(256), 0, st, part, splits, B, n_active, active,
                           bias, d_out, y);
    }
    return hip_ok(hipGetLastError());
}

template <typename T, int BM, int BN, int WGM, int WGN, int NS, int SLAB>
static srigl_status launch_gemm(const void* x, int B, int d_in, const void* Wd, const int32_t* active, int n_active, const float* bias,
                                int d_out, float* y, int splits, float* part, hipStream_t st) {
    if (d_in % (SLAB / (int)sizeof(T)) == 0)
        return launch_gemm_r<T, BM, BN, WGM, WGN, NS, SLAB, false>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
    return launch_gemm_r<T, BM, BN, WGM, WGN, NS, SLAB, true>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
}

// Tile choice and time estimate: a workgroup needs about ns_per_k nanoseconds per element of d_in for its tile (measured on
// MI355X with every compute unit busy), and the tiles take ceil(tiles / 256) rounds over the 256 compute units.  fp32, and either type
// where the caller forces the parts of d_in.
struct TileModel { srigl_gemm_tile tile; int bm, bn; float ns_per_k_bf16, ns_per_k_f32; };
static const TileModel kTileModels[] = {
    {SRIGL_TILE_256x256_H, 256, 256, 28.0f, 233.0f},
    {SRIGL_TILE_256x128, 256, 128, 18.0f, 125.0f},
    {SRIGL_TILE_128x128, 128, 128, 12.0f, 70.0f},
    {SRIGL_TILE_64x64, 64, 64, 3.8f, 19.0f},
};
static srigl_gemm_tile choose_tile(int B, int n_active, bool f32) {
    srigl_gemm_tile best = SRIGL_TILE_64x64;
    double best_cost = 0.0;
    for (const TileModel& m : kTileModels) {
        const long long tiles = (long long)((B + m.bm - 1) / m.bm) * ((n_active + m.bn - 1) / m.bn);
        const long long rounds = (tiles + 255) / 256;
        const double cost = (double)rounds * (f32 ? m.ns_per_k_f32 : m.ns_per_k_bf16);
        if (best_cost == 0.0 || cost < best_cost) { best_cost = cost; best = m.tile; }
    }
    return best;
}

// bf16: a round of tiles costs a part of its own, a part per 1000 elements of d_in and another that follows how full the rounds are; two
// 64 x 64 tiles share a compute unit (up to 256 of them run one to a unit); the bytes of y; ablated neurons' tables; a second launch and the
// partial sums where d_in is cut.  Non-negative least squares on the relative error of 6258 launches, every shape in one part and in the parts
// that parts_of gives, of 920 products (128 to 4096 wide, 100 to 16384 stored rows, batches 8 to 2048, up to half of the neurons ablated, 1 to 20 %
// of the weights present; graphs of 5 to 40 launches): 10 % per shape.  The tile and parts of smallest time are 0.3 % behind the fastest on average on 609
// products of up to 5 M results (at worst 18 %) and 1.4 % (22 %) on 311 larger ones; 0.5 (23) and 2.7 % (28) with constants fitted to calls from
// the host, 13 % too high and most on the smallest, which also left the condensed form calls that the product does faster (4096 -> 4096, K = 410 at batch 64: 17.7 us
// against 13.9).  (256 x 192 tiles: 9000 rows at batch 2048, d_in 4096, 155 us, 157 in 256 x 128 and 180 in 256 x 256; 5023 at 1696, 1136, 35.7, 48 and 36.)
// The last three shapes are for rounds that the others would leave part empty: 192 x 192 has nine sixteenths of a 256 x 256 tile's work to a round, and 4 wavefronts of
// 96 x 96 read fewer fragments per multiplication than 8 of 128 x 64 (13108 rows at batch 2048, d_in 4096, 1.6 rounds of 256 x 256: 205 us -> 197 on one card, 207.7 -> 204.3 on another, which the power of the matrix units limits; 11440 at 1500, 89 -> 68); a
// layer whose 128 x 128 tiles fill three quarters of the chip or a little more than all of it goes into 128 x 96 or 64 x 128 (2335 at 1024, d_in 576, 16.9 -> 13.1; 9012 at 256, 768,
// 18.5 -> 14.6).  Fitted on 918 products beside the time of the shape taken before, plus 6 %: it takes that much of a promise for one of them, in one part
// only (cut into parts they were level or up to 19 % behind).  Not where they gain nothing on average and lose up to 14 % (left_to_others).  Of 1636 random products that come
// to one of them without that rule the 1529 that still do take 0.897 of the time before on average; 19 of them are more than 2 % behind, at worst 20 % (64 x 64 tiles of
// which there are just 282 take 0.8 of the time of their neighbours: 3376 deep, 6007 at 151 rows 25 us, 30 in 64 x 128).
// Shapes that only the library's choice takes: 8 wavefronts of 64x96, 2 LDS stages of 128 bytes; 4 of 96x96, 3 stages; 4 of 32x96, 4; 4 of 32x64, 4
constexpr int kTile256x192 = 7, kTile192x192 = 8, kTile128x96 = 9, kTile64x128 = 10;
struct Bf16TileModel { int tile, bm, bn; float fixed, round, per_k, per_k_full, y, ablated, second, part; };
static const Bf16TileModel kBf16TileModels[] = {
    {SRIGL_TILE_256x256, 256, 256, 0.71f, 6.96f, 15.62f, 4.62f, 0.69f, 2.06f, 1.71f, 1.82f},
    {kTile256x192, 256, 192, 0.0f, 7.08f, 12.05f, 5.64f, 0.83f, 1.88f, 0.0f, 0.0f},
    {SRIGL_TILE_256x128, 256, 128, 1.62f, 4.69f, 8.47f, 2.07f, 0.82f, 1.95f, 1.31f, 2.07f},
    {SRIGL_TILE_128x128, 128, 128, 3.07f, 2.96f, 5.82f, 1.18f, 0.87f, 1.84f, 1.52f, 2.42f},
    {SRIGL_TILE_64x64, 64, 64, 2.76f, 1.07f, 5.60f, 0.0f, 1.22f, 1.34f, 1.46f, 3.18f},
    {kTile192x192, 192, 192, 3.52f, 7.48f, 9.65f, 1.84f, 0.75f, 1.39f, 0.0f, 0.0f},
    {kTile128x96, 128, 96, 1.59f, 5.88f, 4.85f, 1.38f, 0.61f, 1.27f, 0.0f, 0.0f},
    {kTile64x128, 64, 128, 2.35f, 2.71f, 4.81f, 0.30f, 1.31f, 1.64f, 0.0f, 0.0f},
};
// Time (us) of the product in a shape and `splits` parts.
static double bf16_tiles_us(const Bf16TileModel& m, int splits, int B, int d_in, int n_active, int d_out) {
    const double d = d_in * 1e-3 / splits;
    const long long tiles = (long long)((B + m.bm - 1) / m.bm) * ((n_active + m.bn - 1) / m.bn);
    const double groups = (double)(splits > 1 ? (tiles + kXcds - 1) / kXcds * kXcds * splits : tiles);
    const double more = m.y * 1e-6 * B * d_out + (splits > 1 ? m.second + m.part * 1e-6 * splits * B * (double)n_active : n_active < d_out ? m.ablated : 0.0);
    if (m.bn == 64) return more + (groups <= 256 ? 4.17 + 3.67 * d : m.fixed + std::ceil(groups / 512) * (m.round + m.per_k * d));
    return more + m.fixed + std::ceil(groups / 256) * (m.round + m.per_k * d) + groups / 256 * m.per_k_full * d;
}

// Products in which the last two shapes are behind the ones taken before although the estimates promise 6 %: 128 x 96 from 14 MB of results on (with ablated neurons: 256 tiles without any
// hold 12.6) between 384 and 1152 deep (84 products 2 % faster on average, 32 of them 2 to 14 % slower, where shallower and deeper ones are 5 to 10 % faster);
// 64 x 128 where 64 x 64 tiles are just more than one to a compute unit and it fills half of them, with more than eight rows of tiles (23 products, level, 8 of them 2 to 6 % slower).
static bool left_to_others(int tile, int B, int n_active, int d_in, int d_out) {
    if (tile == kTile128x96) return (long long)B * d_out >= 3500000 && d_in >= 384 && d_in < 1152;
    if (tile == kTile64x128) return B > 512 && (B + 63ll) / 64 * ((n_active + 63ll) / 64) <= 272;
    return false;
}

struct GemmChoice { int tile, splits; double us; };

// Several parts of d_in run side by side; their partial sums pass through a workspace and a second launch adds them: worth it
// when the tiles alone reach a fraction of the 256 compute units.  Parts: as many as keep the workgroups (8 runs of tiles,
// padded) within 256, or within 480 for 64x64 tiles, two of which share a compute unit and then run 1.3 (bf16) to 1.85 (fp32) times
// longer each; at most 16, at least 4 stages of 128 bytes each.  Measured on MI355X (3072 -> 768 fp32, 538 stored neurons): batch 256
// 59 us in one part, 18 us in 12; batch 64 57 us and 11 us in 16.
static int parts_of(int B, int n_active, int d_in, bool f32, int bm, int bn) {
    const int stages = (d_in * (f32 ? 4 : 2) + kSlabBytes - 1) / kSlabBytes;
    const long long tiles = (long long)((B + bm - 1) / bm) * ((n_active + bn - 1) / bn), padded = (tiles + kXcds - 1) / kXcds * kXcds;
    const long long wg_cap = bm == 64 && bn == 64 ? 480 : 256;
    const int cap = std::max(1, std::min(stages / 4, kMaxSplits));
    return padded >= wg_cap ? 1 : std::min((int)(wg_cap / padded), cap);
}

// fp32: the partial sums are written once and read once; the second launch and a second pipeline fill are 2.6 us of the 3.5 that the estimate adds, the
// rest is the host's second launch.  (On 78 products with and without parts, 64 x 64 tiles, 100 to 6000 stored rows, batches 16 to 512.)
constexpr double kPartsUs = 1.7 * 8.0 / 4.5e6;
static GemmChoice choose_f32(int B, int n_active, int d_in, int d_out, bool may_split) {
    GemmChoice best{};
    for (const TileModel& m : kTileModels) {
        const long long tiles = (long long)((B + m.bm - 1) / m.bm) * ((n_active + m.bn - 1) / m.bn), padded = (tiles + kXcds - 1) / kXcds * kXcds;
        const int s = may_split ? parts_of(B, n_active, d_in, true, m.bm, m.bn) : 1;
        for (int pass = 0; pass < 2; ++pass) {   // one part, then several
            if (pass == 1 && s == 1) break;
            double us;
            if (pass == 0) {
                const long long rounds = (tiles + 255) / 256;
                us = 2.1 + (double)rounds * m.ns_per_k_f32 * d_in * 1e-3;
            } else {
                const double crowd = (m.bm == 64 && padded * s > 256) ? 1.85 : 1.0;
                us = 3.5 + m.ns_per_k_f32 * crowd * d_in / s * 1e-3 + kPartsUs * s * (double)B * n_active;
            }
            if (best.tile == 0 || us < best.us) best = {m.tile, pass == 0 ? 1 : s, us};
        }
    }
    best.us += 3.5 + 4.0 * (double)B * d_out / 4.5e6;
    return best;
}

static GemmChoice choose_bf16(int B, int n_active, int d_in, int d_out, bool may_split) {
    GemmChoice best{};
    for (const Bf16TileModel& m : kBf16TileModels) {
        if (m.bn > 64 && (long long)std::max(m.bm, m.bn) * d_in * 2 >= (1ll << 31)) continue;   // launch_gemm's byte offsets
        if (left_to_others(m.tile, B, n_active, d_in, d_out)) continue;
        const double one = bf16_tiles_us(m, 1, B, d_in, n_active, d_out);
        if (best.tile == 0 || one < best.us) best = {m.tile, 1, one};
        const int s = may_split ? parts_of(B, n_active, d_in, false, m.bm, m.bn) : 1;
        if (s == 1 || m.tile >= kTile256x192) continue;
        const double several = bf16_tiles_us(m, s, B, d_in, n_active, d_out);
        if (several < best.us) best = {m.tile, s, several};
    }
    return best;
}
static GemmChoice choose_gemm(int B, int n_active, int d_in, int d_out, bool f32, bool may_split) {
    struct Key { int32_t B, n_active, d_in, d_out, form; };
    static thread_local DecisionCache<Key, GemmChoice, 64> cache;
    return cache.get(Key{B, n_active, d_in, d_out, f32 * 2 + may_split}, [&] {
        return f32 ? choose_f32(B, n_active, d_in, d_out, may_split) : choose_bf16(B, n_active, d_in, d_out, may_split);
    });
}

template <typename T>
static srigl_status launch_structured(int tile, const void* x, int B, int d_in, const void* Wd, const int32_t* active, int n_active,
                                      const float* bias, int d_out, float* y, int splits, float* part, hipStream_t st) {
    if constexpr (sizeof(T) == 2) {
        if (tile == kTile192x192) return launch_gemm<T, 192, 192, 2, 2, 3, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        if (tile == kTile128x96) return launch_gemm<T, 128, 96, 4, 1, 4, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        if (tile == kTile64x128) return launch_gemm<T, 64, 128, 2, 2, 4, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        if (tile == kTile256x192) return launch_gemm<T, 256, 192, 4, 2, 2, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
    }
    switch (tile) {
        case SRIGL_TILE_256x256: return launch_gemm<T, 256, 256, 2, 4, 2, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        case SRIGL_TILE_256x256_H: return launch_gemm<T, 256, 256, 2, 4, 5, 64>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        case SRIGL_TILE_256x128_W4: return launch_gemm<T, 256, 128, 2, 2, 3, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        case SRIGL_TILE_256x128: return launch_gemm<T, 256, 128, 4, 2, 3, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        case SRIGL_TILE_128x128: return launch_gemm<T, 128, 128, 2, 2, 4, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        case SRIGL_TILE_64x64: return launch_gemm<T, 64, 64, 2, 2, 4, 128>(x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
        default: return SRIGL_ERR_INVALID_ARG;
    }
}

}  // namespace srigl

using namespace srigl;

extern "C" {

srigl_status srigl_densify(const void* W_c, srigl_dtype w_dtype, const int32_t* idx, int32_t n_active, int32_t K,
                           int32_t d_in, void* Wd, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n_active < 0 || K < 0 || d_in < 0 || K > d_in) return SRIGL_ERR_INVALID_ARG;
    if (w_dtype != SRIGL_F32 && w_dtype != SRIGL_BF16) return SRIGL_ERR_INVALID_ARG;
    if (n_active == 0 || d_in == 0) return SRIGL_OK;
    if (Wd == nullptr || (K > 0 && (W_c == nullptr || idx == nullptr))) return SRIGL_ERR_INVALID_ARG;
    const size_t bytes = (size_t)n_active * d_in * (w_dtype == SRIGL_F32 ? 4 : 2);
    if ((reinterpret_cast<uintptr_t>(Wd) & 15) == 0 && (bytes & 15) == 0) {
        size_t blocks = (bytes / 16 + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        hipLaunchKernelGGL(k_fill_zero16, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<uint4*>(Wd), bytes / 16);
    } else {
        size_t blocks = (bytes + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        hipLaunchKernelGGL(k_fill_zero_bytes, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<unsigned char*>(Wd), bytes);
    }
    const long long n_terms = (long long)n_active * K;
    if (n_terms > 0) {
        long long blocks = (n_terms + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        if (w_dtype == SRIGL_F32)
            hipLaunchKernelGGL(k_scatter_rows<uint32_t>, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const uint32_t*>(W_c), idx,
                               n_terms, K, d_in, static_cast<uint32_t*>(Wd));
        else
            hipLaunchKernelGGL(k_scatter_rows<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const uint16_t*>(W_c), idx,
                               n_terms, K, d_in, static_cast<uint16_t*>(Wd));
    }
    return hip_ok(hipGetLastError());
}

// Estimates in microseconds, calibrated on MI355X measurements of both forms (fp32 and bf16 storage, batches 1..2048,
// 512- to 4096-wide layers, 80-99 % sparsity):
//   condensed  = the estimate of the forward kernel the library's own choice takes for these sizes (condensed_estimate_us); bf16: or of the
//                matrix-core form with its copy made in the call, whichever is faster
//   structured = choose_bf16; fp32:
//              ~ 3.5 + d_in x (rounds of tiles x nanoseconds per element of d_in of the chosen tile) / 1000 / parts of d_in
//                  + the second launch when d_in is cut into parts (srigl_structured_linear_fwd_split)
//                  + 4 B d_out / 4.5e6              (writing the result at HBM speed)
srigl_representation srigl_choose_representation(int32_t B, int32_t d_in, int32_t n_active, int32_t K, int32_t d_out,
                                                 srigl_dtype dtype, float* est_condensed_us, float* est_structured_us) {
    // bf16: on 920 layers and batches timed in both forms (128 to 4096 wide, batches 8 to 2048) the form taken is 1.1 % slower than the faster one on
    // average, beyond 10 % on 22 (fan-ins of 1 to 3 at batches above 700, which the tiles' estimates put too low, among them); on 144 points of 18 named layers 0.3 %, at worst 15 %.
    // (With the constants before, 1.7 % and 0.9 %, beyond 10 % on 48.  While the condensed estimate was the gathering kernels' alone: up to 20 %, and a
    // dense copy of 107 MB on 4096 -> 16384 for what the estimate called 2.7 times.)
    struct Key { int32_t B, d_in, n_active, K, d_out, dtype; };
    struct Estimates { double cond, stru; };
    static thread_local DecisionCache<Key, Estimates, 64> cache;
    const Estimates e = cache.get(Key{B, d_in, n_active, K, d_out, (int32_t)dtype}, [&] {
        Estimates v;
        v.cond = condensed_estimate_us(B, d_in, n_active, K, d_out, dtype == SRIGL_BF16, n_active < d_out);
        const bool f32 = dtype == SRIGL_F32;
        v.stru = choose_gemm(B > 0 ? B : 1, n_active > 0 ? n_active : 1, d_in, d_out, f32, true).us;
        // (1.04: timed beside the products, in the same graphs, the condensed calls take that much longer than the estimates, whatever the batch and the form)
        if (!f32) v.cond = 1.04 * std::min(v.cond, blocked_estimate_us(B, d_in, n_active, K, d_out));
        if ((d_in * (f32 ? 4 : 2)) % 16 != 0) v.stru = 1e30;   // the matrix-core kernel needs rows of whole 16-byte pieces
        return v;
    });
    if (est_condensed_us) *est_condensed_us = (float)e.cond;
    if (est_structured_us) *est_structured_us = (float)e.stru;
    return e.stru < e.cond ? SRIGL_REPR_STRUCTURED : SRIGL_REPR_CONDENSED;
}

static srigl_status structured_core(const void* x, srigl_dtype x_dtype, int32_t B, int32_t d_in, const void* Wd, srigl_dtype w_dtype,
                                    const int32_t* active, int32_t n_active, const float* bias, int32_t d_out, float* y, int tile,
                                    int splits, void* workspace, size_t workspace_bytes, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (B < 0 || d_in < 0 || n_active < 0 || d_out < 0 || n_active > d_out) return SRIGL_ERR_INVALID_ARG;
    if ((x_dtype != SRIGL_F32 && x_dtype != SRIGL_BF16) || (w_dtype != SRIGL_F32 && w_dtype != SRIGL_BF16)) return SRIGL_ERR_INVALID_ARG;
    if (x_dtype != w_dtype) return SRIGL_ERR_UNSUPPORTED;
    if (active == nullptr && n_active != d_out && n_active != 0) return SRIGL_ERR_INVALID_ARG;
    if (splits < 0 || splits > kMaxSplits) return SRIGL_ERR_INVALID_ARG;
    if (B == 0 || d_out == 0) return SRIGL_OK;
    if (y == nullptr) return SRIGL_ERR_INVALID_ARG;
    if (n_active > 0 && d_in > 0 && (x == nullptr || Wd == nullptr)) return SRIGL_ERR_INVALID_ARG;
    const int elem = (x_dtype == SRIGL_F32) ? 4 : 2;
    if (n_active > 0 && d_in > 0) {
        if ((d_in * elem) % 16 != 0 || ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(Wd)) & 15) != 0)
            return SRIGL_ERR_UNSUPPORTED;
    }
    if (n_active == 0) {   // nothing is stored: every column is its bias
        const dim3 grid((unsigned)((d_out + 255) / 256), (unsigned)((B + kFillRows - 1) / kFillRows));
        if (grid.y > 65535u) return SRIGL_ERR_UNSUPPORTED;
        hipLaunchKernelGGL(k_fill_ablated, grid, dim3(256), 0, st, active, n_active, bias, B, d_out, y);
        return hip_ok(hipGetLastError());
    }
    const bool tile_ok = tile >= SRIGL_TILE_AUTO && tile <= SRIGL_TILE_64x64;
    if (splits == 0) {   // the library's choice of parts (and of the tile, unless forced)
        const GemmChoice c = choose_gemm(B, n_active, d_in, d_out, x_dtype == SRIGL_F32, true);
        splits = tile != SRIGL_TILE_AUTO ? 1 : c.splits;   // a forced tile keeps the whole of d_in unless the parts are forced too
        if (tile == SRIGL_TILE_AUTO) tile = c.tile;
    } else if (tile == SRIGL_TILE_AUTO) {   // one part by choice of the entry point, or the caller's parts
        tile = splits == 1 ? choose_gemm(B, n_active, d_in, d_out, x_dtype == SRIGL_F32, false).tile : choose_tile(B, n_active, x_dtype == SRIGL_F32);
    }
    if (splits > 1) {
        const size_t need = (size_t)splits * B * n_active * sizeof(float);
        if (workspace == nullptr || workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 3) != 0) return SRIGL_ERR_CAPACITY;
    }
    if (!tile_ok) return SRIGL_ERR_INVALID_ARG;
    float* part = static_cast<float*>(workspace);
    if (x_dtype == SRIGL_F32) return launch_structured<float>(tile, x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
    return launch_structured<uint16_t>(tile, x, B, d_in, Wd, active, n_active, bias, d_out, y, splits, part, st);
}

srigl_status srigl_structured_linear_fwd_tile(const void* x, srigl_dtype x_dtype, int32_t B, int32_t d_in, const void* Wd,
                                              srigl_dtype w_dtype, const int32_t* active, int32_t n_active,
                                              const float* bias, int32_t d_out, float* y, srigl_gemm_tile tile, void* stream) {
    return structured_core(x, x_dtype, B, d_in, Wd, w_dtype, active, n_active, bias, d_out, y, tile, 1, nullptr, 0, stream);
}

srigl_status srigl_structured_linear_fwd(const void* x, srigl_dtype x_dtype, int32_t B, int32_t d_in, const void* Wd,
                                         srigl_dtype w_dtype, const int32_t* active, int32_t n_active,
                                         const float* bias, int32_t d_out, float* y, void* stream) {
    return structured_core(x, x_dtype, B, d_in, Wd, w_dtype, active, n_active, bias, d_out, y, SRIGL_TILE_AUTO, 1, nullptr, 0, stream);
}

srigl_status srigl_structured_split_plan(int32_t B, int32_t d_in, int32_t n_active, int32_t d_out, srigl_dtype dtype, int32_t* splits,
                                         size_t* workspace_bytes) {
    if (B < 0 || d_in < 0 || n_active < 0 || d_out < 0 || (dtype != SRIGL_F32 && dtype != SRIGL_BF16)) return SRIGL_ERR_INVALID_ARG;
    int s = 1;
    if (B > 0 && d_in > 0 && n_active > 0) s = choose_gemm(B, n_active, d_in, d_out, dtype == SRIGL_F32, true).splits;
    if (splits) *splits = s;
    if (workspace_bytes) *workspace_bytes = s > 1 ? (size_t)s * B * n_active * sizeof(float) : 0;
    return SRIGL_OK;
}

int32_t srigl_structured_tile_query(int32_t B, int32_t d_in, int32_t n_active, int32_t d_out, srigl_dtype dtype, int32_t may_split) {
    if (B <= 0 || d_in <= 0 || n_active <= 0 || d_out < n_active || (dtype != SRIGL_F32 && dtype != SRIGL_BF16)) return 0;
    return choose_gemm(B, n_active, d_in, d_out, dtype == SRIGL_F32, may_split != 0).tile;
}

srigl_status srigl_structured_linear_fwd_split(const void* x, srigl_dtype x_dtype, int32_t B, int32_t d_in, const void* Wd,
                                               srigl_dtype w_dtype, const int32_t* active, int32_t n_active, const float* bias,
                                               int32_t d_out, float* y, srigl_gemm_tile tile, int32_t splits, void* workspace,
                                               size_t workspace_bytes, void* stream) {
    return structured_core(x, x_dtype, B, d_in, Wd, w_dtype, active, n_active, bias, d_out, y, tile, splits, workspace, workspace_bytes, stream);
}

}  // extern "C"
