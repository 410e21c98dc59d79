// ROWLOOP forward kernel (gfx950): the batched formulation of fwd_rowlane.inl (lanes are batch rows, the activation
// tile transposed in LDS, weights and LDS offsets through DPP row broadcasts; Alg. 1 of arXiv 2305.02299 with the bias of
// Sec. 4.4 and the ablated neurons of Sec. 3.1 step 4) for inputs narrow enough that a batch tile holds *every* column of x.
//
// With all of d_in in LDS there is no walk over column chunks: a stored row's K terms are one contiguous range, no partial
// sum has to live across a chunk boundary, and so a wavefront is not limited to the handful of stored rows whose
// accumulators fit its registers.  It walks any number of rows one after the other and parks each finished row in a
// result tile in LDS.  A workgroup can therefore own as many stored rows as the result tile has room for (hundreds), and
// the batch tile of x, which every workgroup of the chunked kernel stages again for every 16-128 stored rows, is staged
// once per several hundred: at 1024 batch rows on a 768-wide input 8 groups of stored rows instead of 24.
//
// Tile: 8, 16, 32 or 64 batch rows (4, 4, 8 or 16 per lane); from 16 rows on the 64 lanes are 16 groups of four, and every group works on a term of its
// own, so a step takes 16 terms of a row: one 16-byte LDS read per four batch rows of a lane, and quad_perm broadcasts put the
// weight into the multiply-add and the column into the LDS address.  (Groups of 16 lanes with two rows per lane, four terms to a step, as this
// kernel was built first, read 8 bytes per lane at 105 bytes per clock and compute unit and issued three vector instructions for
// 128 multiply-adds; here it is ten for 512 and 139 bytes per clock, since random columns of 128 bytes meet in the banks: 219 where they
// do not.  768 -> 3072: K = 77 at batch 256 10.6 -> 9.5 us, at 1024 27.0 -> 21.9, K = 154 at 1024 43.5 -> 34.7; a 16-row tile of 2160
// columns, K = 216 at 256, in place of the chunked kernel 13.7 -> 9.4; 1000 -> 777, K = 50 at 300 15.8 -> 7.4.)
// What bounds it: vector instructions (the multiply-adds are half of them) and LDS reads in equal parts, behind a fixed 5 to 6 us of
// launching 4096 wavefronts, staging the tile and writing y.
// Tiles of 8 batch rows (all that inputs of 2500 to 4096 columns leave room for; also taken on narrower ones where the batch is small or ends inside a
// 16-row tile): 32 groups of two lanes, 32 terms to a step, the same reads and instructions per term and row.  In place of the chunked kernel 3072 -> 768, K = 307 at batch 256 16.8 -> 11.1 us, 538 stored at 64 10.6 -> 8.4,
// 4096 -> 1024, K = 205 at 512 23.9 -> 19.1, 2816 -> 768 bf16, K = 113 at 1527 35.6 -> 27.6; on 147 points that take it 1.49 times faster on
// average, none slower.
// Rows of 64 tiles only pay on inputs up to about 400 columns wide, where they still leave room for a hundred stored rows.
// Terms: 64 consecutive ones of a row to a vector load, requested two rows ahead.
#pragma once
#include "fwd_rowlane.inl"

namespace srigl {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) f32x4 LdsF32x4;
// acc[0..3] += w[lane Q of this group of GL lanes] * x, or = with FIRST.  (The s_nop covers the two wait states a DPP read needs after
// a VALU write of its source: the compiler does not look into the block.)
template <int GL, int Q, bool FIRST>
__device__ __forceinline__ void fmac4_bcast(float* acc, float w, const f32x4& x) {
#define SRIGL_GROUP " quad_perm:[%9,%9,%10,%10] row_mask:0xf bank_mask:0xf bound_ctrl:1"
    if constexpr (FIRST)
        asm("s_nop 1\n\tv_mul_f32_dpp %0, %4, %5" SRIGL_GROUP "\n\tv_mul_f32_dpp %1, %4, %6" SRIGL_GROUP
            "\n\tv_mul_f32_dpp %2, %4, %7" SRIGL_GROUP "\n\tv_mul_f32_dpp %3, %4, %8" SRIGL_GROUP
            : "=&v"(acc[0]), "=&v"(acc[1]), "=&v"(acc[2]), "=&v"(acc[3])
            : "v"(w), "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w), "n"(Q), "n"(GL == 4 ? Q : Q + 2));
    else
        asm("s_nop 1\n\tv_fmac_f32_dpp %0, %4, %5" SRIGL_GROUP "\n\tv_fmac_f32_dpp %1, %4, %6" SRIGL_GROUP
            "\n\tv_fmac_f32_dpp %2, %4, %7" SRIGL_GROUP "\n\tv_fmac_f32_dpp %3, %4, %8" SRIGL_GROUP
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
            : "v"(w), "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w), "n"(Q), "n"(GL == 4 ? Q : Q + 2));
#undef SRIGL_GROUP
}
// (lane Q of this group) ^ piece: the LDS addresses of a term's pieces
template <int GL, int Q>
__device__ __forceinline__ void xor_bcast(int ov, const int (&piece)[1], int (&at)[1]) {
    asm("s_nop 1\n\tv_xor_b32_dpp %0, %1, %2 quad_perm:[%3,%3,%4,%4] row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "=v"(at[0]) : "v"(ov), "v"(piece[0]), "n"(Q), "n"(GL == 4 ? Q : Q + 2));
}
template <int GL, int Q>
__device__ __forceinline__ void xor_bcast(int ov, const int (&piece)[2], int (&at)[2]) {
    static_assert(GL == 4, "one piece per lane in groups of two");
    asm("s_nop 1\n\tv_xor_b32_dpp %0, %2, %3 quad_perm:[%5,%5,%5,%5] row_mask:0xf bank_mask:0xf bound_ctrl:1"
        "\n\tv_xor_b32_dpp %1, %2, %4 quad_perm:[%5,%5,%5,%5] row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "=&v"(at[0]), "=&v"(at[1]) : "v"(ov), "v"(piece[0]), "v"(piece[1]), "n"(Q));
}
template <int GL, int Q>
__device__ __forceinline__ void xor_bcast(int ov, const int (&piece)[4], int (&at)[4]) {
    const int lo[2] = {piece[0], piece[1]}, hi[2] = {piece[2], piece[3]};
    int l[2], h[2];
    xor_bcast<GL, Q>(ov, lo, l);
    xor_bcast<GL, Q>(ov, hi, h);
    at[0] = l[0]; at[1] = l[1]; at[2] = h[0]; at[3] = h[1];
}

constexpr int kQuadBlock = 64;   // terms a wavefront's vector load of W_c / idx brings: 16 groups of lanes x 4 steps, or 32 x 2

// One step: 16 (32) terms, one per group of four (two) lanes; RL rows per lane, read as RL / 4 pieces of 16 bytes.
template <int RL> struct StepX { f32x4 v[RL / 4]; };
template <int RL> struct Pieces { int at[RL / 4]; };   // where in a column the lane's pieces lie
template <int GL, int RL, int Q>
__device__ __forceinline__ void step_reads(StepX<RL>& x, int ov, const Pieces<RL>& pc) {
    int at[RL / 4];
    xor_bcast<GL, Q>(ov, pc.at, at);
#pragma unroll
    for (int h = 0; h < RL / 4; ++h) x.v[h] = *reinterpret_cast<const LdsF32x4*>((unsigned)at[h]);
}
template <int GL, int RL, int Q, bool FIRST>
__device__ __forceinline__ void step_fmacs(float (&acc)[RL], float wv, const StepX<RL>& x) {
#pragma unroll
    for (int h = 0; h < RL / 4; ++h) fmac4_bcast<GL, Q, FIRST>(acc + 4 * h, wv, x.v[h]);
}
// ST steps of NB = ceil(ST / GL) blocks held in registers, in straight-line code (with the number of steps a run-time value the branches
// between them cost a copy of the accumulators at every exit and kept a register per address).  The reads of a step go out two steps
// ahead of its multiply-adds.
template <int GL, int RL, int ST, int NB, bool FIRST, int G = 0>
__device__ __forceinline__ void walk_steps(float (&acc)[RL], const float (&wv)[NB], const int (&ov)[NB], const Pieces<RL>& pc, StepX<RL> (&x)[3]) {
    if constexpr (G < ST) {
        if constexpr (G + 2 < ST) step_reads<GL, RL, (G + 2) % GL>(x[(G + 2) % 3], ov[(G + 2) / GL], pc);
        step_fmacs<GL, RL, G % GL, FIRST && G == 0>(acc, wv[G / GL], x[G % 3]);
        walk_steps<GL, RL, ST, NB, FIRST, G + 1>(acc, wv, ov, pc, x);
    }
}
template <int GL, int RL, int ST, bool FIRST, int NB>
__device__ __forceinline__ void walk_terms(float (&acc)[RL], const float (&wv)[NB], const int (&ov)[NB], const Pieces<RL>& pc) {
    static_assert(NB == (ST + GL - 1) / GL, "blocks of GL steps");
    StepX<RL> x[3];
    step_reads<GL, RL, 0>(x[0], ov[0], pc);
    if constexpr (ST > 1) step_reads<GL, RL, 1>(x[1], ov[0], pc);
    walk_steps<GL, RL, ST, NB, FIRST>(acc, wv, ov, pc, x);
}

// ST: steps a row's first terms take, 64 / GL to a step (rows of more than 256 terms: 4 GL, the rest in a loop).
template <int GL, int RL, int ST, typename XT, typename IT>
__global__ __launch_bounds__(1024) void k_fwd_rowloop(const XT* __restrict__ x, int B, int d_in, const XT* __restrict__ W_c,
                                                      const IT* __restrict__ idx, const int32_t* __restrict__ active, int n_active,
                                                      int K, const float* __restrict__ bias, int d_out, float* __restrict__ y,
                                                      int NG, int n_btiles, int n_groups, int out_off, int span_cap, int act, int bt_major, int nw) {
    extern __shared__ float lds[];   // x tile [C + 1][S]; result tile [BT][NG | 1]; bias [NG], or bias and column table [span_cap] each
    constexpr int BT = GL * RL;              // batch rows per tile
    constexpr int S = BT;                    // words from column to column
    constexpr int S4 = S * 4;
    constexpr int NB = (ST + GL - 1) / GL;   // blocks of terms held in registers
    static_assert((GL == 4 && (RL == 4 || RL == 8 || RL == 16)) || (GL == 2 && RL == 4), "tiles of 8, 16, 32 or 64 rows");

    // consecutive workgroup ids go to different XCDs (one L2 each): either all batch tiles of a group of stored rows share an
    // XCD (its L2 fetches that group's W_c / idx once and all of x), or (bt_major) all groups of a batch tile (its own rows of
    // x, which every workgroup waits for at its start, and all of W_c / idx, which streams in behind the arithmetic)
    const int wg = blockIdx.x;
    const int xcd = wg & 7, inx = wg >> 3;
    const int dec_d = bt_major ? n_groups : n_btiles;
    const int dec_q = inx / dec_d, dec_r = inx - dec_q * dec_d;
    const int bt = bt_major ? dec_q * 8 + xcd : dec_r;
    const int g = bt_major ? dec_r : dec_q * 8 + xcd;
    if (g >= n_groups || bt >= n_btiles) return;

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = bt * BT;
    const int sg0 = g * NG;
    const int ng = min(NG, n_active - sg0);   // > 0: n_groups = ceil(n_active / NG)
    constexpr int UC = BT < 16 ? 32 : 16;      // columns of a unit
    const int C = (d_in + UC - 1) & ~(UC - 1);   // columns of the tile: whole units (what lies past a row's end is named by no index)
    const int tile0 = (int)(unsigned)reinterpret_cast<size_t>((__attribute__((address_space(3))) float*)lds);   // (0: the kernel has no other LDS)
    const int zero_off = tile0 + C * S4;

    // ---- the tile: units of 16 rows x 16 columns (8 x 32); a wavefront takes every nw-th 16 (32) columns, all rows of them ----
    const int dq = lane & 3, db = BT < 16 ? (lane >> 2) & 7 : lane >> 2, half = BT < 16 ? (lane >> 5) * 16 : 0;
    constexpr int RT = BT < 16 ? 1 : BT / 16;  // units to UC columns
    constexpr int CPP = kStageUnits / RT;      // columns / UC a wavefront holds in registers: eight units
    const int n_ct = C / UC;
    const XT* const xtile = x + (size_t)b0 * d_in;
    const int n_rows = min(BT, B - b0);
    const bool last_rows = b0 + BT >= B;
    const int tile_total = n_rows * d_in + (last_rows ? 0 : 16);   // elements of x from the tile's first on that may be read (at least 16, host)
    const bool shifts = (d_in & 15) != 0 && last_rows;             // the last row of x ends inside a unit: its loads start earlier

    // Terms.  A block is 64 consecutive terms of a row, one per lane and array; at step s of the block the GL lanes of group p
    // work on the term that lane s of the group loaded.  Whole blocks are loaded in the order of the lanes (consecutive words), the last,
    // partial one with the term (64 / GL) s + p in lane s of group p, so that a row of K terms takes ceil(K GL / 64) steps.
    // D = 2 rows are in flight ahead of the one being walked.
    const int p16 = lane / GL, q4 = lane % GL;
    const int t_strided = kWave / GL * q4 + p16;
    unsigned t_lane[NB];                       // this lane's term of each preloaded block, clamped into the row
    bool t_real[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int t = kQuadBlock * b + (K - kQuadBlock * b >= kQuadBlock ? lane : t_strided);
        t_real[b] = b < NB - 1 || t < K;
        t_lane[b] = (unsigned)min(t, K - 1);
    }
    constexpr int D = 2;
    XT rw[D][NB];
    int ri[D][NB];
    auto request_row = [&](int j, XT (&w)[NB], int (&i)[NB]) {   // (j is wave-uniform: a scalar base and the lane's constant offset)
        const size_t row = (size_t)(sg0 + j) * (size_t)K;
        const char* const wrow = reinterpret_cast<const char*>(W_c + row);
        const char* const irow = reinterpret_cast<const char*>(idx + row);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            unsigned t = t_lane[b];
            asm("" : "+v"(t));   // (a lane offset from a scalar base only where its 32 bits are seen to be extended next to the load)
            w[b] = *reinterpret_cast<const XT*>(wrow + t * (unsigned)sizeof(XT));
            i[b] = (int)*reinterpret_cast<const IT*>(irow + t * (unsigned)sizeof(IT));
        }
    };
    // a real term becomes (weight, byte offset of its column in the tile), the others weight 0 on the all-zero column; 32-row tiles:
    // the two 32-byte halves of every 64 bytes of a column change places where bit 3 of the column is set
    auto finish = [&](XT w_raw, int i_raw, bool real, float& wv, int& ov) {
        wv = real ? rl_to_f32<XT>(w_raw) : 0.0f;
        const int at = tile0 + (RL > 4 ? (i_raw * S4) | ((i_raw & 8) << 2) : i_raw * S4);
        ov = real ? at : zero_off;
    };

    // What the stores at the end need besides the sums is requested behind the tile and parked in LDS before the first barrier,
    // so that the epilogue reads LDS only (its loads used to cost it two dependent trips to the L2, about a microsecond):
    // without an active list the bias of the workgroup's columns; with one, the run of consecutive columns [c0, c1) that the
    // workgroup writes (the columns behind the previous group's last stored one up to this group's last; the last group also
    // takes the ablated columns up to d_out), the bias of that run and, per column of it, which row of the result tile holds
    // it, if any.  TP entries per thread wait in registers behind the tile's requests; what is beyond goes through a loop.
    constexpr int TP = 1;
    const int nthreads = nw * kWave;
    float* const out = lds + out_off;
    const int OS = NG | 1;                    // odd stride: conflict-free transposed writes
    float* const bsp = out + BT * OS;         // bias of the workgroup's columns
    // the batch row whose sum a lane is left with: 16-lane rows 0..3 hold the group's rows 0, 2, 1, 3
    const int out_row = (p16 & (RL / 4 - 1)) * 16 + 4 * q4 + ((lane >> 5) | ((lane >> 3) & 2));
    int* const tab = reinterpret_cast<int*>(bsp + (active ? span_cap : NG));
    int c0 = 0, c1 = 0, span = 0;
    bool tabled = false;
    if (active != nullptr) {
        c0 = sg0 > 0 ? min(max(active[sg0 - 1] + 1, 0), d_out) : 0;
        c1 = (g == n_groups - 1) ? d_out : min(max(active[sg0 + ng - 1] + 1, c0), d_out);
        span = c1 - c0;
        tabled = span <= span_cap;
    }
    const int n_bias = active ? (tabled ? span : 0) : ng;      // bias entries parked, counted from column (active ? c0 : sg0)
    const int bias0 = active ? c0 : sg0;
    float e_bias[TP];
    int e_col[TP];

    // A pass stages kStageUnits units per wavefront, 16 columns of all rows under one wave-uniform branch (a lane's row past the end
    // re-reads the last one and is dropped afterwards), and the first pass, with 16 wavefronts the only one on inputs up to 4096, 2048, 1024 and 512
    // columns wide in tiles of 8, 16, 32 and 64 rows, is straight-line code: in a loop whose registers a load of the last turn may still own, or with a branch on every
    // load's lanes, the compiler waits for every load in flight before the next one is issued (measured on the staging of this
    // kernel: the six tile loads of a wavefront went out one round trip after the other).
    const float* const bias_src = bias ? bias : reinterpret_cast<const float*>(x);   // never used: entries are 0 without a bias
    unsigned x_lane[RT];                       // element of x the lane loads of column 0, per 16 rows (past B: row B - 1 again, never stored)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) x_lane[rt] = (unsigned)(min(rt * 16 + db, n_rows - 1) * d_in + half + dq * 4);
    // Where the lane's four columns go.  Lanes of neighbouring column groups write different columns of their four at a time: the lanes
    // of a group of four two even and two odd ones, or (16-row tiles) each its own, and with the halves of odd pairs of column
    // groups swapped 32 consecutive lanes meet 32 different banks.
    float* const l_lane = lds + (half + dq * 4) * S + (RL > 4 ? db ^ ((dq & 2) << 2) : db);
    auto stage_pass = [&](int cb, auto first) {
        Staged4<XT> st[CPP][RT];
#pragma unroll
        for (int i = 0; i < CPP; ++i) {
            const int ct = cb + wv_id + i * nw;
            if (ct < n_ct) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    load4_at_element(xtile + min(x_lane[rt] + (unsigned)(ct * UC), (unsigned)(tile_total - 4)), st[i][rt]);
            }
        }
        if constexpr (decltype(first)::value) {
            // behind the tile's first requests: the first rows' terms (vector loads return in order, and the tile's stores
            // into LDS wait for the tile only), and, behind those, what the epilogue needs
#pragma unroll
            for (int d = 0; d < D; ++d) request_row(min(wv_id + d * nw, ng - 1), rw[d], ri[d]);
#pragma unroll
            for (int q = 0; q < TP; ++q) {
                const int e = tid + q * nthreads;
                // (raw values: whether an entry counts is decided where it is written to LDS, so that nothing here waits)
                e_bias[q] = bias_src[bias ? min(bias0 + min(e, max(n_bias - 1, 0)), d_out - 1) : 0];
                e_col[q] = active != nullptr ? active[sg0 + min(e, ng - 1)] : -1;
            }
            if (tabled)
                for (int c = tid; c < span; c += nthreads) tab[c] = -1;
        }
#pragma unroll
        for (int i = 0; i < CPP; ++i) {
            const int ct = cb + wv_id + i * nw;
            if (ct >= n_ct) break;
            if (shifts) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) shift4(st[i][rt], ragged_shift(x_lane[rt] + (unsigned)(ct * UC), tile_total));
            }
            float* const at = l_lane + ct * UC * S;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                float* const d = at + rt * 16;
                const float v0 = st[i][rt].get(0), v1 = st[i][rt].get(1), v2 = st[i][rt].get(2), v3 = st[i][rt].get(3);
                const bool odd = dq & 1;
                if constexpr (RL > 4) {
                    float* const lo = d + (odd ? S : 0);
                    float* const hi = d + (odd ? 0 : S);
                    lo[0] = odd ? v1 : v0; hi[0] = odd ? v0 : v1;
                    lo[2 * S] = odd ? v3 : v2; hi[2 * S] = odd ? v2 : v3;
                } else {
                    const float r0 = odd ? v1 : v0, r1 = odd ? v2 : v1, r2 = odd ? v3 : v2, r3 = odd ? v0 : v3;
                    const bool two = dq & 2;
                    d[dq * S] = two ? r2 : r0; d[((dq + 1) & 3) * S] = two ? r3 : r1;
                    d[((dq + 2) & 3) * S] = two ? r0 : r2; d[((dq + 3) & 3) * S] = two ? r1 : r3;
                }
            }
        }
    };
    stage_pass(0, std::true_type{});
    for (int cb = CPP * nw; cb < n_ct; cb += CPP * nw) stage_pass(cb, std::false_type{});
    if (tid < S) lds[C * S + tid] = 0.0f;   // the all-zero column that padding terms point at
#pragma unroll
    for (int q = 0; q < TP; ++q) {
        const int e = tid + q * nthreads;
        if (e < n_bias) bsp[e] = bias ? e_bias[q] : 0.0f;
    }
    for (int e = tid + TP * nthreads; e < n_bias; e += nthreads) bsp[e] = rl_bias_at(bias, bias0 + e);
    if (tabled) {
        lds_barrier();   // every thread's part of the table is cleared (LDS only: the tile's loads stay in flight)
#pragma unroll
        for (int q = 0; q < TP; ++q) {
            const int col = e_col[q];
            if (tid + q * nthreads < ng && col >= c0 && col < c1) tab[col - c0] = tid + q * nthreads;
        }
        for (int e = tid + TP * nthreads; e < ng; e += nthreads) {
            const int col = active[sg0 + e];
            if (col >= c0 && col < c1) tab[col - c0] = e;
        }
    }
    __syncthreads();

    // ---- the rows of this wavefront, one after the other ----
    // A column is RL / 4 pieces of 64 bytes.  The group at place p of its 16 lanes reads them from piece p on, around, so that the
    // groups served together read different pieces (acc[4 h + k] belongs to row 16 * piece + 4 q + k).
    Pieces<RL> pc;
#pragma unroll
    for (int h = 0; h < RL / 4; ++h) pc.at[h] = ((p16 + h) & (RL / 4 - 1)) * 64 + q4 * 16;
    auto walk_row = [&](int j, XT (&w)[NB], int (&i)[NB]) {
        float acc[RL];
        float pw[NB];
        int po[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) finish(w[b], i[b], t_real[b], pw[b], po[b]);
        // rows of more than 256 terms: their next two blocks are requested now, ahead of the row D rows on (loads return in order)
        XT xw[2];
        int xi[2];
        auto request_block = [&](int t0, XT& w_raw, int& i_raw) {
            const size_t row = (size_t)(sg0 + j) * (size_t)K;
            unsigned t = (unsigned)min(t0 + lane, K - 1);
            w_raw = *reinterpret_cast<const XT*>(reinterpret_cast<const char*>(W_c + row) + t * (unsigned)sizeof(XT));
            i_raw = (int)*reinterpret_cast<const IT*>(reinterpret_cast<const char*>(idx + row) + t * (unsigned)sizeof(IT));
        };
        constexpr int kHeld = 4 * kQuadBlock;
        if constexpr (ST == 4 * GL) {
            if (K > kHeld) {
                request_block(kHeld, xw[0], xi[0]);
                request_block(kHeld + kQuadBlock, xw[1], xi[1]);
            }
        }
        // the buffer is free: the row D rows on goes out now, with the arithmetic of D rows to return in (unconditional, as in
        // the prologue: past the workgroup's last row the last one is read again and never walked; under a branch the wait
        // for the next row's terms would become a wait for everything in flight, these included)
        request_row(min(j + D * nw, ng - 1), w, i);
        walk_terms<GL, RL, ST, true>(acc, pw, po, pc);
        if constexpr (ST == 4 * GL) {
            auto block = [&](int t0, XT& w_raw, int& i_raw) {
                float wc[1];
                int oc[1];
                finish(w_raw, i_raw, t0 + lane < K, wc[0], oc[0]);
                request_block(t0 + 2 * kQuadBlock, w_raw, i_raw);
                walk_terms<GL, RL, GL, false>(acc, wc, oc, pc);
            };
            for (int t0 = kHeld; t0 < K; t0 += 2 * kQuadBlock) {
                block(t0, xw[0], xi[0]);
                if (t0 + kQuadBlock < K) block(t0 + kQuadBlock, xw[1], xi[1]);
            }
        }
        // The groups hold partial sums of the same batch rows.  Every group of a 16-lane row collects the sums of the piece that
        // it reads first; then registers are paired, lanes 0-31 of the sum taking the first and lanes 32-63 the second register's, and
        // again between the odd and even 16-lane rows.  What is left is one batch row per lane of a 64-row tile; in smaller tiles
        // groups that read the same piece first add theirs.
        float m[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            m[k] = acc[k];
            if constexpr (RL >= 8) m[k] += row_ror<4>(acc[4 + k]);
            if constexpr (RL == 16) m[k] += row_ror<8>(acc[8 + k]) + row_ror<12>(acc[12 + k]);
        }
        const auto h0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(m[0]), __float_as_uint(m[1]), false, false);
        const auto h1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(m[2]), __float_as_uint(m[3]), false, false);
        const float u0 = __uint_as_float(h0[0]) + __uint_as_float(h0[1]), u1 = __uint_as_float(h1[0]) + __uint_as_float(h1[1]);
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u0), __float_as_uint(u1), false, false);
        float v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        if constexpr (RL <= 8) v += row_ror<8>(v);
        if constexpr (RL == 4) v += row_ror<4>(v);
        if constexpr (GL == 2) v += row_ror<2>(v);
        if ((p16 & (16 / GL - 1)) < RL / 4) out[out_row * OS + j] = v;
    };
    __builtin_amdgcn_s_setprio(3);
    const int third = ng / 3;
    int j = wv_id;
    for (; j + (D - 1) * nw < ng; j += D * nw) {   // whole turns of the D buffers: straight-line
#pragma unroll
        for (int d = 0; d < D; ++d) walk_row(j + d * nw, rw[d], ri[d]);
        if (j >= 2 * third) __builtin_amdgcn_s_setprio(0);
        else if (j >= third) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(2);
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)                 // the rows of a last, partial turn
        if (j + d * nw < ng) walk_row(j + d * nw, rw[d], ri[d]);
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();

    // ---- results: row-contiguous stores of the workgroup's run of columns ----
    if (active == nullptr) {
        for (int row = wv_id; row < n_rows; row += nw) {
            float* yr = y + (size_t)(b0 + row) * d_out + sg0;
            for (int c = lane; c < ng; c += kWave) {
                const float v = out[row * OS + c] + bsp[c];
                __builtin_nontemporal_store(act == SRIGL_ACT_NONE ? v : apply_act(v, act), &yr[c]);
            }
        }
        return;
    }
    if (tabled) {
        // lanes write the run left to right
        for (int row = wv_id; row < n_rows; row += nw) {
            float* yr = y + (size_t)(b0 + row) * d_out + c0;
            for (int c = lane; c < span; c += kWave) {
                const int t = tab[c];
                const float bv = bsp[c];
                const float v = t >= 0 ? out[row * OS + t] + bv : bv;
                __builtin_nontemporal_store(act == SRIGL_ACT_NONE ? v : apply_act(v, act), &yr[c]);
            }
        }
        return;
    }
    // runs longer than the table (few stored neurons among many ablated ones): every lane writes its stored column and the
    // ablated columns in front of it; the last group's first lane also writes the columns behind the last stored one
    for (int row = wv_id; row < n_rows; row += nw) {
        float* yr = y + (size_t)(b0 + row) * d_out;
        for (int j = lane; j < ng; j += kWave) {
            const int col = active[sg0 + j];
            const int prev = sg0 + j > 0 ? max(active[sg0 + j - 1] + 1, 0) : 0;
            for (int cc = prev; cc < min(col, d_out); ++cc) {
                const float bv = rl_bias_at(bias, cc);
                __builtin_nontemporal_store(act == SRIGL_ACT_NONE ? bv : apply_act(bv, act), &yr[cc]);
            }
            if (col >= 0 && col < d_out) {
                const float v = out[row * OS + j] + rl_bias_at(bias, col);
                __builtin_nontemporal_store(act == SRIGL_ACT_NONE ? v : apply_act(v, act), &yr[col]);
            }
        }
        if (g == n_groups - 1 && lane == 0) {
            for (int cc = max(active[n_active - 1] + 1, 0); cc < d_out; ++cc) {
                const float bv = rl_bias_at(bias, cc);
                __builtin_nontemporal_store(act == SRIGL_ACT_NONE ? bv : apply_act(bv, act), &yr[cc]);
            }
        }
    }
}

template <int GL, int RL, int ST, typename XT, typename IT>
static srigl_status launch_rowloop_f(const FwdArgs& a, const RowloopPlan& p, hipStream_t st) {
    auto kern = k_fwd_rowloop<GL, RL, ST, XT, IT>;
    static LdsLimit lds_limit;
    if (lds_limit.ensure(kern, p.lds) != SRIGL_OK) return SRIGL_ERR_HIP;
    const long long blocks = p.bt_major ? 8LL * ((p.n_btiles + 7) / 8) * p.n_groups : 8LL * ((p.n_groups + 7) / 8) * p.n_btiles;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(p.NW * kWave), p.lds, st, (const XT*)a.x, a.B, a.d_in, (const XT*)a.W_c,
                       (const IT*)a.idx, a.active, a.n_active, a.K, a.bias, a.d_out, a.y, p.NG, p.n_btiles, p.n_groups, p.out_off,
                       p.span_cap, a.act, p.bt_major, p.NW);
    return hip_ok(hipGetLastError());
}

template <int GL, int RL, typename XT, typename IT>
static srigl_status launch_rowloop_r(const FwdArgs& a, const RowloopPlan& p, hipStream_t st) {
    if constexpr (GL == 4) {
        switch (p.ST) {
            case 10: return launch_rowloop_f<GL, RL, 10, XT, IT>(a, p, st);
            case 12: return launch_rowloop_f<GL, RL, 12, XT, IT>(a, p, st);
            case 14: return launch_rowloop_f<GL, RL, 14, XT, IT>(a, p, st);
            case 16: return launch_rowloop_f<GL, RL, 16, XT, IT>(a, p, st);
            default: break;
        }
    }
    switch (p.ST) {
        case 1: return launch_rowloop_f<GL, RL, 1, XT, IT>(a, p, st);
        case 2: return launch_rowloop_f<GL, RL, 2, XT, IT>(a, p, st);
        case 3: return launch_rowloop_f<GL, RL, 3, XT, IT>(a, p, st);
        case 4: return launch_rowloop_f<GL, RL, 4, XT, IT>(a, p, st);
        case 5: return launch_rowloop_f<GL, RL, 5, XT, IT>(a, p, st);
        case 6: return launch_rowloop_f<GL, RL, 6, XT, IT>(a, p, st);
        case 7: return launch_rowloop_f<GL, RL, 7, XT, IT>(a, p, st);
        case 8: return launch_rowloop_f<GL, RL, 8, XT, IT>(a, p, st);
        default: return SRIGL_ERR_UNSUPPORTED;
    }
}

template <typename XT, typename IT>
static srigl_status launch_rowloop_x(const FwdArgs& a, const RowloopPlan& p, hipStream_t st) {
    switch (p.BT) {
        case 8: return launch_rowloop_r<2, 4, XT, IT>(a, p, st);
        case 16: return launch_rowloop_r<4, 4, XT, IT>(a, p, st);
        case 32: return launch_rowloop_r<4, 8, XT, IT>(a, p, st);
        default: return launch_rowloop_r<4, 16, XT, IT>(a, p, st);
    }
}

}  // namespace srigl
