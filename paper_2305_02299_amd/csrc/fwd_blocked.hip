// BLOCKED forward kernel (gfx950, bf16 storage): Alg. 1 of arXiv 2305.02299 on the matrix cores, from a blocked copy of the
// condensed rows.
//
//     y[b][active[s]] = act(bias[active[s]] + sum_k W_c[s][k] * x[b][idx[s][k]])
//
// The gathering kernels read one word of x from LDS per term and batch row, which the LDS serves at 128 bytes per clock and
// compute unit whatever the batch; from a few dozen batch rows on the matrix cores get through the multiplications by the
// pruned positions faster than that.  Nothing dense is kept in memory: a workgroup owns BM batch rows x BN stored rows and
// walks d_in 64 columns at a time; for each piece it clears a BN x 64 weight tile in LDS, writes the piece's terms into it and
// multiplies it with the staged piece of x.  Products of bf16 values are exact in fp32 and the sums run in fp32, as in the
// gathering kernels.
//
// The blocked copy (srigl_block_terms) holds the terms of 32 stored rows x 64 columns next to each other, each as the weight
// beside its place in the LDS tile: 64 lanes fetch up to 256 of them with one 16-byte load each and store them with four 2-byte
// LDS writes each.  (From the row-major copies the same kernel needed 327 us instead of 251 (201 by now) on 4096 -> 16384, 13108 stored
// rows, K = 205, 2048 batch rows: every row's few terms of a piece were a cache line and a lane's predicated writes of their own.)
//
// Pipeline (an iteration is CC pieces of 64 columns): x of the next iteration goes from memory straight into the other of two LDS
// stages while this one is multiplied, and the terms one iteration further ahead into registers.  The weight tile of it + 1 is built while
// the tile of it is multiplied; half of the wavefronts of a 256 x 256 tile build before they multiply, the other half after it, so that
// a SIMD's two wavefronts do different things; by their priorities those that build late multiply first (s_setprio: without it a SIMD's two
// wavefronts came to the end of their multiplications together, and the matrix units waited for the late builds).  A step's fragments
// are read and x is requested between its multiplications, the reads in their first half.
// What bounds it: the matrix units and the build between them; 4096 -> 16384 with 13108 stored rows, batch 2048, in 256 x 256 tiles: an
// iteration of 2048 clocks of multiplications per SIMD took 3400, of which a build 600 and the requests of x 600 (14 instructions of
// addresses each); with the terms in registers instead of an LDS slot, one instruction of addresses per request (a column past the rows' end
// is their last one), reads between the multiplications and the priorities: 237 -> 201 us.  256 wide tiles of other layers 70 -> 58,
// 32.1 -> 26.9, 192 wide 65 -> 57, 128 wide 275 -> 250, 17.5 -> 15.5, 64 wide 440 -> 397, 14.5 -> 13.6.  (Requests of x a step earlier, behind the
// barrier: 242 us, every wavefront's at the same time.)
// LDS layout of a stage: sub-tiles of 64 columns, a row 128 bytes, its 16-byte piece q in slot q ^ ((row >> 1) & 7), as in
// structured.hip.  A wavefront clears and fills whole blocks: no barrier between the two, the LDS serves one wavefront's requests
// in order.
//
// A stored zero times an activation that is not finite is not a term of the layer, but spoils the sum.  The rows of a tile with a sum that is
// not finite are therefore computed again from the terms (mend_rows); finite sums cannot have met such an activation.
#include "mma_tile.h"
#include <algorithm>
#include <cmath>

namespace srigl {

constexpr int kBlockRows = 32;   // stored rows of a block (of kSegCols columns)

// The blocked copy: first the table offs[groups][chunks + 1], in units of four terms from the lists' start, then the lists.  A
// group's lists lie behind each other in chunk order from group * units_per_group on; each is padded to whole units with copies
// of its last term.  A term: weight bits (low half), byte offset in the block's 32 x 128-byte LDS tile (high half).
struct BlockedLayout {
    int groups, chunks, units_per_group;
    size_t table_bytes, bytes;
};
static BlockedLayout blocked_layout(int n_rows, int K, int d_in) {
    BlockedLayout l;
    l.groups = (n_rows + kBlockRows - 1) / kBlockRows;
    l.chunks = (d_in + kSegCols - 1) / kSegCols;
    l.units_per_group = (kBlockRows * K + 3 * l.chunks) / 4 + 1;
    l.table_bytes = ((size_t)l.groups * (l.chunks + 1) * 4 + 15) / 16 * 16;
    l.bytes = l.table_bytes + (size_t)l.groups * l.units_per_group * 16;
    return l;
}

// byte offset of column c (0..63) of row r (0..31) in a block's LDS tile
__device__ __forceinline__ uint32_t block_place(int r, int c) { return (uint32_t)(r * 128) + (((uint32_t)c * 2u) ^ (((uint32_t)(r >> 1) & 7u) << 4)); }

// One workgroup per group of 32 rows, two rows to a wavefront.  The counts per (row, chunk) come from the seg table, lane l having
// chunk l of the wavefront's rows; their sums over the wavefronts below, and along the chunks (which every wavefront sums for itself),
// give each term its place without another pass.  The terms are requested before the table is waited for, and a list is put together in LDS
// (STAGED: where it fits) so that it leaves in whole lines.  A call that brings no copy pays for this in front of its product.  On small
// layers the chain of dependent steps bounds it (200 -> 300 adds 4.2 us to a call, 512 -> 2048 with K = 100 4.9), on large ones the
// terms' way in and out (4096 -> 16384, K = 205, 37 MB: 10.3 us; with the terms fetched behind the sums, each list stored from where its
// terms' lanes were and the sums down the rows by one lane per chunk 15.1).  Eight loads ahead instead of four need more registers than
// two workgroups per compute unit leave (14 us).
constexpr int kBuildThreads = 1024, kBuildWaves = kBuildThreads / 64, kBuildAhead = 4;   // loads of 64 terms per row in flight
static_assert(kBlockRows == 2 * kBuildWaves, "two rows per wavefront");
template <typename IT, bool STAGED>
__global__ __launch_bounds__(kBuildThreads, 8) void k_block_terms(const uint16_t* __restrict__ W_c, const IT* __restrict__ idx,
                                                               const uint16_t* __restrict__ seg, int seg_stride, int n_rows, int K, int chunks,
                                                               int units_per_group, uint32_t* __restrict__ table, uint4* __restrict__ lists) {
    extern __shared__ __attribute__((aligned(16))) uint32_t sh[];
    uint32_t* const stage = sh;                                                   // STAGED: the group's lists
    uint2* const span = reinterpret_cast<uint2*>(sh + (STAGED ? 4 * (size_t)units_per_group : 0));   // [chunks + 1]: the lists' first places, their terms
    uint32_t* const place = reinterpret_cast<uint32_t*>(span + chunks + 1);       // [32][chunks]: place of term 0 of the row if it were in this chunk's list
    uint32_t* const part = place + kBlockRows * chunks;                           // [2][wavefronts][64]: terms per chunk of the wavefront's rows
    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r0 = g * kBlockRows + 2 * wv;
    const int rows = min(max(n_rows - r0, 0), 2);   // of this wavefront
    uint32_t w[2][kBuildAhead], col[2][kBuildAhead];
    auto load = [&](int r, int k0) {
#pragma unroll
        for (int u = 0; u < kBuildAhead; ++u) {
            const size_t at = (size_t)(r0 + r) * K + min(k0 + 64 * u + lane, K - 1);
            if (k0 + 64 * u < K) { w[r][u] = W_c[at]; col[r][u] = (uint32_t)idx[at]; }
        }
    };
#pragma unroll
    for (int r = 0; r < 2; ++r)
        if (r < rows) load(r, 0);
    uint32_t base = 0;   // units of the chunks before
    for (int c0 = 0; c0 < chunks; c0 += 64) {
        const int c = c0 + lane;
        uint32_t s0[2] = {0u, 0u}, n[2] = {0u, 0u};
#pragma unroll
        for (int r = 0; r < 2; ++r)
            if (r < rows && c < chunks) {
                const uint16_t* s = seg + (size_t)(r0 + r) * seg_stride + c;
                s0[r] = s[0];
                n[r] = (uint32_t)max((int)s[1] - (int)s0[r], 0);
            }
        uint32_t* const p = part + (c0 & 64) * kBuildWaves;   // (two places in turn: one barrier)
        p[wv * 64 + lane] = n[0] + n[1];
        __syncthreads();
        uint32_t below = 0, total = 0;
#pragma unroll
        for (int v = 0; v < kBuildWaves; ++v) {
            const uint32_t m = p[v * 64 + lane];
            below += v < wv ? m : 0u;
            total += m;
        }
        const uint32_t units = (total + 3) / 4, incl = wave_prefix(units), first = min(base + incl - units, (uint32_t)units_per_group);
        base += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (c < chunks) {
            place[2 * wv * chunks + c] = 4 * first + below - s0[0];
            place[(2 * wv + 1) * chunks + c] = 4 * first + below + n[0] - s0[1];
            if (wv == 0) span[c] = make_uint2(4 * first, min(total, 4 * ((uint32_t)units_per_group - first)));
        }
    }
    if (tid == 0) span[chunks] = make_uint2(4 * min(base, (uint32_t)units_per_group), 0u);
    __syncthreads();
    const uint32_t group0 = (uint32_t)g * (uint32_t)units_per_group;
    for (int c = tid; c <= chunks; c += kBuildThreads) table[(size_t)g * (chunks + 1) + c] = group0 + span[c].x / 4;
    uint32_t* const out = STAGED ? stage : reinterpret_cast<uint32_t*>(lists + group0);
#pragma unroll
    for (int r = 0; r < 2; ++r)
        for (int k0 = 0; r < rows && k0 < K; k0 += 64 * kBuildAhead) {
            if (k0 != 0) load(r, k0);
            uint32_t at[kBuildAhead];
            uint2 list[kBuildAhead];
#pragma unroll
            for (int u = 0; u < kBuildAhead; ++u)   // (every place is read before the first term is written: LDS answers take a hundred clocks)
                if (k0 + 64 * u < K) {
                    const int c = (int)min(col[r][u] >> 6, (uint32_t)chunks - 1u);
                    list[u] = span[c];
                    at[u] = place[(2 * wv + r) * chunks + c] + (uint32_t)(k0 + 64 * u + lane) - list[u].x;   // within the list
                }
#pragma unroll
            for (int u = 0; u < kBuildAhead; ++u)
                if (k0 + 64 * u + lane < K && at[u] < list[u].y) {   // (else an idx that its seg table does not describe)
                    const uint32_t term = w[r][u] | (block_place(2 * wv + r, (int)(col[r][u] & 63u)) << 16);
                    out[list[u].x + at[u]] = term;
                    if (at[u] + 1u == list[u].y)   // padding: copies of the last term
                        for (uint32_t i = at[u] + 1u; i % 4 != 0; ++i) out[list[u].x + i] = term;
                }
        }
    if (STAGED) {
        __syncthreads();
        for (uint32_t u = tid; u < span[chunks].x / 4; u += kBuildThreads) lists[group0 + u] = reinterpret_cast<const uint4*>(stage)[u];
    }
}

struct BlockedArgs {
    const uint16_t* x;
    const uint32_t* table;
    const unsigned char* lists;
    const uint16_t* W_c;           // W_c / idx: for sums that are not finite
    const void* idx;
    const int32_t* active;
    const float* bias;
    float* y;
    int B, d_in, n_active, K, d_out, idx_u16, act;
    int n_base, tiles_m, tiles_n;   // of the launch: its first stored row, its tiles
};

// The rows of a tile whose bits are set in `spoiled`, computed again from the neurons' own terms: eight rows of x at a time stand in LDS,
// interleaved, so that a term's eight factors come with one 16-byte read; a wavefront takes a neuron, its lanes the terms.  `area` bytes of
// LDS at smem are free (inputs wider than area / 16 columns go through it in runs, the sums so far waiting at `sums`, [bn][8]).
// 4096 -> 16384 (13108 stored, K = 205) at batch 2048: 245 us as it was, 320 with one NaN in the batch, 3.4 ms with one in every row, whatever
// else (the gathering kernel: 0.85 ms); with every sum added up by one lane, term after term from memory, 1.3 ms and 23 ms.  (Rewritten
// operands through the matrix cores once more, four passes, took 2.8 ms for either, and its registers 3 to 7 % of every call.)
constexpr int kMendRows = 8, kMendAhead = 4;   // rows at a time; loads of 64 terms in flight, for two neurons
__device__ __forceinline__ void mend_rows(const BlockedArgs& p, unsigned char* smem, int area, float* sums, const uint32_t* spoiled, int bm, int bn, int waves, int m0, int n0) {
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int stored = min(bn, p.n_active - n0), width = area / (2 * kMendRows) / 64 * 64;
    const int g = ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);   // the row whose sum ends up in this lane
    for (int done = 0;; done += kMendRows) {
        // the next rows: number `done` and on of the set bits
        int rows[kMendRows], n = 0, seen = 0;
        for (int w = 0; w < bm / 32; ++w)
            for (uint32_t bits = spoiled[w]; bits; bits &= bits - 1) {
                if (seen >= done && n < kMendRows) {
                    const int r = m0 + 32 * w + __ffs(bits) - 1;
#pragma unroll
                    for (int q = 0; q < kMendRows; ++q) rows[q] = q >= n ? r : rows[q];   // (rows that are missing repeat the last one)
                    ++n;
                }
                ++seen;
            }
        if (n == 0) return;
        for (int c0 = 0; c0 < p.d_in; c0 += width) {
            const int cols = min(width, p.d_in - c0);
            __syncthreads();   // the run before has been read (at first: the tile)
            for (int c = tid; c < cols; c += waves * kWave) {
                uint32_t h[kMendRows];
#pragma unroll
                for (int q = 0; q < kMendRows; ++q) h[q] = p.x[(size_t)rows[q] * p.d_in + c0 + c];
                *reinterpret_cast<uint4*>(smem + 16 * (size_t)c) = make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
            }
            __syncthreads();
            for (int s0 = 2 * wv; s0 < stored; s0 += 2 * waves) {
                float acc[2][kMendRows];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int q = 0; q < kMendRows; ++q) acc[t][q] = 0.0f;
                for (int k0 = 0; k0 < p.K; k0 += 64 * kMendAhead) {
                    float w[2][kMendAhead];
                    int col[2][kMendAhead];
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int u = 0; u < kMendAhead; ++u) {
                            const int k = k0 + 64 * u + lane;
                            const size_t at = (size_t)(n0 + min(s0 + t, stored - 1)) * p.K + min(k, p.K - 1);
                            w[t][u] = bf16_bits_to_float(p.W_c[at]);
                            const uint32_t c = p.idx_u16 ? static_cast<const uint16_t*>(p.idx)[at] : static_cast<const uint32_t*>(p.idx)[at];
                            col[t][u] = k < p.K ? (int)min(c, (uint32_t)p.d_in - 1u) - c0 : -1;
                        }
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int u = 0; u < kMendAhead; ++u)
                            if (col[t][u] >= 0 && col[t][u] < cols) {
                                const uint4 v = *reinterpret_cast<const uint4*>(smem + 16 * (size_t)col[t][u]);
                                const uint32_t pair[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                                for (int q = 0; q < 4; ++q) {
                                    acc[t][2 * q] = fmaf(w[t][u], __uint_as_float(pair[q] << 16), acc[t][2 * q]);
                                    acc[t][2 * q + 1] = fmaf(w[t][u], __uint_as_float(pair[q] & 0xffff0000u), acc[t][2 * q + 1]);
                                }
                            }
                }
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    float(&v)[kMendRows] = acc[t];
#pragma unroll
                    for (int half = kMendRows / 2, d = 32; half >= 1; half /= 2, d /= 2)   // half of the rows to the upper lanes, half to the lower
#pragma unroll
                        for (int q = 0; q < half; ++q) {
                            const bool up = (lane & d) != 0;
                            v[q] = (up ? v[q + half] : v[q]) + __shfl_xor(up ? v[q] : v[q + half], d, 64);
                        }
                    float sum = v[0];
#pragma unroll
                    for (int d = 4; d >= 1; d /= 2) sum += __shfl_xor(sum, d, 64);
                    const int s = s0 + t;
                    if (s >= stored || (lane & 7) != 0) continue;
                    if (c0 > 0) sum += sums[s * kMendRows + g];
                    if (c0 + cols < p.d_in) {
                        sums[s * kMendRows + g] = sum;
                        continue;
                    }
                    const int out = p.active ? p.active[n0 + s] : n0 + s;
                    if (g < n && out >= 0 && out < p.d_out) {
                        int row = rows[0];
#pragma unroll
                        for (int q = 1; q < kMendRows; ++q) row = q == g ? rows[q] : row;
                        p.y[(size_t)row * p.d_out + out] = apply_act(sum + (p.bias ? p.bias[out] : 0.0f), p.act);
                    }
                }
            }
        }
    }
}

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(2))) Half4 { uint32_t a, b; };

// LDS: two stages of x, two of the weight tile, all of it reused by the epilogue's tile; behind it the epilogue's table
template <int UA, int BM, int BN, int WGM, int WGN, int CC>
constexpr size_t blocked_table_at() {
    constexpr size_t stages = (size_t)CC * 128 * 2 * (BM + BN), tile = EpiLayout<BN, WGM>::TILE_BYTES;
    return stages > tile ? stages : tile;
}

// UA: loads of 256 terms a block's list gets ahead of time (longer lists: the rest is fetched when it is needed)
template <int UA, bool DIRECT, int BM, int BN, int WGM, int WGN, int CC>
__global__ __launch_bounds__(WGM * WGN * 64) void k_fwd_blocked(const BlockedArgs p) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    constexpr int NWAVES = WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN, TM = WTM / 32, TN = WTN / 32;
    constexpr int XSTAGE = CC * BM * 128, WSTAGE = CC * BN * 128;
    constexpr int XP = CC * BM / 8 / NWAVES;   // 1 KB pieces of the x stage per wavefront (8 rows of 128 bytes each)
    constexpr int KSTEPS = 4 * CC;             // MFMA steps of 16 columns per iteration
    constexpr int BLOCKS = CC * BN / kBlockRows;   // of an iteration, one per wavefront
    static_assert(BLOCKS <= NWAVES && (CC == 1 || BLOCKS == NWAVES), "one block per wavefront and iteration");
    static_assert(CC * BM % (8 * NWAVES) == 0 && WTM % 32 == 0 && WTN % 32 == 0 && BM % 16 == 0, "tile shape");
    unsigned char* const wstages = smem + 2 * XSTAGE;
    unsigned char* const table = smem + blocked_table_at<UA, BM, BN, WGM, WGN, CC>();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv / WGN, wn = wv % WGN;
    const int d_in = p.d_in;
    int tile_m, tile_n;
    if (!tile_of_workgroup(blockIdx.x, p.tiles_m, p.tiles_n, &tile_m, &tile_n)) return;
    const int m0 = tile_m * BM, n0 = p.n_base + tile_n * BN;
    const int n_chunks = (d_in + 63) >> 6, n_it = (n_chunks + CC - 1) / CC;

    // ---- x: a lane brings 16 bytes per pass; rows past the batch re-read the last one (never stored), pieces past the end of
    // the rows come from their last columns (DIRECT) or from whatever lies there (they meet zero weights only, and what is not finite
    // in a row spoils its sums wherever it stands)
    uint32_t xoff[XP];   // element offset from the tile's first row, chunk 0 of the iteration
    int xcol[XP];
#pragma unroll
    for (int q = 0; q < XP; ++q) {
        const int row = 8 * (q * NWAVES + wv) + (lane >> 3);   // row of the stage: sub-tile row / BM
        xcol[q] = (row / BM) * 64 + (((lane & 7) ^ ((row >> 1) & 7)) << 3);
        xoff[q] = (uint32_t)min(row % BM, p.B - 1 - m0) * (uint32_t)d_in + (DIRECT ? 0u : (uint32_t)xcol[q]);
    }
    const uint16_t* const xtile = p.x + (size_t)m0 * d_in;
    const uint32_t xtotal = (uint32_t)min(p.B - m0, BM) * (uint32_t)d_in;
    Half4 xr[DIRECT ? 1 : XP][2];
    auto issue_piece = [&](int it, int q) {
        const int c0 = it * CC * 64;
        if (DIRECT) {
            unsigned char* stage = smem + (it & 1) * XSTAGE + 1024 * wv;
            uint32_t off = 2 * (xoff[q] + (uint32_t)min(c0 + xcol[q], d_in - 8));   // (d_in is a multiple of 8: a piece is whole or absent)
            asm("" : "+v"(off));   // (a lane offset from a scalar base: seen to be 32 bits only next to the load)
            __builtin_amdgcn_global_load_lds((gptr_t)(reinterpret_cast<const unsigned char*>(xtile) + off), (lptr_t)(stage + 1024 * NWAVES * q), 16, 0, 0);
        } else {
            const uint16_t* g = xtile + min(xoff[q] + (uint32_t)c0, xtotal - 8u);   // (d_in >= 8: host)
            xr[q][0] = *reinterpret_cast<const Half4*>(g);
            xr[q][1] = *reinterpret_cast<const Half4*>(g + 4);
        }
    };
    auto store_x = [&](int it) {   // !DIRECT
        unsigned char* stage = smem + (it & 1) * XSTAGE + 1024 * wv + 16 * lane;
        const int c0 = it * CC * 64;
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            uint32_t v[4] = {xr[q][0].a, xr[q][0].b, xr[q][1].a, xr[q][1].b};
            // a load that would have run past the tile's last element started up to 8 elements early
            const int sh = min(max((int)(xoff[q] + (uint32_t)c0) - (int)(xtotal - 8u), 0), 7);
            if (__any(sh != 0)) {
                if (sh & 4) { v[0] = v[2]; v[1] = v[3]; v[2] = v[3] = 0; }
                if (sh & 2) { v[0] = v[1]; v[1] = v[2]; v[2] = v[3]; v[3] = 0; }
                if (sh & 1) {
                    v[0] = __builtin_amdgcn_alignbyte(v[1], v[0], 2);
                    v[1] = __builtin_amdgcn_alignbyte(v[2], v[1], 2);
                    v[2] = __builtin_amdgcn_alignbyte(v[3], v[2], 2);
                    v[3] >>= 16;
                }
            }
            *reinterpret_cast<uint4*>(stage + 1024 * NWAVES * q) = make_uint4(v[0], v[1], v[2], v[3]);
        }
    };

    // ---- terms: wavefront wv builds the block of rows 32 * (wv % (BN / 32)) of the tile, sub-tile wv / (BN / 32)
    const int group = n0 / kBlockRows + wv % (BN / kBlockRows), sub = wv / (BN / kBlockRows);
    const bool builds = BLOCKS == NWAVES || wv < BLOCKS;
    const bool has_rows = builds && group * kBlockRows < p.n_active;
    const uint32_t* const offs = p.table + (size_t)(has_rows ? group : 0) * (n_chunks + 1);
    uint32_t list_lo = 0, list_hi = 0;   // lane l: where the lists of iterations 64 i + l begin and end
    auto load_offsets = [&](int it0) {
        const int c = (it0 + lane) * CC + sub;
        const bool in = has_rows && c < n_chunks;
        list_lo = offs[in ? c : 0];
        list_hi = in ? offs[c + 1] : list_lo;
        wait_loads<0>();
    };
    // The units of a list wait in registers for the build, one iteration ahead (past the last iteration the last list again)
    u32x4_t terms[UA];
    uint32_t held_lo = 0, held_n = 0;
    auto load_list = [&](int it) {
        if (!builds) return;
        if ((it & 63) == 0 && it < n_it) load_offsets(it);
        const int at = min(it, n_it - 1) & 63;
        held_lo = (uint32_t)__builtin_amdgcn_readlane((int)list_lo, at);
        held_n = (uint32_t)__builtin_amdgcn_readlane((int)list_hi, at) - held_lo;
#pragma unroll
        for (int i = 0; i < UA; ++i) {
            const uint32_t u = 64u * i + (uint32_t)lane;   // (lanes past the list share one address)
            terms[i] = *reinterpret_cast<const u32x4_t*>(p.lists + (size_t)(held_lo + (u < held_n ? u : 0u)) * 16);
        }
    };
    // (LDS instructions by hand: the compiler would have a write wait for every load into LDS that is in flight)
    auto lds_at = [](const unsigned char* q) { return (uint32_t)(uintptr_t)(lptr_t)q; };
    auto put4 = [&](uint32_t block, u32x4_t v) {
#pragma unroll
        for (int t = 0; t < 4; ++t) asm volatile("ds_write_b16 %0, %1" ::"v"(block + (v[t] >> 16)), "v"(v[t]) : "memory");
    };
    // A block is built from its list: the tile is cleared and the terms are written to their places, behind the zeros in the order of the
    // LDS; the next list is requested into the registers that this one leaves.
    auto build = [&](int it) {
        if (!builds) return;
        const uint32_t block = lds_at(wstages + (it & 1) * WSTAGE + wv * 4096), clear = block + (uint32_t)lane * 16u;
        const u32x4_t zero = {0u, 0u, 0u, 0u};
        asm volatile("ds_write_b128 %0, %1\n\tds_write_b128 %0, %1 offset:1024\n\tds_write_b128 %0, %1 offset:2048\n\t"
                     "ds_write_b128 %0, %1 offset:3072" ::"v"(clear), "v"(zero) : "memory");
        const uint32_t lo = held_lo, n = held_n;
#pragma unroll
        for (int i = 0; i < UA; ++i)
            if (64u * i + (uint32_t)lane < n) put4(block, terms[i]);
        for (uint32_t u = 64u * UA; u < n; u += 64u)
            if (u + (uint32_t)lane < n) {
                const u32x4_t more = *reinterpret_cast<const u32x4_t*>(p.lists + (size_t)(lo + u + (uint32_t)lane) * 16);
                put4(block, more);
            }
        load_list(it + 1);
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    const int swz = ((lane & 31) >> 1) & 7;
    int frag_off[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) frag_off[kk] = (lane & 31) * 128 + (((2 * kk + (lane >> 5)) ^ swz) * 16);
    auto x_frag = [&](int it, int kk, int i) {
        return *reinterpret_cast<const bf16x8_t*>(smem + (it & 1) * XSTAGE + (kk >> 2) * (BM * 128) + (wm * WTM + i * 32) * 128 + frag_off[kk & 3]);
    };
    auto w_frag = [&](int it, int kk, int j) {
        return *reinterpret_cast<const bf16x8_t*>(wstages + (it & 1) * WSTAGE + (kk >> 2) * (BN * 128) + (wn * WTN + j * 32) * 128 + frag_off[kk & 3]);
    };

    uint32_t* const spoiled = reinterpret_cast<uint32_t*>(table + EpiLayout<BN, WGM>::TABLE_BYTES);
    if (tid < BM / 32) spoiled[tid] = 0u;

    // ---- prologue (what the epilogue needs from memory is fetched here too, beside the first requests)
    const long long inputs = 2ll * p.B * p.d_in + 4ll * p.n_active * p.K;
    const TileColumns cols = tile_columns(n0, BN, p.active, p.n_active, p.d_out, line_run(p.B, p.d_out, inputs, EpiLayout<BN, WGM>::LINE_RUN, BN >= 256 ? 77.0f : 46.5f));
    load_list(0);
#pragma unroll
    for (int q = 0; q < XP; ++q) issue_piece(0, q);
    fill_table<BN, WGM, NWAVES * 64>(table, cols.base, cols, n0, p.active, p.bias);
    if (!DIRECT) store_x(0);
    wait_loads<0>();
    build(0);
    lds_barrier();

    // The build of it + 1 stands before or behind the multiplications of it.
    bf16x8_t a[2][TM], b[2][TN];
    constexpr int N_MMA = TM * TN, N_FRAG = TM + TN, N_READ = (N_MMA + 1) / 2;
    auto read_frag = [&](int f, int it, int kk, int set) {   // in the order the products take them: a[0], the b's, the other a's
        if (f >= 1 && f <= TN) b[set][f - 1] = w_frag(it, kk, f - 1);
        else a[set][f ? f - TN : 0] = x_frag(it, kk, f ? f - TN : 0);
    };
#pragma unroll
    for (int f = 0; f < N_FRAG; ++f) read_frag(f, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(a[0][i]));
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(b[0][j]));
    const bool early = NWAVES > 4 && wv < NWAVES / 2;
    for (int it = 0; it < n_it; ++it) {
        const bool next = it + 1 < n_it;
        if (NWAVES > 4) {
            if (early) __builtin_amdgcn_s_setprio(0); else __builtin_amdgcn_s_setprio(1);
        }
        if (early && next) {
            build(it + 1);
        }
        if (!DIRECT && next) {
#pragma unroll
            for (int q = 0; q < XP; ++q) issue_piece(it + 1, q);
        }
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            const bool last = kk + 1 == KSTEPS;
            if (last) {
                if (NWAVES > 4) {
                    if (early) __builtin_amdgcn_s_setprio(1); else __builtin_amdgcn_s_setprio(0);
                }
                if (next) {
                    __builtin_amdgcn_s_waitcnt(kLgkm0);
                    if (!DIRECT) store_x(it + 1);
                    wait_loads<0>();   // x of it + 1; the list
                    if (!early) build(it + 1);
                }
                lds_barrier();   // stage it + 1 is complete, every fragment of stage it is in registers
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < N_MMA; ++m) {
#pragma unroll
                for (int f = m * N_FRAG / N_READ; f < (m + 1) * N_FRAG / N_READ && f < N_FRAG; ++f)
                    read_frag(f, last ? it + 1 : it, last ? 0 : kk + 1, (kk + 1) & 1);
                if (N_MMA > 1) acc[m / TN][m % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk & 1][m / TN], b[kk & 1][m % TN], acc[m / TN][m % TN], 0, 0, 0);
                if (DIRECT && kk == 0) {
#pragma unroll
                    for (int q = m * XP / N_MMA; q < (m + 1) * XP / N_MMA; ++q) issue_piece(it + 1, q);
                }
                if (N_MMA == 1) acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk & 1][0], b[kk & 1][0], acc[0][0], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    wait_loads<0>();   // x past the last iteration
    lds_barrier();
    store_tile<BM, BN, WGM, WGN, true>(smem, table, true, acc, cols, m0, n0, p.B, p.active, p.bias, p.d_out, p.y, p.act, spoiled);
    lds_barrier();
    uint32_t any = 0;
#pragma unroll
    for (int w = 0; w < BM / 32; ++w) any |= spoiled[w];
    if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)any) != 0, 0)) {
        constexpr int SUMS = BN * kMendRows * 4, AREA = (int)blocked_table_at<UA, BM, BN, WGM, WGN, CC>() - SUMS;
        wait_loads<0>();   // the stores above have reached memory; the function starts with a barrier
        mend_rows(p, smem, AREA, reinterpret_cast<float*>(smem + AREA), spoiled, BM, BN, WGM * WGN, m0, n0);
    }
}

template <int UA, bool DIRECT, int BM, int BN, int WGM, int WGN, int CC>
static srigl_status launch_tile(const BlockedArgs& args, int n_rows, hipStream_t st) {
    auto kern = k_fwd_blocked<UA, DIRECT, BM, BN, WGM, WGN, CC>;
    constexpr size_t lds = blocked_table_at<UA, BM, BN, WGM, WGN, CC>() + EpiLayout<BN, WGM>::TABLE_BYTES + BM / 8;
    static_assert(lds <= kLdsMax, "LDS");
    static LdsLimit lds_limit;
    if (lds_limit.ensure(kern, lds) != SRIGL_OK) return SRIGL_ERR_HIP;
    BlockedArgs p = args;
    p.tiles_m = (p.B + BM - 1) / BM;
    p.tiles_n = (n_rows + BN - 1) / BN;
    const long long n_wg = ((long long)p.tiles_m * p.tiles_n + kXcds - 1) / kXcds * kXcds;
    if (n_wg > 0x7fffffffLL) return SRIGL_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kern, dim3((unsigned)n_wg), dim3(WGM * WGN * 64), lds, st, p);
    return hip_ok(hipGetLastError());
}

// stored rows [p.n_base, p.n_base + n_rows) in one tile shape
template <int UA, bool DIRECT>
static srigl_status launch_shape(const BlockedArgs& p, int tile, int n_rows, hipStream_t st) {
    switch (tile) {
        case SRIGL_BLOCKED_256: return launch_tile<UA, DIRECT, 256, 256, 2, 4, 1>(p, n_rows, st);
        case SRIGL_BLOCKED_192: return launch_tile<UA, DIRECT, 256, 192, 4, 2, 1>(p, n_rows, st);
        case SRIGL_BLOCKED_128: return launch_tile<UA, DIRECT, 128, 128, 2, 2, 1>(p, n_rows, st);
        case SRIGL_BLOCKED_64: return launch_tile<UA, DIRECT, 64, 64, 2, 2, 2>(p, n_rows, st);
        default: return SRIGL_ERR_INVALID_ARG;
    }
}
static int blocked_tile_rows(int tile) { return tile == SRIGL_BLOCKED_64 ? 64 : tile == SRIGL_BLOCKED_128 ? 128 : tile == SRIGL_BLOCKED_192 ? 192 : 256; }

// A tile code names the shape in its low four bits; with a second shape in the next four, the stored rows are split: the first `code >>
// 8` tile columns in the first shape, the others in the second.
template <int UA, bool DIRECT>
static srigl_status launch_plan(BlockedArgs& p, int code, hipStream_t st) {
    const int first = code & 15, second = (code >> 4) & 15;
    const long long split = (long long)(code >> 8) * blocked_tile_rows(first);
    p.n_base = 0;
    if (second == 0) return code >> 8 ? SRIGL_ERR_INVALID_ARG : launch_shape<UA, DIRECT>(p, first, p.n_active, st);
    if (code < 0 || split <= 0 || split >= p.n_active || second > SRIGL_BLOCKED_192) return SRIGL_ERR_INVALID_ARG;
    if (const srigl_status rc = launch_shape<UA, DIRECT>(p, first, (int)split, st)) return rc;
    p.n_base = (int)split;
    return launch_shape<UA, DIRECT>(p, second, p.n_active - (int)split, st);
}

// Estimated time (us) of n stored rows in a tile shape, their share of the result `columns` wide.  Least squares on 99 layers and batches
// (200 to 4096 wide, 300 to 16192 stored rows, 80 to 98 % sparse, batches 64 to 2048): a round of workgroups costs a fixed part (prologue,
// epilogue), more with ablated neurons among the columns, and a part per 64 columns of x, more where rows of x go through registers; a
// compute unit holds one workgroup of the two large shapes, or two of the others.  The root mean square of the deviation is 4 to 5 % by shape,
// the shape of smallest estimate 0.3 % behind the fastest on average.
struct BlockedModel { double one, chunk_one, fixed, round, chunk, ragged, ablated, bytes; int slots; };
static double blocked_tile_us(int tile, int B, int n, double columns, int d_in, bool ablated) {
    static const BlockedModel kModels[] = {   // one, chunk_one: all workgroups at once, one to a compute unit
        {6.0, 0.268, 4.8, 0.7, 0.407, 0.113, 1.2, 1.1, 512},
        {8.5, 0.542, 6.2, 1.1, 0.885, 0.196, 3.4, 0.63, 512},
        {11.0, 1.190, 1.8, 9.2, 1.190, 0.226, 6.5, 0.50, 256},
        {10.6, 0.985, 2.3, 8.3, 0.985, 0.241, 1.3, 0.64, 256},
    };
    const BlockedModel& m = kModels[tile - 1];
    const int bn = blocked_tile_rows(tile), bm = bn == 192 ? 256 : bn, chunks = (d_in + kSegCols - 1) / kSegCols;
    const double w = (double)((B + bm - 1) / bm) * ((n + bn - 1) / bn), rounds = std::ceil(w / m.slots);
    const double more = (d_in % 8 != 0 ? m.ragged * chunks : 0.0) + (ablated ? m.ablated : 0.0);
    const double us = w <= 256 ? m.one + m.chunk_one * chunks + more : m.fixed + rounds * (m.round + m.chunk * chunks + more);
    return us + m.bytes * 1e-6 * B * columns;
}

// The tile code of smallest estimate.  The large shapes are also tried for their full rounds of workgroups only, with the stored rows that
// are left in the shape that suits those (3016 -> 9749 at batch 1765 in 256 and then 64 wide tiles 106 us, 135 in one shape).  Two launches take longer
// than their estimates' sum, 1 % with every neuron stored and 9 % with a fifth of them ablated (the second one's start waits for the first one's last rows
// and tables), so that they are taken where the sum promises 8 %.  On 256 points (128 products 768- to 4096-wide, 2560 to 16000 stored rows, batches 600 to
// 2048, with none and with a fifth of the neurons ablated) the code taken is 0.5 % behind the fastest of up to 10 on average, 13 % at worst; 0.6 % (15 %)
// where any promise counts, 1.1 % (16 %) with one shape only.
constexpr double kSplitGain = 0.92;
static int choose_blocked_tile(int B, int d_in, int n_active, int d_out, double* us) {
    constexpr int kShapes[] = {SRIGL_BLOCKED_64, SRIGL_BLOCKED_128, SRIGL_BLOCKED_192, SRIGL_BLOCKED_256};
    const bool ablated = n_active < d_out;
    const double per_row = (double)d_out / n_active;
    int best = 0;
    *us = 0.0;
    auto consider = [&](int code, double t) {
        if (best == 0 || t < *us) { best = code; *us = t; }
    };
    for (int s : kShapes) consider(s, blocked_tile_us(s, B, n_active, d_out, d_in, ablated));
    const double split_below = kSplitGain * *us;
    for (int first : {SRIGL_BLOCKED_256, SRIGL_BLOCKED_192}) {
        const int bn = blocked_tile_rows(first);
        const long long tiles_m = (B + 255) / 256, tiles_n = (n_active + bn - 1) / bn, rounds = tiles_m * tiles_n / 256;
        const long long columns = rounds * 256 / tiles_m;
        if (columns < 1 || columns >= tiles_n || columns >= (1 << 23)) continue;
        const int done = (int)columns * bn, left = n_active - done;
        const double head = blocked_tile_us(first, B, done, done * per_row, d_in, ablated);
        for (int s : kShapes)
            if (s != first) {
                const double both = head + blocked_tile_us(s, B, left, left * per_row, d_in, ablated);
                if (both < split_below) consider(first | s << 4 | (int)columns << 8, both);
            }
    }
    return best;
}

// Taken where its estimate is level with the gathering kernels' or ahead.  On 168 points (21 layers 200 to 4096 wide, batches of 16 to 2048) a call with
// its copy made is then 0.06 % slower on average than with the faster of the two forms throughout, 8 % at worst, one with the copy given 0.1 % (6 %).
constexpr double kBlockedMargin = 1.02;

// What making the copy adds to a call (us): between 4.1 (200 -> 300) and 14 (4096 -> 16384, K = 205) on those layers
static double block_terms_us(int n, int K) { return 4.3 + 2.9e-6 * n * (double)K; }

static bool blocked_fits(int n_active, int K, int d_in) {
    if (n_active <= 0 || K <= 0 || d_in < 8 || d_in > 65536) return false;
    const BlockedLayout l = blocked_layout(n_active, K, d_in);
    return (long long)l.groups * l.units_per_group < (1LL << 30);   // places of terms in 32 bits
}

double blocked_estimate_us(int B, int d_in, int n_active, int K, int d_out) {
    if (B <= 0 || n_active > d_out || K > d_in || !blocked_fits(n_active, K, d_in)) return 1e30;
    double us;
    choose_blocked_tile(B, d_in, n_active, d_out, &us);
    return us + block_terms_us(n_active, K);
}

}  // namespace srigl

using namespace srigl;

extern "C" {

size_t srigl_blocked_bytes(int32_t n_rows, int32_t K, int32_t d_in) {
    if (n_rows <= 0 || K <= 0 || d_in <= 0) return 0;
    return blocked_layout(n_rows, K, d_in).bytes;
}

static int32_t blocked_tile(int32_t B, int32_t d_in, int32_t n_active, int32_t K, int32_t d_out, bool with_copy) {
    if (B <= 0 || n_active > d_out || K > d_in || !blocked_fits(n_active, K, d_in)) return 0;
    struct Key { int32_t B, d_in, n_active, K, d_out, with_copy; };
    static thread_local DecisionCache<Key, int, 64> cache;
    return cache.get(Key{B, d_in, n_active, K, d_out, with_copy}, [&] {
        double us;
        const int tile = choose_blocked_tile(B, d_in, n_active, d_out, &us);
        if (with_copy) us += block_terms_us(n_active, K);
        return us < kBlockedMargin * condensed_estimate_us(B, d_in, n_active, K, d_out, true, n_active < d_out) ? tile : 0;
    });
}
int32_t srigl_blocked_tile(int32_t B, int32_t d_in, int32_t n_active, int32_t K, int32_t d_out) {
    return blocked_tile(B, d_in, n_active, K, d_out, false);
}
int32_t srigl_blocked_tile_with_copy(int32_t B, int32_t d_in, int32_t n_active, int32_t K, int32_t d_out) {
    return blocked_tile(B, d_in, n_active, K, d_out, true);
}

srigl_status srigl_block_terms(const void* W_c, const void* idx, int32_t idx_bits, const uint16_t* seg, int32_t n_rows, int32_t K,
                               int32_t d_in, void* blocked, size_t blocked_bytes, void* stream) {
    if (n_rows < 0 || K < 0 || d_in < 0 || K > d_in || (idx_bits != 32 && idx_bits != 16)) return SRIGL_ERR_INVALID_ARG;
    if (n_rows == 0 || K == 0) return SRIGL_OK;
    if (W_c == nullptr || idx == nullptr || seg == nullptr || blocked == nullptr || reinterpret_cast<uintptr_t>(blocked) % 16 != 0)
        return SRIGL_ERR_INVALID_ARG;
    if (!blocked_fits(n_rows, K, d_in)) return SRIGL_ERR_UNSUPPORTED;
    const BlockedLayout l = blocked_layout(n_rows, K, d_in);
    if (blocked_bytes < l.bytes) return SRIGL_ERR_CAPACITY;
    unsigned char* base = static_cast<unsigned char*>(blocked);
    auto launch = [&](auto kern, LdsLimit& lds_limit, size_t lds, auto* columns) {
        if (lds_limit.ensure(kern, lds) != SRIGL_OK) return SRIGL_ERR_HIP;
        hipLaunchKernelGGL(kern, dim3((unsigned)l.groups), dim3(kBuildThreads), lds, static_cast<hipStream_t>(stream), static_cast<const uint16_t*>(W_c),
                           columns, seg, srigl_seg_stride(d_in), n_rows, K, l.chunks, l.units_per_group, reinterpret_cast<uint32_t*>(base),
                           reinterpret_cast<uint4*>(base + l.table_bytes));
        return hip_ok(hipGetLastError());
    };
    const size_t tables = ((size_t)2 * (l.chunks + 1) + (size_t)kBlockRows * l.chunks + 2 * 64 * kBuildWaves) * 4, staged = tables + 16 * (size_t)l.units_per_group;
    static LdsLimit limit[4];
    const int32_t* wide = static_cast<const int32_t*>(idx);
    const uint16_t* narrow = static_cast<const uint16_t*>(idx);
    if (staged <= kLdsMax)
        return idx_bits == 32 ? launch(k_block_terms<int32_t, true>, limit[0], staged, wide) : launch(k_block_terms<uint16_t, true>, limit[1], staged, narrow);
    return idx_bits == 32 ? launch(k_block_terms<int32_t, false>, limit[2], tables, wide) : launch(k_block_terms<uint16_t, false>, limit[3], tables, narrow);
}

srigl_status srigl_blocked_linear_fwd(const void* x, int32_t B, int32_t d_in, const void* blocked, const void* W_c, const void* idx,
                                           int32_t idx_bits, const int32_t* active, int32_t n_active, int32_t K, const float* bias,
                                           int32_t d_out, float* y, srigl_activation act, int32_t tile, void* stream) {
    if (act != SRIGL_ACT_NONE && act != SRIGL_ACT_RELU && act != SRIGL_ACT_GELU) return SRIGL_ERR_INVALID_ARG;
    if (B < 0 || d_in < 0 || n_active < 0 || K < 0 || d_out < 0 || K > d_in || n_active > d_out || (idx_bits != 32 && idx_bits != 16))
        return SRIGL_ERR_INVALID_ARG;
    if (active == nullptr && n_active != d_out) return SRIGL_ERR_INVALID_ARG;
    if (!blocked_fits(n_active, K, d_in)) return SRIGL_ERR_UNSUPPORTED;
    if (B == 0) return SRIGL_OK;
    if (x == nullptr || blocked == nullptr || W_c == nullptr || idx == nullptr || y == nullptr || reinterpret_cast<uintptr_t>(blocked) % 16 != 0)
        return SRIGL_ERR_INVALID_ARG;
    const BlockedLayout l = blocked_layout(n_active, K, d_in);
    BlockedArgs p;
    const unsigned char* base = static_cast<const unsigned char*>(blocked);
    p.x = static_cast<const uint16_t*>(x); p.table = reinterpret_cast<const uint32_t*>(base); p.lists = base + l.table_bytes;
    p.W_c = static_cast<const uint16_t*>(W_c); p.idx = idx; p.active = active; p.bias = bias; p.y = y;
    p.B = B; p.d_in = d_in; p.n_active = n_active; p.K = K; p.d_out = d_out; p.idx_u16 = idx_bits == 16; p.act = (int)act;
    const bool direct = d_in % 8 == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    // a block's mean number of terms against the 256 a load brings: with up to 230 one load ahead is 0 to 7 % faster (of 132 points on layers of
    // 546 to 4096 columns), from 256 on two are, by up to 20 % (4096 -> 4096 with 400 terms a block, batch 1024: 83.4 and 66.6 us)
    const bool two = 2048.0 * K / d_in > 240.0;
    hipStream_t st = static_cast<hipStream_t>(stream);
    double us;
    if (tile == 0) tile = choose_blocked_tile(B, d_in, n_active, d_out, &us);
    if (direct) return two ? launch_plan<2, true>(p, tile, st) : launch_plan<1, true>(p, tile, st);
    return two ? launch_plan<2, false>(p, tile, st) : launch_plan<1, false>(p, tile, st);
}

}  // extern "C"
