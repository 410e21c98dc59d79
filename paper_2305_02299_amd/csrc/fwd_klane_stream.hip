// KLANE for layers whose terms have to be streamed (gfx950): the small-batch formulation of fwd.hip (lanes share a stored row; Alg. 1 of
// arXiv 2305.02299 with the bias of Sec. 4.4 and the ablated neurons of Sec. 3.1 step 4) with the activations in LDS and two workgroups of
// eight wavefronts per compute unit, each wavefront with four stored rows of one batch row.
//
// The gathering form starts thousands of workgroups of four wavefronts, a stored row each, and takes x from the vector caches, which serve
// a wavefront's 64 scattered words in about as many clocks: 4096 -> 16384 bf16 (13108 stored rows, K = 205, 10.7 MB) at one batch row
// 7.2 us (a call 8.1).  Here a wavefront requests the terms of its four rows, 4 consecutive ones per lane and row in one load per array, before it
// stages its share of x, and the LDS serves 64 scattered words in some ten clocks (a call 5.5).  What bounds it: the start of the wavefronts, the
// trip to memory for the terms and the sums over the lanes, 3.6 us together, and the terms' way in.
#include "srigl_internal.h"
#include "fwd_rowlane.inl"

namespace srigl {

constexpr int kStreamTerms = 4;   // consecutive terms of a lane
constexpr int kStreamChunk = kStreamTerms * kWave;

template <typename T> struct Four { T v[4]; };
__device__ __forceinline__ Four<float> load_four(const float* p) {
    struct __attribute__((packed, aligned(4))) F4 { float v[4]; };
    const F4 f = *reinterpret_cast<const F4*>(p);
    return {{f.v[0], f.v[1], f.v[2], f.v[3]}};
}
__device__ __forceinline__ Four<int32_t> load_four(const int32_t* p) {
    struct __attribute__((packed, aligned(4))) I4 { int32_t v[4]; };
    const I4 f = *reinterpret_cast<const I4*>(p);
    return {{f.v[0], f.v[1], f.v[2], f.v[3]}};
}
__device__ __forceinline__ Four<uint16_t> load_four(const uint16_t* p) {
    struct __attribute__((packed, aligned(2))) U2 { uint32_t x, y; };
    const U2 f = *reinterpret_cast<const U2*>(p);
    return {{(uint16_t)f.x, (uint16_t)(f.x >> 16), (uint16_t)f.y, (uint16_t)(f.y >> 16)}};
}

template <typename XT, typename IT>
__global__ __launch_bounds__(kStreamWaves* kWave, sizeof(XT) + sizeof(IT) < 8 ? 8 : 6) void k_fwd_klane_stream(const XT* __restrict__ x, int d_in, const XT* __restrict__ W_c,
                                                           const IT* __restrict__ idx, const int32_t* __restrict__ active, int n_active, int K,
                                                           const float* __restrict__ bias, int d_out, float* __restrict__ y, int act) {
    extern __shared__ float xs[];   // the columns, then one of zeros for lanes without a term
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    constexpr int kThreads = kStreamWaves * kWave;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (groups of stored rows, batch rows, 1), or (8, batch rows, groups / 8): consecutive workgroups go to different XCDs
    const unsigned b = blockIdx.y;
    const int s0 = (int)((blockIdx.z * 8 + blockIdx.x) * kStreamWaves + wv) * kStreamRows;   // (may lie past the last row)
    if (s0 - wv * kStreamRows >= n_active) return;   // (the whole workgroup)
    const XT* const xr = x + (size_t)b * d_in;
    float* const yr = y + (size_t)b * d_out;
    // after the sums over lanes, 16-lane group g of the wavefront holds row s0 + own (0, 2, 1, 3)
    const int own = ((lane >> 5) | ((lane >> 3) & 2));

    Four<XT> w[kStreamRows];
    Four<IT> c[kStreamRows];
    auto request = [&](int k0, Four<XT> (&wr)[kStreamRows], Four<IT> (&cr)[kStreamRows]) {   // terms k0 + 4 lane and on
        const int at = min(k0 + kStreamTerms * lane, K - kStreamTerms);   // (K >= 4: host; a term of the lane before is dropped where it is used)
#pragma unroll
        for (int r = 0; r < kStreamRows; ++r) {
            const size_t row = (size_t)min(s0 + r, n_active - 1) * (size_t)K;
            wr[r] = load_four(W_c + row + at);
            cr[r] = load_four(idx + row + at);
        }
    };
    request(0, w, c);
    const int s = min(s0 + own, n_active - 1);
    const int col = active ? active[s] : s, prev = s > 0 ? (active ? active[s - 1] : s - 1) : -1;

    // ---- x: four loads per thread in flight ----
    for (int j0 = tid; j0 < d_in; j0 += 4 * kThreads) {
        XT v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = xr[min(j0 + u * kThreads, d_in - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j0 + u * kThreads < d_in) xs[j0 + u * kThreads] = rl_to_f32<XT>(v[u]);
    }
    if (tid == 0) xs[d_in] = 0.0f;
    const bool stored = col >= 0 && col < d_out;
    const float bv = bias && stored ? bias[col] : 0.0f;
    __syncthreads();
    if (s0 >= n_active) return;

    float acc[kStreamRows] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = 0; k0 < K; k0 += kStreamChunk) {
        Four<XT> wn[kStreamRows];
        Four<IT> cn[kStreamRows];
        if (k0 + kStreamChunk < K) request(k0 + kStreamChunk, wn, cn);   // on their way behind these
        const int first = k0 + kStreamTerms * lane, at = min(first, K - kStreamTerms);
        // (the reads of two rows together: left to the compiler they came one at a time, each waited for, in some of its arrangements of this kernel: 3072 -> 448,
        // K = 492 at eight rows 4.7 us for 4.3)
#pragma unroll
        for (int r0 = 0; r0 < kStreamRows; r0 += 2) {
            float xv[2][kStreamTerms];
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int u = 0; u < kStreamTerms; ++u)   // (no real term where first >= K)
                    xv[r][u] = xs[at + u >= first ? min((unsigned)c[r0 + r].v[u], (unsigned)d_in - 1u) : (unsigned)d_in];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int u = 0; u < kStreamTerms; ++u)
                    acc[r0 + r] = fmaf(at + u >= first ? rl_to_f32<XT>(w[r0 + r].v[u]) : 0.0f, xv[r][u], acc[r0 + r]);
        }
#pragma unroll
        for (int r = 0; r < kStreamRows; ++r) { w[r] = wn[r]; c[r] = cn[r]; }
    }
    // registers are paired, lanes 0-31 of the sum taking the first and lanes 32-63 the second register's, and again between the odd and
    // even 16-lane rows; then the sum around each 16-lane row
    const auto h0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[0]), __float_as_uint(acc[1]), false, false);
    const auto h1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[2]), __float_as_uint(acc[3]), false, false);
    const float u0 = __uint_as_float(h0[0]) + __uint_as_float(h0[1]), u1 = __uint_as_float(h1[0]) + __uint_as_float(h1[1]);
    const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(u0), __float_as_uint(u1), false, false);
    float v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    v += row_ror<1>(v);
    const bool mine = s0 + own < n_active;
    if (mine && (lane & 15) == 0 && stored) yr[col] = act == SRIGL_ACT_NONE ? v + bv : apply_act(v + bv, act);
    if (active == nullptr) return;
    // Ablated columns hold their bias: the run in front of each row's column, and the one behind the last row's.  The 16 lanes of a row write
    // its first 16 columns; longer runs are the whole wavefront's, a load of the bias ahead of each store.  By 16 lanes, one load after the
    // other, a run cost 5 ns a column: 1565 -> 7698, K = 140 at two batch rows with 769 neighbours ablated at either end 9.8 us (the gathering
    // form 6.8), now 5.4; 1528 -> 4680, K = 305 at two with 468 7.9 (5.6), now 5.0.
    // (The short runs' bias asked for ahead of the barrier spilled registers: 3 to 13 % slower.)
    constexpr int kOwn = 16;
    auto put = [&](int q, float raw) { yr[q] = act == SRIGL_ACT_NONE ? raw : apply_act(raw, act); };
    const int from = max(prev + 1, 0), to = mine ? min(col, d_out) : from;
    if (from + (lane & 15) < to) put(from + (lane & 15), rl_bias_at(bias, from + (lane & 15)));
    const bool last = s0 + kStreamRows >= n_active;   // (the last row's column then is that of lane 63: rows past it were clamped to it)
    if (!last && !__any(to - from > kOwn)) return;
    const int behind = max(__builtin_amdgcn_readlane(col, kWave - 1) + 1, 0);
#pragma unroll 1
    for (int g = 0; g < kStreamRows + (last ? 1 : 0); ++g) {
        const int lo = g < kStreamRows ? __builtin_amdgcn_readlane(from, 16 * g) + kOwn : behind;
        const int hi = g < kStreamRows ? __builtin_amdgcn_readlane(to, 16 * g) : d_out;
        if (lo >= hi) continue;
        float next = rl_bias_at(bias, min(lo + lane, hi - 1));
#pragma unroll 1
        for (int q = lo + lane; q < hi; q += kWave) {
            const float raw = next;
            next = rl_bias_at(bias, min(q + kWave, hi - 1));
            put(q, raw);
        }
    }
}

template <typename XT, typename IT>
static srigl_status launch_stream_t(const FwdArgs& a, bool by_xcd, hipStream_t st) {
    auto kern = k_fwd_klane_stream<XT, IT>;
    static LdsLimit lds_limit;
    const size_t lds = (size_t)(a.d_in + 1) * sizeof(float);
    if (lds_limit.ensure(kern, lds) != SRIGL_OK) return SRIGL_ERR_HIP;
    const unsigned groups = (unsigned)stream_groups(a);   // (at most 64 batch rows and 32768 rows in all: stream_ahead)
    const dim3 grid = by_xcd ? dim3(8, (unsigned)a.B, (groups + 7) / 8) : dim3(groups, (unsigned)a.B);
    hipLaunchKernelGGL(kern, grid, dim3(kStreamWaves * kWave), lds, st, (const XT*)a.x, a.d_in, (const XT*)a.W_c, (const IT*)a.idx, a.active,
                       a.n_active, a.K, a.bias, a.d_out, a.y, a.act);
    return hip_ok(hipGetLastError());
}

// The form of the small-batch kernel where there are terms to stream (over the batch 1.6 M, or 0.8 M per chunk of 256 terms of a row, whose chunks follow one
// another), four workgroups to a compute unit hold all of them, and a row fills half of its wavefront's lanes or more (3142 -> 16707, K = 314 at one batch
// row 11.1 -> 7.5 us, 3072 -> 768 with 538 stored, K = 307 at 16 6.9 -> 6.2, 4052 -> 4395 bf16, K = 202 at 3 6.6 -> 5.2).  Of 557 points where it may run (300
// to 4096 wide, 128 to 16384 stored rows, batches 2 to 64, both types and index widths) a call takes it on 401, there in 0.86 of the gathering form's time
// on average; on a few it is 3 to 14 % behind (2559 -> 407, 326 stored, K = 281 at 24 rows 6.2 against 5.4: a second chunk for 25 terms).  From 1.0 M terms on
// some would lose 9 to 21 % (3912 -> 3106, K = 391 at 1; 3680 -> 1412, K = 736), with rows that fill fewer lanes 10 % (1011 -> 1884, K = 101 at 12).
bool stream_ahead(const FwdArgs& a) {
    if (a.B <= 0 || a.B > 64 || a.n_active <= 0 || a.K < kStreamTerms || (size_t)(a.d_in + 1) * sizeof(float) > kLdsMax / 4) return false;
    const int chunks = (a.K + kStreamChunk - 1) / kStreamChunk;
    const double terms = (double)a.n_active * a.K * a.B;
    return terms >= 0.8e6 * std::max(2, chunks) && (long long)a.n_active * a.B <= 4 * 256 * kStreamWaves * kStreamRows && 2 * a.K >= chunks * kStreamChunk;
}

static double stream_bytes(const FwdArgs& a) { return (double)a.n_active * a.K * ((a.x_bf16 ? 2 : 4) + (a.idx_u16 ? 2 : 4)); }
// Whether the grid makes every batch row's workgroup of a group of stored rows go to the same XCD, whose L2 then fetches the group's terms once and no
// other's; otherwise a batch row's workgroups go round the XCDs from where the row before ended, which comes to the same where the groups are a multiple of
// eight, and else each meets all terms.  Taken from 2 MB of terms on (level in a loop over one layer up to 4 MB, but two layers' terms then share an L2:
// 915 -> 2745 -> 915 at 11 rows 13.8 -> 11.7 us; 497 points: 0.90 of the time at 8 to 12 MB, 0.68 beyond 20, 2834 -> 3423, K = 481 at four rows 9.9 -> 7.5 us) where
// that keeps the XCDs within a ninth of equal work (172 stored rows, six groups, up to 1.3 times slower).
static bool stream_by_xcd(const FwdArgs& a) {
    const int groups = stream_groups(a);
    return groups % 8 != 0 && stream_bytes(a) > 2e6 && 9 * ((groups + 7) / 8 * 8) <= 10 * groups;
}

// Estimated time (us), for the comparison with the batched kernels: the columns of x that the workgroups stage, the places that the chunks of all
// rows take, the chunks after the first, and the bytes of the terms that the L2s fetch beyond their 32 MB.  Non-negative least squares on the relative
// error of 497 launches on which stream_ahead holds (300 to 4096 wide, 128 to 16384 stored rows, batches 2 to 64, both types and index widths,
// random ablation, cached operands): standard deviation 7.5 %, worst -22 and +21 %.
double stream_estimate_us(const FwdArgs& a) {
    const double chunks = (a.K + kStreamChunk - 1) / kStreamChunk;
    const double bytes = stream_bytes(a), fetched = stream_by_xcd(a) || stream_groups(a) % 8 == 0 ? bytes : bytes * std::min(a.B, 8);
    return 3.40 + 0.460e-6 * stream_groups(a) * a.B * (double)a.d_in + 0.282e-6 * a.n_active * a.B * chunks * kStreamChunk +
           0.098e-6 * std::max(0.0, fetched - 32e6) + 0.28 * (chunks - 1);
}

srigl_status launch_fwd_stream(const FwdArgs& a, hipStream_t st) {
    const bool by_xcd = stream_by_xcd(a);
    if (a.idx_u16) return a.x_bf16 ? launch_stream_t<uint16_t, uint16_t>(a, by_xcd, st) : launch_stream_t<float, uint16_t>(a, by_xcd, st);
    return a.x_bf16 ? launch_stream_t<uint16_t, int32_t>(a, by_xcd, st) : launch_stream_t<float, int32_t>(a, by_xcd, st);
}

}  // namespace srigl
