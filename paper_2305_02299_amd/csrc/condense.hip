// check_fanin and condense kernels (gfx950).
//
// Constant fan-in invariant: Fig. 1a / Sec. 3.1 of arXiv 2305.02299 (every neuron that is not
// ablated keeps exactly K incoming weights).  Condensed form: App. E (an [n][k] array of values and
// an [n][k] array of column indices), with ablated neurons dropped (Sec. 4.4).
//
// All steps are bandwidth work over the mask (1 byte per weight) and, for the compaction, the dense
// weights: one wavefront owns one row, lanes read consecutive mask bytes, and positions inside the row
// come from ballots and prefix popcounts (no atomics).
#include "srigl_internal.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <type_traits>

// Scratch of srigl_condense_static (the condense call for callers that cannot allocate): the rows' bits that srigl_condense
// keeps in its workspace argument.  One copy per GPU, held until the process ends.  The name is a host-side
// stand-in: kernels get the device address that hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[2 * sizeof(int32_t) * (size_t)SRIGL_STATIC_MAX_ROWS + 256];

namespace srigl {

constexpr int kRowsPerBlock = 4;   // 4 wavefronts of 64 lanes, one row each

__device__ __forceinline__ uint32_t lanes_below(uint64_t ballot) {
    // number of set bits of `ballot` that belong to lanes below this one
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
}

// 4 mask bytes of row `m` starting at column `col` (bytes past d_in read as 0), one byte per 8 bits.
__device__ __forceinline__ uint32_t load_mask4(const uint8_t* __restrict__ m, int col, int d_in, bool aligned4) {
    if (col + 4 <= d_in) {
        if (aligned4) return *reinterpret_cast<const uint32_t*>(m + col);
        return (uint32_t)m[col] | ((uint32_t)m[col + 1] << 8) | ((uint32_t)m[col + 2] << 16) | ((uint32_t)m[col + 3] << 24);
    }
    uint32_t v = 0;
    for (int p = 0; p < 4; ++p)
        if (col + p < d_in) v |= (uint32_t)m[col + p] << (8 * p);
    return v;
}

// per-byte non-zero flags of a 32-bit word: bit 7 of each byte
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t w) {
    return (((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u;
}

// counts[r] = number of non-zero mask bytes in row r
__global__ __launch_bounds__(kRowsPerBlock* kWave) void k_row_count(const uint8_t* __restrict__ mask, int n_rows,
                                                                  int d_in, int32_t* __restrict__ counts) {
    const int lane = threadIdx.x & (kWave - 1);
    const int r = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    if (r >= n_rows) return;
    const uint8_t* m = mask + (size_t)r * d_in;
    const bool aligned4 = ((reinterpret_cast<uintptr_t>(m) & 3) == 0);
    int c = 0;
    for (int col = lane * 4; col < d_in; col += kWave * 4) c += __popc(nonzero_bytes(load_mask4(m, col, d_in, aligned4)));
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, kWave);
    if (lane == 0) counts[r] = c;
}

// Index mode: counts[r] = K if row r of idx is in range and strictly ascending, else -1; seg rows.
__global__ __launch_bounds__(kRowsPerBlock* kWave) void k_check_idx(const int32_t* __restrict__ idx, int n_rows, int K,
                                                                  int d_in, int32_t* __restrict__ counts,
                                                                  uint16_t* __restrict__ seg, int seg_stride) {
    const int lane = threadIdx.x & (kWave - 1);
    const int r = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    if (r >= n_rows) return;
    const int32_t* row = idx + (size_t)r * K;
    bool ok = true;
    for (int k = lane; k < K; k += kWave) {
        int32_t cur = row[k];
        if (cur < 0 || cur >= d_in) ok = false;
        if (k > 0 && row[k - 1] >= cur) ok = false;
    }
    const bool row_ok = (__ballot(!ok) == 0ull);
    if (lane == 0) counts[r] = row_ok ? K : -1;
    if (seg == nullptr) return;
    uint16_t* sg = seg + (size_t)r * seg_stride;
    if (!row_ok || K == 0) {
        for (int c = lane; c < seg_stride; c += kWave) sg[c] = 0;
        return;
    }
    // ascending row: seg[c] = position of the first index >= 64*c.  The lane that owns position k
    // fills the entries c in (prev/64, cur/64]; the tail entries hold K.
    for (int k = lane; k < K; k += kWave) {
        const int cur = row[k];
        const int lo = (k == 0) ? 0 : row[k - 1] / kSegCols + 1;
        const int hi = cur / kSegCols;
        for (int c = lo; c <= hi; ++c) sg[c] = (uint16_t)k;
    }
    const int last = row[K - 1] / kSegCols + 1;
    for (int c = last + lane; c < seg_stride; c += kWave) sg[c] = (uint16_t)K;
}

// One workgroup.  Reads counts[], decides K, writes the report of a check.
// index_mode: counts hold K (valid) or -1 (bad); every valid row is "stored" even when K == 0.
__global__ __launch_bounds__(1024) void k_scan_rows(const int32_t* __restrict__ counts, int n_rows, int K_expected,
                                                    int index_mode, srigl_report* __restrict__ report) {
    __shared__ int s_wave[16], s_wave_bad[16];
    __shared__ int s_k, s_min;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
    const int nthreads = blockDim.x, nwaves = nthreads >> 6;

    if (tid == 0) s_min = 0x7fffffff;
    __syncthreads();
    int K = K_expected;
    if (K_expected < 0) {   // fan-in of the first non-empty row
        int first = 0x7fffffff;
        for (int r = tid; r < n_rows; r += nthreads)
            if (counts[r] > 0) { first = r; break; }
        for (int off = 32; off > 0; off >>= 1) first = min(first, __shfl_xor(first, off, kWave));
        if (lane == 0 && first != 0x7fffffff) atomicMin(&s_min, first);
        __syncthreads();
        if (tid == 0) s_k = (s_min == 0x7fffffff) ? 0 : counts[s_min];
        __syncthreads();
        K = s_k;
        __syncthreads();
        if (tid == 0) s_min = 0x7fffffff;
        __syncthreads();
    }
    int n_stored = 0, n_bad = 0, first_bad = 0x7fffffff;
    for (int r = tid; r < n_rows; r += nthreads) {
        const int c = counts[r];
        const bool bad = index_mode ? c != K : (c != 0 && c != K);
        n_stored += (c == K && (index_mode || c > 0)) ? 1 : 0;
        if (bad) { ++n_bad; first_bad = min(first_bad, r); }
    }
    for (int off = 32; off > 0; off >>= 1) {
        n_stored += __shfl_xor(n_stored, off, kWave);
        n_bad += __shfl_xor(n_bad, off, kWave);
        first_bad = min(first_bad, __shfl_xor(first_bad, off, kWave));
    }
    if (lane == 0) {
        s_wave[wv] = n_stored;
        s_wave_bad[wv] = n_bad;
        if (first_bad != 0x7fffffff) atomicMin(&s_min, first_bad);
    }
    __syncthreads();
    if (tid == 0) {
        int n = 0, t = 0;
        for (int w = 0; w < nwaves; ++w) { n += s_wave[w]; t += s_wave_bad[w]; }
        report->K = K;
        report->n_active = n;
        report->n_bad_rows = t;
        report->first_bad_row = (s_min == 0x7fffffff) ? -1 : s_min;
        report->status = t > 0 ? (index_mode ? SRIGL_ERR_INDEX_RANGE : SRIGL_ERR_FANIN) : SRIGL_OK;
        report->reserved[0] = report->reserved[1] = report->reserved[2] = 0;
    }
}

// ---- condense: two launches ----
// k_row_flags reads the mask once and leaves two bits per row (stored: K kept weights; bad: neither 0 nor K).  k_compact_rows
// numbers its rows from those bits by itself (a row's slot is the number of stored rows in front of it: 2 KB of bits for
// 16384 rows, read beside the row's mask), so no launch of one workgroup stands between the two passes over the mask: that
// scan took 5 us at 3072 rows and 31 us at 16384, 128 and 16 times what its bytes need.
constexpr int kFlagRows = 8;       // rows (wavefronts) per workgroup of k_row_flags: one byte of each bit array
constexpr int kMaskCols = 16;      // mask bytes per lane and load
constexpr int kBatchCols = 4 * kWave * kMaskCols;   // columns whose mask bytes a wavefront has in flight

// Kept columns among the kMaskCols columns this lane looks at: `first` (the first of them) and a bit per column.  Rows of any
// alignment: the last lane with columns of the row reads the row's last 16 bytes and drops the ones its neighbour has.
struct MaskPiece {
    uint4 v;
    int first, drop;   // drop: leading columns that are not this lane's (>= 16: none is)
};
__device__ __forceinline__ MaskPiece load_piece(const uint8_t* __restrict__ m, int col, int d_in) {
    MaskPiece p;
    p.first = min(col, d_in - kMaskCols);
    p.drop = col - p.first;
    __builtin_memcpy(&p.v, m + p.first, kMaskCols);   // one 16-byte load at any alignment
    return p;
}
__device__ __forceinline__ uint32_t kept_bits(const MaskPiece& p) {
    // bit 7 of each byte -> four adjacent bits
    auto four = [](uint32_t w) { return ((nonzero_bytes(w) >> 7) * 0x10204080u) >> 28; };
    const uint32_t all = four(p.v.x) | (four(p.v.y) << 4) | (four(p.v.z) << 8) | (four(p.v.w) << 12);
    return p.drop >= kMaskCols ? 0u : (all >> p.drop) << p.drop;
}
// rows shorter than one piece
__device__ __forceinline__ uint32_t kept_bits_short(const uint8_t* __restrict__ m, int col, int d_in) {
    uint32_t b = 0;
    if (col == 0)
        for (int c = 0; c < d_in; ++c) b |= (m[c] != 0 ? 1u : 0u) << c;
    return b;
}

__global__ __launch_bounds__(kFlagRows* kWave) void k_row_flags(const uint8_t* __restrict__ mask, int n_rows, int d_in, int K,
                                                              uint8_t* __restrict__ stored, uint8_t* __restrict__ bad) {
    __shared__ int cnt[kFlagRows];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
    const int r = blockIdx.x * kFlagRows + wv;
    int c = 0;
    if (r < n_rows) {
        const uint8_t* m = mask + (size_t)r * d_in;
        if (d_in >= kMaskCols) {
            for (int col0 = 0; col0 < d_in; col0 += kBatchCols) {
                MaskPiece p[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (col0 + u * kWave * kMaskCols < d_in) p[u] = load_piece(m, col0 + (u * kWave + lane) * kMaskCols, d_in);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (col0 + u * kWave * kMaskCols < d_in) c += __popc(kept_bits(p[u]));
            }
        } else {
            c = __popc(kept_bits_short(m, lane, d_in));
        }
        for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, kWave);
    }
    if (lane == 0) cnt[wv] = r < n_rows ? c : 0;
    __syncthreads();
    if (threadIdx.x < kWave) {
        const int n = lane < kFlagRows ? cnt[lane] : 0;
        const uint64_t is_stored = __ballot(n > 0 && n == K), is_bad = __ballot(n != 0 && n != K);
        if (lane == 0) {
            stored[blockIdx.x] = (uint8_t)is_stored;
            bad[blockIdx.x] = (uint8_t)is_bad;
        }
    }
}

// The same for a caller that adds the rows up itself: a workgroup goes through `groups` groups of 32 rows, two rows to a wavefront, and leaves a word in host
// memory, how many of its rows are stored and bad and the first bad one, beside a mark.  Every word is a write of its own over the bus, 20 to 30 ns at its end (with one
// for every eight rows 384 of them took 7 us on 768 -> 3072), so that there are at most kCountWords.
constexpr unsigned long long kCounted = 1ull << 63;
constexpr int kCountWords = 128, kCountRows = 32, kCountWaves = 16;
__global__ __launch_bounds__(kCountWaves* kWave) void k_row_counts(const uint8_t* __restrict__ mask, int n_rows, int d_in, int K, int groups,
                                                                 uint32_t* __restrict__ stored, uint32_t* __restrict__ bad,
                                                                 unsigned long long* __restrict__ to_host) {
    constexpr int ROWS = kCountRows / kCountWaves, AHEAD = 4;   // rows of a wavefront; loads of each in flight
    __shared__ int cnt[2][kCountRows];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
    unsigned n_stored = 0, n_bad = 0, first_bad = 0;
    for (int g = 0; g < groups; ++g) {
        const int group = blockIdx.x * groups + g, r0 = group * kCountRows + wv * ROWS;
        if (group * kCountRows >= n_rows) break;
        uint32_t c[ROWS] = {};
        if (d_in >= kMaskCols) {
            for (int col0 = 0; col0 < d_in; col0 += AHEAD * kWave * kMaskCols) {
                MaskPiece p[ROWS][AHEAD];
#pragma unroll
                for (int i = 0; i < ROWS; ++i)
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u)
                        if (r0 + i < n_rows && col0 + u * kWave * kMaskCols < d_in)
                            p[i][u] = load_piece(mask + (size_t)(r0 + i) * d_in, col0 + (u * kWave + lane) * kMaskCols, d_in);
#pragma unroll
                for (int i = 0; i < ROWS; ++i)
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u)
                        if (r0 + i < n_rows && col0 + u * kWave * kMaskCols < d_in) c[i] += __popc(kept_bits(p[i][u]));
            }
        } else {
#pragma unroll
            for (int i = 0; i < ROWS; ++i)
                if (r0 + i < n_rows) c[i] = __popc(kept_bits_short(mask + (size_t)(r0 + i) * d_in, lane, d_in));
        }
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const uint32_t n = wave_prefix(c[i]);
            if (lane == kWave - 1) cnt[g & 1][wv * ROWS + i] = (int)n;
        }
        __syncthreads();   // (two places in turn: one barrier)
        if (threadIdx.x < kWave) {
            const int n = lane < kCountRows ? cnt[g & 1][lane] : 0;
            const uint32_t is_stored = (uint32_t)__ballot(n > 0 && n == K), is_bad = (uint32_t)__ballot(n != 0 && n != K);
            if (lane == 0) {
                stored[group] = is_stored;
                bad[group] = is_bad;
            }
            if (is_bad && n_bad == 0) first_bad = g * kCountRows + __builtin_ctz(is_bad);
            n_stored += __popc(is_stored);
            n_bad += __popc(is_bad);
        }
    }
    if (threadIdx.x == 0)
        __hip_atomic_store(&to_host[blockIdx.x], kCounted | (unsigned long long)first_bad << 42 | (unsigned long long)n_bad << 21 | n_stored, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

// One wavefront per row: ordered stream compaction of the kept columns.  T = bit container of one weight (uint32_t for fp32,
// uint16_t for bf16).  The row's kept columns are listed in LDS first (a lane's columns go to consecutive places behind those
// of the lanes below it), then the lanes take the list's entries in turn, so that idx, W_c, the streaming copy (see
// PackedLayout; places behind the K-th term up to the next multiple of four get weight bits 0 and index 0) and the weights'
// gather all run over consecutive terms: three store instructions per 64 terms, where a lane storing its own columns issued
// three per column position.  What bounds it: the mask a second time and the 128-byte lines of W that hold a kept weight (at
// 5 % density nearly all of W).  4096 x 16384 bf16, 20 % of the rows ablated: 161 us for the whole call on the GPU before.
// Workgroup 0 also writes the report, if there is one to write.
template <typename T>
__global__ __launch_bounds__(kRowsPerBlock* kWave) void k_compact_rows(const T* __restrict__ W, const uint8_t* __restrict__ mask,
                                                                     int d_out, int d_in, int K, int cap_rows,
                                                                     const uint8_t* __restrict__ stored, const uint8_t* __restrict__ bad,
                                                                     T* __restrict__ W_c, int32_t* __restrict__ idx, int32_t* __restrict__ active,
                                                                     uint16_t* __restrict__ seg, int seg_stride,
                                                                     unsigned char* __restrict__ packed, PackedLayout pl, int rows_per_block,
                                                                     int list_cap, srigl_report* __restrict__ report) {
    extern __shared__ uint16_t lists[];   // [kRowsPerBlock][list_cap]: kept columns of a row, counted from the batch's first column
    __shared__ int part[kRowsPerBlock], part_bad[kRowsPerBlock], part_first[kRowsPerBlock];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
    const int row0 = blockIdx.x * rows_per_block;
    const uint32_t* const stored_w = reinterpret_cast<const uint32_t*>(stored);
    const uint32_t* const bad_w = reinterpret_cast<const uint32_t*>(bad);
    const int n_words = (d_out + 31) / 32;

    // the first row's mask goes out before the bits are waited for
    MaskPiece ahead[4];
    const bool pieces = d_in >= kMaskCols;
    if (pieces && row0 + wv < d_out) {
        const uint8_t* m = mask + (size_t)(row0 + wv) * d_in;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u * kWave * kMaskCols < d_in) ahead[u] = load_piece(m, (u * kWave + lane) * kMaskCols, d_in);
    }

    // (a workgroup's four rows share a byte)
    const uint32_t own_byte = row0 < d_out ? stored[row0 >> 3] : 0u;
    auto stored_byte = [&](int r) { return (r >> 3) == (row0 >> 3) ? own_byte : (uint32_t)stored[r >> 3]; };

    // bits of the rows [0, row0); workgroup 0 counts all rows, and the bad ones, for the report
    const bool reports = blockIdx.x == 0 && report != nullptr;
    const int upto = reports ? n_words : (row0 + 31) / 32;
    int below = 0, n_bad = 0, first_bad = 0x7fffffff;
    for (int w = tid; w < upto; w += kRowsPerBlock * kWave) {
        uint32_t b = stored_w[w];
        const int left = (reports ? d_out : row0) - 32 * w;   // rows of this word that count
        if (left < 32) b &= (1u << left) - 1u;
        below += __popc(b);
        if (reports) {
            uint32_t q = bad_w[w];
            if (left < 32) q &= (1u << left) - 1u;
            n_bad += __popc(q);
            if (q != 0 && first_bad == 0x7fffffff) first_bad = 32 * w + __ffs(q) - 1;
        }
    }
    for (int off = 32; off > 0; off >>= 1) below += __shfl_xor(below, off, kWave);
    if (reports) {
        for (int off = 32; off > 0; off >>= 1) {
            n_bad += __shfl_xor(n_bad, off, kWave);
            first_bad = min(first_bad, __shfl_xor(first_bad, off, kWave));
        }
    }
    if (lane == 0) { part[wv] = below; part_bad[wv] = n_bad; part_first[wv] = first_bad; }
    __syncthreads();
    int base_slot = part[0] + part[1] + part[2] + part[3];
    static_assert(kRowsPerBlock == 4, "four parts");
    if (reports) {
        if (tid == 0) {
            const int nb = part_bad[0] + part_bad[1] + part_bad[2] + part_bad[3];
            const int fb = min(min(part_first[0], part_first[1]), min(part_first[2], part_first[3]));
            report->K = K;
            report->n_active = base_slot;
            report->n_bad_rows = nb;
            report->first_bad_row = nb ? fb : -1;
            report->reserved[0] = report->reserved[1] = report->reserved[2] = 0;
            // (the status goes last: a caller with the report in host memory may be waiting for it)
            const int st = nb > 0 ? SRIGL_ERR_FANIN : (active && base_slot > cap_rows ? SRIGL_ERR_CAPACITY : SRIGL_OK);
            __hip_atomic_store(&report->status, st, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        base_slot = 0;
    }
    if (K == 0 || cap_rows == 0) return;

    uint16_t* const list = lists + wv * list_cap;
    for (int i = wv; i < rows_per_block; i += kRowsPerBlock) {
        const int r = row0 + i;
        if (r >= d_out) return;
        if (((stored_byte(r) >> (r & 7)) & 1) == 0) continue;   // ablated or invalid
        // stored rows among the workgroup's first i
        int s = base_slot;
        for (int q = row0; q < r; q += 8 - (q & 7)) {
            const uint32_t b = stored_byte(q) >> (q & 7);
            const int n = min(8 - (q & 7), r - q);
            s += __popc(b & ((1u << n) - 1u));
        }
        if (s >= cap_rows) continue;   // no room
        if (lane == 0) active[s] = r;
        const uint8_t* m = mask + (size_t)r * d_in;
        const T* w = W + (size_t)r * d_in;
        T* wc = W_c + (size_t)s * K;
        int32_t* ix = idx + (size_t)s * K;
        uint16_t* sg = seg ? seg + (size_t)s * seg_stride : nullptr;
        unsigned char* pk = packed ? packed + (size_t)s * pl.row_bytes() : nullptr;

        int base = 0;   // kept columns of the batches before (same in every lane)
        for (int col0 = 0; col0 < d_in; col0 += kBatchCols) {
            if (pieces && (i != wv || col0 != 0)) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (col0 + u * kWave * kMaskCols < d_in) ahead[u] = load_piece(m, col0 + (u * kWave + lane) * kMaskCols, d_in);
            }
            int in_batch = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int col = col0 + (u * kWave + lane) * kMaskCols;
                if (col0 + u * kWave * kMaskCols >= d_in) break;
                uint32_t bits = pieces ? kept_bits(ahead[u]) : kept_bits_short(m, col, d_in);
                const int first = (pieces ? ahead[u].first : 0) - col0;
                // kept columns in the lanes below, and in all lanes: bit planes of the lanes' counts (0..16)
                const uint32_t n = __popc(bits);
                int before = 0, total = 0;
#pragma unroll
                for (int p = 0; p < 5; ++p) {
                    const uint64_t bal = __ballot((n >> p) & 1u);
                    before += (int)lanes_below(bal) << p;
                    total += __popcll(bal) << p;
                }
                // every fourth lane starts a 64-column segment
                const int entry = col / kSegCols;
                if (sg && (lane & 3) == 0 && entry < seg_stride) sg[entry] = (uint16_t)(base + in_batch + before);
                int pos = in_batch + before;
                while (bits) {
                    if (base + pos < K && pos < list_cap) list[pos] = (uint16_t)(first + __ffs(bits) - 1);
                    ++pos;
                    bits &= bits - 1;
                }
                in_batch += total;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int n_list = min(min(in_batch, K - base), list_cap);
            for (int t0 = 0; t0 < n_list; t0 += 4 * kWave) {
                int col[4];
                T v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) col[u] = col0 + list[min(t0 + u * kWave + lane, n_list - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = w[col[u]];   // (places past the end re-read the last column)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int t = t0 + u * kWave + lane;
                    if (t < n_list) {
                        ix[base + t] = col[u];
                        wc[base + t] = v[u];
                        if (pk) pl.store(pk, base + t, (uint32_t)v[u], col[u]);
                    }
                }
            }
            base += in_batch;
            __builtin_amdgcn_wave_barrier();   // the list is rewritten by the next batch
        }
        if (sg)   // entries behind the last lane that had columns
            for (int c = (d_in + kMaskCols * kWave - 1) / (kMaskCols * kWave) * (kMaskCols * kWave) / kSegCols + lane; c < seg_stride; c += kWave) sg[c] = (uint16_t)base;
        if (pk)
            for (int t = K + lane; t < pl.terms; t += kWave) pl.store(pk, t, 0u, 0);
    }
}

// The streaming copy from the canonical arrays: one thread per term, padding included.
__global__ __launch_bounds__(256) void k_pack_terms(const void* __restrict__ W_c, const int32_t* __restrict__ idx, int n_rows, int K,
                                                    unsigned char* __restrict__ packed, PackedLayout pl) {
    const long long places = (long long)n_rows * pl.terms;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < places; i += (long long)gridDim.x * blockDim.x) {
        const int s = (int)(i / pl.terms), t = (int)(i - (long long)s * pl.terms);
        uint32_t wbits = 0u;
        int col = 0;
        if (t < K) {
            const size_t e = (size_t)s * K + t;
            wbits = pl.w_bytes == 4 ? static_cast<const uint32_t*>(W_c)[e] : (uint32_t)static_cast<const uint16_t*>(W_c)[e];
            col = idx[e];
        }
        pl.store(packed + (size_t)s * pl.row_bytes(), t, wbits, col);
    }
}

__global__ void k_empty() {}

__global__ __launch_bounds__(256) void k_copy16(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) dst[i] = src[i];
}

}  // namespace srigl

using namespace srigl;

extern "C" {

size_t srigl_workspace_bytes(int32_t n_rows) {
    if (n_rows < 0) n_rows = 0;
    return 2 * sizeof(int32_t) * (size_t)n_rows + 256;
}

int32_t srigl_seg_stride(int32_t d_in) {
    if (d_in < 0) d_in = 0;
    return (d_in + kSegCols - 1) / kSegCols + 1;
}

srigl_status srigl_check_fanin(const uint8_t* mask, const int32_t* idx, int32_t n_rows, int32_t d_in,
                               int32_t K_expected, uint16_t* seg, void* workspace, size_t workspace_bytes,
                               srigl_report* report_dev, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if ((mask == nullptr) == (idx == nullptr)) return SRIGL_ERR_INVALID_ARG;
    if (n_rows < 0 || d_in < 0 || report_dev == nullptr) return SRIGL_ERR_INVALID_ARG;
    if (idx && (K_expected < 0 || K_expected > d_in)) return SRIGL_ERR_INVALID_ARG;
    if (mask && K_expected > d_in) return SRIGL_ERR_INVALID_ARG;
    if (idx && seg && K_expected > 65535) return SRIGL_ERR_UNSUPPORTED;
    if (n_rows > 0 && workspace == nullptr) return SRIGL_ERR_INVALID_ARG;
    if (workspace_bytes < srigl_workspace_bytes(n_rows)) return SRIGL_ERR_CAPACITY;
    int32_t* counts = static_cast<int32_t*>(workspace);
    const int blocks = (n_rows + kRowsPerBlock - 1) / kRowsPerBlock;
    if (n_rows > 0) {
        if (mask) hipLaunchKernelGGL(k_row_count, dim3(blocks), dim3(kRowsPerBlock * kWave), 0, st, mask, n_rows, d_in, counts);
        else      hipLaunchKernelGGL(k_check_idx, dim3(blocks), dim3(kRowsPerBlock * kWave), 0, st, idx, n_rows, K_expected, d_in, counts, seg, srigl_seg_stride(d_in));
    }
    hipLaunchKernelGGL(k_scan_rows, dim3(1), dim3(1024), 0, st, counts, n_rows, K_expected, idx ? 1 : 0, report_dev);
    return hip_ok(hipGetLastError());
}

// What both launches refuse before anything runs.
static srigl_status check_condense(const void* W, srigl_dtype w_dtype, const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K, int32_t cap_rows,
                                   const void* W_c, const int32_t* idx, const int32_t* active, const uint16_t* seg, const void* packed,
                                   size_t packed_bytes, const void* workspace) {
    if (d_out < 0 || d_in < 0 || K < 0 || K > d_in || cap_rows < 0) return SRIGL_ERR_INVALID_ARG;
    if (w_dtype != SRIGL_F32 && w_dtype != SRIGL_BF16) return SRIGL_ERR_INVALID_ARG;
    if (d_out > 0 && d_in > 0 && (W == nullptr || mask == nullptr)) return SRIGL_ERR_INVALID_ARG;
    if (cap_rows > 0 && (active == nullptr || (K > 0 && (W_c == nullptr || idx == nullptr)))) return SRIGL_ERR_INVALID_ARG;
    if (seg && K > 65535) return SRIGL_ERR_UNSUPPORTED;
    if (d_out > 0 && workspace == nullptr) return SRIGL_ERR_INVALID_ARG;
    if (packed) {
        if (reinterpret_cast<uintptr_t>(packed) % 16 != 0) return SRIGL_ERR_INVALID_ARG;
        if (packed_bytes < srigl_packed_bytes(cap_rows, K, d_in, w_dtype)) return SRIGL_ERR_CAPACITY;
    }
    return SRIGL_OK;
}

// two bits per row in the workspace (8 bytes per row of room)
static uint8_t* bad_bits(uint8_t* stored, int32_t d_out) { return stored ? stored + (size_t)(d_out + 127) / 128 * 16 : nullptr; }

// How the rows are shared out among k_row_counts' workgroups: groups of 32 to a workgroup, workgroups.
struct CountShape { int groups, words; };
static CountShape count_shape(int32_t d_out) {
    const int all = (d_out + kCountRows - 1) / kCountRows, groups = (all + kCountWords - 1) / kCountWords;
    return {groups, groups ? (all + groups - 1) / groups : 0};
}

static void launch_flags(const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K, void* workspace, unsigned long long* to_host, hipStream_t st) {
    uint8_t* const stored = static_cast<uint8_t*>(workspace);
    uint8_t* const bad = bad_bits(stored, d_out);
    if (d_out <= 0) return;
    if (to_host) {
        const CountShape c = count_shape(d_out);
        hipLaunchKernelGGL(k_row_counts, dim3((unsigned)c.words), dim3(kCountWaves * kWave), 0, st, mask, d_out, d_in, K, c.groups,
                           reinterpret_cast<uint32_t*>(stored), reinterpret_cast<uint32_t*>(bad), to_host);
    } else {
        hipLaunchKernelGGL(k_row_flags, dim3((unsigned)((d_out + kFlagRows - 1) / kFlagRows)), dim3(kFlagRows * kWave), 0, st, mask, d_out, d_in, K, stored, bad);
    }
}

static void launch_compact(const void* W, srigl_dtype w_dtype, const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K, int32_t cap_rows, void* W_c,
                           int32_t* idx, int32_t* active, uint16_t* seg, void* packed, void* workspace, srigl_report* report, hipStream_t st) {
    const PackedLayout pl = packed_layout(K, d_in, w_dtype == SRIGL_BF16);
    const uint8_t* stored = static_cast<const uint8_t*>(workspace);
    const uint8_t* bad = bad_bits(static_cast<uint8_t*>(workspace), d_out);
    // one row per wavefront; layers of more than 131072 rows several, so that the bits every workgroup reads stay a small part
    int rows_per_block = kRowsPerBlock;
    while ((d_out + rows_per_block - 1) / rows_per_block > 32768) rows_per_block *= 2;
    const int blocks = d_out > 0 ? (d_out + rows_per_block - 1) / rows_per_block : 1;   // (no rows: workgroup 0 writes the report)
    const int list_cap = (K < kBatchCols ? K : kBatchCols) + 1;
    const size_t lds = sizeof(uint16_t) * kRowsPerBlock * (size_t)list_cap;
    auto launch = [&](auto kern, const auto* weights, auto* out) {
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(kRowsPerBlock * kWave), lds, st, weights, mask, d_out, d_in, K, cap_rows, stored, bad, out, idx, active,
                           seg, srigl_seg_stride(d_in), static_cast<unsigned char*>(packed), pl, rows_per_block, list_cap, report);
    };
    if (w_dtype == SRIGL_F32) launch(k_compact_rows<uint32_t>, static_cast<const uint32_t*>(W), static_cast<uint32_t*>(W_c));
    else launch(k_compact_rows<uint16_t>, static_cast<const uint16_t*>(W), static_cast<uint16_t*>(W_c));
}

static srigl_status condense_core(const void* W, srigl_dtype w_dtype, const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K,
                                  int32_t cap_rows, void* W_c, int32_t* idx, int32_t* active, uint16_t* seg, void* packed,
                                  size_t packed_bytes, void* workspace, srigl_report* report_dev, hipStream_t st) {
    if (report_dev == nullptr) return SRIGL_ERR_INVALID_ARG;
    if (const srigl_status rc = check_condense(W, w_dtype, mask, d_out, d_in, K, cap_rows, W_c, idx, active, seg, packed, packed_bytes, workspace)) return rc;
    launch_flags(mask, d_out, d_in, K, workspace, nullptr, st);
    launch_compact(W, w_dtype, mask, d_out, d_in, K, cap_rows, W_c, idx, active, seg, packed, workspace, report_dev, st);
    return hip_ok(hipGetLastError());
}

// Layers whose rows 128 workgroups count in the 4.5 us that the host gains by it: two groups of 32 rows to a workgroup, and so little to read, all of them together and
// each by itself, that k_row_flags with a workgroup for every eight rows would not have been done sooner.  Calls of condense_layer with counts beside calls
// with the second launch's report (us; K = a tenth of d_in): 3072 x 768 13.0 / 16.3, 329 x 128 0.69 of the time, 8192 x 512 0.96, 4096 x 1536 0.97, 2048 x 2048 0.88, 1024 x 3072 0.92,
// 512 x 4096 0.93, 256 x 5120 0.93; beyond the line 12288 x 256 1.04, 20000 x 24 1.17, 3072 x 2048 0.98, 4096 x 2048 1.08, 2048 x 3072 1.02, 1024 x 4096 1.01, 512 x 6144 1.15, 64 x 16384 1.31.
size_t srigl_condense_count_bytes(int32_t d_out, int32_t d_in) {
    if (d_out <= 0 || d_in <= 0 || d_out > 2 * kCountRows * kCountWords) return 0;
    const CountShape c = count_shape(d_out);
    const long long rows_of_one = (long long)kCountRows * c.groups;   // what a workgroup reads by itself takes 42 times as long as its part of what all read
    return (d_out + 42 * rows_of_one) * d_in <= 8500000 ? c.words * sizeof(unsigned long long) : 0;
}

// The layers whose rows k_row_counts counts when it is asked to: 2^20 rows are the fields of a word.
static bool counts_fit(int32_t d_out, int32_t d_in) { return d_out > 0 && d_in > 0 && d_out <= 1 << 20 && (long long)d_out * d_in <= 8 << 20; }

srigl_status srigl_condense_count(const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K, void* workspace, size_t workspace_bytes, void* counts,
                                  size_t counts_bytes, void* stream) {
    if (d_out < 0 || d_in < 0 || K < 0 || K > d_in || (d_out > 0 && d_in > 0 && mask == nullptr)) return SRIGL_ERR_INVALID_ARG;
    if (d_out > 0 && (workspace == nullptr || reinterpret_cast<uintptr_t>(counts) % 8 != 0)) return SRIGL_ERR_INVALID_ARG;
    const size_t need = counts_fit(d_out, d_in) ? count_shape(d_out).words * sizeof(unsigned long long) : 0;
    if (workspace_bytes < srigl_workspace_bytes(d_out) || (counts && counts_bytes < need)) return SRIGL_ERR_CAPACITY;
    if (counts && need == 0) return SRIGL_ERR_UNSUPPORTED;
    if (counts) std::memset(counts, 0, need);
    std::atomic_thread_fence(std::memory_order_release);
    launch_flags(mask, d_out, d_in, K, workspace, static_cast<unsigned long long*>(counts), static_cast<hipStream_t>(stream));
    return hip_ok(hipGetLastError());
}

srigl_status srigl_condense_write(const void* W, srigl_dtype w_dtype, const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K, int32_t cap_rows,
                                  void* W_c, int32_t* idx, int32_t* active, uint16_t* seg, void* packed, size_t packed_bytes, void* workspace,
                                  size_t workspace_bytes, srigl_report* report, void* stream) {
    if (d_out >= 0 && workspace_bytes < srigl_workspace_bytes(d_out)) return SRIGL_ERR_CAPACITY;
    if (const srigl_status rc = check_condense(W, w_dtype, mask, d_out, d_in, K, cap_rows, W_c, idx, active, seg, packed, packed_bytes, workspace)) return rc;
    launch_compact(W, w_dtype, mask, d_out, d_in, K, cap_rows, W_c, idx, active, seg, packed, workspace, report, static_cast<hipStream_t>(stream));
    return hip_ok(hipGetLastError());
}

int32_t srigl_condense_counted(const void* counts, int32_t d_out, int32_t K, int32_t cap_rows, int32_t* from, srigl_report* report) {
    const unsigned long long* const words = static_cast<const unsigned long long*>(counts);
    const CountShape c = count_shape(std::max(d_out, 0));
    if (*from <= 0) {
        *report = srigl_report{};
        report->first_bad_row = -1;
    }
    for (; *from < c.words; ++*from) {
        const unsigned long long w = __atomic_load_n(&words[*from], __ATOMIC_ACQUIRE);
        if ((w & kCounted) == 0) return 0;
        const int wrong = (int)((w >> 21) & 0x1fffff);
        report->n_active += (int)(w & 0x1fffff);
        report->n_bad_rows += wrong;
        if (wrong && report->first_bad_row < 0) report->first_bad_row = *from * c.groups * kCountRows + (int)((w >> 42) & 0x1fffff);
    }
    report->K = K;
    report->status = report->n_bad_rows > 0 ? SRIGL_ERR_FANIN : cap_rows >= 0 && report->n_active > cap_rows ? SRIGL_ERR_CAPACITY : SRIGL_OK;
    return 1;
}

srigl_status srigl_condense(const void* W, srigl_dtype w_dtype, const uint8_t* mask, int32_t d_out,
                            int32_t d_in, int32_t K, int32_t cap_rows, void* W_c, int32_t* idx,
                            int32_t* active, uint16_t* seg, void* packed, size_t packed_bytes, void* workspace,
                            size_t workspace_bytes, srigl_report* report_dev, void* stream) {
    if (d_out >= 0 && workspace_bytes < srigl_workspace_bytes(d_out)) return SRIGL_ERR_CAPACITY;
    return condense_core(W, w_dtype, mask, d_out, d_in, K, cap_rows, W_c, idx, active, seg, packed, packed_bytes, workspace,
                         report_dev, static_cast<hipStream_t>(stream));
}

// Device address of `scratch` on the current device, looked up once per device.
static srigl_status scratch_on_current_device(void** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptr[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return SRIGL_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return SRIGL_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return SRIGL_ERR_HIP;
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return SRIGL_OK;
}

srigl_status srigl_condense_static(const void* W, srigl_dtype w_dtype, const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K,
                                   int32_t cap_rows, void* W_c, int32_t* idx, int32_t* active, uint16_t* seg, void* packed,
                                   size_t packed_bytes, srigl_report* report_dev, void* stream) {
    if (d_out > SRIGL_STATIC_MAX_ROWS) return SRIGL_ERR_CAPACITY;   // more rows than the built-in scratch holds
    void* ws = nullptr;
    const srigl_status st = scratch_on_current_device(&ws);
    if (st != SRIGL_OK) return st;
    // every bit of rows [0, d_out) is written by the first kernel before the second reads it, so what an earlier call left in
    // the scratch is never seen and nothing has to be cleared
    return condense_core(W, w_dtype, mask, d_out, d_in, K, cap_rows, W_c, idx, active, seg, packed, packed_bytes, ws, report_dev,
                         static_cast<hipStream_t>(stream));
}

size_t srigl_packed_bytes(int32_t n_rows, int32_t K, int32_t d_in, srigl_dtype w_dtype) {
    if (n_rows <= 0 || K <= 0 || d_in <= 0 || (w_dtype != SRIGL_F32 && w_dtype != SRIGL_BF16)) return 0;
    return (size_t)n_rows * packed_layout(K, d_in, w_dtype == SRIGL_BF16).row_bytes();
}

srigl_status srigl_pack_terms(const void* W_c, srigl_dtype w_dtype, const int32_t* idx, int32_t n_rows, int32_t K, int32_t d_in,
                              void* packed, size_t packed_bytes, void* stream) {
    if (n_rows < 0 || K < 0 || d_in < 0 || K > d_in || (w_dtype != SRIGL_F32 && w_dtype != SRIGL_BF16)) return SRIGL_ERR_INVALID_ARG;
    if (n_rows == 0 || K == 0) return SRIGL_OK;
    if (W_c == nullptr || idx == nullptr || packed == nullptr || reinterpret_cast<uintptr_t>(packed) % 16 != 0) return SRIGL_ERR_INVALID_ARG;
    if (packed_bytes < srigl_packed_bytes(n_rows, K, d_in, w_dtype)) return SRIGL_ERR_CAPACITY;
    const PackedLayout pl = packed_layout(K, d_in, w_dtype == SRIGL_BF16);
    long long blocks = ((long long)n_rows * pl.terms + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_pack_terms, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(stream), W_c, idx, n_rows, K,
                       static_cast<unsigned char*>(packed), pl);
    return hip_ok(hipGetLastError());
}

srigl_status srigl_launch_empty(void* stream) {
    hipLaunchKernelGGL(k_empty, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream));
    return hip_ok(hipGetLastError());
}

srigl_status srigl_copy_bytes(const void* src, void* dst, size_t n_bytes, void* stream) {
    if (n_bytes == 0) return SRIGL_OK;
    if (src == nullptr || dst == nullptr || (n_bytes & 15) != 0) return SRIGL_ERR_INVALID_ARG;
    if (((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) != 0) return SRIGL_ERR_INVALID_ARG;
    const size_t n16 = n_bytes / 16;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint4*>(src), static_cast<uint4*>(dst), n16);
    return hip_ok(hipGetLastError());
}

const char* srigl_status_str(srigl_status s) {
    switch (s) {
        case SRIGL_OK: return "ok";
        case SRIGL_ERR_INVALID_ARG: return "invalid argument";
        case SRIGL_ERR_FANIN: return "a row holds neither 0 nor K kept weights";
        case SRIGL_ERR_CAPACITY: return "buffer too small";
        case SRIGL_ERR_INDEX_RANGE: return "index out of range or row not strictly ascending";
        case SRIGL_ERR_UNSUPPORTED: return "unsupported configuration";
        case SRIGL_ERR_HIP: return "HIP call failed";
    }
    return "unknown status";
}

}  // extern "C"
