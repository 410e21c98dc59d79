// One SRigL connectivity update of a layer on the GPU (gfx950): Sec. 3.1 of arXiv 2305.02299, steps 1-7 (prune / grow
// criteria, salient weights per neuron, neuron ablation with threshold gamma_sal, new fan-in k', layer-wide pruning, per-neuron
// regrowth), fp32 weights and gradients, dense [d_out][d_in] storage with a byte mask.  Readings of the text are listed in
// include/srigl.h next to srigl_mask_update.
//
// Every ranking is a selection of the K largest of unique 64-bit keys, (magnitude bits, position): equal magnitudes are
// ordered by position, so the selected set is unique and no sort is needed.
//
// Layer-wide selections (steps 3 and 6).  The top bit of a key is zero; its next 12 bits (exponent and 4 mantissa bits) are
// the first digit.  k_hist counts the digits of the whole layer, k_collect lists the keys of the digit that holds the K-th
// (about a percent of a layer with real-valued contents), k_final finishes the walk on that list in one workgroup.  So the
// layer is read twice per selection pair, and both selections of step 3 share the reads (an element belongs to exactly one).
// Contents with more keys in that digit than the list has room for (few distinct magnitudes: gradients that are zero, quantised or signed
// weights) go without a list: k_collect counts the next 12 bits instead, and k_final's launch, which has a workgroup per compute unit
// or so standing by for that, counts the last 7 bits of the magnitude in one pass (finish_wide).  Step 6 ranks the weights of the neurons that remain: the per-neuron kernel takes
// the ablated neurons' keys out of step 3's counts, so step 6 starts at k_collect, and with no neuron ablated it is step 3's
// answer.  Row-wise selections (step 7) are a search for the threshold by its bits, one wavefront per row, keys in registers,
// counts from ballots: no LDS, no barrier.
//
// Eight launches.  768 x 3072, 90 % sparse: the walk by 8-bit digits through 19 launches took 98 us, 48 of them for three
// passes whose LDS counters met in one bank, 19 for the row-wise radix walk.
#include "scan_tail.h"
#include "srigl_internal.h"
#include <cstddef>

namespace srigl {

struct SelState {
    unsigned long long prefix;      // the leading bits of the K-th largest key found so far (right-aligned); at the end: the key itself
    unsigned long long k_rem;       // how many of the keys with this prefix are still wanted
    unsigned long long total;       // number of candidate keys
    unsigned int in_bin;            // keys with this prefix
    int done;                       // the threshold is final (nothing wanted: ~0; everything wanted: 0; or the walk has ended)
};

constexpr int kDigitBits = 12, kDigits = 1 << kDigitBits, kDigitShift = 63 - kDigitBits;   // the first digit of a key
constexpr int kCoarse = 256, kFine = kDigits / kCoarse;   // the digit is found among 256 coarse counts first, then among 16
// Copies of the layer-wide counters (a workgroup adds into copy w % 8: one per die), and of the neuron counters: a launch ends
// with one atomic per non-empty digit and workgroup, and atomics on one address take turns.
constexpr int kHistCopies = 8;
constexpr int kCountCopies = 64;
constexpr int kNextCopies = 4;   // of the counters of step 3's second digits (a hundredth as many adds)
constexpr int kWideParts = 256;  // parts of the layer in finish_wide, at most

// Head of the workspace.  Selections: 0 = smallest kept weights of the layer, 1 = largest gradients at pruned positions,
// 2 = smallest kept weights of the remaining neurons (counted in hist[0] once the ablated neurons are out of it).
struct UpdateScratch {
    unsigned int hist[2][kHistCopies][kDigits];
    unsigned int coarse[2][kHistCopies][kCoarse];
    // second digits of the keys with the picked first one: selections 0 and 1 always (copies), selection 2 (one) where it has no list
    unsigned int next[2 * kNextCopies + 1][kDigits];
    unsigned int cnt_remaining[kCountCopies], cnt_ablated[kCountCopies];   // steps 4-5: neurons that stay / are ablated now
    unsigned long long cand_count[3];   // keys in the selection's list
    unsigned int arrived[4];            // finish_wide: parts of the selection that have been counted
    SelState picked[3];                 // after the first digit (written by k_collect)
    SelState fin[3];                    // the finished selections (k_final)
    unsigned long long t_prune;         // step 6's threshold and the new fan-in (k_final of step 6)
    long long k_new;
};
__device__ __forceinline__ unsigned int* next_digits(UpdateScratch* s, int sel, int copy) {
    return s->next[sel == 2 ? 2 * kNextCopies : sel * kNextCopies + copy % kNextCopies];
}
constexpr size_t kZeroWords = (offsetof(UpdateScratch, picked) + 15) / 16;   // 16-byte pieces cleared before an update

__device__ __forceinline__ unsigned int mag_bits(float v) { return __float_as_uint(v) & 0x7fffffffu; }
// larger key = smaller magnitude, then lower position
__device__ __forceinline__ unsigned long long key_small_first(unsigned int mag, unsigned int pos) {
    return ((unsigned long long)(0x7fffffffu - mag) << 32) | (0xffffffffu - pos);
}
// larger key = larger magnitude, then lower position
__device__ __forceinline__ unsigned long long key_large_first(unsigned int mag, unsigned int pos) {
    return ((unsigned long long)mag << 32) | (0xffffffffu - pos);
}
__device__ __forceinline__ unsigned int digit_small_first(unsigned int mag) { return (0x7fffffffu - mag) >> (kDigitShift - 32); }
__device__ __forceinline__ unsigned int digit_large_first(unsigned int mag) { return mag >> (kDigitShift - 32); }

constexpr int kInitBlocks = 64;
__global__ __launch_bounds__(256) void k_update_init(uint4* __restrict__ head) {
    const uint4 z = {0u, 0u, 0u, 0u};
    for (size_t i = blockIdx.x * 256 + threadIdx.x; i < kZeroWords; i += (size_t)kInitBlocks * 256) head[i] = z;
}

// The part of the layer that workgroup w works on, in every launch that reads the layer: consecutive workgroup ids go round the eight dies, and each of
// them stays with the same eighth of the layer.  (What a die keeps of it between launches the counters do not say: under them, one launch at a time, k_row_salient misses its L2 on
// 167 of 185 thousand requests with this order and on 168 without.)  A die's eighth is four runs, so that contents whose
// expensive rows lie together (weights of few magnitudes lose their first rows) do not leave dies without work.  Whole updates against ones with no order (and results
// not yet streamed): real-valued contents 0.83 to 0.95 of the time (3072 x 768 43.8 -> 40.6 us, 4096 x 1024 61.4 -> 51.2, 1953 x 4096 87.9 -> 81.9), few magnitudes 0.97 to
// 1.03, 1.05 at worst (signed weights on 4096 x 1024 185 -> 187, 1953 x 4096 351 -> 345; mostly ones on 1024 x 4096 200 -> 207).  One run a die: signed weights another 1 to 3 % slower.
// Eight runs: those 0.94 to 0.99 of four, but real-valued ones 1.01 to 1.06 (a die then meets twice as many pages); eight on layers of 4 to 7 M elements only: signed weights on
// 4096 x 1024 178, real-valued ones 51.7, and the choice itself 0.5 to 1 us on every other layer.
constexpr unsigned int kRuns = 4;
__device__ __forceinline__ unsigned int part_of_workgroup(unsigned int w, unsigned int workgroups) {
    if (workgroups % kDies) return w;
    const unsigned int of_die = workgroups / kDies, die = w % kDies, j = w / kDies;
    unsigned int first = 0, next = (of_die + kRuns - 1) / kRuns;   // the run's first workgroup of each die, and the next run's
#pragma unroll
    for (unsigned int r = 1; r < kRuns; ++r)
        if (j >= next) {
            first = next;
            next = ((r + 1) * of_die + kRuns - 1) / kRuns;
        }
    return kDies * first + die * (next - first) + j - first;
}

// Four consecutive elements of the flat layer.
struct Quad {
    uint32_t m;
    float4 w, g;
};
// What a workgroup of k_hist / k_collect works on: a run of quads, kQuads per thread in flight.
constexpr int kScanThreads = 1024, kQuads = 4;
template <bool GRAD>
__device__ __forceinline__ void load_quads(Quad (&q)[kQuads], const float* __restrict__ W, const uint8_t* __restrict__ mask,
                                           const float* __restrict__ grad, unsigned int first, unsigned int end) {
#pragma unroll
    for (int u = 0; u < kQuads; ++u) {
        const unsigned int i = min(first + u * kScanThreads + threadIdx.x, end - 1);   // (past the end: re-read and dropped)
        q[u].m = reinterpret_cast<const uint32_t*>(mask)[i];
        q[u].w = reinterpret_cast<const float4*>(W)[i];
        if (GRAD) q[u].g = reinterpret_cast<const float4*>(grad)[i];
    }
}
// The elements of a quad, or of the layer's last ones (fewer than four, or all of them when the arrays are not 16-byte aligned).
template <typename Element>
__device__ __forceinline__ void each_of_quad(const Quad& q, unsigned int base, Element element) {
    element(base + 0, q.m & 0xffu, q.w.x, q.g.x);
    element(base + 1, (q.m >> 8) & 0xffu, q.w.y, q.g.y);
    element(base + 2, (q.m >> 16) & 0xffu, q.w.z, q.g.z);
    element(base + 3, q.m >> 24, q.w.w, q.g.w);
}

// Counts the first digits of both selections of step 3.  n4 quads, then the elements [4 n4, N) one by one.  LDS counters: the
// digits of one wavefront's values spread over some fifty of the 4096, so its adds meet at most a few times per address.
__global__ __launch_bounds__(kScanThreads) void k_hist(const float* __restrict__ W, const uint8_t* __restrict__ mask, const float* __restrict__ grad,
                                                       unsigned int N, unsigned int n4, unsigned int n_wg, unsigned int per, UpdateScratch* __restrict__ s) {
    __shared__ __align__(16) unsigned int h[2][kDigits];
    const int t = threadIdx.x;
    const unsigned int q0 = min(part_of_workgroup(blockIdx.x, n_wg) * per, n4), q1 = min(q0 + per, n4);
    Quad q[kQuads];
    if (q0 < q1) load_quads<true>(q, W, mask, grad, q0, q1);
    for (int i = t; i < 2 * kDigits / 4; i += kScanThreads) reinterpret_cast<uint4*>(&h[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    auto element = [&](unsigned int, unsigned int m, float w, float g) {
        const unsigned int d = m ? digit_small_first(mag_bits(w)) : digit_large_first(mag_bits(g));
        atomicAdd(&h[m ? 0 : 1][d], 1u);
    };
    for (unsigned int b = q0; b < q1; b += kQuads * kScanThreads) {
        if (b != q0) load_quads<true>(q, W, mask, grad, b, q1);
#pragma unroll
        for (int u = 0; u < kQuads; ++u)
            if (b + u * kScanThreads + t < q1) each_of_quad(q[u], 0, element);
    }
    each_of_tail(N, n4, blockIdx.x * kScanThreads + t, n_wg * kScanThreads, [&](unsigned int i) { element(i, mask[i], W[i], grad[i]); });
    __syncthreads();
    // neighbouring lanes add to neighbouring digits (an atomic instruction costs by the lines it touches: with four digits in a
    // row per thread the flush took half of the kernel's 11 us)
    const int copy = blockIdx.x % kHistCopies;
#pragma unroll
    for (int sel = 0; sel < 2; ++sel) {
#pragma unroll
        for (int j = 0; j < kDigits / kScanThreads; ++j) {
            const unsigned int n = h[sel][t + j * kScanThreads];
            if (n) atomicAdd(&s->hist[sel][copy][t + j * kScanThreads], n);
        }
    }
    if (t < 2 * kCoarse) {
        const int sel = t / kCoarse, c = t % kCoarse;
        unsigned int n = 0;
#pragma unroll
        for (int j = 0; j < kFine / 4; ++j) {
            const uint4 v = reinterpret_cast<const uint4*>(&h[sel][c * kFine])[j];
            n += v.x + v.y + v.z + v.w;
        }
        if (n) atomicAdd(&s->coarse[sel][copy][c], n);
    }
}
static_assert(kFine == 16 && kDigits == 4 * kScanThreads, "sixteen digits per coarse count, four per thread");

__device__ __forceinline__ unsigned int wave_total(unsigned int v) { return (unsigned)__builtin_amdgcn_readlane((int)wave_prefix(v), 63); }

// With n keys in this lane's bin: the bin d with suffix(d) >= want > suffix(d + 1), suffix(d) = keys in bins d and above;
// `above` = suffix(d + 1), `in_bin` = the bin's keys, `total` = suffix(0).  The results are the same on every lane.
__device__ __forceinline__ void pick_lane(unsigned int n, unsigned int want, int& bin, unsigned int& above, unsigned int& in_bin,
                                          unsigned int& total) {
    const unsigned int incl = wave_prefix(n);
    total = (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
    const unsigned int beyond = total - incl;   // keys in the bins above this lane's
    const uint64_t owner = __ballot(beyond < want && beyond + n >= want);
    bin = owner ? __builtin_ctzll(owner) : 0;
    above = (unsigned)__builtin_amdgcn_readlane((int)beyond, bin);
    in_bin = (unsigned)__builtin_amdgcn_readlane((int)n, bin);
}

// The state of a selection after its first digit, from the layer-wide counters.  One whole wavefront; the same on every lane.
__device__ SelState pick_first(const UpdateScratch* __restrict__ s, int hist, unsigned long long K, int lane) {
    unsigned int v[4] = {0u, 0u, 0u, 0u};   // coarse counts 4 lane .. 4 lane + 3
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) {
        const uint4 q = reinterpret_cast<const uint4*>(s->coarse[hist][c])[lane];
        v[0] += q.x; v[1] += q.y; v[2] += q.z; v[3] += q.w;
    }
    SelState st;
    st.prefix = 0; st.k_rem = K; st.in_bin = 0; st.done = 0;
    int group, sub, fine;
    unsigned int above, in_bin, total;
    pick_lane(v[0] + v[1] + v[2] + v[3], K == 0 ? 1u : (unsigned)min(K, 0xffffffffull), group, above, in_bin, total);
    st.total = total;
    if (K == 0 || total < K) {
        st.prefix = K == 0 ? ~0ull : 0ull;   // nothing / everything
        st.done = 1;
        return st;
    }
    unsigned int want = (unsigned)K - above;
    // the coarse digit inside the chosen group of four, then the digit inside the coarse one
    unsigned int mine = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const unsigned int x = (unsigned)__builtin_amdgcn_readlane((int)v[j], group);
        if (lane == j) mine = x;
    }
    pick_lane(mine, want, sub, above, in_bin, total);
    want -= above;
    const int coarse = 4 * group + sub;
    unsigned int n = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; c += 4) n += s->hist[hist][c + (lane >> 4)][coarse * kFine + (lane & 15)];
    n += __shfl_xor(n, 16, 64);
    n += __shfl_xor(n, 32, 64);
    pick_lane(lane < kFine ? n : 0u, want, fine, above, in_bin, total);
    st.k_rem = want - above;
    st.prefix = coarse * kFine + fine;
    st.in_bin = in_bin;
    if (st.k_rem == in_bin) {   // every key of the digit is wanted: the threshold is the smallest key with this prefix
        st.prefix <<= kDigitShift;
        st.done = 1;
    }
    return st;
}

// add(d, n) for the lanes that are `on`: those with the first one's digit add together, the others for themselves (contents of few magnitudes
// have whole wavefronts on one counter, whose atomics take turns).
template <typename Add>
__device__ __forceinline__ void add_by_digit(bool on, unsigned int d, Add add) {
    const uint64_t any = __ballot(on);
    if (any == 0) return;
    const int lead = __builtin_ctzll(any);
    const unsigned int first = (unsigned)__builtin_amdgcn_readlane((int)d, lead);
    const uint64_t same = __ballot(on && d == first);
    if (on && d != first) add(d, 1u);
    if ((int)(threadIdx.x & 63) == lead) add(first, (unsigned)__popcll(same));
}

// Sum of the 64 copies of a neuron counter.  Called by one whole wavefront; the result is the same on every lane.
__device__ __forceinline__ unsigned int sum_copies(const unsigned int (&c)[kCountCopies], int lane) {
    return wave_total(c[lane]);
}

// Lists the keys of the first digit that holds the K-th key.  PAIR: selections 0 and 1 together, otherwise selection 2 (kept
// weights of the remaining neurons; nothing to do when no neuron was ablated).  A workgroup collects up to kStage keys per
// selection in LDS and appends them with one update of the list's length; what does not fit goes out one by one.  PAIR also counts the
// next 12 bits of the keys it lists, so that k_final, one workgroup on its own, goes through the list once instead of twice (768 x 3072,
// 23000 keys: 9.5 -> 5.6 us there for 0.7 here).  Counting a neuron's salient elements here and in k_final, to spare k_row_salient the
// layer, cost k_final more than k_row_salient saved.  A selection whose digit holds more keys than a list has room for gets the next 12 bits
// of its keys counted instead (in LDS, in the place of the collected keys).
constexpr int kStage = 2048;
template <bool PAIR>
__global__ __launch_bounds__(kScanThreads) void k_collect(const float* __restrict__ W, const uint8_t* __restrict__ mask,
                                                          const float* __restrict__ grad, UpdateScratch* __restrict__ s, unsigned long long K,
                                                          unsigned int n4, unsigned int n_wg, unsigned int per, unsigned int N,   // (preloaded)
                                                          const int* __restrict__ remains, int d_in, unsigned long long* __restrict__ candA,
                                                          unsigned long long* __restrict__ candB, unsigned long long cap) {
    __shared__ __align__(16) unsigned long long stage[PAIR ? 2 : 1][kStage];
    __shared__ SelState cur[2];
    __shared__ unsigned int n_staged[2];
    __shared__ unsigned long long base[2];
    const int t = threadIdx.x;
    constexpr int selA = PAIR ? 0 : 2;
    const unsigned int q0 = min(part_of_workgroup(blockIdx.x, n_wg) * per, n4), q1 = min(q0 + per, n4);
    Quad q[kQuads];
    if (!PAIR && sum_copies(s->cnt_ablated, t & 63) == 0) return;
    if (q0 < q1) load_quads<PAIR>(q, W, mask, grad, q0, q1);   // (before the counters are waited for)
    if (t < (PAIR ? 128 : 64)) {
        const int k = t >> 6;
        const SelState st = pick_first(s, k, K, t & 63);
        if ((t & 63) == 0) {
            cur[k] = st;
            n_staged[k] = 0;
            if (blockIdx.x == 0) s->picked[k == 0 ? selA : 1] = st;
        }
    }
    __syncthreads();
    const bool openA = !cur[0].done, openB = PAIR && !cur[1].done;
    if (!openA && !openB) return;
    const bool wideA = openA && cur[0].in_bin > cap, wideB = openB && cur[1].in_bin > cap;
    const unsigned int digA = openA ? (unsigned int)cur[0].prefix : ~0u, digB = openB ? (unsigned int)cur[1].prefix : ~0u;
    if (wideA || wideB) {
        for (int i = t; i < kStage; i += kScanThreads) {
            if (wideA) stage[0][i] = 0ull;
            if (wideB) stage[PAIR ? 1 : 0][i] = 0ull;
        }
        __syncthreads();
    }
    auto second_digit = [](unsigned long long key) { return (unsigned int)(key >> (kDigitShift - kDigitBits)) & (kDigits - 1); };
    auto count_next = [&](int k, unsigned long long key) {
        add_by_digit(true, second_digit(key), [&](unsigned int d, unsigned int n) { atomicAdd(next_digits(s, k, blockIdx.x) + d, n); });
    };
    auto put = [&](int k, unsigned long long key) {
        if (k == 0 ? wideA : wideB) {
            atomicAdd(reinterpret_cast<unsigned int*>(stage[PAIR ? k : 0]) + second_digit(key), 1u);
            return;
        }
        const unsigned int slot = atomicAdd(&n_staged[k], 1u);
        if (slot < (unsigned)kStage) {
            stage[k][slot] = key;
        } else {
            const unsigned long long at = atomicAdd(&s->cand_count[k == 0 ? selA : 1], 1ull);
            if (PAIR) count_next(k, key);
            if (at < cap) (k == 0 ? candA : candB)[at] = key;
        }
    };
    auto element = [&](unsigned int i, unsigned int m, float w, float g) {
        if (m) {
            const unsigned int mag = mag_bits(w);
            if (digit_small_first(mag) == digA && (PAIR || remains[i / (unsigned)d_in] != 0)) put(0, key_small_first(mag, i));
        } else if (PAIR) {
            const unsigned int mag = mag_bits(g);
            if (digit_large_first(mag) == digB) put(1, key_large_first(mag, i));
        }
    };
    auto flush = [&] {
        __syncthreads();
        if (t < (PAIR ? 2 : 1)) {   // (nothing was put in place of a selection that counts)
            const unsigned int n = min(n_staged[t], (unsigned)kStage);
            base[t] = n ? atomicAdd(&s->cand_count[t == 0 ? selA : 1], (unsigned long long)n) : 0ull;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < (PAIR ? 2 : 1); ++k) {
            const unsigned int n = min(n_staged[k], (unsigned)kStage);
            for (unsigned int e = t; e < n; e += kScanThreads) {
                const unsigned long long key = stage[k][e];
                if (base[k] + e < cap) (k == 0 ? candA : candB)[base[k] + e] = key;
                if (PAIR) count_next(k, key);
            }
        }
        __syncthreads();
        if (t < 2) n_staged[t] = 0;
        __syncthreads();
    };
    int batches = 0;
    for (unsigned int b = q0; b < q1; b += kQuads * kScanThreads) {
        if (b != q0) load_quads<PAIR>(q, W, mask, grad, b, q1);
#pragma unroll
        for (int u = 0; u < kQuads; ++u) {
            const unsigned int i = b + u * kScanThreads + t;
            if (i < q1) each_of_quad(q[u], 4 * i, element);
        }
        if (++batches % 4 == 0 && b + kQuads * kScanThreads < q1) flush();   // (65536 elements, three percent of which the stage holds)
    }
    each_of_tail(N, n4, blockIdx.x * kScanThreads + t, n_wg * kScanThreads,
                 [&](unsigned int i) { element(i, mask[i], W[i], PAIR ? grad[i] : 0.0f); });
    flush();
#pragma unroll
    for (int k = 0; k < (PAIR ? 2 : 1); ++k) {
        if (!(k == 0 ? wideA : wideB)) continue;
#pragma unroll
        for (int j = 0; j < kDigits / kScanThreads; ++j) {
            const unsigned int d = t + j * kScanThreads, n = reinterpret_cast<const unsigned int*>(stage[k])[d];
            if (n) atomicAdd(next_digits(s, k == 0 ? selA : 1, blockIdx.x) + d, n);
        }
    }
}
static_assert(2 * kStage == kDigits, "the counters take the place of the collected keys");

// With c4 keys in the digits 4t .. 4t + 3 of thread t (c4.x in the lowest): the digit with the k_rem-th key becomes part of `st`, whose prefix
// grows by `bits`; `left` bits of the key follow.  The whole workgroup; the same on every thread.  wave_sum, cur: its LDS.
__device__ __forceinline__ void pick_next(SelState& st, const uint4 c4, int bits, int left, unsigned int (&wave_sum)[kScanThreads / 64], SelState& cur) {
    const int t = threadIdx.x, lane = t & 63;
    // keys in the digits above a thread's: in its wavefront's higher lanes and the higher wavefronts
    const unsigned int mine = c4.x + c4.y + c4.z + c4.w, incl = wave_prefix(mine);
    if (lane == 63) wave_sum[t >> 6] = incl;
    __syncthreads();
    unsigned int beyond = (unsigned)__builtin_amdgcn_readlane((int)incl, 63) - incl;
    for (int w = kScanThreads / 64 - 1; w > (t >> 6); --w) beyond += wave_sum[w];
    const unsigned int want = (unsigned)st.k_rem;
    if (beyond < want && beyond + mine >= want) {
        unsigned int above = beyond, in_bin = c4.w;
        int digit = 4 * t + 3;
        if (above + in_bin < want) { above += c4.w; in_bin = c4.z; --digit; }
        if (digit == 4 * t + 2 && above + in_bin < want) { above += c4.z; in_bin = c4.y; --digit; }
        if (digit == 4 * t + 1 && above + in_bin < want) { above += c4.y; in_bin = c4.x; --digit; }
        SelState c = st;
        c.k_rem = want - above;
        c.prefix = (c.prefix << bits) | (unsigned)digit;
        c.in_bin = in_bin;
        if (c.k_rem == in_bin || left == 0) {
            c.prefix <<= left;
            c.done = 1;
        }
        cur = c;
    }
    __syncthreads();
    st = cur;
    __syncthreads();   // (cur is written again by the next pick)
}
static_assert(kDigits == 4 * kScanThreads, "four digits per thread");

// The end of a selection without a list, after its second digit: the magnitudes still open differ in their last 7 bits.  Every workgroup
// of the selection counts them over a part of the layer; the last one to arrive finds the magnitude, the part in which the k_rem-th of
// its positions lies, and that position.  Two passes over the layer in all, by many workgroups, and one over a part.  (One workgroup that
// walked the layer digit by digit took 8.6 ms on 768 x 3072 with zero gradients, 55 on 1953 x 4096 with signed weights; the whole update takes
// 79 and 335 us now, with a fence per wavefront instead of one 108 and 376.)
// `count`: [parts][128] in the place of the list.  false: another workgroup finishes.
constexpr int kLastBits = kDigitShift - kDigitBits - 32, kLast = 1 << kLastBits;
static_assert(kLast == 128, "two values per lane");
__device__ bool finish_wide(SelState& st, int sel, int part, int parts, const float* __restrict__ W, const uint8_t* __restrict__ mask,
                            const float* __restrict__ grad, const int* __restrict__ remains, unsigned int N, int d_in, unsigned int* arrived,
                            unsigned int* __restrict__ count, unsigned int* sh) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    constexpr int U = 4, WAVES = kScanThreads / 64;
    unsigned int* const total = sh;                // [kLast]
    unsigned int* const found = sh + kLast;        // magnitude value, keys wanted of it, part, keys wanted in the part
    unsigned int* const wave_n = found + 4;        // [WAVES]
    unsigned int* const of_part = wave_n + WAVES;  // [kWideParts]
    const float* const src = sel == 1 ? grad : W;
    const unsigned long long prefix = st.prefix;   // the two digits
    const unsigned int per = (unsigned int)(((unsigned long long)N + parts - 1) / parts);
    auto part_begin = [&](int p) { return (unsigned int)min((unsigned long long)p * per, (unsigned long long)N); };
    // Visits [lo, hi) in steps of U x `width` elements, `at` of them this thread's first; f(position, value or ~0) with all lanes of the wavefront.
    auto visit = [&](unsigned int lo, unsigned int hi, unsigned int at, unsigned int width, auto f) {
        for (unsigned long long b = lo; b < hi; b += (unsigned long long)U * width) {
            unsigned int m[U], i[U];
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                i[u] = (unsigned int)min(b + (unsigned long long)u * width + at, (unsigned long long)N - 1);
                m[u] = mask[i[u]];
                v[u] = src[i[u]];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned long long key = sel == 1 ? key_large_first(mag_bits(v[u]), i[u]) : key_small_first(mag_bits(v[u]), i[u]);
                bool in = b + (unsigned long long)u * width + at < hi && (m[u] != 0) == (sel != 1) && (key >> (32 + kLastBits)) == prefix;
                if (sel == 2) in = in && remains[i[u] / (unsigned)d_in] != 0;
                if (!f(i[u], in ? (unsigned int)(key >> 32) & (kLast - 1) : ~0u)) return;
            }
        }
    };
    for (int i = t; i < kLast; i += kScanThreads) total[i] = 0;
    __syncthreads();
    visit(part_begin(part), part_begin(part + 1), t, kScanThreads, [&](unsigned int, unsigned int v) {
        add_by_digit(v != ~0u, v, [&](unsigned int d, unsigned int n) { atomicAdd(&total[d], n); });
        return true;
    });
    __syncthreads();
    for (int i = t; i < kLast; i += kScanThreads) count[part * kLast + i] = total[i];
    __syncthreads();
    if (t == 0) {   // (one wavefront's fences: behind and in front of the workgroup's barriers they stand for all of it)
        __threadfence();
        found[0] = atomicAdd(arrived, 1u);
        __threadfence();
    }
    __syncthreads();
    if (found[0] != (unsigned)parts - 1) return false;
    __syncthreads();
    // ---- the magnitude
    for (int i = t; i < kLast; i += kScanThreads) total[i] = 0;
    __syncthreads();
    {
        unsigned int n = 0;
        for (int p = t / kLast; p < parts; p += kScanThreads / kLast) n += __hip_atomic_load(&count[p * kLast + t % kLast], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (n) atomicAdd(&total[t % kLast], n);
    }
    __syncthreads();
    if (wv == 0) {
        const unsigned int lo = total[2 * lane], hi = total[2 * lane + 1];
        int pair;
        unsigned int above, in_pair, all;
        pick_lane(lo + hi, (unsigned)st.k_rem, pair, above, in_pair, all);
        const unsigned int top = (unsigned)__builtin_amdgcn_readlane((int)hi, pair), want = (unsigned)st.k_rem - above;
        if (lane == 0) {
            found[0] = 2 * pair + (want <= top ? 1 : 0);
            found[1] = want <= top ? want : want - top;
        }
    }
    __syncthreads();
    const unsigned int value = found[0];
    st.k_rem = found[1];
    st.in_bin = total[value];
    st.prefix = (prefix << kLastBits) | value;
    st.done = 1;
    if (st.k_rem == st.in_bin) {   // every position of the magnitude: the smallest key with it
        st.prefix <<= 32;
        return true;
    }
    // ---- the part, lower positions first
    for (int p = t; p < parts; p += kScanThreads) of_part[p] = __hip_atomic_load(&count[p * kLast + value], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    // the group of 64 entries (or the entry) in which the want-th lies; want becomes its number in there
    auto walk = [&](const unsigned int* n, int entries, unsigned int want) {
        for (int e0 = 0; e0 < entries; e0 += 64) {
            const unsigned int mine = e0 + lane < entries ? n[e0 + lane] : 0u, incl = wave_prefix(mine);
            const uint64_t owner = __ballot(incl >= want && incl - mine < want);
            if (owner) {
                const int l = __builtin_ctzll(owner);
                if (lane == 0) {
                    found[2] = e0 + l;
                    found[3] = want - ((unsigned)__builtin_amdgcn_readlane((int)incl, l) - (unsigned)__builtin_amdgcn_readlane((int)mine, l));
                }
                return;
            }
            want -= (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
        }
    };
    if (wv == 0) walk(of_part, parts, (unsigned)st.k_rem);
    __syncthreads();
    // ---- the position: a run of the part per wavefront, counted; then the run that holds it once more
    const unsigned int lo = part_begin(found[2]), hi = part_begin(found[2] + 1), want = found[3], run = (hi - lo + WAVES - 1) / WAVES;
    auto run_begin = [&](int w) { return lo + min((unsigned)w * run, hi - lo); };
    unsigned int n = 0;
    visit(run_begin(wv), run_begin(wv + 1), lane, 64, [&](unsigned int, unsigned int v) {
        n += (unsigned)__popcll(__ballot(v == value));
        return true;
    });
    if (lane == 0) wave_n[wv] = n;
    __syncthreads();
    if (wv == 0) walk(wave_n, WAVES, want);
    __syncthreads();
    if (wv == (int)found[2]) {
        unsigned int left = found[3];
        visit(run_begin(wv), run_begin(wv + 1), lane, 64, [&](unsigned int i, unsigned int v) {
            const uint64_t here = __ballot(v == value);
            const unsigned int c = (unsigned)__popcll(here);
            if (left > c) { left -= c; return true; }
            const unsigned int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(here >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)here, 0u));
            if (v == value && rank + 1 == left) found[0] = 0xffffffffu - i;
            return false;
        });
    }
    __syncthreads();
    st.prefix = (st.prefix << 32) | found[0];
    return true;
}

// The end of a selection: workgroups of selection 0 and 1 in turn (PAIR), or of selection 2.  With a list the selection's first workgroup does
// it all and the others return at once; without one they share the work (finish_wide).  One workgroup runs the code for a list once, so its
// length counts: with the list held in registers and every loop unrolled over it, fetching the instructions took most of 10 us.  12-bit
// digits until at most kDirect keys share the prefix (step 3: the first of them from k_collect's counters, which is enough on
// real-valued contents), which are then ranked against each other.  (Eight loads ahead instead of four, for
// the same reason: updates of 4096 x 1024 52.1 us instead of 50.9, 1953 x 4096 83.7 instead of 81.9, smaller ones level.)
// Step 6's first workgroup also takes the new fan-in from the neuron counters (step 5) and writes the report.
constexpr int kAhead = 4, kDirect = 256;
template <bool PAIR>
__global__ __launch_bounds__(kScanThreads) void k_final(UpdateScratch* __restrict__ s, unsigned long long* candA, unsigned long long* candB,
                                                        unsigned long long cap, unsigned long long K, long long budget, int parts, int d_in,   // (preloaded)
                                                        const float* __restrict__ W, const uint8_t* __restrict__ mask, const float* __restrict__ grad,
                                                        const int* __restrict__ remains, unsigned int N, long long* __restrict__ report) {
    __shared__ __align__(16) unsigned int h[kDigits];
    __shared__ unsigned int wave_sum[kScanThreads / 64];
    __shared__ SelState cur;
    __shared__ unsigned long long direct[kDirect];
    __shared__ unsigned int n_direct;
    const int t = threadIdx.x, lane = t & 63;
    const int sel = PAIR ? (int)blockIdx.x & 1 : 2, part = PAIR ? (int)blockIdx.x >> 1 : (int)blockIdx.x;   // of `parts` for each selection
    SelState st;
    if (!PAIR) {
        const unsigned int n_ablated = sum_copies(s->cnt_ablated, lane);
        if (part != 0 && n_ablated == 0) return;
        st = n_ablated == 0 ? s->fin[0] : s->picked[2];   // no neuron ablated: the same candidates and count as in step 3
        if (part == 0) {
            const unsigned int n_remaining = sum_copies(s->cnt_remaining, lane);
            if (t == 0) {
                long long k = n_remaining > 0 ? budget / (long long)n_remaining : 0;
                if (k > d_in) k = d_in;
                s->k_new = k;
                report[0] = k;
                report[1] = n_remaining;
                report[2] = n_ablated;
                report[3] = (long long)(K < st.total ? K : st.total);
            }
        }
    } else {
        st = s->picked[sel];
    }
    auto finish = [&] {
        if (t == 0) {
            s->fin[sel] = st;
            if (!PAIR) s->t_prune = st.prefix;
        }
    };
    const bool wide = !st.done && st.in_bin > cap;
    if (part != 0 && !wide) return;
    if (st.done) { finish(); return; }
    auto counted_where_listed = [&] {
        uint4 c4 = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int c = 0; c < (PAIR ? kNextCopies : 1); ++c) {
            const uint4 v = reinterpret_cast<const uint4*>(next_digits(s, sel, c))[t];
            c4.x += v.x; c4.y += v.y; c4.z += v.z; c4.w += v.w;
        }
        return c4;
    };
    if (wide) {
        pick_next(st, counted_where_listed(), kDigitBits, kDigitShift - kDigitBits, wave_sum, cur);
        if (st.done ? part == 0 : finish_wide(st, sel, part, parts, W, mask, grad, remains, N, d_in, &s->arrived[sel],
                                              reinterpret_cast<unsigned int*>(sel == 1 ? candB : candA), h))
            finish();
        return;
    }
    const unsigned int n = st.in_bin;   // every key of the digit is in the list
    const unsigned long long* const list = sel == 1 ? candB : candA;
    auto each = [&](auto f) {
#pragma unroll 1
        for (unsigned int i0 = t; 2 * i0 < n; i0 += kAhead * kScanThreads) {   // two keys per load
            ulonglong2 key[kAhead];
#pragma unroll
            for (int j = 0; j < kAhead; ++j) key[j] = reinterpret_cast<const ulonglong2*>(list)[min(i0 + j * kScanThreads, (n - 1u) / 2u)];
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const unsigned int i = 2 * (i0 + j * kScanThreads);
                if (i < n) f(key[j].x);
                if (i + 1 < n) f(key[j].y);
            }
        }
    };
    int shift = kDigitShift;   // key >> shift == st.prefix: still in the walk
    for (;;) {
        if (st.in_bin <= (unsigned)kDirect) {
            if (t == 0) n_direct = 0;
            __syncthreads();
            each([&](unsigned long long k) {
                if ((k >> shift) == st.prefix) direct[min(atomicAdd(&n_direct, 1u), (unsigned)kDirect - 1)] = k;
            });
            __syncthreads();
            const unsigned int n_here = min(n_direct, (unsigned)kDirect);
            if (t < (int)n_here) {   // the k_rem-th largest
                const unsigned long long mine = direct[t];
                unsigned int larger = 0;
                for (unsigned int j = 0; j < n_here; ++j) larger += direct[j] > mine ? 1u : 0u;
                if (larger + 1 == st.k_rem) cur.prefix = mine;
            }
            __syncthreads();
            st.prefix = cur.prefix;
            st.done = 1;
            finish();
            return;
        }
        const int bits = min(kDigitBits, shift), next = shift - bits;
        uint4 c4;
        if (PAIR && shift == kDigitShift) {   // counted where the list was made
            c4 = counted_where_listed();
        } else {
            for (int i = t; i < kDigits; i += kScanThreads) h[i] = 0;
            __syncthreads();
            each([&](unsigned long long k) {
                add_by_digit((k >> shift) == st.prefix, (unsigned int)(k >> next) & ((1u << bits) - 1u),
                             [&](unsigned int d, unsigned int c) { atomicAdd(&h[d], c); });
            });
            __syncthreads();
            c4 = reinterpret_cast<const uint4*>(h)[t];
        }
        pick_next(st, c4, bits, next, wave_sum, cur);
        shift = next;
        if (st.done) { finish(); return; }
    }
}
static_assert((kLast + 4 + kScanThreads / 64 + kWideParts) <= kDigits, "finish_wide's LDS");

// Four consecutive columns of a row, at any alignment of the row: the last group of a row that does not end on a group
// boundary reads the row's last four columns and owns only those its neighbour does not have.
struct RowQuad {
    uint32_t m;
    float4 w, g;
};
__device__ __forceinline__ int quad_first(int c0, int d_in) { return min(c0, d_in - 4); }
__device__ __forceinline__ void load_row_quad(RowQuad& q, const float* __restrict__ W, const uint8_t* __restrict__ mask,
                                              const float* __restrict__ grad, size_t at) {
    __builtin_memcpy(&q.m, mask + at, 4);
    struct __attribute__((packed, aligned(4))) F4 { float x, y, z, w; };
    const F4 w = *reinterpret_cast<const F4*>(W + at), g = *reinterpret_cast<const F4*>(grad + at);
    q.w = make_float4(w.x, w.y, w.z, w.w);
    q.g = make_float4(g.x, g.y, g.z, g.w);
}
// rows of fewer than four columns
__device__ __forceinline__ void load_row_short(RowQuad& q, const float* __restrict__ W, const uint8_t* __restrict__ mask,
                                               const float* __restrict__ grad, size_t at, int n) {
    auto w = [&](int j) { return j < n ? W[at + j] : 0.0f; };
    auto g = [&](int j) { return j < n ? grad[at + j] : 0.0f; };
    auto m = [&](int j) { return j < n ? (uint32_t)mask[at + j] << (8 * j) : 0u; };
    q.m = m(0) | m(1) | m(2) | m(3);
    q.w = make_float4(w(0), w(1), w(2), w(3));
    q.g = make_float4(g(0), g(1), g(2), g(3));
}

// Steps 3 to 5 up to the counts: per neuron, how many weights it holds and how many salient ones, whether it stays
// (remains[r]; a neuron without weights stays ablated), and the layer's numbers of staying and newly ablated neurons (one
// atomic per workgroup and counter, spread over copies; read by the launches after this one).  One wavefront per row.  An
// ablated neuron's weights leave the counts of selection 0.
__global__ __launch_bounds__(256) void k_row_salient(const float* __restrict__ W, const uint8_t* __restrict__ mask,
                                                     const float* __restrict__ grad, int d_out, int d_in, unsigned int n_wg, int k, int gamma_percent,
                                                     UpdateScratch* __restrict__ s, int* __restrict__ remains) {
    __shared__ int wg_stay, wg_ablated;
    __shared__ __align__(16) unsigned int gone[kDigits];
    bool ablates = false;
    const int lane = threadIdx.x & 63;
    const unsigned int r = part_of_workgroup(blockIdx.x, n_wg) * 4 + (threadIdx.x >> 6);
    const bool row = is_row(r, d_out);
    if (threadIdx.x == 0) { wg_stay = 0; wg_ablated = 0; }
    const size_t row0 = (size_t)r * d_in;
    const bool quads = d_in >= 4;
    // the row's first kAhead steps are requested before the thresholds are (they do not depend on them)
    constexpr int kAhead = 4;
    RowQuad p[kAhead];
    if (row && quads) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (256 * u < d_in) load_row_quad(p[u], W, mask, grad, row0 + quad_first(4 * lane + 256 * u, d_in));
    }
    const unsigned long long t_small = s->fin[0].prefix, t_grad = s->fin[1].prefix;
    __syncthreads();
    int h = 0, sal = 0;
    auto element = [&](int c, int own, unsigned int m, float w, float g) {   // columns below `own` belong to the neighbour
        if (c < own || c >= d_in) return;
        const unsigned int i = (unsigned int)row0 + c;
        if (m) {
            ++h;
            if (key_small_first(mag_bits(w), i) < t_small) ++sal;    // survives the layer-wide pruning
        } else if (key_large_first(mag_bits(g), i) >= t_grad) {
            ++sal;                                                    // would be grown
        }
    };
    auto quad = [&](const RowQuad& q, int first, int own) {
        element(first + 0, own, q.m & 0xffu, q.w.x, q.g.x);
        element(first + 1, own, (q.m >> 8) & 0xffu, q.w.y, q.g.y);
        element(first + 2, own, (q.m >> 16) & 0xffu, q.w.z, q.g.z);
        element(first + 3, own, q.m >> 24, q.w.w, q.g.w);
    };
    if (row) {
        if (quads) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (256 * u < d_in) quad(p[u], quad_first(4 * lane + 256 * u, d_in), 4 * lane + 256 * u);
            for (int c = 4 * lane + 256 * kAhead; c < d_in; c += 256) {
                RowQuad q;
                load_row_quad(q, W, mask, grad, row0 + quad_first(c, d_in));
                quad(q, quad_first(c, d_in), c);
            }
        } else if (lane == 0) {
            RowQuad q;
            load_row_short(q, W, mask, grad, row0, d_in);
            quad(q, 0, 0);
        }
        h = (int)wave_total((unsigned)h);
        sal = (int)wave_total((unsigned)sal);
        const bool ablated = h > 0 && (sal < 1 || (long long)sal * 100 < (long long)gamma_percent * k);
        if (lane == 0) {
            if (ablated) atomicAdd(&wg_ablated, 1);
            if (h > 0 && !ablated) atomicAdd(&wg_stay, 1);
            remains[r] = h > 0 && !ablated ? 1 : 0;
        }
        ablates = ablated;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (wg_stay) atomicAdd(&s->cnt_remaining[blockIdx.x % kCountCopies], (unsigned int)wg_stay);
        if (wg_ablated) atomicAdd(&s->cnt_ablated[blockIdx.x % kCountCopies], (unsigned int)wg_ablated);
    }
    if (wg_ablated == 0) return;
    // The ablated rows' digits are counted in LDS first: an atomic in memory for every kept weight of theirs (and one for the coarse
    // digit) was most of the update where many neurons go (768 x 3072: 887 of 3072 ablated 104 us, 2969 of them 283).
    for (int i = threadIdx.x; i < kDigits / 4; i += 256) reinterpret_cast<uint4*>(gone)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    if (ablates)
        for (int c = lane; c < d_in; c += 64)
            if (mask[row0 + c] != 0) atomicAdd(&gone[digit_small_first(mag_bits(W[row0 + c]))], 1u);
    __syncthreads();
    const int copy = blockIdx.x % kHistCopies;   // (modulo 2^32 per copy: the copies' sum is what counts)
#pragma unroll
    for (int j = 0; j < kDigits / 256; ++j) {
        const unsigned int n = gone[threadIdx.x + 256 * j];
        if (n) atomicSub(&s->hist[0][copy][threadIdx.x + 256 * j], n);
    }
    static_assert(kCoarse == 256, "a coarse count per thread");
    unsigned int n = 0;
#pragma unroll
    for (int j = 0; j < kFine / 4; ++j) {
        const uint4 v = reinterpret_cast<const uint4*>(gone)[threadIdx.x * (kFine / 4) + j];
        n += v.x + v.y + v.z + v.w;
    }
    if (n) atomicSub(&s->coarse[0][copy][threadIdx.x], n);
}

// Steps 6 (applied) and 7.  WPR wavefronts per row (1, four rows to a workgroup, or 4); lane l of them holds columns
// 4 (l + 64 WPR q) .. + 3, q < NQ (d_in <= 256 WPR NQ).  Rows of more than 1024 columns take four wavefronts: with one, a wavefront's
// hundreds of instructions per count ran one after the other on two thirds of a machine that few rows fill (2240 x 1896
// 27 -> 18 us, 4096 x 1953 41 -> 25; shorter rows would pay for the barrier behind every count).  A column
// is ranked by one number (its weight's magnitude if it survives step 6, else its gradient's), equal numbers by column.  The
// `want`-th largest among the row's candidates is searched by counting (NQ x 4 compares, their ballots counted by scalar
// instructions) until a threshold splits off exactly `want`.
template <int NQ, int WPR, bool BESIDE>
__global__ __launch_bounds__(256) void k_row_update(const float* __restrict__ W, const uint8_t* __restrict__ mask, const float* __restrict__ grad,
                                                    int d_out, int d_in, unsigned int n_wg, const int* __restrict__ remains, const UpdateScratch* __restrict__ s,
                                                    uint8_t* __restrict__ mask_out, float* __restrict__ W_out) {
    constexpr int N = 4 * NQ;
    constexpr bool HOLD = NQ <= 4;   // the weights stay in registers (else they are read again where they are kept)
    static_assert(WPR == 1 || WPR == 4, "the workgroup's barrier is the row's");
    __shared__ int part[2][4];
    const int lane = WPR == 1 ? threadIdx.x & 63 : threadIdx.x;
    const unsigned int part_no = part_of_workgroup(blockIdx.x, n_wg), r = WPR == 1 ? part_no * 4 + (threadIdx.x >> 6) : part_no;
    if (!is_row(r, d_out)) return;
    const size_t row0 = (size_t)r * d_in;
    const bool quads = NQ > 1 || WPR > 1 || d_in >= 4;
    struct __attribute__((packed, aligned(4))) F4 { float x, y, z, w; };
    auto col0 = [&](int q) { return 4 * (lane + 64 * WPR * q); };
    // a number of each of the row's wavefronts, summed (two places in turn: one barrier per sum)
    int turn = 0;
    auto row_sum = [&](int n) {
        if (WPR == 1) return n;
        if ((threadIdx.x & 63) == 0) part[turn][threadIdx.x >> 6] = n;
        __syncthreads();
        const int total = part[turn][0] + part[turn][1] + part[turn][2] + part[turn][3];
        turn ^= 1;
        return __builtin_amdgcn_readfirstlane(total);
    };

    int rank[N];             // magnitude bits (below 2^31), or -1: not a column of the row
    uint32_t surv[(N + 31) / 32];
#pragma unroll
    for (int i = 0; i < (N + 31) / 32; ++i) surv[i] = 0u;
    float4 held[HOLD ? NQ : 1];
    const unsigned long long t_prune = s->t_prune;
    const long long k_new = s->k_new;
    const bool stays = remains[r] != 0;
    constexpr int STEP = NQ <= 6 ? NQ : 4;   // groups in flight
#pragma unroll
    for (int q0 = 0; q0 < NQ; q0 += STEP) {
        RowQuad in[STEP];
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
            if (q0 + u < NQ && ((BESIDE && q0 == 0) || stays)) {   // (BESIDE: the first ones beside `stays`, not behind it)
                if (quads) load_row_quad(in[u], W, mask, grad, row0 + quad_first(col0(q0 + u), d_in));
                else load_row_short(in[u], W, mask, grad, row0, d_in);
            }
        }
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
            const int q = q0 + u;
            if (q >= NQ) break;
            const int own = col0(q), first = quads ? quad_first(own, d_in) : 0;
            auto take = [&](int j, unsigned int m, float w, float g) {
                const int c = first + j;
                const bool valid = stays && c >= own && c < d_in;
                const bool sv = valid && m != 0 && key_small_first(mag_bits(w), (unsigned int)row0 + c) < t_prune;
                rank[4 * q + j] = valid ? (int)mag_bits(sv ? w : g) : -1;
                if (sv) surv[(4 * q + j) / 32] |= 1u << ((4 * q + j) % 32);
            };
            take(0, in[u].m & 0xffu, in[u].w.x, in[u].g.x);
            take(1, (in[u].m >> 8) & 0xffu, in[u].w.y, in[u].g.y);
            take(2, (in[u].m >> 16) & 0xffu, in[u].w.z, in[u].g.z);
            take(3, in[u].m >> 24, in[u].w.w, in[u].g.w);
            if (HOLD) held[q] = in[u].w;
        }
    }
    auto survives = [&](int e) { return ((surv[e / 32] >> (e % 32)) & 1u) != 0; };

    int kept = 0;
    {
        int mine = 0;
#pragma unroll
        for (int i = 0; i < (N + 31) / 32; ++i) mine += __popc(surv[i]);
        kept = row_sum((int)wave_total((unsigned)mine));
    }
    const int target = (int)k_new;   // at most d_in
    // trim: the row keeps its `target` largest surviving weights; grow: the `target - kept` largest gradients among its free positions
    const bool trim = kept > target;
    const int want = trim ? target : target - kept;
    int T = 0, last_col = d_in;      // a candidate is chosen if its rank is above T, or T and its column at most last_col
    if (stays && want > 0) {
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (survives(e) != trim) rank[e] = -1 - (rank[e] >= 0 ? 1 : 0);   // not a candidate (-2: a column all the same)
        auto count = [&](int thr) {
            int n = 0;
#pragma unroll
            for (int e = 0; e < N; ++e) n += __popcll(__ballot(rank[e] >= thr));
            return row_sum(n);
        };
        // count(T) >= want > count(hi).  Rows regrow close to the layer-wide gradient threshold of step 3, so the walk starts
        // there with steps that double, and halves the interval it lands in: about 8 counts on real-valued contents, where
        // the 31 bits one after the other took 22 (768 columns 12.1 -> 9.6 us, 2048 31.4 -> 24).
        int at_T = -1, hi = 0x7fffffff;
        if (!trim) {
            const unsigned int near = (unsigned int)(s->fin[1].prefix >> 32);
            int g = (int)min(max(near, 1u), 0x7ffffffeu), step = 1 << 20;   // (an eighth of an octave)
            const int n = count(g);
            if (n >= want) {
                T = g; at_T = n;
                while (at_T != want && step <= 0x7ffffffe - T) {
                    const int m = count(T + step);
                    if (m < want) { hi = T + step; break; }
                    T += step; at_T = m; step *= 2;
                }
            } else {
                hi = g;
                while (step < hi) {
                    const int m = count(hi - step);
                    if (m >= want) { T = hi - step; at_T = m; break; }
                    hi -= step; step *= 2;
                }
            }
        }
        while (at_T != want && hi - T > 1) {
            const int mid = T + (hi - T) / 2, n = count(mid);
            if (n >= want) { T = mid; at_T = n; } else hi = mid;
        }
        if (at_T != want && hi == 0x7fffffff && T == hi - 1) {   // (the one magnitude the walk leaves out)
            const int n = count(hi);
            if (n >= want) { T = hi; at_T = n; }
        }
        if (at_T != want) {   // equal ranks on both sides of the border (or T = 0): the lowest columns of them
            const int r_eq = want - (T == 0x7fffffff ? 0 : count(T + 1));
            auto eq_below = [&](int col) {
                int n = 0;
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    const int own = col0(e / 4), c = (quads ? quad_first(own, d_in) : 0) + e % 4;
                    n += __popcll(__ballot(rank[e] == T && c < col));
                }
                return row_sum(n);
            };
            int c = 0;            // the largest column with fewer than r_eq equal ranks in front of it
            for (int bit = 13; bit >= 0; --bit)
                if (c + (1 << bit) <= d_in && eq_below(c + (1 << bit)) < r_eq) c += 1 << bit;
            last_col = c;
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int own = col0(q), first = quads ? quad_first(own, d_in) : 0;
        if (own >= d_in) continue;
        bool keep[4], grow[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = 4 * q + j, c = first + j;
            const bool sv = survives(e);
            const bool chosen = want > 0 && rank[e] >= 0 && (rank[e] > T || (rank[e] == T && c <= last_col));
            keep[j] = stays && sv && (!trim || chosen);
            grow[j] = stays && !sv && !trim && chosen;
        }
        float4 w = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (HOLD) {
            if (stays) w = held[q];
        } else if (keep[0] || keep[1] || keep[2] || keep[3]) {
            const F4 v = *reinterpret_cast<const F4*>(W + row0 + first);   // (rows this long have whole groups)
            w = make_float4(v.x, v.y, v.z, v.w);
        }
        const F4 o = {keep[0] ? w.x : 0.0f, keep[1] ? w.y : 0.0f, keep[2] ? w.z : 0.0f, keep[3] ? w.w : 0.0f};
        const uint32_t m = (uint32_t)(keep[0] || grow[0]) | ((uint32_t)(keep[1] || grow[1]) << 8) | ((uint32_t)(keep[2] || grow[2]) << 16) |
                           ((uint32_t)(keep[3] || grow[3]) << 24);
        if (quads && first == own) {
            // (streamed: what stays in the L2 is written to memory at the launch's end, behind the last row's search: 3072 x 768 10.0 us of launch -> 9.0)
            typedef uint32_t U1 __attribute__((aligned(1)));
            typedef float F4v __attribute__((ext_vector_type(4), aligned(4)));
            const F4v ov = {o.x, o.y, o.z, o.w};
            __builtin_nontemporal_store(m, reinterpret_cast<U1*>(mask_out + row0 + first));
            __builtin_nontemporal_store(ov, reinterpret_cast<F4v*>(W_out + row0 + first));
        } else {
            const float of[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = first + j;
                if (c >= own && c < d_in) {
                    mask_out[row0 + c] = (uint8_t)(m >> (8 * j));
                    W_out[row0 + c] = of[j];
                }
            }
        }
    }
}

// A layer without elements: nothing stays, nothing is pruned.
__global__ void k_update_report_empty(long long* __restrict__ report) {
    if (threadIdx.x < 4) report[threadIdx.x] = 0;
}

// Keys per candidate list: a thirty-second of the layer, at least 4096.  A list holds the keys that share the threshold's first digit: about
// a percent of real-valued contents, three at most; more are contents of few magnitudes, which do better without a list (7 levels of
// weights and gradients on 768 x 3072, 5 % of the layer in one digit: 749 us with a list).
static size_t cand_capacity(int32_t d_out, int32_t d_in) {
    const size_t n = (d_out > 0 && d_in > 0) ? (size_t)d_out * (size_t)d_in : 0;
    const size_t c = n / 32;
    return c < 4096 ? 4096 : c / 2 * 2;   // (even: the second list is 16-byte aligned too)
}
static size_t update_head_bytes(int32_t d_out) {
    const size_t rows = d_out > 0 ? (size_t)d_out : 0;
    return ((sizeof(UpdateScratch) + rows * sizeof(int32_t) + 255) / 256) * 256;
}

}  // namespace srigl

using namespace srigl;

extern "C" {

size_t srigl_mask_update_workspace_bytes(int32_t d_out, int32_t d_in) {
    return update_head_bytes(d_out) + 2 * cand_capacity(d_out, d_in) * sizeof(unsigned long long);
}

srigl_status srigl_mask_update(const float* W, const uint8_t* mask, const float* grad, int32_t d_out, int32_t d_in, int32_t k,
                               int64_t K_upd, int32_t gamma_percent, int64_t budget, uint8_t* mask_out, float* W_out,
                               void* workspace, size_t workspace_bytes, int64_t* report_dev, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (d_out < 0 || d_in < 0 || k < 0 || k > d_in || K_upd < 0 || gamma_percent < 0 || budget < 0 || report_dev == nullptr)
        return SRIGL_ERR_INVALID_ARG;
    if ((long long)d_out * d_in >= (1ll << 32)) return SRIGL_ERR_UNSUPPORTED;   // positions are ranked as 32-bit numbers
    if (d_in > 8192) return SRIGL_ERR_UNSUPPORTED;                              // a row is held in the registers of one wavefront
    if (workspace == nullptr) return SRIGL_ERR_INVALID_ARG;
    if (workspace_bytes < srigl_mask_update_workspace_bytes(d_out, d_in)) return SRIGL_ERR_CAPACITY;
    const unsigned int N = (unsigned int)((long long)d_out * d_in);
    if (N > 0 && (W == nullptr || mask == nullptr || grad == nullptr || mask_out == nullptr || W_out == nullptr)) return SRIGL_ERR_INVALID_ARG;
    UpdateScratch* s = static_cast<UpdateScratch*>(workspace);
    int* remains = reinterpret_cast<int*>(static_cast<unsigned char*>(workspace) + sizeof(UpdateScratch));
    const unsigned long long cap = cand_capacity(d_out, d_in);
    unsigned long long* candA = reinterpret_cast<unsigned long long*>(static_cast<unsigned char*>(workspace) + update_head_bytes(d_out));
    unsigned long long* candB = candA + cap;
    long long* report = reinterpret_cast<long long*>(report_dev);
    if (N == 0) {
        hipLaunchKernelGGL(k_update_report_empty, dim3(1), dim3(64), 0, st, report);
        return hip_ok(hipGetLastError());
    }
    // Eight launches, each reading what the ones before it counted.  (What a kernel needs to know of its grid is an argument: gridDim, and blockDim, come
    // with 256 bytes of arguments of the runtime's own, which every launch of the kernel writes.)
    hipLaunchKernelGGL(k_update_init, dim3(kInitBlocks), dim3(256), 0, st, reinterpret_cast<uint4*>(s));
    // quads of the flat layer (16-byte moves need aligned arrays; rows of any length); at most one workgroup per compute unit
    const bool vec = reinterpret_cast<uintptr_t>(W) % 16 == 0 && reinterpret_cast<uintptr_t>(grad) % 16 == 0 && reinterpret_cast<uintptr_t>(mask) % 4 == 0;
    const unsigned int n4 = vec ? N / 4 : 0;
    unsigned int blocks = (unsigned int)(((unsigned long long)N + 4 * kScanThreads - 1) / (4 * kScanThreads));
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL(k_hist, dim3(blocks), dim3(kScanThreads), 0, st, W, mask, grad, N, n4, blocks, (n4 + blocks - 1) / blocks, s);
    hipLaunchKernelGGL(k_collect<true>, dim3(blocks), dim3(kScanThreads), 0, st, W, mask, grad, s, (unsigned long long)K_upd, n4, blocks,
                       (n4 + blocks - 1) / blocks, N, remains, d_in, candA, candB, cap);
    // Workgroups of k_final that stand by for a selection without a list (otherwise their start is all they cost: 45.0 us with 64, 44.7 with
    // none on 768 x 3072).  With 16 / 32 / 64 of them an update of that layer with zero gradients takes 127 / 92 / 79 us; on 4096 x 4097 64 take
    // 330 us and 256 285, on smaller layers 256 have too little to do each (1953 x 4096: 276, with 64 212).
    const unsigned int parts = N < (1u << 24) ? std::min(blocks, 64u) : (unsigned)kWideParts;
    hipLaunchKernelGGL(k_final<true>, dim3(2 * parts), dim3(kScanThreads), 0, st, s, candA, candB, cap, (unsigned long long)K_upd, (long long)budget,
                       (int)parts, d_in, W, mask, grad, remains, N, report);
    const dim3 row_grid(row_workgroups(d_out, 4));
    hipLaunchKernelGGL(k_row_salient, row_grid, dim3(256), 0, st, W, mask, grad, d_out, d_in, row_grid.x, k, gamma_percent, s, remains);
    // (most updates ablate nothing and this launch returns at once: it takes few workgroups, whose start is then all it costs)
    const unsigned int few = std::min(blocks, 64u);
    hipLaunchKernelGGL(k_collect<false>, dim3(few), dim3(kScanThreads), 0, st, W, mask, grad, s, (unsigned long long)K_upd, n4, few,
                       (n4 + few - 1) / few, N, remains, d_in, candA, candB, cap);
    hipLaunchKernelGGL(k_final<false>, dim3(parts), dim3(kScanThreads), 0, st, s, candA, candB, cap, (unsigned long long)K_upd, (long long)budget,
                       (int)parts, d_in, W, mask, grad, remains, N, report);
    // A row is requested beside the flag that says whether it stays where the layer is still near (real-valued, all rows staying: 1953 x 4096 82.5 us, 83.7
    // behind the flag); from 8 M elements on the memory's rate counts and rows that don't stay are not read: 4096 x 4096 with a fifth of the rows ablated 137 us -> 132,
    // 16384 x 4096 549 -> 528, 4096 x 2048 with a tenth 79 either way.
    const dim3 one_row_grid(row_workgroups(d_out, 1));
#define SRIGL_ROW_UPDATE(NQ, WPR)                                                                                                               \
    hipLaunchKernelGGL((N < (1u << 23) ? k_row_update<NQ, WPR, true> : k_row_update<NQ, WPR, false>), WPR == 1 ? row_grid : one_row_grid,       \
                       dim3(256), 0, st, W, mask, grad, d_out, d_in, (WPR == 1 ? row_grid : one_row_grid).x, remains, s, mask_out, W_out)
    const int nq = (d_in + 255) / 256;
    if (nq <= 1) SRIGL_ROW_UPDATE(1, 1);
    else if (nq <= 2) SRIGL_ROW_UPDATE(2, 1);
    else if (nq <= 3) SRIGL_ROW_UPDATE(3, 1);
    else if (nq <= 4) SRIGL_ROW_UPDATE(4, 1);
    else if (nq <= 8) SRIGL_ROW_UPDATE(2, 4);
    else if (nq <= 12) SRIGL_ROW_UPDATE(3, 4);
    else if (nq <= 16) SRIGL_ROW_UPDATE(4, 4);
    else if (nq <= 24) SRIGL_ROW_UPDATE(6, 4);
    else SRIGL_ROW_UPDATE(8, 4);
#undef SRIGL_ROW_UPDATE
    return hip_ok(hipGetLastError());
}

}  // extern "C"
