// Workgroup-level rank selection shared by the selection kernels and the fused decode kernel.
//
// One strict total order on channels: higher score first, equal scores by lower channel index.  Scores are
// mapped to order-preserving 32-bit keys; an MSB-first radix select over four 8-bit digits finds the key of
// the n-th best element, and a block scan in index order admits elements equal to that key until the count
// is exact.  One workgroup handles one selection, so the result is deterministic.
#pragma once
#include "pop_internal.h"

namespace pop {

constexpr int kSelMaxWaves = 16;
constexpr int kSelLdsKeys = 4096;  // candidate keys staged in LDS when they fit (16 KiB)

struct SelShared {
    // digit histograms of three consecutive radix passes (radix_threshold), or 1024 intervals (interval_threshold)
    __attribute__((aligned(16))) unsigned int hist[4][256];
    uint32_t list[kWave], extreme[2][kSelMaxWaves];
    int wave_tot[6][kSelMaxWaves];
    int digit;
    int remaining;
    int list_len;
    uint32_t keys[kSelLdsKeys];
};

// Inclusive prefix sum over the 64 lanes of a wave with DPP moves (register-to-register: a few cycles per step,
// where a shuffle through the LDS crossbar costs a full LDS round trip per step).
__device__ __forceinline__ int wave_incl_scan(int v)
{
    // within each row of 16 lanes: shifts by 1, 2, 4, 8 (lanes without a source keep 0)
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    // across rows: last lane of row 0 -> row 1, of row 2 -> row 3; then last lane of row 1 -> rows 2 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

// Exclusive block scan of N integer streams at once.  Returns the exclusive prefix in v[], block totals in
// tot[].  All threads of the block must call.
template <int N>
__device__ __forceinline__ void block_excl_scan(int (&v)[N], int (&tot)[N], SelShared &sh)
{
    int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, nw = (blockDim.x + kWave - 1) / kWave;
    int inc[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        inc[q] = wave_incl_scan(v[q]);
        if (lane == kWave - 1) sh.wave_tot[q][wave] = inc[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) {
        // lane l < nw reads the total of wave l; a second in-wave scan gives every wave's base
        const int t = lane < nw ? sh.wave_tot[q][lane] : 0;
        const int ts = wave_incl_scan(t);
        const int base = wave > 0 ? __builtin_amdgcn_readlane(ts, wave - 1) : 0;
        const int total = __builtin_amdgcn_readlane(ts, kWave - 1);
        v[q] = base + inc[q] - v[q];
        tot[q] = total;
    }
    __syncthreads();
}

// op over each row of 16 lanes (every lane of the row gets it).
template <class Op>
__device__ __forceinline__ uint32_t row_reduce(uint32_t v, Op op)
{
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true));   // quad_perm 1,0,3,2
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true));   // quad_perm 2,3,0,1
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true));  // row_half_mirror
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true));  // row_mirror
    return v;
}

// op over the wave, in its last lane.
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce_last(uint32_t v, Op op)
{
    v = row_reduce(v, op);
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xa, 0xf, false));  // row_bcast:15
    return op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xc, 0xf, false));  // row_bcast:31
}

// hist[d] += 1 for every lane with valid set, d < 256.  Lanes of a wave that hold the same digit as its first
// valid lane are counted by that lane, and again for the rest as long as such a group covers a quarter of the wave;
// whatever is left adds on its own.  Scores of one layer share their exponent bits, so without this the leading
// digit of every key would hit one LDS word, one lane at a time; for well-spread digits the loop ends after one try.
__device__ __forceinline__ void wave_hist_add(unsigned int *hist, uint32_t d, bool valid)
{
    unsigned long long todo = __ballot(valid);
    const int lane = threadIdx.x % kWave;
#pragma unroll 1
    for (int it = 0; it < 4 && todo; ++it) {
        const int leader = __builtin_ctzll(todo);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, leader);
        const unsigned long long same = __ballot(valid && d == d0) & todo;
        const int n_same = __popcll(same);
        if (lane == leader) atomicAdd(&hist[d0], (unsigned int)n_same);
        todo &= ~same;
        if (n_same < kWave / 4) break;
    }
    if ((todo >> lane) & 1ull) atomicAdd(&hist[d], 1u);
}

// Key of the n_top-th best element among key(0..n), and how many elements equal to that key belong to the
// top n_top (taken in index order).  n_top == 0 gives take_eq = 0 with kth = 0xffffffff.
// MSB-first radix select over 8-bit digits, starting below the bits that all keys have in common.
template <class KeyFn>
__device__ __forceinline__ void radix_threshold(KeyFn key, int n, int n_top, SelShared &sh, uint32_t &kth,
                                                int &take_eq)
{
    if (n_top <= 0) {
        kth = 0xffffffffu;
        take_eq = 0;
        return;
    }
    // bits in which any two keys differ: OR over all keys of (key ^ key(0))
    unsigned int *scratch = &sh.hist[2][0];
    if (threadIdx.x == 0) scratch[0] = 0;
    if (threadIdx.x < 256) sh.hist[0][threadIdx.x] = 0;
    if (blockDim.x < 256)
        for (int i = threadIdx.x + blockDim.x; i < 256; i += blockDim.x) sh.hist[0][i] = 0;
    __syncthreads();
    const uint32_t k0 = key(0);
    uint32_t diff = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) diff |= key(i) ^ k0;
    diff |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)diff, 0xB1, 0xf, 0xf, true);   // quad_perm 1,0,3,2
    diff |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)diff, 0x4E, 0xf, 0xf, true);   // quad_perm 2,3,0,1
    diff |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)diff, 0x141, 0xf, 0xf, true);  // row_half_mirror
    diff |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)diff, 0x140, 0xf, 0xf, true);  // row_mirror
    if (threadIdx.x % 16 == 0 && diff) atomicOr(&scratch[0], diff);  // one lane per row of 16
    __syncthreads();
    diff = scratch[0];
    if (diff == 0) {  // all keys equal
        __syncthreads();
        kth = k0;
        take_eq = n_top;
        return;
    }
    const int top_bit = 31 - __builtin_clz(diff);          // highest bit in which keys differ
    const int n_pass = top_bit / 8 + 1;                     // digits below and including that bit
    uint32_t known = top_bit == 31 ? 0u : ~((2u << top_bit) - 1u);  // the common leading bits
    uint32_t prefix = k0 & known;
    int remaining = n_top;
    const int lane = threadIdx.x % kWave;
    // Pass p counts into hist[p % 3], and clears hist[(p + 1) % 3] for the next pass: that one was last read in
    // pass p - 2, which every wave had finished before any wave could pass the barrier of pass p - 1.  Every wave
    // then finds the digit for itself, so a pass has a single barrier.
    int pass = 0;
    for (int shift = (n_pass - 1) * 8; shift >= 0; shift -= 8, ++pass) {
        unsigned int *hist = sh.hist[pass % 3], *next = sh.hist[(pass + 1) % 3];
        if (threadIdx.x < 256) next[threadIdx.x] = 0;
        if (blockDim.x < 256)
            for (int i = threadIdx.x + blockDim.x; i < 256; i += blockDim.x) next[i] = 0;
        const int n_round = (n + blockDim.x - 1) / blockDim.x * blockDim.x;  // whole waves take part in the ballots
        if (pass == 0) {
            // leading digit: scores of one layer crowd into a few values of it
            for (int i = threadIdx.x; i < n_round; i += blockDim.x) {
                const uint32_t k = i < n ? key(i) : 0u;
                wave_hist_add(hist, (k >> shift) & 255u, i < n && (k & known) == prefix);
            }
        } else {
            // later digits are spread out (and few keys are left): one atomic each
            for (int i = threadIdx.x; i < n; i += blockDim.x) {
                const uint32_t k = key(i);
                if ((k & known) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
            }
        }
        __syncthreads();
        // lane l owns the four digits 255-4l .. 252-4l, scanned from the largest digit down
        int c[4], lane_tot = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = (int)hist[255 - (4 * lane + q)];
            lane_tot += c[q];
        }
        int before = wave_incl_scan(lane_tot) - lane_tot;
        int digit = -1, rem_new = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (before < remaining && remaining <= before + c[q]) {
                digit = 255 - (4 * lane + q);
                rem_new = remaining - before;
            }
            before += c[q];
        }
        const int owner = __builtin_ctzll(__ballot(digit >= 0));  // exactly one lane holds the digit
        digit = __builtin_amdgcn_readlane(digit, owner);
        remaining = __builtin_amdgcn_readlane(rem_new, owner);
        prefix |= ((uint32_t)digit) << shift;
        known |= 255u << shift;
    }
    __syncthreads();  // the caller may reuse the histograms
    kth = prefix;
    take_eq = remaining;
}

// The same for keys that are in LDS, with `cut` set when only some of the elements equal to kth belong to the top.  One histogram
// over 1024 equal intervals between the largest and the smallest key leaves the threshold in an interval of a few keys, which are
// ranked pairwise; an interval of more than 64 is cut again, down to equal keys.  Every wave reads the histogram and ranks the list for
// itself: three barriers and three sweeps over the keys (extremes, histogram, list), where the digits above take seven and five.
// Lanes that add to one word do so one at a time, so an interval that holds an eighth of the keys is measured before it is cut again, and
// keys equal to the smallest (the scores of dead channels, zero) are counted by the wave, in sets of more than 2048 (below, the look whether there
// are such costs a step of d 512, m 1376 0.3 us and saves less) where a wave's first keys show eight of them.  4096 candidates, nine tenths of
// them zero, whole call: half selected 26.6 us without these two, 11.2 with, 22.5 by digits; a twentieth selected 17.5, 14.4 and 14.6.
// One float32 step at d 512, m 1376 (550 candidates, two waves) 20.1 -> 16.1 us, two of d 1024, m 4000 39.7 -> 32.4, re-scoring all of 11008
// channels 134.4 -> 124.9 (two layers).
constexpr int kSelBits = 10, kSelBins = 1 << kSelBits;
template <class KeyFn>
__device__ __forceinline__ void interval_threshold(KeyFn key, int n, int n_top, SelShared &sh, uint32_t &kth, int &take, bool &cut)
{
    cut = false;
    if (n_top <= 0) {
        kth = 0xffffffffu;
        take = 0;
        return;
    }
    const auto larger = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int nw = (blockDim.x + kWave - 1) / kWave;
    unsigned int *const bins = &sh.hist[0][0];
    uint32_t *const list = &sh.list[0];
    for (int i = threadIdx.x; i < kSelBins / 4; i += blockDim.x) reinterpret_cast<uint4 *>(bins)[i] = make_uint4(0, 0, 0, 0);
    if (threadIdx.x == 0) sh.list_len = 0;
    // largest value and (as the largest complement) smallest over the workgroup; a barrier inside
    auto extremes = [&](uint32_t &most, uint32_t &inv_least) {
        most = wave_reduce_last(most, larger), inv_least = wave_reduce_last(inv_least, larger);
        if (lane == kWave - 1) sh.extreme[0][wave] = most, sh.extreme[1][wave] = inv_least;
        __syncthreads();
        const bool some = lane % 16 < nw;
        most = __builtin_amdgcn_readfirstlane(row_reduce(some ? sh.extreme[0][lane % 16] : 0u, larger));
        inv_least = __builtin_amdgcn_readfirstlane(row_reduce(some ? sh.extreme[1][lane % 16] : 0u, larger));
    };
    uint32_t key_max = 0u, inv_min = 0u;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const uint32_t k = key(i);
        key_max = larger(key_max, k), inv_min = larger(inv_min, ~k);
    }
    extremes(key_max, inv_min);
    const uint32_t range = key_max - ~inv_min;
    int remaining = n_top, matching = n;
    uint32_t lo = 0u;  // distances from the largest key; the interval is [lo, lo + 2^shift)
    int shift = 0;
    if (range != 0u) {
        shift = max(0, 32 - __builtin_clz(range) - kSelBits);
        int i = threadIdx.x;
        if (n > 2048 && __popcll(__ballot(i < n && key_max - key(i) == range)) >= 8) {
            int at_least = 0;  // of the wave, in its first lane, which takes part in every round
            for (; i < n; i += blockDim.x) {
                const uint32_t u = key_max - key(i);
                at_least += __popcll(__ballot(u == range));
                if (u != range) atomicAdd(&bins[u >> shift], 1u);
            }
            if (lane == 0) atomicAdd(&bins[range >> shift], (unsigned int)at_least);
        } else {
            for (; i < n; i += blockDim.x) atomicAdd(&bins[(key_max - key(i)) >> shift], 1u);
        }
        for (;;) {
            __syncthreads();
            // lane l owns bins 16 l .. 16 l + 15
            int c[16], sum = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint4 v = reinterpret_cast<const uint4 *>(bins)[4 * lane + q];
                c[4 * q] = (int)v.x, c[4 * q + 1] = (int)v.y, c[4 * q + 2] = (int)v.z, c[4 * q + 3] = (int)v.w;
                sum += (c[4 * q] + c[4 * q + 1]) + (c[4 * q + 2] + c[4 * q + 3]);
            }
            int before = wave_incl_scan(sum) - sum;
            const int owner = __builtin_ctzll(__ballot(before < remaining && remaining <= before + sum));
            int bin = 0, rest = 0, in_bin = 0;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                if (before < remaining && remaining <= before + c[q]) bin = 16 * lane + q, rest = remaining - before, in_bin = c[q];
                before += c[q];
            }
            lo += (uint32_t)__builtin_amdgcn_readlane(bin, owner) << shift;
            remaining = __builtin_amdgcn_readlane(rest, owner);
            matching = __builtin_amdgcn_readlane(in_bin, owner);
            if (matching <= kWave || shift == 0) break;
            __syncthreads();
            for (int i = threadIdx.x; i < kSelBins / 4; i += blockDim.x)
                reinterpret_cast<uint4 *>(bins)[i] = make_uint4(0, 0, 0, 0);
            uint32_t width = (1u << shift) - 1u;
            if (matching > n / 8) {
                // a crowd: cut what its keys span, which may be nothing (equal keys add to one word, one lane at a time)
                uint32_t inv_least = 0u, u_max = 0u;
                for (int i = threadIdx.x; i < n; i += blockDim.x) {
                    const uint32_t u = key_max - key(i);
                    if (u >= lo && u - lo <= width) u_max = larger(u_max, u), inv_least = larger(inv_least, ~u);
                }
                extremes(u_max, inv_least);
                lo = ~inv_least, width = u_max - lo;
                if (width == 0u) {
                    shift = 0;
                    break;
                }
                shift = 32 - __builtin_clz(width);
            } else {
                __syncthreads();
            }
            shift = max(0, shift - kSelBits);
            for (int i = threadIdx.x; i < n; i += blockDim.x) {
                const uint32_t u = key_max - key(i);
                if (u >= lo && u - lo <= width) atomicAdd(&bins[(u - lo) >> shift], 1u);
            }
        }
    }
    if (shift == 0) {  // equal keys
        kth = key_max - lo;
        take = remaining;
        cut = remaining < matching;
        return;
    }
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const uint32_t u = key_max - key(i);
        if (u >= lo && (u - lo) >> shift == 0) list[atomicAdd(&sh.list_len, 1)] = u;
    }
    __syncthreads();
    const uint32_t u = lane < matching ? list[lane] : 0xffffffffu;
    int less = 0, equal = 0;
    for (int q = 0; q < matching; ++q) {
        const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)u, q);
        less += v < u, equal += v == u;
    }
    const int at = __builtin_ctzll(__ballot(lane < matching && less < remaining && remaining <= less + equal));
    kth = key_max - (uint32_t)__builtin_amdgcn_readlane((int)u, at);
    take = remaining - __builtin_amdgcn_readlane(less, at);
    cut = take < __builtin_amdgcn_readlane(equal, at);
}

struct SelectNoHook {
    __device__ __forceinline__ void operator()(int) const {}
    __device__ __forceinline__ void operator()() const {}
};

// Select the best k of n_cand candidates (cs[i] is the score of channel cand_idx[i], cand_idx ascending).
// Writes, each if non-null: mk[cand_idx[i]] = selected (candidate bytes only; the bytes of retained and pruned
// channels are constant for a partition and written when the partition is made), act_sel[0..k) = selected
// channels ascending, selpos[i] = selected (by position in cand_idx).  on_selected(i) is called for every selected position before any of those global writes,
// then after_selected() by every thread (it may contain barriers): callers that only need the positions get
// them without waiting for the index loads.  All threads of the block must call.
// kCoherentScores: the scores were just written by other workgroups of the same kernel with write-through stores;
// read them with device-coherent loads (no cache invalidation needed).  kCoherentFlags: selpos is written through,
// for another workgroup of the same kernel to read.
template <bool kCoherentScores = false, class OnSelected = SelectNoHook, class AfterSelected = SelectNoHook,
          bool kCoherentFlags = false>
__device__ __forceinline__ void block_select_candidates(const float *__restrict__ cs, const int *__restrict__ cand_idx,
                                                        int n_cand, int k, unsigned char *__restrict__ mk,
                                                        int *__restrict__ act_sel, SelShared &sh,
                                                        OnSelected on_selected = OnSelected(),
                                                        AfterSelected after_selected = AfterSelected(),
                                                        unsigned long long *tr = nullptr,
                                                        unsigned char *__restrict__ selpos = nullptr,
                                                        int selpos_stride = 1, bool keys_ready = false,
                                                        uint32_t *keys_ext = nullptr, int keys_cap = 0)
{
#define SEL_STAMP(k) do { if (tr && threadIdx.x == 0) tr[k] = wall_clock64(); } while (0)
    SEL_STAMP(0);
    auto score = [&](int i) -> float {
        return kCoherentScores ? __hip_atomic_load(&cs[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : cs[i];
    };
    // keys_ready: the caller has put score_key(score) of every candidate into sh.keys (n_cand <= kSelLdsKeys) and
    // synchronised the block.  keys_ext: LDS of the caller's, 2 * keys_cap words, used instead of sh.keys (a large
    // candidate set then stays out of global memory after the first sweep as well; the second half stages the
    // decisions for the output pass)
    uint32_t *const keys = keys_ext ? keys_ext : sh.keys;
    const bool in_lds = n_cand <= (keys_ext ? keys_cap : kSelLdsKeys);
    // (large sets: the channel numbers the output pass needs are requested now, so that they are there by then)
    constexpr int kAhead = 12;
    int jj[kAhead];
    if (keys_ext && in_lds) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = u * blockDim.x + threadIdx.x;
            jj[u] = i < n_cand ? cand_idx[i] : 0;
        }
    }
    if (in_lds && !keys_ready) {
        // twelve independent loads in flight per thread: under a streaming load a trip to memory takes microseconds
        constexpr int kLoads = 12;
        for (int base = 0; base < n_cand; base += kLoads * blockDim.x) {
            float v[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int i = base + u * blockDim.x + threadIdx.x;
                v[u] = score(i < n_cand ? i : 0);
            }
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int i = base + u * blockDim.x + threadIdx.x;
                if (i < n_cand) keys[i] = score_key(v[u]);
            }
        }
        __syncthreads();
    }
    auto key = [&](int i) -> uint32_t { return in_lds ? keys[i] : score_key(score(i)); };
    uint32_t kth;
    int take;
    SEL_STAMP(1);
    bool cut = true;  // some of the elements equal to kth are out: which, their order says
    if (in_lds)
        interval_threshold(key, n_cand, k, sh, kth, take, cut);
    else
        radix_threshold(key, n_cand, k, sh, kth, take);
    SEL_STAMP(2);

    const int E = (n_cand + blockDim.x - 1) / blockDim.x;
    const int lo = min(n_cand, (int)threadIdx.x * E), hi = min(n_cand, lo + E);
    int cnt[2] = {0, 0}, tot[2];
    if (!cut) {  // (where the selected stand among themselves is of no interest yet)
        for (int i = threadIdx.x; i < n_cand; i += blockDim.x)
            if (k > 0 && key(i) >= kth) on_selected(i);
        after_selected();
    }
    for (int i = lo; i < hi; ++i) {
        uint32_t kv = key(i);
        cnt[0] += (kv == kth);
        cnt[1] += (kv > kth);
    }
    block_excl_scan<2>(cnt, tot, sh);
    SEL_STAMP(3);
    if (cut) {
        int eq = cnt[0];
        for (int i = lo; i < hi; ++i) {
            uint32_t kv = key(i);
            if ((kv > kth) || (kv == kth && eq < take)) on_selected(i);
            eq += (kv == kth);
        }
        SEL_STAMP(4);
        after_selected();
    }
    SEL_STAMP(5);
    // position of a selected element = (# greater before it) + (# admitted equal before it)
    if (keys_ext && in_lds) {
        // Large sets (the caller's LDS holds n_cand more words behind the keys): every thread leaves the decisions of
        // its contiguous range in LDS - the position among the selected, or -1 - and the outputs are then written
        // by consecutive threads for consecutive candidates: whole cache lines instead of one byte per lane 11 apart.
        int *code = reinterpret_cast<int *>(keys_ext + n_cand);
        int eq = cnt[0], gt = cnt[1];
        for (int i = lo; i < hi; ++i) {
            const uint32_t kv = key(i);
            const bool sel = (kv > kth) || (kv == kth && eq < take);
            code[i] = sel ? gt + min(eq, take) : -1;
            eq += (kv == kth);
            gt += (kv > kth);
        }
        __syncthreads();
        for (int base = 0; base < n_cand; base += kAhead * blockDim.x) {
            if (base > 0) {  // (beyond what was requested at the start)
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int i = base + u * blockDim.x + threadIdx.x;
                    jj[u] = i < n_cand ? cand_idx[i] : 0;
                }
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int i = base + u * blockDim.x + threadIdx.x;
                if (i < n_cand) {
                    const int c = code[i];
                    if (mk) mk[jj[u]] = c >= 0 ? 1 : 0;
                    if (selpos) {
                        if (kCoherentFlags)
                            coherent_store(&selpos[(size_t)i * selpos_stride], (unsigned char)(c >= 0 ? 1 : 0));
                        else
                            selpos[(size_t)i * selpos_stride] = c >= 0 ? 1 : 0;
                    }
                    if (c >= 0 && act_sel) act_sel[c] = jj[u];
                }
            }
        }
        return;
    }
    // the channel numbers of this thread's range are requested together, not one trip to memory per element
    constexpr int kPre = 12;
    int jpre[kPre];
#pragma unroll
    for (int u = 0; u < kPre; ++u) jpre[u] = lo + u < hi ? cand_idx[lo + u] : 0;
    int eq = cnt[0], gt = cnt[1];
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
        const int i = lo + u;
        if (i < hi) {
            uint32_t kv = key(i);
            bool sel = (kv > kth) || (kv == kth && eq < take);
            int pos = gt + min(eq, take);
            eq += (kv == kth);
            gt += (kv > kth);
            const int j = jpre[u];
            if (mk) mk[j] = sel ? 1 : 0;
            if (selpos) {  // the same decision by candidate position
                if (kCoherentFlags)
                    coherent_store(&selpos[(size_t)i * selpos_stride], (unsigned char)(sel ? 1 : 0));
                else
                    selpos[(size_t)i * selpos_stride] = sel ? 1 : 0;
            }
            if (sel && act_sel) act_sel[pos] = j;
        }
    }
    for (int i = lo + kPre; i < hi; ++i) {
        uint32_t kv = key(i);
        bool sel = (kv > kth) || (kv == kth && eq < take);
        int pos = gt + min(eq, take);
        eq += (kv == kth);
        gt += (kv > kth);
        int j = cand_idx[i];
        if (mk) mk[j] = sel ? 1 : 0;
        if (selpos) {
            if (kCoherentFlags)
                coherent_store(&selpos[(size_t)i * selpos_stride], (unsigned char)(sel ? 1 : 0));
            else
                selpos[(size_t)i * selpos_stride] = sel ? 1 : 0;
        }
        if (sel && act_sel) act_sel[pos] = j;
    }
}

}  // namespace pop
