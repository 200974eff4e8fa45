// Rank-based selection kernels: the three-region partition at prefill (Sec. 3.3 "Prefilling Stage"), the
// per-step candidate top-k (Sec. 3.3 "Decoding Stage") and the index-list compactions around them.
//
// All selections use one strict total order on channels: higher score first, equal scores by lower channel
// index.  Scores are mapped to order-preserving 32-bit keys; the n-th best element is found in equal intervals of their range
// (by digits from the most significant bits down where they do not fit the LDS), so the result is deterministic.
#include "pop_select_dev.h"

namespace pop {

// ---------------------------------------------------------------- three-region partition
// One launch: every workgroup finds the rank thresholds for itself, from all keys, and then writes what belongs to its
// own 1024 channels.  Finding them in one place and handing them on would cost a launch or a grid-wide wait, as long as
// the search itself; done by everybody at once it costs nothing more, and the outputs (a dozen arrays in a layer's
// prefill) are written by the whole chip.
// Search: the keys sit in registers (NS per thread), as distances u from the largest key, so that the best channel has 0.
// One histogram over 8192 equal intervals between the largest and the smallest key leaves a threshold in an interval of a
// dozen keys, whose ranks are counted out pairwise.  (Intervals of the keys' range and not leading bits of the keys: scores on
// both sides of a power of two differ in their leading bits however close they are.)  An interval that holds more than a list
// is cut into 2048 again; where that ends at equal keys, they are counted out in channel order (part_equal_key).  One score far
// from the others (a channel of zeros, an infinity) makes every interval wide, and some hundred keys share one: then the second
// cut runs, 11008 channels 9.0 -> 12.3 us (leading bits took 15.6), 14336 11.2 -> 14.5 (18.3), 1376 7.4 -> 8.5 (9.0).
// A threshold is an element (key, channel): channels up to it in the order (key descending, channel ascending) are in.
// Bound by the sixteen waves' issue and the barriers: a sweep over all keys takes 0.6 to 1 us, a phase between two barriers half
// a microsecond at least, so there are seven phases of which two sweep.  Launches back to back: 11008 channels 13.6 -> 9.1 us,
// 14336 16.0 -> 10.3, up to 2800 at the rate of launches (the kernel itself 8.8 -> 5 us at 1376), against leading bits of the
// keys, a second histogram in most partitions and scans of each output's count; eight distinct scores 18.9 -> 18.0, all equal
// 8.5 -> 8.1.
constexpr int kPartThreads = 1024;
constexpr int kPartWaves = kPartThreads / kWave;
constexpr int kPartBits = 13, kPartBins = 1 << kPartBits;          // intervals of the first histogram
constexpr int kPartMoreBits = 11, kPartMoreBins = 1 << kPartMoreBits;  // of a further one (three of them at a time)
constexpr int kPartList = 64;      // keys of an interval counted out pairwise at most, one per lane
constexpr int kPartMaxSlots = 32;  // keys per thread held in registers at most: 32768 channels

struct PartShared {
    __attribute__((aligned(16))) unsigned int hist[kPartBins];
    __attribute__((aligned(16))) uint32_t list_u[3][kPartList];
    __attribute__((aligned(16))) int list_idx[3][kPartList];
    int list_len[3];
    uint32_t lo[3];                     // start of the threshold's interval
    int remaining[3], matching[3];      // rank within it, keys in it
    uint32_t thr_u[3];
    int thr_idx[3], base_list[3];       // base_list: keys of the list that are in and belong to earlier channels
    uint32_t extreme[2][kPartWaves], bits[kPartWaves];
    int wave_tot[3][kPartWaves];
    uint32_t own[2][3][kPartWaves];
};

// Inclusive scan within each row of 16 lanes.
__device__ __forceinline__ uint32_t row_incl_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
    return v;
}

// Exclusive scan of N streams over the workgroup.
template <int N>
__device__ __forceinline__ void part_scan(int (&v)[N], PartShared &sh)
{
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int inc[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        inc[q] = wave_incl_scan(v[q]);
        if (lane == kWave - 1) sh.wave_tot[q][wave] = inc[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const uint32_t ts = row_incl_scan((uint32_t)sh.wave_tot[q][lane % kPartWaves]);
        v[q] = (wave > 0 ? __builtin_amdgcn_readlane((int)ts, wave - 1) : 0) + inc[q] - v[q];
    }
}

// *idx = the rank-th (1 ..) channel among those whose key is key_max - want.  Every wave counts its own 64 channels of every
// key slot, 32 slots at a time, then finds the slot and wave where the rank is reached from all the counts (count: 512 words;
// counted: they are there already, from a call for the same key).  More than four keys per thread are read again: held in
// registers for this, they cost every partition half a microsecond.
template <int NS, int NK>
__device__ __forceinline__ void part_equal_key(const float *__restrict__ scores, const uint32_t (&u)[NK], int m,
                                               uint32_t key_max, uint32_t want, int rank, bool counted, int *count, int *idx)
{
    constexpr int kWaves = kPartWaves;
    const uint32_t want_key = key_max - want;
    static_assert(kPartMaxSlots * kWaves == 8 * kWave && 8 * kWave <= kPartBins, "eight counts per lane, in a histogram");
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (int base = 0; base < m; base += kPartMaxSlots * kPartThreads) {
        if (!counted) {
            int mine = 0;
            if constexpr (NS > 0 && NS <= 4) {
#pragma unroll
                for (int s = 0; s < NK; ++s) {
                    const int c = __builtin_popcountll(__ballot(s * kPartThreads + (int)threadIdx.x < m && u[s] == want));
                    mine = lane == s ? c : mine;
                }
            } else {
#pragma unroll 1
                for (int s = 0; s < kPartMaxSlots && base + s * kPartThreads < m; s += 8) {
                    float v[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {  // (requested together)
                        const int i = base + (s + q) * kPartThreads + (int)threadIdx.x;
                        v[q] = scores[i < m ? i : 0];
                    }
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const int i = base + (s + q) * kPartThreads + (int)threadIdx.x;
                        const int c = __builtin_popcountll(__ballot(i < m && score_key(v[q]) == want_key));
                        mine = lane == s + q ? c : mine;
                    }
                }
            }
            __syncthreads();  // the counts' readers are done
            if (lane < kPartMaxSlots) count[lane * kWaves + wave] = mine;
            __syncthreads();
        }
        int v[8], sum = 0;  // (slot, wave) in channel order
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = count[8 * lane + q], sum += v[q];
        const int inc = wave_incl_scan(sum);
        const unsigned long long hit = __ballot(inc - sum < rank && rank <= inc);
        if (hit == 0) {  // beyond these slots
            rank -= __builtin_amdgcn_readlane(inc, kWave - 1);
            continue;
        }
        const int at = __builtin_ctzll(hit);
        int before = __builtin_amdgcn_readlane(inc - sum, at), entry = 8 * at;
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            const int c = __builtin_amdgcn_readlane(v[q], at);
            if (entry == 8 * at + q && before + c < rank) before += c, ++entry;
        }
        if (wave == entry % kWaves) {
            const int i = base + entry / kWaves * kPartThreads + (int)threadIdx.x;
            const bool eq = i < m && score_key(scores[i < m ? i : 0]) == want_key;
            const unsigned long long eqs = __ballot(eq);
            if (eq && before + __builtin_popcountll(eqs & ((1ull << lane) - 1ull)) == rank - 1) *idx = i;
        }
        return;
    }
}

// What one channel's place in the partition writes; r, c, t: retained, candidate and top channels before it.
__device__ __forceinline__ void write_channel(const PartitionOutputs &o, int m, int n_cand, int j, int region, bool top,
                                              int r, int c, int t)
{
    if (o.scores_copy) o.scores_copy[j] = o.scores[j];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (o.region[q]) o.region[q][j] = (unsigned char)region;
        if (o.top_mask[q]) o.top_mask[q][j] = top ? 1 : 0;
    }
    for (int b = 0; b < o.rows; ++b) o.mask[(size_t)b * m + j] = region == POP_REGION_RETAINED ? 1 : 0;
    if (region == POP_REGION_CANDIDATE) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (o.cand_idx[q]) o.cand_idx[q][c] = j;
        if (o.rc_idx) o.rc_idx[c] = j;
    } else if (region == POP_REGION_RETAINED) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (o.ret_idx[q]) o.ret_idx[q][r] = j;
        for (int b = 0; b < o.rows; ++b) o.active_idx[(size_t)b * o.act_stride + r] = j;
        if (o.rc_idx) o.rc_idx[n_cand + r] = j;
        if (o.ulist) o.ulist[r] = j;
    }
    if (top && o.top_list) o.top_list[t] = j;
}

// NS keys per thread in registers, thread t those of channels t, t + 1024, ...; NS = 0: any number of channels, read again
// in every sweep, by one workgroup that writes all outputs.
template <int NS>
__global__ __launch_bounds__(kPartThreads) void partition_kernel(const float *__restrict__ scores, int m, int n_ret,
                                                                 int n_cand, int n_top, PartitionOutputs o)
{
    __shared__ PartShared sh;
    constexpr int NT = 3, NK = NS > 0 ? NS : 1;
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint32_t u[NK];
    if (NS > 0) {
        float v[NK];
#pragma unroll
        for (int s = 0; s < NK; ++s) {
            const int i = s * kPartThreads + tid;
            v[s] = scores[i < m ? i : 0];
        }
#pragma unroll
        for (int s = 0; s < NK; ++s) u[s] = __float_as_uint(v[s]);
    }
    if (blockIdx.x == 0 && tid < o.n_sync) o.sync[tid] = 0;
    if (blockIdx.x == 0 && tid == 0 && o.top_count) *o.top_count = n_top;
    for (int i = tid; i < kPartBins / 4; i += kPartThreads) reinterpret_cast<uint4 *>(sh.hist)[i] = make_uint4(0, 0, 0, 0);
    if (tid < NT) sh.list_len[tid] = sh.base_list[tid] = 0;
    if (tid < NT * kPartList) (&sh.list_u[0][0])[tid] = 0xffffffffu, (&sh.list_idx[0][0])[tid] = 0x7fffffff;  // (before nothing)

    const auto larger = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    const auto smaller = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
    const auto either = [](uint32_t a, uint32_t b) { return a | b; };
    uint32_t key_max = 0u, key_min = 0xffffffffu, bits = 0u;  // (bits: in which any two keys differ)
    if (NS > 0) {
#pragma unroll
        for (int s = 0; s < NK; ++s) u[s] = score_key(__uint_as_float(u[s]));
        const uint32_t key_0 = __builtin_amdgcn_readfirstlane(u[0]);
#pragma unroll
        for (int s = 0; s < NK; ++s) {  // (slots beyond the last channel repeat channel 0)
            key_max = larger(key_max, u[s]), key_min = smaller(key_min, u[s]), bits |= u[s] ^ key_0;
        }
    } else {
        const uint32_t key_0 = score_key(scores[0]);
        for (int i = tid; i < m; i += kPartThreads) {
            const uint32_t k = score_key(scores[i]);
            key_max = larger(key_max, k), key_min = smaller(key_min, k), bits |= k ^ key_0;
        }
    }
    key_max = wave_reduce_last(key_max, larger), key_min = wave_reduce_last(key_min, smaller);
    bits = wave_reduce_last(bits, either);
    if (lane == kWave - 1) sh.extreme[0][wave] = key_max, sh.extreme[1][wave] = key_min, sh.bits[wave] = bits;
    __syncthreads();
    key_max = __builtin_amdgcn_readfirstlane(row_reduce(sh.extreme[0][lane % kPartWaves], larger));
    key_min = __builtin_amdgcn_readfirstlane(row_reduce(sh.extreme[1][lane % kPartWaves], smaller));
    bits = __builtin_amdgcn_readfirstlane(row_reduce(sh.bits[lane % kPartWaves] | (sh.extreme[0][lane % kPartWaves] ^ key_max), either));
    // f(distance from the largest key, channel) for every key of this thread
    auto sweep = [&](auto f) {
        if (NS > 0) {
#pragma unroll
            for (int s = 0; s < NK; ++s) {
                const int i = s * kPartThreads + tid;
                if (i < m) f(u[s], i);
            }
        } else {
            for (int i = tid; i < m; i += kPartThreads) f(key_max - score_key(scores[i]), i);
        }
    };
    const uint32_t range = key_max - key_min;
    // Intervals are 2^shift wide; below the lowest bit in which keys differ there is nothing to cut (a few coarse scores come
    // to lie in neighbouring words of the histogram, and what stays crowded there is equal).
    const int low = bits ? __builtin_ctz(bits) : 0;
    int shift = max(low, 32 - kPartBits - (range ? __builtin_clz(range) : 32));
    if (NS > 0) {
#pragma unroll
        for (int s = 0; s < NK; ++s) u[s] = key_max - u[s];
    }

    // thresholds: retained (rank n_ret), retained + candidate (rank n_ret + n_cand), the n_top best; a set of none needs no
    // search (matching 0) and is closed at the end
    const int want[NT] = {n_ret, n_ret + n_cand, n_top};
    uint32_t lo[NT];
    int remaining[NT], matching[NT];
    auto take_interval = [&]() {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            lo[t] = __builtin_amdgcn_readfirstlane(sh.lo[t]);
            remaining[t] = __builtin_amdgcn_readfirstlane(sh.remaining[t]);
            matching[t] = __builtin_amdgcn_readfirstlane(sh.matching[t]);
        }
    };
    if (range == 0) {  // all equal (11008 additions to one word would take as long as all the rest)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            lo[t] = 0u, remaining[t] = max(want[t], 1), matching[t] = want[t] > 0 ? m : 0;
            if (tid == t) sh.remaining[t] = remaining[t];
        }
    } else {
        sweep([&](uint32_t v, int) { atomicAdd(&sh.hist[v >> shift], 1u); });
        __syncthreads();
        const uint4 h0 = reinterpret_cast<const uint4 *>(sh.hist)[2 * tid], h1 = reinterpret_cast<const uint4 *>(sh.hist)[2 * tid + 1];
        const int c[8] = {(int)h0.x, (int)h0.y, (int)h0.z, (int)h0.w, (int)h1.x, (int)h1.y, (int)h1.z, (int)h1.w};
        int v[1] = {((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]))};
        const int sum = v[0];
        part_scan<1>(v, sh);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int rank = max(want[t], 1);
            if (v[0] < rank && rank <= v[0] + sum) {
                int before = v[0], bin = 8 * tid, in_bin = 0;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const bool here = before < rank && rank <= before + c[q];
                    if (here) sh.remaining[t] = rank - before, bin = 8 * tid + q, in_bin = c[q];
                    before += c[q];
                }
                sh.lo[t] = (uint32_t)bin << shift, sh.matching[t] = want[t] > 0 ? in_bin : 0;
            }
        }
        __syncthreads();
        take_interval();
    }
    auto crowded = [&]() { return matching[0] > kPartList || matching[1] > kPartList || matching[2] > kPartList; };
    while (crowded() && shift > low) {
        const int next = max(shift - kPartMoreBits, low);
        for (int i = tid; i < NT * kPartMoreBins / 4; i += kPartThreads)
            reinterpret_cast<uint4 *>(sh.hist)[i] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        sweep([&](uint32_t v, int) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (v >= lo[t] && (v - lo[t]) >> shift == 0)
                    atomicAdd(&sh.hist[t * kPartMoreBins + ((v - lo[t]) >> next)], 1u);
        });
        __syncthreads();
        int c[NT][2], v[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const uint2 two = reinterpret_cast<const uint2 *>(sh.hist + t * kPartMoreBins)[tid];
            c[t][0] = (int)two.x, c[t][1] = (int)two.y;
            v[t] = c[t][0] + c[t][1];
        }
        part_scan<NT>(v, sh);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            int before = v[t];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (before < remaining[t] && remaining[t] <= before + c[t][q]) {
                    sh.lo[t] = lo[t] + ((uint32_t)(2 * tid + q) << next), sh.remaining[t] = remaining[t] - before;
                    sh.matching[t] = want[t] > 0 ? c[t][q] : 0;
                }
                before += c[t][q];
            }
        }
        __syncthreads();
        take_interval();
        shift = next;
    }
    // Each threshold's interval into its list; and how many channels before this workgroup's own (key slot blockIdx.x) lie in
    // the intervals before it.
    const int s_first = blockIdx.x, first = s_first * kPartThreads;
    bool listed[NT];
    uint32_t at[NT];
    int base[NT] = {0, 0, 0};  // (of this wave)
#pragma unroll
    for (int t = 0; t < NT; ++t) listed[t] = matching[t] > 0 && matching[t] <= kPartList, at[t] = matching[t] > 0 ? lo[t] >> shift : 0u;
    const bool lists = listed[0] || listed[1] || listed[2];
    if (lists) sweep([&](uint32_t v, int i) {
        const uint32_t p = v >> shift;
        if (p == at[0] || p == at[1] || p == at[2]) {  // (few)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (listed[t] && p == at[t]) {
                    const int e = atomicAdd(&sh.list_len[t], 1);
                    sh.list_u[t][e] = v, sh.list_idx[t][e] = i;
                }
        }
    });
    uint32_t mine = 0u;
    if (NS > 0) {
#pragma unroll
        for (int s = 0; s < NK; ++s) {
            if (s == s_first) mine = u[s];
            if (s < s_first && !crowded()) {
#pragma unroll
                for (int t = 0; t < NT; ++t) base[t] += __builtin_popcountll(__ballot(u[s] >> shift < at[t]));
            }
        }
    }
    if (lists) __syncthreads();
    if (lists && wave < NT) {  // a wave per threshold, a lane per key
        const int t = wave, len = __builtin_amdgcn_readfirstlane(sh.list_len[t]), rank = __builtin_amdgcn_readfirstlane(sh.remaining[t]);
        const uint32_t v = sh.list_u[t][lane];
        const int i = sh.list_idx[t][lane];
        int before = 0;
        for (int q0 = 0; q0 < len; q0 += 16) {  // (sixteen at a time: one LDS latency for all of them)
            uint4 uq[4];
            int4 iq[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uq[w] = *reinterpret_cast<const uint4 *>(&sh.list_u[t][q0 + 4 * w]);
                iq[w] = *reinterpret_cast<const int4 *>(&sh.list_idx[t][q0 + 4 * w]);
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                before += uq[w].x < v || (uq[w].x == v && iq[w].x < i);
                before += uq[w].y < v || (uq[w].y == v && iq[w].y < i);
                before += uq[w].z < v || (uq[w].z == v && iq[w].z < i);
                before += uq[w].w < v || (uq[w].w == v && iq[w].w < i);
            }
        }
        const bool have = lane < len;
        if (have && before == rank - 1) sh.thr_u[t] = v, sh.thr_idx[t] = i;
        const int earlier = __builtin_popcountll(__ballot(have && before < rank && i < first));
        if (lane == 0) sh.base_list[t] = earlier;
    }
    if (crowded()) {
        // more equal keys than a list holds: the remaining-th of them in channel order
        __syncthreads();
        int last = -1;
#pragma unroll 1
        for (int t = 0; t < NT; ++t) {  // (one copy of the code)
            if ((t == 0 ? matching[0] : (t == 1 ? matching[1] : matching[2])) <= kPartList) continue;
            const uint32_t v = t == 0 ? lo[0] : (t == 1 ? lo[1] : lo[2]);
            const int rank = t == 0 ? remaining[0] : (t == 1 ? remaining[1] : remaining[2]);
            if (tid == 0) sh.thr_u[t] = v;
            if (range == 0) {  // every key
                if (tid == 0) sh.thr_idx[t] = rank - 1;
            } else {
                const bool counted = m <= kPartMaxSlots * kPartThreads && last >= 0 && sh.lo[last] == v;
                part_equal_key<NS>(scores, u, m, key_max, v, rank, counted, reinterpret_cast<int *>(sh.hist), &sh.thr_idx[t]);
                last = t;
            }
        }
        __syncthreads();
    } else {
        __syncthreads();
    }
    uint32_t thr_u[NT];
    int thr_idx[NT], total[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        thr_u[t] = want[t] > 0 ? sh.thr_u[t] : 0u;
        thr_idx[t] = want[t] > 0 ? sh.thr_idx[t] : -1;
        total[t] = NS > 0 && !crowded() ? sh.base_list[t] : 0;
    }
    auto within = [&](int t, uint32_t v, int j) { return v < thr_u[t] || (v == thr_u[t] && j <= thr_idx[t]); };
    if (NS > 0 && crowded()) {  // (the channels before, with the thresholds at hand)
#pragma unroll
        for (int s = 0; s < NK; ++s)
            if (s < s_first) {
#pragma unroll
                for (int t = 0; t < NT; ++t) base[t] += __builtin_popcountll(__ballot(within(t, u[s], s * kPartThreads + tid)));
            }
    }
    const int s_last = NS > 0 ? s_first + 1 : (m + kPartThreads - 1) / kPartThreads;
    for (int s = s_first; s < s_last; ++s) {
        const int j = s * kPartThreads + tid;
        const uint32_t v = NS > 0 ? mine : key_max - score_key(scores[j < m ? j : 0]);
        bool in[NT];
        int pre[NT], all[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            in[t] = j < m && within(t, v, j);
            const unsigned long long b = __ballot(in[t]);
            all[t] = __builtin_popcountll(b);
            pre[t] = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
        }
        // the waves' counts (1024 together at most) and their shares of the channels before (below 32768), two to a word
        uint32_t(&own)[3][kPartWaves] = sh.own[s & 1];
        if (lane == 0) {
            own[0][wave] = (uint32_t)all[0] | (uint32_t)all[1] << 16;
            own[1][wave] = (uint32_t)all[2] | (uint32_t)base[2] << 16;
            own[2][wave] = (uint32_t)base[0] | (uint32_t)base[1] << 16;
        }
        __syncthreads();
        uint32_t sum[3], until[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint32_t ts = row_incl_scan(own[q][lane % kPartWaves]);
            until[q] = wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)ts, wave - 1) : 0u;
            sum[q] = (uint32_t)__builtin_amdgcn_readlane((int)ts, kPartWaves - 1);
        }
        const int n_in[NT] = {(int)(sum[0] & 0xffffu), (int)(sum[0] >> 16), (int)(sum[1] & 0xffffu)};
        const int earlier[NT] = {(int)(sum[2] & 0xffffu), (int)(sum[2] >> 16), (int)(sum[1] >> 16)};
        const int waves_before[NT] = {(int)(until[0] & 0xffffu), (int)(until[0] >> 16), (int)(until[1] & 0xffffu)};
        int place[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) place[t] = total[t] + earlier[t] + waves_before[t] + pre[t];
        if (j < m)
            write_channel(o, m, n_cand, j, in[0] ? POP_REGION_RETAINED : (in[1] ? POP_REGION_CANDIDATE : POP_REGION_PRUNED),
                          in[2], place[0], place[1] - place[0], place[2]);
#pragma unroll
        for (int t = 0; t < NT; ++t) total[t] += n_in[t];
    }
}

hipError_t launch_partition(const float *scores, int m, int n_ret, int n_cand, int n_top, const PartitionOutputs &o,
                            hipStream_t s)
{
    // A build per number of key slots in registers: a wider one than needed costs its empty slots' part of every sweep (11008
    // channels in 11 slots 9.1 us, 14336 in 14 slots 10.3, 20000 in 20 slots 11.8).
    const int slots = (m + kPartThreads - 1) / kPartThreads;
#define POP_PART(NS, WGS) \
    hipLaunchKernelGGL(partition_kernel<NS>, dim3(WGS), dim3(kPartThreads), 0, s, scores, m, n_ret, n_cand, n_top, o)
    if (slots <= 2) POP_PART(2, slots);
    else if (slots <= 4) POP_PART(4, slots);
    else if (slots <= 8) POP_PART(8, slots);
    else if (slots <= 11) POP_PART(11, slots);
    else if (slots <= 14) POP_PART(14, slots);
    else if (slots <= 20) POP_PART(20, slots);
    else if (slots <= kPartMaxSlots) POP_PART(kPartMaxSlots, slots);
    else POP_PART(0, 1);
#undef POP_PART
    return hipGetLastError();
}

// hc[t][c] = h_all[t][list[c]] for c < *n_list, and zero columns from there up to the next multiple of 64 (the
// direct-load GEMM reads them, against rows of zeros: they must not keep what an earlier, longer list left there).  A
// workgroup gathers 512 columns of kCompactRows tokens; a thread owns two adjacent columns (one 32-bit store).
constexpr int kCompactRows = 8;
__global__ __launch_bounds__(256) void compact_hidden_kernel(const uint16_t *__restrict__ h_all, int ldh, int T,
                                                             const int *__restrict__ list,
                                                             const int *__restrict__ n_list, uint16_t *__restrict__ hc,
                                                             int ldhc)
{
    const int a = *n_list;
    const int c = (blockIdx.x * 256 + (int)threadIdx.x) * 2;
    const int t0 = blockIdx.y * kCompactRows, t1 = min(T, t0 + kCompactRows);
    if (c >= a) {
        if (c < min((a + 63) / 64 * 64, ldhc))
            for (int t = t0; t < t1; ++t) *reinterpret_cast<uint32_t *>(hc + (size_t)t * ldhc + c) = 0u;
        return;
    }
    const int j0 = list[c], j1 = c + 1 < a ? list[c + 1] : -1;
    uint32_t v[kCompactRows];
#pragma unroll
    for (int u = 0; u < kCompactRows; ++u) {  // (requested together)
        const uint16_t *row = h_all + (size_t)min(t0 + u, T - 1) * ldh;
        v[u] = (uint32_t)row[j0] | (j1 >= 0 ? (uint32_t)row[j1] << 16 : 0u);
    }
#pragma unroll
    for (int u = 0; u < kCompactRows; ++u)
        if (t0 + u < t1) *reinterpret_cast<uint32_t *>(hc + (size_t)(t0 + u) * ldhc + c) = v[u];
}

hipError_t launch_compact_hidden(const uint16_t *h_all, int ldh, int T, const int *list, const int *n_list, int max_list,
                                 uint16_t *hc, int ldhc, hipStream_t s)
{
    // (63 columns beyond the longest list, for the zeros)
    dim3 grid((max_list + 63 + 511) / 512, (T + kCompactRows - 1) / kCompactRows);
    hipLaunchKernelGGL(compact_hidden_kernel, grid, dim3(256), 0, s, h_all, ldh, T, list, n_list, hc, ldhc);
    return hipGetLastError();
}

// ---------------------------------------------------------------- per-step candidate top-k
unsigned long long *g_select_trace = nullptr;  // profiling builds: where topk_kernel stamps its phases (else null)
void set_select_trace(unsigned long long *p) { g_select_trace = p; }

// One workgroup per sequence b.  Only candidate-dependent state is written: the candidate bytes of mask[b][:]
// and the selected suffix of active_idx[b][:]; the retained / pruned bytes and the retained prefix are constant
// for a partition (partition_kernel).
// With a union request (B > 1) every workgroup also leaves one byte per candidate position, and the workgroup
// that finishes last (an arrival counter; nobody waits) compacts the candidates selected by any sequence into
// list[n_ret..] and rewinds the counter.
__global__ __launch_bounds__(1024) void topk_kernel(const float *__restrict__ cscore, int cs_stride,
                                                    const int *__restrict__ cand_idx, int n_cand, int n_ret, int m,
                                                    BatchK kk, int act_stride, unsigned char *__restrict__ mask,
                                                    int *__restrict__ active_idx, int *__restrict__ n_active,
                                                    int *__restrict__ sel_idx, unsigned char *selflag,
                                                    int *union_ctr, int *__restrict__ union_list,
                                                    int *__restrict__ n_union, int keys_in_ext,
                                                    unsigned long long *tr)
{
    __shared__ SelShared sh;
    __shared__ int s_last;
    extern __shared__ uint32_t topk_keys[];  // [2 n_cand] when the launch gave it: candidate sets beyond sh.keys
    const int b = blockIdx.x, B = gridDim.x, k = kk.k[b];
    unsigned char *mk = mask ? mask + (size_t)b * m : nullptr;
    int *act = active_idx ? active_idx + (size_t)b * act_stride + n_ret : (b == 0 ? sel_idx : nullptr);
    // selflag: [n_cand][POP_MAX_BATCH], one 8-byte word per candidate position
    block_select_candidates(cscore + (size_t)b * cs_stride, cand_idx, n_cand, k, mk, act, sh, SelectNoHook(),
                            SelectNoHook(), b == 0 ? tr : nullptr, selflag ? selflag + b : nullptr, POP_MAX_BATCH, false,
                            keys_in_ext ? topk_keys : nullptr, keys_in_ext ? n_cand : 0);
    if (tr && b == 0 && threadIdx.x == 0) tr[6] = wall_clock64();
    if (n_active && threadIdx.x == 0) n_active[b] = n_ret + k;
    if (!union_list) return;
    // the flags of this sequence are written; the last workgroup to get here sees every sequence's flags
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(union_ctr, 1) == B - 1;
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    static_assert(POP_MAX_BATCH == 8, "one 64-bit word of flags per candidate position");
    const unsigned long long live = B >= 8 ? ~0ull : ((1ull << (8 * B)) - 1ull);  // bytes of sequences >= B are stale
    const unsigned long long *flags = reinterpret_cast<const unsigned long long *>(selflag);
    int E = (n_cand + blockDim.x - 1) / blockDim.x;
    int lo = min(n_cand, (int)threadIdx.x * E), hi = min(n_cand, lo + E);
    int c[1] = {0}, tot[1];
    for (int i = lo; i < hi; ++i) c[0] += (flags[i] & live) != 0;
    block_excl_scan<1>(c, tot, sh);
    int p = n_ret + c[0];
    for (int i = lo; i < hi; ++i)
        if ((flags[i] & live) != 0) union_list[p++] = cand_idx[i];
    if (threadIdx.x == 0) {
        *n_union = n_ret + tot[0];
        *union_ctr = 0;
    }
}

hipError_t launch_topk(const float *cscore, int cs_stride, const int *cand_idx, int n_cand, int n_ret, int m, int B,
                       BatchK k, int act_stride, unsigned char *mask, int *active_idx, int *n_active, int *sel_idx,
                       unsigned char *selflag, int *union_ctr, int *union_list, int *n_union, hipStream_t s)
{
    int threads = n_cand <= 2048 ? 256 : 1024;
    // candidate sets beyond the select's own key buffer (re-scoring all channels of a layer) get theirs from the launch
    const bool ext = n_cand > kSelLdsKeys && n_cand <= 16384;  // (keys and staged decisions: 8 bytes per candidate)
    const size_t lds = ext ? (size_t)n_cand * 8 : 0;
    if (lds > 32 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&topk_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(topk_kernel, dim3(B), dim3(threads), lds, s, cscore, cs_stride, cand_idx, n_cand, n_ret, m, k,
                       act_stride, mask, active_idx, n_active, sel_idx, selflag, union_ctr, union_list, n_union,
                       ext ? 1 : 0, g_select_trace);
    return hipGetLastError();
}

// mask[j] = 1 for retained channels, 0 for the others (until a selection sets candidates).
__global__ __launch_bounds__(256) void retained_mask_kernel(const unsigned char *__restrict__ region, int m,
                                                            unsigned char *__restrict__ mask)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < m) mask[j] = region[j] == POP_REGION_RETAINED ? 1 : 0;
}

hipError_t launch_retained_mask(const unsigned char *region, int m, unsigned char *mask, hipStream_t s)
{
    hipLaunchKernelGGL(retained_mask_kernel, dim3((m + 255) / 256), dim3(256), 0, s, region, m, mask);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void fill_int_kernel(int *__restrict__ p, int n, int value)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

hipError_t launch_fill_int(int *p, int n, int value, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_int_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n, value);
    return hipGetLastError();
}

// ---------------------------------------------------------------- list compaction
// list = ascending channels j with mask[r][j] != 0 for some row r < rows.
__global__ __launch_bounds__(1024) void mask_to_list_kernel(const unsigned char *__restrict__ mask, int rows, int m,
                                                            int *__restrict__ list, int *__restrict__ n_list,
                                                            uint16_t *__restrict__ pad_hc, int pad_ld, int pad_T)
{
    __shared__ SelShared sh;
    int E = (m + blockDim.x - 1) / blockDim.x;
    int lo = min(m, (int)threadIdx.x * E), hi = min(m, lo + E);
    int c[1] = {0}, tot[1];
    for (int j = lo; j < hi; ++j) {
        int any = 0;
        for (int r = 0; r < rows; ++r) any |= mask[(size_t)r * m + j];
        c[0] += (any != 0);
    }
    block_excl_scan<1>(c, tot, sh);
    int p = c[0];
    for (int j = lo; j < hi; ++j) {
        int any = 0;
        for (int r = 0; r < rows; ++r) any |= mask[(size_t)r * m + j];
        if (any) list[p++] = j;
    }
    if (threadIdx.x == 0) *n_list = tot[0];
    if (pad_hc) {
        const int a = tot[0], a_end = min((a + 63) / 64 * 64, pad_ld), w = a_end - a;
        for (int e = threadIdx.x; e < w * pad_T; e += blockDim.x) pad_hc[(size_t)(e / w) * pad_ld + a + e % w] = 0;
    }
}

// One mask: every workgroup of 1024 channels counts the whole mask for itself (a thread up to 64 channels, 16 at a time where the
// mask is aligned), so nobody waits for anybody and the list leaves in whole lines; the zero columns behind the list
// are dealt by token rows.  Latency is all there is to it: one trip for the mask and one barrier.  Whole call of 24 tokens,
// against one workgroup that reads the mask byte by byte, twice: d 1024, m 3000 23.1 -> 22.4 us, d 512, m 16383 30.8 -> 21.8;
// the launch alone at 13824 channels 7.5 -> 4.8.  (Bytes behind the last whole sixteen in a loop, which waits for each of them by
// itself, and sums over the lanes by way of the LDS: 23.7 and 23.1.)
constexpr int kListMaxChannels = 65536;
__global__ __launch_bounds__(1024) void mask_row_to_list_kernel(const unsigned char *__restrict__ mask, int m,
                                                                int *__restrict__ list, int *__restrict__ n_list,
                                                                uint16_t *__restrict__ pad_hc, int pad_ld, int pad_T)
{
    __shared__ int w_all[16], w_before[16], w_own[16];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int c0 = blockIdx.x * 1024, mine = c0 + tid;
    // Every request of a thread goes out before the first is waited for: no branch but the loops around them, and the bytes
    // behind the last whole sixteen are dealt to sixteen threads.
    const unsigned char own = mask[min(mine, m - 1)];
    uint32_t counts = 0;  // of the whole mask | of the blocks before this one << 16 (64 of a thread at most)
    if ((reinterpret_cast<uintptr_t>(mask) & 15) == 0) {
        const int rest = m / 16 * 16 + tid;  // (never before a block)
        const unsigned char last = mask[min(rest, m - 1)];
        for (int j = tid * 16; j + 16 <= m; j += 16 * 1024) {
            const uint4 v = *reinterpret_cast<const uint4 *>(mask + j);
            const uint32_t q[4] = {v.x, v.y, v.z, v.w};
            uint32_t n = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i)  // (any bit of a byte into its top bit)
                n += __popc((((q[i] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | q[i]) & 0x80808080u);
            counts += n | (j < c0 ? n << 16 : 0u);  // (c0 is a multiple of 16)
        }
        counts += rest < m && last != 0;
    } else {
        for (int j = tid * 16; j < m; j += 16 * 1024) {
            unsigned char v[16];
            uint32_t n = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = mask[min(j + i, m - 1)];
#pragma unroll
            for (int i = 0; i < 16; ++i) n += j + i < m && v[i] != 0;
            counts += n | (j < c0 ? n << 16 : 0u);
        }
    }
    counts = (uint32_t)wave_incl_scan((int)counts);  // (4096 of a wave at most)
    const bool on = mine < m && own != 0;
    const unsigned long long votes = __ballot(on);
    if (lane == kWave - 1) w_all[wave] = counts & 0xffff, w_before[wave] = counts >> 16, w_own[wave] = __popcll(votes);
    __syncthreads();
    int total = 0, at = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        total += w_all[q];
        at += w_before[q] + (q < wave ? w_own[q] : 0);
    }
    if (on) list[at + __popcll(votes & ((1ull << lane) - 1))] = mine;
    if (mine == 0) *n_list = total;
    if (pad_hc) {
        const int c = total + lane;  // (fewer than 64 columns)
        if (c < min((total + 63) / 64 * 64, pad_ld))
            for (int t = blockIdx.x * 16 + wave; t < pad_T; t += gridDim.x * 16) pad_hc[(size_t)t * pad_ld + c] = 0;
    }
}

hipError_t launch_mask_to_list(const unsigned char *mask, int rows, int m, int *list, int *n_list, hipStream_t s,
                               uint16_t *pad_hc, int pad_ld, int pad_T)
{
    if (rows == 1 && m <= kListMaxChannels) {
        hipLaunchKernelGGL(mask_row_to_list_kernel, dim3((m + 1023) / 1024), dim3(1024), 0, s, mask, m, list, n_list, pad_hc,
                           pad_ld, pad_T);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(mask_to_list_kernel, dim3(1), dim3(1024), 0, s, mask, rows, m, list, n_list, pad_hc, pad_ld,
                       pad_T);
    return hipGetLastError();
}

// any[j] = 1 where mask[r][j] != 0 for some row r.  any is cleared first; a thread owns 4 adjacent channels and a
// group of 32 rows and writes 1 where it saw a set byte (writers of one byte all write the same value).
constexpr int kAnyRows = 32;
__global__ __launch_bounds__(256) void mask_any_kernel(const unsigned char *__restrict__ mask, int rows, int m,
                                                       unsigned char *__restrict__ any)
{
    const int j = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (j >= m) return;
    const int n = min(4, m - j);
    const int r0 = blockIdx.y * kAnyRows, r1 = min(rows, r0 + kAnyRows);
    unsigned char acc[4] = {0, 0, 0, 0};
    for (int r = r0; r < r1; ++r)
        for (int q = 0; q < n; ++q) acc[q] |= mask[(size_t)r * m + j + q];
    for (int q = 0; q < n; ++q)
        if (acc[q]) any[j + q] = 1;
}

// any must have room for m rounded up to a multiple of 4 bytes.
hipError_t launch_mask_any(const unsigned char *mask, int rows, int m, unsigned char *any, hipStream_t s)
{
    hipError_t e = launch_fill_int((int *)any, (m + 3) / 4, 0, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mask_any_kernel, dim3((m + 1023) / 1024, (rows + kAnyRows - 1) / kAnyRows), dim3(256), 0, s, mask,
                       rows, m, any);
    return hipGetLastError();
}

// Scores of one batch step aggregated over its B sequences (Eq. 3 with the step's tokens and samples):
// cs[b][p] = n_j |h_bj| on entry; on exit every row holds sqrt(sum_b cs[b][p]^2) = n_j * ||h_{:,j}||_2.
__global__ __launch_bounds__(256) void aggregate_scores_kernel(float *__restrict__ cs, int cs_stride, int B, int n)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    double acc = 0.0;
    for (int b = 0; b < B; ++b) {
        const double v = (double)cs[(size_t)b * cs_stride + p];
        acc += v * v;
    }
    const float r = (float)sqrt(acc);
    for (int b = 0; b < B; ++b) cs[(size_t)b * cs_stride + p] = r;
}

hipError_t launch_aggregate_scores(float *cs, int cs_stride, int B, int n, hipStream_t s)
{
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(aggregate_scores_kernel, dim3((n + 255) / 256), dim3(256), 0, s, cs, cs_stride, B, n);
    return hipGetLastError();
}

}  // namespace pop
