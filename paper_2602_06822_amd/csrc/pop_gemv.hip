// Decode-step GEMVs over gathered channel rows (Sec. 3.4 two-step decoding), batch-general form.  Both are
// HBM-bandwidth bound: every weight byte of an active channel is read exactly once per step with 128-bit
// loads, contiguous per channel thanks to the channel-major layout w[j] = [gate | up | down].  The single-
// sequence decode step uses the fused kernel in pop_decode_fused.hip instead.
//
//   gateup: for each listed channel j and each of the B sequences,
//           h[b][j] = silu(x_b . W_gate[j,:]) * (x_b . W_up[j,:]); the first n_score listed channels (the
//           candidates) also get their step score I_j(t) = n_j * |h[b][j]| (Eq. 3 with a single token).
//   down:   y[b][:] = sum over listed j of h[b][j] * W_down[:, j], optionally masked per sequence.
//
// A wave owns a whole row at a time (gateup) or a 64-vector column chunk of a slab of rows (down); lanes
// stride the row in 16-byte vectors, so each wave-level load instruction fetches 1 KiB of contiguous HBM.
#include "pop_select_dev.h"
#include "pop_vec.h"

namespace pop {

// ---------------------------------------------------------------- gate/up GEMV
constexpr int kGuUnroll = 8;  // 16-byte loads per matrix in flight per lane within one group

// One listed channel j (list position p), one wave: h[b][j] = silu(x_b . gate_j) * (x_b . up_j) for the B sequences
// whose x is staged in LDS (xs [B][nvec]); positions p < n_score also get their step score.  kCoherent: the scores
// are written through, for workgroups of the same launch to read.
template <class V, int B, bool kCoherent>
__device__ __forceinline__ void gateup_row(const typename V::vec_t *__restrict__ w, int nvec,
                                           const typename V::vec_t *xs, int j, int p, int lane, float *__restrict__ h,
                                           int m, const float *__restrict__ nrm, float *cscore, int cs_stride,
                                           int n_score)
{
    typedef typename V::vec_t vec_t;
    // (many sequences: fewer row vectors in flight per lane, so that the sequences' accumulators stay in registers)
    constexpr int U = B >= 5 ? kGuUnroll / 2 : kGuUnroll;
    const int group = kWave * U;
    const int nvec_full = nvec / group * group;
    j = __builtin_amdgcn_readfirstlane(j);  // (one channel per wave)
    // The start of each row as one value: taken apart by the compiler (the base, the channel and the lane in one sum, per load) the
    // addresses cost registers and with them loads in flight.  Two layers: 13B shape, four sequences 122.5 -> 120.0 us, five
    // 124.1 -> 122.7; 7B shape, four 97.7 -> 95.4, six 100.0 -> 98.8; float32 d 1024, m 2816, three 48.6 -> 47.4, eight
    // 65.3 -> 64.0; two and three sequences of bf16 layers the same.  The pointers say that they are global: what comes out
    // of the asm as a plain pointer is read by flat loads, which count as LDS operations too and are waited for all at once.
    typedef __attribute__((address_space(1))) const raw_vec_t row_t;
    auto row_vec = [](row_t *p) -> decltype(auto) {
        if constexpr (V::kStream)
            return __builtin_nontemporal_load(p);
        else
            return (*p);  // (a reference)
    };
    row_t *g = (row_t *)(w + (uint64_t)(uint32_t)j * (uint32_t)channel_vectors(nvec, V::kElems == 8));
    row_t *u = g + nvec;
    asm("" : "+s"(g));
    asm("" : "+s"(u));
    // Two 16-byte vectors' products (sixteen exact products for bf16 rows) are summed in the row's accumulator type,
    // the pairs of a lane and then the lanes in double: a long float32 chain would round every add at the magnitude
    // of the largest product met so far, and so would a float32 tree over the lanes.
    static_assert(U % 2 == 0, "vectors are taken in pairs");
    double ag[B], au[B];
#pragma unroll
    for (int b = 0; b < B; ++b) ag[b] = au[b] = 0.0;

    for (int c0 = 0; c0 < nvec_full; c0 += group) {
        vec_t wg[U], wu[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            wg[q] = __builtin_bit_cast(vec_t, row_vec(&g[c0 + q * kWave + lane]));
            wu[q] = __builtin_bit_cast(vec_t, row_vec(&u[c0 + q * kWave + lane]));
        }
#pragma unroll
        for (int q = 0; q < U; q += 2) {
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const vec_t x0 = xs[b * nvec + c0 + q * kWave + lane], x1 = xs[b * nvec + c0 + (q + 1) * kWave + lane];
                ag[b] += (double)V::dot(wg[q + 1], x1, V::dot(wg[q], x0, (typename V::acc_t)0));
                au[b] += (double)V::dot(wu[q + 1], x1, V::dot(wu[q], x0, (typename V::acc_t)0));
            }
        }
    }
    // (two at a time: 13B shape, three sequences 117.7-118.5 -> 116.3-116.9 us, d 3200 76.2 -> 75.0, float32 d 1024, two sequences
    // 44.6 -> 43.7.  Not four sequences of float32 rows, whose sums spill: d 1000, four tokens 18.9 instead of 17.9.)
    constexpr int kTailUnroll = B <= (V::kElems == 8 ? 4 : 3) ? 2 : 1;
#pragma unroll kTailUnroll
    for (int c = nvec_full + lane; c < nvec; c += kWave) {
        const vec_t wg = __builtin_bit_cast(vec_t, row_vec(&g[c])), wu = __builtin_bit_cast(vec_t, row_vec(&u[c]));
#pragma unroll
        for (int b = 0; b < B; ++b) {
            vec_t xv = xs[b * nvec + c];
            ag[b] += (double)V::dot(wg, xv, (typename V::acc_t)0);
            au[b] += (double)V::dot(wu, xv, (typename V::acc_t)0);
        }
    }
    // Lanes: four values at a time (gate and up sums of two sequences) through halving exchanges inside the rows of
    // 16 lanes, then across the four rows; lanes 0 and 1 end up with the gate sums of the two sequences and fetch
    // the matching up sums from lanes 2 and 3.
#pragma unroll
    for (int b0 = 0; b0 < B; b0 += 2) {
        const double v4[4] = {ag[b0], au[b0], b0 + 1 < B ? ag[b0 + 1] : 0.0, b0 + 1 < B ? au[b0 + 1] : 0.0};
        double z = butterfly4_row_sum(v4, lane);
        z += __shfl_xor(z, 16, kWave);
        z += __shfl_xor(z, 32, kWave);
        const double zu = dpp_move<0x4E>(z);  // quad_perm 2,3,0,1
        const int b = b0 + lane;
        if (lane < 2 && b < B) {
            const float hv = silu_mul((float)z, (float)zu);
            h[(size_t)b * m + j] = hv;
            if (p < n_score) {
                const float sc = nrm[j] * fabsf(hv);
                if (kCoherent)
                    coherent_store(&cscore[(size_t)b * cs_stride + p], sc);
                else
                    cscore[(size_t)b * cs_stride + p] = sc;
            }
        }
    }
}

template <class V, int B>
__global__ __launch_bounds__(1024) void gateup_kernel(const typename V::vec_t *__restrict__ w, int nvec,
                                                     const typename V::vec_t *__restrict__ x,
                                                     const int *__restrict__ rows, int n_rows,
                                                     const int *__restrict__ n_rows_dev, float *__restrict__ h, int m,
                                                     const float *__restrict__ nrm, float *__restrict__ cscore,
                                                     int cs_stride, int n_score)
{
    typedef typename V::vec_t vec_t;
    extern __shared__ uint4 xs_raw[];
    vec_t *xs = reinterpret_cast<vec_t *>(xs_raw);  // [B][nvec]
    for (int i = threadIdx.x; i < B * nvec; i += blockDim.x) xs[i] = x[i];
    __syncthreads();

    const int n = n_rows_dev ? *n_rows_dev : n_rows;
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n_waves = gridDim.x * (blockDim.x / kWave);

    for (int p = blockIdx.x * (blockDim.x / kWave) + wave; p < n; p += n_waves)
        gateup_row<V, B, false>(w, nvec, xs, rows[p], p, lane, h, m, nrm, cscore, cs_stride, n_score);
}

// Batched decode with the selection inside: rows = candidates (n_cand) then retained channels (n_ret).  All but
// the last B workgroups evaluate the rows, candidates first, and signal an arrival once their candidate scores are
// acknowledged.  The last B workgroups wait, bounded, for all arrivals and run one sequence's top-k each, the last of
// them also the union of the selections, while the others go on with the retained channels: the selection costs
// no time of its own.  All workgroups are resident (at most one per compute unit is launched), so the wait ends;
// if it ever expires the error flag is raised and the step's selection is not made.
// The arrival counter is never rewound: a second word holds the arrivals expected before this launch, the selectors
// wait for that plus this launch's workers, and the last selector moves the word on.  Every worker arrives exactly
// once before the launch ends, whether or not a selector was still waiting for it, so the two words agree again
// at the start of the next launch whatever happened in this one.
struct GateupSelectArgs {
    const int *cand_idx;
    int n_cand, n_ret;
    BatchK k;
    int act_stride;
    unsigned char *mask;
    int *active_idx, *n_active;
    unsigned char *selflag;
    int *union_list, *n_union;
    int *counters;  // [0] arrivals (ever growing), [1] selectors done, [2] arrivals expected before this launch
    int *err_flag;
    int spin_limit;  // looks a selector's wait takes before it gives up
};

template <class V, int B>
__global__ __launch_bounds__(1024) void gateup_select_kernel(const typename V::vec_t *__restrict__ w, int nvec,
                                                            const typename V::vec_t *__restrict__ x,
                                                            const int *__restrict__ rows, float *__restrict__ h, int m,
                                                            const float *__restrict__ nrm, float *cscore, int cs_stride,
                                                            GateupSelectArgs sa)
{
    typedef typename V::vec_t vec_t;
    extern __shared__ uint4 xs_raw[];
    __shared__ SelShared sh;
    __shared__ int s_flag;
    vec_t *xs = reinterpret_cast<vec_t *>(xs_raw);  // [B][nvec]
    for (int i = threadIdx.x; i < B * nvec; i += blockDim.x) xs[i] = x[i];
    __syncthreads();

    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wpb = blockDim.x / kWave, n_wg = gridDim.x;
    const int n_cand = sa.n_cand, n = sa.n_cand + sa.n_ret;

    const int n_work = n_wg - B;  // workgroups that evaluate rows; the last B select
    if ((int)blockIdx.x < n_work) {
        // Rows are dealt to the waves of the working workgroups in list order, candidates first.  A workgroup
        // signals its arrival after its last round that holds a candidate (at once if it has none): its scores are
        // then acknowledged (write-through stores, counter wait, barrier).
        const int wg = blockIdx.x, stride = n_work * wpb;
        const int cand_rounds = wg * wpb < n_cand ? (n_cand - wg * wpb + stride - 1) / stride : 0;
        if (cand_rounds == 0 && threadIdx.x == 0) atomicAdd(&sa.counters[0], 1);
        for (int it = 0; it * stride + wg * wpb < n; ++it) {
            const int p = it * stride + wg * wpb + wave;
            if (p < n_cand)
                gateup_row<V, B, true>(w, nvec, xs, rows[p], p, lane, h, m, nrm, cscore, cs_stride, n_cand);
            else if (p < n)
                gateup_row<V, B, false>(w, nvec, xs, rows[p], p, lane, h, m, nrm, cscore, cs_stride, n_cand);
            if (it == cand_rounds - 1) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's scores are acknowledged
                __syncthreads();
                if (threadIdx.x == 0) atomicAdd(&sa.counters[0], 1);
            }
        }
        return;
    }

    const int b = blockIdx.x - n_work;  // this workgroup selects for sequence b
    const int target = sa.counters[2] + n_work;  // (written by the previous launch: an ordinary load)
    if (threadIdx.x == 0) {
        const bool ok = spin_until(&sa.counters[0], target, sa.spin_limit);
        if (!ok) *sa.err_flag = 1;
        s_flag = ok ? 1 : 0;
    }
    __syncthreads();
    if (s_flag) {
        block_select_candidates<true, SelectNoHook, SelectNoHook, true>(
            cscore + (size_t)b * cs_stride, sa.cand_idx, n_cand, sa.k.k[b], sa.mask + (size_t)b * m,
            sa.active_idx + (size_t)b * sa.act_stride + sa.n_ret, sh, SelectNoHook(), SelectNoHook(), nullptr,
            sa.selflag + b, POP_MAX_BATCH);
        if (threadIdx.x == 0) sa.n_active[b] = sa.n_ret + sa.k.k[b];
    }
    // The flags went out as write-through stores; once they are acknowledged the selector signs off.  The last
    // selector to do so reads every sequence's flags (coherent loads): union of the selections, counters rewound.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) s_flag = atomicAdd(&sa.counters[1], 1) == B - 1;
    __syncthreads();
    if (!s_flag) return;
    static_assert(POP_MAX_BATCH == 8, "one 64-bit word of flags per candidate position");
    const unsigned long long live = B >= 8 ? ~0ull : ((1ull << (8 * B)) - 1ull);
    const unsigned long long *flags = reinterpret_cast<const unsigned long long *>(sa.selflag);
    // this thread's candidate positions: flags and channel numbers requested together
    constexpr int kPre = 4;
    const int E = (n_cand + blockDim.x - 1) / blockDim.x;
    const int lo = min(n_cand, (int)threadIdx.x * E), hi = min(n_cand, lo + E);
    unsigned long long fpre[kPre];
    int jpre[kPre];
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
        fpre[u] = lo + u < hi ? coherent_load(&flags[lo + u]) & live : 0ull;
        jpre[u] = lo + u < hi ? sa.cand_idx[lo + u] : 0;
    }
    int c[1] = {0}, tot[1];
#pragma unroll
    for (int u = 0; u < kPre; ++u) c[0] += fpre[u] != 0;
    for (int i = lo + kPre; i < hi; ++i) c[0] += (coherent_load(&flags[i]) & live) != 0;
    block_excl_scan<1>(c, tot, sh);
    int pos = sa.n_ret + c[0];
#pragma unroll
    for (int u = 0; u < kPre; ++u)
        if (fpre[u] != 0) sa.union_list[pos++] = jpre[u];
    for (int i = lo + kPre; i < hi; ++i)
        if ((coherent_load(&flags[i]) & live) != 0) sa.union_list[pos++] = sa.cand_idx[i];
    if (threadIdx.x == 0) {
        *sa.n_union = sa.n_ret + tot[0];
        sa.counters[1] = 0;
        sa.counters[2] = target;
    }
}

template <class V>
static hipError_t gateup_dispatch(const void *w, int nvec, const void *x, int B, const int *rows, int n_rows,
                                  const int *n_rows_dev, float *h, int m, const float *nrm, float *cscore, int cs_stride,
                                  int n_score, int n_cu, hipStream_t s)
{
    typedef typename V::vec_t vec_t;
    if (n_rows <= 0) return hipSuccess;
    // x is staged in LDS by every workgroup: with several sequences it fills most of it, so one large workgroup
    // per compute unit (16 waves sharing the copy) takes the place of many small ones
    size_t lds = (size_t)B * nvec * sizeof(vec_t);
    const int threads = lds > 16 * 1024 ? 1024 : 256;
    const int wpb = threads / kWave;
    int blocks = (n_rows + wpb - 1) / wpb;
    const int cap = threads == 1024 ? n_cu : 1024;
    if (blocks > cap) blocks = cap;
#define POP_GU(BB)                                                                                                  \
    case BB:                                                                                                        \
        if (lds > 48 * 1024) {                                                                                      \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gateup_kernel<V, BB>),               \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);               \
            if (e != hipSuccess) return e;                                                                          \
        }                                                                                                           \
        hipLaunchKernelGGL((gateup_kernel<V, BB>), dim3(blocks), dim3(threads), lds, s, (const vec_t *)w, nvec,          \
                           (const vec_t *)x, rows, n_rows, n_rows_dev, h, m, nrm, cscore, cs_stride, n_score);       \
        break;
    switch (B) {
        POP_GU(1) POP_GU(2) POP_GU(3) POP_GU(4) POP_GU(5) POP_GU(6) POP_GU(7) POP_GU(8)
        default: return hipErrorInvalidValue;
    }
#undef POP_GU
    return hipGetLastError();
}

hipError_t launch_gateup(const void *w, int is_bf16, int d, int m, const void *x, int B, const int *rows, int n_rows,
                         const int *n_rows_dev, float *h, const float *nrm, float *cscore, int cs_stride, int n_score,
                         int n_cu, long long stream_from, hipStream_t s)
{
    if (stream_rows(d, m, is_bf16, stream_from))
        return gateup_dispatch<StreamBF16>(w, d / 8, x, B, rows, n_rows, n_rows_dev, h, m, nrm, cscore, cs_stride,
                                           n_score, n_cu, s);
    if (is_bf16)
        return gateup_dispatch<VecBF16>(w, d / 8, x, B, rows, n_rows, n_rows_dev, h, m, nrm, cscore, cs_stride,
                                        n_score, n_cu, s);
    return gateup_dispatch<VecF32>(w, d / 4, x, B, rows, n_rows, n_rows_dev, h, m, nrm, cscore, cs_stride, n_score,
                                   n_cu, s);
}

template <class V>
static hipError_t gateup_select_dispatch(const void *w, int nvec, const void *x, int B, const int *rows, float *h, int m,
                                         const float *nrm, float *cscore, int cs_stride, const GateupSelectArgs &sa,
                                         int n_cu, bool *fused, hipStream_t s)
{
    typedef typename V::vec_t vec_t;
    *fused = false;
    const int n_rows = sa.n_cand + sa.n_ret, threads = 1024, wpb = threads / kWave;
    const size_t lds = (size_t)B * nvec * sizeof(vec_t);
    int blocks = (n_rows + wpb - 1) / wpb;
    if (blocks > n_cu) blocks = n_cu;
    if (B < 2 || blocks < 2 * B || sa.n_cand < 1) return hipSuccess;  // too small to set workgroups aside
#define POP_GS(BB)                                                                                                  \
    case BB: {                                                                                                      \
        const void *fn = reinterpret_cast<const void *>(&gateup_select_kernel<V, BB>);                               \
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                \
        if (e != hipSuccess) return e;                                                                               \
        int per_cu = 0;                                                                                              \
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gateup_select_kernel<V, BB>, threads, lds);        \
        if (e != hipSuccess) return e;                                                                               \
        if (per_cu < 1) return hipSuccess; /* not resident: the caller uses the two-launch form */                   \
        hipLaunchKernelGGL((gateup_select_kernel<V, BB>), dim3(blocks), dim3(threads), lds, s, (const vec_t *)w,     \
                           nvec, (const vec_t *)x, rows, h, m, nrm, cscore, cs_stride, sa);                          \
        break;                                                                                                       \
    }
    switch (B) {
        POP_GS(2) POP_GS(3) POP_GS(4) POP_GS(5) POP_GS(6) POP_GS(7) POP_GS(8)
        default: return hipErrorInvalidValue;
    }
#undef POP_GS
    *fused = true;
    return hipGetLastError();
}

hipError_t launch_gateup_select(const void *w, int is_bf16, int d, int m, const void *x, int B, const int *rows,
                                float *h, const float *nrm, float *cscore, int cs_stride, const int *cand_idx,
                                int n_cand, int n_ret, BatchK k, int act_stride, unsigned char *mask, int *active_idx,
                                int *n_active, unsigned char *selflag, int *union_list, int *n_union, int *counters,
                                int *err_flag, int spin_limit, int n_cu, bool *fused, hipStream_t s)
{
    GateupSelectArgs sa = {cand_idx, n_cand, n_ret, k, act_stride, mask, active_idx, n_active, selflag,
                           union_list, n_union, counters, err_flag, spin_limit};
    if (stream_rows(d, m, is_bf16, kStreamStepBytes))
        return gateup_select_dispatch<StreamBF16>(w, d / 8, x, B, rows, h, m, nrm, cscore, cs_stride, sa, n_cu, fused, s);
    if (is_bf16)
        return gateup_select_dispatch<VecBF16>(w, d / 8, x, B, rows, h, m, nrm, cscore, cs_stride, sa, n_cu, fused, s);
    return gateup_select_dispatch<VecF32>(w, d / 4, x, B, rows, h, m, nrm, cscore, cs_stride, sa, n_cu, fused, s);
}

// ---------------------------------------------------------------- down projection
// grid = (column chunks of 64 vectors, slabs).  A workgroup first stages its slab's channel list and the B
// sequences' hidden activations of those channels (zeroed where a sequence's mask excludes the channel) in LDS,
// with independent loads, so that the streaming loop touches global memory for weight rows only.  The 4 waves
// then split the slab's rows, keep float32 accumulators for their 64-vector column chunk, and are combined
// through LDS in wave order; the slab partials are then summed in slab order by down_reduce_kernel, so y does
// not depend on scheduling.
constexpr int kDownUnroll = 8;
constexpr int kDownSlabRows = 256;  // rows of a slab staged at a time

template <class V, int B>
__global__ __launch_bounds__(256) void down_kernel(const typename V::vec_t *__restrict__ w, int nvec,
                                                   const int *__restrict__ list, int n_host,
                                                   const int *__restrict__ n_dev, const float *__restrict__ h, int m,
                                                   const unsigned char *__restrict__ mask, int mask_stride,
                                                   float *__restrict__ partial, int d)
{
    typedef typename V::vec_t vec_t;
    constexpr int E = V::kElems;
    __shared__ float red[3][kWave * 8];
    __shared__ int js[kDownSlabRows];
    __shared__ float hs[B][kDownSlabRows];
    const int n = n_dev ? *n_dev : n_host;
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n_slabs = gridDim.y, slab = blockIdx.y;
    const int col = blockIdx.x * kWave + lane;  // vector column
    const bool col_ok = col < nvec;
    const uint32_t chan = channel_vectors(nvec, V::kElems == 8);
    const vec_t *w_down = w + 2 * nvec + col;
    const int per_slab = (n + n_slabs - 1) / n_slabs;
    const int s0 = min(n, slab * per_slab), s1 = min(n, s0 + per_slab);

    float acc[B][8];
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[b][e] = 0.f;

    for (int c0 = s0; c0 < s1; c0 += kDownSlabRows) {
        const int nc = min(kDownSlabRows, s1 - c0);
        __syncthreads();  // the previous chunk's readers are done
        for (int i = threadIdx.x; i < nc; i += blockDim.x) {
            const int j = list[c0 + i];
            js[i] = j;
            float hv[B];
            unsigned char mk[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                hv[b] = h[(size_t)b * m + j];
                mk[b] = mask ? mask[(size_t)b * mask_stride + j] : (unsigned char)1;
            }
#pragma unroll
            for (int b = 0; b < B; ++b) hs[b][i] = mk[b] ? hv[b] : 0.f;
        }
        __syncthreads();
        // rows of this wave within the chunk
        const int per_wave = (nc + 3) / 4;
        const int r0 = min(nc, wave * per_wave), r1 = min(nc, r0 + per_wave);
        int i = r0;
        for (; i + kDownUnroll <= r1; i += kDownUnroll) {
            vec_t wv[kDownUnroll];
#pragma unroll
            for (int q = 0; q < kDownUnroll; ++q)
                wv[q] = col_ok ? load_row<V>(w_down, (uint64_t)(uint32_t)js[i + q] * chan) : V::zero();
#pragma unroll
            for (int q = 0; q < kDownUnroll; ++q)
#pragma unroll
                for (int b = 0; b < B; ++b) V::axpy(hs[b][i + q], wv[q], acc[b]);
        }
        for (; i < r1; ++i) {
            const vec_t wv1 = col_ok ? load_row<V>(w_down, (uint64_t)(uint32_t)js[i] * chan) : V::zero();
#pragma unroll
            for (int b = 0; b < B; ++b) V::axpy(hs[b][i], wv1, acc[b]);
        }
    }

    // combine the 4 waves in wave order, one sequence at a time
#pragma unroll
    for (int b = 0; b < B; ++b) {
        __syncthreads();
        if (wave > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) red[wave - 1][e * kWave + lane] = acc[b][e];
        }
        __syncthreads();
        if (wave == 0 && col_ok) {
            float *dst = partial + ((size_t)slab * B + b) * d + (size_t)col * E;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                float v = acc[b][e];
                v += red[0][e * kWave + lane];
                v += red[1][e * kWave + lane];
                v += red[2][e * kWave + lane];
                dst[e] = v;
            }
        }
    }
}

// y[b][o] = sum over slabs of partial[slab][b][o]; total = B*d outputs.  A workgroup owns 64 outputs; its 4
// waves each sum a contiguous quarter of the slabs (independent loads, added in slab order) and are combined in
// wave order, so the result does not depend on scheduling.  Sums in double: the slabs' partial sums are of the size of
// the result, so a float32 chain over them would cost more than everything before it.
__global__ __launch_bounds__(256) void down_reduce_kernel(const float *__restrict__ partial, int n_slabs, int total,
                                                          void *__restrict__ y, int y_bf16, StepCopy copy)
{
    const int main_blocks = (total + kWave - 1) / kWave;
    if ((int)blockIdx.x >= main_blocks) {  // what the step's caller takes of its selection
        copy_step_block(copy, blockIdx.x - main_blocks, gridDim.x - main_blocks);
        return;
    }
    __shared__ double part[4][kWave];
    const int lane = threadIdx.x % kWave, q = threadIdx.x / kWave;
    const int i = blockIdx.x * kWave + lane;
    const int per = (n_slabs + 3) / 4, s0 = min(n_slabs, q * per), s1 = min(n_slabs, s0 + per);
    double acc = 0.0;
    if (i < total) {
        int s = s0;
        for (; s + 8 <= s1; s += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(s + u) * total + i];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += (double)v[u];
        }
        for (; s < s1; ++s) acc += (double)partial[(size_t)s * total + i];
    }
    part[q][lane] = acc;
    __syncthreads();
    if (q == 0 && i < total) {
        const float v = (float)(((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]);
        if (y_bf16)
            ((uint16_t *)y)[i] = f32_to_bf16(v);
        else
            ((float *)y)[i] = v;
    }
}

static hipError_t launch_down_reduce(const float *partial, int n_slabs, int total, void *y, int y_bf16, const StepCopy *copy,
                                     hipStream_t s)
{
    const StepCopy c = copy ? *copy : StepCopy{};
    hipLaunchKernelGGL(down_reduce_kernel, dim3((total + kWave - 1) / kWave + c.blocks(256)), dim3(256), 0, s, partial, n_slabs,
                       total, y, y_bf16, c);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void step_copy_kernel(StepCopy c) { copy_step_block(c, blockIdx.x, gridDim.x); }

hipError_t launch_step_copy(const StepCopy &c, hipStream_t s)
{
    const int blocks = c.blocks(256);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(step_copy_kernel, dim3(blocks), dim3(256), 0, s, c);
    return hipGetLastError();
}

template <class V>
static hipError_t down_dispatch(const void *w, int nvec, int d, int m, const int *list, const int *n_dev, int n_host,
                                const float *h, const unsigned char *mask, int mask_stride, int B, float *partial,
                                int n_slabs, void *y, int y_bf16, hipStream_t s, const StepCopy *copy)
{
    typedef typename V::vec_t vec_t;
    dim3 grid((nvec + kWave - 1) / kWave, n_slabs);
#define POP_DN(BB)                                                                                                  \
    case BB:                                                                                                        \
        hipLaunchKernelGGL((down_kernel<V, BB>), grid, dim3(256), 0, s, (const vec_t *)w, nvec, list, n_host,        \
                           n_dev, h, m, mask, mask_stride, partial, d);                                              \
        break;
    switch (B) {
        POP_DN(1) POP_DN(2) POP_DN(3) POP_DN(4) POP_DN(5) POP_DN(6) POP_DN(7) POP_DN(8)
        default: return hipErrorInvalidValue;
    }
#undef POP_DN
    int total = B * d;
    return launch_down_reduce(partial, n_slabs, total, y, y_bf16, copy, s);
}

int down_num_slabs(int d, int is_bf16)
{
    int nvec = d / (is_bf16 ? 8 : 4);
    int chunks = (nvec + kWave - 1) / kWave;
    int slabs = (512 + chunks - 1) / chunks;  // about 512 workgroups = 2048 waves
    if (slabs < 1) slabs = 1;
    if (slabs > 256) slabs = 256;
    return slabs;
}

hipError_t launch_down(const void *w, int is_bf16, int d, int m, const int *list, const int *n_dev, int n_host,
                       const float *h, const unsigned char *mask, int mask_stride, int B, float *partial, int n_slabs,
                       void *y, int y_bf16, long long stream_from, hipStream_t s, const StepCopy *copy)
{
    if (stream_rows(d, m, is_bf16, stream_from))
        return down_dispatch<StreamBF16>(w, d / 8, d, m, list, n_dev, n_host, h, mask, mask_stride, B, partial, n_slabs,
                                         y, y_bf16, s, copy);
    if (is_bf16)
        return down_dispatch<VecBF16>(w, d / 8, d, m, list, n_dev, n_host, h, mask, mask_stride, B, partial, n_slabs,
                                      y, y_bf16, s, copy);
    return down_dispatch<VecF32>(w, d / 4, d, m, list, n_dev, n_host, h, mask, mask_stride, B, partial, n_slabs, y,
                                 y_bf16, s, copy);
}

// ---------------------------------------------------------------- down projection of up to 32 tokens on the matrix cores
// y[t][:] = sum over listed j of h[t][j] * W_down[:, j], h in float32.  Bound by the weight stream: the vector kernel above
// spends a fused multiply-add per token and weight (eight sequences: 27 us where the rows take 15), and takes eight tokens
// at a time.  Here a float32 h is the exact sum of three bf16 values, so three 16x16x32 products per 16 tokens give what
// float32 multiplies would: products are exact, sums are float32.
// A workgroup owns 128 columns and a slab of the list, its eight waves 32 channels each of every 256.  Lane (c, g) =
// (lane % 16, lane / 16) loads 16 bytes of the rows of channels 8 g .. 8 g + 7 at columns 8 c .. 8 c + 7 (256 contiguous
// bytes per row), which is a transposed operand: one byte permute per register pairs the values of two channels, and
// product e takes column 8 c + e of every lane.  A wave sees to its own channels alone, h included, which passes through a piece of LDS
// of its own: no barrier stands between requests and products, every wait leaves the rows of the wave's next group in flight, and the
// eight waves run apart.  (With h staged by the workgroup, three bf16 planes of 256 channels between two barriers, its loads had to be
// waited for behind the rows in flight, and were made for 16 tokens whether they existed or not: 13B shape, two layers, batch of 4
// 110.5 us a step instead of 104.9, of 8 123.3 instead of 121.8.)
constexpr int kSkThreads = 512;
constexpr int kSkList = 4096;      // channels of a slab whose numbers are in LDS at a time
constexpr int kSkCols = 128;       // columns per workgroup
constexpr int kSkPair = 68;        // floats between two pairs of tokens' h (64, and four banks)
constexpr int kSkChunk = 256;      // channels staged at a time (skinny_staged_kernel)
constexpr int kSkLd = kSkChunk + 8;  // LDS row stride of the staged h planes (16-byte aligned, rows four banks apart)

// f = hi + mid + lo exactly for finite f (24 significant bits in three bf16 values of 8; the rests are exact differences)
__device__ __forceinline__ void split3(float f, uint16_t &hi, uint16_t &mid, uint16_t &lo)
{
    const uint32_t b0 = __float_as_uint(f) & 0xffff0000u;
    const float r1 = f - __uint_as_float(b0);
    const uint32_t b1 = __float_as_uint(r1) & 0xffff0000u;
    const float r2 = r1 - __uint_as_float(b1);
    hi = (uint16_t)(b0 >> 16), mid = (uint16_t)(b1 >> 16), lo = (uint16_t)(__float_as_uint(r2) >> 16);
}

// TQ pairs of tokens, of which T exist; kMask: masks per token (else none)
template <class V, int TQ, bool kMask>
__global__ __launch_bounds__(kSkThreads) void skinny_down_kernel(const uint4 *__restrict__ w, int nvec,
                                                                 const int *__restrict__ list, const int *__restrict__ n_dev,
                                                                 const float *__restrict__ h, int m,
                                                                 const unsigned char *__restrict__ mask, int mask_stride,
                                                                 int T, float *__restrict__ partial, int d)
{
    typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    constexpr int TG = 1;  // group of 16 tokens
    constexpr int kWaves = kSkThreads / kWave;
    static_assert(TQ <= 8 * TG, "pairs of tokens");
    extern __shared__ __attribute__((aligned(16))) unsigned char sk_lds[];
    int *js = reinterpret_cast<int *>(sk_lds);  // [kSkList] channels of the slab
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // this wave's h of 32 channels, [16 TG tokens][32]: pairs of tokens kSkPair floats apart (fragment reads hit all banks)
    float *hw = reinterpret_cast<float *>(sk_lds + kSkList * 4) + wave * (8 * TG * kSkPair);
    const int c = lane % 16, g = lane / 16;
    const int n = *n_dev;
    const int n_slabs = gridDim.y, per_slab = (n + n_slabs - 1) / n_slabs;
    const int s0 = min(n, (int)blockIdx.y * per_slab), s1 = min(n, s0 + per_slab);
    const int vcol = blockIdx.x * (kSkCols / 8) + c;  // this lane's vector column
    const bool col_ok = vcol < nvec;
    const uint32_t chan = channel_vectors(nvec, 1);
    const uint4 *wc = w + 2 * nvec + (col_ok ? vcol : 0);

    f32x4_t acc[TG][8];
#pragma unroll
    for (int t = 0; t < TG; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[t][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    uint4 rows[2][8];
    float hv[TQ];                // of tokens 2 q + lane / 32, channel lane % 32 of the group
    unsigned char hm[kMask ? TQ : 1];
    // group i of this wave: entries 32 (wave + kWaves i) .. + 31 of the list in LDS, of which `have` exist (the rest repeat the last)
    auto entry = [&](int i, int k, int have) { return js[min(32 * (wave + kWaves * i) + k, have - 1)]; };
    auto request_rows = [&](uint4 (&r)[8], int i, int have) {
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = load_row<V>(wc, (uint64_t)(uint32_t)entry(i, 8 * g + q, have) * chan);
    };
    auto request_h = [&](int i, int have) {
        const int j = entry(i, lane % 32, have);
        int half = lane / 32;
        asm volatile("" : "+v"(half));  // (offsets made afresh: kept for all tokens they cost the registers of a group's rows)
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
            const int t = 2 * q + half < T ? 2 * q + half : 0;
            // (atomic in name only: a plain load may move, and moves down to where its value is used)
            hv[q] = __hip_atomic_load(h + (size_t)((uint32_t)t * (uint32_t)m + (uint32_t)j), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            if (kMask)
                hm[q] = __hip_atomic_load(mask + (size_t)((uint32_t)t * (uint32_t)mask_stride + (uint32_t)j), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    };
    // h to LDS; zero beyond the list, beyond T and where a mask says so
    auto place_h = [&](int i, int have) {
        const bool live = 32 * (wave + kWaves * i) + lane % 32 < have;
#pragma unroll
        for (int q = 0; q < TQ; ++q)
            hw[q * kSkPair + lane] = live && 2 * q + lane / 32 < T && (!kMask || hm[kMask ? q : 0]) ? hv[q] : 0.f;
    };
    auto multiply = [&](const uint4 (&r)[8]) {
#pragma unroll
        for (int t = 0; t < TG; ++t) {
            const float4 *at = reinterpret_cast<const float4 *>(hw + (8 * t + c / 2) * kSkPair + c % 2 * 32 + 8 * g);
            const float4 f0 = at[0], f1 = at[1];
            const float f[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
            uint32_t p[3][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint16_t a[3], b[3];
                split3(f[2 * q], a[0], a[1], a[2]);
                split3(f[2 * q + 1], b[0], b[1], b[2]);
#pragma unroll
                for (int k = 0; k < 3; ++k) p[k][q] = (uint32_t)a[k] | (uint32_t)b[k] << 16;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint4 &r0 = r[2 * q], &r1 = r[2 * q + 1];
                    const uint32_t a0 = e / 2 == 0 ? r0.x : (e / 2 == 1 ? r0.y : (e / 2 == 2 ? r0.z : r0.w));
                    const uint32_t a1 = e / 2 == 0 ? r1.x : (e / 2 == 1 ? r1.y : (e / 2 == 2 ? r1.z : r1.w));
                    v[q] = __builtin_amdgcn_perm(a1, a0, e % 2 ? 0x07060302u : 0x05040100u);
                }
                const bf16x8_t bw = __builtin_bit_cast(bf16x8_t, make_uint4(v[0], v[1], v[2], v[3]));
#pragma unroll
                for (int k = 2; k >= 0; --k)  // (small parts first)
                    acc[t][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, make_uint4(p[k][0], p[k][1], p[k][2], p[k][3])), bw, acc[t][e], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int q = TQ; q < 8 * TG; ++q) hw[q * kSkPair + lane] = 0.f;
    for (int l0 = s0; l0 < s1; l0 += kSkList) {
        const int have = min(kSkList, s1 - l0);
        __syncthreads();  // the readers of the list before are done
        for (int i = threadIdx.x; i < have; i += kSkThreads) js[i] = list[l0 + i];
        __syncthreads();
        const int groups = (have + 32 * kWaves - 1) / (32 * kWaves);
        request_rows(rows[0], 0, have);
        request_h(0, have);
        request_rows(rows[1], 1, have);
        auto step = [&](uint4 (&r)[8], int i) {
            place_h(i, have);
            request_h(i + 1, have);
            __builtin_amdgcn_sched_barrier(0);  // (requests where they are written: earlier they cost registers)
            multiply(r);
            __builtin_amdgcn_sched_barrier(0);
            request_rows(r, i + 2, have);
            __builtin_amdgcn_sched_barrier(0);
        };
        int i = 0;
        for (; i + 2 <= groups; i += 2) {
            step(rows[0], i);
            step(rows[1], i + 1);
        }
        if (i < groups) {
            place_h(i, have);
            multiply(rows[0]);
        }
    }
    // the waves' sums in wave order, 16 tokens at a time; register v of product e is token 4 g + v, column 8 c + e
    float *red = reinterpret_cast<float *>(sk_lds);  // [waves][16 tokens][128 columns]
#pragma unroll
    for (int t = 0; t < TG; ++t) {
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float4 *dst = reinterpret_cast<float4 *>(red + ((size_t)(wave * 16 + 4 * g + v)) * kSkCols + 8 * c);
            dst[0] = make_float4(acc[t][0][v], acc[t][1][v], acc[t][2][v], acc[t][3][v]);
            dst[1] = make_float4(acc[t][4][v], acc[t][5][v], acc[t][6][v], acc[t][7][v]);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < 16 * kSkCols; i += kSkThreads) {
            const int tok = 16 * t + i / kSkCols, col = blockIdx.x * kSkCols + i % kSkCols;
            if (tok < T && col < d) {
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < kSkThreads / kWave; ++q) s += (double)red[q * 16 * kSkCols + i];
                float v = (float)s;
                if (!__builtin_isfinite(v)) {
                    // An infinity is not the sum of three parts, and parts that are zero make NaN of an infinite weight:
                    // here the sum is what the vector kernel's multiply-adds give.
                    v = 0.f;
                    for (int p = s0; p < s1; ++p) {
                        const int j = list[p];
                        const float hv = !kMask || mask[(size_t)tok * mask_stride + j] ? h[(size_t)tok * m + j] : 0.f;
                        const uint16_t wv = reinterpret_cast<const uint16_t *>(w)[(size_t)j * channel_elems_bf16(d) + 2 * d + col];
                        v = fmaf(hv, __uint_as_float((uint32_t)wv << 16), v);
                    }
                }
                partial[((size_t)blockIdx.y * T + tok) * d + col] = v;
            }
        }
    }
}

// TG groups of 16 tokens, two of 17 to 32 tokens: the workgroup stages h for all its waves, as three bf16 planes of 256 channels.  (Eight
// waves that each see to their own have no registers for two groups' sums and two steps of rows, and with four the float32 sums are twice
// as long: 24 tokens 62.7 us instead of 63.3 for the whole call, at a fifth more error.)
template <class V, int TG, bool kMask>
__global__ __launch_bounds__(kSkThreads) void skinny_staged_kernel(const uint4 *__restrict__ w, int nvec,
                                                                 const int *__restrict__ list, const int *__restrict__ n_dev,
                                                                 const float *__restrict__ h, int m,
                                                                 const unsigned char *__restrict__ mask, int mask_stride,
                                                                 int T, float *__restrict__ partial, int d)
{
    typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) unsigned char sk_lds[];
    constexpr int kPlanes = 3 * 16 * TG * kSkLd * 2;        // bytes
    uint16_t *hp = reinterpret_cast<uint16_t *>(sk_lds);  // [3][16 TG][kSkLd]: planes of h, rows by token
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int c = lane % 16, g = lane / 16;
    const int n = *n_dev;
    const int n_slabs = gridDim.y, per_slab = (n + n_slabs - 1) / n_slabs;
    const int s0 = min(n, (int)blockIdx.y * per_slab), s1 = min(n, s0 + per_slab);
    const int vcol = blockIdx.x * (kSkCols / 8) + c;  // this lane's vector column
    const bool col_ok = vcol < nvec;
    const uint32_t chan = channel_vectors(nvec, 1);
    const uint4 *wc = w + 2 * nvec + (col_ok ? vcol : 0);

    f32x4_t acc[TG][8];
#pragma unroll
    for (int t = 0; t < TG; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[t][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // channels of two chunks behind the planes: chunk q's in js[q % 2], loaded two chunks ahead
    int *js = reinterpret_cast<int *>(sk_lds + kPlanes);  // [2][kSkChunk]
    const int li = threadIdx.x % kSkChunk, half = threadIdx.x / kSkChunk;
    auto channel = [&](int at) { return list[min(at + li, s1 - 1)]; };  // beyond the slab: its last channel (h is 0 there)
    uint4 rows[2][8];
    auto request = [&](int set) {
#pragma unroll
        for (int i = 0; i < 8; ++i) rows[set][i] = load_row<V>(wc, (uint64_t)(uint32_t)js[set * kSkChunk + 32 * wave + 8 * g + i] * chan);
    };
    // h of the 256 channels at `at` as three planes; zero beyond the slab, beyond T and where a mask says so
    auto stage = [&](int set, int at) {
        const int j = js[set * kSkChunk + li];
        float v[8 * TG];
        unsigned char mk[8 * TG];
#pragma unroll
        for (int q = 0; q < 8 * TG; ++q) {
            const int t = min(2 * q + half, T - 1);
            v[q] = h[(size_t)t * m + j];
            if (kMask) mk[q] = mask[(size_t)t * mask_stride + j];
        }
#pragma unroll
        for (int q = 0; q < 8 * TG; ++q) {
            const int t = 2 * q + half;
            uint16_t a, b, e;
            split3(t < T && at + li < s1 && (!kMask || mk[q]) ? v[q] : 0.f, a, b, e);
            hp[(0 * 16 * TG + t) * kSkLd + li] = a;
            hp[(1 * 16 * TG + t) * kSkLd + li] = b;
            hp[(2 * 16 * TG + t) * kSkLd + li] = e;
        }
    };
    auto multiply = [&](int set) {
        bf16x8_t bw[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            uint32_t v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint4 &r0 = rows[set][2 * q], &r1 = rows[set][2 * q + 1];
                const uint32_t a0 = e / 2 == 0 ? r0.x : (e / 2 == 1 ? r0.y : (e / 2 == 2 ? r0.z : r0.w));
                const uint32_t a1 = e / 2 == 0 ? r1.x : (e / 2 == 1 ? r1.y : (e / 2 == 2 ? r1.z : r1.w));
                v[q] = __builtin_amdgcn_perm(a1, a0, e % 2 ? 0x07060302u : 0x05040100u);
            }
            bw[e] = __builtin_bit_cast(bf16x8_t, make_uint4(v[0], v[1], v[2], v[3]));
        }
#pragma unroll
        for (int t = 0; t < TG; ++t)
#pragma unroll
            for (int part = 2; part >= 0; --part) {  // (small parts first)
                const bf16x8_t ha = *reinterpret_cast<const bf16x8_t *>(
                    &hp[((part * TG + t) * 16 + c) * kSkLd + 32 * wave + 8 * g]);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    acc[t][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ha, bw[e], acc[t][e], 0, 0, 0);
            }
    };
    if (s0 < s1) {
        if (half == 0) js[li] = channel(s0), js[kSkChunk + li] = channel(s0 + kSkChunk);
        __syncthreads();
        request(0);
        auto step = [&](int set, int at) {
            const int next = channel(at + 2 * kSkChunk);
            stage(set, at);
            if (at + kSkChunk < s1) request(set ^ 1);
            __syncthreads();
            if (half == 0) js[set * kSkChunk + li] = next;
            multiply(set);
            __syncthreads();  // the planes' readers are done, the channels are there
        };
        for (int at = s0; at < s1; at += 2 * kSkChunk) {
            step(0, at);
            if (at + kSkChunk < s1) step(1, at + kSkChunk);
        }
    }
    // the eight waves' sums in wave order, 16 tokens at a time; register v of product e is token 4 g + v, column 8 c + e
    float *red = reinterpret_cast<float *>(sk_lds);  // [8 waves][16 tokens][128 columns]
#pragma unroll
    for (int t = 0; t < TG; ++t) {
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float4 *dst = reinterpret_cast<float4 *>(red + ((size_t)(wave * 16 + 4 * g + v)) * kSkCols + 8 * c);
            dst[0] = make_float4(acc[t][0][v], acc[t][1][v], acc[t][2][v], acc[t][3][v]);
            dst[1] = make_float4(acc[t][4][v], acc[t][5][v], acc[t][6][v], acc[t][7][v]);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < 16 * kSkCols; i += kSkThreads) {
            const int tok = 16 * t + i / kSkCols, col = blockIdx.x * kSkCols + i % kSkCols;
            if (tok < T && col < d) {
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < kSkThreads / kWave; ++q) s += (double)red[q * 16 * kSkCols + i];
                float v = (float)s;
                if (!__builtin_isfinite(v)) {
                    // An infinity is not the sum of three parts, and parts that are zero make NaN of an infinite weight:
                    // here the sum is what the vector kernel's multiply-adds give.
                    v = 0.f;
                    for (int p = s0; p < s1; ++p) {
                        const int j = list[p];
                        const float hv = !kMask || mask[(size_t)tok * mask_stride + j] ? h[(size_t)tok * m + j] : 0.f;
                        const uint16_t wv = reinterpret_cast<const uint16_t *>(w)[(size_t)j * channel_elems_bf16(d) + 2 * d + col];
                        v = fmaf(hv, __uint_as_float((uint32_t)wv << 16), v);
                    }
                }
                partial[((size_t)blockIdx.y * T + tok) * d + col] = v;
            }
        }
    }
}

// Slabs of the list so that the column blocks fill the chip once.
int skinny_down_slabs(int is_bf16, int d, int m, int n_cu)
{
    if (!is_bf16) return f32_down_slabs(d, m, n_cu);
    const int cols = (d + kSkCols - 1) / kSkCols;
    const int slabs = n_cu / cols;
    return slabs < 1 ? 1 : (slabs > 64 ? 64 : slabs);
}

template <class V>
static hipError_t launch_skinny_down_partials(const void *w, int d, int m, const int *list, const int *n_dev,
                                              const float *h, const unsigned char *mask, int mask_stride, int T,
                                              float *partial, int n_slabs, hipStream_t s)
{
    if (T < 1 || T > kSkMaxTokens) return hipErrorInvalidValue;
    const dim3 grid((d + kSkCols - 1) / kSkCols, n_slabs);
    hipError_t e = hipSuccess;
    constexpr size_t red = (size_t)8 * 16 * kSkCols * 4;
#define POP_SK(KERNEL, STAGE)                                                                                             \
    do {                                                                                                                  \
        constexpr size_t stage = STAGE, lds = stage > red ? stage : red;                                                  \
        const auto kernel = KERNEL;                                                                                       \
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,       \
                                (int)lds);                                                                                \
        if (e != hipSuccess) return e;                                                                                    \
        hipLaunchKernelGGL(kernel, grid, dim3(kSkThreads), lds, s, (const uint4 *)w, d / 8, list, n_dev, h, m, mask,      \
                           mask_stride, T, partial, d);                                                                   \
    } while (0)
#define POP_SKQ(TQ)                                                                          \
    POP_SK((mask ? skinny_down_kernel<V, TQ, true> : skinny_down_kernel<V, TQ, false>), \
           (size_t)kSkList * 4 + (size_t)8 * 8 * kSkPair * 4)
    // (pairs of tokens are loaded whether they exist or not, h and mask byte of each channel: as many as that as rows.  With the eight
    // pairs of 9 to 16 tokens that is what a wave's own h costs, so there h is staged, except where a slab is a single group of every
    // wave's or masks are loaded over a long list.  Whole FFN of 12 tokens, three layers in turn, waves on their own / staged: one mask, d 2048,
    // m 5504 78.9 / 80.0 us, d 2560, m 6144 93.1 / 92.2, d 3072 102.1 / 100.2, d 4096, m 5504 118.0 / 116.5, m 11008 143.0 / 141.6; own
    // masks, d 2048, m 5504 114.7 / 111.5, d 2560 128.4 / 125.0, d 4096, m 5504 151.9 / 151.6, m 8192 166.8 / 167.4, m 14336 238.7 / 244.5)
    if (T <= 4) POP_SKQ(2);
    else if (T <= 6) POP_SKQ(3);
    else if (T <= 8) POP_SKQ(4);
    else if (T <= 16 && (mask ? m >= 8192 : m <= 384 * n_slabs)) POP_SKQ(8);
    else if (T <= 16)
        POP_SK((mask ? skinny_staged_kernel<V, 1, true> : skinny_staged_kernel<V, 1, false>), (size_t)3 * 16 * kSkLd * 2 + 2 * kSkChunk * 4);
    else
        POP_SK((mask ? skinny_staged_kernel<V, 2, true> : skinny_staged_kernel<V, 2, false>), (size_t)3 * 32 * kSkLd * 2 + 2 * kSkChunk * 4);
#undef POP_SKQ
#undef POP_SK
    return hipGetLastError();
}

hipError_t launch_skinny_down(const void *w, int is_bf16, int d, int m, const int *list, const int *n_dev, const float *h,
                              const unsigned char *mask, int mask_stride, int T, float *partial, int n_slabs, void *y,
                              int y_bf16, long long stream_from, hipStream_t s, const StepCopy *copy)
{
    const bool stream = stream_rows(d, m, is_bf16, stream_from);
    hipError_t e =
        stream    ? launch_skinny_down_partials<StreamBF16>(w, d, m, list, n_dev, h, mask, mask_stride, T, partial, n_slabs, s)
        : is_bf16 ? launch_skinny_down_partials<VecBF16>(w, d, m, list, n_dev, h, mask, mask_stride, T, partial, n_slabs, s)
                  : launch_down_f32_partials(w, d, m, list, n_dev, h, mask, mask_stride, T, partial, n_slabs, s);
    if (e != hipSuccess) return e;
    return launch_down_reduce(partial, n_slabs, T * d, y, y_bf16, copy, s);
}

}  // namespace pop
