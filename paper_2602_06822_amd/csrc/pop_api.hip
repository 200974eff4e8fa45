// C ABI of the POP pruned-FFN library: argument validation, layer state and kernel sequencing.
// Every step of the path runs in the HIP kernels of the sibling files; nothing here computes on the host
// except the integer region counts.
#include <stddef.h>
#include <stdint.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <new>

#include "pop_internal.h"

using namespace pop;

namespace {

thread_local char g_hip_err[256] = "";

int hip_fail(hipError_t e, const char *what)
{
    snprintf(g_hip_err, sizeof g_hip_err, "%s: %s", what, hipGetErrorString(e));
    return POP_EHIP;
}

#define POP_HIP(call)                                      \
    do {                                                   \
        hipError_t e__ = (call);                           \
        if (e__ != hipSuccess) return hip_fail(e__, #call); \
    } while (0)

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// The kernels read activations and weights, and write y, with 16-byte accesses.
inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

#ifdef POP_TRACE
unsigned long long *g_trace = nullptr;  // profiling builds: device buffer the fused kernel stamps into
#endif

}  // namespace

struct pop_layer {
    int d = 0, m = 0, esize = 0, is_bf16 = 0, max_tokens = 0, max_batch = 0;
    void *w = nullptr;     // gate row, up row, down column of each channel, channel_vectors() apart
    float *nrm = nullptr;  // [m]
    int n_cu = 0, wg_target = 0;
    bool shared_mask = false;    // B > 1: one selection for the batch from scores aggregated over its sequences
    bool input_side = false;     // importance from the first projections and the FFN input (pop_layer_set_importance)
    float *in_s2 = nullptr;      // [max_batch][d]: squared input norms (input-side importance)
    double *in_part = nullptr;   // [row groups][d]: their partial sums over a prompt
    // partition
    bool has_partition = false;
    int n_ret = 0, n_cand = 0;
    float *scores = nullptr;           // [m]
    float *s2_part = nullptr;          // [tiles][m]
    int *pf_ctr = nullptr;             // [m] arrival counters of the prefill kernel's channel chunks (zero at rest)
    int tiles_cap = 0;
    unsigned char *region = nullptr;   // [m]
    int *ret_idx = nullptr;            // [m]
    int *cand_idx = nullptr;           // [m]
    int *rc_idx = nullptr;             // [m]: candidates then retained
    // decode step
    bool has_step = false, step_fused = false, ulist_prefix_ok = false;
    int strat_n_ret = -1, strat_n_cand = -1, strat_k = -1;  // decode strategy of the layer (pop_layer_set_strategy)
    int step_B = 0;
    bool fused_ok = false;             // the fused kernel supports this partition
    FusedPlan plan = {};
    int *sync = nullptr;               // [16]: [2] error flag of the batched kernels, [8..9] and [10..12] their counters
    // what the fused kernel's workgroups hand to each other: 64-bit words {value, epoch}
    unsigned long long *hc = nullptr;     // [m] a candidate's h, by candidate position
    unsigned long long *selw = nullptr;   // per-workgroup selection words
    int *fctr = nullptr;                  // [16]: [0] epoch, [1] finished workgroups, [2] sticky error flag
    int spin_limit = 1 << 16;             // looks a bounded in-kernel wait takes before it gives up
    BatchK step_k = {};
    float *h = nullptr;                // [chunk][m]
    float *cscore = nullptr;           // [max_batch][m]
    unsigned char *mask = nullptr;     // [max_batch][m]
    unsigned char *selflag = nullptr;  // [m][POP_MAX_BATCH]: per-sequence selection by candidate position (B > 1)
    int *active_idx = nullptr;         // [max_batch][m]
    int *n_active = nullptr;           // [max_batch]
    int *ulist = nullptr;              // [m]
    int *n_ulist = nullptr;            // [1]
    float *partial = nullptr;          // max([n_slabs][chunk][d], [fused workgroups][d], [skinny slabs][32 or 64][d])
    int n_slabs = 0;
    // whole-prompt pruned FFN on the matrix cores (bf16 layers), allocated at its first use
    uint16_t *ffn_hc = nullptr;        // [tokens][ldh] bf16: H of the active channels, compact
    size_t ffn_hc_cap = 0;             // elements
    uint16_t *ffn_hall = nullptr;      // [m][tokens, in 64s] or [tokens][ldh] bf16: H of all channels, kept by pop_prefill_forward
    size_t ffn_hall_cap = 0;           // elements
    float *ffn_part = nullptr;         // [splits][tokens][d]: partial outputs of the split contraction
    size_t ffn_part_cap = 0;           // elements
    unsigned char *ffn_any = nullptr;  // [m]: the prompt's mask, or channels active in any row of a per-token mask
    int *top_list = nullptr;           // [m] + 1: the prompt's own active channels (ascending), then their number
    // pruned FFN of a few tokens
    int chunk = 0;                     // tokens the decode kernels take at a time
    float *hs = nullptr;               // [precise_max_tokens][m] float32
    uint16_t *zero_row = nullptr;      // kZeroRowBytes of zeros: stands in for rows beyond a channel list
};

namespace {

// Launch shape of the fused single-sequence step for the layer's current region sizes, sized to be co-resident.
int plan_fused_step(pop_layer *L)
{
    L->fused_ok = fused_plan(L->d, L->m, L->is_bf16, L->n_ret, L->n_cand, L->wg_target, &L->plan);
    if (L->fused_ok) {
        int max_wg = 0;
        POP_HIP(fused_resident_limit(L->is_bf16, L->plan, L->n_cu, &max_wg));
        if (max_wg < 2) {
            L->fused_ok = false;
        } else if (L->plan.n_wg > max_wg) {
            L->fused_ok = fused_plan(L->d, L->m, L->is_bf16, L->n_ret, L->n_cand, max_wg, &L->plan) && L->plan.n_wg <= max_wg;
        }
    }
    return POP_OK;
}

// What the caller takes of the step's selection results, from the layer's state (each destination may be null).
StepCopy step_copy(const pop_layer *L, int B, float *cand_scores, unsigned char *mask, int *active_idx, int *n_active)
{
    StepCopy c;
    c.B = B, c.m = L->m, c.n_cand = L->n_cand, c.n_list = L->n_ret + L->n_cand;
    c.cscore = L->cscore, c.mask_src = L->mask, c.act_src = L->active_idx, c.n_act_src = L->n_active;
    c.cand_scores = cand_scores, c.mask = mask, c.active_idx = active_idx, c.n_active = n_active;
    return c;
}

// From this many tokens on a bf16 layer's stand-alone pruned FFN runs on the matrix cores with H rounded to bf16.
constexpr int kFfnMfmaMinTokens = 32;

// A stand-alone FFN of a few tokens: one pass of the decode kernels over a list where T fits one and T x m is below this, else
// the pass whose time hardly grows with T (bf16 / float32 matrix cores).  Whole call, layers in turn, decode / other, shared mask: 7B shape
// (m 11008) 2 tokens 41.5 / 45.2 us, 5 tokens 45.7 / 45.9, 6 tokens 48.3 / 46.4, 8 tokens 50.8 / 46.7; d 2048, m 5632, 6 tokens 24.2 / 25.8, 8 tokens
// 26.3 / 26.0; float32 d 2048, m 5632, 4 tokens 28.9 / 30.6, 8 tokens 32.0 / 31.0.  The line fits these; since waves see to their own channels in
// the other pass it lies too high by up to a half elsewhere (d 2048, m 14336, 3 tokens 37.1 / 36.1, 4 tokens 38.3 / 36.8; 13B shape, 3 tokens
// 63.6 / 62.8, 4 tokens 65.7 / 63.1; d 1024, m 4000, 5 tokens 18.9 / 18.7, 8 tokens 21.3 / 18.7).
constexpr int kFewTokenChannels = 60000;

// Per-token masks of up to this many bytes become a list in one launch; larger ones are combined by the whole chip first, two
// launches more (d 512, m 768, 8 tokens: 20 us against 25; m 11008, 2 tokens: 54.4 / 55.6, 8 tokens: 76 / 58).
constexpr int kMaskListBytes = 24576;

// From this many sequences on a bf16 layer's batched step takes the matrix cores for its down projection: the vector
// kernel's multiply-adds grow with the batch, the matrix-core kernel's time does not.  The line was drawn for a matrix-core kernel whose
// workgroups staged h, which was behind below it (7B shape, 3 sequences 50.0 / 50.7 us; 13B 73.1 / 74.4; d 8192, m 28672, 5 sequences
// 198.7 / 201.8).  Whole step, vector / matrix, weights from memory, with the waves on their own: d 1024, m 2816, 2 sequences 21.1 / 18.3, 3
// 22.5 / 19.0; d 4104, m 5000, 2 36.2 / 33.8; 7B shape at sparsity .35 2 43.6 / 42.3, 3 45.6 / 43.5, 4 47.4 / 44.9, at .5 2 41.0 / 37.9, 3 41.3 / 38.6; 13B
// shape 2 63.8 / 61.7 and 49.9 / 48.8, 3 66.6 / 63.5 and 52.3 / 50.3, 4 69.0 / 65.9 and 55.4 / 52.2, 8 82.6 / 77.9; d 8192, m 28672 2 163.5 / 162.8, 3 167.7 /
// 168.3, 5 180.3 / 181.3, 8 207.7 / 206.5.  So it lies too high by now on all but the largest layers.
int skinny_min_batch(int d, int m)
{
    const long long weights = (long long)d * m;
    return weights > (128ll << 20) ? 6 : (weights > (32ll << 20) ? 4 : 3);
}

// hipMalloc that leaves no pending error behind when it fails (a later launch check would report it as its own).
bool dev_alloc(void **p, size_t bytes)
{
    if (hipMalloc(p, bytes) == hipSuccess) return true;
    (void)hipGetLastError();
    *p = nullptr;
    return false;
}

// Makes *p hold at least `need` elements of esize bytes; the old contents are dropped.  Growing frees first, which
// synchronises the device.
int grow(void **p, size_t *cap, size_t need, size_t esize)
{
    if (need <= *cap) return POP_OK;
    if (*p) POP_HIP(hipFree(*p));
    *p = nullptr, *cap = 0;
    if (!dev_alloc(p, need * esize)) return POP_ENOMEM;
    *cap = need;
    return POP_OK;
}

// Scratch of the prompt-sized forward pass for T tokens: compact H, split partials, the byte mask; with keep_all
// also H of all channels.  (A forward pass with H by channel does not read compact H; a pruned FFN of as many tokens after it, captured
// in a graph perhaps, finds its scratch there.)  Returns the row stride of the H buffers and the number of contraction splits.
int ffn_scratch(pop_layer *L, int T, bool keep_all, int *ldh, int *n_split, hipStream_t s, bool shorter_too = false)
{
    // rows are whole 64-channel k-steps long: the direct-load GEMM reads the columns between a list's end and the end
    // of its last k-step (times rows of zeros, so they only have to be finite; every writer of compact H zeroes them).
    // New buffers are cleared by a kernel on the caller's stream, ahead of the kernels that read them.
    *ldh = (L->m + 63) / 64 * 64;
    *n_split = down_gemm_splits(T, L->d, L->n_cu);
    const size_t hc_before = L->ffn_hc_cap;
    int rc = grow((void **)&L->ffn_hc, &L->ffn_hc_cap, (size_t)T * *ldh, sizeof(uint16_t));
    if (rc == POP_OK && L->ffn_hc_cap != hc_before)
        POP_HIP(launch_fill_int((int *)L->ffn_hc, (int)(L->ffn_hc_cap / 2), 0, s));
    if (rc == POP_OK && !L->zero_row) {
        if (!dev_alloc((void **)&L->zero_row, kZeroRowBytes)) return POP_ENOMEM;
        POP_HIP(launch_fill_int((int *)L->zero_row, kZeroRowBytes / 4, 0, s));
    }
    size_t part_rows = *n_split > 1 ? (size_t)*n_split * T : 0;
    if (shorter_too)  // a shorter prompt is split more ways: room for every prompt length up to T
        for (int t = 1; t < T; ++t) {
            const size_t r = (size_t)down_gemm_splits(t, L->d, L->n_cu) * t;
            if (r > part_rows) part_rows = r;
        }
    if (rc == POP_OK && part_rows)
        rc = grow((void **)&L->ffn_part, &L->ffn_part_cap, part_rows * L->d, sizeof(float));
    // (by token or by channel)
    if (rc == POP_OK && keep_all)
        rc = grow((void **)&L->ffn_hall, &L->ffn_hall_cap, (size_t)((T + 63) / 64 * 64) * *ldh + kRowsSlack, sizeof(uint16_t));
    return rc;
}

// Whole-prompt pruned FFN (Sec. 3.4: forward pass under the pruning structure): active list from the mask(s),
// gate/up over the listed channels with H written in compact bf16 form, then the K-gathered down-projection GEMM.
int pruned_ffn_mfma(pop_layer *L, const void *x, int T, const unsigned char *mask, int mask_rows, void *y, int y_bf16,
                    hipStream_t s)
{
    const int m = L->m, d = L->d;
    int ldh, n_split;
    { int rc = ffn_scratch(L, T, false, &ldh, &n_split, s); if (rc != POP_OK) return rc; }
    const unsigned char *tmask = nullptr;
    if (mask_rows == 1) {
        POP_HIP(launch_mask_to_list(mask, 1, m, L->ulist, L->n_ulist, s, L->ffn_hc, ldh, T));
    } else {
        POP_HIP(launch_mask_any(mask, T, m, L->ffn_any, s));
        POP_HIP(launch_mask_to_list(L->ffn_any, 1, m, L->ulist, L->n_ulist, s, L->ffn_hc, ldh, T));
        tmask = mask;
    }
    POP_HIP(launch_gateup_list_bf16(L->w, d, m, x, T, L->ulist, L->n_ulist, tmask, L->ffn_hc, ldh, L->n_cu,
                                   kStreamFfnBytes, s));
    POP_HIP(launch_down_gemm_bf16(L->w, d, L->ulist, L->n_ulist, L->ffn_hc, ldh, T, n_split, L->n_cu, L->ffn_part, y, y_bf16, s,
                                  L->zero_row));
    return POP_OK;
}

// Pruned FFN of x under the given masks.
int pruned_ffn(pop_layer *L, const void *x, int T, const unsigned char *mask, int mask_rows, void *y, int y_bf16, hipStream_t s)
{
    const int m = L->m, d = L->d, ysize = y_bf16 ? 2 : 4;
    L->has_step = false;  // the step scratch is reused below
    L->ulist_prefix_ok = false;
    if (L->is_bf16 && T >= kFfnMfmaMinTokens) return pruned_ffn_mfma(L, x, T, mask, mask_rows, y, y_bf16, s);
    const int few = precise_max_tokens(L->is_bf16, d);
    if (few > 0 && T > 1 && (T > L->chunk || (long long)T * m >= kFewTokenChannels)) {
        // a few tokens (bf16 layers: all of them) per pass over the weights
        if (mask_rows > 1 && (long long)mask_rows * m > kMaskListBytes) {
            POP_HIP(launch_mask_any(mask, T, m, L->ffn_any, s));
            POP_HIP(launch_mask_to_list(L->ffn_any, 1, m, L->ulist, L->n_ulist, s));
        } else {
            POP_HIP(launch_mask_to_list(mask, mask_rows, m, L->ulist, L->n_ulist, s));
        }
        for (int t0 = 0; t0 < T; t0 += few) {
            const int n = T - t0 < few ? T - t0 : few;
            POP_HIP(launch_precise_gateup(L->w, L->is_bf16, d, m, (const char *)x + (size_t)t0 * d * L->esize, n, L->ulist,
                                          L->n_ulist, L->hs, nullptr, nullptr, L->n_cu, kStreamFfnBytes, s));
            POP_HIP(launch_skinny_down(L->w, L->is_bf16, d, m, L->ulist, L->n_ulist, L->hs,
                                       mask_rows > 1 ? mask + (size_t)t0 * m : nullptr, m, n, L->partial,
                                       skinny_down_slabs(L->is_bf16, d, m, L->n_cu),
                                       (char *)y + (size_t)t0 * d * ysize, y_bf16, kStreamFfnBytes, s));
        }
        return POP_OK;
    }
    if (mask_rows == 1) POP_HIP(launch_mask_to_list(mask, 1, m, L->ulist, L->n_ulist, s));
    const long long stream_from = T > L->chunk ? kStreamAgainBytes : kStreamFfnBytes;  // (every pass reads the same rows)
    for (int t0 = 0; t0 < T; t0 += L->chunk) {
        const int Bc = (T - t0 < L->chunk) ? T - t0 : L->chunk;
        const unsigned char *mk = mask_rows == 1 ? nullptr : mask + (size_t)t0 * m;
        if (mk) POP_HIP(launch_mask_to_list(mk, Bc, m, L->ulist, L->n_ulist, s));
        const char *xc = (const char *)x + (size_t)t0 * d * L->esize;
        POP_HIP(launch_gateup(L->w, L->is_bf16, d, m, xc, Bc, L->ulist, m, L->n_ulist, L->h, nullptr, nullptr, 0, 0,
                              L->n_cu, stream_from, s));
        POP_HIP(launch_down(L->w, L->is_bf16, d, m, L->ulist, L->n_ulist, 0, L->h, mk, m, Bc, L->partial, L->n_slabs,
                            (char *)y + (size_t)t0 * d * ysize, y_bf16, stream_from, s));
    }
    return POP_OK;
}

// Scores, partition and partition-constant step state from s2_part (the second half of the prefilling stage).
// n_top: size of the prompt's own mask; `o` says what the caller wants of it.
int finish_partition(pop_layer *L, int T, int n_ret, int n_cand, float *scores, unsigned char *region, int *ret_idx,
                     int *cand_idx, hipStream_t s, bool scores_ready, int n_top = 0,
                     PartitionOutputs o = PartitionOutputs{})
{
    const int m = L->m;
    if (!scores_ready)
        POP_HIP(launch_scores_from_partials(L->s2_part, prefill_rows_used(T, L->d, m, L->n_cu), m, L->nrm,
                                            L->scores, s));
    o.scores = L->scores, o.scores_copy = scores;
    o.region[0] = L->region, o.region[1] = region;
    o.ret_idx[0] = L->ret_idx, o.ret_idx[1] = ret_idx;
    o.cand_idx[0] = L->cand_idx, o.cand_idx[1] = cand_idx;
    o.rows = L->max_batch, o.act_stride = m, o.mask = L->mask, o.active_idx = L->active_idx;
    o.rc_idx = L->rc_idx, o.ulist = L->ulist;
    o.sync = L->sync, o.n_sync = 16;
    POP_HIP(launch_partition(L->scores, m, n_ret, n_cand, n_top, o, s));
    L->ulist_prefix_ok = true;
    L->n_ret = n_ret;
    L->n_cand = n_cand;
    { int rc = plan_fused_step(L); if (rc != POP_OK) return rc; }
    L->has_partition = true;
    return POP_OK;
}

// Arguments of the fused single-sequence kernel for the layer's current partition.
FusedParams fused_params(pop_layer *L, const void *x_t, int k)
{
    FusedParams p = {};
    p.w = L->w;
    p.x = x_t;
    p.nvec = L->d / (L->is_bf16 ? 8 : 4);
    p.d = L->d;
    p.m = L->m;
    p.ret_idx = L->ret_idx;
    p.n_ret = L->n_ret;
    p.cand_idx = L->cand_idx;
    p.n_cand = L->n_cand;
    p.k = k;
    p.nrm = L->nrm;
    p.h = L->h;
    p.cscore = L->cscore;
    p.mask = L->mask;
    p.active_idx = L->active_idx;
    p.n_active = L->n_active;
    p.hc = L->hc;
    p.selw = L->selw;
    p.partial = L->partial;
    p.ctr = L->fctr;
    p.spin_limit = L->spin_limit;
    p.input_side = L->input_side ? 1 : 0;
#ifdef POP_TRACE
    p.trace = g_trace;
#endif
    return p;
}

}  // namespace

extern "C" {

int pop_version(void) { return 100; }

const char *pop_strerror(int status)
{
    switch (status) {
        case POP_OK: return "ok";
        case POP_EINVAL: return "invalid argument";
        case POP_ESHAPE: return "inconsistent sizes";
        case POP_ENOMEM: return "out of device memory";
        case POP_EHIP: return "HIP call failed";
        case POP_ESTATE: return "call order violated";
        case POP_EUNSUPPORTED: return "unsupported configuration";
        case POP_EDEVICE: return "a kernel gave up a bounded wait";
        default: return "unknown status";
    }
}

const char *pop_last_hip_error(void) { return g_hip_err; }

int pop_region_counts(int m, double f_ret, double f_cand, int *n_ret, int *n_cand, int *n_prn)
{
    if (!n_ret || !n_cand || !n_prn) return POP_EINVAL;
    if (m <= 0 || !(f_ret >= 0.0) || !(f_cand >= 0.0) || !(f_ret + f_cand <= 1.0 + 1e-12)) return POP_EINVAL;
    long long a = (long long)floor(f_ret * (double)m + 0.5);
    long long b = (long long)floor((f_ret + f_cand) * (double)m + 0.5);
    if (a > m) a = m;
    if (b > m) b = m;
    if (b < a) b = a;
    *n_ret = (int)a;
    *n_cand = (int)(b - a);
    *n_prn = (int)(m - b);
    return POP_OK;
}

int pop_k_for_ratio(int m, double r, int n_ret, int n_cand, int *k)
{
    if (!k) return POP_EINVAL;
    if (m <= 0 || !(r >= 0.0) || !(r <= 1.0) || n_ret < 0 || n_cand < 0 || n_ret + n_cand > m) return POP_EINVAL;
    long long a = (long long)floor((1.0 - r) * (double)m + 0.5);
    long long kk = a - n_ret;
    if (kk < 0) kk = 0;
    if (kk > n_cand) kk = n_cand;
    *k = (int)kk;
    return POP_OK;
}

int pop_strategy_counts(int strategy, int m, double r, double gamma, int *n_ret, int *n_cand, int *k)
{
    if (!n_ret || !n_cand || !k) return POP_EINVAL;
    if (m <= 0 || !(r >= 0.0) || !(r <= 1.0) || !(gamma >= 0.0) || !(gamma <= 1.0)) return POP_EINVAL;
    const int a = (int)floor((1.0 - r) * (double)m + 0.5);  // active channels per token
    switch (strategy) {
    case POP_STRATEGY_STATIC_MASK:
        *n_ret = a, *n_cand = 0, *k = 0;
        return POP_OK;
    case POP_STRATEGY_RESCORE_ALL:
        *n_ret = 0, *n_cand = m, *k = a;
        return POP_OK;
    case POP_STRATEGY_POP: {
        if (1.0 - r - gamma / 2 < 0.0 || 1.0 - r + gamma / 2 > 1.0) return POP_EINVAL;
        int n_prn = 0;
        int rc = pop_region_counts(m, 1.0 - r - gamma / 2, gamma, n_ret, n_cand, &n_prn);
        if (rc != POP_OK) return rc;
        return pop_k_for_ratio(m, r, *n_ret, *n_cand, k);
    }
    default:
        return POP_EINVAL;
    }
}

int pop_layer_destroy(pop_layer_t *L)
{
    if (!L) return POP_EINVAL;
    void *ptrs[] = {L->w,      L->nrm, L->scores, L->s2_part, L->region,     L->ret_idx,  L->cand_idx, L->rc_idx,
                    L->h,      L->cscore, L->mask, L->selflag, L->active_idx, L->n_active, L->ulist, L->n_ulist,  L->partial,
                    L->sync,   L->hc, L->selw, L->fctr, L->pf_ctr, L->ffn_hc, L->ffn_part, L->ffn_any, L->ffn_hall, L->in_s2, L->in_part, L->top_list, L->zero_row, L->hs};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    delete L;
    return POP_OK;
}

int pop_layer_create(pop_layer_t **out, int d, int m, pop_dtype_t wdtype, const void *w_gate, const void *w_up,
                     const void *w_down, int max_tokens, int max_batch, void *stream)
{
    if (!out) return POP_EINVAL;
    *out = nullptr;
    if (!w_gate || !w_up || !w_down) return POP_EINVAL;
    if (!aligned16(w_gate) || !aligned16(w_up) || !aligned16(w_down)) return POP_EINVAL;
    if (wdtype != POP_F32 && wdtype != POP_BF16) return POP_EINVAL;
    if (d <= 0 || m <= 0 || max_tokens < 1) return POP_ESHAPE;
    if (max_batch < 1 || max_batch > POP_MAX_BATCH) return POP_ESHAPE;
    const int is_bf16 = wdtype == POP_BF16, esize = is_bf16 ? 2 : 4;
    if ((d * esize) % 16 != 0) return POP_EUNSUPPORTED;
    if ((long long)m * 3 * d >= (1LL << 34)) return POP_EUNSUPPORTED;  // 16-byte vectors of w are indexed with 32 bits

    int dev = 0, lds_max = 0, n_cu = 0;
    POP_HIP(hipGetDevice(&dev));
    POP_HIP(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    POP_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    if ((long long)max_batch * d * esize > lds_max) return POP_EUNSUPPORTED;  // x_t is staged in LDS

    pop_layer *L = new (std::nothrow) pop_layer;
    if (!L) return POP_ENOMEM;
    L->d = d;
    L->m = m;
    L->esize = esize;
    L->is_bf16 = is_bf16;
    L->max_tokens = max_tokens;
    L->max_batch = max_batch;
    L->tiles_cap = prefill_num_tiles(max_tokens, is_bf16);
    L->n_slabs = down_num_slabs(d, is_bf16);
    L->n_cu = n_cu;
    L->wg_target = n_cu;  // one workgroup per compute unit; POP_FUSED_WGS overrides (tuning)
    if (const char *e = getenv("POP_FUSED_WGS")) {
        int v = atoi(e);
        if (v >= 2 && v <= fused_max_workgroups()) L->wg_target = v;
    }
    if (L->wg_target > fused_max_workgroups()) L->wg_target = fused_max_workgroups();
    if (const char *e = getenv("POP_WAIT_LIMIT")) L->spin_limit = atoi(e) < 0 ? 0 : atoi(e);  // (tuning, tests)

    // tokens of a stand-alone FFN that the decode kernels take at a time: as many as they can, whatever the batch
    L->chunk = max_batch;
    while (L->chunk < POP_MAX_BATCH && (long long)(L->chunk + 1) * d * esize <= lds_max) ++L->chunk;
    const int few_tokens = precise_max_tokens(is_bf16, d);

    const size_t mm = (size_t)m, B = (size_t)max_batch, C = (size_t)L->chunk;
    size_t partial_rows = (size_t)L->n_slabs * C;
    if (partial_rows < (size_t)fused_max_workgroups()) partial_rows = (size_t)fused_max_workgroups();
    const size_t skinny_rows = (size_t)skinny_down_slabs(is_bf16, d, m, n_cu) * (is_bf16 ? kSkMaxTokens : kF32MaxTokens);
    if (partial_rows < skinny_rows) partial_rows = skinny_rows;
    struct Req { void **p; size_t bytes; };
    Req reqs[] = {
        {&L->w, mm * channel_vectors(d * esize / 16, is_bf16) * 16},
        {(void **)&L->nrm, mm * 4},
        {(void **)&L->scores, mm * 4},
        {(void **)&L->s2_part, (size_t)L->tiles_cap * mm * 4},
        {(void **)&L->region, mm},
        {(void **)&L->ret_idx, mm * 4},
        {(void **)&L->cand_idx, mm * 4},
        {(void **)&L->rc_idx, mm * 4},
        {(void **)&L->h, C * mm * 4},
        {(void **)&L->cscore, B * mm * 4},
        {(void **)&L->mask, B * mm},
        {(void **)&L->selflag, (size_t)POP_MAX_BATCH * mm},
        {(void **)&L->active_idx, B * mm * 4},
        {(void **)&L->n_active, B * 4},
        {(void **)&L->ulist, mm * 4},
        {(void **)&L->n_ulist, 4},
        {(void **)&L->partial, partial_rows * d * 4},
        {(void **)&L->sync, 64},
        {(void **)&L->hc, mm * 8},
        {(void **)&L->selw, fused_selw_words() * 8},
        {(void **)&L->fctr, 64},
        {(void **)&L->pf_ctr, mm * 4},
        {(void **)&L->ffn_any, (mm + 3) / 4 * 4},
        {(void **)&L->top_list, (mm + 1) * 4},
        {(void **)&L->hs, (size_t)few_tokens * mm * 4},
    };
    for (const Req &r : reqs) {
        if (r.bytes == 0) continue;
        hipError_t e = hipMalloc(r.p, r.bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            pop_layer_destroy(L);
            return e == hipErrorOutOfMemory ? POP_ENOMEM : hip_fail(e, "hipMalloc");
        }
    }
    hipStream_t s = as_stream(stream);
    hipError_t e = launch_repack(w_gate, w_up, w_down, d, m, esize, L->w, L->nrm, is_bf16, s);
    if (e == hipSuccess) e = launch_fill_int(L->sync, 16, 0, s);
    // the words the fused kernel's workgroups exchange start out with epoch 0, the counter at 1: nothing stale can
    // ever look valid
    if (e == hipSuccess) e = hipMemsetAsync(L->hc, 0, mm * 8, s);
    if (e == hipSuccess) e = hipMemsetAsync(L->selw, 0, fused_selw_words() * 8, s);
    if (e == hipSuccess) e = launch_fill_int(L->fctr, 16, 0, s);
    if (e == hipSuccess) e = launch_fill_int(L->pf_ctr, m, 0, s);
    if (e == hipSuccess) e = launch_fill_int(L->fctr, 1, 1, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        pop_layer_destroy(L);
        return hip_fail(e, "layer repack");
    }
    *out = L;
    return POP_OK;
}

int pop_prefill_partition(pop_layer_t *L, const void *x, int T, int n_ret, int n_cand, float *scores,
                          unsigned char *region, int *ret_idx, int *cand_idx, void *stream)
{
    if (!L) return POP_EINVAL;
    if (T < 0 || T > L->max_tokens) return POP_ESHAPE;
    if (T > 0 && (!x || !aligned16(x))) return POP_EINVAL;
    if (n_ret == POP_FROM_STRATEGY && n_cand == POP_FROM_STRATEGY) {
        if (L->strat_n_ret < 0) return POP_ESTATE;
        n_ret = L->strat_n_ret, n_cand = L->strat_n_cand;
    }
    if (n_ret < 0 || n_cand < 0 || (long long)n_ret + n_cand > L->m) return POP_ESHAPE;
    hipStream_t s = as_stream(stream);
    const int m = L->m;
    const bool few = !L->input_side && T <= precise_max_tokens(L->is_bf16, L->d);
    L->has_partition = false;
    L->has_step = false;
    if (T == 0) {
        // no tokens: every importance is zero under either reading, and the order falls back on the channel index
        POP_HIP(launch_fill_int((int *)L->scores, m, 0, s));
    } else if (L->input_side) {
        POP_HIP(launch_input_norms(x, L->is_bf16, T, L->d, L->in_part, L->in_s2, s));
        POP_HIP(launch_input_side_scores(L->w, L->is_bf16, L->d, L->in_s2, 1, nullptr, m, L->scores, m, kStreamPartBytes, s));
    } else {
        const PrefillScores fin{L->pf_ctr, L->nrm, L->scores};
        if (few)  // (the same launch as pop_prefill_forward's: the same scores, bit for bit)
            POP_HIP(launch_precise_gateup(L->w, L->is_bf16, L->d, m, x, T, nullptr, nullptr, L->hs, L->s2_part, &fin, L->n_cu, kStreamPromptBytes,
                                          s));
        else
            POP_HIP(launch_prefill_gateup(L->w, L->is_bf16, L->d, m, x, T, L->s2_part, L->n_cu, s, &fin));
    }
    return finish_partition(L, T, n_ret, n_cand, scores, region, ret_idx, cand_idx, s,
                            T == 0 || L->input_side || few || prefill_forms_scores(L->is_bf16, T, L->d, m, L->n_cu));
}

int pop_prefill_forward(pop_layer_t *L, const void *x, int T, int n_ret, int n_cand, int k0, void *y, pop_dtype_t ydtype,
                        float *scores, unsigned char *region, int *ret_idx, int *cand_idx, unsigned char *mask,
                        void *stream)
{
    if (!L) return POP_EINVAL;
    if (T < 0 || T > L->max_tokens) return POP_ESHAPE;
    if (T > 0 && (!x || !y || !aligned16(x) || !aligned16(y))) return POP_EINVAL;
    if (ydtype != POP_F32 && ydtype != POP_BF16) return POP_EINVAL;
    if (n_ret == POP_FROM_STRATEGY && n_cand == POP_FROM_STRATEGY) {
        if (L->strat_n_ret < 0) return POP_ESTATE;
        n_ret = L->strat_n_ret, n_cand = L->strat_n_cand;
        if (k0 == POP_FROM_STRATEGY) k0 = L->strat_k;
    }
    if (n_ret < 0 || n_cand < 0 || (long long)n_ret + n_cand > L->m) return POP_ESHAPE;
    if (k0 < 0 || k0 > n_cand) return POP_ESHAPE;
    hipStream_t s = as_stream(stream);
    const int m = L->m, d = L->d;
    // H of the importance contraction is kept and the output runs on the matrix cores (the input-side importance
    // has no such contraction: partition first, then the masked FFN)
    const bool keep = L->is_bf16 && T >= kFfnMfmaMinTokens && !L->input_side;
    // a short prompt: H of all channels in float32 from the same pass that scores them
    const bool few = !L->input_side && T > 0 && T <= precise_max_tokens(L->is_bf16, d);
    L->has_partition = false;
    L->has_step = false;
    int ldh = 0, n_split = 1;
    const bool by_channel = down_gemm_by_channel(d);
    const int ldt = (T + 63) / 64 * 64;
    if (keep) {
        int rc = ffn_scratch(L, T, true, &ldh, &n_split, s);
        if (rc != POP_OK) return rc;
        const PrefillScores fin{L->pf_ctr, L->nrm, L->scores};
        POP_HIP(launch_prefill_gateup_keep_bf16(L->w, d, m, x, T, L->s2_part, L->ffn_hall, by_channel ? ldt : ldh, by_channel, L->n_cu,
                                                s, &fin));
    } else {
        if (T == 0) {
            POP_HIP(launch_fill_int((int *)L->scores, m, 0, s));  // no tokens: all importances zero
        } else if (L->input_side) {
            POP_HIP(launch_input_norms(x, L->is_bf16, T, d, L->in_part, L->in_s2, s));
            POP_HIP(launch_input_side_scores(L->w, L->is_bf16, d, L->in_s2, 1, nullptr, m, L->scores, m, kStreamTwiceBytes, s));
        } else if (few) {
            const PrefillScores fin{L->pf_ctr, L->nrm, L->scores};
            POP_HIP(launch_precise_gateup(L->w, L->is_bf16, d, m, x, T, nullptr, nullptr, L->hs, L->s2_part, &fin, L->n_cu, kStreamPromptBytes,
                                          s));
        } else {
            const PrefillScores fin{L->pf_ctr, L->nrm, L->scores};
            POP_HIP(launch_prefill_gateup(L->w, L->is_bf16, d, m, x, T, L->s2_part, L->n_cu, s, &fin));
        }
    }
    // prefill mask: retained channels plus the best k0 candidates by prefill score, i.e. the n_ret + k0 best channels
    // of the partition's own order: the partition launch emits them as well (mask bytes and ascending list)
    // (the byte mask only where somebody reads it: the caller, or the path below that works from a mask)
    PartitionOutputs o;
    o.top_list = L->top_list, o.top_count = L->top_list + m;
    o.top_mask[0] = keep || few ? nullptr : L->ffn_any, o.top_mask[1] = mask;
    {
        int rc = finish_partition(L, T, n_ret, n_cand, scores, region, ret_idx, cand_idx, s,
                                  T == 0 || L->input_side || few || prefill_forms_scores(L->is_bf16, T, L->d, m, L->n_cu),
                                  n_ret + k0, o);
        if (rc != POP_OK) return rc;
    }
    if (T == 0) return POP_OK;  // no token rows to produce
    if (keep && by_channel) {
        POP_HIP(launch_down_gemm_rows(L->w, d, m, L->top_list, n_ret + k0, L->ffn_hall, ldt, T, n_split, L->n_cu, L->ffn_part, y,
                                      ydtype == POP_BF16, s, L->zero_row));
        return POP_OK;
    }
    if (keep) {
        POP_HIP(launch_compact_hidden(L->ffn_hall, ldh, T, L->top_list, L->top_list + m, n_ret + k0, L->ffn_hc, ldh, s));
        POP_HIP(launch_down_gemm_bf16(L->w, d, L->top_list, L->top_list + m, L->ffn_hc, ldh, T, n_split, L->n_cu, L->ffn_part, y,
                                      ydtype == POP_BF16, s, L->zero_row));
        return POP_OK;
    }
    if (few) {
        POP_HIP(launch_skinny_down(L->w, L->is_bf16, d, m, L->top_list, L->top_list + m, L->hs, nullptr, 0, T, L->partial,
                                   skinny_down_slabs(L->is_bf16, d, m, L->n_cu), y, ydtype == POP_BF16, kStreamPromptBytes, s));
        return POP_OK;
    }
    return pruned_ffn(L, x, T, L->ffn_any, 1, y, ydtype == POP_BF16, s);
}

// Pass 1 and the selection of a decode step; the results stay in the layer's state.
static int decode_select(pop_layer_t *L, const void *x_t, int B, const int *k, void *stream)
{
    if (!L || !x_t || !aligned16(x_t)) return POP_EINVAL;
    if (!L->has_partition) return POP_ESTATE;
    if (!k && L->strat_k < 0) return POP_EINVAL;  // no per-sequence counts and no strategy to take them from
    if (B < 1 || B > L->max_batch) return POP_ESHAPE;
    BatchK kk = {};
    for (int b = 0; b < B; ++b) {
        const int kb = k ? k[b] : L->strat_k;
        if (kb < 0 || kb > L->n_cand) return POP_ESHAPE;
        kk.k[b] = kb;
    }
    hipStream_t s = as_stream(stream);
    const int m = L->m, n_ret = L->n_ret, n_cand = L->n_cand;
    L->has_step = false;
    if (B == 1 && L->fused_ok) {
        FusedParams p = fused_params(L, x_t, kk.k[0]);
        POP_HIP(launch_decode_fused(L->plan, L->is_bf16, p, s));
        L->step_fused = true;
    } else {
        if (B > 1) {
            if (!L->ulist_prefix_ok && n_ret)
                POP_HIP(hipMemcpyAsync(L->ulist, L->ret_idx, (size_t)n_ret * 4, hipMemcpyDeviceToDevice, s));
            L->ulist_prefix_ok = true;
        }
        if (L->input_side) {
            // (a single sequence on a shape the fused kernel takes went there: it scores the candidates from the same
            // rows it reads for h.)  Here candidates are scored from their gate and up rows and |x_t| alone, so the
            // selection comes first and the forward pass runs over retained and selected channels only
            const bool shared = B > 1 && L->shared_mask;
            if (shared)
                for (int b = 1; b < B; ++b)
                    if (kk.k[b] != kk.k[0]) return POP_ESHAPE;
            POP_HIP(launch_input_squares(x_t, L->is_bf16, B, L->d, L->in_s2, s));
            POP_HIP(launch_input_side_scores(L->w, L->is_bf16, L->d, L->in_s2, B, L->cand_idx, n_cand, L->cscore, m, kStreamStepBytes,
                                             s));
            // one mask for the batch: the root of the sum of the sequences' squared scores is this reading's importance
            // over the step's B rows (Eq. 1-2 with s_k over tokens and samples); every row gets it
            if (shared) POP_HIP(launch_aggregate_scores(L->cscore, m, B, n_cand, s));
            POP_HIP(launch_topk(L->cscore, m, L->cand_idx, n_cand, n_ret, m, B, kk, m, L->mask, L->active_idx,
                                L->n_active, nullptr, B > 1 ? L->selflag : nullptr, L->sync + 8, B > 1 ? L->ulist : nullptr, L->n_ulist,
                                s));
            if (B == 1)
                POP_HIP(launch_gateup(L->w, L->is_bf16, L->d, m, x_t, 1, L->active_idx, n_ret + kk.k[0], nullptr, L->h,
                                      nullptr, nullptr, 0, 0, L->n_cu, kStreamStepBytes, s));
            else
                POP_HIP(launch_gateup(L->w, L->is_bf16, L->d, m, x_t, B, L->ulist, m, L->n_ulist, L->h, nullptr, nullptr,
                                      0, 0, L->n_cu, kStreamStepBytes, s));
            L->step_fused = false;
            L->step_B = B;
            L->step_k = kk;
            L->has_step = true;
            return POP_OK;
        }
        bool sel_inside = false;
        const bool shared = B > 1 && L->shared_mask;
        if (shared)
            for (int b = 1; b < B; ++b)
                if (kk.k[b] != kk.k[0]) return POP_ESHAPE;
        if (B > 1 && !shared)  // per-sequence top-k and their union inside the gate/up kernel, behind the retained channels
            POP_HIP(launch_gateup_select(L->w, L->is_bf16, L->d, m, x_t, B, L->rc_idx, L->h, L->nrm, L->cscore, m,
                                         L->cand_idx, n_cand, n_ret, kk, m, L->mask, L->active_idx, L->n_active,
                                         L->selflag, L->ulist, L->n_ulist, L->sync + 10, L->sync + 2, L->spin_limit,
                                         L->n_cu, &sel_inside, s));
        if (!sel_inside) {
            POP_HIP(launch_gateup(L->w, L->is_bf16, L->d, m, x_t, B, L->rc_idx, n_ret + n_cand, nullptr, L->h, L->nrm,
                                  L->cscore, m, n_cand, L->n_cu, kStreamStepBytes, s));
            // one mask for the batch: every sequence's row gets the scores aggregated over the batch, so the B
            // selections below come out identical
            if (shared) POP_HIP(launch_aggregate_scores(L->cscore, m, B, n_cand, s));
            // B > 1: the kernel also builds the union of the B selections for the batched down projection
            POP_HIP(launch_topk(L->cscore, m, L->cand_idx, n_cand, n_ret, m, B, kk, m, L->mask, L->active_idx,
                                L->n_active, nullptr, B > 1 ? L->selflag : nullptr, L->sync + 8, B > 1 ? L->ulist : nullptr, L->n_ulist,
                                s));
        }
        L->step_fused = false;
    }
    L->step_B = B;
    L->step_k = kk;
    L->has_step = true;
    return POP_OK;
}

// The output of the decode step in the layer's state; `copy` rides along with its last launch.
static int decode_output(pop_layer_t *L, int T, void *y, pop_dtype_t ydtype, const StepCopy *copy, hipStream_t s)
{
    const int m = L->m, d = L->d, y_bf16 = ydtype == POP_BF16;
    if (!L->has_step) return POP_ESTATE;
    if (T != L->step_B) return POP_ESHAPE;
    if (L->step_fused)
        POP_HIP(launch_decode_tail(L->partial, L->plan.n_wg, d, y, y_bf16, s, copy));
    else if (T == 1)
        POP_HIP(launch_down(L->w, L->is_bf16, d, m, L->active_idx, nullptr, L->n_ret + L->step_k.k[0], L->h, nullptr, 0, 1,
                            L->partial, L->n_slabs, y, y_bf16, kStreamStepBytes, s, copy));
    else if (L->is_bf16 && T >= skinny_min_batch(d, m))
        POP_HIP(launch_skinny_down(L->w, L->is_bf16, d, m, L->ulist, L->n_ulist, L->h, L->mask, m, T, L->partial,
                                   skinny_down_slabs(L->is_bf16, d, m, L->n_cu), y, y_bf16, kStreamStepBytes, s, copy));
    else
        POP_HIP(launch_down(L->w, L->is_bf16, d, m, L->ulist, L->n_ulist, 0, L->h, L->mask, m, T, L->partial, L->n_slabs, y,
                            y_bf16, kStreamStepBytes, s, copy));
    return POP_OK;
}

int pop_decode_mask(pop_layer_t *L, const void *x_t, int B, const int *k, float *cand_scores, unsigned char *mask,
                    int *active_idx, int *n_active, void *stream)
{
    const int rc = decode_select(L, x_t, B, k, stream);
    if (rc != POP_OK) return rc;
    POP_HIP(launch_step_copy(step_copy(L, B, cand_scores, mask, active_idx, n_active), as_stream(stream)));
    return POP_OK;
}

int pop_decode_step(pop_layer_t *L, const void *x_t, int B, const int *k, void *y, pop_dtype_t ydtype,
                    float *cand_scores, unsigned char *mask, int *active_idx, int *n_active, void *stream)
{
    if (!L || !x_t || !y || !aligned16(x_t) || !aligned16(y)) return POP_EINVAL;
    if (ydtype != POP_F32 && ydtype != POP_BF16) return POP_EINVAL;
    if (!L->has_partition) return POP_ESTATE;
    if (!k && L->strat_k < 0) return POP_EINVAL;
    if (B < 1 || B > L->max_batch) return POP_ESHAPE;
    for (int b = 0; b < B; ++b) {
        const int kb = k ? k[b] : L->strat_k;
        if (kb < 0 || kb > L->n_cand) return POP_ESHAPE;
    }
    // the launches of the two calls (a single-sequence step on a shape the fused kernel takes: that kernel, then the
    // small kernel that sums its workgroups' partial outputs), the last of which also copies what the caller takes
    const int rc = decode_select(L, x_t, B, k, stream);
    if (rc != POP_OK) return rc;
    const StepCopy copy = step_copy(L, B, cand_scores, mask, active_idx, n_active);
    return decode_output(L, B, y, ydtype, &copy, as_stream(stream));
}

int pop_pruned_ffn(pop_layer_t *L, const void *x, int T, const unsigned char *mask, int mask_rows, void *y,
                   pop_dtype_t ydtype, void *stream)
{
    if (!L || !y || !aligned16(y)) return POP_EINVAL;
    if (ydtype != POP_F32 && ydtype != POP_BF16) return POP_EINVAL;
    hipStream_t s = as_stream(stream);
    const int y_bf16 = ydtype == POP_BF16;
    if (!mask) return decode_output(L, T, y, ydtype, nullptr, s);
    if (!x || !aligned16(x)) return POP_EINVAL;
    if (T < 1) return POP_ESHAPE;
    if (mask_rows != 1 && mask_rows != T) return POP_ESHAPE;
    return pruned_ffn(L, x, T, mask, mask_rows, y, y_bf16, s);
}

int pop_partition_from_scores(const float *scores, int m, int n_ret, int n_cand, unsigned char *region, int *ret_idx,
                              int *cand_idx, void *stream)
{
    if (!scores) return POP_EINVAL;
    if (m <= 0 || n_ret < 0 || n_cand < 0 || (long long)n_ret + n_cand > m) return POP_ESHAPE;
    PartitionOutputs o;
    o.region[0] = region, o.ret_idx[0] = ret_idx, o.cand_idx[0] = cand_idx;
    POP_HIP(launch_partition(scores, m, n_ret, n_cand, 0, o, as_stream(stream)));
    return POP_OK;
}

int pop_partition_top_from_scores(const float *scores, int m, int n_ret, int n_cand, int n_top, unsigned char *region,
                                  int *ret_idx, int *cand_idx, unsigned char *top_mask, int *top_list, void *stream)
{
    if (!scores || !top_list) return POP_EINVAL;
    if (m <= 0 || n_ret < 0 || n_cand < 0 || (long long)n_ret + n_cand > m) return POP_ESHAPE;
    if (n_top < 0 || n_top > m) return POP_ESHAPE;
    PartitionOutputs o;
    o.region[0] = region, o.ret_idx[0] = ret_idx, o.cand_idx[0] = cand_idx;
    o.top_mask[0] = top_mask, o.top_list = top_list;
    POP_HIP(launch_partition(scores, m, n_ret, n_cand, n_top, o, as_stream(stream)));
    return POP_OK;
}

int pop_topk_from_scores(const float *cand_scores, const int *cand_idx, int n_cand, int k, const unsigned char *region,
                         int m, unsigned char *mask, int *sel_idx, void *stream)
{
    if (m <= 0 || n_cand < 0 || n_cand > m || k < 0 || k > n_cand) return POP_ESHAPE;
    if (n_cand > 0 && (!cand_scores || !cand_idx)) return POP_EINVAL;
    if (mask && !region) return POP_EINVAL;
    BatchK kk = {};
    kk.k[0] = k;
    if (mask) POP_HIP(launch_retained_mask(region, m, mask, as_stream(stream)));
    POP_HIP(launch_topk(cand_scores, n_cand, cand_idx, n_cand, 0, m, 1, kk, 0, mask, nullptr, nullptr, sel_idx,
                        nullptr, nullptr, nullptr, nullptr, as_stream(stream)));
    return POP_OK;
}

int pop_importance_reduce(const void *h, pop_dtype_t hdtype, int T, int m, const float *nrm, float *scores,
                          void *stream)
{
    if (!h || !nrm || !scores) return POP_EINVAL;
    if (hdtype != POP_F32 && hdtype != POP_BF16) return POP_EINVAL;
    if (T < 1 || m < 1) return POP_ESHAPE;
    hipStream_t s = as_stream(stream);
    const size_t bytes = importance_reduce_scratch_bytes(h, hdtype == POP_BF16, T, m);
    if (bytes == 0) {
        POP_HIP(launch_importance_reduce(h, hdtype == POP_BF16, T, m, nrm, scores, nullptr, s));
        return POP_OK;
    }
    // long prompts of few channels: the per-chunk partial sums live in stream-ordered scratch
    void *scratch = nullptr;
    hipError_t e = hipMallocAsync(&scratch, bytes, s);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e == hipErrorOutOfMemory ? POP_ENOMEM : hip_fail(e, "hipMallocAsync");
    }
    e = launch_importance_reduce(h, hdtype == POP_BF16, T, m, nrm, scores, scratch, s);
    const hipError_t ef = hipFreeAsync(scratch, s);
    if (e != hipSuccess) return hip_fail(e, "importance reduction");
    if (ef != hipSuccess) return hip_fail(ef, "hipFreeAsync");
    return POP_OK;
}

int pop_layer_reserve_prompt(pop_layer_t *L, int T, void *stream)
{
    if (!L) return POP_EINVAL;
    if (T < 1 || T > L->max_tokens) return POP_ESHAPE;
    if (!L->is_bf16 || T < kFfnMfmaMinTokens) return POP_OK;  // those forward passes use the layer's fixed scratch
    int ldh = 0, n_split = 1;
    { int rc = ffn_scratch(L, T, true, &ldh, &n_split, as_stream(stream), true); if (rc != POP_OK) return rc; }
    return POP_OK;
}

int pop_probe_read(const void *buf, size_t bytes, int workgroups, unsigned int *sink, void *stream)
{
    if (!buf || !sink || !aligned16(buf)) return POP_EINVAL;
    if (bytes < 16 || workgroups < 1 || workgroups > 65535) return POP_ESHAPE;
    POP_HIP(launch_probe_read(buf, bytes, workgroups, sink, as_stream(stream)));
    return POP_OK;
}

int pop_probe_step_read(pop_layer_t *L, int k, int workgroups, unsigned int *sink, void *stream)
{
    if (!L || !sink) return POP_EINVAL;
    if (!L->has_partition) return POP_ESTATE;
    if (k < 0 || k > L->n_cand || workgroups < 1 || workgroups > 65535) return POP_ESHAPE;
    if (L->n_ret + L->n_cand == 0) return POP_OK;
    POP_HIP(launch_probe_step_read(L->w, L->d / (L->is_bf16 ? 8 : 4), channel_vectors(L->d / (L->is_bf16 ? 8 : 4), L->is_bf16), L->rc_idx, L->n_ret + L->n_cand, L->ret_idx,
                                   L->n_ret, L->cand_idx, k, workgroups, sink, stream_rows(L->d, L->m, L->is_bf16, kStreamStepBytes), as_stream(stream)));
    return POP_OK;
}

int pop_layer_get_norms(pop_layer_t *L, float *nrm, void *stream)
{
    if (!L) return POP_EINVAL;
    if (nrm) POP_HIP(hipMemcpyAsync(nrm, L->nrm, (size_t)L->m * 4, hipMemcpyDeviceToDevice, as_stream(stream)));
    return POP_OK;
}

#ifdef POP_TRACE
void pop_trace_set_buffer(void *dev_ptr)
{
    g_trace = (unsigned long long *)dev_ptr;
    set_select_trace(g_trace ? g_trace + 1010 * 8 : nullptr);
}
#endif

int pop_layer_sync_status(pop_layer_t *L, void *stream)
{
    if (!L) return POP_EINVAL;
    int flag = 0, flag_fused = 0;
    POP_HIP(hipMemcpyAsync(&flag, L->sync + 2, 4, hipMemcpyDeviceToHost, as_stream(stream)));
    POP_HIP(hipMemcpyAsync(&flag_fused, L->fctr + 2, 4, hipMemcpyDeviceToHost, as_stream(stream)));
    POP_HIP(hipStreamSynchronize(as_stream(stream)));
    if (flag) POP_HIP(launch_fill_int(L->sync + 2, 1, 0, as_stream(stream)));  // reported once
    if (flag_fused) POP_HIP(launch_fill_int(L->fctr + 2, 1, 0, as_stream(stream)));
    return (flag || flag_fused) ? POP_EDEVICE : POP_OK;
}

int pop_layer_set_importance(pop_layer_t *L, int reading)
{
    if (!L) return POP_EINVAL;
    if (reading != POP_IMPORTANCE_OUTPUT_SIDE && reading != POP_IMPORTANCE_INPUT_SIDE) return POP_EINVAL;
    if (reading == POP_IMPORTANCE_INPUT_SIDE) {
        const size_t groups = (size_t)input_side_groups(L->max_tokens);
        if (!L->in_s2 && !dev_alloc((void **)&L->in_s2, (size_t)L->max_batch * L->d * sizeof(float)))
            return POP_ENOMEM;
        if (!L->in_part && !dev_alloc((void **)&L->in_part, groups * L->d * sizeof(double)))
            return POP_ENOMEM;
    }
    L->input_side = reading == POP_IMPORTANCE_INPUT_SIDE;
    L->has_partition = false;
    L->has_step = false;
    return POP_OK;
}

int pop_layer_set_shared_batch_mask(pop_layer_t *L, int on)
{
    if (!L) return POP_EINVAL;
    L->shared_mask = on != 0;
    L->has_step = false;
    return POP_OK;
}

int pop_layer_set_strategy(pop_layer_t *L, int strategy, double r, double gamma)
{
    if (!L) return POP_EINVAL;
    int n_ret = 0, n_cand = 0, k = 0;
    const int rc = pop_strategy_counts(strategy, L->m, r, gamma, &n_ret, &n_cand, &k);
    if (rc != POP_OK) return rc;
    L->strat_n_ret = n_ret, L->strat_n_cand = n_cand, L->strat_k = k;
    return POP_OK;
}

int pop_layer_set_wait_limit(pop_layer_t *L, int looks)
{
    if (!L || looks < 0) return POP_EINVAL;
    L->spin_limit = looks;
    return POP_OK;
}

int pop_layer_step_kind(pop_layer_t *L, int *workgroups)
{
    if (!L) return POP_EINVAL;
    if (workgroups) *workgroups = (L->has_partition && L->fused_ok) ? L->plan.n_wg : 0;
    return !L->has_step ? 0 : (L->step_fused ? 1 : 2);
}

int pop_layer_get_hidden(pop_layer_t *L, float *h, int B, void *stream)
{
    if (!L) return POP_EINVAL;
    if (B < 1 || B > L->max_batch) return POP_ESHAPE;
    if (h) POP_HIP(hipMemcpyAsync(h, L->h, (size_t)B * L->m * 4, hipMemcpyDeviceToDevice, as_stream(stream)));
    return POP_OK;
}

}  // extern "C"
