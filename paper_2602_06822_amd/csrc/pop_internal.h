// Internal declarations shared by the HIP translation units of the POP library.
// Each .hip file defines its kernels and a host launcher; pop_api.hip holds the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "pop.h"

namespace pop {

constexpr int kWave = 64;

// Order-preserving key of a float32 score: larger score <=> larger key; -0.0 maps to the key of +0.0.
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t b = __float_as_uint(s);
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }

// round-to-nearest-even float32 -> bf16 bits (finite inputs)
__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + expf(-g)) * u; }

// 16-byte vectors between the weights of one channel [gate row | up row | down column] (nvec vectors each) and the next
// channel's.  A 128-byte line on bf16 layers whose rows are 8 or 16 KB: the contraction of a prompt, whose workgroups all
// ask for the same columns of their rows at about the same time, otherwise keeps hitting the same few memory channels.  Prompt
// calls with weights from memory, without / with it: d 4096, m 14336, 256 tokens 82.0 / 80.1 us (the contraction alone, before its
// third step of token rows, 95 / 72), m 11008, 512 tokens 90.2 / 86.8, eight experts 1142 / 1098; d 8192, m 14336, 256 tokens
// 154.6 / 140.4, 512 tokens 232.5 / 225.5.  Two or three lines gain the same or less.  Not on other rows: 2, 4, 6 and 10 KB (d 1024 to
// 5120) are within 1 % with and without, 12 KB (d 6144, m 16384) 128-138 / 126 at 256 tokens and 193-200 / 190 at 512.  Not on 24 and
// 32 KB either (d 16384, m 16384, 256 tokens 324 / 291): there the single-sequence step's kernel keeps 190 registers in scratch
// memory, and its build with the gap takes 1 to 3 % longer than the one without.  None behind each row: the decode step reads
// a channel's rows together and was 0.7 % slower with gaps between them.
__host__ __device__ __forceinline__ constexpr int channel_gap(int nvec, int is_bf16)
{
    return is_bf16 && (nvec == 512 || nvec == 1024) ? 8 : 0;
}
// Weight rows that a launch reads once are loaded past the caches (non-temporal) on layers too large for the next pass to find
// them there.  A plain read of rows from memory: 5.7-6.0 TB/s with ordinary loads, 6.4 with these; but what they read does not stay in
// the 256 MB last-level cache, so where it would have been there for the next pass they lose.  A call cannot know what runs before
// the next one on its layer: the rule is the size of the layer's weights (3 d m, bf16), drawn where no call was slower
// with several layers in turn and half of their channels active.  Time of a call past the caches over its time with ordinary loads:
//   decode steps, six layers: of 50 MB 1.02-1.11 (half of the channels active; .65 of them 1.02-1.08), of 68 MB 1.01-1.07 (.97-.98), of 79 MB
//   .98-1.01, of 86 MB .98-1.00 (.93-.97), of 113 MB .94-.97, of 270 MB .90-.93; twelve layers: of 50 MB .96-.98, of 86 MB .92-.94
//   a prompt's own forward pass (all of gate and up), three layers, 4 to 60 tokens: of 94 MB 1.00-1.08, of 113 MB .98-1.00, of 138 MB
//   .96-.98, of 270 MB .92-.94
//   a prompt's partition (gate and up alone), three layers, 40 tokens: of 138 MB 1.07, of 157 MB .92
//   a stand-alone FFN (what is active of the layer), three layers, 1 to 40 tokens: of 157 MB 1.01-1.04 (.65 active .96-1.00), of 201 MB 1.00-1.02
//   (.93-.98), of 226 MB .96-1.02, of 251 MB .93-1.00, of 270 MB .92-.98 (.90-.97); three tenths active, of 270 MB still 1.04
// A layer run by itself, all of what a step reads in that cache, is slower: 7B shape 33.4 / 34.2 us, eight sequences 46.4 / 49.7, 13B shape, two 60.0 / 63.2.
// Rows that the same call asks for again stay in the cache, as long as it holds them: gate and up rows that scores of the
// input-side reading come from and the prompt's forward pass reads after them (three layers, 40 tokens: of 138 MB 1.05, of 201 MB 1.02-1.07, of
// 270 MB .98-.99), and the rows of an FFN that takes its tokens in several passes (24 tokens: of 74 MB 1.08, of 197 MB 1.03-1.04, of 271 MB
// 1.02-1.04).
constexpr long long kStreamStepBytes = 80ll << 20, kStreamPromptBytes = 128ll << 20, kStreamPartBytes = 144ll << 20;
constexpr long long kStreamFfnBytes = 240ll << 20, kStreamTwiceBytes = 240ll << 20, kStreamAgainBytes = 384ll << 20;
inline bool stream_rows(int d, int m, int is_bf16, long long limit) { return is_bf16 && 6ll * d * m >= limit; }

// From one channel's weights to the next's.
__host__ __device__ __forceinline__ constexpr int channel_vectors(int nvec, int is_bf16)
{
    return 3 * nvec + channel_gap(nvec, is_bf16);
}
// The same in elements of a bf16 layer.
__host__ __device__ __forceinline__ int channel_elems_bf16(int d) { return channel_vectors(d / 8, 1) * 8; }

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

struct BatchK {
    int k[POP_MAX_BATCH];
};

// Device-coherent (agent scope) accesses for values that workgroups of one kernel hand to each other: the
// loads bypass stale cache lines, the stores write through, so no cache write-back or invalidation is needed.
__device__ __forceinline__ int coherent_load(const int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void coherent_store(int *p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void coherent_store(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void coherent_store(unsigned char *p, unsigned char v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float coherent_load(const float *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long coherent_load(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Bounded wait until the counter *addr, which only ever grows (and may wrap), has reached target: at most `limit`
// looks, at least one (a launch that waits is sized so that all its workgroups are resident).
__device__ __forceinline__ bool spin_until(const int *addr, int target, int limit)
{
    for (int it = 0;; ++it) {
        if (coherent_load(addr) - target >= 0) return true;
        if (it >= limit) return false;
        __builtin_amdgcn_s_sleep(2);
    }
}

// ---- setup (pop_setup.hip) ----
// w[j][0][:] = w_gate[j][:], w[j][1][:] = w_up[j][:], w[j][2][o] = w_down[o][j];  nrm[j] = ||w_down[:,j]||.
hipError_t launch_repack(const void *w_gate, const void *w_up, const void *w_down, int d, int m, int esize,
                         void *w, float *nrm, int is_bf16, hipStream_t s);

// ---- selection (pop_select.hip) ----
// What the partition of scores[m] writes; every pointer may be null.  Two destinations where a layer keeps its own copy.
struct PartitionOutputs {
    const float *scores = nullptr;  // read for scores_copy
    float *scores_copy = nullptr;
    unsigned char *region[2] = {nullptr, nullptr};
    int *ret_idx[2] = {nullptr, nullptr}, *cand_idx[2] = {nullptr, nullptr};
    // the n_top best channels of the same order (the prompt's own mask, Sec. 3.4: the retained channels plus the best
    // candidates by prefill score are the n_top best overall): bytes, ascending list, its length
    unsigned char *top_mask[2] = {nullptr, nullptr};
    int *top_list = nullptr, *top_count = nullptr;
    // partition-constant step state: mask[b][j] = (region[j] == retained), active_idx[b][0..n_ret) = ret_idx for b < rows,
    // rc_idx = cand_idx ++ ret_idx, ulist[0..n_ret) = ret_idx
    int rows = 0, act_stride = 0;
    unsigned char *mask = nullptr;
    int *active_idx = nullptr, *rc_idx = nullptr, *ulist = nullptr;
    int *sync = nullptr;  // n_sync <= 1024 counters to clear
    int n_sync = 0;
};
void set_select_trace(unsigned long long *p);  // profiling builds: phase stamps of topk_kernel (8 words), or null
// Regions by rank of scores[m]: the best n_ret channels, the next n_cand, the rest; and the n_top best.
hipError_t launch_partition(const float *scores, int m, int n_ret, int n_cand, int n_top, const PartitionOutputs &o,
                            hipStream_t s);
// hc[t][c] = h_all[t][list[c]] for c < *n_list <= max_list, t < T (bf16 bits), and zero columns up to the next multiple
// of 64.  ldhc even.
hipError_t launch_compact_hidden(const uint16_t *h_all, int ldh, int T, const int *list, const int *n_list, int max_list,
                                 uint16_t *hc, int ldhc, hipStream_t s);
// Per sequence b (grid = B): select k.k[b] of n_cand candidates by cscore[b*cs_stride + i]; writes the candidate
// bytes of mask[b][m], active_idx[b*act_stride + n_ret .. n_ret+k), n_active[b], sel_idx (sequence 0, only when
// active_idx is null), each if non-null.  With union_list non-null also: selflag [B][n_cand] (scratch), and the
// union of the B selections: union_list[n_ret..] = candidates selected by any b (ascending), *n_union = n_ret +
// their number; the prefix union_list[0..n_ret) = ret_idx is written by the caller once per partition.  union_ctr
// is a zeroed counter that the kernel leaves at zero.
hipError_t launch_topk(const float *cscore, int cs_stride, const int *cand_idx, int n_cand, int n_ret, int m, int B,
                       BatchK k, int act_stride, unsigned char *mask, int *active_idx, int *n_active, int *sel_idx,
                       unsigned char *selflag, int *union_ctr, int *union_list, int *n_union, hipStream_t s);
// mask[j] = (region[j] == retained)
hipError_t launch_retained_mask(const unsigned char *region, int m, unsigned char *mask, hipStream_t s);
// mask rows -> ascending list of channels active in any row.  With pad_hc given ([pad_T][pad_ld] bf16, pad_ld a
// multiple of 64) the launch also zeroes its columns from the list's length up to the next multiple of 64 (what the
// direct-load GEMM reads beyond a compact H's last column).
hipError_t launch_mask_to_list(const unsigned char *mask, int rows, int m, int *list, int *n_list, hipStream_t s,
                               uint16_t *pad_hc = nullptr, int pad_ld = 0, int pad_T = 0);

// What the caller of a decode step takes of its selection, copied from the layer's state by extra workgroups of the step's
// last launch (or of a launch of its own): every destination may be null.
struct StepCopy {
    int B = 0, m = 0, n_cand = 0, n_list = 0;  // rows of the layer's arrays are m apart; n_list = n_ret + n_cand
    const float *cscore = nullptr;
    const unsigned char *mask_src = nullptr;   // (16-byte aligned)
    const int *act_src = nullptr, *n_act_src = nullptr;
    float *cand_scores = nullptr;              // [B][n_cand]
    unsigned char *mask = nullptr;             // [B][m]
    int *active_idx = nullptr, *n_active = nullptr;  // [B][n_list], [B]
    bool any() const { return (cand_scores && n_cand) || mask || (active_idx && n_list) || n_active; }
    // workgroups of `threads` threads that copy it, a few elements per thread
    int blocks(int threads) const
    {
        if (!any()) return 0;
        const long n = (cand_scores ? (long)B * n_cand : 0) + (mask ? (long)B * m / 16 : 0) + (active_idx ? (long)B * n_list : 0);
        const long b = (n + 4L * threads - 1) / (4L * threads);
        return b < 1 ? 1 : (b > 64 ? 64 : (int)b);
    }
};
// workgroup `block` of n_blocks
__device__ __forceinline__ void copy_step_block(const StepCopy &c, int block, int n_blocks)
{
    const int at = block * blockDim.x + threadIdx.x, step = n_blocks * blockDim.x;
    if (c.cand_scores)
        for (int i = at; i < c.B * c.n_cand; i += step)
            c.cand_scores[i] = c.cscore[(size_t)(i / c.n_cand) * c.m + i % c.n_cand];
    if (c.active_idx)
        for (int i = at; i < c.B * c.n_list; i += step)
            c.active_idx[i] = c.act_src[(size_t)(i / c.n_list) * c.m + i % c.n_list];
    if (c.n_active && block == 0 && (int)threadIdx.x < c.B) c.n_active[threadIdx.x] = c.n_act_src[threadIdx.x];
    if (c.mask) {
        const int n = c.B * c.m, n16 = (reinterpret_cast<uintptr_t>(c.mask) & 15u) == 0 ? n / 16 : 0;
        for (int i = at; i < n16; i += step)
            reinterpret_cast<uint4 *>(c.mask)[i] = reinterpret_cast<const uint4 *>(c.mask_src)[i];
        for (int i = n16 * 16 + at; i < n; i += step) c.mask[i] = c.mask_src[i];
    }
}
hipError_t launch_step_copy(const StepCopy &c, hipStream_t s);

// ---- decode GEMVs (pop_gemv.hip) ----
// h[b][j] = silu(x_b . gate_j) * (x_b . up_j) for j in rows[0..n_rows); if cscore != null, rows [0, n_score)
// also get cscore[b][pos] = nrm[j] * |h|.  n_rows_dev (optional) overrides n_rows with a device-side count.
// stream_from, here and below: the size of layer from which rows go past the caches (stream_rows).
hipError_t launch_gateup(const void *w, int is_bf16, int d, int m, const void *x, int B, const int *rows, int n_rows,
                         const int *n_rows_dev, float *h, const float *nrm, float *cscore, int cs_stride, int n_score,
                         int n_cu, long long stream_from, hipStream_t s);
// y[b][:] = sum_{i<n} hm(b, list[i]) * w[list[i]][2][:], hm = h[b][j] (masked by mask[b][j] when mask != null).
// Two stages: slab partials then a fixed-order reduction; y written as float32 or bf16.
hipError_t launch_down(const void *w, int is_bf16, int d, int m, const int *list, const int *n_dev, int n_host,
                       const float *h, const unsigned char *mask, int mask_stride, int B, float *partial, int n_slabs,
                       void *y, int y_bf16, long long stream_from, hipStream_t s, const StepCopy *copy = nullptr);
int down_num_slabs(int d, int is_bf16);
// The same for up to kSkMaxTokens (bf16 layers) or kF32MaxTokens rows of h ([T][m] float32, by channel) on the matrix cores; masks one row per token
// (mask_stride) or null.  partial: [n_slabs][T][d] float32.
constexpr int kSkMaxTokens = 32;  // (bf16)
int skinny_down_slabs(int is_bf16, int d, int m, int n_cu);
hipError_t launch_skinny_down(const void *w, int is_bf16, int d, int m, const int *list, const int *n_dev, const float *h,
                              const unsigned char *mask, int mask_stride, int T, float *partial, int n_slabs, void *y,
                              int y_bf16, long long stream_from, hipStream_t s, const StepCopy *copy = nullptr);
// Batched decode (2 <= B <= POP_MAX_BATCH) with the per-sequence selection inside the gate/up kernel: the listed
// rows are the n_cand candidates followed by the n_ret retained channels; all workgroups evaluate the candidates
// first, then the last B workgroups wait (bounded) for everybody's candidate scores and select for one sequence
// each while the others evaluate the retained channels.  Outputs as launch_gateup + launch_topk with a union
// request.  counters: [0] arrivals, [1] selectors done (both zero between launches); err_flag is set if a wait
// expired.  *fused = false (and nothing launched) when the shape does not allow it: use the two launches.
hipError_t launch_gateup_select(const void *w, int is_bf16, int d, int m, const void *x, int B, const int *rows,
                                float *h, const float *nrm, float *cscore, int cs_stride, const int *cand_idx,
                                int n_cand, int n_ret, BatchK k, int act_stride, unsigned char *mask, int *active_idx,
                                int *n_active, unsigned char *selflag, int *union_list, int *n_union, int *counters,
                                int *err_flag, int spin_limit, int n_cu, bool *fused, hipStream_t s);

// ---- fused single-sequence decode step (pop_decode_fused.hip) ----
struct FusedParams {
    const void *w;
    const void *x;
    int nvec, d, m;
    const int *ret_idx;
    int n_ret;
    const int *cand_idx;
    int n_cand, k;
    const float *nrm;
    float *h;                   // [m]
    float *cscore;              // [n_cand]
    unsigned char *mask;        // [m]
    int *active_idx;            // [>= n_ret + k]
    int *n_active;              // [1]
    // what the workgroups hand to each other: 64-bit words {value, epoch}
    unsigned long long *hc;     // [n_cand] a candidate's h (input-side reading: its step score), by candidate position
    unsigned long long *selw;   // [n_wg] per-workgroup selection word (selected candidate slots), 128 bytes apart
    float *partial;             // [n_wg][d] partial output rows (summed by decode_tail_kernel)
    int *ctr;                   // [0] epoch (>= 1), [1] workgroups that finished (back at zero when the kernel ends),
                                // [2] sticky error flag: a bounded wait gave up
    int spin_limit;             // looks a bounded wait takes before it gives up
    int input_side;             // candidates are ranked by || [gate_j, up_j] * |x_t| ||_2 instead of n_j |h_j|
    int n_static;               // retained rounds per worker
    unsigned long long *trace;  // profiling builds only: 8 timestamps per workgroup, else null
};

struct FusedPlan {
    int n_wg, block, per;
    int n_static;  // retained rounds per worker
    bool gap;      // the layer's channels are channel_gap() apart
    bool stream;   // weight rows past the caches (stream_rows)
};
int fused_max_workgroups();
size_t fused_selw_words();  // 64-bit words of the selection-word buffer (one per workgroup, spaced apart)
// Launch shape for (d, dtype, region sizes); false when the fused kernel does not support the shape.
bool fused_plan(int d, int m, int is_bf16, int n_ret, int n_cand, int wg_target, FusedPlan *pl);
// Largest grid of this shape that is co-resident on n_cu compute units.
hipError_t fused_resident_limit(int is_bf16, const FusedPlan &pl, int n_cu, int *max_wg);
hipError_t launch_decode_fused(const FusedPlan &pl, int is_bf16, FusedParams &p, hipStream_t s);
hipError_t launch_decode_tail(const float *partial, int n_wg, int d, void *y, int y_bf16, hipStream_t s,
                              const StepCopy *copy = nullptr);
hipError_t launch_fill_int(int *p, int n, int value, hipStream_t s);

// ---- measurement aids (pop_probe.hip): bare reads, nothing of the method ----
hipError_t launch_probe_read(const void *buf, size_t bytes, int workgroups, unsigned int *sink, hipStream_t s);
hipError_t launch_probe_step_read(const void *w, int nvec, int chan, const int *gu_list, int n_gu, const int *dn_ret,
                                  int n_dn_ret, const int *dn_sel, int n_dn_sel, int workgroups, unsigned int *sink,
                                  bool stream, hipStream_t s);

// ---- prefill (pop_prefill.hip) ----
// s2_part[tile][j] = sum over the tile's tokens of H[t][j]^2, one row per token tile.
int prefill_num_tiles(int T, int is_bf16);  // upper bound on the rows used, for sizing s2_part
int prefill_rows_used(int T, int d, int m, int n_cu);  // rows the launch below writes for this T (bf16)
// With `fin`, launches for which prefill_forms_scores holds (float32 layers; bf16 ones with one tile per compute unit at most) also leave scores[j] = nrm[j] * sqrt(sum over the token tiles, in tile
// order and in double, of s2_part[tile][j]) (Eq. 3): the token tile of a channel chunk that finishes last does the sum.
// chunk_ctr: one int per channel chunk (m of them suffice), zero before the launch and zero again after it.
struct PrefillScores {
    int *chunk_ctr;
    const float *nrm;
    float *scores;
};
bool prefill_forms_scores(int is_bf16, int T, int d, int m, int n_cu);
hipError_t launch_prefill_gateup(const void *w, int is_bf16, int d, int m, const void *x, int T, float *s2_part,
                                 int n_cu, hipStream_t s, const PrefillScores *fin = nullptr);
// bf16 layers: gate/up over the channels of a device-resident list (n_list: its length, on the device);
// hc[t][c] = bf16(H[t][list[c]]), times tmask[t][list[c]] if tmask ([T][m]) is given.  ldh % 8 == 0.
hipError_t launch_gateup_list_bf16(const void *w, int d, int m, const void *x, int T, const int *list, const int *n_list,
                                   const unsigned char *tmask, uint16_t *hc, int ldh, int n_cu, long long stream_from, hipStream_t s);
// y[t][n] = sum_c hc[t][c] * w[list[c]][2][n] on the matrix cores; part (float32 [n_split][T][d]) is needed when
// n_split = down_gemm_splits(...) > 1.  With zero_row (256 bytes of zeros), d % 128 == 0 and ldh % 64 == 0 the
// operands go straight into LDS; that form reads hc columns up to the list length rounded up to 64, which must hold
// finite values.
int down_gemm_splits(int T, int d, int n_cu);
hipError_t launch_down_gemm_bf16(const void *w, int d, const int *list, const int *n_list, const uint16_t *hc, int ldh,
                                 int T, int n_split, int n_cu, float *part, void *y, int y_bf16, hipStream_t s,
                                 const uint16_t *zero_row = nullptr);
// The same with H of all m channels by channel, ht[j][ldt] (ldt a multiple of 64, kRowsSlack elements readable behind the last row):
// rows are read by the list, nothing is gathered.  down_gemm_by_channel: widths it takes.  zero_row: kZeroRowBytes of zeros.
constexpr int kRowsSlack = 512, kZeroRowBytes = 1024;
bool down_gemm_by_channel(int d);
hipError_t launch_down_gemm_rows(const void *w, int d, int m, const int *list, int n_list, const uint16_t *ht, int ldt,
                                 int T, int n_split, int n_cu, float *part, void *y, int y_bf16, hipStream_t s,
                                 const uint16_t *zero_row);
// bf16 layers: the prefill contraction (s2_part as in launch_prefill_gateup) that also keeps H:
// h_all[t][j] = bf16(H[t][j]), row stride ldh, or by channel (d a multiple of 64): h_all[j][t], ldh >= T a multiple of 64.
hipError_t launch_prefill_gateup_keep_bf16(const void *w, int d, int m, const void *x, int T, float *s2_part,
                                           uint16_t *h_all, int ldh, bool by_channel, int n_cu, hipStream_t s,
                                           const PrefillScores *fin = nullptr);
// Gate/up of up to precise_max_tokens tokens (0: not for such layers) with sums in double and h[t][j] in float32 ([T][m],
// by channel).  Without a list: all channels, and their scores as fin says (chunk_ctr zero before and after).  With one
// (n_list: its length, on the device): the listed channels, no scores.
constexpr int kF32MaxTokens = 64;
int precise_max_tokens(int is_bf16, int d);
hipError_t launch_precise_gateup(const void *w, int is_bf16, int d, int m, const void *x, int T, const int *list,
                                 const int *n_list, float *h, float *s2_part, const PrefillScores *fin, int n_cu,
                                 long long stream_from, hipStream_t s);
// float32 layers, T <= kF32MaxTokens: the slab partials of the down projection (summed by launch_skinny_down)
int f32_down_slabs(int d, int m, int n_cu);
hipError_t launch_down_f32_partials(const void *w, int d, int m, const int *list, const int *n_dev, const float *h,
                                    const unsigned char *mask, int mask_stride, int T, float *partial, int n_slabs,
                                    hipStream_t s);
// ---- input-side importance (pop_input_side.hip) ----
int input_side_groups(int T);  // row groups of a T-token prompt (sizes part below: [groups][d] doubles)
// s2[k] = sum_t x[t][k]^2 over the T rows (fixed summation order)
hipError_t launch_input_norms(const void *x, int is_bf16, int T, int d, double *part, float *s2, hipStream_t s);
// s2[b][k] = x[b][k]^2
hipError_t launch_input_squares(const void *x, int is_bf16, int B, int d, float *s2, hipStream_t s);
// out[q][p] = sqrt(sum_k (w_gate[j][k]^2 + w_up[j][k]^2) s2[q][k]), j = rows ? rows[p] : p, q < S, p < n_rows
hipError_t launch_input_side_scores(const void *w, int is_bf16, int d, const float *s2, int S, const int *rows,
                                    int n_rows, float *out, int out_stride, long long stream_from, hipStream_t s);
// cs[b][p] <- sqrt(sum over b' < B of cs[b'][p]^2) for every b < B, p < n
hipError_t launch_aggregate_scores(float *cs, int cs_stride, int B, int n, hipStream_t s);
// any[j] = 1 if mask[t][j] != 0 for some t < rows, else 0
hipError_t launch_mask_any(const unsigned char *mask, int rows, int m, unsigned char *any, hipStream_t s);
// scores[j] = nrm[j] * sqrt(sum_tile s2_part[tile][j])
hipError_t launch_scores_from_partials(const float *s2_part, int n_tiles, int m, const float *nrm, float *scores,
                                       hipStream_t s);
// stand-alone column reduction of a materialised H[T][m] (pop_importance.hip); scratch: device memory of
// importance_reduce_scratch_bytes(h, is_bf16, T, m) bytes (0: none), 8-byte aligned, for the per-chunk partial sums
size_t importance_reduce_scratch_bytes(const void *h, int is_bf16, int T, int m);
hipError_t launch_importance_reduce(const void *h, int is_bf16, int T, int m, const float *nrm, float *scores,
                                    void *scratch, hipStream_t s);

// s2[k] = sum_t x[t][k]^2 in one launch (not for very long prompts)
bool column_squares_takes(int T);
hipError_t launch_column_squares(const void *x, int is_bf16, int T, int d, float *s2, hipStream_t s);

}  // namespace pop
