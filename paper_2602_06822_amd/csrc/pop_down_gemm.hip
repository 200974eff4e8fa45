// Down projection of a whole prompt under the pruning structure (Sec. 3.4: the forward pass over the active channels):
//     Y[t][n] = sum over list positions c < a of  Hc[t][c] * W_down[n][list[c]],
// a K-gathered bf16 MFMA GEMM: the contraction runs over the a active channels, whose down columns are the rows
// w[list[c]][2][:] of the channel-major weights, contiguous along n.
//
// The matrix cores want both operands with the contraction index fastest inside a lane (8 consecutive k per lane for
// the 32x32x16 tile).  Hc is stored that way; the weight rows are not (n is contiguous, k jumps from row to row).
// They are staged into LDS as they come, [k][n], and fetched with the transposing LDS read of this chip: a block of
// 16 lanes points at a 4 (k) x 16 (n) patch, lane i at the 4 values of row i / 4 starting at column 4 (i % 4), and
// receives it transposed, lane j the 4 k-values of column j.  Two such reads make the 8 values of one B fragment.
//
// Short prompts do not give enough tiles to fill the chip, so the contraction is split into n_split ranges whose float32
// partial results are summed, in split order, by a second kernel (deterministic).  Kernels:
//  * down_gemm_rows_kernel (a prompt's own forward pass, d a multiple of 128): H by channel, [m][T], both operands are rows of the list;
//  * down_gemm_dma_kernel (d a multiple of 128): both operands go from global memory straight into rings of unpadded,
//    swizzled LDS buffers, with one exact wait per k-step (described at the kernel);
//  * down_gemm_bf16_kernel (other d): 256 tokens x 128 columns per workgroup, 8 waves (4 along the tokens x 2 along n), wave
//    tile 64 x 64 = 2 x 2 products of 32x32x16, k-steps of 64 channels; an LDS double buffer filled through registers with
//    the rows of two k-steps in flight; channel numbers are fetched a step further ahead so the weight loads never wait for
//    them.  Its weight tile has a row stride of 160 elements, which puts the 4 rows of a patch, and the two patches a read
//    instruction's half-wave touches, into disjoint banks.
#include "pop_internal.h"

namespace pop {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));

constexpr int kDgBM = 256;            // tokens per workgroup tile
constexpr int kDgBN = 128;            // output columns per workgroup tile
constexpr int kDgBK = 64;             // channels per k-step
constexpr int kDgLdA = kDgBK + 8;     // LDS row stride of the Hc tile in elements (144 B: conflict-free 16-byte reads)
constexpr int kDgLdB = kDgBN + 32;    // LDS row stride of the weight tile in elements (320 B)
constexpr int kDgMaxSplit = 8;

__device__ __forceinline__ int dg_xcd_logical_block(int bid, int per_xcd) { return (bid % 8) * per_xcd + bid / 8; }

__global__ __launch_bounds__(512) void down_gemm_bf16_kernel(const uint16_t *__restrict__ w, int d,
                                                             const int *__restrict__ list,
                                                             const int *__restrict__ n_list,
                                                             const uint16_t *__restrict__ hc, int ldh, int T, int n_tt,
                                                             int n_nt, int n_split, int per_xcd,
                                                             float *__restrict__ part, void *__restrict__ y, int y_bf16)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t dg_lds[];
    uint16_t *As = dg_lds;                          // [2][kDgBM * kDgLdA]
    uint16_t *Bs = dg_lds + 2 * kDgBM * kDgLdA;     // [2][kDgBK * kDgLdB]

    const int logical = dg_xcd_logical_block(blockIdx.x, per_xcd);
    if (logical >= n_tt * n_nt * n_split) return;
    // token tiles of one (split, column tile) are neighbours: they share its weight rows in the XCD's L2
    const int ttile = logical % n_tt, ntile = (logical / n_tt) % n_nt, split = logical / (n_tt * n_nt);
    const int t0 = ttile * kDgBM, n0 = ntile * kDgBN;

    const int a = *n_list;
    const int steps_all = (a + kDgBK - 1) / kDgBK, steps_per = (steps_all + n_split - 1) / n_split;
    const int ks0 = min(split * steps_per, steps_all), ks1 = min(ks0 + steps_per, steps_all);

    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int wm = wave / 2, wn = wave % 2;

    // staging.  Hc tile: 8 vectors of 16 bytes per row, 64 rows per pass, 4 passes; weight tile: 16 vectors per row,
    // 32 rows per pass, 2 passes
    const int a_row = tid / 8, a_kv = tid % 8;
    const int b_row = tid / 16, b_nv = tid % 16;
    // Every load below is unconditional (addresses clamped into valid memory, the value replaced afterwards where it
    // must not count), so that the loads of two k-steps can be in flight at once: with loads under branches the
    // compiler can only wait for all of them.  Token rows beyond T are clamped and never stored.
    const uint16_t *pa[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) pa[p] = hc + (size_t)min(t0 + a_row + p * 64, T - 1) * ldh;
    const bool n_ok = n0 + b_nv * 8 < d;
    const int n_col = n_ok ? n0 + b_nv * 8 : 0;
    uint4 ra[2][4], rb[2][2];  // two k-steps on their way through registers, as loaded
    uint32_t rb_on[2][2];      // all ones where the weight row exists, else 0
    int chn[2][2], chn_off[2][2];  // channels of this thread's two weight rows, two k-steps, as loaded; -1 where the
                                   // row does not exist, else 0 (kept apart so that nothing touches the loaded value
                                   // before its use a step later)
    auto load_channels = [&](int set, int ks) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int c = ks * kDgBK + b_row + p * 32;
            chn[set][p] = list[min(c, a - 1)];
            chn_off[set][p] = -(int)(ks >= ks1 || c >= a);
        }
    };
    auto load_global = [&](int set, int ks) {
        const int k = min(ks, ks1 - 1) * kDgBK + a_kv * 8;
        const int kc = k < a ? k : 0;
#pragma unroll
        for (int p = 0; p < 4; ++p) ra[set][p] = *reinterpret_cast<const uint4 *>(pa[p] + kc);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int j = chn[set][p] | chn_off[set][p];
            rb[set][p] = *reinterpret_cast<const uint4 *>(w + (size_t)max(j, 0) * channel_elems_bf16(d) + 2 * d + n_col);
            rb_on[set][p] = (j >= 0 && n_ok) ? 0xffffffffu : 0u;
        }
    };
    // writes the rows of k-step ks, loaded into set `buf`, to LDS buffer `buf`; what lies beyond the a channels or
    // the d columns is cleared here, where the loaded values are first touched
    auto store_lds = [&](int buf, int ks) {
        const int keep = a - (min(ks, ks1 - 1) * kDgBK + a_kv * 8);  // columns of the Hc vector that hold data
        uint32_t keep_bits[4];                                       // 16-bit elements, two per word
#pragma unroll
        for (int q = 0; q < 4; ++q)
            keep_bits[q] = 2 * q >= keep ? 0u : (2 * q + 1 >= keep ? 0xffffu : 0xffffffffu);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const uint4 v = ra[buf][p];
            *reinterpret_cast<uint4 *>(&As[(buf * kDgBM + a_row + p * 64) * kDgLdA + a_kv * 8]) =
                make_uint4(v.x & keep_bits[0], v.y & keep_bits[1], v.z & keep_bits[2], v.w & keep_bits[3]);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint4 v = rb[buf][p];
            const uint32_t on = rb_on[buf][p];
            *reinterpret_cast<uint4 *>(&Bs[(buf * kDgBK + b_row + p * 32) * kDgLdB + b_nv * 8]) =
                make_uint4(v.x & on, v.y & on, v.z & on, v.w & on);
        }
    };

    f32x16_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][f][v] = 0.f;

    // A fragment: row lane % 32 of the token fragment, k = kk + 8 (lane / 32) .. + 7.
    // B fragment, read r (k = kk + 8 (lane / 32) + 4 r .. + 3): this lane points at row (lane % 16) / 4 of that
    // group, columns 16 ((lane / 16) % 2) + 4 (lane % 4) .. + 3 of the fragment, and receives column lane % 32.
    const int a_off = (wm * 64 + lane % 32) * kDgLdA + (lane / 32) * 8;
    const int b_off = ((lane / 32) * 8 + (lane % 16) / 4) * kDgLdB + wn * 64 + 16 * ((lane / 16) % 2) + 4 * (lane % 4);
    auto multiply = [&](int buf) {
        const uint16_t *Ab = As + buf * kDgBM * kDgLdA + a_off;
        const uint16_t *Bb = Bs + buf * kDgBK * kDgLdB + b_off;
#pragma unroll
        for (int kk = 0; kk < kDgBK; kk += 16) {
            bf16x8_t af[2], bf[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const uint16_t *q = Bb + kk * kDgLdB + f * 32;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (s16x4_t __attribute__((address_space(3))) *)(q));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (s16x4_t __attribute__((address_space(3))) *)(q + 4 * kDgLdB));
                const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                bf[f] = __builtin_bit_cast(bf16x8_t, both);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) af[i] = *reinterpret_cast<const bf16x8_t *>(Ab + i * 32 * kDgLdA + kk);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int f = 0; f < 2; ++f)
                    acc[i][f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bf[f], acc[i][f], 0, 0, 0);
        }
    };

    // Step ks multiplies LDS buffer (ks - ks0) % 2.  Meanwhile the rows of step ks + 1 are in registers (set of the
    // other parity, requested one step earlier, written to the other buffer after the products), the rows of step
    // ks + 2 are requested into the set this buffer was filled from, and the channel numbers of step ks + 3 are
    // requested ahead of them, so that no wait for an older request also waits for a younger one that is not needed yet.
    const int n_steps = ks1 - ks0;
    if (n_steps > 0) {
        load_channels(0, ks0);
        load_global(0, ks0);
        load_channels(1, ks0 + 1);
        load_global(1, ks0 + 1);
        load_channels(0, ks0 + 2);
        store_lds(0, ks0);
        __syncthreads();
        auto step = [&](int ks, int b) {
            load_channels(b ^ 1, ks + 3);
            load_global(b, ks + 2);
            __builtin_amdgcn_sched_barrier(0);  // (keeps the requests ahead of the products in the instruction stream)
            multiply(b);
            __builtin_amdgcn_sched_barrier(0);
            store_lds(b ^ 1, ks + 1);
            __syncthreads();
        };
        int i = 0;
        for (; i + 1 < n_steps; i += 2) {
            step(ks0 + i, 0);
            step(ks0 + i + 1, 1);
        }
        if (i < n_steps) multiply(0);  // (an odd last step: its rows were stored by the step before)
    }

    // register v of a fragment is token row (v / 4) * 8 + (lane / 32) * 4 + v % 4, column lane % 32
    float *yp = part ? part + (size_t)split * T * d : nullptr;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const int n = n0 + wn * 64 + f * 32 + lane % 32;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = t0 + wm * 64 + i * 32 + (v / 4) * 8 + (lane / 32) * 4 + v % 4;
                if (t < T && n < d) {
                    const size_t o = (size_t)t * d + n;
                    if (yp) yp[o] = acc[i][f][v];
                    else if (y_bf16) ((uint16_t *)y)[o] = f32_to_bf16(acc[i][f][v]);
                    else ((float *)y)[o] = acc[i][f][v];
                }
            }
        }
}

// Both operands loaded straight into LDS (global_load_lds).  A tile is 64 MF tokens x 128 columns; four waves of 16 MF
// tokens x 128 columns each, 16x16x32 products.  Hc tile: rows of 128 bytes, unpadded, the 16-byte units of row r stored at
// unit ^ ((r / 2) % 8) (conflict-free 16-byte fragment reads).  Weight tile: 64 rows x 256 bytes as they come: a quarter
// wave reads one whole row.  The weight fragments are transposed in registers (two 16-byte rows, one byte permute per
// register), which measured the same as the transposing LDS read and leaves all reads to the compiler's own counting.
// One wave per SIMD, pipelined by hand like the prefill contraction (16x16x32 products move fewer accumulator bytes, four
// waves read 48 KB of fragments per 32-element slice where eight of 64 x 64 read 64 KB): while the
// products of one slice issue, the fragments of the next are read; a k-step is two slices, the first with the requests for
// weight rows and channel numbers, then the barrier, the second with the requests for Hc rows.
// Every wave issues the same loads in every k-step, so a step waits with an exact count for its own rows only.  Nothing is
// masked: token rows beyond T are pointed at the last token and never stored, list positions beyond the a channels are
// pointed at a row of zeros (zero_row, 256 bytes), which makes it irrelevant what the Hc columns beyond a hold, as long as
// it is finite (the buffer is cleared when it is allocated and only ever holds H values).  Needs d % 128 == 0 and
// ldh >= a rounded up to 64.
// What bounds it: no one thing.  The 48 KB of a k-step's loads at MF = 4 and its 96 KB of fragment reads take the LDS 1430 cycles (850 for
// the loads alone, 58 bytes a cycle from the L2; the two do not overlap) of the 2060 it takes at 2048 tokens, its products 1024.  Without the
// products 2048 tokens take 94 us of 133, 333 tokens at the 13B shape 31 of 42, an expert's 256 tokens 30 of 32; with the channel
// numbers counted up instead of read, or all rows from 64 channels, at most 2 us less in any of them.
// With one wave per SIMD, whatever does not fit between two products (12 cycles) comes on top, so the permutes of a fragment
// stand between the products of the one before it and a weight row's address is one multiply-add (both in a bunch in front of their use
// before): 333 tokens at the 13B shape 42.7 -> 40.5 us, 2048 tokens at d 4096 169 -> 159 (under the kernel trace), 256 tokens 33.6 -> 32.8,
// of which 8-15 us are the start, the first rows and the partials' way out.
constexpr int kDdThreads = 256;
constexpr int kDdMaxMF = 5;
constexpr int kDdSlots = 8;  // k-steps whose channel numbers are kept
template <int MF>
struct DdRing {
    static constexpr int NA = MF >= 5 ? 2 : (MF >= 3 ? 3 : 4);
    static constexpr int NB = MF == 4 ? 3 : 4;
    static constexpr size_t kBytes = (size_t)(NA * 64 * MF * kDgBK + NB * kDgBK * kDgBN) * sizeof(uint16_t) + kDdSlots * kDgBK * 4;
};

// The tile's results: register v of product e is token 4 (lane / 16) + v of the fragment, column 8 (lane % 16) + e; row0 is register
// 0's token in fragment 0, fragments are `apart` tokens apart.
template <int MF>
__device__ __forceinline__ void dd_store(const f32x4_t (&acc)[MF][kDgBN / 16], int row0, int apart, size_t col, int split, int T,
                                         int d, float *__restrict__ part, void *__restrict__ y, int y_bf16)
{
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int t = row0 + i * apart + v;
            if (t >= T) continue;
            if (part || !y_bf16) {
                float4 *dst = reinterpret_cast<float4 *>((part ? part + (size_t)split * T * d : (float *)y) + (size_t)t * d + col);
                dst[0] = make_float4(acc[i][0][v], acc[i][1][v], acc[i][2][v], acc[i][3][v]);
                dst[1] = make_float4(acc[i][4][v], acc[i][5][v], acc[i][6][v], acc[i][7][v]);
            } else {
                uint32_t q[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    q[e] = (uint32_t)f32_to_bf16(acc[i][2 * e][v]) | ((uint32_t)f32_to_bf16(acc[i][2 * e + 1][v]) << 16);
                *reinterpret_cast<uint4 *>((uint16_t *)y + (size_t)t * d + col) = make_uint4(q[0], q[1], q[2], q[3]);
            }
        }
}

template <int MF, bool kStream>
__device__ __forceinline__ void dd_tile(const uint16_t *__restrict__ w, int d, const int *__restrict__ list,
                                        const int *__restrict__ n_list, const uint16_t *__restrict__ hc, int ldh, int T,
                                        int n_tt, int n_nt, int n_split, int per_xcd, const uint16_t *__restrict__ zero_row,
                                        float *__restrict__ part, void *__restrict__ y, int y_bf16)
{
    typedef __attribute__((address_space(3))) void lds_t;
    typedef __attribute__((address_space(1))) const void glb_t;
    constexpr int NA = DdRing<MF>::NA, NB = DdRing<MF>::NB, F = kDgBN / 16;
    constexpr int BM = 64 * MF, AT = BM * kDgBK, BT = kDgBK * kDgBN;  // elements per stage
    constexpr int PA = BM / 32, PB = 4;  // direct loads per wave and k-step (and one of channel numbers)
    extern __shared__ __attribute__((aligned(16))) uint16_t dg_lds[];
    uint16_t *As = dg_lds;            // [NA][64 MF * 64]
    uint16_t *Bs = dg_lds + NA * AT;  // [NB][64 * 128]
    int *Cs = reinterpret_cast<int *>(Bs + NB * BT);  // [8][64]

    const int logical = dg_xcd_logical_block(blockIdx.x, per_xcd);
    if (logical >= n_tt * n_nt * n_split) return;
    // token tiles of one (split, column tile) are neighbours: they share its weight rows in the XCD's L2
    const int ttile = logical % n_tt, ntile = (logical / n_tt) % n_nt, split = logical / (n_tt * n_nt);
    const int t0 = ttile * BM, n0 = ntile * kDgBN;

    const int a = *n_list;
    const int steps_all = (a + kDgBK - 1) / kDgBK, steps_per = (steps_all + n_split - 1) / n_split;
    const int ks0 = min(split * steps_per, steps_all), ks1 = min(ks0 + steps_per, steps_all);
    const int n_steps = ks1 - ks0;

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);

    f32x4_t acc[MF][F];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][f][v] = 0.f;

    if (n_steps > 0) {
        // direct loads.  Hc: pass p of wave w covers rows 32 p + 8 w + lane / 8, this lane the unit that belongs at
        // position lane % 8 of its row.  Weights: pass p covers rows 16 p + 4 w + lane / 16, unit lane % 16.
        const int a_row = wave * 8 + lane / 8;
        const int a_src = ((lane % 8) ^ ((a_row / 2) % 8)) * 8;  // (passes are 32 rows apart: same swizzle term)
        // (32 bits reach over the 32 rows of a pass whatever their length: 44 million channels at most)
        const uint16_t *hc_pass[PA];  // the pass's first row
        uint32_t a_off[PA];           // bytes from there
#pragma unroll
        for (int p = 0; p < PA; ++p) {
            const int first = min(t0 + p * 32, T - 1);
            hc_pass[p] = hc + (size_t)first * ldh;
            a_off[p] = 2 * ((uint32_t)(min(t0 + a_row + p * 32, T - 1) - first) * (uint32_t)ldh + a_src);
        }
        const int b_row = wave * 4 + lane / 16;
        const uintptr_t b_col = (uintptr_t)(w + 2 * d + n0 + (lane % 16) * 8), b_zero = (uintptr_t)(zero_row + (lane % 16) * 8);
        const uint32_t b_stride = (uint32_t)(channel_elems_bf16(d) * sizeof(uint16_t));
        // Channel numbers of a k-step: one direct load of 64 of them into slot step % 8 of a small ring, two steps before
        // they are needed (every wave loads the same, so that its own waits cover it).
        auto load_channels = [&](int step) {
            const int *src = list + min(min(ks0 + step, ks1 - 1) * kDgBK + lane, a - 1);
            __builtin_amdgcn_global_load_lds((glb_t *)src, (lds_t *)(Cs + step % kDdSlots * kDgBK), 4, 0, 0);
        };
        // (read with their own wait: seen as an ordinary read it would be taken to alias the direct loads in flight and wait
        // for all of them)
        auto channels = [&](int (&c)[PB], int step) {
            const uint32_t at = (uint32_t)(uintptr_t)(Cs + step % kDdSlots * kDgBK + b_row);
            asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:64\n\tds_read_b32 %2, %4 offset:128\n\t"
                         "ds_read_b32 %3, %4 offset:192\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(c[0]), "=&v"(c[1]), "=&v"(c[2]), "=&v"(c[3])
                         : "v"(at)
                         : "memory");
        };
        auto load_a = [&](int p, int buf, int step) {
            const char *k = (const char *)(hc_pass[p] + min(ks0 + step, ks1 - 1) * kDgBK);
            __builtin_amdgcn_global_load_lds((glb_t *)(k + a_off[p]), (lds_t *)(As + buf * AT + (p * 32 + wave * 8) * kDgBK), 16, 0, 0);
        };
        // (the row is selected with a mask: a conditional would put the load under a branch and make its wait inexact; one 64-bit
        // multiply-add for the address: what does not fit between two products is time lost)
        auto load_b = [&](int c, int p, int buf, int step) {
            const int ks = ks0 + step, n_live = ks < ks1 ? a - ks * kDgBK - p * 16 : 0;
            const uintptr_t live = -(uintptr_t)(b_row < n_live);
            const uintptr_t row = b_col + (uint64_t)(uint32_t)c * b_stride;
            __builtin_amdgcn_global_load_lds((glb_t *)(b_zero ^ ((row ^ b_zero) & live)),
                                             (lds_t *)(Bs + buf * BT + (p * 16 + wave * 4) * kDgBN), 16, 0,
                                             kStream ? 2 : 0);  // (2: non-temporal)
        };
        // Fragment reads.  A: row lane % 16 of the token fragment, unit 4 q + lane / 16 under the row's swizzle.  Weights: lane
        // (c, g) = (lane % 16, lane / 16) reads columns 8 c .. 8 c + 7 of rows 32 q + 8 g .. + 7, which is a transposed
        // operand: one byte permute per register pairs the values of two rows, and product e takes column 8 c + e of every
        // lane.
        const uint16_t *Al = As + (wave * MF * 16 + lane % 16) * kDgBK;
        const uint16_t *Bl = Bs + (lane / 16) * 8 * kDgBN + (lane % 16) * 8;
        int koff[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) koff[q] = ((q * 4 + lane / 16) ^ ((lane % 16) / 2)) * 8;
        bf16x8_t af[2][MF];
        bf16x8_t rows[2][8];
        constexpr int NR = 8 + MF, NP = MF * F;
        auto fetch = [&](const uint16_t *Ab, const uint16_t *Bb, int i, int q, int set) {
            if (i < 8)
                rows[set][i] = *reinterpret_cast<const bf16x8_t *>(Bb + (q * 32 + i) * kDgBN);
            else
                af[set][i - 8] = *reinterpret_cast<const bf16x8_t *>(Ab + (i - 8) * 16 * kDgBK + koff[q]);
        };
        // product i: fragment i / MF of the columns, i % MF of the tokens.  The permutes that make a fragment of the columns
        // stand between the products of the fragment before it; those of the next slice's first fragment between the last ones
        // of this slice, when its rows have been read (one token fragment: reads last to the end, `first_pairs` follows them).
        uint32_t bw[2][4];
        auto pair = [&](int e, int q, int set) {
            const u32x4_t r0 = __builtin_bit_cast(u32x4_t, rows[set][2 * q]);
            const u32x4_t r1 = __builtin_bit_cast(u32x4_t, rows[set][2 * q + 1]);
            bw[e % 2][q] = __builtin_amdgcn_perm(r1[e / 2], r0[e / 2], e % 2 ? 0x07060302u : 0x05040100u);
        };
        auto product = [&](int i, int set) {
            const int e = i / MF, m_ = i % MF;
            const u32x4_t b = {bw[e % 2][0], bw[e % 2][1], bw[e % 2][2], bw[e % 2][3]};
            // (two wait states behind the last permute, which the compiler does not see that a product needs: two products
            // where a fragment has three or more.  Nothing else writes an operand that late as long as the loop below stays one
            // body: a second copy of it for an odd last step had the compiler move every accumulator out and back in between
            // its products.)
            if (MF < 3 && m_ == 0)
                asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[m_][e]) : "v"(af[set][m_]), "v"(b));
            else
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[m_][e]) : "v"(af[set][m_]), "v"(b));
            constexpr int kGaps = MF < 3 ? 1 : MF - 2;
            if (m_ < kGaps && (MF > 1 || e + 1 < F)) {
#pragma unroll
                for (int q = m_ * 4 / kGaps; q < (m_ + 1) * 4 / kGaps; ++q) pair((e + 1) % F, q, e + 1 < F ? set : set ^ 1);
            }
        };
        auto first_pairs = [&](int set) {
#pragma unroll
            for (int q = 0; q < 4; ++q) pair(0, q, set);
        };
        // Requests in program order: ... A(s + NA - 1) | C(s + NB + 1), B(s + NB - 1) [wait for step s + 1] A(s + NA) | ...: the
        // wait may leave in flight what was issued after A(s + 1), B(s + 1) and the C that the next B requests use
        constexpr int kAfterA = (NA - 1) * (PB + 1) + (NA - 2) * PA, kAfterB = (NB - 2) * (PA + PB + 1);
        constexpr int kAfterC = PA + 2 * PB + 1;
        constexpr int kRows = kAfterA < kAfterB ? kAfterA : kAfterB, kYounger = kRows < kAfterC ? kRows : kAfterC;
        static_assert(kYounger < 64 && (NB - 2) * PB + (NA - 1) * PA < 64, "vmcnt is a 6-bit counter");
        // What steps before the first would have requested: channel numbers up to step NB, then the first NB - 1 steps of
        // weight rows and the first NA of token rows, step by step; the first two waits leave what comes after their step.
        static_assert(NB + 2 <= kDdSlots && NA >= 2 && NB >= 3, "rings");
        static_assert(kYounger <= (NB - 3) * PB + (NA - 2) * PA + PB + 1, "the wait of the first step");
        for (int q = 0; q <= NB; ++q) load_channels(q);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int chn[PB];
        constexpr int kDeep = NA > NB - 1 ? NA : NB - 1;
#pragma unroll
        for (int q = 0; q < kDeep; ++q) {
            if (q < NB - 1) {
                channels(chn, q);
#pragma unroll
                for (int p = 0; p < PB; ++p) load_b(chn[p], p, q, q);
            }
            if (q < NA) {
#pragma unroll
                for (int p = 0; p < PA; ++p) load_a(p, q, q);
            }
        }
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NB - 2) * PB + (NA - 1) * PA) : "memory");
        int abuf = 0, bbuf = 0, bprev = NB - 1;
        constexpr int kSpread = NP > 8 ? NP * 3 / 4 : NP;  // products the reads are spread over: the last have time to arrive
#pragma unroll
        for (int i = 0; i < NR; ++i) fetch(Al, Bl, i, 0, 0);
        first_pairs(0);
        auto k_step = [&](int s) {
            const uint16_t *Ab = Al + abuf * AT, *Bb = Bl + bbuf * BT;
            load_channels(s + NB + 1);
            channels(chn, s + NB - 1);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                product(i, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = min(i, kSpread) * NR / kSpread; r < min(i + 1, kSpread) * NR / kSpread; ++r) fetch(Ab, Bb, r, 1, 1);
#pragma unroll
                for (int p = i * PB / NP; p < (i + 1) * PB / NP; ++p) load_b(chn[p], p, bprev, s + NB - 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (MF == 1) first_pairs(1);
            // this wave's reads of the buffers are over and its rows of the next step have landed; after the barrier so are
            // everybody's and have everybody's
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kYounger) : "memory");
            const int a_free = abuf;
            bprev = bbuf;
            abuf = abuf + 1 == NA ? 0 : abuf + 1;
            bbuf = bbuf + 1 == NB ? 0 : bbuf + 1;
            Ab = Al + abuf * AT, Bb = Bl + bbuf * BT;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                product(i, 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = min(i, kSpread) * NR / kSpread; r < min(i + 1, kSpread) * NR / kSpread; ++r) fetch(Ab, Bb, r, 0, 0);
#pragma unroll
                for (int p = i * PA / NP; p < (i + 1) * PA / NP; ++p) load_a(p, a_free, s + NA);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (MF == 1) first_pairs(0);
        };
        for (int s = 0; s < n_steps; ++s) k_step(s);
        // the surplus requests, before the LDS is given up; the products' results before they are read (the compiler does
        // not see the products, so it adds no wait states for them)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int f = 0; f < F; ++f) asm volatile("" : "+a"(acc[i][f]));  // (no read of them moves ahead of the wait)
    }

    dd_store<MF>(acc, t0 + wave * MF * 16 + lane / 16 * 4, 16, n0 + lane % 16 * 8, split, T, d, part, y, y_bf16);
}

template <int MF>
__global__ __launch_bounds__(kDdThreads, 1) void down_gemm_dma_kernel(const uint16_t *__restrict__ w, int d,
                                                                      const int *__restrict__ list,
                                                                      const int *__restrict__ n_list,
                                                                      const uint16_t *__restrict__ hc, int ldh, int T,
                                                                      int n_tt, int n_nt, int n_split, int per_xcd,
                                                                      const uint16_t *__restrict__ zero_row,
                                                                      float *__restrict__ part, void *__restrict__ y,
                                                                      int y_bf16)
{
    dd_tile<MF, false>(w, d, list, n_list, hc, ldh, T, n_tt, n_nt, n_split, per_xcd, zero_row, part, y, y_bf16);
}

// The same with weight rows past the caches: one token tile, so every row is read once, on layers of stream_rows.
template <int MF>
__global__ __launch_bounds__(kDdThreads, 1) void down_gemm_stream_kernel(const uint16_t *__restrict__ w, int d,
                                                                         const int *__restrict__ list,
                                                                         const int *__restrict__ n_list,
                                                                         const uint16_t *__restrict__ hc, int ldh, int T,
                                                                         int n_tt, int n_nt, int n_split, int per_xcd,
                                                                         const uint16_t *__restrict__ zero_row,
                                                                         float *__restrict__ part, void *__restrict__ y,
                                                                         int y_bf16)
{
    dd_tile<MF, true>(w, d, list, n_list, hc, ldh, T, n_tt, n_nt, n_split, per_xcd, zero_row, part, y, y_bf16);
}

// Loads straight into LDS, 16 or 4 bytes a lane to consecutive places from `to` on (the same in all lanes).  Inline assembly: the compiler
// takes some LDS reads (of channel numbers, transposing ones) for reads of what direct loads write, and would wait for all of those in
// flight in front of each.  They have no register results, and the kernels' own counted waits are the only ones they need.  m0 is a
// reserved register and cannot be named as changed: nothing else in these kernels may use it, which the listing's test looks after
// (saved and put back around every load: 13B shape, 2048 tokens 707 -> 723 us, eight experts' sizes up to 1 %).
__device__ __forceinline__ int dd_lds(const void *to) { return __builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)to); }
template <bool kStream>
__device__ __forceinline__ void dd_load16(const void *to, uintptr_t from)
{
    if constexpr (kStream)  // (non-temporal)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" : : "s"(dd_lds(to)), "v"(from));
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(dd_lds(to)), "v"(from));
}
__device__ __forceinline__ void dd_load4(const void *to, const void *from)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(dd_lds(to)), "v"(from));
}

// The same contraction over H by channel, ht[j][ldt] of all m channels (written so by the prompt's own contraction): both operands
// are rows of the listed channels, so there is no gather of H's columns in front (17 us at 2048 tokens, 6 at an expert's 256).
// H tile: MF panels of 64 channels x 64 tokens, rows of 128 bytes as they come; a wave owns 16 tokens of every panel (its fragment i
// is of panel i) and fetches them with the transposing LDS read: of each 16 lanes, lane l points at the 4 tokens 4 (l % 4) .. of
// row l / 4 and receives the 4 channels of token l, twice for the 8 of a fragment.  The 32-byte pieces of row r are stored at piece
// ^ ((r / 2) % 2 + 2 ((r / 8) % 2)): the eight rows of a half wave's read fall into different banks.
// Everything else as in dd_tile: list positions beyond the a channels are rows of zeros in both operands; tokens beyond T belong to
// rows that are not stored (behind the last row kRowsSlack elements are readable).  A step's channel numbers are read once, for the
// H rows NA steps and the weight rows NB - 1 steps ahead, and loaded a step earlier than there.
template <int MF, bool kStream>
__global__ __launch_bounds__(kDdThreads, 1) void down_gemm_rows_kernel(const uint16_t *__restrict__ w, int d,
                                                                       const int *__restrict__ list, int a,
                                                                       const uint16_t *__restrict__ ht, int ldt, int T,
                                                                       int n_tt, int n_nt, int n_split, int per_xcd,
                                                                       const uint16_t *__restrict__ zero_row,
                                                                       float *__restrict__ part, void *__restrict__ y,
                                                                       int y_bf16)
{
    constexpr int NA = DdRing<MF>::NA, NB = DdRing<MF>::NB, F = kDgBN / 16;
    constexpr int BM = 64 * MF, PT = 64 * kDgBK, AT = MF * PT, BT = kDgBK * kDgBN;  // elements per panel and stage
    constexpr int PA = 2 * MF, PB = 4;  // direct loads per wave and k-step (and one of channel numbers)
    extern __shared__ __attribute__((aligned(16))) uint16_t dg_lds[];
    uint16_t *As = dg_lds;            // [NA][MF][64 * 64]
    uint16_t *Bs = dg_lds + NA * AT;  // [NB][64 * 128]
    int *Cs = reinterpret_cast<int *>(Bs + NB * BT);  // [8][64]

    const int logical = dg_xcd_logical_block(blockIdx.x, per_xcd);
    if (logical >= n_tt * n_nt * n_split) return;
    const int ttile = logical % n_tt, ntile = (logical / n_tt) % n_nt, split = logical / (n_tt * n_nt);
    const int t0 = ttile * BM, n0 = ntile * kDgBN;

    const int steps_all = (a + kDgBK - 1) / kDgBK, steps_per = (steps_all + n_split - 1) / n_split;
    const int ks0 = min(split * steps_per, steps_all), ks1 = min(ks0 + steps_per, steps_all);
    const int n_steps = ks1 - ks0;

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);

    f32x4_t acc[MF][F];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][f][v] = 0.f;

    if (n_steps > 0) {
        // direct loads.  H: half q of a panel is 32 rows, 8 of them by this wave, this lane the unit that belongs at position lane % 8
        // of row a_row; the same rows of every panel.  Weights: pass p covers rows 16 p + 4 w + lane / 16, unit lane % 16.
        const int a_row = wave * 8 + lane / 8;
        const int a_src = ((lane % 8 / 2) ^ (lane / 16 % 2 + 2 * (wave % 2))) * 16 + lane % 2 * 8;
        const uintptr_t a_col = (uintptr_t)(ht + t0 + a_src), a_zero = (uintptr_t)(zero_row + a_src);
        const uint32_t a_stride = (uint32_t)ldt * (uint32_t)sizeof(uint16_t);
        const int b_row = wave * 4 + lane / 16;
        const uintptr_t b_col = (uintptr_t)(w + 2 * d + n0 + (lane % 16) * 8), b_zero = (uintptr_t)(zero_row + (lane % 16) * 8);
        const uint32_t b_stride = (uint32_t)(channel_elems_bf16(d) * sizeof(uint16_t));
        auto load_channels = [&](int step) {
            dd_load4(Cs + step % kDdSlots * kDgBK, list + min(min(ks0 + step, ks1 - 1) * kDgBK + lane, a - 1));
        };
        auto channels = [&](int (&ca)[2], int (&cb)[PB], int step_a, int step_b) {
            const int *at_a = Cs + step_a % kDdSlots * kDgBK + a_row, *at_b = Cs + step_b % kDdSlots * kDgBK + b_row;
            ca[0] = at_a[0], ca[1] = at_a[32];
#pragma unroll
            for (int p = 0; p < PB; ++p) cb[p] = at_b[16 * p];
        };
        // A row's address, with a row of zeros beyond the list (selected with masks: no branch around a load).
        auto row_of = [&](int c, int row, int step, uintptr_t col, uint32_t stride, uintptr_t zero) {
            const int ks = ks0 + step, n_live = ks < ks1 ? a - ks * kDgBK : 0;
            const uintptr_t live = -(uintptr_t)(row < n_live), at = col + (uint64_t)(uint32_t)c * stride;
            return zero ^ ((at ^ zero) & live);
        };
        // pass p: panel p / 2, rows 32 (p % 2) ..
        auto load_a = [&](const uintptr_t (&rows)[2], int p, int buf) {
            dd_load16<false>(As + buf * AT + p / 2 * PT + (p % 2 * 32 + wave * 8) * 64, rows[p % 2] + p / 2 * 128);
        };
        auto load_b = [&](int c, int p, int buf, int step) {
            dd_load16<kStream>(Bs + buf * BT + (p * 16 + wave * 4) * kDgBN, row_of(c, b_row + 16 * p, step, b_col, b_stride, b_zero));
        };
        // Fragment reads.  H: lanes 16 g .. + 15 read rows 32 q + 8 g + 4 half + (lane % 16) / 4.  Weights as in dd_tile.
        const uint16_t *Al = As + (lane / 16 * 8 + lane % 16 / 4) * 64 +
                             (wave ^ (lane % 16 / 8 + 2 * (lane / 16 % 2))) * 16 + lane % 4 * 4;
        const uint16_t *Bl = Bs + (lane / 16) * 8 * kDgBN + (lane % 16) * 8;
        s16x4_t af[2][MF][2];
        bf16x8_t rows[2][8];
        constexpr int NR = 8 + 2 * MF, NP = MF * F;
        auto fetch = [&](const uint16_t *Ab, const uint16_t *Bb, int i, int q, int set) {
            if (i < 8)
                rows[set][i] = *reinterpret_cast<const bf16x8_t *>(Bb + (q * 32 + i) * kDgBN);
            else
                af[set][(i - 8) / 2][i % 2] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (s16x4_t __attribute__((address_space(3))) *)(Ab + (i - 8) / 2 * PT + (q * 32 + i % 2 * 4) * 64));
        };
        uint32_t bw[2][4];
        auto pair = [&](int e, int q, int set) {
            const u32x4_t r0 = __builtin_bit_cast(u32x4_t, rows[set][2 * q]);
            const u32x4_t r1 = __builtin_bit_cast(u32x4_t, rows[set][2 * q + 1]);
            bw[e % 2][q] = __builtin_amdgcn_perm(r1[e / 2], r0[e / 2], e % 2 ? 0x07060302u : 0x05040100u);
        };
        auto product = [&](int i, int set) {
            const int e = i / MF, m_ = i % MF;
            const u32x4_t b = {bw[e % 2][0], bw[e % 2][1], bw[e % 2][2], bw[e % 2][3]};
            const s16x8_t h = __builtin_shufflevector(af[set][m_][0], af[set][m_][1], 0, 1, 2, 3, 4, 5, 6, 7);
            // (wait states as in dd_tile)
            if (MF < 3 && m_ == 0)
                asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[m_][e]) : "v"(h), "v"(b));
            else
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[m_][e]) : "v"(h), "v"(b));
            constexpr int kGaps = MF < 3 ? 1 : MF - 2;
            if (m_ < kGaps && (MF > 1 || e + 1 < F)) {
#pragma unroll
                for (int q = m_ * 4 / kGaps; q < (m_ + 1) * 4 / kGaps; ++q) pair((e + 1) % F, q, e + 1 < F ? set : set ^ 1);
            }
        };
        auto first_pairs = [&](int set) {
#pragma unroll
            for (int q = 0; q < 4; ++q) pair(0, q, set);
        };
        // Requests in program order: ... A(s + NA - 1) | C(s + NB + 2), B(s + NB - 1) [wait for step s + 1] A(s + NA) | ...: the
        // wait may leave in flight what was issued after A(s + 1), B(s + 1) and the C that step s + 1 reads, C(s + 1 + NB) at most,
        // issued one step before
        constexpr int kAfterA = (NA - 1) * (PB + 1) + (NA - 2) * PA, kAfterB = (NB - 2) * (PA + PB + 1);
        constexpr int kAfterC = PA + 2 * PB + 1;
        constexpr int kRows = kAfterA < kAfterB ? kAfterA : kAfterB, kYounger = kRows < kAfterC ? kRows : kAfterC;
        static_assert(kYounger < 64 && (NB - 2) * PB + (NA - 1) * PA < 64, "vmcnt is a 6-bit counter");
        static_assert(NB + 3 <= kDdSlots && NA <= NB && NA >= 2 && NB >= 3, "rings");
        static_assert(kYounger <= (NB - 3) * PB + (NA - 2) * PA + PB + 1, "the wait of the first step");
        for (int q = 0; q <= NB + 1; ++q) load_channels(q);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int cha[2], chn[PB];
        uintptr_t ra[2];
        constexpr int kDeep = NA > NB - 1 ? NA : NB - 1;
#pragma unroll
        for (int q = 0; q < kDeep; ++q) {
            channels(cha, chn, q, q);
            if (q < NB - 1) {
#pragma unroll
                for (int p = 0; p < PB; ++p) load_b(chn[p], p, q, q);
            }
            if (q < NA) {
#pragma unroll
                for (int e = 0; e < 2; ++e) ra[e] = row_of(cha[e], a_row + 32 * e, q, a_col, a_stride, a_zero);
#pragma unroll
                for (int p = 0; p < PA; ++p) load_a(ra, p, q);
            }
        }
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NB - 2) * PB + (NA - 1) * PA) : "memory");
        int abuf = 0, bbuf = 0, bprev = NB - 1;
        constexpr int kSpread = NP > 8 ? NP * 3 / 4 : NP;  // products the reads are spread over: the last have time to arrive
#pragma unroll
        for (int i = 0; i < NR; ++i) fetch(Al, Bl, i, 0, 0);
        first_pairs(0);
        for (int s = 0; s < n_steps; ++s) {
            const uint16_t *Ab = Al + abuf * AT, *Bb = Bl + bbuf * BT;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                product(i, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (i == 0) channels(cha, chn, s + NA, s + NB - 1);
                if (i == 1) load_channels(s + NB + 2);
#pragma unroll
                for (int r = min(i, kSpread) * NR / kSpread; r < min(i + 1, kSpread) * NR / kSpread; ++r) fetch(Ab, Bb, r, 1, 1);
#pragma unroll
                for (int p = i * PB / NP; p < (i + 1) * PB / NP; ++p) load_b(chn[p], p, bprev, s + NB - 1);
                if (i >= NP - 2) ra[i - (NP - 2)] = row_of(cha[i - (NP - 2)], a_row + 32 * (i - (NP - 2)), s + NA, a_col, a_stride, a_zero);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (MF == 1) first_pairs(1);
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kYounger) : "memory");
            const int a_free = abuf;
            bprev = bbuf;
            abuf = abuf + 1 == NA ? 0 : abuf + 1;
            bbuf = bbuf + 1 == NB ? 0 : bbuf + 1;
            Ab = Al + abuf * AT, Bb = Bl + bbuf * BT;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                product(i, 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = min(i, kSpread) * NR / kSpread; r < min(i + 1, kSpread) * NR / kSpread; ++r) fetch(Ab, Bb, r, 0, 0);
#pragma unroll
                for (int p = i * PA / NP; p < (i + 1) * PA / NP; ++p) load_a(ra, p, a_free);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (MF == 1) first_pairs(0);
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int f = 0; f < F; ++f) asm volatile("" : "+a"(acc[i][f]));  // (no read of them moves ahead of the wait)
    }
    dd_store<MF>(acc, t0 + wave * 16 + lane / 16 * 4, 64, n0 + lane % 16 * 8, split, T, d, part, y, y_bf16);
}

// y = sum over the splits, in split order, of part[split]; n4 = T * d / 4 vectors.
__global__ __launch_bounds__(256) void down_gemm_reduce_kernel(const float4 *__restrict__ part, int n_split, size_t n4,
                                                               void *__restrict__ y, int y_bf16)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    float4 s = part[i];
    for (int q = 1; q < n_split; ++q) {
        const float4 v = part[(size_t)q * n4 + i];
        s.x += v.x, s.y += v.y, s.z += v.z, s.w += v.w;
    }
    if (y_bf16) {
        uint2 o;
        o.x = (uint32_t)f32_to_bf16(s.x) | ((uint32_t)f32_to_bf16(s.y) << 16);
        o.y = (uint32_t)f32_to_bf16(s.z) | ((uint32_t)f32_to_bf16(s.w) << 16);
        ((uint2 *)y)[i] = o;
    } else {
        ((float4 *)y)[i] = s;
    }
}

// Token fragments per wave (tiles of 64 MF tokens) and ranges the contraction is split into so that the tiles fill the
// compute units.  A tile's time per k-slice: its products (16 cycles each on one matrix pipe) and what the LDS and the loads
// add; splits shorten it, tiles beyond one per compute unit lengthen it.
static int dd_shape(int T, int d, int n_cu, int *n_split)
{
    int best = 4;
    long best_cost = -1;
    for (int mf = kDdMaxMF; mf >= 1; --mf) {
        const long tiles = (long)((T + 64 * mf - 1) / (64 * mf)) * ((d + kDgBN - 1) / kDgBN);
        long split = n_cu / tiles;
        if (split < 1) split = 1;
        if (split > kDgMaxSplit) split = kDgMaxSplit;
        const long cost = (tiles * split + n_cu - 1) / n_cu * (144 * mf + 100) * 840 / split;
        if (best_cost < 0 || cost < best_cost) best_cost = cost, best = mf, *n_split = (int)split;
    }
    return best;
}

int down_gemm_splits(int T, int d, int n_cu)
{
    int n_split = 1;
    if (d % kDgBN == 0) {
        dd_shape(T, d, n_cu, &n_split);
        return n_split;
    }
    const int tiles = ((T + kDgBM - 1) / kDgBM) * ((d + kDgBN - 1) / kDgBN);
    n_split = n_cu / tiles;
    if (n_split < 1) n_split = 1;
    if (n_split > kDgMaxSplit) n_split = kDgMaxSplit;
    return n_split;
}

template <int MF>
static hipError_t launch_dd(const void *w, int d, const int *list, const int *n_list, const uint16_t *hc, int ldh, int T,
                            int n_split, float *part, void *y, int y_bf16, hipStream_t s, const uint16_t *zero_row)
{
    const size_t lds = DdRing<MF>::kBytes;
    const int n_tt = (T + 64 * MF - 1) / (64 * MF), n_nt = d / kDgBN, per_xcd = (n_tt * n_nt * n_split + 7) / 8;
    // (ldh: the layer's channels rounded up to 64)
    const bool stream = n_tt == 1 && stream_rows(d, ldh, 1, kStreamFfnBytes);
    const auto kernel = stream ? down_gemm_stream_kernel<MF> : down_gemm_dma_kernel<MF>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(per_xcd * 8), dim3(kDdThreads), lds, s, (const uint16_t *)w, d, list,
                       n_list, hc, ldh, T, n_tt, n_nt, n_split, per_xcd, zero_row, part, y, y_bf16);
    return hipGetLastError();
}

static hipError_t down_gemm_reduce(const float *part, int n_split, int T, int d, void *y, int y_bf16, hipStream_t s)
{
    if (n_split <= 1) return hipSuccess;
    const size_t n4 = (size_t)T * d / 4;
    hipLaunchKernelGGL(down_gemm_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, (const float4 *)part,
                       n_split, n4, y, y_bf16);
    return hipGetLastError();
}

bool down_gemm_by_channel(int d) { return d % kDgBN == 0; }

hipError_t launch_down_gemm_rows(const void *w, int d, int m, const int *list, int n_list, const uint16_t *ht, int ldt,
                                 int T, int n_split, int n_cu, float *part, void *y, int y_bf16, hipStream_t s,
                                 const uint16_t *zero_row)
{
    if (!down_gemm_by_channel(d) || ldt % 64 || ldt < T) return hipErrorInvalidValue;
    int split = 1;
    void (*kernel)(const uint16_t *, int, const int *, int, const uint16_t *, int, int, int, int, int, int, const uint16_t *, float *,
                   void *, int);
    size_t lds = 0;
    const int mf = dd_shape(T, d, n_cu, &split), n_tt = (T + 64 * mf - 1) / (64 * mf);
    const bool stream = n_tt == 1 && stream_rows(d, m, 1, kStreamPromptBytes);
    switch (mf) {
#define POP_DR(MF)                                                                           \
    case MF:                                                                                 \
        kernel = stream ? down_gemm_rows_kernel<MF, true> : down_gemm_rows_kernel<MF, false>; \
        lds = DdRing<MF>::kBytes;                                                            \
        break;
        POP_DR(5) POP_DR(4) POP_DR(3) POP_DR(2) POP_DR(1)
#undef POP_DR
        default: return hipErrorInvalidValue;
    }
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    const int n_nt = d / kDgBN, per_xcd = (n_tt * n_nt * n_split + 7) / 8;
    hipLaunchKernelGGL(kernel, dim3(per_xcd * 8), dim3(kDdThreads), lds, s, (const uint16_t *)w, d, list, n_list, ht, ldt, T, n_tt,
                       n_nt, n_split, per_xcd, zero_row, n_split > 1 ? part : nullptr, y, y_bf16);
    e = hipGetLastError();
    return e != hipSuccess ? e : down_gemm_reduce(part, n_split, T, d, y, y_bf16, s);
}

// bf16 only; d % 8 == 0, ldh % 8 == 0.  part: float32 [n_split][T][d], needed when n_split > 1.  zero_row: 256 bytes
// of zeros (optional); with it, d % 128 == 0 and ldh % 64 == 0 the direct-load kernel runs, which reads Hc columns up to
// the list length rounded up to 64.
hipError_t launch_down_gemm_bf16(const void *w, int d, const int *list, const int *n_list, const uint16_t *hc, int ldh,
                                 int T, int n_split, int n_cu, float *part, void *y, int y_bf16, hipStream_t s,
                                 const uint16_t *zero_row)
{
    float *parts = n_split > 1 ? part : nullptr;
    hipError_t e = hipSuccess;
    if (zero_row && d % kDgBN == 0 && ldh % kDgBK == 0) {
        int split = 1;
#define POP_DD(MF) \
    case MF: e = launch_dd<MF>(w, d, list, n_list, hc, ldh, T, n_split, parts, y, y_bf16, s, zero_row); break;
        switch (dd_shape(T, d, n_cu, &split)) {
            POP_DD(5) POP_DD(4) POP_DD(3) POP_DD(2) POP_DD(1)
            default: return hipErrorInvalidValue;
        }
#undef POP_DD
        if (e != hipSuccess) return e;
    } else {
        const int n_tt = (T + kDgBM - 1) / kDgBM, n_nt = (d + kDgBN - 1) / kDgBN;
        const int per_xcd = (n_tt * n_nt * n_split + 7) / 8;
        const size_t lds = (size_t)2 * (kDgBM * kDgLdA + kDgBK * kDgLdB) * sizeof(uint16_t);
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&down_gemm_bf16_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(down_gemm_bf16_kernel, dim3(per_xcd * 8), dim3(512), lds, s, (const uint16_t *)w, d, list,
                           n_list, hc, ldh, T, n_tt, n_nt, n_split, per_xcd, parts, y, y_bf16);
    }
    e = hipGetLastError();
    return e != hipSuccess ? e : down_gemm_reduce(part, n_split, T, d, y, y_bf16, s);
}

}  // namespace pop
