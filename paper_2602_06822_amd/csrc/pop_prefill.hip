// Prefill: gate/up contraction over all m channels and all T prompt tokens, fused with the column-wise
// importance reduction  s2[j] = sum_t H[t][j]^2  (Sec. 3.3 "Prefilling Stage"; Eq. 3: activation norm over
// tokens and samples).  In its plain form H is never written to memory.
//
// bf16: matrix-core tiles.  Rows that are whole k-steps long (d a multiple of 64) run prefill_mma_kernel, described
// there; other row lengths are staged through registers (prefill_bf16_kernel): a workgroup owns BM tokens (256 with 8
// waves, 4 along the tokens x 2 along the B rows; 128 with 4 waves for short prompts) and a chunk of up to 96 channels,
// i.e. up to 192 rows of the B operand (gate and up rows of the channel-major blocks w[j] = [gate row | up row | down
// column]); a wave owns 64 tokens x 48 channels = 96 B rows.  The 96 B rows of a wave are three fragments of 32x32x16
// products: gate of its channels 0..31, up of the same channels (same lane and register slot in the two accumulators,
// so silu(g)*u needs no exchange), and a mixed fragment [gate 32..47 | up 32..47] whose halves meet through one
// cross-lane move in the epilogue.  A second tile form drops the mixed fragment (64 channels per chunk, 64 B rows per
// wave).  The chunk size is chosen so that the tiles divide evenly over the compute units (one or a whole number of
// tiles each).  Either way an accumulator lane holds several token rows of one channel column, so the token reduction
// is in-register adds, cross-lane adds and an LDS combine of the token waves.  Token tiles write separate partial rows
// that are summed in tile order.
// Two more forms of the same kernels serve the forward pass of a whole prompt under the pruning structure
// (Sec. 3.4): one also writes H (rounded to bf16) as [T][m]; one runs its chunks over a device-resident list of
// active channels instead of all m and writes H (optionally times a per-token mask) in compact form
// [T][list position] for the down projection instead of reducing its squares.
// float32: FP64 matrix-core tiles (gateup_f32_kernel), described there.
#include <stdlib.h>

#include <type_traits>

#include "pop_internal.h"

namespace pop {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kPfBMmin = 64;      // smallest token tile (sizes the partial-row buffer)
constexpr int kPfChunk = 96;      // channels per workgroup tile at most
constexpr int kPfBK = 64;         // k elements per stage
constexpr int kPfLd = kPfBK + 8;  // padded LDS row stride in elements (144 B): conflict-free 16-byte reads

constexpr int kPf32BM = 16;       // smallest token tile of the float32 form

int prefill_num_tiles(int T, int is_bf16)
{
    return is_bf16 ? (T + kPfBMmin - 1) / kPfBMmin : (T + kPf32BM - 1) / kPf32BM;
}

// Workgroups are dealt round-robin to the 8 XCDs; renumber so that consecutive logical tiles (the token tiles
// of one channel chunk, which share the weight rows) land on the same XCD and meet in its L2.
__device__ __forceinline__ int xcd_logical_block(int bid, int per_xcd) { return (bid % 8) * per_xcd + bid / 8; }

// Channel (relative to the chunk) and matrix (0 gate, 1 up) of B row r of the workgroup tile.  A wave owns NF
// fragments of 32 rows: gate and up of its channels 0..31 and, with NF = 3, the mixed fragment of channels 32..47.
template <int NF>
__device__ __forceinline__ void pf_row_channel(int r, int &ch, int &which)
{
    const int half = r / (NF * 32), rr = r % (NF * 32);
    if (rr < 64) {
        ch = half * (NF * 16) + rr % 32;
        which = rr / 32;
    } else {
        ch = half * 48 + 32 + rr % 16;
        which = (rr - 64) / 16;
    }
}

// Tile geometry: channel chunks of at most 96 channels (three fragments per wave) or at most 64 (two fragments), as
// many as make the tiles a whole number per compute unit; of the two forms the one that is cheaper on the busiest
// compute unit.  The kernel is bound by its LDS fragment reads, so a tile's cost is taken as the reads per k-slice
// of a wave: 2 token fragments + the B fragments (measured: a two-fragment tile takes 0.8 of a three-fragment one).
// Host and device share this because the list form learns its channel count on the device.
struct PfGeom {
    int chunk, n_ct, total, per_xcd, nf;
};
__host__ __device__ inline PfGeom prefill_geometry_nf(int n_ch, int n_tt, int n_cu, int nf)
{
    PfGeom g;
    g.nf = nf;
    const int cap = nf * 32;
    const int min_ct = (n_ch + cap - 1) / cap;
    const int per_cu = (min_ct * n_tt + n_cu - 1) / n_cu;
    int n_ct = per_cu * n_cu / n_tt;
    if (n_ct < min_ct) n_ct = min_ct;
    if (n_ct > n_ch) n_ct = n_ch;
    g.chunk = (n_ch + n_ct - 1) / n_ct;
    g.n_ct = (n_ch + g.chunk - 1) / g.chunk;
    g.total = n_tt * g.n_ct;
    g.per_xcd = (g.total + 7) / 8;
    return g;
}
__host__ __device__ inline PfGeom prefill_geometry(int n_ch, int n_tt, int n_cu)
{
    if (n_ch <= 0) return PfGeom{1, 0, 0, 0, 3};
    const PfGeom g3 = prefill_geometry_nf(n_ch, n_tt, n_cu, 3), g2 = prefill_geometry_nf(n_ch, n_tt, n_cu, 2);
    const int cost3 = (g3.total + n_cu - 1) / n_cu * 5, cost2 = (g2.total + n_cu - 1) / n_cu * 4;
    return cost2 < cost3 ? g2 : g3;
}

// silu(g) * u for the tile epilogue (96 values per lane, with no other tile to hide behind): hardware exp2 and
// reciprocal, each good to one unit in the last place, instead of the library exponential and the exact quotient
// (a fifth of the instructions).  g -> -inf gives g * 0, g -> +inf gives g * 1.
__device__ __forceinline__ float silu_mul_tile(float g, float u)
{
    const float e = __builtin_amdgcn_exp2f(g * -1.44269504088896341f);
    return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

// What the list form adds to the plain prefill arguments.
struct PfStore {
    const int *list;            // active channels, ascending
    const int *n_list;          // their number (device)
    uint16_t *hc;               // [T][ldh] bf16: H of list position c in column c
    int ldh;
    const unsigned char *tmask; // per-token masks [T][m], or null
    int n_cu;
    float *h32 = nullptr;       // [T][m] float32, by channel (precise modes)
    // scores formed in the same launch (modes 0 and 2; null = leave that to the caller): the token tile of a
    // channel chunk that finishes last sums the chunk's partial rows
    int *fin_ctr = nullptr;     // one arrival counter per channel chunk; zero between launches
    const float *nrm = nullptr; // [m]
    float *scores = nullptr;    // [m]
};

// The tile's partial row from its waves' column sums and, where asked for, the chunk's scores.
template <int TW>
__device__ __forceinline__ void pf_chunk_scores(const float (&colsum)[TW][kPfChunk], int m, int n_ttiles, int ttile,
                                                int ctile, int c0, int cn, float *__restrict__ s2_part, const PfStore &st)
{
    const int tid = threadIdx.x;
    __syncthreads();
    if (tid < cn) {
        float tot = 0.f;
#pragma unroll
        for (int q = 0; q < TW; ++q) tot += colsum[q][tid];
        if (st.fin_ctr && n_ttiles == 1)  // (no other tile to wait for)
            st.scores[c0 + tid] = (float)((double)st.nrm[c0 + tid] * sqrt((double)tot));
        else if (st.fin_ctr)
            coherent_store(&s2_part[(size_t)ttile * m + c0 + tid], tot);
        else
            s2_part[(size_t)ttile * m + c0 + tid] = tot;
    }
    if (st.fin_ctr && n_ttiles > 1) {
        // Scores of this chunk's channels (Eq. 3): I_j = n_j * sqrt(sum over the token tiles, in tile order and in
        // double, of the partial sums).  The partial rows are written through and read with device-coherent loads;
        // a tile counts itself in once its own row has been acknowledged, and the tile that completes the count does
        // the sum and puts the counter back to zero for the next launch.  Nobody waits for anybody.
        __shared__ int fin_last;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            const bool last = atomicAdd(&st.fin_ctr[ctile], 1) == n_ttiles - 1;
            if (last) coherent_store(&st.fin_ctr[ctile], 0);
            fin_last = last;
        }
        __syncthreads();
        if (fin_last && tid < cn) {
            double acc = 0.0;
            for (int t = 0; t < n_ttiles; ++t) acc += (double)coherent_load(&s2_part[(size_t)t * m + c0 + tid]);
            st.scores[c0 + tid] = (float)((double)st.nrm[c0 + tid] * sqrt(acc));
        }
    }
}

// kMode 0: scores only (s2_part).  1: channels from st.list, H stored compact (no s2_part).  2: all m channels,
// s2_part and H stored as [T][m padded].  Of the direct-load kernel also 3 and 4, for prompts too short for H in bf16: all
// channels with s2_part, or those of st.list without, sums in double and H in float32 by channel; and 5, as 2 with H by channel,
// [m][ldh] with ldh >= T tokens a multiple of 64: rows that the down projection reads by the list of active channels.
template <int BM, int NW, int NF, int kMode>
__global__ __launch_bounds__(NW * 64) void prefill_bf16_kernel(const uint16_t *__restrict__ w,
                                                           const uint16_t *__restrict__ x, int T, int d, int m,
                                                           int n_ttiles, int chunk, int n_items, int per_xcd,
                                                           float *__restrict__ s2_part, PfStore st)
{
    constexpr int TW = NW / 2;          // waves along the tokens (2 along the B rows)
    constexpr int MT = BM / (32 * TW);  // 32-token fragments per wave
    constexpr int RP = NW * 8;          // rows one staging pass of the workgroup covers
    constexpr int BR = NF * 64;         // B rows of the workgroup tile
    constexpr int WC = NF * 16;         // channels per wave
    constexpr int LD = kPfLd;           // LDS rows: 64 elements padded to 72
    extern __shared__ __attribute__((aligned(16))) uint16_t pf_lds[];
    uint16_t *As = pf_lds;                    // [2][BM * LD]
    uint16_t *Bs = pf_lds + 2 * BM * LD;      // [2][BR * LD]
    __shared__ float colsum[TW][kPfChunk];

    constexpr bool kList = kMode == 1, kStore = kMode != 0;
    int n_ch = m;  // channels the chunks run over
    if (kList) {
        n_ch = *st.n_list;
        const PfGeom g = prefill_geometry(n_ch, n_ttiles, st.n_cu);
        if (g.nf != NF) return;  // the other instantiation runs this list length
        chunk = g.chunk, n_items = g.total, per_xcd = g.per_xcd;
        if ((int)blockIdx.x >= per_xcd * 8) return;  // the grid was sized for the longest list
    }
    const int logical = xcd_logical_block(blockIdx.x, per_xcd);
    if (logical >= n_items) return;
    const int ctile = logical / n_ttiles, ttile = logical % n_ttiles;
    const int t0 = ttile * BM, c0 = ctile * chunk;
    const int cn = min(chunk, n_ch - c0);  // channels in this chunk

    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int wm = wave / 2, wn = wave % 2;  // wave tile: tokens wm*BM/TW.., B rows wn*NF*32..

    // global -> LDS staging: 8 vectors of 16 bytes per 64-element row; the workgroup covers RP rows per pass
    const int ld_row = tid / 8, ld_kv = tid % 8;
    constexpr int PA = BM / RP, PB = BR / RP;
    static_assert(BM % RP == 0 && BR % RP == 0, "whole staging passes");
    uint4 ra[PA], rb[PB];
    // row starts; null for a row of zeros (tokens beyond T, channels beyond the chunk)
    const uint16_t *pa[PA], *pb[PB];
#pragma unroll
    for (int p = 0; p < PA; ++p) {
        const int t = t0 + ld_row + p * RP;
        pa[p] = t < T ? x + (size_t)t * d : nullptr;
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        int ch, which;
        pf_row_channel<NF>(ld_row + p * RP, ch, which);
        pb[p] = nullptr;
        if (ch < cn) {
            const int j = kList ? st.list[c0 + ch] : c0 + ch;
            pb[p] = w + (size_t)j * channel_elems_bf16(d) + which * d;
        }
    }
    auto load_global = [&](int k0) {
        const int k = k0 + ld_kv * 8;
        const bool k_ok = k < d;
#pragma unroll
        for (int p = 0; p < PA; ++p)
            ra[p] = (k_ok && pa[p]) ? *reinterpret_cast<const uint4 *>(pa[p] + k) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int p = 0; p < PB; ++p)
            rb[p] = (k_ok && pb[p]) ? *reinterpret_cast<const uint4 *>(pb[p] + k) : make_uint4(0, 0, 0, 0);
    };
    auto store_lds = [&](int buf) {
#pragma unroll
        for (int p = 0; p < PA; ++p)
            *reinterpret_cast<uint4 *>(&As[(buf * BM + ld_row + p * RP) * LD + ld_kv * 8]) = ra[p];
#pragma unroll
        for (int p = 0; p < PB; ++p)
            *reinterpret_cast<uint4 *>(&Bs[(buf * BR + ld_row + p * RP) * LD + ld_kv * 8]) = rb[p];
    };
    f32x16_t acc[MT][NF];  // [token fragment][0 = gate 0..31, 1 = up 0..31, 2 = gate 32..47 | up 32..47]
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][f][v] = 0.f;

    const int n_k = (d + kPfBK - 1) / kPfBK;
    const int arow = wm * (BM / TW) + (lane % 32), brow = wn * (NF * 32) + (lane % 32), koff = (lane / 32) * 8;
    auto multiply = [&](int buf) {
        const uint16_t *Ab = As + (buf * BM + arow) * LD + koff;
        const uint16_t *Bb = Bs + (buf * BR + brow) * LD + koff;
        // the fragments of k-slice q + 1 are requested before the products of slice q are issued (two register
        // sets), so that their LDS latency runs under the matrix pipe
        bf16x8_t bf[2][NF], af[2][MT];
        auto fetch = [&](int q, int set) {
#pragma unroll
            for (int f = 0; f < NF; ++f) bf[set][f] = *reinterpret_cast<const bf16x8_t *>(Bb + f * 32 * LD + q * 16);
#pragma unroll
            for (int a = 0; a < MT; ++a) af[set][a] = *reinterpret_cast<const bf16x8_t *>(Ab + a * 32 * LD + q * 16);
        };
        fetch(0, 0);
#pragma unroll
        for (int q = 0; q < kPfBK / 16; ++q) {
            if (q + 1 < kPfBK / 16) fetch(q + 1, (q + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    acc[a][f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[q & 1][a], bf[q & 1][f], acc[a][f], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // step ks multiplies LDS buffer ks % 2 while the rows of step ks + 1 are on their way through registers
    load_global(0);
    store_lds(0);
    __syncthreads();
    for (int ks = 0; ks < n_k; ++ks) {
        const int buf = ks & 1;
        if (ks + 1 < n_k) load_global((ks + 1) * kPfBK);
        multiply(buf);
        if (ks + 1 < n_k) store_lds(buf ^ 1);
        __syncthreads();
    }

    // epilogue: lane holds 16 * MT token rows of column (lane % 32) of each fragment; rows of padded tokens and columns
    // of padded channels are exactly 0
    // H of the tile (modes 1 and 2), written after the partial sums have gone out: the tile's arrival is counted once
    // its partial row is acknowledged, and that wait should not take in the much larger H.
    auto store_h = [&]() {
        // register v of a fragment is token row (v / 4) * 8 + (lane / 32) * 4 + v % 4, column lane % 32
        const int col = lane % 32;
        const int c01 = wn * WC + col, c2 = wn * WC + 32 + col;
        const bool ok01 = c01 < cn, ok2 = NF == 3 && col < 16 && c2 < cn;
        const int j01 = (kList && st.tmask && ok01) ? st.list[c0 + c01] : 0;
        const int j2 = (kList && st.tmask && ok2) ? st.list[c0 + c2] : 0;
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = t0 + wm * (BM / TW) + a * 32 + (v / 4) * 8 + (lane / 32) * 4 + v % 4;
                float h01 = silu_mul_tile(acc[a][0][v], acc[a][1][v]);
                float h2 = 0.f;
                if (NF == 3) {
                    const float g2 = acc[a][NF - 1][v];
                    const float u2 = __shfl_xor(g2, 16, kWave);
                    h2 = silu_mul_tile(g2, u2);
                }
                if (t < T) {
                    uint16_t *row = st.hc + (size_t)t * st.ldh + c0;
                    if (ok01) {
                        if (kList && st.tmask && !st.tmask[(size_t)t * m + j01]) h01 = 0.f;
                        row[c01] = f32_to_bf16(h01);
                    }
                    if (ok2) {
                        if (kList && st.tmask && !st.tmask[(size_t)t * m + j2]) h2 = 0.f;
                        row[c2] = f32_to_bf16(h2);
                    }
                }
            }
    };
    if (kList) {
        store_h();
        return;
    }
    float ss01 = 0.f, ss2 = 0.f;
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float hv = silu_mul_tile(acc[a][0][v], acc[a][1][v]);
            ss01 = fmaf(hv, hv, ss01);
            if (NF == 3) {
                // mixed fragment: the up value of column c < 16 sits in lane c + 16, same register
                const float g2 = acc[a][NF - 1][v];
                const float u2 = __shfl_xor(g2, 16, kWave);
                const float h2 = silu_mul_tile(g2, u2);
                ss2 = fmaf(h2, h2, ss2);
            }
        }
    ss01 += __shfl_xor(ss01, 32, kWave);
    ss2 += __shfl_xor(ss2, 32, kWave);
    if (lane < 32) colsum[wm][wn * WC + lane] = ss01;
    if (NF == 3 && lane < 16) colsum[wm][wn * WC + 32 + lane] = ss2;
    pf_chunk_scores<TW>(colsum, m, n_ttiles, ttile, ctile, c0, cn, s2_part, st);
    if (kStore) store_h();
}

// ---- rows that are whole k-steps long (d a multiple of 64): the direct-load kernel
//
// A tile is 64 MF tokens x 8 F channels (16 F rows of the B operand); four waves, 16 MF tokens each.  F comes from a
// short ladder and MF is 1..5, so that ragged prompts and channel counts waste little: a tile's last rows are padding.
constexpr int kPmThreads = 256;
constexpr int kPmMaxMF = 5;
constexpr int kPmMaxF = 12;
// LDS ring depths (k-steps of 64 elements): token rows, which mostly come from L2, and weight rows, which come from
// memory; as deep as 160 KB allow with F = 12.
template <int MF>
struct PmRing {
    static constexpr int NA = MF >= 4 ? 2 : (MF >= 2 ? 3 : 4);
    static constexpr int NB = MF >= 3 ? 3 : (MF == 2 ? 4 : 5);
    static constexpr size_t kBytes = (size_t)(NA * 64 * MF + NB * 16 * kPmMaxF) * kPfBK * sizeof(uint16_t);
};
// Narrow chunks of four token fragments (F up to kPmDeepF): their weight rows leave room for a third step of token rows.  A wave's
// requests return in order, so with two steps of token rows every wait for the next one is also a wait for all but
// the youngest step of weight rows, however many their ring holds; with three both have a step longer.  d 4096, m 14336, F 7, with
// weights from memory: 256 tokens 80.4 -> 72.9 us (from the last-level cache 58.8 -> 55.1), 512 tokens at the 13B shape 145 ->
// 139.5.  Wider chunks: no room; five fragments leave none for token rows at any width that is used.
constexpr int kPmDeepMF = 4, kPmDeepF = 8;
struct PmDeepRing {
    static constexpr int NA = 3, NB = 3;
    static constexpr size_t kBytes = (size_t)(NA * 64 * kPmDeepMF + NB * 16 * kPmDeepF) * kPfBK * sizeof(uint16_t);
};

// Channel (relative to the chunk) and matrix (0 gate, 1 up) of B row r: fragments of 16 rows go in pairs, the gate rows
// of 16 channels and the up rows of the same; an odd last fragment is [gate of 8 channels | up of the same 8].
template <int F>
__device__ __forceinline__ void pm_row_channel(int r, int &ch, int &which)
{
    const int f = r / 16, c = r % 16;
    if (F % 2 && f >= F - 1) {
        ch = 8 * (F - 1) + c % 8, which = c / 8;
    } else {
        ch = f / 2 * 16 + c, which = f % 2;
    }
}

// Tiles of one launch: F and the counts that follow.  Shared by host and device (the list form learns its channel
// count on the device).  Every width of the ladder is a code path of each kernel; without 9 and 5 a chunk is at most a
// ninth or a fifth wider than the best one.
struct PmTiles {
    int f, n_ct, total, per_xcd;
};
// Relative time of a tile on its compute unit, per 32 elements of the contraction, in cycles: its products (16 cycles
// each on one matrix pipe) and the LDS and L2 traffic next to them, or the memory time of its weight rows where few
// token tiles share them.
__host__ __device__ inline int pm_tile_cost(int mf, int f, int n_tt)
{
    const int work = 16 * mf * f + 8 * (4 * mf + f) + 60, mem = 100 * f / n_tt;
    return work > mem ? work : mem;
}
__host__ __device__ inline PmTiles pm_tiles(int n_ch, int n_tt, int mf, int n_cu, int *cost = nullptr)
{
    PmTiles best{kPmMaxF, 0, 0, 0};
    int best_cost = 0;
    const int ladder[7] = {12, 11, 10, 8, 7, 6, 4};
    for (int i = 0; i < 7; ++i) {
        const int f = ladder[i], n_ct = (n_ch + 8 * f - 1) / (8 * f), total = n_ct * n_tt;
        const int c = (total + n_cu - 1) / n_cu * pm_tile_cost(mf, f, n_tt);
        if (i == 0 || c < best_cost) best_cost = c, best = PmTiles{f, n_ct, total, (total + 7) / 8};
    }
    if (cost) *cost = best_cost;
    return best;
}

// Bound by the LDS, the matrix pipe and the chip's power together.  Direct loads of lines that the L2 holds deliver 58 bytes a cycle and
// compute unit (135 bytes/ns, nothing else running, any depth from 8 loads a wave on), but fragment reads, 128 bytes a cycle, do not overlap with
// them: 48 KB of loads take 850 cycles, with 96 KB of reads 1430, with 120 KB 1750.  So the 54 KB and 120 KB of a k-step at MF = 4, F = 11 are about
// 1850 cycles of the LDS next to 1390 of products, of the 2040 it takes (512 tokens: pipe busy for 61-68 % of the waves' time), and with the pipe that busy
// the clock falls to about 2.0 GHz: without its products the launch takes 51 instead of 77 us, 2048 tokens 231 instead of 309.  An expert's
// 256 tokens (F 7) leave the pipe idle for two thirds of the time, the clock near 2.4 GHz, and take as long without products (71
// of 72 us: weights from memory).  So what counts is work per byte loaded and per product: 16x16x32 products move fewer accumulator bytes per flop than 32x32x16 ones (7 % faster here at
// equal cycles), a wave keeps all 16 F rows against its 16 MF tokens (MF + F fragment reads of 1 KB for MF * F products
// of 16 cycles), and F follows the channel count in eights instead of padding it to 96.  Token rows straight into
// registers instead (a wave is the only reader of its own) were bit-identical and a third slower (512 tokens 75 -> 100
// us): a fragment's load touches 16 lines per 16 lanes, a direct load two.
// One wave per SIMD has nobody to hide behind, so the stream is pipelined by hand: while the products of one 32-element
// slice issue, the fragments of the next are read, and direct loads go out a few products apart (bunched together they
// hold up the wave's issue).  A k-step is two slices: the first carries the requests for weight rows, then this wave's
// reads of the step's buffers are over (the second slice's fragments are in registers), the barrier makes the next
// step's rows visible, and the second slice carries the requests for token rows and the reads of the next step's first
// slice.
// Operand rows go straight from global memory into LDS (global_load_lds: 1 KB = 8 unpadded 128-byte rows per wave
// instruction, the 16-byte units of row r stored at unit ^ ((r / 2) % 8): conflict-free fragment reads).  Every wave
// issues the same loads in every k-step (rows beyond T or beyond the chunk are pointed at a row that exists, steps
// beyond the last at the last step), so each wait counts exactly.
// Measured, d 4096, m 11008 (before: eight waves of 64 tokens x 96 rows, 32x32x16 products, reads and products of all
// waves in lockstep): 512 tokens 102 -> 80 us (1.16 PFLOP/s), 2048 tokens 380 -> 292 us (1.26), 256 tokens 54 us.
template <int MF, int F, int kMode, class Ring, bool kStream>
__device__ __forceinline__ void pm_tile(const uint16_t *__restrict__ w, const uint16_t *__restrict__ x, int T, int d,
                                        int m, int n_ch, int n_tt, int logical, float *__restrict__ s2_part,
                                        const PfStore &st, uint16_t *lds, float (&colsum)[4][kPfChunk])
{
    typedef __attribute__((address_space(3))) void lds_t;
    typedef __attribute__((address_space(1))) const void glb_t;
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    constexpr int NA = Ring::NA, NB = Ring::NB;
    constexpr bool kList = kMode == 1 || kMode == 4, kPrecise = kMode == 3 || kMode == 4, kRows = kMode == 5;
    // An odd F leaves 16 rows for the last pass: half a request of each wave (without: two waves' whole ones, and the other two ask for
    // rows again that are there, 2 KB of the 48 to 56 of a k-step.  With: eight experts 1015 -> 1005 us; 512 and 24 tokens the same).  Not in the
    // kernels with ordinary loads that store no H by channel: twelve partitions and FFNs with F of 7 and 11 between 1 % faster and 1 % slower.
    constexpr bool kHalf = (kStream || kRows) && F % 2;
    constexpr int BM = 64 * MF, BC = 8 * F;             // tokens and channels of the tile
    constexpr int PA = BM / 32, PB = (F + 1) / 2;       // direct loads per wave and k-step (32 rows a pass)
    constexpr int AT = BM * kPfBK, BT = PB * 32 * kPfBK;  // elements of one buffer
    uint16_t *As = lds;            // [NA][BM * 64]
    uint16_t *Bs = lds + NA * AT;  // [NB][PB * 32 * 64]

    const int ctile = logical / n_tt, ttile = logical % n_tt;
    const int t0 = ttile * BM, c0 = ctile * BC, cn = min(BC, n_ch - c0);
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);

    // direct loads: this lane's 16 bytes land at LDS unit lane % 8 of row ld_row of the pass, so it fetches the
    // k-vector that belongs there under the swizzle (passes are 32 rows apart: same swizzle term)
    const int ld_row = tid / 8, src_kv = ((tid % 8) ^ ((ld_row / 2) % 8)) * 8;
    const uint16_t *pa[PA], *pb[PB];
#pragma unroll
    for (int p = 0; p < PA; ++p) pa[p] = x + (size_t)min(t0 + ld_row + p * 32, T - 1) * d + src_kv;
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        int ch, which;
        const bool half = kHalf && p == PB - 1;
        const int row = p * 32 + (half ? wave * 4 + lane / 8 : ld_row);
        pm_row_channel<F>(row, ch, which);
        const int cc = min(ch, cn - 1);
        const int j = kList ? st.list[c0 + cc] : c0 + cc;
        pb[p] = w + (size_t)j * channel_elems_bf16(d) + which * d + (half ? ((lane % 8) ^ ((row / 2) % 8)) * 8 : src_kv);
    }
    const int n_k = d / kPfBK;
    // k-step s is columns kof(s) (steps beyond the last repeat it).  Sums in float32 take the columns in the same order in
    // every tile: a sum must not depend on its channel's place, or channels with equal weights would not tie.  Rows are a
    // power of two apart in most models, and tiles in step with each other keep asking the same few memory channels.  So
    // the sums in double, where the order is lost in the rounding to float32, start at a column of their own per chunk (24
    // tokens, d 4096, m 11008: whole call 83 -> 73 us); in one tile of float32 sums it gained as much (270 tokens, m 14336: 98
    // -> 80 us).
    const int rot = kPrecise ? ctile % n_k : 0;
    auto kof = [&](int step) {
        const int q = min(step, n_k - 1) + rot;
        return (q >= n_k ? q - n_k : q) * kPfBK;
    };
    auto load_a = [&](int p, int buf, int k0) {
        __builtin_amdgcn_global_load_lds((glb_t *)(pa[p] + k0), (lds_t *)(As + buf * AT + (p * 32 + wave * 8) * kPfBK), 16,
                                         0, 0);
    };
    auto load_b = [&](int p, int buf, int k0) {
        if (kHalf && p == PB - 1) {
            // (32 lanes; inline assembly, for there may be no branch around a load.  It leaves m0 and exec as they were.)
            const int to = __builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)(Bs + buf * BT + (p * 32 + wave * 4) * kPfBK));
            int m0_was;
            if constexpr (kStream)
                asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_mov_b32 exec_hi, 0\n\tglobal_load_lds_dwordx4 %2, off nt\n\t"
                             "s_mov_b32 exec_hi, -1\n\ts_mov_b32 m0, %0" : "=&s"(m0_was) : "s"(to), "v"(pb[p] + k0));
            else
                asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_mov_b32 exec_hi, 0\n\tglobal_load_lds_dwordx4 %2, off\n\t"
                             "s_mov_b32 exec_hi, -1\n\ts_mov_b32 m0, %0" : "=&s"(m0_was) : "s"(to), "v"(pb[p] + k0));
            return;
        }
        __builtin_amdgcn_global_load_lds((glb_t *)(pb[p] + k0), (lds_t *)(Bs + buf * BT + (p * 32 + wave * 8) * kPfBK), 16,
                                         0, kStream ? 2 : 0);  // (2: non-temporal)
    };

    f32x4_t acc[MF][F];
#pragma unroll
    for (int a = 0; a < MF; ++a)
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[a][f][v] = 0.f;

    // fragment reads: row lane % 16 of the fragment, unit 4 q + lane / 16 under the row's swizzle (fragments are 16 rows
    // apart: same term); the order is the one their products need
    int koff[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) koff[q] = ((q * 4 + lane / 16) ^ ((lane % 16) / 2)) * 8;
    const uint16_t *Al = As + (wave * MF * 16 + lane % 16) * kPfBK, *Bl = Bs + (lane % 16) * kPfBK;
    bf16x8_t af[2][MF], bf[2][F];
    auto fetch = [&](const uint16_t *Ab, const uint16_t *Bb, int i, int q, int set) {
        if (i == 0)
            af[set][0] = *reinterpret_cast<const bf16x8_t *>(Ab + koff[q]);
        else if (i <= F)
            bf[set][i - 1] = *reinterpret_cast<const bf16x8_t *>(Bb + (i - 1) * 16 * kPfBK + koff[q]);
        else
            af[set][i - F] = *reinterpret_cast<const bf16x8_t *>(Ab + (i - F) * 16 * kPfBK + koff[q]);
    };
    // (inline assembly ties the accumulator to itself: left to choose, the compiler gives products of this size other
    // destinations and copies them back, which costs more than the products)
    // Precise modes: a k-step's two products run from zero and their sums are added up in double, one step later.
    double sum[kPrecise ? MF : 1][kPrecise ? F : 1][4] = {};
    auto product = [&](int i, int set) {
        if constexpr (kPrecise) {
            const f32x4_t from = set == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : acc[i / F][i % F];
            acc[i / F][i % F] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[set][i / F], bf[set][i % F], from, 0, 0, 0);
        } else {
            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                         : "+a"(acc[i / F][i % F])
                         : "v"(af[set][i / F]), "v"(bf[set][i % F]));
        }
    };
    auto add_up = [&]() {
        if constexpr (kPrecise) {
#pragma unroll
            for (int i = 0; i < MF * F; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) sum[i / F][i % F][v] += (double)acc[i / F][i % F][v];
        }
    };

    // Requests in program order: ... A(s + NA - 1) | B(s + NB - 1) [wait for step s + 1] A(s + NA) | B(s + NB) [...: the
    // wait may leave in flight what was issued after both A(s + 1) and B(s + 1).
    constexpr int kAfterA = (NA - 1) * PB + (NA - 2) * PA, kAfterB = (NB - 2) * (PA + PB);
    constexpr int kYounger = kAfterA < kAfterB ? kAfterA : kAfterB;
    static_assert(kYounger + PA < 64, "vmcnt is a 6-bit counter");
    constexpr int kFirst = NA > NB - 1 ? NA : NB - 1;
#pragma unroll
    for (int j = -kFirst; j < 0; ++j) {  // what steps j < 0 would have requested
        if (j - 1 + NB >= 0) {
#pragma unroll
            for (int p = 0; p < PB; ++p) load_b(p, j - 1 + NB, kof(j - 1 + NB));
        }
        if (j + NA >= 0) {
#pragma unroll
            for (int p = 0; p < PA; ++p) load_a(p, j + NA, kof(j + NA));
        }
    }
    // the wait "before step 0", with the token rows requested behind it in flight as well
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kYounger + PA) : "memory");
    constexpr int NP = MF * F, NR = MF + F;    // products and fragment reads of a slice
    constexpr int kSpread = NP > 8 ? NP * 3 / 4 : NP;  // products the reads are spread over: the last have time to arrive
#pragma unroll
    for (int i = 0; i < NR; ++i) fetch(Al, Bl, i, 0, 0);
    int abuf = 0, bbuf = 0, bprev = NB - 1;
    for (int ks = 0; ks < n_k; ++ks) {
        const uint16_t *Ab = Al + abuf * AT, *Bb = Bl + bbuf * BT;
        const int kb = kof(ks + NB - 1), ka = kof(ks + NA);
        add_up();  // (the step before; zeroes first)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            product(i, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = min(i, kSpread) * NR / kSpread; r < min(i + 1, kSpread) * NR / kSpread; ++r) fetch(Ab, Bb, r, 1, 1);
#pragma unroll
            for (int p = i * PB / NP; p < (i + 1) * PB / NP; ++p) load_b(p, bprev, kb);
            __builtin_amdgcn_sched_barrier(0);
        }
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
            for (int p = i * PA / NP; p < (i + 1) * PA / NP; ++p) load_a(p, a_free, ka);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // the surplus requests, before the LDS is used for something else; the products' results before they are read (the
    // compiler does not see the products, so it adds no wait states for them)
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __syncthreads();
    if constexpr (!kPrecise) {
#pragma unroll
        for (int i = 0; i < MF * F; ++i) asm volatile("" : "+a"(acc[i / F][i % F]));  // (no read of them moves ahead of the wait)
    }
    if constexpr (kPrecise) {
        add_up();
#pragma unroll
        for (int i = 0; i < MF * F; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i / F][i % F][v] = (float)sum[i / F][i % F][v];
    }

    // Accumulator register v of a lane: token 4 (lane / 16) + v of the fragment, B row lane % 16 of the fragment.  An odd
    // last fragment holds gate values in lanes 0..7 of each 16 and up values of the same channels in lanes 8..15: the
    // halves trade two registers each, so that every lane forms two of the four.
    uint16_t *hs = lds;                 // [BM][BC + 8], by channel [BC][BM + 8] bf16: H of the tile on its way out
    constexpr int HS = kRows ? BM + 8 : BC + 8;
    const int col = lane % 16, row0 = wave * MF * 16 + lane / 16 * 4;  // first token row of this lane
    const bool upper = col >= 8;
    const int c_odd = 8 * (F - 1) + col % 8, r_odd = upper ? 2 : 0;
    // (a lane's squares are summed rows 0 and 1 of each fragment first, then rows 2 and 3, as the two lanes that share a
    // channel of the odd fragment do it: a channel's score does not depend on its place in the tile)
    float ss[(F + 1) / 2];
#pragma unroll
    for (int p = 0; p < F / 2; ++p) {
        const int c = 16 * p + col;
        const bool live_c = c < cn;
        const int j = (kList && (kPrecise || st.tmask) && live_c) ? st.list[c0 + c] : c0 + c;
        float sq[2] = {0.f, 0.f};
#pragma unroll
        for (int a = 0; a < MF; ++a) {
            uint32_t four[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = t0 + row0 + a * 16 + v;
                float h = kPrecise ? silu_mul(acc[a][2 * p][v], acc[a][2 * p + 1][v])
                                   : silu_mul_tile(acc[a][2 * p][v], acc[a][2 * p + 1][v]);
                h = (t < T && live_c) ? h : 0.f;  // (padding holds products of the rows its loads were pointed at)
                sq[v / 2] = fmaf(h, h, sq[v / 2]);
                if (kPrecise) {
                    if (t < T && live_c) st.h32[(size_t)t * m + j] = h;
                } else if (kRows) {
                    four[v] = f32_to_bf16(h);
                } else if (kMode != 0) {
                    if (kList && st.tmask && t < T && live_c && !st.tmask[(size_t)t * m + j]) h = 0.f;
                    hs[(row0 + a * 16 + v) * HS + c] = f32_to_bf16(h);
                }
            }
            if (kRows)
                *reinterpret_cast<uint2 *>(hs + c * HS + row0 + a * 16) = make_uint2(four[0] | four[1] << 16, four[2] | four[3] << 16);
        }
        ss[p] = sq[0] + sq[1];
    }
    if (F % 2) {
        const bool live_c = c_odd < cn;
        const int j = (kList && (kPrecise || st.tmask) && live_c) ? st.list[c0 + c_odd] : c0 + c_odd;
        ss[F / 2] = 0.f;
#pragma unroll
        for (int a = 0; a < MF; ++a) {
            uint32_t two[2];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const float mine = upper ? acc[a][F - 1][v + 2] : acc[a][F - 1][v];
                const float give = upper ? acc[a][F - 1][v] : acc[a][F - 1][v + 2];
                const float got = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x128, 0xf, 0xf, true));  // row_ror:8
                const int t = t0 + row0 + a * 16 + r_odd + v;
                const float gate = upper ? got : mine, up = upper ? mine : got;
                float h = kPrecise ? silu_mul(gate, up) : silu_mul_tile(gate, up);
                h = (t < T && live_c) ? h : 0.f;
                ss[F / 2] = fmaf(h, h, ss[F / 2]);
                if (kPrecise) {
                    if (t < T && live_c) st.h32[(size_t)t * m + j] = h;
                } else if (kRows) {
                    two[v] = f32_to_bf16(h);
                } else if (kMode != 0) {
                    if (kList && st.tmask && t < T && live_c && !st.tmask[(size_t)t * m + j]) h = 0.f;
                    hs[(row0 + a * 16 + r_odd + v) * HS + c_odd] = f32_to_bf16(h);
                }
            }
            if (kRows) *reinterpret_cast<uint32_t *>(hs + c_odd * HS + row0 + a * 16 + r_odd) = two[0] | two[1] << 16;
        }
    }
    if (!kList) {
#pragma unroll
        for (int p = 0; p < (F + 1) / 2; ++p) {
            float s = ss[p];
            if (p == F / 2) s += __shfl_xor(s, 8, kWave);
            s += __shfl_xor(s, 16, kWave);
            s += __shfl_xor(s, 32, kWave);
            if (lane < 16 && (p < F / 2 || lane < 8)) colsum[wave][16 * p + lane] = s;
        }
        pf_chunk_scores<4>(colsum, m, n_tt, ttile, ctile, c0, cn, s2_part, st);
    }
    if (kRows) {
        __syncthreads();
        for (int i = tid; i < BC * (BM / 8); i += kPmThreads) {
            const int c = i / (BM / 8), t = t0 + i % (BM / 8) * 8;
            if (c < cn && t < st.ldh)
                *reinterpret_cast<uint4 *>(st.hc + (size_t)(c0 + c) * st.ldh + t) =
                    *reinterpret_cast<const uint4 *>(hs + c * HS + i % (BM / 8) * 8);
        }
    }
    if (kMode == 1 || kMode == 2) {
        __syncthreads();
        for (int i = tid; i < BM * F; i += kPmThreads) {
            const int r = i / F, v = i % F;
            if (t0 + r < T && c0 + v * 8 < st.ldh)
                *reinterpret_cast<uint4 *>(st.hc + (size_t)(t0 + r) * st.ldh + c0 + v * 8) =
                    *reinterpret_cast<const uint4 *>(hs + r * HS + v * 8);
        }
    }
}

// One workgroup per compute unit; each walks its share of the tiles of its XCD (the token tiles of a channel chunk are
// neighbours there and meet in its L2).  prefill_stream_kernel: weight rows past the caches, for layers of stream_rows and up to
// two token tiles per chunk, which ask for a row at the same time (2048 tokens no change); with the narrow chunks' deeper ring where it is
// used.  512 tokens, d 4096, m 11008, in turn on one card: 87.8 -> 84.4 us.  Two tiles from 240 MB of weights on; three layers in turn, past
// the caches over ordinary, 128 and 256 tokens: partition, of 138 MB 1.08 and 1.04, of 157 MB 1.01, of 201 MB .96 and .97; forward pass .95-.98;
// but 200 tokens 1.15, 1.14, 1.02, of 226 MB 1.05, of 251 MB .98, and forward 1.02-1.05 up to 226 MB.  The second tile has to be seven eighths
// full, half on rows of up to 8 KB where a compute unit runs one tile: one with few tokens of its own has its other rows from the cache, runs
// ahead, the further the longer the rows, and what it asked for is gone when the first tile comes to it, a read of every row from memory by each.
// Partition, us of three or two layers, by how full the second tile is: 13B shape (two tiles a compute unit) .09 242 / 311, .33 278 / 306, .56 289 / 295,
// .80 298 / 294; d 8192, m 28672 .09 464 / 632; one tile a compute unit, 7B shape .09 157 / 168, .33 164 / 169, .56 182 / 171; d 6144, m 8192 .56 156 /
// 161, .75 161 / 161, .88 166 / 162; d 12288, m 6000 .56 218 / 255, .75 230 / 246, .88 235 / 237, 1.0 241 / 239.
// A list of channels: one token tile (two, 333 tokens at the 13B shape: 107.6 without / 108.3 with).
template <int MF, int kMode>
inline bool pm_streams(int d, int m, int T, bool one_each, long long stream_from)
{
    if (T <= 64 * MF) return stream_rows(d, m, 1, stream_from);
    if (kMode == 1 || kMode == 4 || T > 128 * MF || T < (one_each && d <= 4096 ? 96 : 120) * MF) return false;
    return stream_rows(d, m, 1, stream_from < kStreamTwiceBytes ? kStreamTwiceBytes : stream_from);
}
constexpr bool pm_deep(int mf, int f, int mode) { return mf == kPmDeepMF && f <= kPmDeepF && (mode == 0 || mode == 2 || mode == 5); }
template <int MF, int kMode, bool kStream>
__device__ __forceinline__ void pm_walk(const uint16_t *__restrict__ w, const uint16_t *__restrict__ x, int T, int d, int m,
                                        int n_tt, PmTiles g, float *__restrict__ s2_part, const PfStore &st)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t pf_lds[];
    __shared__ float colsum[4][kPfChunk];
    int n_ch = m;  // channels the chunks run over
    if (kMode == 1 || kMode == 4) {
        n_ch = *st.n_list;
        g = pm_tiles(n_ch, n_tt, MF, st.n_cu);
    }
    for (int i = blockIdx.x / 8; i < g.per_xcd; i += gridDim.x / 8) {
        const int logical = (blockIdx.x % 8) * g.per_xcd + i;
        if (logical >= g.total) break;
        switch (g.f) {
#define POP_PM(FF)                                                                                                         \
    case FF: {                                                                                                             \
        typedef typename std::conditional<pm_deep(MF, FF, kMode), PmDeepRing, PmRing<MF>>::type ring_t;                    \
        pm_tile<MF, FF, kMode, ring_t, kStream>(w, x, T, d, m, n_ch, n_tt, logical, s2_part, st, pf_lds, colsum);             \
        break;                                                                                                             \
    }
            POP_PM(12) POP_PM(11) POP_PM(10) POP_PM(8) POP_PM(7) POP_PM(6) POP_PM(4)
#undef POP_PM
        }
        __syncthreads();  // the next tile's direct loads overwrite the LDS
    }
}

template <int MF, int kMode>
__global__ __launch_bounds__(kPmThreads, 1) void prefill_stream_kernel(const uint16_t *__restrict__ w,
                                                                       const uint16_t *__restrict__ x, int T, int d, int m,
                                                                       int n_tt, PmTiles g, float *__restrict__ s2_part,
                                                                       PfStore st)
{
    pm_walk<MF, kMode, true>(w, x, T, d, m, n_tt, g, s2_part, st);
}

// H by channel (mode 5).
template <int MF, bool kStream>
__global__ __launch_bounds__(kPmThreads, 1) void prefill_rows_kernel(const uint16_t *__restrict__ w,
                                                                     const uint16_t *__restrict__ x, int T, int d, int m,
                                                                     int n_tt, PmTiles g, float *__restrict__ s2_part,
                                                                     PfStore st)
{
    pm_walk<MF, 5, kStream>(w, x, T, d, m, n_tt, g, s2_part, st);
}

template <int MF, int kMode>
__global__ __launch_bounds__(kPmThreads, 1) void prefill_mma_kernel(const uint16_t *__restrict__ w,
                                                                    const uint16_t *__restrict__ x, int T, int d, int m,
                                                                    int n_tt, PmTiles g, float *__restrict__ s2_part,
                                                                    PfStore st)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t pf_lds[];
    __shared__ float colsum[4][kPfChunk];
    int n_ch = m;  // channels the chunks run over
    if (kMode == 1 || kMode == 4) {
        n_ch = *st.n_list;
        g = pm_tiles(n_ch, n_tt, MF, st.n_cu);
    }
    for (int i = blockIdx.x / 8; i < g.per_xcd; i += gridDim.x / 8) {
        const int logical = (blockIdx.x % 8) * g.per_xcd + i;
        if (logical >= g.total) break;
        switch (g.f) {
#define POP_PM(FF)                                                                               \
    case FF:                                                                                                 \
        pm_tile<MF, FF, kMode, PmRing<MF>, false>(w, x, T, d, m, n_ch, n_tt, logical, s2_part, st, pf_lds, colsum); \
        break;
            POP_PM(12) POP_PM(11) POP_PM(10) POP_PM(8) POP_PM(7) POP_PM(6) POP_PM(4)
#undef POP_PM
        }
        __syncthreads();  // the next tile's direct loads overwrite the LDS
    }
}

// The same for four token fragments and narrow chunks: three steps of token rows in the ring.
template <int kMode>
__global__ __launch_bounds__(kPmThreads, 1) void prefill_deep_kernel(const uint16_t *__restrict__ w,
                                                                     const uint16_t *__restrict__ x, int T, int d, int m,
                                                                     int n_tt, PmTiles g, float *__restrict__ s2_part,
                                                                     PfStore st)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t pf_lds[];
    __shared__ float colsum[4][kPfChunk];
    for (int i = blockIdx.x / 8; i < g.per_xcd; i += gridDim.x / 8) {
        const int logical = (blockIdx.x % 8) * g.per_xcd + i;
        if (logical >= g.total) break;
        switch (g.f) {
#define POP_PM(FF)                                                                                                \
    case FF:                                                                                                      \
        pm_tile<kPmDeepMF, FF, kMode, PmDeepRing, false>(w, x, T, d, m, m, n_tt, logical, s2_part, st, pf_lds, colsum); \
        break;
            POP_PM(8) POP_PM(7) POP_PM(6) POP_PM(4)
#undef POP_PM
        }
        __syncthreads();  // the next tile's direct loads overwrite the LDS
    }
}

// ---- float32 layers: both projections of a few tokens on the FP64 matrix cores
//
// Products of float32 values are exact in double, so the sums are good to double whatever their order, and the decode
// steps' float64 dot products lose nothing to these.  16x16x4 products (64 cycles; lane (c, g) = (lane % 16, lane / 16)
// holds row c, k = g of either operand; register v of the result is row 4 v + g, column c).  The contraction index may be
// taken in any order as long as both operands agree, so a lane loads 16 bytes along k and feeds four products.
// Small layers are bound by latency: the four waves of a workgroup split the contraction and meet through LDS, and the
// tile (16 TA tokens x 8 NB channels) is small where that takes to fill the chip.  64 tokens, d 512, m 1376: 12 us
// with the scores, against 62 + 5 us for a float32 multiply-add tile on 43 workgroups and the launch that summed its rows.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
constexpr int kF32Waves = 4;
constexpr int kF32Steps = 4;  // k-steps of 16 elements whose loads are in flight per lane

// B rows of a fragment: gate rows of 8 channels, then the up rows of the same.  list: channels (null: all m), n_list on
// the device.  h32 [T][m] by channel and s2_part / scores as asked for.
template <int TA, int NB>
__global__ __launch_bounds__(kF32Waves * 64) void gateup_f32_kernel(const float *__restrict__ w, const float *__restrict__ x,
                                                                    int T, int d, int m, int n_tt,
                                                                    float *__restrict__ s2_part, PfStore st)
{
    constexpr int BM = 16 * TA, BC = 8 * NB;
    extern __shared__ __attribute__((aligned(16))) double f32_lds[];  // [4 waves][BM][16 NB], then h [BM][BC] floats
    __shared__ float colsum[1][kPfChunk];
    const int n_ch = st.list ? *st.n_list : m;
    const int c0 = blockIdx.x * BC, ttile = blockIdx.y, t0 = ttile * BM;
    if (c0 >= n_ch) return;
    const int cn = min(BC, n_ch - c0);
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c = lane % 16, g = lane / 16;

    const float *pa[TA], *pb[NB];
#pragma unroll
    for (int a = 0; a < TA; ++a) pa[a] = x + (size_t)min(t0 + 16 * a + c, T - 1) * d;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int cc = c0 + min(8 * b + c % 8, cn - 1);
        const int j = st.list ? st.list[cc] : cc;
        pb[b] = w + ((size_t)j * 3 + c / 8) * d;
    }
    f64x4_t acc[TA][NB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    for (int s = wave; s * 16 < d; s += kF32Waves * kF32Steps) {
        float4 va[kF32Steps][TA], vb[kF32Steps][NB];
#pragma unroll
        for (int u = 0; u < kF32Steps; ++u) {
            const int k = (s + u * kF32Waves) * 16 + 4 * g, kk = k < d ? k : 0;
#pragma unroll
            for (int a = 0; a < TA; ++a) va[u][a] = *reinterpret_cast<const float4 *>(pa[a] + kk);
#pragma unroll
            for (int b = 0; b < NB; ++b) vb[u][b] = *reinterpret_cast<const float4 *>(pb[b] + kk);
        }
#pragma unroll
        for (int u = 0; u < kF32Steps; ++u) {
            if ((s + u * kF32Waves) * 16 + 4 * g >= d) {  // (beyond the row: zeros of both operands, an infinite weight may stand
                                                         // at the row's start)
#pragma unroll
                for (int a = 0; a < TA; ++a) va[u][a] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int b = 0; b < NB; ++b) vb[u][b] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int a = 0; a < TA; ++a) {
                    const float4 &q = va[u][a];
                    const double fa = (double)(e == 0 ? q.x : (e == 1 ? q.y : (e == 2 ? q.z : q.w)));
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const float4 &r = vb[u][b];
                        const double fb = (double)(e == 0 ? r.x : (e == 1 ? r.y : (e == 2 ? r.z : r.w)));
                        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa, fb, acc[a][b], 0, 0, 0);
                    }
                }
        }
    }
    constexpr int RW = 16 * NB;
    double *mine = f32_lds + (size_t)wave * BM * RW;
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) mine[(16 * a + 4 * v + g) * RW + 16 * b + c] = acc[a][b][v];
    __syncthreads();
    float *hs = reinterpret_cast<float *>(f32_lds + (size_t)kF32Waves * BM * RW);  // [BM][BC]
    for (int i = tid; i < BM * BC; i += kF32Waves * kWave) {
        const int r = i / BC, ch = i % BC, at = r * RW + 16 * (ch / 8) + ch % 8;
        double gs = 0.0, us = 0.0;
#pragma unroll
        for (int q = 0; q < kF32Waves; ++q) {
            gs += f32_lds[(size_t)q * BM * RW + at];
            us += f32_lds[(size_t)q * BM * RW + at + 8];
        }
        const bool live = t0 + r < T && ch < cn;
        const float h = live ? silu_mul((float)gs, (float)us) : 0.f;
        hs[i] = h;
        if (live && st.h32) st.h32[(size_t)(t0 + r) * m + (st.list ? st.list[c0 + ch] : c0 + ch)] = h;
    }
    if (!s2_part) return;
    __syncthreads();
    if (tid < BC) {
        double tot = 0.0;
        for (int r = 0; r < BM; ++r) tot += (double)hs[r * BC + tid] * (double)hs[r * BC + tid];
        colsum[0][tid] = (float)tot;
    }
    pf_chunk_scores<1>(colsum, m, n_tt, ttile, blockIdx.x, c0, cn, s2_part, st);
}

template <int TA, int NB>
static hipError_t launch_gateup_f32(const void *w, int d, int m, const void *x, int T, float *s2_part, const PfStore &st,
                                    hipStream_t s)
{
    const size_t lds = (size_t)kF32Waves * 16 * TA * 16 * NB * sizeof(double) + (size_t)16 * TA * 8 * NB * sizeof(float);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gateup_f32_kernel<TA, NB>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int n_tt = (T + 16 * TA - 1) / (16 * TA);
    hipLaunchKernelGGL((gateup_f32_kernel<TA, NB>), dim3((m + 8 * NB - 1) / (8 * NB), n_tt), dim3(kF32Waves * kWave), lds, s,
                       (const float *)w, (const float *)x, T, d, m, n_tt, s2_part, st);
    return hipGetLastError();
}

// Tile of a float32 contraction: 64 tokens x 16 channels where that still gives every compute unit two workgroups, else
// 16 tokens x 8 channels.
static bool f32_large_tile(int T, int m, int n_cu) { return (T + 63) / 64 * ((m + 15) / 16) >= 2 * n_cu; }

static hipError_t launch_gateup_f32_any(const void *w, int d, int m, const void *x, int T, float *s2_part, int n_cu,
                                        const PfStore &st, hipStream_t s)
{
    return f32_large_tile(T, m, n_cu) ? launch_gateup_f32<4, 2>(w, d, m, x, T, s2_part, st, s)
                                      : launch_gateup_f32<1, 1>(w, d, m, x, T, s2_part, st, s);
}

// partial[slab][t][:] = sum over the slab's list positions of h[t][j] * w[j][2][:], t < T <= 16 TA.  A workgroup owns 64
// columns and a slab, its waves every fourth group of four channels; lane (c, g) loads 16 bytes of channel g's row at
// columns 4 c, product e takes column 4 c + e of every lane.
template <int TA>
__global__ __launch_bounds__(kF32Waves * 64) void down_f32_kernel(const float4 *__restrict__ w, int nvec,
                                                                  const int *__restrict__ list,
                                                                  const int *__restrict__ n_dev,
                                                                  const float *__restrict__ h, int m,
                                                                  const unsigned char *__restrict__ mask, int mask_stride,
                                                                  int T, float *__restrict__ partial, int d)
{
    __shared__ double red[kF32Waves][16 * 64];
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c = lane % 16, g = lane / 16;
    const int n = *n_dev, n_slabs = gridDim.y, per_slab = (n + n_slabs - 1) / n_slabs;
    const int s0 = min(n, (int)blockIdx.y * per_slab), s1 = min(n, s0 + per_slab);
    const int vcol = blockIdx.x * 16 + c;
    const float4 *wc = w + (vcol < nvec ? vcol : 0);
    f64x4_t acc[TA][4];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[a][e] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    constexpr int U = 4;
    for (int p0 = s0 + 4 * wave; p0 < s1; p0 += 4 * kF32Waves * U) {
        float4 vw[U];
        float va[U][TA];
        unsigned char mk[U][TA];
        int js[U];
#pragma unroll
        for (int u = 0; u < U; ++u) js[u] = list[min(p0 + 4 * kF32Waves * u + g, s1 - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            vw[u] = wc[((size_t)js[u] * 3 + 2) * nvec];
#pragma unroll
            for (int a = 0; a < TA; ++a) {
                const int t = min(16 * a + c, T - 1);
                va[u][a] = h[(size_t)t * m + js[u]];
                mk[u][a] = mask ? mask[(size_t)t * mask_stride + js[u]] : (unsigned char)1;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = p0 + 4 * kF32Waves * u + g < s1;
            // (beyond the slab: zeros of both operands, an infinite weight may stand in the row read there)
            const float4 q = live ? vw[u] : make_float4(0.f, 0.f, 0.f, 0.f);
            const double fw[4] = {(double)q.x, (double)q.y, (double)q.z, (double)q.w};
#pragma unroll
            for (int a = 0; a < TA; ++a) {
                const double fa = live && mk[u][a] ? (double)va[u][a] : 0.0;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[a][e] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa, fw[e], acc[a][e], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int a = 0; a < TA; ++a) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][(4 * v + g) * 64 + 4 * c + e] = acc[a][e][v];
        __syncthreads();
        for (int i = tid; i < 16 * 64; i += kF32Waves * kWave) {
            const int t = 16 * a + i / 64, col = blockIdx.x * 64 + i % 64;
            if (t < T && col < d)
                partial[((size_t)blockIdx.y * T + t) * d + col] = (float)((red[0][i] + red[1][i]) + (red[2][i] + red[3][i]));
        }
    }
}

int f32_down_slabs(int d, int m, int n_cu)
{
    const int cols = (d + 63) / 64;
    int slabs = 2 * n_cu / cols;
    if (slabs > (m + 31) / 32) slabs = (m + 31) / 32;  // (a few channels per wave at least)
    return slabs < 1 ? 1 : (slabs > 64 ? 64 : slabs);
}

hipError_t launch_down_f32_partials(const void *w, int d, int m, const int *list, const int *n_dev, const float *h,
                                    const unsigned char *mask, int mask_stride, int T, float *partial, int n_slabs,
                                    hipStream_t s)
{
    if (T < 1 || T > kF32MaxTokens) return hipErrorInvalidValue;
    const dim3 grid((d + 63) / 64, n_slabs);
    if (T <= 16)
        hipLaunchKernelGGL(down_f32_kernel<1>, grid, dim3(kF32Waves * kWave), 0, s, (const float4 *)w, d / 4, list, n_dev, h,
                           m, mask, mask_stride, T, partial, d);
    else
        hipLaunchKernelGGL(down_f32_kernel<4>, grid, dim3(kF32Waves * kWave), 0, s, (const float4 *)w, d / 4, list, n_dev, h,
                           m, mask, mask_stride, T, partial, d);
    return hipGetLastError();
}

// Token tile of the register-staged kernel: 256 or 128 tokens, whichever gives the cheaper schedule: tiles per compute
// unit on the busiest one (after the chunks are evened out) times a tile's measured relative cost - 1 for 256 tokens x
// three fragments, 0.8 with two fragments, and 0.6 of either for the 128-token form.
static int prefill_token_tile(int T, int n_ch, int n_cu)
{
    int best_bm = 256;
    long best = -1;
    for (int bm = 256; bm >= 128; bm -= 128) {
        const PfGeom g = prefill_geometry(n_ch, (T + bm - 1) / bm, n_cu);
        const long waves = (g.total + n_cu - 1) / n_cu;
        const long cost = waves * (g.nf == 3 ? 5 : 4) * (bm == 256 ? 5 : 3);
        if (best < 0 || cost < best) best = cost, best_bm = bm;
    }
    return best_bm;
}

// Rows that are whole k-steps long take the direct-load kernel.
static bool prefill_direct(int d) { return d % kPfBK == 0; }

// Token fragments per wave of the direct-load kernel: the cheapest schedule over the tile heights.
static int pm_token_fragments(int T, int n_ch, int n_cu, PmTiles *tiles)
{
    int best = 1, best_cost = 0;
    for (int mf = 1; mf <= kPmMaxMF; ++mf) {
        int cost = 0;
        const PmTiles g = pm_tiles(n_ch, (T + 64 * mf - 1) / (64 * mf), mf, n_cu, &cost);
        if (mf == 1 || cost < best_cost) best_cost = cost, best = mf, *tiles = g;
    }
    return best;
}

int prefill_rows_used(int T, int d, int m, int n_cu)
{
    if (prefill_direct(d)) {
        PmTiles g;
        const int bm = 64 * pm_token_fragments(T, m, n_cu, &g);
        return (T + bm - 1) / bm;
    }
    const int bm = prefill_token_tile(T, m, n_cu);
    return (T + bm - 1) / bm;
}

template <int BM, int NW, int NF, int kMode>
static hipError_t launch_pf_bf16(int blocks, hipStream_t s, const void *w, const void *x, int T, int d, int m, int n_tt,
                                 const PfGeom &g, float *s2_part, const PfStore &st)
{
    const size_t lds = (size_t)2 * (BM + NF * 64) * kPfLd * sizeof(uint16_t);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&prefill_bf16_kernel<BM, NW, NF, kMode>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((prefill_bf16_kernel<BM, NW, NF, kMode>), dim3(blocks), dim3(NW * 64), lds, s,
                       (const uint16_t *)w, (const uint16_t *)x, T, d, m, n_tt, g.chunk, g.total, g.per_xcd, s2_part, st);
    return hipGetLastError();
}

template <int MF, int kMode>
static hipError_t launch_pm(const void *w, int d, int m, const void *x, int T, const PmTiles &g, float *s2_part, int n_cu,
                            const PfStore &st, long long stream_from, hipStream_t s)
{
    void (*kernel)(const uint16_t *, const uint16_t *, int, int, int, int, PmTiles, float *, PfStore);
    const int n_tt = (T + 64 * MF - 1) / (64 * MF);
    // (the list form learns its F on the device; wider chunks do not leave the room)
    const bool deep = pm_deep(MF, g.f, kMode), stream = pm_streams<MF, kMode>(d, m, T, g.total <= n_cu, stream_from);
    const size_t lds = deep ? PmDeepRing::kBytes : PmRing<MF>::kBytes;
    if constexpr (kMode == 5) {
        kernel = stream ? prefill_rows_kernel<MF, true> : prefill_rows_kernel<MF, false>;
    } else {
        kernel = stream ? prefill_stream_kernel<MF, kMode> : prefill_mma_kernel<MF, kMode>;
        if constexpr (MF == kPmDeepMF && (kMode == 0 || kMode == 2))
            if (deep && !stream) kernel = prefill_deep_kernel<kMode>;
    }
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    const int all = kMode == 1 || kMode == 4 ? n_cu : (g.total < n_cu ? g.total : n_cu);
    hipLaunchKernelGGL(kernel, dim3((all + 7) / 8 * 8), dim3(kPmThreads), lds, s, (const uint16_t *)w, (const uint16_t *)x, T,
                       d, m, n_tt, g, s2_part, st);
    return hipGetLastError();
}

template <int kMode>
static hipError_t launch_pm_all(const void *w, int d, int m, const void *x, int T, float *s2_part, int n_cu,
                                const PfStore &st, long long stream_from, hipStream_t s)
{
    PmTiles g;
    switch (pm_token_fragments(T, m, n_cu, &g)) {  // (list form: priced as all m channels, cut up on the device)
    case 1: return launch_pm<1, kMode>(w, d, m, x, T, g, s2_part, n_cu, st, stream_from, s);
    case 2: return launch_pm<2, kMode>(w, d, m, x, T, g, s2_part, n_cu, st, stream_from, s);
    case 3: return launch_pm<3, kMode>(w, d, m, x, T, g, s2_part, n_cu, st, stream_from, s);
    case 4: return launch_pm<4, kMode>(w, d, m, x, T, g, s2_part, n_cu, st, stream_from, s);
    default: return launch_pm<5, kMode>(w, d, m, x, T, g, s2_part, n_cu, st, stream_from, s);
    }
}

// Whether the contraction's launch forms the scores itself: when every compute unit runs one tile at most.  The tile
// that completes a chunk learns so through a write-through store, its acknowledgement and a counted arrival, a few
// microseconds that nothing hides at the end of a launch with one tile per compute unit anyway, but that would stand
// between the tiles a compute unit runs back to back on a long prompt (measured: +14 us at 2048 tokens).
bool prefill_forms_scores(int is_bf16, int T, int d, int m, int n_cu)
{
    if (T < 1) return false;
    if (!is_bf16) return true;  // (small tiles, many per compute unit: one's wait hides behind the others)
    if (prefill_direct(d)) {
        PmTiles g;
        pm_token_fragments(T, m, n_cu, &g);
        return g.total <= n_cu;
    }
    const int bm = prefill_token_tile(T, m, n_cu);
    return prefill_geometry(m, (T + bm - 1) / bm, n_cu).total <= n_cu;
}

template <int kMode>
static hipError_t launch_pf_bf16_all(const void *w, int d, int m, const void *x, int T, float *s2_part, int n_cu,
                                     PfStore st, hipStream_t s)
{
    if (!prefill_forms_scores(1, T, d, m, n_cu)) st.fin_ctr = nullptr;
    if (prefill_direct(d)) return launch_pm_all<kMode>(w, d, m, x, T, s2_part, n_cu, st, kMode == 0 ? kStreamPartBytes : kStreamPromptBytes, s);
    const int bm = prefill_token_tile(T, m, n_cu);
    const int n_tt = (T + bm - 1) / bm;
    const PfGeom g = prefill_geometry(m, n_tt, n_cu);
    const int blocks = g.per_xcd * 8;
    // 256-token tiles run with 8 waves (two per SIMD: one wave's waits for staging loads, LDS writes and the
    // k-step barrier are covered by the other's products), 128-token tiles with 4
    if (bm == 256 && g.nf == 3) return launch_pf_bf16<256, 8, 3, kMode>(blocks, s, w, x, T, d, m, n_tt, g, s2_part, st);
    if (bm == 256) return launch_pf_bf16<256, 8, 2, kMode>(blocks, s, w, x, T, d, m, n_tt, g, s2_part, st);
    if (g.nf == 3) return launch_pf_bf16<128, 4, 3, kMode>(blocks, s, w, x, T, d, m, n_tt, g, s2_part, st);
    return launch_pf_bf16<128, 4, 2, kMode>(blocks, s, w, x, T, d, m, n_tt, g, s2_part, st);
}

// bf16 only: the prefill contraction that also keeps H, h_all[t][j] = bf16(H[t][j]) with row stride ldh, or by_channel (d a
// multiple of 64) h_all[j][t] with ldh >= T a multiple of 64.
hipError_t launch_prefill_gateup_keep_bf16(const void *w, int d, int m, const void *x, int T, float *s2_part,
                                           uint16_t *h_all, int ldh, bool by_channel, int n_cu, hipStream_t s,
                                           const PrefillScores *fin)
{
    PfStore st{nullptr, nullptr, h_all, ldh, nullptr, n_cu};
    if (fin) st.fin_ctr = fin->chunk_ctr, st.nrm = fin->nrm, st.scores = fin->scores;
    if (by_channel) {
        if (!prefill_direct(d)) return hipErrorInvalidValue;
        if (!prefill_forms_scores(1, T, d, m, n_cu)) st.fin_ctr = nullptr;
        return launch_pm_all<5>(w, d, m, x, T, s2_part, n_cu, st, kStreamPromptBytes, s);
    }
    return launch_pf_bf16_all<2>(w, d, m, x, T, s2_part, n_cu, st, s);
}

hipError_t launch_prefill_gateup(const void *w, int is_bf16, int d, int m, const void *x, int T, float *s2_part,
                                 int n_cu, hipStream_t s, const PrefillScores *fin)
{
    if (is_bf16) {
        PfStore st{};
        if (fin) st.fin_ctr = fin->chunk_ctr, st.nrm = fin->nrm, st.scores = fin->scores;
        return launch_pf_bf16_all<0>(w, d, m, x, T, s2_part, n_cu, st, s);
    }
    PfStore st{};
    if (fin) st.fin_ctr = fin->chunk_ctr, st.nrm = fin->nrm, st.scores = fin->scores;
    return launch_gateup_f32_any(w, d, m, x, T, s2_part, n_cu, st, s);
}

// bf16 only.  Gate/up over the channels of a device-resident list; hc[t][c] = bf16(H[t][list[c]]) (times
// tmask[t][list[c]] if tmask is given).  The list's length is known on the device only.  Direct-load kernel: every
// workgroup cuts the list up for itself.  Register-staged kernel: both tile forms are launched, each sized for the
// longest possible list (m channels), and the one the length does not call for exits at once.
hipError_t launch_gateup_list_bf16(const void *w, int d, int m, const void *x, int T, const int *list, const int *n_list,
                                   const unsigned char *tmask, uint16_t *hc, int ldh, int n_cu, long long stream_from, hipStream_t s)
{
    PfStore st{list, n_list, hc, ldh, tmask, n_cu};
    if (prefill_direct(d)) return launch_pm_all<1>(w, d, m, x, T, nullptr, n_cu, st, stream_from, s);
    const int bm = prefill_token_tile(T, m, n_cu);  // (the list's length is not known here: priced as all m channels)
    const int n_tt = (T + bm - 1) / bm;
    PfGeom g{};
    hipError_t e = hipSuccess;
    for (int nf = 3; nf >= 2 && e == hipSuccess; --nf) {
        // an upper bound of the tile count over all list lengths <= m (the count before chunks are evened out)
        const int min_ct = (m + nf * 32 - 1) / (nf * 32);
        const int per_cu = (min_ct * n_tt + n_cu - 1) / n_cu;
        int n_ct = per_cu * n_cu / n_tt;
        if (n_ct < min_ct) n_ct = min_ct;
        const int blocks = (n_tt * n_ct + 7) / 8 * 8;
        if (bm == 256 && nf == 3) e = launch_pf_bf16<256, 8, 3, 1>(blocks, s, w, x, T, d, m, n_tt, g, nullptr, st);
        else if (bm == 256) e = launch_pf_bf16<256, 8, 2, 1>(blocks, s, w, x, T, d, m, n_tt, g, nullptr, st);
        else if (nf == 3) e = launch_pf_bf16<128, 4, 3, 1>(blocks, s, w, x, T, d, m, n_tt, g, nullptr, st);
        else e = launch_pf_bf16<128, 4, 2, 1>(blocks, s, w, x, T, d, m, n_tt, g, nullptr, st);
    }
    return e;
}

int precise_max_tokens(int is_bf16, int d) { return is_bf16 ? (prefill_direct(d) ? 31 : 0) : kF32MaxTokens; }

// (bf16: one token tile, bound by the weight stream, so the sums in double are free: 24 tokens, d 4096, m 11008 take 34 us,
// the same as without.)
hipError_t launch_precise_gateup(const void *w, int is_bf16, int d, int m, const void *x, int T, const int *list,
                                 const int *n_list, float *h, float *s2_part, const PrefillScores *fin, int n_cu,
                                 long long stream_from, hipStream_t s)
{
    PfStore st{list, n_list, nullptr, 0, nullptr, n_cu};
    st.h32 = h;
    if (fin && !list) st.fin_ctr = fin->chunk_ctr, st.nrm = fin->nrm, st.scores = fin->scores;
    if (!is_bf16) return launch_gateup_f32_any(w, d, m, x, T, list ? nullptr : s2_part, n_cu, st, s);
    if (list) return launch_pm<1, 4>(w, d, m, x, T, PmTiles{}, nullptr, n_cu, st, stream_from, s);
    return launch_pm<1, 3>(w, d, m, x, T, pm_tiles(m, 1, 1, n_cu), s2_part, n_cu, st, stream_from, s);
}

// scores[j] = nrm[j] * sqrt(sum over token tiles, in tile order, of s2_part[tile][j])   (Eq. 3)
__global__ __launch_bounds__(256) void scores_from_partials_kernel(const float *__restrict__ s2_part, int n_tiles, int m,
                                                                   const float *__restrict__ nrm,
                                                                   float *__restrict__ scores)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    double acc = 0.0;
    for (int t = 0; t < n_tiles; ++t) acc += (double)s2_part[(size_t)t * m + j];
    scores[j] = (float)((double)nrm[j] * sqrt(acc));
}

hipError_t launch_scores_from_partials(const float *s2_part, int n_tiles, int m, const float *nrm, float *scores,
                                       hipStream_t s)
{
    hipLaunchKernelGGL(scores_from_partials_kernel, dim3((m + 255) / 256), dim3(256), 0, s, s2_part, n_tiles, m, nrm,
                       scores);
    return hipGetLastError();
}

}  // namespace pop
