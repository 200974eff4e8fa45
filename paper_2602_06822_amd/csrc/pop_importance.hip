// Column-wise importance reduction over materialised activations (Sec. 3.4 Eq. 3):
//     scores[j] = nrm[j] * sqrt( sum over tokens t of H[t][j]^2 ),   H: [T][m] float32 or bf16.
//
// HBM-bound: every element of H is read once, sums in double (a float32 running sum over a long prompt would lose more
// than the 1e-5 the scores are held to), the summation order fixed by (T, m, the alignment) alone, so the result is
// bit-reproducible.  Two forms:
//  * importance_columns_kernel: one workgroup takes 64 columns and all tokens, so nothing is left to add up afterwards and
//    no scratch is needed.  A row segment is one or two cache lines; 16 waves x 8 loads of 16 bytes per lane keep 128 KB on
//    their way per compute unit, so a 1024-token prompt is a single round trip.  1024 x 13824 bf16: 7 us, against 20 + 6 us
//    for the two launches below and the allocation of their scratch around them.
//  * long prompts of few columns (fewer than kIrMinGroups workgroups, more than kIrLongPrompt tokens; or narrow rows that
//    can only be read one element at a time) would leave most of the chip idle for many rounds: tokens split into chunks,
//    per-chunk partial sums in scratch.  8192 x 1000 bf16: 24 us in columns, 41 in chunks; 16384 x 8200: 69 and 207.
//      stage 1  part[chunk][j] = sum over the chunk's tokens of H[t][j]^2; 256 adjacent columns of one token chunk per
//               workgroup, a lane one column of each 64-column group, eight rows in flight per lane; the four waves take
//               the chunk's rows round robin and meet through LDS in wave order.
//      stage 2  scores[j] = nrm[j] * sqrt(sum over chunks, in chunk order, of part[chunk][j]).
//    `part` is scratch: [n_chunks][m] doubles beyond the inputs and outputs.
#include <mutex>

#include "pop_internal.h"

namespace pop {

constexpr int kIrCols = 256;      // columns per workgroup
constexpr int kIrWaves = 4;       // waves per workgroup: rows of the chunk round robin
constexpr int kIrRows = 8;        // rows in flight per lane
constexpr int kIrMaxChunks = 32;  // token chunks at most

template <bool BF16>
__device__ __forceinline__ float ir_load(const void *h, size_t i)
{
    return BF16 ? __uint_as_float(((uint32_t)((const uint16_t *)h)[i]) << 16) : ((const float *)h)[i];
}

constexpr int kIcCols = 64;        // columns per workgroup
constexpr int kIcWaves = 16;
constexpr int kIcRows = 8;         // loads in flight per lane
constexpr int kIrMinGroups = 128;
constexpr int kIrLongPrompt = 8192;
// Narrow rows read one element at a time: a few workgroups with a sixteenth of the bytes in flight (8192 x 1001 bf16: 47 us
// in columns, 41 in chunks; 8192 x 63: 41 and 26; 8192 x 1001 float32: 45 and 84; 5000 x 1001 bf16: 29 and 31).
constexpr int kIrLongPromptSingle = 5120;
constexpr int kIrNarrowRow = 2048;  // bytes

// E columns per lane: 16-byte loads (8 bf16, 4 float32; rows and base 16-byte aligned) or, E = 1, one element.
// nrm == nullptr: the sums themselves.
template <bool BF16, int E>
__global__ __launch_bounds__(kIcWaves * kWave) void importance_columns_kernel(const void *__restrict__ h, int T, int m,
                                                                              const float *__restrict__ nrm,
                                                                              float *__restrict__ scores)
{
    __shared__ double red[kIcWaves][kIcCols];
    constexpr int LPR = kIcCols / E;        // lanes per row
    constexpr int RPW = kWave / LPR;        // rows a wave's load covers
    constexpr int step = kIcWaves * RPW;
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int col = blockIdx.x * kIcCols + lane % LPR * E, r0 = wave * RPW + lane / LPR;
    const bool ok = col < m;                // (E columns at once: m is a multiple of E there)
    double acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.0;
    for (int t = r0; t < T; t += step * kIcRows) {
        if constexpr (E == 1) {
            float v[kIcRows];
#pragma unroll
            for (int u = 0; u < kIcRows; ++u) {
                const int tr = t + u * step;
                v[u] = ir_load<BF16>(h, (size_t)min(tr, T - 1) * m + (ok ? col : 0));
                v[u] = tr < T ? v[u] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kIcRows; ++u) acc[0] = fma((double)v[u], (double)v[u], acc[0]);
        } else {
            uint4 v[kIcRows];
#pragma unroll
            for (int u = 0; u < kIcRows; ++u) {
                const size_t at = (size_t)min(t + u * step, T - 1) * m + (ok ? col : 0);
                v[u] = *reinterpret_cast<const uint4 *>((const unsigned char *)h + at * (BF16 ? 2 : 4));
            }
#pragma unroll
            for (int u = 0; u < kIcRows; ++u) {
                const uint32_t q[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                const bool live = t + u * step < T;
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const float f = BF16 ? (e % 2 ? bf16_hi(q[e / 2]) : bf16_lo(q[e / 2])) : __uint_as_float(q[e % 4]);
                    const double d = live ? (double)f : 0.0;
                    acc[e] = fma(d, d, acc[e]);
                }
            }
        }
    }
    // rows of the wave's lanes, then the waves in order
#pragma unroll
    for (int e = 0; e < E; ++e) {
#pragma unroll
        for (int off = LPR; off < kWave; off <<= 1) acc[e] += __shfl_xor(acc[e], off, kWave);
        if (lane < LPR) red[wave][lane * E + e] = acc[e];
    }
    __syncthreads();
    const int j = blockIdx.x * kIcCols + (int)threadIdx.x;
    if (threadIdx.x < kIcCols && j < m) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < kIcWaves; ++w) tot += red[w][threadIdx.x];
        scores[j] = nrm ? (float)((double)nrm[j] * sqrt(tot)) : (float)tot;
    }
}

template <bool BF16>
__global__ __launch_bounds__(kIrWaves * kWave) void importance_partial_kernel(const void *__restrict__ h, int T, int m,
                                                                              int rows_per_chunk,
                                                                              double *__restrict__ part)
{
    __shared__ double red[kIrWaves][kIrCols];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int c0 = blockIdx.x * kIrCols, chunk = blockIdx.y;
    const int t_lo = chunk * rows_per_chunk, t_hi = min(T, t_lo + rows_per_chunk);
    constexpr int G = kIrCols / kWave;  // column groups of a lane
    int col[G];
    bool ok[G];
    double acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        col[g] = c0 + g * kWave + lane;
        ok[g] = col[g] < m;
        acc[g] = 0.0;
    }
    // wave w takes rows t_lo + w, t_lo + w + 4, ...; kIrRows of them requested together
    for (int t = t_lo + wave; t < t_hi; t += kIrWaves * kIrRows) {
        float v[kIrRows][G];
#pragma unroll
        for (int r = 0; r < kIrRows; ++r) {
            const int tr = t + r * kIrWaves;
#pragma unroll
            for (int g = 0; g < G; ++g) v[r][g] = (tr < t_hi && ok[g]) ? ir_load<BF16>(h, (size_t)tr * m + col[g]) : 0.f;
        }
#pragma unroll
        for (int r = 0; r < kIrRows; ++r)
#pragma unroll
            for (int g = 0; g < G; ++g) acc[g] = fma((double)v[r][g], (double)v[r][g], acc[g]);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) red[wave][g * kWave + lane] = acc[g];
    __syncthreads();
    const int c = c0 + (int)threadIdx.x;
    if (c < m) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < kIrWaves; ++w) tot += red[w][threadIdx.x];
        part[(size_t)chunk * m + c] = tot;
    }
}

__global__ __launch_bounds__(256) void importance_finish_kernel(const double *__restrict__ part, int n_chunks, int m,
                                                                const float *__restrict__ nrm,
                                                                float *__restrict__ scores)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    double tot = 0.0;
    for (int c = 0; c < n_chunks; ++c) tot += part[(size_t)c * m + j];
    scores[j] = (float)((double)nrm[j] * sqrt(tot));
}

// Token chunks for (T, m): enough workgroups to fill the chip a few times over, at least 32 rows per chunk.
static int importance_chunks(int T, int m)
{
    const int col_blocks = (m + kIrCols - 1) / kIrCols;
    int n = (1024 + col_blocks - 1) / col_blocks;
    if (n > kIrMaxChunks) n = kIrMaxChunks;
    if (n > (T + 31) / 32) n = (T + 31) / 32;
    return n < 1 ? 1 : n;
}

// Whether rows can be read 16 bytes at a time.
static bool importance_vec(const void *h, int is_bf16, int m)
{
    return (reinterpret_cast<uintptr_t>(h) & 15u) == 0 && m % (is_bf16 ? 8 : 4) == 0;
}

static bool importance_in_chunks(const void *h, int is_bf16, int T, int m)
{
    if (!importance_vec(h, is_bf16, m) && T > kIrLongPromptSingle && (long long)m * (is_bf16 ? 2 : 4) <= kIrNarrowRow) return true;
    return T > kIrLongPrompt && (m + kIcCols - 1) / kIcCols < kIrMinGroups;
}

size_t importance_reduce_scratch_bytes(const void *h, int is_bf16, int T, int m)
{
    return importance_in_chunks(h, is_bf16, T, m) ? (size_t)importance_chunks(T, m) * m * sizeof(double) : 0;
}

static hipError_t launch_importance_columns(const void *h, int is_bf16, int T, int m, const float *nrm, float *scores,
                                            hipStream_t s)
{
    const dim3 grid((m + kIcCols - 1) / kIcCols), block(kIcWaves * kWave);
    const bool vec = importance_vec(h, is_bf16, m);
    if (is_bf16 && vec)
        hipLaunchKernelGGL((importance_columns_kernel<true, 8>), grid, block, 0, s, h, T, m, nrm, scores);
    else if (is_bf16)
        hipLaunchKernelGGL((importance_columns_kernel<true, 1>), grid, block, 0, s, h, T, m, nrm, scores);
    else if (vec)
        hipLaunchKernelGGL((importance_columns_kernel<false, 4>), grid, block, 0, s, h, T, m, nrm, scores);
    else
        hipLaunchKernelGGL((importance_columns_kernel<false, 1>), grid, block, 0, s, h, T, m, nrm, scores);
    return hipGetLastError();
}

hipError_t launch_importance_reduce(const void *h, int is_bf16, int T, int m, const float *nrm, float *scores,
                                    void *scratch, hipStream_t s)
{
    if (!importance_in_chunks(h, is_bf16, T, m)) return launch_importance_columns(h, is_bf16, T, m, nrm, scores, s);
    const int n_chunks = importance_chunks(T, m);
    const int rows_per_chunk = (T + n_chunks - 1) / n_chunks;
    double *part = (double *)scratch;
    dim3 grid((m + kIrCols - 1) / kIrCols, n_chunks);
    if (is_bf16)
        hipLaunchKernelGGL(importance_partial_kernel<true>, grid, dim3(kIrWaves * kWave), 0, s, h, T, m, rows_per_chunk,
                           part);
    else
        hipLaunchKernelGGL(importance_partial_kernel<false>, grid, dim3(kIrWaves * kWave), 0, s, h, T, m, rows_per_chunk,
                           part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(importance_finish_kernel, dim3((m + 255) / 256), dim3(256), 0, s, part, n_chunks, m, nrm, scores);
    return hipGetLastError();
}

bool column_squares_takes(int T) { return T <= kIrLongPrompt; }

hipError_t launch_column_squares(const void *x, int is_bf16, int T, int d, float *s2, hipStream_t s)
{
    return launch_importance_columns(x, is_bf16, T, d, nullptr, s2, s);
}

}  // namespace pop

// ---------------------------------------------------------------- the variant that allocates nothing
// Scratch of the variant below: a file-scope device array (every GPU the library runs on holds its own copy until
// the process ends).  Host code never passes the array's name to a kernel: the name is a host-side stand-in, not a
// device address.  Its device address is looked up once per device and used from then on.
namespace {

constexpr int kStaticMaxChannels = 32768;  // largest m of the allocation-free variant
constexpr size_t kStaticScratchBytes = (size_t)pop::kIrMaxChunks * kStaticMaxChannels * sizeof(double);  // 8 MiB
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each device, once looked up

// Device address of the static scratch on the current device (looked up at the first call on that device).
hipError_t static_scratch(void **ptr)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

extern "C" int pop_importance_reduce_static(const void *h, pop_dtype_t hdtype, int T, int m, const float *nrm,
                                            float *scores, void *stream)
{
    if (!h || !nrm || !scores) return POP_EINVAL;
    if (hdtype != POP_F32 && hdtype != POP_BF16) return POP_EINVAL;
    if (T < 1 || m < 1) return POP_ESHAPE;
    const size_t bytes = pop::importance_reduce_scratch_bytes(h, hdtype == POP_BF16, T, m);
    if (m > kStaticMaxChannels || bytes > kStaticScratchBytes)
        return POP_EUNSUPPORTED;  // beyond the static scratch: use pop_importance_reduce
    void *ptr = nullptr;
    if (bytes > 0 && static_scratch(&ptr) != hipSuccess) {
        (void)hipGetLastError();
        return POP_EHIP;
    }
    // stage 1 writes every partial sum that stage 2 reads, so nothing in the array has to start at zero
    const hipError_t e = pop::launch_importance_reduce(h, hdtype == POP_BF16, T, m, nrm, scores, ptr,
                                                       reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return POP_EHIP;
    return POP_OK;
}
