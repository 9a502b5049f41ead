// FP64 vector kernels for the Krylov solver (HBM-bound level-1/level-2 work).
// Reductions are two-pass with a fixed block count and fixed order, so every
// result is bitwise reproducible from run to run.
#include <algorithm>

#include "common.hpp"

namespace ertvie {

namespace {

constexpr int kBlk = 256;
constexpr int kRedBlocks = 240;   // partial sums per column
constexpr int kColGroup = 8;      // columns reduced together per pass over w

constexpr int kWave = 64;
constexpr int kWavesPerBlk = kBlk / kWave;
constexpr int kHChunk = 1024;     // coefficients of one subtraction pass, in LDS

// Sum over the 64 lanes of a wave (butterfly: every lane ends with the same bits).
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) v += __shfl_xor(v, s, kWave);
    return v;
}

// Column sums of the partials [nblk][ncols], columns c0 .. c0 + n - 1, into sh[0 .. n): one
// wave per column, lanes over the blocks, then the butterfly (fixed order).
__device__ __forceinline__ void sum_partials(const double* __restrict__ part, int nblk, int ncols, int c0, int n,
                                             double* sh)
{
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    for (int c = wave; c < n; c += kWavesPerBlk) {
        double s = 0.0;
        for (int b = lane; b < nblk; b += kWave) s += part[(long)b * ncols + c0 + c];
        s = wave_sum(s);
        if (lane == 0) sh[c] = s;
    }
}

// One pass of a Gram-Schmidt step over the workgroup's piece of w:
//   SUB   h = column sums of pin; w -= V h (block 0 writes h to hout, added to it with ADD);
//   DOTS  pout[block][c] = partial <V[:,c], w> of the (updated) piece;
//   NORM  pout[block] = partial <w, w>.
// The sums that a pass needs from the whole of w cross the launch boundary as partials,
// and every workgroup sums them again for itself (nblk * ncols values from L2): a
// Gram-Schmidt step with one re-orthogonalisation is then three launches and a final
// one, instead of nine, three of them a one-thread-per-column sum of the partials of 25 us
// (2D 512^2 solve of 9 steps with the FFT-based preconditioner: 5.62 ms before, 4.31 ms
// after).  Bound: HBM for many columns, launch latency for few.
template <bool SUB, bool ADD, bool DOTS, bool NORM>
__global__ __launch_bounds__(kBlk) void k_orth(const double* __restrict__ V, long ldv, int ncols, double* __restrict__ w,
                                               long N, const double* __restrict__ pin, double* __restrict__ hout,
                                               double* __restrict__ pout)
{
    __shared__ double sh[SUB ? kHChunk : 1];
    __shared__ double red[kWavesPerBlk][kColGroup];
    const long chunk = (N + gridDim.x - 1) / gridDim.x;
    const long lo = blockIdx.x * chunk;
    const long hi = (lo + chunk) < N ? (lo + chunk) : N;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    double nn = 0.0;
    if constexpr (SUB) {
        for (int c0 = 0; c0 < ncols; c0 += kHChunk) {
            const int n = min(kHChunk, ncols - c0);
            __syncthreads();
            sum_partials(pin, gridDim.x, ncols, c0, n, sh);
            __syncthreads();
            if (blockIdx.x == 0)
                for (int c = threadIdx.x; c < n; c += kBlk) hout[c0 + c] = ADD ? hout[c0 + c] + sh[c] : sh[c];
            for (long i = lo + threadIdx.x; i < hi; i += kBlk) {
                double s = 0.0;
                const double* v = V + (long)c0 * ldv + i;
                int c = 0;
                for (; c + 8 <= n; c += 8) {
                    double x[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[u] = v[(long)(c + u) * ldv];
#pragma unroll
                    for (int u = 0; u < 8; ++u) s += x[u] * sh[c + u];
                }
                for (; c < n; ++c) s += v[(long)c * ldv] * sh[c];
                const double wi = w[i] - s;
                w[i] = wi;
                if (NORM && c0 + kHChunk >= ncols) nn += wi * wi;
            }
        }
    }
    if constexpr (DOTS) {
        for (int c0 = 0; c0 < ncols; c0 += kColGroup) {
            double acc[kColGroup];
#pragma unroll
            for (int c = 0; c < kColGroup; ++c) acc[c] = 0.0;
            for (long i = lo + threadIdx.x; i < hi; i += kBlk) {
                const double wi = w[i];
#pragma unroll
                for (int c = 0; c < kColGroup; ++c)
                    if (c0 + c < ncols) acc[c] += V[(long)(c0 + c) * ldv + i] * wi;
            }
            __syncthreads();                              // the previous group's sums are read
#pragma unroll
            for (int c = 0; c < kColGroup; ++c) {
                const double s = wave_sum(acc[c]);
                if (lane == 0) red[wave][c] = s;
            }
            __syncthreads();
            if (threadIdx.x < kColGroup && c0 + (int)threadIdx.x < ncols) {
                double s = red[0][threadIdx.x];
                for (int q = 1; q < kWavesPerBlk; ++q) s += red[q][threadIdx.x];
                pout[(long)blockIdx.x * ncols + c0 + threadIdx.x] = s;
            }
        }
    }
    if constexpr (NORM) {
        nn = wave_sum(nn);
        __syncthreads();
        if (lane == 0) red[wave][0] = nn;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = red[0][0];
            for (int q = 1; q < kWavesPerBlk; ++q) s += red[q][0];
            pout[blockIdx.x] = s;
        }
    }
}

// out[c] = column sums of the partials (one wave per column).
__global__ __launch_bounds__(kBlk) void k_multidot_final(const double* __restrict__ part, int nblk, int ncols,
                                                         double* __restrict__ out)
{
    __shared__ double sh[kWavesPerBlk];
    const int c0 = blockIdx.x * kWavesPerBlk, n = min(kWavesPerBlk, ncols - c0);
    sum_partials(part, nblk, ncols, c0, n, sh);
    __syncthreads();
    if ((int)threadIdx.x < n) out[c0 + threadIdx.x] = sh[threadIdx.x];
}

// The end of a Gram-Schmidt step: the squared norm from its partials, and the column of
// the Hessenberg matrix (h, then the squared norm) to page-locked host memory.
__global__ __launch_bounds__(kBlk) void k_orth_final(const double* __restrict__ part, int nblk,
                                                     const double* __restrict__ h, int ncols,
                                                     double* __restrict__ host)
{
    __shared__ double sh[1];
    sum_partials(part, nblk, 1, 0, 1, sh);
    for (int c = threadIdx.x; c < ncols; c += kBlk) host[c] = h[c];
    __syncthreads();
    if (threadIdx.x == 0) host[ncols] = sh[0];
}

__global__ __launch_bounds__(kBlk) void k_gemv(const double* __restrict__ V, long ldv, int ncols,
                                               const double* __restrict__ coef, double* __restrict__ w, long N)
{
    const long i = blockIdx.x * (long)kBlk + threadIdx.x;
    if (i >= N) return;
    double s = 0.0;
    for (int c = 0; c < ncols; ++c) s += V[(long)c * ldv + i] * coef[c];
    w[i] += s;
}

__global__ void k_scale(double* __restrict__ y, const double* __restrict__ x, double a, long N)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < N) y[i] = a * x[i];
}

__global__ void k_sub(double* __restrict__ y, const double* __restrict__ a, const double* __restrict__ b, long N)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < N) y[i] = a[i] - b[i];
}

__global__ void k_add(double* __restrict__ y, const double* __restrict__ x, long N)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < N) y[i] += x[i];
}

__global__ void k_zero(double* __restrict__ y, long N)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < N) y[i] = 0.0;
}

// workgroups of a reduction: about 64 values each at least, at most kRedBlocks
inline int red_blocks(long N)
{
    int nb = kRedBlocks;
    if ((long)nb * 64 > N) nb = (int)((N + 63) / 64);
    return nb < 1 ? 1 : nb;
}

inline unsigned nblocks(long N) { return (unsigned)((N + kBlk - 1) / kBlk); }

}  // namespace

ert_status dev_multidot(hipStream_t s, const double* V, long ldv, int ncols, const double* w, long N,
                        double* partial, double* out)
{
    if (ncols <= 0) return ERT_OK;
    const int nb = red_blocks(N);
    // (w is only read: the instance has no subtraction)
    hipLaunchKernelGGL((k_orth<false, false, true, false>), dim3(nb), dim3(kBlk), 0, s, V, ldv, ncols,
                       const_cast<double*>(w), N, (const double*)nullptr, (double*)nullptr, partial);
    ERT_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_multidot_final, dim3((ncols + kWavesPerBlk - 1) / kWavesPerBlk), dim3(kBlk), 0, s,
                       (const double*)partial, nb, ncols, out);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status dev_orthogonalise(hipStream_t s, const double* V, long ldv, int ncols, double* w, long N, double* partial,
                             double* partial2, double* h, double* host)
{
    const int nb = red_blocks(N);
    const dim3 grid(nb), blk(kBlk);
    hipLaunchKernelGGL((k_orth<false, false, true, false>), grid, blk, 0, s, V, ldv, ncols, w, N,
                       (const double*)nullptr, (double*)nullptr, partial);
    hipLaunchKernelGGL((k_orth<true, false, true, false>), grid, blk, 0, s, V, ldv, ncols, w, N,
                       (const double*)partial, h, partial2);
    hipLaunchKernelGGL((k_orth<true, true, false, true>), grid, blk, 0, s, V, ldv, ncols, w, N,
                       (const double*)partial2, h, partial);
    hipLaunchKernelGGL(k_orth_final, dim3(1), blk, 0, s, (const double*)partial, nb, (const double*)h, ncols, host);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status dev_gemv_add(hipStream_t s, const double* V, long ldv, int ncols, const double* coef, double* x,
                        long N)
{
    if (ncols <= 0) return ERT_OK;
    hipLaunchKernelGGL(k_gemv, dim3(nblocks(N)), dim3(kBlk), 0, s, V, ldv, ncols, coef, x, N);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status dev_scale(hipStream_t s, double* y, const double* x, double alpha, long N)
{
    hipLaunchKernelGGL(k_scale, dim3(nblocks(N)), dim3(kBlk), 0, s, y, x, alpha, N);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status dev_sub(hipStream_t s, double* y, const double* a, const double* b, long N)
{
    hipLaunchKernelGGL(k_sub, dim3(nblocks(N)), dim3(kBlk), 0, s, y, a, b, N);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status dev_add(hipStream_t s, double* y, const double* x, long N)
{
    hipLaunchKernelGGL(k_add, dim3(nblocks(N)), dim3(kBlk), 0, s, y, x, N);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status dev_zero(hipStream_t s, double* y, long N)
{
    hipLaunchKernelGGL(k_zero, dim3(nblocks(N)), dim3(kBlk), 0, s, y, N);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

}  // namespace ertvie

// ------------------------------------------------------------ level 3 ----
// C = beta C + alpha A B with element strides (A(i,k) = A[i*sAi + k*sAk], ...).
// 64 x 64 output tiles, 4 x 4 per thread, reduction chunks of 16 staged in LDS.
// Long reductions (tall-skinny products) are split over gridDim.z slices whose
// partial tiles go to a workspace and are summed in slice order (deterministic).
namespace ertvie {
namespace {

struct DG {
    int M, N;
    long K;
    double alpha, beta;
    const double* A; long sAi, sAk;
    const double* B; long sBk, sBj;
    double* C; long sCi, sCj;
    double* part;      // split-K workspace [nz][M][N] (row-major), or null
    long kchunk;       // reduction length per slice
};

__global__ __launch_bounds__(256) void k_dgemm(DG g)
{
    __shared__ double As[16][65], Bs[16][65];
    const int i0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const long klo = (long)blockIdx.z * g.kchunk;
    const long khi = (klo + g.kchunk) < g.K ? (klo + g.kchunk) : g.K;
    double acc[4][4] = {};
    for (long k0 = klo; k0 < khi; k0 += 16) {
        for (int e = threadIdx.x; e < 16 * 64; e += 256) {
            const int kk = e / 64, r = e % 64;
            const long k = k0 + kk;
            const int i = i0 + r, j = j0 + r;
            As[kk][r] = (i < g.M && k < khi) ? g.A[i * g.sAi + k * g.sAk] : 0.0;
            Bs[kk][r] = (j < g.N && k < khi) ? g.B[k * g.sBk + j * g.sBj] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            double a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = As[kk][ty * 4 + u];
                b[u] = Bs[kk][tx * 4 + u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] += a[u] * b[v];
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + ty * 4 + u, j = j0 + tx * 4 + v;
            if (i >= g.M || j >= g.N) continue;
            if (g.part) {
                g.part[((long)blockIdx.z * g.M + i) * g.N + j] = acc[u][v];
            } else {
                double* c = g.C + i * g.sCi + j * g.sCj;
                *c = (g.beta == 0.0 ? 0.0 : g.beta * *c) + g.alpha * acc[u][v];
            }
        }
}

__global__ void k_dgemm_reduce(DG g, int nz)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (t >= (long)g.M * g.N) return;
    const int i = (int)(t / g.N), j = (int)(t % g.N);
    double s = 0.0;
    for (int z = 0; z < nz; ++z) s += g.part[((long)z * g.M + i) * g.N + j];
    double* c = g.C + i * g.sCi + j * g.sCj;
    *c = (g.beta == 0.0 ? 0.0 : g.beta * *c) + g.alpha * s;
}

}  // namespace

ert_status dev_dgemm(hipStream_t s, int M, int N, long K, double alpha, const double* A, long sAi, long sAk,
                     const double* B, long sBk, long sBj, double beta, double* C, long sCi, long sCj, double* work,
                     size_t work_elems)
{
    if (M <= 0 || N <= 0) return ERT_OK;
    DG g{M, N, K, alpha, beta, A, sAi, sAk, B, sBk, sBj, C, sCi, sCj, nullptr, K};
    const long tiles = (long)((M + 63) / 64) * ((N + 63) / 64);
    int nz = 1;
    if (tiles < 256 && K > 4096 && work) {
        nz = (int)std::min<long>(std::max<long>(1, 512 / tiles), (K + 4095) / 4096);
        while (nz > 1 && (size_t)nz * M * N > work_elems) --nz;
    }
    if (nz > 1) {
        g.part = work;
        g.kchunk = ((K + nz - 1) / nz + 15) / 16 * 16;
        nz = (int)((K + g.kchunk - 1) / g.kchunk);
    }
    dim3 grid((unsigned)((M + 63) / 64), (unsigned)((N + 63) / 64), (unsigned)nz);
    hipLaunchKernelGGL(k_dgemm, grid, dim3(256), 0, s, g);
    ERT_HIP(hipGetLastError());
    if (nz > 1) {
        const long n = (long)M * N;
        hipLaunchKernelGGL(k_dgemm_reduce, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, nz);
        ERT_HIP(hipGetLastError());
    }
    return ERT_OK;
}

}  // namespace ertvie
