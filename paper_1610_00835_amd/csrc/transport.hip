// Algorithm 1 step S.3: the angular solution Phi(x, v) from U by the
// scattering-free transport equation v . grad Phi + sigma_t Phi = Q,
// Q = sigma_s U + f, with no inflow, solved along characteristics: from each
// cell centre the ray is followed backwards to the boundary of the box
// [0, n_a h]^d in m = ceil(s_b / (h/2)) equal steps (with a 1e-12 relative margin); on each step sigma_t and Q
// take their (clamped d-linear) values at the step midpoint and the step is
// integrated exactly for those constants (step characteristics), so a constant
// medium and source give Q (1 - exp(-sigma_t s_b)) / sigma_t exactly.
//
// One thread per (cell, direction), FP64; the medium and the source are read
// through the d-linear interpolation the kernel's ray rule uses, from boxes of
// the two fields interleaved per cell in LDS.  exp(-tau) is carried as a
// running product of the steps' factors.
#include "common.hpp"

#include <cmath>
#include <mutex>

namespace ertvie {

// Device scratch of the allocation-free entry point (ert_vie_transport_noalloc):
// the interleaved (sigma_t, Q) pairs, 2 N doubles, then the directions, dim * ndir
// doubles.  32.5 MiB per device, held from the library's first use of it on that
// device until the process ends.  Host code never passes this name to a kernel
// or a copy: it uses the device address from hipGetSymbolAddress (scratch_base).
constexpr size_t kTransportScratch = (size_t(1) << 22) + (size_t(1) << 16);   // doubles
static __device__ __align__(256) double scratch[kTransportScratch];

namespace {

// (sigma_t, Q) per cell, interleaved so that one 16-byte load serves both fields
__global__ __launch_bounds__(256) void k_source(const double* __restrict__ U, const double* __restrict__ f,
                                                const double* __restrict__ st, const double* __restrict__ ss, long N,
                                                double2* __restrict__ sq)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i >= N) return;
    sq[i] = make_double2(st[i], (U ? ss[i] * U[i] : 0.0) + (f ? f[i] : 0.0));
}

// Taylor coefficients 1 / (k + 1)! of (1 - exp(-x)) / x in -x, by falling k; a kernel argument so
// that they sit in scalar registers.
struct Phi1 {
    double c[11];
};
constexpr Phi1 kPhi1 = {{1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0,
                         1.0 / 5040.0, 1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5}};

// phi(x) = (1 - exp(-x)) / x for 0 <= x <= 1/4 by its Taylor sum (truncated at 2^-56); to 1 by
// two doublings, phi(2 x) = phi(x) (1 - x phi(x) / 2), of x / 4.
__device__ __forceinline__ double phi1_quarter(const Phi1& f, double x)
{
    double p = f.c[0];
#pragma unroll
    for (int k = 1; k < 11; ++k) p = fma(p, -x, f.c[k]);
    return fma(p, -x, 1.0);
}
__device__ __forceinline__ double phi1_one(const Phi1& f, double x)
{
    const double y = 0.25 * x;
    double p = phi1_quarter(f, y);
    p *= fma(-0.5 * y, p, 1.0);
    return p * fma(-y, p, 1.0);
}

// exp(-x) - 1; a call, so that its constants don't sit in registers through the march
__device__ __noinline__ double thick_step(double x) { return expm1(-x); }

// One step of length D in (sigma_t, Q) = s: att = exp(-tau) before the step.
__device__ __forceinline__ void ray_step(const Phi1& coef, double2 s, double D, double& acc, double& att)
{
    const double sd = s.x * D;
    double step, em;         // integral of exp over the step, exp(-sigma D) - 1
    if (!__ballot(!(sd >= 0.0 && sd <= 0.25))) {
        const double p = phi1_quarter(coef, sd);
        step = D * p;
        em = -sd * p;
    } else if (!__ballot(!(sd >= 0.0 && sd <= 1.0))) {
        const double p = phi1_one(coef, sd);
        step = D * p;
        em = -sd * p;
    } else {
        em = thick_step(sd);
        step = sd > 1e-300 ? -em / s.x : D;
    }
    acc = fma(att * s.y, step, acc);
    att = fma(att, em, att);
}

// A workgroup's cells, 2^s per axis: 8 x 8 x 8 in 3D and 32 x 16 in 2D; grids thinner than that
// give the rest to their longer axes (4 x 128 at most: no side is below kThin + 1).  Compact
// tiles keep the rays of a wave near each other in length (64 cells of a row: a third of the
// steps were idle).
//
// Grids whose shortest side is at most kThin cells take one ray per thread with its samples from
// memory (k_sweep_thin): their rays have a few steps, and staging and its barriers cost more
// than the gathers.  Staged and gathered: 1 x 1 x 4096, 8 directions, 31 and 26 us a call; 2 x 300 x
// 300, 4 directions, 89 and 83; 3 x 300 x 300 129 and 116; 4 x 300 x 300 148 and 163; 2D 2 x 4096
// 31 and 29, 4 x 4096 37 and 38.
constexpr int kThin = 3;
constexpr int kSweepThreads = 512;
constexpr double kSlack = 1e-6;        // cells
constexpr int kSweepCells = 3328;      // staged box, (sigma_t, Q) pairs: three workgroups per CU
struct SweepTile {
    int s[3];
};
SweepTile sweep_tile(const Geo& g)
{
    const int n[3] = {g.n0, g.n1, g.dim > 2 ? g.n2 : 1};
    SweepTile t = g.dim > 2 ? SweepTile{{3, 3, 3}} : SweepTile{{5, 4, 0}};
    for (int a = 0; a < g.dim; ++a)
        while (t.s[a] > 0 && (1 << (t.s[a] - 1)) >= n[a]) {
            --t.s[a];
            int best = -1;
            for (int b = 0; b < g.dim; ++b)
                if (b != a && (1 << t.s[b]) < n[b] && (best < 0 || n[b] >> t.s[b] > n[best] >> t.s[best])) best = b;
            if (best >= 0) ++t.s[best];
        }
    return t;
}

// One ray per thread, window by window in the distance: the cells that the rays of the tile pass
// between distances w W and (w + 1) W (in cells) are a box, staged in LDS before the window, cells
// outside the grid with the value of the face (the clamped rule).  In cells the sample q = 1/2,
// 3/2, .. of cell i sits at i - q e per axis (cell centres are whole numbers); the box allows it
// a rounding of kSlack.  W is the largest whose box fits for this direction, 16 cells at most.
// Bound: FP64 arithmetic (75 instructions per step; a hundred and fifty with clamps, expm1 and a
// division), then LDS reads (eight corners of 16 bytes; as gathers through L1 at half the rate
// they were the bound).  64^3 x 26 directions: 2.46 -> 1.53 ms; 512^2 x 26: 12.5 -> 5.8 ms.
template <int DIM>
__global__ __launch_bounds__(kSweepThreads, 6) void k_sweep(Geo g, SweepTile tile, Phi1 coef,
                                                            const double2* __restrict__ sq,
                                                            const double* __restrict__ dirs, long N,
                                                            double* __restrict__ phi)
{
    __shared__ double2 sl[kSweepCells];
    const int d = blockIdx.y, tid = threadIdx.x;
    const double h = g.h;
    const int n[3] = {g.n0, g.n1, DIM > 2 ? g.n2 : 1};
    int lo[DIM], c[DIM];             // first cell of the tile, cell of the thread
    double v[DIM];
    bool in = true;
    {
        int blk = blockIdx.x, t = tid;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const int nt = (n[a] + (1 << tile.s[a]) - 1) >> tile.s[a];
            lo[a] = (blk % nt) << tile.s[a];
            blk /= nt;
            c[a] = lo[a] + (t & ((1 << tile.s[a]) - 1));
            t >>= tile.s[a];
            in = in && c[a] < n[a];
            v[a] = dirs[DIM * d + a];
        }
        in = in && t == 0;
    }
    // distance backwards along -v to the box boundary
    double sb = 1e300;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const double x = h * (c[a] + 0.5);
        if (v[a] > 0.0) sb = fmin(sb, x / v[a]);
        else if (v[a] < 0.0) sb = fmin(sb, (n[a] * h - x) / (-v[a]));
    }
    // the relative margin keeps the count of an exact multiple of h/2 (every
    // axis-parallel ray) independent of the last bit of sb
    const double q0 = ceil(sb / (0.5 * h) * (1.0 - 1e-12));
    const int m = !in ? 0 : q0 < 1.0 ? 1 : (int)q0;
    const double D = in ? sb / (double)m : h;
    const double per_cell = h / D;   // steps per cell length
    double e[DIM];
#pragma unroll
    for (int a = 0; a < DIM; ++a) e[a] = -D * v[a] / h;
    // the window
    int W = 16;
    for (; W > 1; --W) {
        int vol = 1;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            vol *= (int)((1 << tile.s[a]) - 1 + W * fabs(v[a]) + 2.0 * kSlack) + 3;
        }
        if (vol <= kSweepCells) break;
    }
    double acc = 0.0, att = 1.0;     // att = exp(-tau) before the step
    double q = 0.5;
    int k = 0;
    for (int w = 0;; ++w) {
        // cells low .. low + ext - 1 of the window
        int low[DIM], ext[DIM];
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const int last = lo[a] + (1 << tile.s[a]) - 1, top = last < n[a] - 1 ? last : n[a] - 1;
            const double ta = w * W * v[a], tb = (w + 1) * W * v[a];
            low[a] = (int)floor(lo[a] - fmax(ta, tb) - kSlack);
            ext[a] = (int)floor(top - fmin(ta, tb) + kSlack) + 2 - low[a];
        }
        const int vol = ext[0] * ext[1] * (DIM > 2 ? ext[DIM - 1] : 1);
        if (!__syncthreads_or(k < m)) break;       // also: the previous window's reads are done
        {
            const float i0 = 1.0f / (float)ext[0], i1 = 1.0f / (float)ext[1];
            for (int s = tid; s < vol; s += kSweepThreads) {
                const int row = (int)(((float)s + 0.5f) * i0), x = s - row * ext[0];
                const int z = DIM > 2 ? (int)(((float)row + 0.5f) * i1) : 0, y = row - z * ext[1];
                const int cx = min(max(low[0] + x, 0), n[0] - 1), cy = min(max(low[1] + y, 0), n[1] - 1);
                long at = cx + (long)n[0] * cy;
                if constexpr (DIM > 2) at += (long)n[0] * n[1] * min(max(low[DIM - 1] + z, 0), n[2] - 1);
                sl[s] = sq[at];
            }
        }
        __syncthreads();
        const double end = (w + 1) * W * per_cell + 0.5;
        const int kend = end < (double)m ? (int)end : m;
        const double p1 = (double)ext[0], p2 = (double)(ext[0] * ext[1]);
        const int o1 = ext[0], o2 = ext[0] * ext[1];
        double x0[DIM];
#pragma unroll
        for (int a = 0; a < DIM; ++a) x0[a] = (double)(c[a] - low[a]);
        for (; k < kend; ++k, q += 1.0) {
            double t[DIM], f[DIM];
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                const double u = fma(q, e[a], x0[a]);
                f[a] = floor(u);
                t[a] = u - f[a];
            }
            double at = fma(p1, f[1], f[0]);
            if constexpr (DIM > 2) at = fma(p2, f[DIM - 1], at);
            const double2* b = sl + (int)at;
            auto line = [&](const double2* r) {
                const double2 x = r[0], y = r[1];
                return make_double2(fma(t[0], y.x - x.x, x.x), fma(t[0], y.y - x.y, x.y));
            };
            auto plane = [&](const double2* r) {
                const double2 x = line(r), y = line(r + o1);
                return make_double2(fma(t[1], y.x - x.x, x.x), fma(t[1], y.y - x.y, x.y));
            };
            double2 s = plane(b);
            if constexpr (DIM > 2) {
                const double2 y = plane(b + o2);
                s = make_double2(fma(t[DIM - 1], y.x - s.x, s.x), fma(t[DIM - 1], y.y - s.y, s.y));
            }
            ray_step(coef, s, D, acc, att);
        }
    }
    if (!in) return;
    long j = c[0] + (long)n[0] * c[1];
    if constexpr (DIM > 2) j += (long)n[0] * n[1] * c[DIM - 1];
    phi[(long)d * N + j] = acc;
}

// One ray per thread with its samples from memory: grids of at most kThin cells on some axis.
template <int DIM>
__global__ __launch_bounds__(256) void k_sweep_thin(Geo g, Phi1 coef, const double2* __restrict__ sq,
                                                    const double* __restrict__ dirs, long N, double* __restrict__ phi)
{
    const long j = blockIdx.x * 256L + threadIdx.x;
    if (j >= N) return;
    const int d = blockIdx.y;
    const double h = g.h;
    const int n[3] = {g.n0, g.n1, DIM > 2 ? g.n2 : 1};
    int c[DIM];
    double v[DIM], e[DIM];
    long rest = j;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        c[a] = (int)(rest % n[a]);
        rest /= n[a];
        v[a] = dirs[DIM * d + a];
    }
    // the ray and its steps as in k_sweep (one function for both took 3 more registers to memory there)
    double sb = 1e300;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const double x = h * (c[a] + 0.5);
        if (v[a] > 0.0) sb = fmin(sb, x / v[a]);
        else if (v[a] < 0.0) sb = fmin(sb, (n[a] * h - x) / (-v[a]));
    }
    const double q0 = ceil(sb / (0.5 * h) * (1.0 - 1e-12));
    const int m = q0 < 1.0 ? 1 : (int)q0;
    const double D = sb / (double)m;
#pragma unroll
    for (int a = 0; a < DIM; ++a) e[a] = -D * v[a] / h;
    double acc = 0.0, att = 1.0, q = 0.5;
    for (int k = 0; k < m; ++k, q += 1.0) {
        double t[DIM];
        long at[DIM][2];
        long stride = 1;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const double u = fma(q, e[a], (double)c[a]), f = floor(u);
            const int i = (int)f;
            t[a] = u - f;
            at[a][0] = stride * min(max(i, 0), n[a] - 1);
            at[a][1] = stride * min(max(i + 1, 0), n[a] - 1);
            stride *= n[a];
        }
        auto line = [&](long o) {
            const double2 x = sq[at[0][0] + o], y = sq[at[0][1] + o];
            return make_double2(fma(t[0], y.x - x.x, x.x), fma(t[0], y.y - x.y, x.y));
        };
        auto plane = [&](long o) {
            const double2 x = line(at[1][0] + o), y = line(at[1][1] + o);
            return make_double2(fma(t[1], y.x - x.x, x.x), fma(t[1], y.y - x.y, x.y));
        };
        double2 s = plane(DIM > 2 ? at[DIM - 1][0] : 0);
        if constexpr (DIM > 2) {
            const double2 y = plane(at[DIM - 1][1]);
            s = make_double2(fma(t[DIM - 1], y.x - s.x, s.x), fma(t[DIM - 1], y.y - s.y, s.y));
        }
        ray_step(coef, s, D, acc, att);
    }
    phi[(long)d * N + j] = acc;
}

// Directions (host, ndir x dim): finite unit vectors.
ert_status check_dirs(int dim, const double* dirs_host, int ndir)
{
    for (int d = 0; d < ndir; ++d) {
        double nn = 0.0;
        for (int a = 0; a < dim; ++a) {
            const double c = dirs_host[(size_t)d * dim + a];
            if (!std::isfinite(c)) {
                record_error("ert_vie_transport: non-finite direction");
                return ERT_EINVAL;
            }
            nn += c * c;
        }
        if (std::fabs(nn - 1.0) > 1e-10) {
            record_error("ert_vie_transport: directions must be unit vectors");
            return ERT_EINVAL;
        }
    }
    return ERT_OK;
}

// The sweep with caller-provided device buffers: sq (N pairs) and dd (dim * ndir),
// which receives the directions.  Synchronises the plan's stream before returning
// (the directions are copied from the caller's host array).
ert_status sweep_into(ert_plan_impl* p, const double* U, const double* f, const double* dirs_host, int ndir,
                      double* phi, double2* sq, double* dd)
{
    const long N = p->N;
    const int dim = p->o.dim;
    ert_status st = ERT_HIPST(hipMemcpyAsync(dd, dirs_host, sizeof(double) * dim * (size_t)ndir,
                                             hipMemcpyHostToDevice, p->stream));
    if (st == ERT_OK) {
        hipLaunchKernelGGL(k_source, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, p->stream, U, f, p->d_st,
                           p->d_ss, N, sq);
        st = ERT_HIPST(hipGetLastError());
    }
    const SweepTile tile = sweep_tile(p->geo);
    const int n[3] = {p->geo.n0, p->geo.n1, dim > 2 ? p->geo.n2 : 1};
    const bool thin = std::min(std::min(n[0], n[1]), dim > 2 ? n[2] : n[1]) <= kThin;
    long tiles = 1;
    for (int a = 0; a < dim; ++a) tiles *= (n[a] + (1 << tile.s[a]) - 1) >> tile.s[a];
    // directions in slabs of at most 65535 (grid.y)
    for (int d0 = 0; d0 < ndir && st == ERT_OK; d0 += 65535) {
        const int nd = std::min(65535, ndir - d0);
        if (thin)
            hipLaunchKernelGGL((dim == 2 ? k_sweep_thin<2> : k_sweep_thin<3>), dim3((unsigned)((N + 255) / 256), (unsigned)nd),
                               dim3(256), 0, p->stream, p->geo, kPhi1, sq, dd + (size_t)dim * d0, N, phi + (size_t)d0 * N);
        else
            hipLaunchKernelGGL((dim == 2 ? k_sweep<2> : k_sweep<3>), dim3((unsigned)tiles, (unsigned)nd),
                               dim3(kSweepThreads), 0, p->stream, p->geo, tile, kPhi1, sq, dd + (size_t)dim * d0, N,
                               phi + (size_t)d0 * N);
        st = ERT_HIPST(hipGetLastError());
    }
    const ert_status ss = ERT_HIPST(hipStreamSynchronize(p->stream));
    return st != ERT_OK ? st : ss;
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on device `dev` (made current by the caller), looked
// up once per device.
ert_status scratch_base(int dev, double** out)
{
    if (dev < 0 || dev >= kMaxDevices) {
        record_error("ert_vie_transport_noalloc: device index out of range");
        return ERT_EDEVICE;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            record_hip_error("hipGetSymbolAddress(scratch)", e != hipSuccess ? e : hipErrorInvalidSymbol, __FILE__,
                             __LINE__);
            return ERT_EDEVICE;
        }
        g_scratch_ptr[dev] = static_cast<double*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return ERT_OK;
}

}  // namespace

ert_status transport_sweep(ert_plan_impl* p, const double* U, const double* f, const double* dirs_host, int ndir,
                           double* phi)
{
    ERT_TRY(check_dirs(p->o.dim, dirs_host, ndir));
    const long N = p->N;
    double* buf = nullptr;
    ERT_HIP(hipMalloc(&buf, sizeof(double) * (2 * N + (size_t)p->o.dim * ndir)));
    const ert_status st = sweep_into(p, U, f, dirs_host, ndir, phi, reinterpret_cast<double2*>(buf), buf + 2 * N);
    (void)hipFree(buf);
    return st;
}

ert_status transport_sweep_noalloc(ert_plan_impl* p, const double* U, const double* f, const double* dirs_host,
                                   int ndir, double* phi)
{
    ERT_TRY(check_dirs(p->o.dim, dirs_host, ndir));
    const size_t need = 2 * (size_t)p->N + (size_t)p->o.dim * ndir;
    if (need > kTransportScratch) {
        record_error("ert_vie_transport_noalloc: 2 N + dim * ndir exceeds the scratch of 4259840 doubles");
        return ERT_EINVAL;
    }
    int cur = 0;
    ERT_HIP(hipGetDevice(&cur));
    if (cur != p->device) ERT_HIP(hipSetDevice(p->device));
    double* base = nullptr;
    ert_status st = scratch_base(p->device, &base);
    if (st == ERT_OK)
        st = sweep_into(p, U, f, dirs_host, ndir, phi, reinterpret_cast<double2*>(base), base + 2 * p->N);
    if (cur != p->device) {
        const hipError_t e = hipSetDevice(cur);
        if (st == ERT_OK && e != hipSuccess) {
            record_hip_error("hipSetDevice", e, __FILE__, __LINE__);
            st = ERT_EDEVICE;
        }
    }
    return st;
}

}  // namespace ertvie
