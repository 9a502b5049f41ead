// Diffusion preconditioner (Sec. 4.4, eq. EQ:DA): the diffusion approximation
//   -div(D grad U) + mu_a U = f,  U + l dU/dn = 0,  D = 1/(d sigma_t), l = 2 D,
// models f -> U = (I - K)^{-1} A f, so (I - K)^{-1} = I + (I - K)^{-1} A S is
// approximated by  M r = r + L^{-1} (sigma_s r),  L^{-1} by two V-cycles.
//
// Cell-centred finite differences per unit volume on the solver's grid:
//   (L U)_j = sum_interior faces Df (U_j - U_k) / h^2 + sum_boundary faces 2 D_j / (h (h + 2 l_j)) U_j
//           + mu_a_j U_j,   Df = harmonic mean of D_j, D_k.
// Multigrid: levels by halving each axis (ceil) down to at most 4 cells per
// axis, coarse sigma_t / sigma_s the averages of the children, rediscretised
// with 2h; red-black Gauss-Seidel (red = even i0+i1+i2 first), 2 sweeps before
// and after the coarse correction; restriction by averaging the children,
// constant prolongation; 60 sweeps on the coarsest level.  All FP64.
//
// How a cycle runs.  The work is a few hundred dependent half-sweeps over small
// arrays, so what bounds it is the number of dependent launches:
//  - The cycle below a level of at most kDenseCells cells, started from zero, is a
//    fixed linear map of the level's right-hand side.  Its matrix is formed once,
//    one unit vector per workgroup (k_small_matrix), and every cycle then applies
//    it as one matrix-vector product (k_dense) instead of about 170 dependent
//    half-sweeps of one workgroup (177 us at 2D 264^2).
//  - 2D levels above it take one launch down (both pre-sweeps, residual and
//    restriction) and one up (prolongation and both post-sweeps) over LDS tiles with
//    a halo as wide as the half-sweeps reach (k_tile), instead of five and five.
//    With both, a 2D 264^2 solve of 10 steps takes 2.05 ms instead of 10.7.
//  - In 3D such tiles would be mostly halo (an 8^3 tile of an 18^3 box), so the
//    larger levels keep one launch per half-sweep.
// Face coefficients are stored divided by h^2 and the smoother multiplies by the
// inverse diagonal.  Cells and threads are 32-bit: a plan has at most 2^30 cells.
#include "common.hpp"

#include <algorithm>
#include <vector>

namespace ertvie {

struct DiffLevel {
    int n[3] = {1, 1, 1};
    double h = 0.0;
    long N = 0;
    double* st = nullptr;
    double* ss = nullptr;
    double* idiag = nullptr;                       // 1 / diagonal
    double* df[3] = {nullptr, nullptr, nullptr};   // face to the upper neighbour along axis a, over h^2
    double* U = nullptr;                           // iterate after the pre-sweeps
    double* V = nullptr;                           // 2D: iterate after the post-sweeps (tiles read U's halos)
    double* B = nullptr;
};

struct DiffPc {
    int dim = 0;
    std::vector<DiffLevel> lv;
    int dense = 0;               // level whose cycle is the matrix `mat`
    double* mat = nullptr;       // [n][n], row major, n = cells of level `dense`
    long bytes = 0;
};

namespace {

constexpr int kPre = 2, kPost = 2, kCoarseSweeps = 60, kCoarsest = 4, kCycles = 2;

constexpr int kDenseCells = 512;   // 2 MB of matrix; one thread per cell of a workgroup forms its columns
constexpr int kMaxSmall = 8;       // levels of at most kDenseCells cells (a 512 x 1 grid has 8)

struct LvArgs {
    int dim, n0, n1, n2;
    double h;
    const double* st;
    const double* ss;
    double* idiag;
    double* dfx;
    double* dfy;
    double* dfz;
};

__device__ __forceinline__ void unravel(long j, int n0, int n1, int i[3])
{
    i[0] = (int)(j % n0);
    i[1] = (int)((j / n0) % n1);
    i[2] = (int)(j / ((long)n0 * n1));
}

__global__ void k_avg_children(int dim, int f0, int f1, int f2, const double* __restrict__ fine, int c0, int c1,
                               int c2, double* __restrict__ coarse)
{
    const long c = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (c >= (long)c0 * c1 * c2) return;
    int ic[3];
    unravel(c, c0, c1, ic);
    double s = 0.0;
    int cnt = 0;
    for (int oz = 0; oz < (dim > 2 ? 2 : 1); ++oz)
        for (int oy = 0; oy < 2; ++oy)
            for (int ox = 0; ox < 2; ++ox) {
                const int a = 2 * ic[0] + ox, b = 2 * ic[1] + oy, z = 2 * ic[2] + oz;
                if (a < f0 && b < f1 && z < f2) {
                    s += fine[a + (long)f0 * (b + (long)f1 * z)];
                    ++cnt;
                }
            }
    coarse[c] = s / cnt;
}

__global__ void k_faces(LvArgs a)
{
    const long N = (long)a.n0 * a.n1 * a.n2;
    const long j = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (j >= N) return;
    int i[3];
    unravel(j, a.n0, a.n1, i);
    const int n[3] = {a.n0, a.n1, a.n2};
    const long s[3] = {1, a.n0, (long)a.n0 * a.n1};
    double* df[3] = {a.dfx, a.dfy, a.dfz};
    const double Dj = 1.0 / (a.dim * a.st[j]);
    for (int ax = 0; ax < 3; ++ax) {
        double v = 0.0;
        if (ax < a.dim && i[ax] < n[ax] - 1) {
            const double Dk = 1.0 / (a.dim * a.st[j + s[ax]]);
            v = 2.0 * Dj * Dk / (Dj + Dk) / (a.h * a.h);
        }
        df[ax][j] = v;
    }
}

__global__ void k_diag(LvArgs a)
{
    const long N = (long)a.n0 * a.n1 * a.n2;
    const long j = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (j >= N) return;
    int i[3];
    unravel(j, a.n0, a.n1, i);
    const int n[3] = {a.n0, a.n1, a.n2};
    const long s[3] = {1, a.n0, (long)a.n0 * a.n1};
    const double* df[3] = {a.dfx, a.dfy, a.dfz};
    const double Dj = 1.0 / (a.dim * a.st[j]);
    const double rob = 2.0 * Dj / (a.h * (a.h + 4.0 * Dj));
    double d = a.st[j] - a.ss[j];
    for (int ax = a.dim - 1; ax >= 0; --ax) {
        if (i[ax] < n[ax] - 1) d += df[ax][j];
        if (i[ax] > 0) d += df[ax][j - s[ax]];
        if (i[ax] == 0) d += rob;
        if (i[ax] == n[ax] - 1) d += rob;
    }
    a.idiag[j] = 1.0 / d;
}

// sum over interior faces of (Df / h^2) U_k (a face on the boundary has a zero coefficient)
__device__ __forceinline__ double offdiag(const LvArgs& a, const double* U, int j, int x, int y, int z)
{
    double o = 0.0;
    if (a.dim > 2) {
        const int s2 = a.n0 * a.n1;
        if (z < a.n2 - 1) o += a.dfz[j] * U[j + s2];
        if (z > 0) o += a.dfz[j - s2] * U[j - s2];
    }
    if (y < a.n1 - 1) o += a.dfy[j] * U[j + a.n0];
    if (y > 0) o += a.dfy[j - a.n0] * U[j - a.n0];
    if (x < a.n0 - 1) o += a.dfx[j] * U[j + 1];
    if (x > 0) o += a.dfx[j - 1] * U[j - 1];
    return o;
}

// One colour of a 3D level: thread = one cell of the colour (two per x pair).
__global__ __launch_bounds__(256) void k_rbgs(LvArgs a, double* __restrict__ U, const double* __restrict__ B,
                                              int colour)
{
    const int hx = (a.n0 + 1) / 2;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= hx * a.n1 * a.n2) return;
    const int r = t / hx, y = r % a.n1, z = r / a.n1;
    const int x = 2 * (t - r * hx) + ((y + z + colour) & 1);
    if (x >= a.n0) return;
    const int j = x + a.n0 * r;
    U[j] = (B[j] + offdiag(a, U, j, x, y, z)) * a.idiag[j];
}

// B_c = average over the children of the residual B - (diag U - offdiag U), and U_c = 0
// (the coarser correction starts from zero).
__global__ __launch_bounds__(256) void k_restrict_residual(LvArgs a, const double* __restrict__ U,
                                                           const double* __restrict__ B, int c0, int c1, int c2,
                                                           double* __restrict__ Bc, double* __restrict__ Uc)
{
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= c0 * c1 * c2) return;
    const int r = q / c0, qx = q - r * c0, qy = r % c1, qz = r / c1;
    double s = 0.0;
    int cnt = 0;
    for (int o = 0; o < 8; ++o) {
        const int x = 2 * qx + (o & 1), y = 2 * qy + ((o >> 1) & 1), z = 2 * qz + (o >> 2);
        if (x >= a.n0 || y >= a.n1 || z >= a.n2) continue;
        const int j = x + a.n0 * (y + a.n1 * z);
        s += B[j] - (U[j] / a.idiag[j] - offdiag(a, U, j, x, y, z));
        ++cnt;
    }
    Bc[q] = s / cnt;
    Uc[q] = 0.0;
}

__global__ void k_prolong_add(int f0, int f1, int f2, double* __restrict__ Uf, int c0, int c1,
                              const double* __restrict__ Ec)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= f0 * f1 * f2) return;
    const int r = j / f0, x = j - r * f0, y = r % f1, z = r / f1;
    Uf[j] += Ec[x / 2 + c0 * (y / 2 + c1 * (z / 2))];
}

// ------------------------------------------------------------- 2D tiles ----

// One half of a cycle on a 2D level.  A workgroup owns a TILE x TILE tile and holds
// the tile and a halo of kHalo cells in LDS (iterate) and registers (right-hand side
// and coefficients of its cells).  The four half-sweeps run on the whole box; a
// half-sweep spoils one more ring of cells, counted from the box's edge, and the
// residual reads one ring further, so the tile's own values are exact.
//   down (UP = false): U_out = smooth(U_in) (U_in = 0 when null), and the restricted
//     residual to Bc.  The black cells' residual is zero after the last half-sweep.
//     With r, the right-hand side is ss r, formed here and stored to Bout.
//   up (UP = true): U_out = smooth(U_in + prolong(Ec)); with r, U_out receives
//     r + that (the preconditioner's output; r and U_out may be the same buffer).
// Neighbouring tiles read each other's U_in, so U_out is another buffer.
// Bound: launch latency, the load of a cell's nine values and the four barriers.  Tiles of 16
// cells, one cell of the box per thread, spread a level over the chip: 264^2, 66 us per
// application (18 launches); 86 us with tiles of 32 and two cells per thread, 150 us with
// seven.  The larger tile pays where a level has more of them than the chip holds at once
// (2048^2: 414 against 562 us): its halo doubles a cell's traffic instead of tripling it.
constexpr int kHalo = 5;
constexpr long kLargeLevel = 400000;              // cells
template <int TILE_, int THREADS_>
struct TileForm {
    static constexpr int TILE = TILE_, THREADS = THREADS_;
    static constexpr int BOX = TILE + 2 * kHalo, PITCH = BOX + 1, PER = (BOX * BOX + THREADS - 1) / THREADS;
};
using TileSmall = TileForm<16, 704>;
using TileLarge = TileForm<32, 1024>;

template <bool UP, typename F>
__global__ __launch_bounds__(F::THREADS) void k_tile(LvArgs a, const double* Uin, const double* Bin, const double* r,
                                              const double* __restrict__ ss, int c0, int c1,
                                              const double* __restrict__ Ec, double* Uout, double* Bout,
                                              double* __restrict__ Bc)
{
    constexpr int kTile = F::TILE, kTileThreads = F::THREADS, kBox = F::BOX, kPitch = F::PITCH, kBoxPer = F::PER;
    __shared__ double u[kBox * kPitch];
    __shared__ double res[UP ? 1 : kTile * (kTile + 1)];
    const int tx0 = blockIdx.x * kTile, ty0 = blockIdx.y * kTile;
    double b[kBoxPer], id[kBoxPer], ce[kBoxPer], cw[kBoxPer], cn[kBoxPer], cs[kBoxPer];
    int at[kBoxPer];                              // LDS index
    unsigned red = 0, upd = 0;                    // bit k: cell k is red, is updated by the sweeps
#pragma unroll
    for (int k = 0; k < kBoxPer; ++k) {
        const int e = threadIdx.x + kTileThreads * k;
        const int ex = e % kBox, ey = e / kBox, x = tx0 + ex - kHalo, y = ty0 + ey - kHalo;
        const bool box = e < kBox * kBox;
        const bool in = box && x >= 0 && x < a.n0 && y >= 0 && y < a.n1;
        const int j = in ? x + a.n0 * y : 0;
        at[k] = ex + kPitch * ey;
        double v = 0.0;
        b[k] = id[k] = ce[k] = cw[k] = cn[k] = cs[k] = 0.0;
        if (in) {
            if (UP) v = Uin[j] + Ec[(x >> 1) + c0 * (y >> 1)];
            else if (Uin) v = Uin[j];
            b[k] = (!UP && r) ? ss[j] * r[j] : Bin[j];
            id[k] = a.idiag[j];
            ce[k] = a.dfx[j];
            cn[k] = a.dfy[j];
            if (x > 0) cw[k] = a.dfx[j - 1];
            if (y > 0) cs[k] = a.dfy[j - a.n0];
        }
        if (box) u[at[k]] = v;
        if (in && ex > 0 && ex < kBox - 1 && ey > 0 && ey < kBox - 1) upd |= 1u << k;
        if (((x + y) & 1) == 0) red |= 1u << k;
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2 * (UP ? kPost : kPre); ++h) {
        const unsigned todo = upd & ((h & 1) ? ~red : red);
#pragma unroll
        for (int k = 0; k < kBoxPer; ++k)
            if (todo >> k & 1u) {
                const int i = at[k];
                const double o = cn[k] * u[i + kPitch] + cs[k] * u[i - kPitch] + ce[k] * u[i + 1] + cw[k] * u[i - 1];
                u[i] = (b[k] + o) * id[k];
            }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kBoxPer; ++k) {
        const int e = threadIdx.x + kTileThreads * k;
        const int ex = e % kBox - kHalo, ey = e / kBox - kHalo, x = tx0 + ex, y = ty0 + ey;
        if (e >= kBox * kBox || ex < 0 || ex >= kTile || ey < 0 || ey >= kTile) continue;
        double rv = 0.0;
        if (x < a.n0 && y < a.n1) {
            const int j = x + a.n0 * y, i = at[k];
            if (UP) {
                Uout[j] = r ? r[j] + u[i] : u[i];
            } else {
                Uout[j] = u[i];
                if (r) Bout[j] = b[k];
                if (red >> k & 1u) {
                    const double o =
                        cn[k] * u[i + kPitch] + cs[k] * u[i - kPitch] + ce[k] * u[i + 1] + cw[k] * u[i - 1];
                    rv = b[k] - (u[i] / id[k] - o);
                }
            }
        }
        if (!UP) res[ex + (kTile + 1) * ey] = rv;
    }
    if (UP) return;
    __syncthreads();
    const int qx = threadIdx.x % (kTile / 2), qy = threadIdx.x / (kTile / 2);
    const int X = tx0 / 2 + qx, Y = ty0 / 2 + qy;
    if (qy >= kTile / 2 || X >= c0 || Y >= c1) return;
    const double* p = res + 2 * qx + (kTile + 1) * 2 * qy;
    const int cnt = (2 * X + 1 < a.n0 ? 2 : 1) * (2 * Y + 1 < a.n1 ? 2 : 1);
    Bc[X + c0 * Y] = (p[0] + p[1] + p[kTile + 1] + p[kTile + 2]) / cnt;
}

// ---------------------------------------------------------- dense levels ----

struct SmallLevels {
    int nl;                       // levels from the dense one down to the coarsest
    int cycles;                   // 1; 2 when the dense level is the finest (both cycles in the matrix)
    LvArgs a[kMaxSmall];
};

__device__ __forceinline__ void small_rbgs(const LvArgs& a, int N, double* U, const double* B, int sweeps)
{
    for (int sw = 0; sw < sweeps; ++sw)
        for (int colour = 0; colour < 2; ++colour) {
            for (int j = threadIdx.x; j < N; j += blockDim.x) {
                const int r = j / a.n0, x = j - r * a.n0, y = r % a.n1, z = r / a.n1;
                if (((x + y + z) & 1) == colour) U[j] = (B[j] + offdiag(a, U, j, x, y, z)) * a.idiag[j];
            }
            __syncthreads();
        }
}

// Column blockIdx.x of the cycle's matrix: the cycle(s) from zero for that unit vector.
__global__ __launch_bounds__(kDenseCells) void k_small_matrix(SmallLevels c, double* __restrict__ mat)
{
    __shared__ double Us[2 * kDenseCells], Bs[2 * kDenseCells];   // sum of the levels' cells < 2 kDenseCells
    int off[kMaxSmall], cells[kMaxSmall], total = 0;
    for (int k = 0; k < c.nl; ++k) {
        off[k] = total;
        cells[k] = c.a[k].n0 * c.a[k].n1 * c.a[k].n2;
        total += cells[k];
    }
    for (int j = threadIdx.x; j < total; j += blockDim.x) {
        Us[j] = 0.0;
        Bs[j] = j == (int)blockIdx.x ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int cy = 0; cy < c.cycles; ++cy) {
        for (int k = 0; k + 1 < c.nl; ++k) {
            const LvArgs& a = c.a[k];
            const LvArgs& q = c.a[k + 1];
            double *U = Us + off[k], *B = Bs + off[k];
            small_rbgs(a, cells[k], U, B, kPre);
            for (int t = threadIdx.x; t < cells[k + 1]; t += blockDim.x) {
                const int r = t / q.n0, qx = t - r * q.n0, qy = r % q.n1, qz = r / q.n1;
                double s = 0.0;
                int cnt = 0;
                for (int o = 0; o < 8; ++o) {
                    const int x = 2 * qx + (o & 1), y = 2 * qy + ((o >> 1) & 1), z = 2 * qz + (o >> 2);
                    if (x >= a.n0 || y >= a.n1 || z >= a.n2) continue;
                    const int j = x + a.n0 * (y + a.n1 * z);
                    s += B[j] - (U[j] / a.idiag[j] - offdiag(a, U, j, x, y, z));
                    ++cnt;
                }
                Bs[off[k + 1] + t] = s / cnt;
                Us[off[k + 1] + t] = 0.0;
            }
            __syncthreads();
        }
        small_rbgs(c.a[c.nl - 1], cells[c.nl - 1], Us + off[c.nl - 1], Bs + off[c.nl - 1], kCoarseSweeps);
        for (int k = c.nl - 2; k >= 0; --k) {
            const LvArgs& a = c.a[k];
            const LvArgs& q = c.a[k + 1];
            double* U = Us + off[k];
            for (int j = threadIdx.x; j < cells[k]; j += blockDim.x) {
                const int r = j / a.n0, x = j - r * a.n0, y = r % a.n1, z = r / a.n1;
                U[j] += Us[off[k + 1] + x / 2 + q.n0 * (y / 2 + q.n1 * (z / 2))];
            }
            __syncthreads();
            small_rbgs(a, cells[k], U, Bs + off[k], kPost);
        }
    }
    for (int j = threadIdx.x; j < cells[0]; j += blockDim.x) mat[(long)j * cells[0] + blockIdx.x] = Us[j];
}

// y = mat b, one wave per row.  FINEST: y = r + mat (ss r), the whole preconditioner of a
// grid of at most kDenseCells cells; r and y may be the same buffer, so one workgroup
// reads all of r before it writes.
template <bool FINEST>
__global__ __launch_bounds__(FINEST ? 1024 : 256) void k_dense(const double* __restrict__ mat, int n, const double* b,
                                                              const double* __restrict__ ss, double* y)
{
    __shared__ double sb[kDenseCells];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int i = threadIdx.x; i < n; i += blockDim.x) sb[i] = FINEST ? ss[i] * b[i] : b[i];
    __syncthreads();
    for (int row = blockIdx.x * nw + wave; row < n; row += gridDim.x * nw) {
        const double* m = mat + (long)row * n;
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < kDenseCells / 64; ++k) {
            const int i = 64 * k + lane;
            if (i < n) s += m[i] * sb[i];
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) s += __shfl_xor(s, d, 64);
        if (lane == 0) y[row] = FINEST ? b[row] + s : s;
    }
}

__global__ void k_scaled(const double* __restrict__ r, const double* __restrict__ ss, long N, double* __restrict__ b,
                         double* __restrict__ u)
{
    const long j = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (j >= N) return;
    b[j] = ss[j] * r[j];
    u[j] = 0.0;
}

__global__ void k_add_out(const double* r, const double* __restrict__ u, long N, double* z)
{
    const long j = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (j < N) z[j] = r[j] + u[j];
}

inline unsigned nblk(long n) { return (unsigned)((n + 255) / 256); }

LvArgs args_of(const DiffPc* d, const DiffLevel& L)
{
    return LvArgs{d->dim, L.n[0], L.n[1], L.n[2], L.h, L.st, L.ss, L.idiag, L.df[0], L.df[1], L.df[2]};
}

ert_status dense(hipStream_t s, DiffPc* d)
{
    DiffLevel& L = d->lv[d->dense];
    hipLaunchKernelGGL(k_dense<false>, dim3((unsigned)((L.N + 3) / 4)), dim3(256), 0, s, (const double*)d->mat, (int)L.N,
                       (const double*)L.B, (const double*)nullptr, d->dim == 2 ? L.V : L.U);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

template <bool UP, typename F>
void launch_tile(hipStream_t s, const LvArgs& a, const double* Uin, const double* B, const double* r, const double* ss,
                 const DiffLevel& C, const double* Ec, double* Uout, double* Bout, double* Bc)
{
    const dim3 grid((unsigned)((a.n0 + F::TILE - 1) / F::TILE), (unsigned)((a.n1 + F::TILE - 1) / F::TILE));
    hipLaunchKernelGGL((k_tile<UP, F>), grid, dim3(F::THREADS), 0, s, a, Uin, B, r, ss, C.n[0], C.n[1], Ec, Uout, Bout, Bc);
}

// One cycle from level k down in 2D.  first: the iterate starts at zero; r (finest level
// only): the residual the preconditioner acts on; out: r + U instead of the level's V.
ert_status vcycle2(hipStream_t s, DiffPc* d, int k, bool first, const double* r, double* out)
{
    if (k == d->dense) return dense(s, d);
    DiffLevel& L = d->lv[k];
    DiffLevel& C = d->lv[k + 1];
    const LvArgs a = args_of(d, L);
    const bool large = L.N >= kLargeLevel;
    const auto down = large ? launch_tile<false, TileLarge> : launch_tile<false, TileSmall>;
    const auto up = large ? launch_tile<true, TileLarge> : launch_tile<true, TileSmall>;
    down(s, a, first ? nullptr : L.V, L.B, first ? r : nullptr, L.ss, C, nullptr, L.U, L.B, C.B);
    ERT_HIP(hipGetLastError());
    ERT_TRY(vcycle2(s, d, k + 1, true, nullptr, nullptr));
    up(s, a, L.U, L.B, out ? r : nullptr, nullptr, C, C.V, out ? out : L.V, nullptr, nullptr);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status vcycle3(hipStream_t s, DiffPc* d, int k)
{
    if (k == d->dense) return dense(s, d);
    DiffLevel& L = d->lv[k];
    DiffLevel& C = d->lv[k + 1];
    const LvArgs a = args_of(d, L);
    const dim3 half(nblk((long)((L.n[0] + 1) / 2) * L.n[1] * L.n[2]));
    for (int h = 0; h < 2 * kPre; ++h)
        hipLaunchKernelGGL(k_rbgs, half, dim3(256), 0, s, a, L.U, (const double*)L.B, h & 1);
    hipLaunchKernelGGL(k_restrict_residual, dim3(nblk(C.N)), dim3(256), 0, s, a, (const double*)L.U,
                       (const double*)L.B, C.n[0], C.n[1], C.n[2], C.B, C.U);
    ERT_HIP(hipGetLastError());
    ERT_TRY(vcycle3(s, d, k + 1));
    hipLaunchKernelGGL(k_prolong_add, dim3(nblk(L.N)), dim3(256), 0, s, L.n[0], L.n[1], L.n[2], L.U, C.n[0], C.n[1],
                       (const double*)C.U);
    for (int h = 0; h < 2 * kPost; ++h)
        hipLaunchKernelGGL(k_rbgs, half, dim3(256), 0, s, a, L.U, (const double*)L.B, h & 1);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status diffpc_build(ert_plan_impl* p)
{
    if (p->diffpc) return ERT_OK;
    DiffPc* d = new DiffPc();
    d->dim = p->o.dim;
    hipStream_t s = p->stream;
    int n[3] = {p->geo.n0, p->geo.n1, d->dim == 3 ? p->geo.n2 : 1};
    double h = p->geo.h;
    ert_status st = ERT_OK;
    auto alloc = [&](double** q, long cnt) {
        if (st != ERT_OK) return;
        if (hipMalloc(q, sizeof(double) * std::max<long>(1, cnt)) != hipSuccess) {
            record_error("diffusion preconditioner: allocation failed");
            st = ERT_ENOMEM;
        }
        d->bytes += sizeof(double) * cnt;
    };
    while (st == ERT_OK) {
        DiffLevel L;
        for (int a = 0; a < 3; ++a) L.n[a] = n[a];
        L.h = h;
        L.N = (long)n[0] * n[1] * n[2];
        alloc(&L.st, L.N);
        alloc(&L.ss, L.N);
        alloc(&L.idiag, L.N);
        for (int a = 0; a < 3; ++a) alloc(&L.df[a], L.N);
        alloc(&L.U, L.N);
        if (d->dim == 2) alloc(&L.V, L.N);
        alloc(&L.B, L.N);
        d->lv.push_back(L);
        if (st != ERT_OK) break;
        const int mx = std::max(n[0], std::max(n[1], n[2]));
        if (mx <= kCoarsest) break;
        for (int a = 0; a < 3; ++a) n[a] = (n[a] + 1) / 2;
        h *= 2.0;
    }
    long nd = 0;
    if (st == ERT_OK) {
        while (d->lv[d->dense].N > kDenseCells) ++d->dense;   // the coarsest has at most 4^3
        nd = d->lv[d->dense].N;
        alloc(&d->mat, nd * nd);
    }
    if (st == ERT_OK) {
        DiffLevel& L0 = d->lv[0];
        st = ERT_HIPST(hipMemcpyAsync(L0.st, p->d_st, sizeof(double) * L0.N, hipMemcpyDeviceToDevice, s));
        if (st == ERT_OK)
            st = ERT_HIPST(hipMemcpyAsync(L0.ss, p->d_ss, sizeof(double) * L0.N, hipMemcpyDeviceToDevice, s));
        for (size_t k = 1; k < d->lv.size() && st == ERT_OK; ++k) {
            DiffLevel& F = d->lv[k - 1];
            DiffLevel& C = d->lv[k];
            hipLaunchKernelGGL(k_avg_children, dim3(nblk(C.N)), dim3(256), 0, s, d->dim, F.n[0], F.n[1], F.n[2],
                               (const double*)F.st, C.n[0], C.n[1], C.n[2], C.st);
            hipLaunchKernelGGL(k_avg_children, dim3(nblk(C.N)), dim3(256), 0, s, d->dim, F.n[0], F.n[1], F.n[2],
                               (const double*)F.ss, C.n[0], C.n[1], C.n[2], C.ss);
            st = ERT_HIPST(hipGetLastError());
        }
        for (size_t k = 0; k < d->lv.size() && st == ERT_OK; ++k) {
            const LvArgs a = args_of(d, d->lv[k]);
            hipLaunchKernelGGL(k_faces, dim3(nblk(d->lv[k].N)), dim3(256), 0, s, a);
            hipLaunchKernelGGL(k_diag, dim3(nblk(d->lv[k].N)), dim3(256), 0, s, a);
            st = ERT_HIPST(hipGetLastError());
        }
        if (st == ERT_OK) {
            SmallLevels c{};
            c.nl = (int)d->lv.size() - d->dense;
            c.cycles = d->dense == 0 ? kCycles : 1;
            for (int q = 0; q < c.nl; ++q) c.a[q] = args_of(d, d->lv[d->dense + q]);
            hipLaunchKernelGGL(k_small_matrix, dim3((unsigned)nd), dim3(kDenseCells), 0, s, c, d->mat);
            st = ERT_HIPST(hipGetLastError());
        }
        if (st == ERT_OK) st = ERT_HIPST(hipStreamSynchronize(s));
    }
    if (st != ERT_OK) {
        diffpc_destroy(d);
        return st;
    }
    p->diffpc = d;
    return ERT_OK;
}

}  // namespace

void diffpc_destroy(DiffPc* d)
{
    if (!d) return;
    for (auto& L : d->lv) {
        (void)hipFree(L.st);
        (void)hipFree(L.ss);
        (void)hipFree(L.idiag);
        for (auto* q : L.df) (void)hipFree(q);
        (void)hipFree(L.U);
        (void)hipFree(L.V);
        (void)hipFree(L.B);
    }
    (void)hipFree(d->mat);
    delete d;
}

ert_status diffpc_apply(ert_plan_impl* p, const double* r, double* z, int nrhs)
{
    ERT_TRY(diffpc_build(p));
    DiffPc* d = p->diffpc;
    hipStream_t s = p->stream;
    DiffLevel& L0 = d->lv[0];
    for (int c = 0; c < nrhs; ++c) {
        const double* rc = r + (size_t)c * p->N;
        double* zc = z + (size_t)c * p->N;
        if (d->dense == 0) {
            hipLaunchKernelGGL(k_dense<true>, dim3(1), dim3(1024), 0, s, (const double*)d->mat, (int)p->N, rc,
                               (const double*)p->d_ss, zc);
            ERT_HIP(hipGetLastError());
        } else if (d->dim == 2) {
            for (int cy = 0; cy < kCycles; ++cy)
                ERT_TRY(vcycle2(s, d, 0, cy == 0, rc, cy + 1 == kCycles ? zc : nullptr));
        } else {
            hipLaunchKernelGGL(k_scaled, dim3(nblk(p->N)), dim3(256), 0, s, rc, (const double*)p->d_ss, p->N, L0.B, L0.U);
            for (int cy = 0; cy < kCycles; ++cy) ERT_TRY(vcycle3(s, d, 0));
            hipLaunchKernelGGL(k_add_out, dim3(nblk(p->N)), dim3(256), 0, s, rc, (const double*)L0.U, p->N, zc);
            ERT_HIP(hipGetLastError());
        }
    }
    return ERT_OK;
}

}  // namespace ertvie
