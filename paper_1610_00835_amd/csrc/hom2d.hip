// FP64 apply of a homogeneous 2D medium (leaves of 8 x 8 cells): the multilevel passes of
// Sec. 3.3 in a few launches.
//
// A 2D level is small (64 values per leaf, n^2 <= 64 nodes per box), so an apply is
// bound by its chain of dependent launches, not by its arithmetic: with one launch
// per pass and level (gather, P2M, M2M, compression, translation, sum, expansion, L2L,
// L2P, assembly) 512^2 took 31 launches, 231 us, and 64^2 14 launches, 78 us.  Here
//   up       a workgroup takes a box two levels above the leaves with its 16 leaves: weighted
//            charges, P2M, and M2M over both levels in LDS; then the same from there,
//            two levels per launch, up to level 2;
//   products the translations of all levels and the near field, which depend on
//            nothing but the up pass, in one launch on the matrix cores;
//   down     two levels of L2L per launch; the last one goes on to L2P, adds the near
//            field and assembles y.
// 512^2 (order 6): 5 launches, 231 -> 63 us; 64^2 (order 8): 3 launches, 78 -> 30 us; 2048^2
// (order 8) 1380 -> 1180 us, now bound by the FP64 matrix pipe (24 GFLOP).  64 right-hand
// sides: 64^2 147 -> 133 us, 512^2 (order 6) 3.65 -> 1.88 ms.
//
// The compressed translations U C_o U^T (shared basis U per level) act here as the full
// matrices of the same map, n^2 x n^2, formed once at plan time: the compression and
// expansion passes go, and n^2 is at most twice the rank.
#include <algorithm>

#include "fmm.hpp"

namespace ertvie {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kCells = 64;                     // cells per leaf
constexpr int kSubMax = 16;                    // boxes of the lowest level in a workgroup

// Matrix fragments: [matrix][row tile][step s][lane], the entry of row 16 rt + lane % 16 and
// column (lane / 16) KS + s (KS = columns / 4): a lane's four-column groups are consecutive
// in its source vector, and a wave reads a fragment as one line of 512 bytes.
__global__ void k_fragments(const double* __restrict__ src, int ld, int K, int KS, int RT, long nmat,
                            double* __restrict__ dst)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const long per = (long)RT * KS * 64;
    if (i >= nmat * per) return;
    const long m = i / per;
    const int e = (int)(i - m * per), lane = e & 63, s = (e >> 6) % KS, rt = (e >> 6) / KS;
    const int r = 16 * rt + (lane & 15), c = (lane >> 4) * KS + s;
    dst[i] = (r < K && c < K) ? src[(m * ld + r) * ld + c] : 0.0;
}

// A box of level `low` in the workgroup's subtree: group g of 64 threads, depth = low - top.
struct SubBox {
    int x, y;
    bool ok;
};
__device__ __forceinline__ SubBox sub_box(const Hom2d& t, int top, int level, int g)
{
    const int j = level - top, side = 1 << j;
    const int bx = blockIdx.x % t.nl0[top], by = blockIdx.x / t.nl0[top];
    SubBox b;
    b.x = (bx << j) + (g & (side - 1));
    b.y = (by << j) + (g >> j);
    b.ok = b.x < t.nl0[level] && b.y < t.nl1[level];
    return b;
}

// Up pass from level `low` to level `top`; LEAVES: low = L, from the charges.
template <bool LEAVES>
__global__ __launch_bounds__(64 * kSubMax) void k_up(Hom2dUp u)
{
    __shared__ double cur[kSubMax][64], tmp[kSubMax][64], P[64], M[128];
    const Hom2d& t = u.t;
    if (LEAVES && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *u.io = u.a;
    const int tid = threadIdx.x, g = tid >> 6, lane = tid & 63, rhs = blockIdx.y;
    const int nc = t.nc, K = t.K, low = u.low, top = u.top;
    for (int i = tid; i < 2 * nc * nc; i += blockDim.x) M[i] = t.M1[i];
    const SubBox b = sub_box(t, top, low, g);
    const long box = b.x + (long)t.nl0[low] * b.y;
    double* Wl = t.W[low] + ((long)rhs * t.nl0[low] * t.nl1[low] + box) * t.ld;
    if constexpr (LEAVES) {
        for (int i = tid; i < 8 * nc; i += blockDim.x) P[i] = t.P1[i];
        const int x = 8 * b.x + (lane & 7), y = 8 * b.y + (lane >> 3);
        double v = 0.0;
        if (b.ok && x < t.n0 && y < t.n1) {
            const long j = x + (long)t.n0 * y;
            const double xv = u.a.x[(long)rhs * t.N + j];
            v = u.a.op != ERT_OP_G ? u.ss[j] * xv : xv;
        }
        cur[g][lane] = v;
        if (b.ok) t.q[((long)rhs * t.nl0[low] * t.nl1[low] + box) * kCells + lane] = v;
        __syncthreads();
        if (lane < 8 * nc) {
            const int m0 = lane % nc, row = lane / nc;
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) s += P[m0 * 8 + i] * cur[g][row * 8 + i];
            tmp[g][lane] = s;
        }
        __syncthreads();
        if (lane < K) {
            const int m0 = lane % nc, m1 = lane / nc;
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) s += P[m1 * 8 + i] * tmp[g][i * nc + m0];
            cur[g][lane] = s;
            if (b.ok) Wl[lane] = s;
        }
    } else {
        if (lane < K) cur[g][lane] = b.ok ? Wl[lane] : 0.0;
    }
    __syncthreads();
    for (int j = low - top - 1; j >= 0; --j) {
        const int np = 1 << (2 * j), side = 1 << j;
        double* z = &tmp[0][0];                 // [parent][cy][k1][m0]
        for (int e = tid; e < np * 2 * K; e += blockDim.x) {
            const int p = e / (2 * K), r = e - p * 2 * K, cy = r / K, m = r - cy * K, m0 = m % nc, row = m - m0;
            const int child = 2 * (p & (side - 1)) + ((2 * (p >> j) + cy) << (j + 1));
            double s = 0.0;
            for (int cx = 0; cx < 2; ++cx)
                for (int k = 0; k < nc; ++k) s += M[(cx * nc + m0) * nc + k] * cur[child + cx][row + k];
            z[e] = s;
        }
        __syncthreads();
        const int level = top + j;
        for (int e = tid; e < np * K; e += blockDim.x) {
            const int p = e / K, m = e - p * K, m0 = m % nc, m1 = m / nc;
            double s = 0.0;
            for (int cy = 0; cy < 2; ++cy)
                for (int k = 0; k < nc; ++k) s += M[(cy * nc + m1) * nc + k] * z[(p * 2 + cy) * K + k * nc + m0];
            cur[p][m] = s;
            const SubBox pb = sub_box(t, top, level, p);
            if (pb.ok)
                t.W[level][((long)rhs * t.nl0[level] * t.nl1[level] + pb.x + (long)t.nl0[level] * pb.y) * t.ld + m] = s;
        }
        __syncthreads();
    }
}

// Down pass from level `top` (whose locals are complete) to level `low`; LEAVES: low = L, on to y.
template <bool LEAVES>
__global__ __launch_bounds__(64 * kSubMax) void k_down(Hom2dDown d)
{
    __shared__ double cur[2][kSubMax][64], tmp[kSubMax][64], P[64], M[128];
    const Hom2d& t = d.t;
    const int tid = threadIdx.x, g = tid >> 6, lane = tid & 63, rhs = blockIdx.y;
    const int nc = t.nc, K = t.K, low = d.low, top = d.top;
    for (int i = tid; i < 2 * nc * nc; i += blockDim.x) M[i] = t.M1[i];
    if constexpr (LEAVES)
        for (int i = tid; i < 8 * nc; i += blockDim.x) P[i] = t.P1[i];
    const long nbt = (long)t.nl0[top] * t.nl1[top];
    if (g == 0 && lane < K) cur[0][0][lane] = t.Lc[top][((long)rhs * nbt + blockIdx.x) * t.ld + lane];
    // the leaf's operands of the assembly and the near field, on their way during the passes
    double xj = 0.0, sj = 0.0, dj = 0.0, near = 0.0;
    long j = -1;
    double* y = nullptr;
    int op = 0;
    if constexpr (LEAVES) {
        const SubBox b = sub_box(t, top, low, g);
        const int x = 8 * b.x + (lane & 7), yy = 8 * b.y + (lane >> 3);
        if (b.ok && x < t.n0 && yy < t.n1) {
            j = x + (long)t.n0 * yy;
            xj = d.io->x[(long)rhs * t.N + j];
            sj = d.ss[j];
            dj = d.diag[j];
            near = t.pot[((long)rhs * t.nl0[low] * t.nl1[low] + b.x + (long)t.nl0[low] * b.y) * kCells + lane];
        }
        y = d.io->y;
        op = d.io->op;
    }
    int at = 0;
    __syncthreads();
    for (int k = 1; k <= low - top; ++k, at ^= 1) {
        const int level = top + k, nb = 1 << (2 * k), side = 1 << k;
        const SubBox b = sub_box(t, top, level, g);
        const bool on = g < nb && b.ok && lane < K;
        const int parent = ((g & (side - 1)) >> 1) + (((g >> k) >> 1) << (k - 1));
        const int m0 = lane % nc, m1 = lane / nc;
        double* own = t.Lc[level] + ((long)rhs * t.nl0[level] * t.nl1[level] + b.x + (long)t.nl0[level] * b.y) * t.ld;
        double v = on ? own[lane] : 0.0;        // the level's translations
        if (on) {
            const double* mx = M + (b.x & 1) * nc * nc + m0;
            double s = 0.0;
            for (int i = 0; i < nc; ++i) s += mx[i * nc] * cur[at][parent][m1 * nc + i];
            tmp[g][lane] = s;
        }
        __syncthreads();
        if (on) {
            const double* my = M + (b.y & 1) * nc * nc + m1;
            double s = 0.0;
            for (int i = 0; i < nc; ++i) s += my[i * nc] * tmp[g][i * nc + m0];
            v += s;
            cur[at ^ 1][g][lane] = v;
            if (!LEAVES && level == low) own[lane] = v;
        }
        __syncthreads();
    }
    if constexpr (LEAVES) {
        const SubBox b = sub_box(t, top, low, g);
        if (b.ok && lane < 8 * nc) {
            const int m1 = lane >> 3, lx = lane & 7;
            double s = 0.0;
            for (int i = 0; i < nc; ++i) s += P[i * 8 + lx] * cur[at][g][m1 * nc + i];
            tmp[g][lane] = s;
        }
        __syncthreads();
        if (j < 0) return;
        double far = 0.0;
        for (int i = 0; i < nc; ++i) far += P[i * 8 + (lane >> 3)] * tmp[g][i * 8 + (lane & 7)];
        const double w = op == ERT_OP_G ? xj : sj * xj;
        const double v = d.hd * (near + far) + dj * w;
        y[(long)rhs * t.N + j] = op == ERT_OP_A ? xj - v : v;
    }
}

// Sum over the offsets of this wave (every fourth) of op_o W[t + o] for the 16 targets of a
// column tile, row tiles rt0 .. rt0 + RTB - 1: D holds rows lane / 16 + 4 i of target lane % 16.
template <int KS, int RT, int RTB>
__device__ __forceinline__ void offset_sum(const BoxOffset* __restrict__ offs, int noff, const double* __restrict__ F,
                                           const double* __restrict__ W, int ldw, int n0, int n1, int tx, int ty,
                                           bool tok, int rt0, v4d (&acc)[RTB])
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, grp = lane >> 4;
    for (int oi = wave; oi < noff; oi += 4) {
        const BoxOffset o = offs[oi];
        const int x = tx + o.o0, y = ty + o.o1;
        const bool in = tok && x >= 0 && x < n0 && y >= 0 && y < n1;
        if (!__any(in)) continue;
        const double* w = W + (long)(in ? x + (long)n0 * y : 0) * ldw + grp * KS;
        double b[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) b[s] = w[s];
#pragma unroll
        for (int s = 0; s < KS; ++s) b[s] = in ? b[s] : 0.0;
        const double* f = F + ((long)o.op * RT + rt0) * KS * 64 + lane;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int r = 0; r < RTB; ++r)
                acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[(r * KS + s) * 64], b[s], acc[r], 0, 0, 0);
    }
}

// Translations of every level and the near field.  Workgroup: a column tile of 16 target
// boxes (of one parity class of a level, which shares its interaction list; or of leaves
// for the near field) and all row tiles, or one of them (SPLIT) where the tiles are too
// few to fill the chip.  The four waves take every fourth offset; their sums are added
// in wave order.  Bound: the latency of the fragments (L2) and the FP64 matrix pipe.
template <int NC, bool SPLIT>
__global__ __launch_bounds__(256) void k_products(Hom2dProducts p)
{
    constexpr int K = NC * NC, KS = (K + 3) / 4, RT = (K + 15) / 16;
    constexpr int RTF = SPLIT ? 1 : RT, RTN = SPLIT ? 1 : 4;
    __shared__ double red[3 * RTN * 256];
    const Hom2d& t = p.t;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, grp = lane >> 4, li = lane & 15, rhs = blockIdx.z;
    const int rt0 = SPLIT ? blockIdx.y : 0;
    int blk = blockIdx.x;
    const int L = t.L;
    const bool near = blk < p.near_tiles;
    int level = L, cls = 0;
    if (!near) {
        blk -= p.near_tiles;
        while (blk >= p.tiles[level]) blk -= p.tiles[level--];
        if (rt0 >= RT) return;                  // uniform
    }
    const int n0 = t.nl0[level], n1 = t.nl1[level];
    int c0 = n0, c1 = n1, px = 0, py = 0, step = 1;
    if (!near) {
        step = 2;
        for (;; ++cls) {
            px = cls & 1;
            py = cls >> 1;
            c0 = (n0 - px + 1) / 2;
            c1 = (n1 - py + 1) / 2;
            const int nt = (c0 * c1 + 15) / 16;
            if (blk < nt || cls == 3) break;
            blk -= nt;
        }
    }
    const int col = 16 * blk + li;
    const bool tok = col < c0 * c1;
    const int ax = tok ? col % c0 : 0, ay = tok ? col / c0 : 0;
    const int tx = step * ax + px, ty = step * ay + py;
    const long nbox = (long)n0 * n1, box = tx + (long)n0 * ty;
    auto store = [&](v4d* acc, int nrt, double* out, int ld, int rows) {
        if (wave > 0)
            for (int r = 0; r < nrt; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) red[((wave - 1) * nrt + r) * 256 + i * 64 + lane] = acc[r][i];
        __syncthreads();
        if (wave != 0 || !tok) return;
        for (int r = 0; r < nrt; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * (rt0 + r) + grp + 4 * i;
                const double* q = red + r * 256 + i * 64 + lane;
                if (row < rows) out[box * ld + row] = ((acc[r][i] + q[0]) + q[nrt * 256]) + q[2 * nrt * 256];
            }
    };
    if (near) {
        v4d acc[RTN];
#pragma unroll
        for (int r = 0; r < RTN; ++r) acc[r] = v4d{0, 0, 0, 0};
        offset_sum<16, 4, RTN>(p.near_offs, 9, p.near, t.q + (long)rhs * nbox * kCells, kCells, n0, n1, tx, ty, tok, rt0,
                               acc);
        store(acc, RTN, t.pot + (long)rhs * nbox * kCells, kCells, kCells);
    } else {
        v4d acc[RTF];
#pragma unroll
        for (int r = 0; r < RTF; ++r) acc[r] = v4d{0, 0, 0, 0};
        offset_sum<KS, RT, RTF>(p.far_offs + 27 * cls, 27, p.far[level], t.W[level] + (long)rhs * nbox * t.ld, t.ld, n0, n1,
                                tx, ty, tok, rt0, acc);
        store(acc, RTF, t.Lc[level] + (long)rhs * nbox * t.ld, t.ld, K);
    }
}

int far_tiles(const Hom2d& t, int l)
{
    int n = 0;
    for (int c = 0; c < 4; ++c) n += ((t.nl0[l] - (c & 1) + 1) / 2 * ((t.nl1[l] - (c >> 1) + 1) / 2) + 15) / 16;
    return n;
}

template <int NC>
void launch_products(hipStream_t s, const Hom2dProducts& p, int tiles, int nrhs)
{
    // fewer tiles than two per CU: a workgroup per 16 rows (64^2: 4 + 20 tiles, 512^2: 600)
    if ((long)tiles * nrhs < 512)
        hipLaunchKernelGGL((k_products<NC, true>), dim3(tiles, 4, nrhs), dim3(256), 0, s, p);
    else
        hipLaunchKernelGGL((k_products<NC, false>), dim3(tiles, 1, nrhs), dim3(256), 0, s, p);
}

}  // namespace

size_t hom2d_fragment_elems(int K) { return (size_t)((K + 15) / 16) * ((K + 3) / 4) * 64; }

ert_status hom2d_fragments(hipStream_t s, const double* src, int ld, int K, long nmat, double* dst)
{
    const long n = nmat * (long)hom2d_fragment_elems(K);
    hipLaunchKernelGGL(k_fragments, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, ld, K, (K + 3) / 4,
                       (K + 15) / 16, nmat, dst);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

const void* hom2d_first_kernel() { return (const void*)k_up<true>; }

dim3 hom2d_up_grid(const Hom2dUp& u, int nrhs) { return dim3((unsigned)(u.t.nl0[u.top] * u.t.nl1[u.top]), (unsigned)nrhs); }
dim3 hom2d_up_block(const Hom2dUp& u) { return dim3(64u << (2 * (u.low - u.top))); }

ert_status hom2d_up(hipStream_t s, const Hom2dUp& first, int nrhs)
{
    hipLaunchKernelGGL(k_up<true>, hom2d_up_grid(first, nrhs), hom2d_up_block(first), 0, s, first);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status hom2d_up_rest(hipStream_t s, Hom2dUp u, int nrhs, int step)
{
    while (u.top > 2) {
        u.low = u.top;
        u.top = std::max(2, u.low - step);
        hipLaunchKernelGGL(k_up<false>, hom2d_up_grid(u, nrhs), hom2d_up_block(u), 0, s, u);
    }
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status hom2d_products(hipStream_t s, Hom2dProducts p, int nrhs, bool near, bool far)
{
    const Hom2d& t = p.t;
    p.near_tiles = near ? (t.nl0[t.L] * t.nl1[t.L] + 15) / 16 : 0;
    int tiles = p.near_tiles;
    for (int l = 2; l <= t.L && far; ++l) tiles += p.tiles[l] = far_tiles(t, l);
    switch (t.nc) {
    case 2: launch_products<2>(s, p, tiles, nrhs); break;
    case 3: launch_products<3>(s, p, tiles, nrhs); break;
    case 4: launch_products<4>(s, p, tiles, nrhs); break;
    case 5: launch_products<5>(s, p, tiles, nrhs); break;
    case 6: launch_products<6>(s, p, tiles, nrhs); break;
    case 7: launch_products<7>(s, p, tiles, nrhs); break;
    case 8: launch_products<8>(s, p, tiles, nrhs); break;
    default: record_error("FMM: Chebyshev order outside 2..8"); return ERT_EINVAL;
    }
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status hom2d_down(hipStream_t s, Hom2dDown d, int nrhs, int last, int step)
{
    const Hom2d& t = d.t;
    // an odd step first, then `step` levels each
    for (int top = 2; top < last;) {
        const int low = std::min(last, top + ((last - top) % step ? 1 : step));
        d.top = top;
        d.low = low;
        hipLaunchKernelGGL(k_down<false>, dim3((unsigned)(t.nl0[top] * t.nl1[top]), (unsigned)nrhs),
                           dim3(64u << (2 * (low - top))), 0, s, d);
        top = low;
    }
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status hom2d_out(hipStream_t s, Hom2dDown d, int nrhs, int last)
{
    const Hom2d& t = d.t;
    d.top = last;
    d.low = t.L;
    hipLaunchKernelGGL(k_down<true>, dim3((unsigned)(t.nl0[last] * t.nl1[last]), (unsigned)nrhs),
                       dim3(64u << (2 * (t.L - last))), 0, s, d);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

}  // namespace ertvie
