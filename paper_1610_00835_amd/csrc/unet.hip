// Learned right preconditioner: a three-level 3D convolutional U-Net (widths
// w1/w2/w3, 3x3x3 convolutions, 2x2x2 average pooling, nearest upsampling,
// skip connections by concatenation), trained on the device.
//
// Data layout: activations are FP32, channels-last ([batch][voxel][channel],
// voxel = x-fastest cell index of the solver grid), so one voxel's channels are
// contiguous and a 3x3x3 convolution is an implicit GEMM with a reduction over
// (tap, input channel).  Convolutions of the forward pass and the input
// gradients of the backward pass run on the matrix cores as BF16 x BF16 -> FP32
// (v_mfma_f32_16x16x32_bf16), BF16 weights times the FP32 activations split
// into two BF16 parts (hi + lo, two products, so activations keep ~16 mantissa
// bits and rounding noise does not compound layer after layer): rows are output
// channels, columns are voxels, so
// each lane ends with four consecutive channels of one voxel (one 16-byte
// store).  Weight gradients use FP32 operands (v_mfma_f32_16x16x4f32) with the
// voxel sum split into slabs and summed in a fixed order (deterministic).
// Parameters live in one flat FP32 vector in the canonical layout documented in
// include/ertvie.h; BF16 copies in GEMM order are rebuilt after every update.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "common.hpp"
#include "up2.hpp"

namespace ertvie {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kNetLayers = 11;
constexpr int kCinPad = 8;          // input feature channels as stored (3 used)

// Round-to-nearest-even FP32 -> BF16 (the rounding of the reference).
__device__ __forceinline__ __bf16 to_bf16(float f)
{
    unsigned u = __float_as_uint(f);
    u = u + 0x7FFFu + ((u >> 16) & 1u);
    unsigned short h = (unsigned short)(u >> 16);
    return __builtin_bit_cast(__bf16, h);
}

struct Tensor {          // channels-last view: element (b, v, c) at b * bstride + v * stride + off + c
    float* p;
    long bstride;
    int stride;
    int off;
};

struct ConvArgs {
    const float* in;
    long in_b;
    int in_stride, in_off, cin;     // cin: multiple of 8
    float* out;
    long out_b;
    int out_stride, out_off;
    const __bf16* W;                // [cout][Kpad], k = tap * cin + ci
    int Kpad;
    const float* bias;
    const float* mask;              // MODE 1: out *= (mask > 0)
    long mask_b;
    int mask_stride, mask_off;
    int n0, n1, n2;
    long V;
    int flip;                       // 1: taps mirrored (input-gradient convolution)
};

// MODE 0: bias + ReLU; MODE 1: multiply by the mask (x > 0); MODE 2: plain.
template <int CT, int MODE>
__global__ __launch_bounds__(256) void k_conv3(ConvArgs a)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, grp = lane >> 4;
    const long v0 = ((long)blockIdx.x * 4 + wave) * 16;
    if (v0 >= a.V) return;                      // uniform over the wave
    const int b = blockIdx.y;
    const long v = v0 + (lane & 15);
    const bool vok = v < a.V;
    const int x = (int)(v % a.n0), y = (int)((v / a.n0) % a.n1), z = (int)(v / ((long)a.n0 * a.n1));
    const float* in = a.in + (long)b * a.in_b + a.in_off;
    v4f acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = v4f{0.f, 0.f, 0.f, 0.f};
    const int Kreal = 27 * a.cin;
    for (int k0 = 0; k0 < a.Kpad; k0 += 32) {
        const int k = k0 + 8 * grp;
        v8bf bf;
        float xs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (vok && k < Kreal) {
            const int tap = k / a.cin, ci = k - tap * a.cin;
            const int t = a.flip ? 26 - tap : tap;
            const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
            const int xx = x + dx, yy = y + dy, zz = z + dz;
            if (xx >= 0 && xx < a.n0 && yy >= 0 && yy < a.n1 && zz >= 0 && zz < a.n2) {
                const float* src = in + (xx + (long)a.n0 * (yy + (long)a.n1 * zz)) * a.in_stride + ci;
                const v4f p = *(const v4f*)src, q = *(const v4f*)(src + 4);
                xs[0] = p[0]; xs[1] = p[1]; xs[2] = p[2]; xs[3] = p[3];
                xs[4] = q[0]; xs[5] = q[1]; xs[6] = q[2]; xs[7] = q[3];
            }
        }
        v8bf bl;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const __bf16 h = to_bf16(xs[e]);
            bf[e] = h;
            bl[e] = to_bf16(xs[e] - (float)h);
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const v8bf wf = *(const v8bf*)(a.W + (long)(16 * c + (lane & 15)) * a.Kpad + k);
            acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, bf, acc[c], 0, 0, 0);
            acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, bl, acc[c], 0, 0, 0);
        }
    }
    if (!vok) return;
    float* out = a.out + (long)b * a.out_b + v * a.out_stride + a.out_off;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int co = 16 * c + 4 * grp;
        v4f r = acc[c];
        if constexpr (MODE == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float t = r[i] + a.bias[co + i];
                r[i] = t > 0.f ? t : 0.f;
            }
        } else if constexpr (MODE == 1) {
            const v4f m = *(const v4f*)(a.mask + (long)b * a.mask_b + v * a.mask_stride + a.mask_off + co);
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = m[i] > 0.f ? r[i] : 0.f;
        }
        *(v4f*)(out + co) = r;
    }
}

// The same convolution with the input staged in LDS, for inputs of at most kTileCin
// channels.  A workgroup owns an 8 x 4 x (2 VT) box of voxels and stages it with its
// one-voxel halo, split into the two BF16 parts once (k_conv3 loads and splits every
// input value 27 times, and finds each of its taps by divisions).  Wave w takes VT times
// 16 voxels (two rows of 8) and the workgroup's 16 CT output channels: all of them, or 16
// where whole layers would leave CUs idle; a lane's eight channels of a tap are one
// 16-byte LDS read per part.  The reduction goes through the same chunks of 32 in
// the same order as k_conv3's, so the results are the same bits.  An LDS position is
// padded so that eight neighbouring ones start in different 16-byte banks.
// 32^3 x 4: 16 -> 16 channels 39 -> 16 us, 48 -> 16 channels 33 us.  Bound: LDS reads (one
// per product at 16 output channels) and, on the coarse levels, the latency of the weights.
constexpr int kTileCin = 128;
constexpr int kHx = 10, kHy = 6;                // staged box: 10 x 6 x (2 VT + 2) voxels
constexpr int kTileThreads = 256;

inline int tile_pitch(int cin) { return (cin / 8) % 2 ? cin : cin + 8; }
// bytes of LDS: the two parts, one zero vector, the offset of every group of 8 reduction
// indices (and of up to three chunks past the end)
inline size_t tile_lds(int cin, int Kpad, int vt)
{
    return (size_t)2 * kHx * kHy * (2 * vt + 2) * tile_pitch(cin) * sizeof(__bf16) + 16 + (size_t)(Kpad / 8 + 12) * sizeof(int);
}

template <int CT, int MODE, int VT>
__global__ __launch_bounds__(kTileThreads) void k_conv3_tile(ConvArgs a, int pitch, int t0, int t1)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int HZ = 2 * VT + 2, NPOS = kHx * kHy * HZ;
    __bf16* hi = (__bf16*)smem;
    __bf16* lo = hi + NPOS * pitch;
    __bf16* zero = lo + NPOS * pitch;
    int* koff = (int*)(zero + 8);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, grp = lane >> 4, li = lane & 15;
    const int b = blockIdx.y, cb = 16 * CT * blockIdx.z;   // first output channel
    const int bx = blockIdx.x % t0, by = (blockIdx.x / t0) % t1, bz = blockIdx.x / (t0 * t1);
    const int x0 = 8 * bx, y0 = 4 * by, z0 = 2 * VT * bz;
    const float* in = a.in + (long)b * a.in_b + a.in_off;
    for (int k = tid; k < a.Kpad / 8 + 12; k += kTileThreads) {
        const int tap = 8 * k / a.cin, ci = 8 * k - tap * a.cin;
        const int t = a.flip ? 26 - tap : tap;
        koff[k] = tap < 27 ? ((t / 9 * kHy + (t / 3) % 3) * kHx + t % 3) * pitch + ci : -1;
    }
    if (tid < 8) zero[tid] = (__bf16)0.f;
    // four groups of eight channels per thread and round, their loads together
    const int c8 = a.cin / 8, items = NPOS * c8;
    for (int e0 = tid; e0 < items; e0 += 4 * kTileThreads) {
        v4f u[4], v[4];
        int at[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int e = e0 + k * kTileThreads;
            const int p = e / c8, c = 8 * (e - p * c8);
            const int x = x0 + p % kHx - 1, y = y0 + (p / kHx) % kHy - 1, z = z0 + p / (kHx * kHy) - 1;
            at[k] = e < items ? p * pitch + c : -1;
            u[k] = v[k] = v4f{0.f, 0.f, 0.f, 0.f};
            if (e < items && x >= 0 && x < a.n0 && y >= 0 && y < a.n1 && z >= 0 && z < a.n2) {
                const float* src = in + (x + (long)a.n0 * (y + (long)a.n1 * z)) * a.in_stride + c;
                u[k] = *(const v4f*)src;
                v[k] = *(const v4f*)(src + 4);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (at[k] < 0) continue;
            v8bf h, l;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float f = q < 4 ? u[k][q] : v[k][q - 4];
                h[q] = (__bf16)f;                // v_cvt_pk_bf16_f32: to nearest even, as to_bf16
                l[q] = (__bf16)(f - (float)h[q]);
            }
            *(v8bf*)(hi + at[k]) = h;
            *(v8bf*)(lo + at[k]) = l;
        }
    }
    __syncthreads();
    // voxel li of tile vt: x li % 8, y 2 (..) + li / 8
    int base[VT];
#pragma unroll
    for (int t = 0; t < VT; ++t) {
        const int yp = VT == 2 ? t : (wave & 1), zz = VT == 2 ? wave : (wave >> 1);
        base[t] = ((zz * kHy + 2 * yp + (li >> 3)) * kHx + (li & 7)) * pitch;
    }
    const int zoff = (int)(zero - hi), lo_off = NPOS * pitch;
    v4f acc[VT][CT];
#pragma unroll
    for (int t = 0; t < VT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] = v4f{0.f, 0.f, 0.f, 0.f};
    const __bf16* W = a.W + (long)(cb + li) * a.Kpad + 8 * grp;
    // G chunks at a time, the next G's weights on their way; chunks past the end multiply zeros
    constexpr int G = CT <= 2 ? 4 : CT <= 4 ? 2 : 1;
    auto weights = [&](int k0, v8bf (&w)[G][CT]) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int k = k0 + 32 * u < a.Kpad ? k0 + 32 * u : 0;
#pragma unroll
            for (int c = 0; c < CT; ++c) w[u][c] = *(const v8bf*)(W + (long)16 * c * a.Kpad + k);
        }
    };
    v8bf wn[G][CT];
    weights(0, wn);
    for (int k0 = 0; k0 < a.Kpad; k0 += 32 * G) {
        v8bf w[G][CT];
        int ko[G];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            ko[u] = koff[k0 / 8 + 4 * u + grp];
#pragma unroll
            for (int c = 0; c < CT; ++c) w[u][c] = wn[u][c];
        }
        weights(k0 + 32 * G, wn);
#pragma unroll
        for (int u = 0; u < G; ++u) {
            v8bf bh[VT], bl[VT];
#pragma unroll
            for (int t = 0; t < VT; ++t) {
                bh[t] = *(const v8bf*)(hi + (ko[u] >= 0 ? base[t] + ko[u] : zoff));
                bl[t] = *(const v8bf*)(hi + (ko[u] >= 0 ? base[t] + ko[u] + lo_off : zoff));
            }
#pragma unroll
            for (int t = 0; t < VT; ++t)
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][c], bh[t], acc[t][c], 0, 0, 0);
                    acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][c], bl[t], acc[t][c], 0, 0, 0);
                }
        }
    }
#pragma unroll
    for (int t = 0; t < VT; ++t) {
        const int x = x0 + (li & 7), y = y0 + 2 * (VT == 2 ? t : (wave & 1)) + (li >> 3);
        const int z = z0 + (VT == 2 ? wave : (wave >> 1));
        if (x >= a.n0 || y >= a.n1 || z >= a.n2) continue;
        const long v = x + (long)a.n0 * (y + (long)a.n1 * z);
        float* out = a.out + (long)b * a.out_b + v * a.out_stride + a.out_off;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int co = cb + 16 * c + 4 * grp;
            v4f r = acc[t][c];
            if constexpr (MODE == 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float q = r[i] + a.bias[co + i];
                    r[i] = q > 0.f ? q : 0.f;
                }
            } else if constexpr (MODE == 1) {
                const v4f m = *(const v4f*)(a.mask + (long)b * a.mask_b + v * a.mask_stride + a.mask_off + co);
#pragma unroll
                for (int i = 0; i < 4; ++i) r[i] = m[i] > 0.f ? r[i] : 0.f;
            }
            *(v4f*)(out + co) = r;
        }
    }
}

// Weight gradients of a 3x3x3 layer.  A workgroup takes one pair of 16 input and 16
// output channels and a few tiles of 8 x 4 x 4 voxels: the tile of the output gradient and
// the tile with its one-voxel halo of the input are staged in LDS (FP32, the next ones in
// flight), and each of the twelve waves multiplies one plane of voxels, four to a
// v_mfma_f32_16x16x4f32, into the nine taps of one dz (nine accumulators, each operand one
// conflict-free LDS read; with all 27 in a wave only one workgroup fits a CU, 254 us).
// The waves' sums are added in wave order, the workgroups' by k_grad_reduce in slab order.  The bias gradient is summed beside the first input
// channels' pair.  All layers go in one launch after the backward pass, so that the small
// ones fill the chip beside the large ones.  Before, every (tap, 16 channels) was a workgroup of its own that read
// both operands from memory four bytes per lane: 32^3 x 4, all layers, 1620 us with
// their sums, now 181 + 16 us (105 us of products).  Bound: the FP32 matrix pipe.
struct DwArgs {
    const float* in;
    long in_b;
    int in_stride, in_off, cin;
    const float* g;                 // output gradient (after the activation mask)
    long g_b;
    int cout;
    int n0, n1, n2;
    int t0, t1, t2;                 // tiles per axis
    int ntile;                      // tiles over all batch columns
    int per, nslab, nco, npair;     // tiles per slab, slabs; pairs are (ci block, co block), co fastest
    float* part;                    // [slab][pair][kPairVals]
    int first;                      // workgroups of the layers before (k_conv_wgrad)
};
struct DwLayers {
    DwArgs l[10];
};

constexpr int kTapVals = 27 * 256;            // [tap][ci][co]
constexpr int kPairVals = kTapVals + 16;      // and the bias row
constexpr int kWgParts = 4, kWgThreads = 64 * 3 * kWgParts;

__global__ __launch_bounds__(kWgThreads, 6) void k_conv_wgrad(DwLayers G)
{
    int layer = 0;
    while (layer + 1 < 10 && (int)blockIdx.x >= G.l[layer + 1].first) ++layer;
    const DwArgs& a = G.l[layer];
    constexpr int NPOS = kHx * kHy * 6, NIN = NPOS * 4, PER = (NIN + kWgThreads - 1) / kWgThreads;
    constexpr int TILE = NPOS * 16 + 128 * 16;    // floats: input with halo, gradient
    __shared__ __align__(16) float sm[2 * TILE];
    static_assert(9 * kWgParts * 256 <= 2 * TILE, "one round of the waves' sums");
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, grp = lane >> 4, li = lane & 15;
    const int dz = wave / kWgParts, part = wave % kWgParts;
    const int pair = ((int)blockIdx.x - a.first) % a.npair, slab = ((int)blockIdx.x - a.first) / a.npair;
    const int ci0 = pair / a.nco * 16, co0 = pair % a.nco * 16;
    v4f rin[PER], rg;
    auto fetch = [&](int t) {
        const int per = a.t0 * a.t1 * a.t2, b = t / per, q = t - b * per;
        const int x0 = 8 * (q % a.t0), y0 = 4 * ((q / a.t0) % a.t1), z0 = 4 * (q / (a.t0 * a.t1));
        const float* in = a.in + (long)b * a.in_b + a.in_off + ci0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = tid + kWgThreads * k, p = e >> 2, c = 4 * (e & 3);
            const int x = x0 + p % kHx - 1, y = y0 + (p / kHx) % kHy - 1, z = z0 + p / (kHx * kHy) - 1;
            const bool ok = e < NIN && ci0 + c < a.cin && x >= 0 && x < a.n0 && y >= 0 && y < a.n1 && z >= 0 && z < a.n2;
            rin[k] = ok ? *(const v4f*)(in + (x + (long)a.n0 * (y + (long)a.n1 * z)) * a.in_stride + c)
                        : v4f{0.f, 0.f, 0.f, 0.f};
        }
        const int v = tid >> 2, c = 4 * (tid & 3);
        const int x = x0 + (v & 7), y = y0 + ((v >> 3) & 3), z = z0 + (v >> 5);
        const bool ok = v < 128 && x < a.n0 && y < a.n1 && z < a.n2;
        rg = ok ? *(const v4f*)(a.g + (long)b * a.g_b + (x + (long)a.n0 * (y + (long)a.n1 * z)) * a.cout + co0 + c)
                : v4f{0.f, 0.f, 0.f, 0.f};
    };
    auto stash = [&](float* d) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = tid + kWgThreads * k;
            if (e < NIN) *(v4f*)(d + 4 * e) = rin[k];
        }
        if (tid < 512) *(v4f*)(d + NPOS * 16 + 4 * tid) = rg;
    };
    v4f acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    // a slab's tiles are consecutive (neighbours share their halo in the cache)
    const int t0 = slab * a.per, t1 = min(a.ntile, t0 + a.per);
    fetch(t0);
    stash(sm);
    __syncthreads();
    int cur = 0;
    for (int t = t0; t < t1; ++t, cur ^= 1) {
        const bool more = t + 1 < t1;             // uniform
        if (more) fetch(t + 1);
        const float* si = sm + cur * TILE;
        const float* sg = si + NPOS * 16;
#pragma unroll 2
        for (int i = 0; i < 8; ++i) {
            // four voxels along x: plane `part` of the tile, row i / 2, half i % 2
            const int x = 4 * (i & 1) + grp, y = i >> 1;
            const float gv = sg[((part * 4 + y) * 8 + x) * 16 + li];
            const float* A = si + (((part + dz) * kHy + y) * kHx + x) * 16 + li;
            bsum += gv;
#pragma unroll
            for (int tap = 0; tap < 9; ++tap)
                acc[tap] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[(tap / 3 * kHx + tap % 3) * 16], gv, acc[tap], 0, 0, 0);
        }
        if (more) stash(sm + (cur ^ 1) * TILE);
        __syncthreads();
    }
    float* dst = a.part + ((long)slab * a.npair + pair) * kPairVals;
#pragma unroll
    for (int q = 0; q < 3; ++q) {                 // taps 9 dz + 3 q ..
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                sm[((dz * 3 + t) * kWgParts + part) * 256 + (4 * grp + i) * 16 + li] = acc[3 * q + t][i];
        __syncthreads();
        for (int e = tid; e < 9 * 256; e += kWgThreads) {
            const int t = e >> 8;
            const float* p = sm + t * kWgParts * 256 + (e & 255);
            dst[(t / 3 * 9 + 3 * q + t % 3) * 256 + (e & 255)] = ((p[0] + p[256]) + p[512]) + p[768];
        }
        __syncthreads();
    }
    if (ci0 != 0) return;
    if (dz == 0) sm[(part * 4 + grp) * 16 + li] = bsum;
    __syncthreads();
    if (tid < 16) {
        float s = sm[tid];
        for (int k = 1; k < 4 * kWgParts; ++k) s += sm[k * 16 + tid];
        dst[kTapVals + tid] = s;
    }
}

// Weight and bias gradient of the 1x1x1 output layer: part[slab][0 .. C) and [C].
__global__ __launch_bounds__(256) void k_head_wgrad(const float* __restrict__ x, const float* __restrict__ gy, int C,
                                                    long n, int nslab, float* __restrict__ part)
{
    __shared__ float red[256], rb[256];
    const int c = threadIdx.x % C, row = threadIdx.x / C, rows = 256 / C;
    float s = 0.f, sb = 0.f;
    if (row < rows)
#pragma unroll 4
        for (long v = (long)blockIdx.x * rows + row; v < n; v += (long)nslab * rows) {
            const float g = gy[v];
            s += x[v * C + c] * g;
            sb += g;
        }
    red[threadIdx.x] = s;
    rb[threadIdx.x] = sb;
    __syncthreads();
    if (threadIdx.x > C) return;
    const int q = threadIdx.x < C ? threadIdx.x : 0;
    const float* p = threadIdx.x < C ? red : rb;
    float t = p[q];
    for (int k = 1; k < rows; ++k) t += p[k * C + q];
    part[(long)blockIdx.x * (C + 1) + threadIdx.x] = t;
}

// All layers' slabs summed in slab order (four consecutive quarters, then those) into the
// canonical gradient.  Workgroup: 64 partial values of one layer, four waves over the
// slabs; consecutive lanes read consecutive values.
struct GradLayer {
    const float* part;
    float* gw;
    float* gb;
    int ntaps, cin_real, cout, nco, npair, nslab, first;   // first: workgroups of the layers before
};
struct GradLayers {
    GradLayer l[11];
};

__global__ __launch_bounds__(256) void k_grad_reduce(GradLayers G)
{
    __shared__ float red[256];
    int li = 0;
    while (li + 1 < 11 && (int)blockIdx.x >= G.l[li + 1].first) ++li;
    const GradLayer& l = G.l[li];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int vals = l.ntaps == 27 ? l.npair * kPairVals : l.cin_real + 1;
    const int e = ((int)blockIdx.x - l.first) * 64 + lane;
    const int per = (l.nslab + 3) / 4, k0 = wave * per, k1 = min(l.nslab, k0 + per);
    float s = 0.f;
    if (e < vals)
#pragma unroll 8
        for (int k = k0; k < k1; ++k) s += l.part[(long)k * vals + e];
    red[threadIdx.x] = s;
    __syncthreads();
    if (wave != 0 || e >= vals) return;
    s = ((red[lane] + red[64 + lane]) + red[128 + lane]) + red[192 + lane];
    if (l.ntaps != 27) {
        if (e < l.cin_real) l.gw[e] = s;
        else l.gb[0] = s;
        return;
    }
    const int pair = e / kPairVals, r = e - pair * kPairVals;
    const int ci0 = pair / l.nco * 16, co0 = pair % l.nco * 16;
    if (r >= kTapVals) {
        if (ci0 == 0) l.gb[co0 + r - kTapVals] = s;
        return;
    }
    const int tap = r >> 8, ci = ci0 + ((r >> 4) & 15), co = co0 + (r & 15);
    if (ci < l.cin_real) l.gw[((long)co * l.cin_real + ci) * 27 + tap] = s;
}

// BF16 weights in GEMM order.  Forward: Wf[co][tap * cin_pad + ci] = W[co][ci][tap].
// Input gradient: Wb[ci][tap * cout + co] = W[co][ci][tap] (taps mirrored at use).
__global__ void k_prep_w(const float* W, int cout, int cin_real, int cin_pad, int Kpad, __bf16* Wf, __bf16* Wb,
                         int KpadB)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < (long)cout * Kpad) {
        const int co = (int)(i / Kpad), k = (int)(i % Kpad);
        float w = 0.f;
        if (k < 27 * cin_pad) {
            const int tap = k / cin_pad, ci = k % cin_pad;
            if (ci < cin_real) w = W[((long)co * cin_real + ci) * 27 + tap];
        }
        Wf[i] = to_bf16(w);
    }
    if (Wb && i < (long)cin_pad * KpadB) {
        const int ci = (int)(i / KpadB), k = (int)(i % KpadB);
        float w = 0.f;
        if (k < 27 * cout && ci < cin_real) {
            const int tap = k / cout, co = k % cout;
            w = W[((long)co * cin_real + ci) * 27 + tap];
        }
        Wb[i] = to_bf16(w);
    }
}

// Input channels: r / s, log sigma_t, sigma_s / sigma_t, zero padding.
__global__ void k_features(const double* r, const double* st, const double* ss, long N, const double* scale,
                           int media_per_rhs, float* X)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (i >= N) return;
    const long m = media_per_rhs ? (long)b * N + i : i;
    float* d = X + ((long)b * N + i) * kCinPad;
    d[0] = (float)(r[(long)b * N + i] / scale[b]);
    d[1] = (float)log(st[m]);
    d[2] = (float)(ss[m] / st[m]);
#pragma unroll
    for (int c = 3; c < kCinPad; ++c) d[c] = 0.f;
}

// rms of each column (two passes: block partials, then one block per column).
__global__ void k_sumsq_partial(const double* x, long N, double* part, int nblk)
{
    __shared__ double sh[256];
    const int b = blockIdx.y;
    double s = 0.0;
    for (long i = blockIdx.x * 256L + threadIdx.x; i < N; i += (long)nblk * 256) {
        const double v = x[(long)b * N + i];
        s += v * v;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(long)b * nblk + blockIdx.x] = sh[0];
}

__global__ void k_rms_final(const double* part, int nblk, long N, double* scale)
{
    __shared__ double sh[64];                // nblk <= 64; loaded together, added in order
    const int b = blockIdx.x;
    if ((int)threadIdx.x < nblk) sh[threadIdx.x] = part[(long)b * nblk + threadIdx.x];
    __syncthreads();
    if (threadIdx.x != 0) return;
    double s = 0.0;
    for (int k = 0; k < nblk; ++k) s += sh[k];
    const double r = sqrt(s / (double)N);
    scale[b] = r > 0.0 ? r : 1.0;
}

__global__ void k_pool2(const float* src, long s_b, int s_stride, int s_off, int C, float* dst, long d_b, int n0,
                        int n1, int n2)
{
    const int m0 = n0 / 2, m1 = n1 / 2, m2 = n2 / 2;
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (i >= (long)m0 * m1 * m2 * C) return;
    const int c = (int)(i % C);
    const long p = i / C;
    const int x = (int)(p % m0), y = (int)((p / m0) % m1), z = (int)(p / ((long)m0 * m1));
    float s = 0.f;
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) {
                const long v = (2 * x + dx) + (long)n0 * ((2 * y + dy) + (long)n1 * (2 * z + dz));
                s += src[(long)b * s_b + v * s_stride + s_off + c];
            }
    dst[(long)b * d_b + p * C + c] = s * 0.125f;
}

// dst (fine grid n) channels [d_off, d_off + C) = src (coarse grid) nearest value; four
// channels per thread (every stride and offset is a multiple of 8)
__global__ void k_up2(const float* src, long s_b, int C, float* dst, long d_b, int d_stride, int d_off, int n0,
                      int n1, int n2)
{
    const Up2Cell q = up2_cell(blockIdx.x, blockDim.x, threadIdx.x, C, n0, n1);
    const int b = blockIdx.y;
    if (q.z >= (unsigned)n2) return;
    const long p = q.x / 2 + (long)(n0 / 2) * (q.y / 2 + (long)(n1 / 2) * (q.z / 2));
    *(v4f*)(dst + (long)b * d_b + (long)q.v * d_stride + d_off + q.c) = *(const v4f*)(src + (long)b * s_b + p * C + q.c);
}

// dst (coarse) = (sum over the 8 children of g channels [g_off, g_off + C)) * (mask > 0)
__global__ void k_up2_grad_mask(const float* g, long g_b, int g_stride, int g_off, int C, const float* mask,
                                long m_b, float* dst, long d_b, int n0, int n1, int n2)
{
    const int m0 = n0 / 2, m1 = n1 / 2, m2 = n2 / 2;
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (i >= (long)m0 * m1 * m2 * C) return;
    const int c = (int)(i % C);
    const long p = i / C;
    const int x = (int)(p % m0), y = (int)((p / m0) % m1), z = (int)(p / ((long)m0 * m1));
    float s = 0.f;
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) {
                const long v = (2 * x + dx) + (long)n0 * ((2 * y + dy) + (long)n1 * (2 * z + dz));
                s += g[(long)b * g_b + v * g_stride + g_off + c];
            }
    dst[(long)b * d_b + p * C + c] = mask[(long)b * m_b + p * C + c] > 0.f ? s : 0.f;
}

// dst (fine, dense C) = (skip gradient + coarse gradient / 8) * (mask > 0)
__global__ void k_pool2_grad_add_mask(const float* gs, long gs_b, int gs_stride, int gs_off, const float* gp,
                                      long gp_b, const float* mask, long m_b, int m_stride, int m_off, int C,
                                      float* dst, long d_b, int n0, int n1, int n2)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (i >= (long)n0 * n1 * n2 * C) return;
    const int c = (int)(i % C);
    const long v = i / C;
    const int x = (int)(v % n0), y = (int)((v / n0) % n1), z = (int)(v / ((long)n0 * n1));
    const long p = x / 2 + (long)(n0 / 2) * (y / 2 + (long)(n1 / 2) * (z / 2));
    const float s = gs[(long)b * gs_b + v * gs_stride + gs_off + c] + gp[(long)b * gp_b + p * C + c] * 0.125f;
    dst[(long)b * d_b + v * C + c] = mask[(long)b * m_b + v * m_stride + m_off + c] > 0.f ? s : 0.f;
}

// 1x1x1 output layer: y = sum_c w[c] x[v][c] + b
__global__ void k_head(const float* x, long x_b, int C, const float* w, const float* bias, float* y, long V)
{
    const long v = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (v >= V) return;
    const float* xv = x + (long)b * x_b + v * C;
    float s = 0.f;
    for (int c = 0; c < C; ++c) s += w[c] * xv[c];
    y[(long)b * V + v] = s + bias[0];
}

// Targets t = (e - r) / s (FP32) and, per column, partial sums of (y - t)^2 and t^2.
__global__ void k_loss_partial(const float* y, const double* e, const double* r, const double* scale, long V,
                               float* t, double* part, int nblk)
{
    __shared__ double s1[256], s2[256];
    const int b = blockIdx.y;
    double a = 0.0, c = 0.0;
    for (long i = blockIdx.x * 256L + threadIdx.x; i < V; i += (long)nblk * 256) {
        const float tv = (float)((e[(long)b * V + i] - r[(long)b * V + i]) / scale[b]);
        t[(long)b * V + i] = tv;
        const double d = (double)y[(long)b * V + i] - (double)tv;
        a += d * d;
        c += (double)tv * (double)tv;
    }
    s1[threadIdx.x] = a;
    s2[threadIdx.x] = c;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            s1[threadIdx.x] += s1[threadIdx.x + w];
            s2[threadIdx.x] += s2[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[((long)b * nblk + blockIdx.x) * 2] = s1[0];
        part[((long)b * nblk + blockIdx.x) * 2 + 1] = s2[0];
    }
}

// loss = mean over columns of sum (y - t)^2 / sum t^2; tt[b] = sum t^2
__global__ void k_loss_final(const double* part, int nblk, int B, double* tt, double* loss)
{
    double L = 0.0;
    for (int b = 0; b < B; ++b) {
        // one wave, nblk <= 64: lane k holds block k's sums
        const bool ok = (int)threadIdx.x < nblk;
        double a = ok ? part[((long)b * nblk + threadIdx.x) * 2] : 0.0;
        double c = ok ? part[((long)b * nblk + threadIdx.x) * 2 + 1] : 0.0;
        for (int d = 1; d < 64; d <<= 1) {
            a += __shfl_xor(a, d, 64);
            c += __shfl_xor(c, d, 64);
        }
        const double t = c > 0.0 ? c : 1.0;
        if (threadIdx.x == 0) tt[b] = t;
        L += a / t;
    }
    if (threadIdx.x == 0) loss[0] = L / B;
}

// gy = 2 (y - t) / (tt B); G = w[c] gy * (x[v][c] > 0) (head and last ReLU); four channels
// per thread
__global__ void k_head_grad(const float* y, const float* t, const double* tt, int B, long V, const float* w,
                            const float* x, int C, float* gy, float* G)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int b = blockIdx.y, C4 = C / 4;
    const long v = i / C4;
    const int c = 4 * (int)(i - v * C4);
    if (v >= V) return;
    const float g = (float)(2.0 * ((double)y[(long)b * V + v] - (double)t[(long)b * V + v]) / (tt[b] * B));
    if (c == 0) gy[(long)b * V + v] = g;
    const v4f xv = *(const v4f*)(x + ((long)b * V + v) * C + c);
    v4f r;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = xv[k] > 0.f ? w[c + k] * g : 0.f;
    *(v4f*)(G + ((long)b * V + v) * C + c) = r;
}

__global__ void k_adam(float* p, const float* g, float* m, float* v, long n, float lr, float b1, float b2,
                       float eps, float c1, float c2)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// z = r + s y (FP64 output): the identity part of the correction plus the network's
__global__ void k_out(const float* y, const double* r, const double* scale, long V, double* z)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (i >= V) return;
    z[(long)b * V + i] = r[(long)b * V + i] + (double)y[(long)b * V + i] * scale[b];
}

// z = r + scale * y(parent cell) on the fine grid (n0 x n1 x n2, x fastest): the
// network's output on the grid coarsened by f, extended piecewise constant.
__global__ void k_out_prolong(const float* y, const double* r, const double* scale, int n0, int n1, int n2, int f,
                              double* z)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const long N = (long)n0 * n1 * n2;
    if (i >= N) return;
    const int i0 = (int)(i % n0), i1 = (int)((i / n0) % n1), i2 = (int)(i / ((long)n0 * n1));
    const int c0 = n0 / f, c1 = n1 / f;
    const long c = i0 / f + (long)c0 * (i1 / f + (long)c1 * (i2 / f));
    z[i] = r[i] + (double)y[c] * scale[0];
}

inline unsigned nblocks(long n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// Cell averages over f x f x f blocks: y[c] = f^-3 sum of x over the fine cells of coarse
// cell c (fine grid n0 x n1 x n2, every n_a a multiple of f, x fastest; fixed summation
// order: z, then y, then x).  nrhs columns of N fine / N / f^3 coarse values.
__global__ void k_restrict(const double* __restrict__ x, int n0, int n1, int n2, int f, double* __restrict__ y)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    const int c0 = n0 / f, c1 = n1 / f, c2 = n2 / f;
    const long Nc = (long)c0 * c1 * c2, N = (long)n0 * n1 * n2;
    if (i >= Nc) return;
    const int j0 = (int)(i % c0) * f, j1 = (int)((i / c0) % c1) * f, j2 = (int)(i / ((long)c0 * c1)) * f;
    const double* xb = x + (long)b * N;
    double s = 0.0;
    for (int dz = 0; dz < f; ++dz)
        for (int dy = 0; dy < f; ++dy)
            for (int dx = 0; dx < f; ++dx) s += xb[(j0 + dx) + (long)n0 * ((j1 + dy) + (long)n1 * (j2 + dz))];
    y[(long)b * Nc + i] = s / (double)(f * f * f);
}

ert_status restrict_avg(hipStream_t s, const double* x, const int n[3], int f, double* y, int nrhs)
{
    const long Nc = (long)(n[0] / f) * (n[1] / f) * (n[2] / f);
    hipLaunchKernelGGL(k_restrict, dim3(nblocks(Nc), nrhs), dim3(256), 0, s, x, n[0], n[1], n[2], f, y);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

// ----------------------------------------------------------------- host ----

constexpr int kHeadSlabs = 512;     // workgroups of the output layer's weight gradient

// Grid level of a layer: 0 full, 1 half, 2 quarter resolution.
inline int layer_level(int li) { return (li < 2 || li >= 8) ? 0 : ((li < 4 || li >= 6) ? 1 : 2); }

struct NetLayer {
    int cin_real, cin, cout, k;     // cin: as stored (multiple of 8)
    long w_off, b_off;              // canonical parameter offsets
    int Kpad, KpadB;
    size_t part_off;                // partial weight gradients in NetImpl::part
    __bf16* Wf = nullptr;
    __bf16* Wb = nullptr;
};

struct NetImpl {
    ert_net_opts o;
    hipStream_t s = nullptr;
    int n[3];
    long V, V2, V4;
    int B;            // batch capacity
    int B_run = 1;    // batch of the current call
    int w1, w2, w3;
    NetLayer L[kNetLayers];
    long nparam = 0;
    float *P = nullptr, *G = nullptr, *M = nullptr, *Vv = nullptr;
    long step = 0;
    // activations (per batch slot: [V][C])
    float *X = nullptr, *A1 = nullptr, *C1 = nullptr, *P1 = nullptr, *A2 = nullptr, *C2 = nullptr, *P2 = nullptr,
          *A3 = nullptr, *A3b = nullptr, *D2 = nullptr, *D2b = nullptr, *D1 = nullptr, *D1b = nullptr, *Y = nullptr;
    // gradients
    float *T = nullptr, *gY = nullptr, *Gf1 = nullptr, *Gf2 = nullptr, *GC1 = nullptr, *Gh1 = nullptr,
          *Gh2 = nullptr, *GC2 = nullptr, *Gq1 = nullptr, *Gq2 = nullptr, *gP2 = nullptr, *Gh3 = nullptr,
          *Gh4 = nullptr, *gP1 = nullptr, *Gf3 = nullptr, *Gf4 = nullptr, *part = nullptr;
    double *scale = nullptr, *red = nullptr, *tt = nullptr, *loss = nullptr;
    int red_blk = 64;
    double* coarse = nullptr;   // restricted residual and media (3 V) for use on a finer plan grid
    std::vector<void*> allocs;

    ert_status alloc(void* pp, size_t bytes)
    {
        void** q = (void**)pp;
        if (hipMalloc(q, bytes ? bytes : 16) != hipSuccess) {
            record_error("net: device allocation failed");
            return ERT_ENOMEM;
        }
        allocs.push_back(*q);
        return ERT_OK;
    }
    ~NetImpl()
    {
        for (void* q : allocs) (void)hipFree(q);
    }
};

namespace {

ert_status conv(NetImpl* n, int li, const float* in, long in_b, int in_stride, int in_off, float* out, long out_b,
                int out_stride, int out_off, int level, int mode, bool backward, const float* mask = nullptr,
                long mask_b = 0, int mask_stride = 0, int mask_off = 0)
{
    const NetLayer& l = n->L[li];
    const int f = 1 << level;
    ConvArgs a;
    a.in = in; a.in_b = in_b; a.in_stride = in_stride; a.in_off = in_off;
    a.out = out; a.out_b = out_b; a.out_stride = out_stride; a.out_off = out_off;
    a.mask = mask; a.mask_b = mask_b; a.mask_stride = mask_stride; a.mask_off = mask_off;
    a.n0 = n->n[0] / f; a.n1 = n->n[1] / f; a.n2 = n->n[2] / f;
    a.V = (long)a.n0 * a.n1 * a.n2;
    a.bias = n->P + l.b_off;
    int cout;
    if (!backward) {
        a.cin = l.cin; a.W = l.Wf; a.Kpad = l.Kpad; a.flip = 0; cout = l.cout;
    } else {
        a.cin = l.cout; a.W = l.Wb; a.Kpad = l.KpadB; a.flip = 1; cout = l.cin;
    }
    const dim3 grid(nblocks(a.V, 64), n->B_run);
    const int ct = cout / 16;
    if (ct < 1 || ct > 8 || ct == 5 || ct == 7) {       // whatever the grid: one rule for every form
        record_error("net: unsupported channel count");
        return ERT_EUNSUPPORTED;
    }
    // tiles of 128 voxels while they fill the chip twice over and two fit a CU's LDS, else of 64
    const int t0 = (a.n0 + 7) / 8, t1 = (a.n1 + 3) / 4;
    const bool big = (long)t0 * t1 * ((a.n2 + 3) / 4) * n->B_run >= 512 && tile_lds(a.cin, a.Kpad, 2) <= 80 * 1024;
    const int vt = big ? 2 : 1;
    const dim3 tiles((unsigned)(t0 * t1 * ((a.n2 + 2 * vt - 1) / (2 * vt))), n->B_run);
    const size_t lds = tile_lds(a.cin, a.Kpad, vt);
    const int pitch = tile_pitch(a.cin);
    // coarse levels (few tiles): a workgroup per 16 output channels
    if (a.cin <= kTileCin && (long)tiles.x * tiles.y < 512) {
        const dim3 split(tiles.x, tiles.y, ct);
        if (mode == 0) hipLaunchKernelGGL((k_conv3_tile<1, 0, 1>), split, dim3(kTileThreads), lds, n->s, a, pitch, t0, t1);
        else if (mode == 1)
            hipLaunchKernelGGL((k_conv3_tile<1, 1, 1>), split, dim3(kTileThreads), lds, n->s, a, pitch, t0, t1);
        else hipLaunchKernelGGL((k_conv3_tile<1, 2, 1>), split, dim3(kTileThreads), lds, n->s, a, pitch, t0, t1);
        ERT_HIP(hipGetLastError());
        return ERT_OK;
    }
#define ERT_CONV_M(CT, MODE)                                                                                     \
    if (a.cin > kTileCin)                                                                                        \
        hipLaunchKernelGGL((k_conv3<CT, MODE>), grid, dim3(256), 0, n->s, a);                                    \
    else if (vt == 2)                                                                                            \
        hipLaunchKernelGGL((k_conv3_tile<CT, MODE, 2>), tiles, dim3(kTileThreads), lds, n->s, a, pitch, t0, t1); \
    else                                                                                                         \
        hipLaunchKernelGGL((k_conv3_tile<CT, MODE, 1>), tiles, dim3(kTileThreads), lds, n->s, a, pitch, t0, t1);
#define ERT_CONV(CT)                             \
    if (mode == 0) { ERT_CONV_M(CT, 0) }         \
    else if (mode == 1) { ERT_CONV_M(CT, 1) }    \
    else { ERT_CONV_M(CT, 2) }
    switch (ct) {
    case 1: ERT_CONV(1) break;
    case 2: ERT_CONV(2) break;
    case 3: ERT_CONV(3) break;
    case 4: ERT_CONV(4) break;
    case 6: ERT_CONV(6) break;
    default: ERT_CONV(8) break;
    }
#undef ERT_CONV
#undef ERT_CONV_M
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}


// Tiles, pairs and slabs of the 3x3x3 layers' weight gradients for a batch of B: a workgroup
// takes enough tiles of one pair that about eight workgroups per CU do all layers, so
// that the launch ends evenly and the partial sums stay small.
void wgrad_shapes(const NetImpl* n, int B, DwLayers& G)
{
    long units = 0;
    for (int li = 0; li < kNetLayers - 1; ++li) {
        const NetLayer& l = n->L[li];
        DwArgs& a = G.l[li];
        const int f = 1 << layer_level(li);
        a.cin = l.cin;
        a.cout = l.cout;
        a.n0 = n->n[0] / f; a.n1 = n->n[1] / f; a.n2 = n->n[2] / f;
        a.t0 = (a.n0 + 7) / 8; a.t1 = (a.n1 + 3) / 4; a.t2 = (a.n2 + 3) / 4;
        a.ntile = a.t0 * a.t1 * a.t2 * B;
        a.nco = l.cout / 16;
        a.npair = (l.cin + 15) / 16 * a.nco;
        units += (long)a.ntile * a.npair;
    }
    const int per = (int)std::min<long>(16, std::max<long>(1, units / 2048));
    int first = 0;
    for (int li = 0; li < kNetLayers - 1; ++li) {
        DwArgs& a = G.l[li];
        a.per = per;
        a.nslab = (a.ntile + per - 1) / per;
        a.first = first;
        first += a.nslab * a.npair;
    }
}

// Inputs of layer li's weight gradient: activations `in` (stride/offset) and the output
// gradient after its mask `g` (dense cout channels).
void wgrad(DwLayers& G, int li, const float* in, long in_b, int in_stride, int in_off, const float* g, long g_b)
{
    DwArgs& a = G.l[li];
    a.in = in; a.in_b = in_b; a.in_stride = in_stride; a.in_off = in_off;
    a.g = g; a.g_b = g_b;
}

// The weight gradients of every layer into n->G.
ert_status weight_gradients(NetImpl* n, DwLayers& W, const float* head_in, const float* head_g)
{
    GradLayers G;
    int first = 0;
    for (int li = 0; li < kNetLayers; ++li) {
        const NetLayer& l = n->L[li];
        GradLayer& g = G.l[li];
        g.part = n->part + l.part_off;
        g.gw = n->G + l.w_off;
        g.gb = n->G + l.b_off;
        g.ntaps = l.k == 3 ? 27 : 1;
        g.cin_real = l.cin_real;
        g.cout = l.cout;
        g.first = first;
        if (l.k == 3) {
            W.l[li].part = n->part + l.part_off;
            g.nco = W.l[li].nco;
            g.npair = W.l[li].npair;
            g.nslab = W.l[li].nslab;
            first += (g.npair * kPairVals + 63) / 64;
        } else {
            g.nco = g.npair = 1;
            g.nslab = kHeadSlabs;
            first += (l.cin_real + 1 + 63) / 64;
        }
    }
    const DwArgs& last = W.l[kNetLayers - 2];
    hipLaunchKernelGGL(k_conv_wgrad, dim3(last.first + last.nslab * last.npair), dim3(kWgThreads), 0, n->s, W);
    hipLaunchKernelGGL(k_head_wgrad, dim3(kHeadSlabs), dim3(256), 0, n->s, head_in, head_g, n->w1, n->V * n->B_run,
                       kHeadSlabs, n->part + n->L[kNetLayers - 1].part_off);
    hipLaunchKernelGGL(k_grad_reduce, dim3(first), dim3(256), 0, n->s, G);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status prep_weights(NetImpl* n)
{
    for (int li = 0; li < kNetLayers; ++li) {
        NetLayer& l = n->L[li];
        if (l.k != 3) continue;
        const long cnt = std::max((long)l.cout * l.Kpad, l.Wb ? (long)l.cin * l.KpadB : 0L);
        hipLaunchKernelGGL(k_prep_w, dim3(nblocks(cnt)), dim3(256), 0, n->s, (const float*)(n->P + l.w_off), l.cout,
                           l.cin_real, l.cin, l.Kpad, l.Wf, l.Wb, l.KpadB);
        ERT_HIP(hipGetLastError());
    }
    return ERT_OK;
}

// features + column scales of r (FP64 N x B)
ert_status features(NetImpl* n, const double* r, const double* st, const double* ss, int media_per_rhs)
{
    const int B = n->B_run;
    hipLaunchKernelGGL(k_sumsq_partial, dim3(n->red_blk, B), dim3(256), 0, n->s, r, n->V, n->red, n->red_blk);
    hipLaunchKernelGGL(k_rms_final, dim3(B), dim3(64), 0, n->s, (const double*)n->red, n->red_blk, n->V, n->scale);
    hipLaunchKernelGGL(k_features, dim3(nblocks(n->V), B), dim3(256), 0, n->s, r, st, ss, n->V,
                       (const double*)n->scale, media_per_rhs, n->X);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ert_status forward(NetImpl* n)
{
    const int w1 = n->w1, w2 = n->w2, w3 = n->w3, B = n->B_run;
    const long V = n->V, V2 = n->V2, V4 = n->V4;
    const int c1s = w2 + w1, c2s = w3 + w2;
    const int n0 = n->n[0], n1 = n->n[1], n2 = n->n[2];
    ERT_TRY(conv(n, 0, n->X, V * kCinPad, kCinPad, 0, n->A1, V * w1, w1, 0, 0, 0, false));
    ERT_TRY(conv(n, 1, n->A1, V * w1, w1, 0, n->C1, V * c1s, c1s, w2, 0, 0, false));
    hipLaunchKernelGGL(k_pool2, dim3(nblocks(V2 * w1), B), dim3(256), 0, n->s, (const float*)n->C1, V * c1s, c1s, w2,
                       w1, n->P1, V2 * w1, n0, n1, n2);
    ERT_TRY(conv(n, 2, n->P1, V2 * w1, w1, 0, n->A2, V2 * w2, w2, 0, 1, 0, false));
    ERT_TRY(conv(n, 3, n->A2, V2 * w2, w2, 0, n->C2, V2 * c2s, c2s, w3, 1, 0, false));
    hipLaunchKernelGGL(k_pool2, dim3(nblocks(V4 * w2), B), dim3(256), 0, n->s, (const float*)n->C2, V2 * c2s, c2s, w3,
                       w2, n->P2, V4 * w2, n0 / 2, n1 / 2, n2 / 2);
    ERT_TRY(conv(n, 4, n->P2, V4 * w2, w2, 0, n->A3, V4 * w3, w3, 0, 2, 0, false));
    ERT_TRY(conv(n, 5, n->A3, V4 * w3, w3, 0, n->A3b, V4 * w3, w3, 0, 2, 0, false));
    hipLaunchKernelGGL(k_up2, dim3(nblocks(V2 * w3 / 4), B), dim3(256), 0, n->s, (const float*)n->A3b, V4 * w3, w3, n->C2,
                       V2 * c2s, c2s, 0, n0 / 2, n1 / 2, n2 / 2);
    ERT_TRY(conv(n, 6, n->C2, V2 * c2s, c2s, 0, n->D2, V2 * w2, w2, 0, 1, 0, false));
    ERT_TRY(conv(n, 7, n->D2, V2 * w2, w2, 0, n->D2b, V2 * w2, w2, 0, 1, 0, false));
    hipLaunchKernelGGL(k_up2, dim3(nblocks(V * w2 / 4), B), dim3(256), 0, n->s, (const float*)n->D2b, V2 * w2, w2, n->C1,
                       V * c1s, c1s, 0, n0, n1, n2);
    ERT_TRY(conv(n, 8, n->C1, V * c1s, c1s, 0, n->D1, V * w1, w1, 0, 0, 0, false));
    ERT_TRY(conv(n, 9, n->D1, V * w1, w1, 0, n->D1b, V * w1, w1, 0, 0, 0, false));
    hipLaunchKernelGGL(k_head, dim3(nblocks(V), B), dim3(256), 0, n->s, (const float*)n->D1b, V * w1, w1,
                       (const float*)(n->P + n->L[10].w_off), (const float*)(n->P + n->L[10].b_off), n->Y, V);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

// loss and gradient (n->G) for corrections e of residuals r (FP64 N x B), after forward()
ert_status backward(NetImpl* n, const double* r, const double* e)
{
    const int w1 = n->w1, w2 = n->w2, w3 = n->w3, B = n->B_run;
    const long V = n->V, V2 = n->V2, V4 = n->V4;
    const int c1s = w2 + w1, c2s = w3 + w2;
    const int n0 = n->n[0], n1 = n->n[1], n2 = n->n[2];
    // every layer's output gradient keeps a buffer of its own until the weight gradients
    DwLayers W;
    wgrad_shapes(n, B, W);
    hipLaunchKernelGGL(k_loss_partial, dim3(n->red_blk, B), dim3(256), 0, n->s, (const float*)n->Y, e, r,
                       (const double*)n->scale, V, n->T, n->red, n->red_blk);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(64), 0, n->s, (const double*)n->red, n->red_blk, B, n->tt, n->loss);
    // head: gY and the masked gradient of L10's output (Gf1)
    hipLaunchKernelGGL(k_head_grad, dim3(nblocks(V * w1 / 4), B), dim3(256), 0, n->s, (const float*)n->Y, (const float*)n->T,
                       (const double*)n->tt, B, V, (const float*)(n->P + n->L[10].w_off), (const float*)n->D1b, w1,
                       n->gY, n->Gf1);
    ERT_HIP(hipGetLastError());
    // L10
    wgrad(W, 9, n->D1, V * w1, w1, 0, n->Gf1, V * w1);
    ERT_TRY(conv(n, 9, n->Gf1, V * w1, w1, 0, n->Gf2, V * w1, w1, 0, 0, 1, true, n->D1, V * w1, w1, 0));
    // L9 (input: concat [up(D2b), s1])
    wgrad(W, 8, n->C1, V * c1s, c1s, 0, n->Gf2, V * w1);
    ERT_TRY(conv(n, 8, n->Gf2, V * w1, w1, 0, n->GC1, V * c1s, c1s, 0, 0, 2, true));
    hipLaunchKernelGGL(k_up2_grad_mask, dim3(nblocks(V2 * w2), B), dim3(256), 0, n->s, (const float*)n->GC1, V * c1s,
                       c1s, 0, w2, (const float*)n->D2b, V2 * w2, n->Gh1, V2 * w2, n0, n1, n2);
    // L8
    wgrad(W, 7, n->D2, V2 * w2, w2, 0, n->Gh1, V2 * w2);
    ERT_TRY(conv(n, 7, n->Gh1, V2 * w2, w2, 0, n->Gh2, V2 * w2, w2, 0, 1, 1, true, n->D2, V2 * w2, w2, 0));
    // L7 (input: concat [up(A3b), s2])
    wgrad(W, 6, n->C2, V2 * c2s, c2s, 0, n->Gh2, V2 * w2);
    ERT_TRY(conv(n, 6, n->Gh2, V2 * w2, w2, 0, n->GC2, V2 * c2s, c2s, 0, 1, 2, true));
    hipLaunchKernelGGL(k_up2_grad_mask, dim3(nblocks(V4 * w3), B), dim3(256), 0, n->s, (const float*)n->GC2,
                       V2 * c2s, c2s, 0, w3, (const float*)n->A3b, V4 * w3, n->Gq1, V4 * w3, n0 / 2, n1 / 2, n2 / 2);
    // L6
    wgrad(W, 5, n->A3, V4 * w3, w3, 0, n->Gq1, V4 * w3);
    ERT_TRY(conv(n, 5, n->Gq1, V4 * w3, w3, 0, n->Gq2, V4 * w3, w3, 0, 2, 1, true, n->A3, V4 * w3, w3, 0));
    // L5 (input: pool(s2)); its input gradient has w2 channels
    wgrad(W, 4, n->P2, V4 * w2, w2, 0, n->Gq2, V4 * w3);
    ERT_TRY(conv(n, 4, n->Gq2, V4 * w3, w3, 0, n->gP2, V4 * w2, w2, 0, 2, 2, true));
    hipLaunchKernelGGL(k_pool2_grad_add_mask, dim3(nblocks(V2 * w2), B), dim3(256), 0, n->s, (const float*)n->GC2,
                       V2 * c2s, c2s, w3, (const float*)n->gP2, V4 * w2, (const float*)n->C2, V2 * c2s, c2s, w3, w2,
                       n->Gh3, V2 * w2, n0 / 2, n1 / 2, n2 / 2);
    // L4
    wgrad(W, 3, n->A2, V2 * w2, w2, 0, n->Gh3, V2 * w2);
    ERT_TRY(conv(n, 3, n->Gh3, V2 * w2, w2, 0, n->Gh4, V2 * w2, w2, 0, 1, 1, true, n->A2, V2 * w2, w2, 0));
    // L3 (input: pool(s1)); its input gradient has w1 channels
    wgrad(W, 2, n->P1, V2 * w1, w1, 0, n->Gh4, V2 * w2);
    ERT_TRY(conv(n, 2, n->Gh4, V2 * w2, w2, 0, n->gP1, V2 * w1, w1, 0, 1, 2, true));
    hipLaunchKernelGGL(k_pool2_grad_add_mask, dim3(nblocks(V * w1), B), dim3(256), 0, n->s, (const float*)n->GC1,
                       V * c1s, c1s, w2, (const float*)n->gP1, V2 * w1, (const float*)n->C1, V * c1s, c1s, w2, w1,
                       n->Gf3, V * w1, n0, n1, n2);
    // L2
    wgrad(W, 1, n->A1, V * w1, w1, 0, n->Gf3, V * w1);
    ERT_TRY(conv(n, 1, n->Gf3, V * w1, w1, 0, n->Gf4, V * w1, w1, 0, 0, 1, true, n->A1, V * w1, w1, 0));
    // L1 (features; no input gradient)
    wgrad(W, 0, n->X, V * kCinPad, kCinPad, 0, n->Gf4, V * w1);
    return weight_gradients(n, W, n->D1b, n->gY);
}

}  // namespace

// Solver-side use: z = M(r) for one residual column on the plan's media (grid pn).
// A network on the plan's grid coarsened by f (pn = f n) acts on the cell averages of
// r, sigma_t and sigma_s over f^3 blocks, and its output is extended piecewise
// constant: z = r + P(s_c y(R r)).
ert_status net_precond(NetImpl* n, const double* r, const double* st, const double* ss, double* z, hipStream_t s,
                       const int* pn)
{
    const int f = pn[0] / n->n[0];
    hipStream_t keep = n->s;
    n->s = s;
    n->B_run = 1;
    ert_status st_ = ERT_OK;
    if (f > 1) {
        if (!n->coarse) st_ = n->alloc(&n->coarse, 3 * (size_t)n->V * sizeof(double));
        if (st_ == ERT_OK) st_ = restrict_avg(s, r, pn, f, n->coarse, 1);
        if (st_ == ERT_OK) st_ = restrict_avg(s, st, pn, f, n->coarse + n->V, 1);
        if (st_ == ERT_OK) st_ = restrict_avg(s, ss, pn, f, n->coarse + 2 * n->V, 1);
        if (st_ == ERT_OK) st_ = features(n, n->coarse, n->coarse + n->V, n->coarse + 2 * n->V, 0);
    } else {
        st_ = features(n, r, st, ss, 0);
    }
    if (st_ == ERT_OK) st_ = forward(n);
    if (st_ == ERT_OK) {
        if (f > 1) {
            const long N = (long)pn[0] * pn[1] * pn[2];
            hipLaunchKernelGGL(k_out_prolong, dim3(nblocks(N), 1), dim3(256), 0, s, (const float*)n->Y, r,
                               (const double*)n->scale, pn[0], pn[1], pn[2], f, z);
        } else {
            hipLaunchKernelGGL(k_out, dim3(nblocks(n->V), 1), dim3(256), 0, s, (const float*)n->Y, r,
                               (const double*)n->scale, n->V, z);
        }
        if (hipGetLastError() != hipSuccess) st_ = ERT_EDEVICE;
    }
    n->s = keep;
    return st_;
}

const int* net_grid(const NetImpl* n) { return n->n; }

}  // namespace ertvie

using namespace ertvie;

struct ert_net_s : public NetImpl {};

namespace ertvie {
NetImpl* net_impl(ert_net_t net) { return static_cast<NetImpl*>(net); }
}  // namespace ertvie

extern "C" {

ERT_API long ert_net_param_count(const ert_net_opts* o)
{
    if (!o) return -1;
    const int w1 = o->width[0] ? o->width[0] : 16, w2 = o->width[1] ? o->width[1] : 32,
              w3 = o->width[2] ? o->width[2] : 64;
    const int sh[kNetLayers][3] = {{w1, 3, 3}, {w1, w1, 3}, {w2, w1, 3}, {w2, w2, 3}, {w3, w2, 3}, {w3, w3, 3},
                                   {w2, w3 + w2, 3}, {w2, w2, 3}, {w1, w2 + w1, 3}, {w1, w1, 3}, {1, w1, 1}};
    long c = 0;
    for (int i = 0; i < kNetLayers; ++i) c += (long)sh[i][0] * sh[i][1] * sh[i][2] * sh[i][2] * sh[i][2] + sh[i][0];
    return c;
}

ERT_API ert_status ert_net_create(const ert_net_opts* o, void* hip_stream, ert_net_t* out)
{
    if (!o || !out) {
        record_error("ert_net_create: null argument");
        return ERT_EINVAL;
    }
    *out = nullptr;
    const int w1 = o->width[0] ? o->width[0] : 16, w2 = o->width[1] ? o->width[1] : 32,
              w3 = o->width[2] ? o->width[2] : 64;
    if (o->dim != 3) {
        record_error("ert_net_create: the network is three-dimensional (dim must be 3)");
        return o->dim == 2 ? ERT_EUNSUPPORTED : ERT_EINVAL;
    }
    for (int a = 0; a < 3; ++a)
        if (o->n[a] < 4 || o->n[a] % 4 != 0) {
            record_error("ert_net_create: every grid extent must be a positive multiple of 4");
            return ERT_EINVAL;
        }
    if (w1 % 16 || w2 % 16 || w3 % 16 || w1 > 128 || w2 > 128 || w3 > 128 || w1 < 16 || w2 < 16 || w3 < 16) {
        record_error("ert_net_create: widths must be multiples of 16 in [16, 128]");
        return ERT_EINVAL;
    }
    for (int i = 0; i < 4; ++i)
        if (o->reserved[i]) {
            record_error("ert_net_create: reserved fields must be 0");
            return ERT_EINVAL;
        }
    const int B = o->batch_max > 0 ? o->batch_max : 1;
    ert_net_s* n = new (std::nothrow) ert_net_s();
    if (!n) return ERT_ENOMEM;
    n->o = *o;
    n->s = (hipStream_t)hip_stream;
    for (int a = 0; a < 3; ++a) n->n[a] = o->n[a];
    n->V = (long)o->n[0] * o->n[1] * o->n[2];
    n->V2 = n->V / 8;
    n->V4 = n->V / 64;
    n->B = B;
    n->w1 = w1; n->w2 = w2; n->w3 = w3;
    const int sh[kNetLayers][3] = {{w1, 3, 3}, {w1, w1, 3}, {w2, w1, 3}, {w2, w2, 3}, {w3, w2, 3}, {w3, w3, 3},
                                   {w2, w3 + w2, 3}, {w2, w2, 3}, {w1, w2 + w1, 3}, {w1, w1, 3}, {1, w1, 1}};
    long off = 0;
    ert_status st = ERT_OK;
    for (int i = 0; i < kNetLayers && st == ERT_OK; ++i) {
        NetLayer& l = n->L[i];
        l.cout = sh[i][0];
        l.cin_real = sh[i][1];
        l.cin = i == 0 ? kCinPad : l.cin_real;
        l.k = sh[i][2];
        l.w_off = off;
        off += (long)l.cout * l.cin_real * l.k * l.k * l.k;
        l.b_off = off;
        off += l.cout;
        if (l.k == 3) {
            l.Kpad = (27 * l.cin + 31) / 32 * 32;
            st = n->alloc(&l.Wf, (size_t)l.cout * l.Kpad * sizeof(__bf16));
            if (i > 0 && st == ERT_OK) {
                l.KpadB = (27 * l.cout + 31) / 32 * 32;
                st = n->alloc(&l.Wb, (size_t)l.cin * l.KpadB * sizeof(__bf16));
            }
        }
    }
    n->nparam = off;
    const long V = n->V, V2 = n->V2, V4 = n->V4;
    auto fl = [&](float** p, long elems) {
        if (st == ERT_OK) st = n->alloc(p, (size_t)elems * B * sizeof(float));
    };
    if (st == ERT_OK) st = n->alloc(&n->P, n->nparam * sizeof(float));
    if (st == ERT_OK) st = n->alloc(&n->G, n->nparam * sizeof(float));
    if (st == ERT_OK) st = n->alloc(&n->M, n->nparam * sizeof(float));
    if (st == ERT_OK) st = n->alloc(&n->Vv, n->nparam * sizeof(float));
    fl(&n->X, V * kCinPad);
    fl(&n->A1, V * w1);
    fl(&n->C1, V * (w2 + w1));
    fl(&n->P1, V2 * w1);
    fl(&n->A2, V2 * w2);
    fl(&n->C2, V2 * (w3 + w2));
    fl(&n->P2, V4 * w2);
    fl(&n->A3, V4 * w3);
    fl(&n->A3b, V4 * w3);
    fl(&n->D2, V2 * w2);
    fl(&n->D2b, V2 * w2);
    fl(&n->D1, V * w1);
    fl(&n->D1b, V * w1);
    fl(&n->Y, V);
    fl(&n->T, V);
    fl(&n->gY, V);
    fl(&n->Gf1, V * w1);
    fl(&n->Gf2, V * w1);
    fl(&n->GC1, V * (w2 + w1));
    fl(&n->Gh1, V2 * w2);
    fl(&n->Gh2, V2 * w2);
    fl(&n->GC2, V2 * (w3 + w2));
    fl(&n->Gq1, V4 * w3);
    fl(&n->Gq2, V4 * w3);
    fl(&n->gP2, V4 * w2);
    fl(&n->Gh3, V2 * w2);
    fl(&n->Gh4, V2 * w2);
    fl(&n->gP1, V2 * w1);
    fl(&n->Gf3, V * w1);
    fl(&n->Gf4, V * w1);
    // partial weight gradients: a layer's slabs are most for some batch up to B
    size_t need = 0;
    {
        int most[kNetLayers - 1] = {};
        DwLayers G;
        for (int q = 1; q <= B; ++q) {
            wgrad_shapes(n, q, G);
            for (int i = 0; i < kNetLayers - 1; ++i) most[i] = std::max(most[i], G.l[i].nslab);
        }
        for (int i = 0; i < kNetLayers; ++i) {
            n->L[i].part_off = need;
            need += i < kNetLayers - 1 ? (size_t)most[i] * G.l[i].npair * kPairVals : (size_t)kHeadSlabs * (n->L[i].cin + 1);
        }
    }
    if (st == ERT_OK) st = n->alloc(&n->part, need * sizeof(float));
    if (st == ERT_OK) st = n->alloc(&n->scale, (size_t)B * sizeof(double));
    if (st == ERT_OK) st = n->alloc(&n->tt, (size_t)B * sizeof(double));
    if (st == ERT_OK) st = n->alloc(&n->loss, sizeof(double));
    if (st == ERT_OK) st = n->alloc(&n->red, (size_t)B * n->red_blk * 2 * sizeof(double));
    if (st == ERT_OK && (hipMemsetAsync(n->P, 0, n->nparam * sizeof(float), n->s) != hipSuccess ||
                         hipMemsetAsync(n->M, 0, n->nparam * sizeof(float), n->s) != hipSuccess ||
                         hipMemsetAsync(n->Vv, 0, n->nparam * sizeof(float), n->s) != hipSuccess))
        st = ERT_EDEVICE;
    if (st != ERT_OK) {
        delete n;
        return st;
    }
    *out = n;
    return ERT_OK;
}

ERT_API long ert_net_size(ert_net_t net) { return net ? net->nparam : -1; }

ERT_API ert_status ert_net_set_params(ert_net_t net, const float* params)
{
    if (!net || !params) {
        record_error("ert_net_set_params: null argument");
        return ERT_EINVAL;
    }
    ERT_HIP(hipMemcpyAsync(net->P, params, net->nparam * sizeof(float), hipMemcpyHostToDevice, net->s));
    ERT_HIP(hipMemsetAsync(net->M, 0, net->nparam * sizeof(float), net->s));
    ERT_HIP(hipMemsetAsync(net->Vv, 0, net->nparam * sizeof(float), net->s));
    net->step = 0;
    ERT_TRY(prep_weights(net));
    ERT_HIP(hipStreamSynchronize(net->s));
    return ERT_OK;
}

ERT_API ert_status ert_net_get_params(ert_net_t net, float* params)
{
    if (!net || !params) {
        record_error("ert_net_get_params: null argument");
        return ERT_EINVAL;
    }
    ERT_HIP(hipMemcpyAsync(params, net->P, net->nparam * sizeof(float), hipMemcpyDeviceToHost, net->s));
    ERT_HIP(hipStreamSynchronize(net->s));
    return ERT_OK;
}

static ert_status net_check(ert_net_t net, const void* a, const void* b, int batch, const char* who)
{
    if (!net || !a || !b) {
        record_error(who);
        return ERT_EINVAL;
    }
    if (batch < 1 || batch > net->B) {
        record_error("net: batch outside 1..batch_max");
        return ERT_EINVAL;
    }
    return ERT_OK;
}

ERT_API ert_status ert_net_forward(ert_net_t net, const double* r, const double* sigma_t, const double* sigma_s,
                                   double* z, int batch)
{
    ERT_TRY(net_check(net, r, z, batch, "ert_net_forward: null argument"));
    if (!sigma_t || !sigma_s) {
        record_error("ert_net_forward: null medium");
        return ERT_EINVAL;
    }
    net->B_run = batch;
    ERT_TRY(features(net, r, sigma_t, sigma_s, 1));
    ERT_TRY(forward(net));
    hipLaunchKernelGGL(k_out, dim3(nblocks(net->V), batch), dim3(256), 0, net->s, (const float*)net->Y, r,
                       (const double*)net->scale, net->V, z);
    ERT_HIP(hipGetLastError());
    return ERT_OK;
}

ERT_API ert_status ert_net_grad(ert_net_t net, const double* r, const double* e, const double* sigma_t,
                                const double* sigma_s, int batch, double* loss, float* grad)
{
    ERT_TRY(net_check(net, r, e, batch, "ert_net_grad: null argument"));
    if (!sigma_t || !sigma_s) {
        record_error("ert_net_grad: null medium");
        return ERT_EINVAL;
    }
    net->B_run = batch;
    ERT_TRY(features(net, r, sigma_t, sigma_s, 1));
    ERT_TRY(forward(net));
    ERT_TRY(backward(net, r, e));
    if (loss) ERT_HIP(hipMemcpyAsync(loss, net->loss, sizeof(double), hipMemcpyDeviceToHost, net->s));
    if (grad) ERT_HIP(hipMemcpyAsync(grad, net->G, net->nparam * sizeof(float), hipMemcpyDeviceToHost, net->s));
    ERT_HIP(hipStreamSynchronize(net->s));
    return ERT_OK;
}

ERT_API ert_status ert_net_train_step(ert_net_t net, const double* r, const double* e, const double* sigma_t,
                                      const double* sigma_s, int batch, const ert_net_train_opts* opts, double* loss)
{
    ERT_TRY(net_check(net, r, e, batch, "ert_net_train_step: null argument"));
    if (!sigma_t || !sigma_s || !opts) {
        record_error("ert_net_train_step: null medium or options");
        return ERT_EINVAL;
    }
    const double lr = opts->lr > 0 ? opts->lr : 1e-3, b1 = opts->beta1 > 0 ? opts->beta1 : 0.9,
                 b2 = opts->beta2 > 0 ? opts->beta2 : 0.999, eps = opts->eps > 0 ? opts->eps : 1e-8;
    if (!(lr < 1.0) || !(b1 < 1.0) || !(b2 < 1.0)) {
        record_error("ert_net_train_step: lr, beta1 and beta2 must lie in (0, 1)");
        return ERT_EINVAL;
    }
    net->B_run = batch;
    ERT_TRY(features(net, r, sigma_t, sigma_s, 1));
    ERT_TRY(forward(net));
    ERT_TRY(backward(net, r, e));
    net->step += 1;
    const float c1 = (float)(1.0 - std::pow(b1, (double)net->step)), c2 = (float)(1.0 - std::pow(b2, (double)net->step));
    hipLaunchKernelGGL(k_adam, dim3(nblocks(net->nparam)), dim3(256), 0, net->s, net->P, (const float*)net->G, net->M,
                       net->Vv, net->nparam, (float)lr, (float)b1, (float)b2, (float)eps, c1, c2);
    ERT_HIP(hipGetLastError());
    ERT_TRY(prep_weights(net));
    if (loss) {
        ERT_HIP(hipMemcpyAsync(loss, net->loss, sizeof(double), hipMemcpyDeviceToHost, net->s));
        ERT_HIP(hipStreamSynchronize(net->s));
    }
    return ERT_OK;
}

ERT_API void ert_net_destroy(ert_net_t net) { delete net; }

}  // extern "C"
