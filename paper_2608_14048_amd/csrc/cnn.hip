// cnn.hip -- the learned subgrid flux-correction closure of the coarse MHD step.
//
// An extension of this library, not part of the paper's method (the paper only
// remarks, Sec. "Discussion and Summary", that a neural surrogate could replace an
// expensive cell-local solve such as astrochemistry).  The construction around the
// network follows the method: the network sees the 8
// primitive channels of the coarse state at the start of a step and returns 15 face-
// flux corrections (rho, M_x, M_y, M_z, E through the low x, y and z face of each cell)
// and 3 edge-EMF corrections (E_x on edge (i, j-1/2, k-1/2), E_y on (i-1/2, j, k-1/2),
// E_z on (i-1/2, j-1/2, k)); they are added to the plain step in flux form (eq.
// (fv_update)) and in constrained-transport form (eq. (ct)), so the corrected step
// stays conservative and keeps div B.
//
// Network: 4 periodic 3x3x3 convolutions, widths 8 -> 32 -> 32 -> 32 -> 18, ReLU after
// the first three.  Every convolution is an implicit GEMM on the matrix cores: BF16
// operands, FP32 accumulation, v_mfma_f32_16x16x32_bf16 for the 32-channel inputs and
// v_mfma_f32_16x16x16_bf16 for the first layer's 16 (8 padded).  Activations are
// stored channel-last ([voxel][channel], channels padded to 16 or 32) so that one
// lane's K values are one 8- or 16-byte read.  Persistent workgroups hold the weight
// fragments of all 27 taps in registers and take 16 x 4 x 8 voxel blocks (flat ones on
// grids of few planes or rows) through LDS (k_conv).  The backward data pass is the
// same kernel on reflected, transposed weights with the ReLU mask of the layer below;
// the weight and bias gradients are a GEMM over voxels per tap (MFMA with K along
// voxels, k_grad) with one partial per workgroup.
// Master weights and Adam moments are FP32; the BF16 copies are refreshed after each
// update.
//
// Conventions (shared with the FP64 reference, implemented independently there): tap
// t = (dz+1)*9 + (dy+1)*3 + (dx+1); y[v][co] = b[co] + sum_{t,ci} W[t][ci][co] x[v+off(t)][ci];
// parameters in order, per layer: W [27][cin][cout], then b [cout].
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <new>
#include <vector>

#include "../../include/mhd950.h"
#include "launch.hpp"

using namespace mhd;

namespace {

constexpr int kLayers = 4;
constexpr int kCin[kLayers] = {8, 32, 32, 32};
constexpr int kCout[kLayers] = {32, 32, 32, 18};
constexpr int kCinPad[kLayers] = {16, 32, 32, 32};
constexpr int kNPad = 32;        // padded output width of every layer
constexpr int kThreads = 256;    // 4 wavefronts

typedef unsigned short bf16_t;
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

constexpr size_t layer_w(int l) { return (size_t)27 * kCin[l] * kCout[l]; }
constexpr size_t layer_params(int l) { return layer_w(l) + kCout[l]; }
size_t param_offset(int l)
{
    size_t o = 0;
    for (int q = 0; q < l; ++q) o += layer_params(q);
    return o;
}
size_t total_params() { return param_offset(kLayers); }

__device__ __forceinline__ bf16_t f2bf(float x)
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) return (bf16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even
    return (bf16_t)(u >> 16);
}
// two at once, the first in the low half (the hardware conversion: nearest even too)
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi)
{
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, bf2{(__bf16)lo, (__bf16)hi});
}
__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ int wrap1(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// i taken periodically into [0, n) from any distance
__device__ __forceinline__ int wrapn(int i, int n)
{
    const int r = i % n;
    return r < 0 ? r + n : r;
}

// voxel index of (x, y, z) displaced by tap t
__device__ __forceinline__ unsigned int tap_voxel(const Geo& g, int x, int y, int z, int t)
{
    const int dx = t % 3 - 1, dy = (t / 3) % 3 - 1, dz = t / 9 - 1;
    return ((unsigned int)wrap1(z + dz, g.nz) * (unsigned int)g.ny + (unsigned int)wrap1(y + dy, g.ny)) *
               (unsigned int)g.nx + (unsigned int)wrap1(x + dx, g.nx);
}

}  // namespace

namespace mhd {

// ----------------------------------------------------------------------------------
// kernels
// ----------------------------------------------------------------------------------

// Normalised primitive channels of a canonical FP64 state -> X0 [n][16] (8 used).
__global__ __launch_bounds__(kThreads) void k_cnn_input(Geo g, double gamma, const double* __restrict__ U,
                                                        const float* __restrict__ mu, const float* __restrict__ sd,
                                                        bf16_t* __restrict__ X0)
{
    const unsigned int c = blockIdx.x * kThreads + threadIdx.x;
    if (c >= (unsigned int)g.n) return;
    const unsigned int n = (unsigned int)g.n;
    const int x = (int)(c % (unsigned int)g.nx), y = (int)((c / (unsigned int)g.nx) % (unsigned int)g.ny);
    const int z = (int)(c / ((unsigned int)g.nx * (unsigned int)g.ny));
    const unsigned int cx = tap_voxel(g, x, y, z, 14), cy = tap_voxel(g, x, y, z, 16), cz = tap_voxel(g, x, y, z, 22);
    const double rho = U[c];
    const double v[3] = {U[n + c] / rho, U[2 * n + c] / rho, U[3 * n + c] / rho};
    const double b[3] = {0.5 * (U[5 * n + c] + U[5 * n + cx]), 0.5 * (U[6 * n + c] + U[6 * n + cy]),
                         0.5 * (U[7 * n + c] + U[7 * n + cz])};
    const double ke = 0.5 * rho * ((v[0] * v[0] + v[1] * v[1]) + v[2] * v[2]);
    const double p = (gamma - 1.0) * ((U[4 * n + c] - ke) - 0.5 * ((b[0] * b[0] + b[1] * b[1]) + b[2] * b[2]));
    const double w[8] = {rho, v[0], v[1], v[2], p, b[0], b[1], b[2]};
    // the voxel's 16 channels (8 used, 8 zero padding) as two 16-byte stores
    uint32_t h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        h[q] = (uint32_t)f2bf((float)((w[2 * q] - mu[2 * q]) / sd[2 * q])) |
               (uint32_t)f2bf((float)((w[2 * q + 1] - mu[2 * q + 1]) / sd[2 * q + 1])) << 16;
    uint4* o = reinterpret_cast<uint4*>(X0 + (size_t)c * 16);
    o[0] = uint4{h[0], h[1], h[2], h[3]};
    o[1] = uint4{0u, 0u, 0u, 0u};
}

// Y[v][nn] = sum_t sum_k X[v + off(t)][k] B[t][nn][k] (+ bias), 32 outputs.
// MODE 0: + bias, ReLU, store BF16 [n][32].  MODE 1: + bias, store FP32 planar O[nn][v]
// for nn < nstore.  MODE 2: times (M[v][nn] > 0), store BF16 [n][32].
//
// Persistent workgroups of eight waves, two per SIMD, so that a wave may hold 256
// registers: its 16 output channels' weight fragments of all 27 taps stay in them (108 at
// 32 input channels), read from memory once per wave instead of once per block.  A block
// is 16 x 4 x 8 voxels, its input with a one-voxel halo (18 x 6 x 10 voxels) is staged in
// LDS while the loads of the next block's are in flight, and wave w computes channels
// 16 (w % 2) .. of the 4 rows of planes 2 (w / 2) and the one above.  An input row's
// fragment is read once per dx and serves every (dy, dz) that reaches it: 72 LDS reads for
// 216 matrix instructions (one read per instruction when each tap read its own).  Every
// output still adds its taps in the order t = 0 .. 26.  Rows past the grid's edge are
// computed from any rows and not stored.  64^3, 32 -> 32 channels: 30.8 -> 22.2 us forward,
// 41.5 -> 24.5 us with the ReLU mask, against a block per workgroup of four waves that
// fetched each tap's weights from L2 (of 22 us about 7 are the launch and the staging of
// two blocks, 4 the weights, 10 the matrix instructions and their LDS reads).  The weight
// fragments are the first operand where the output is channel-last, so that a lane ends
// up with four channels of a voxel and stores 8 bytes.
//
// A block is GY x GZ groups of WY rows x WZ planes, two waves each: 2 x 4 (four rows, eight
// planes) above; a grid of few planes, or few rows, takes 32 rows of one plane, or one row
// of 32 planes, where 4 x 8 blocks would be mostly padding (see conv).
constexpr int kConvThreads = 512, kConvWaves = kConvThreads / 64;
constexpr int kConvGroups = 256;  // persistent workgroups at most: one per CU

template <int CINP>
struct ConvFrag;
template <>
struct ConvFrag<32> {
    typedef s8 T;
    // D rows are the first operand's, columns the second's
    __device__ static f4 mma(T a, T b, f4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
    }
};
template <>
struct ConvFrag<16> {
    typedef s4 T;
    __device__ static f4 mma(T a, T b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }
};

template <int CINP, int MODE, int WY, int WZ, int GY, int GZ>
__global__ __launch_bounds__(kConvThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_conv(
    Geo g, const bf16_t* __restrict__ X, const bf16_t* __restrict__ B, const float* __restrict__ bias,
    const bf16_t* __restrict__ M, bf16_t* __restrict__ Y, float* __restrict__ O, int nstore, unsigned int nty,
    unsigned int nblk)
{
    using Frag = ConvFrag<CINP>;
    using T = typename Frag::T;
    constexpr int KL = CINP / 4;                     // K values of a lane
    constexpr int CH = CINP / 8;                     // 16-byte chunks of a voxel
    static_assert(2 * GY * GZ == kConvWaves && WY * WZ == 8, "two waves a group, eight rows a wave");
    constexpr int TY = WY * GY, TZ = WZ * GZ;        // rows and planes of a block
    constexpr int HY = TY + 2, HZ = TZ + 2, ROWS = HY * HZ;
    constexpr int VY = WY + 2, VZ = WZ + 2;          // a wave's rows and planes with their halo
    constexpr int NR = (ROWS + kConvWaves - 1) / kConvWaves;
    // a wave stages rows w, w + 8, ..: one load for a row's first 16 voxels (all 18 where
    // they fit the 64 lanes), and one for the last two voxels of eight rows
    constexpr int MV = CH == 2 ? 18 : 16, NTAIL = CH == 2 ? 0 : (NR + 7) / 8;
    // chunk c of a voxel in column x sits at c ^ swz(x): sixteen consecutive voxels of one
    // chunk then spread over all banks
    __shared__ __align__(16) bf16_t sA[18 * ROWS * CINP];
    auto swz = [](int x) { return CINP == 32 ? (x >> 2) & 3 : (x >> 3) & 1; };
    const int lane = (int)threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // this wave's first row and plane in the block, and its channel half
    const int yp = (w >> 1) % GY * WY, zp = (w >> 1) / GY * WZ, cb = w & 1;
    const int lr = lane & 15, lg = lane >> 4;
    const unsigned int ntx = (unsigned int)g.nx / 16u, n = (unsigned int)g.n;

    const int mvox = lane / CH, mpos = lane % CH;          // this lane's voxel and chunk of a row
    const int tvox = 16 + (lane >> 2 & 1), tpos = lane & 3;  // and of a row's tail
    u4 v[NR], tail[NTAIL > 0 ? NTAIL : 1];
    auto fetch = [&](unsigned int blk) {
        const int x0 = (int)(blk % ntx) * 16, y0 = (int)((blk / ntx) % nty) * TY;
        const int z0 = (int)(blk / (ntx * nty)) * TZ;
        // first voxel of halo row r of the block (periodic)
        auto line = [&](int r) {
            int y = y0 + r % HY - 1, z = z0 + r / HY - 1;
            if (y < 0) y += g.ny;
            if (z < 0) z += g.nz;
            while (y >= g.ny) y -= g.ny;
            while (z >= g.nz) z -= g.nz;
            return ((unsigned int)z * (unsigned int)g.ny + (unsigned int)y) * (unsigned int)g.nx;
        };
        const unsigned int mo = (unsigned int)wrap1(x0 + mvox - 1, g.nx) * CINP + (mpos ^ swz(mvox)) * 8;
#pragma unroll
        for (int m = 0; m < NR; ++m) {
            const int r = w + kConvWaves * m;
            const bf16_t* p = X + (size_t)line(r < ROWS ? r : 0) * CINP;  // (row 0 again past the last)
            if (mvox < MV) v[m] = *reinterpret_cast<const u4*>(reinterpret_cast<const char*>(p) + mo * 2u);
        }
#pragma unroll
        for (int m = 0; m < NTAIL; ++m) {
            const int rr = m * 8 + (lane >> 3);
            if (w + kConvWaves * rr < ROWS) {
                const unsigned int gv = line(w + kConvWaves * rr) + (unsigned int)wrap1(x0 + tvox - 1, g.nx);
                tail[m] = *reinterpret_cast<const u4*>(X + (size_t)gv * CINP + (tpos ^ swz(tvox)) * 8);
            }
        }
    };
    fetch(blockIdx.x);  // the grid has at most nblk workgroups
    T wt[27];
#pragma unroll
    for (int t = 0; t < 27; ++t)  // (a scalar base and one lane offset: no address registers)
        wt[t] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(B + (t * kNPad + cb * 16) * CINP) +
                                            (unsigned int)(lr * CINP + lg * KL) * 2u);

    // where this lane reads the fragments of its first halo row (the others lie a constant
    // number of bytes further on)
    const bf16_t* a0[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        const int x = lr + dx, chunk = CINP == 32 ? lg : lg >> 1, part = CINP == 32 ? 0 : (lg & 1) * 4;
        a0[dx] = sA + ((zp * HY + yp) * 18 + x) * CINP + (chunk ^ swz(x)) * 8 + part;
    }

    for (unsigned int blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        __syncthreads();  // the block before is read
#pragma unroll
        for (int m = 0; m < NR; ++m)
            if (mvox < MV && w + kConvWaves * m < ROWS)
                *reinterpret_cast<u4*>(sA + (size_t)((w + kConvWaves * m) * 18 + mvox) * CINP + mpos * 8) = v[m];
#pragma unroll
        for (int m = 0; m < NTAIL; ++m) {
            const int rr = m * 8 + (lane >> 3);
            if (w + kConvWaves * rr < ROWS)
                *reinterpret_cast<u4*>(sA + (size_t)((w + kConvWaves * rr) * 18 + tvox) * CINP + tpos * 8) = tail[m];
        }
        __syncthreads();
        if (blk + gridDim.x < nblk) fetch(blk + gridDim.x);

        // acc[rb]: row yp + rb % WY of plane zp + rb / WY
        f4 acc[8];
#pragma unroll
        for (int rb = 0; rb < 8; ++rb) acc[rb] = f4{0.f, 0.f, 0.f, 0.f};
        // the fragments of input row r (row yp + r % VY of plane zp + r / VY of the halo
        // block), one per dx; those of row r + 1 are read while row r multiplies
        auto row = [&](int r, int dx) {
            return *reinterpret_cast<const T*>(a0[dx] + (r / VY * HY + r % VY) * (18 * CINP));
        };
        T cur[3], nxt[3];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) cur[dx] = nxt[dx] = row(0, dx);
#pragma unroll
        for (int r = 0; r < VY * VZ; ++r) {
            if (r + 1 < VY * VZ) {
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) nxt[dx] = row(r + 1, dx);
            }
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int z = 0; z < WZ; ++z)
#pragma unroll
                    for (int y = 0; y < WY; ++y) {
                        const int dz = r / VY - z, dy = r % VY - y;
                        if (dz < 0 || dz > 2 || dy < 0 || dy > 2) continue;
                        const int t = dz * 9 + dy * 3 + dx;
                        f4& d = acc[z * WY + y];
                        d = MODE == 1 ? Frag::mma(cur[dx], wt[t], d) : Frag::mma(wt[t], cur[dx], d);
                    }
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) cur[dx] = nxt[dx];
            __builtin_amdgcn_sched_barrier(0);  // (all rows' reads at once would not fit the registers)
        }
        // MODE 1: element i of lane l is voxel 4 (l / 16) + i of the row, channel l % 16;
        // else voxel l % 16, channel 4 (l / 16) + i: four voxels or four channels per store
        const int x0 = (int)(blk % ntx) * 16, y0 = (int)((blk / ntx) % nty) * TY + yp;
        const int z0 = (int)(blk / (ntx * nty)) * TZ + zp;
#pragma unroll
        for (int rb = 0; rb < 8; ++rb) {
            const int y = y0 + rb % WY, z = z0 + rb / WY;
            if (y >= g.ny || z >= g.nz) continue;
            const unsigned int vrow = ((unsigned int)z * (unsigned int)g.ny + (unsigned int)y) * (unsigned int)g.nx +
                                      (unsigned int)x0;
            const f4 a = acc[rb];
            if constexpr (MODE == 1) {
                const int nn = cb * 16 + lr;
                if (nn < nstore) {
                    const float b = bias[nn];
                    *reinterpret_cast<float4*>(O + (size_t)nn * n + vrow + lg * 4) =
                        float4{a[0] + b, a[1] + b, a[2] + b, a[3] + b};
                }
            } else {
                const size_t at = (size_t)(vrow + lr) * kNPad + cb * 16 + lg * 4;
                float o[4];
                if constexpr (MODE == 0) {
                    const float4 b = *reinterpret_cast<const float4*>(bias + cb * 16 + lg * 4);
                    o[0] = fmaxf(a[0] + b.x, 0.f); o[1] = fmaxf(a[1] + b.y, 0.f);
                    o[2] = fmaxf(a[2] + b.z, 0.f); o[3] = fmaxf(a[3] + b.w, 0.f);
                } else {
                    const uint2 mk = *reinterpret_cast<const uint2*>(M + at);
                    o[0] = __uint_as_float(mk.x << 16) > 0.f ? a[0] : 0.f;
                    o[1] = __uint_as_float(mk.x & 0xffff0000u) > 0.f ? a[1] : 0.f;
                    o[2] = __uint_as_float(mk.y << 16) > 0.f ? a[2] : 0.f;
                    o[3] = __uint_as_float(mk.y & 0xffff0000u) > 0.f ? a[3] : 0.f;
                }
                *reinterpret_cast<uint2*>(Y + at) = uint2{f2bf2(o[0], o[1]), f2bf2(o[2], o[3])};
            }
        }
    }
}

// Weight and bias gradients of one layer, dW[t][k][nn] = sum_v X[v + off(t)][k] D[v][nn]
// and db[nn] = sum_v D[v][nn], one partial per workgroup (k_grad_sum adds them up).
//
// A GEMM per tap with K along the voxels, v_mfma_f32_32x32x16_bf16 (lane l holds A row and
// B column l % 32 at K 8 (l / 32) + 0..7).  The operands are channel-last in memory and a
// lane needs eight voxels of one channel, so a block of 16 x 4 x 4 voxels (X with its
// one-voxel halo) is transposed into LDS once, four voxels per write, and all 27 taps
// read it there: wave w owns the three taps dx = -1, 0, 1 of one (dy, dz), which are three
// windows of the same ten voxels (dx = 0 is the odd one, shifted out of its neighbours).
// Nine waves, 48 accumulator registers each, kept over all the blocks a workgroup takes.
// 64^3, 32 -> 32 channels: gathering two bytes at a time for every tap with one atomic add
// per gradient and chunk took 239 us and the bias gradient's own pass 32; this takes 29,
// and 6 to add the partials up.  Two workgroups per CU (96 registers, spilling, twice the
// partials) took 38 + 9.
constexpr int kGradWaves = 9, kGradThreads = 64 * kGradWaves;
constexpr int kGradGroups = 256;  // workgroups at most (one per CU), each with its own partial
constexpr int kXRow = 10;                      // dwords of a staged X row: voxels x0 - 1 .. x0 + 16, padded
constexpr int kXStr = 36 * kXRow + 2;          // dwords of a channel (36 rows), bank-spread
constexpr int kDStr = 16 * 8 + 4;              // dwords of a D channel (16 rows of 16 voxels)

typedef float f16v __attribute__((ext_vector_type(16)));

// Eight channels of four voxels (v[j]: voxel j) transposed: q[c] = channel c's four voxels.
__device__ __forceinline__ void transpose_8x4(const u4 v[4], uint2 q[8])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const unsigned int a = v[0][c], b = v[1][c], d = v[2][c], e = v[3][c];
        q[2 * c] = uint2{(a & 0xffffu) | b << 16, (d & 0xffffu) | e << 16};
        q[2 * c + 1] = uint2{a >> 16 | (b & 0xffff0000u), d >> 16 | (e & 0xffff0000u)};
    }
}

template <int CINP>
__global__ __launch_bounds__(kGradThreads) void k_grad(Geo g, const bf16_t* __restrict__ X,
                                                       const bf16_t* __restrict__ D, float* __restrict__ part, int cin,
                                                       int cout, unsigned int nty, unsigned int nblk)
{
    constexpr int CH = CINP / 8;
    constexpr int XI = 36 * 5 * CH, DI = 16 * 4 * 4;  // staging items: 4 voxels x 8 channels
    __shared__ __align__(16) unsigned int sX[CINP * kXStr];
    __shared__ __align__(16) unsigned int sD[32 * kDStr];
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int lr = lane & 31, lh = lane >> 5;
    const int dy = w % 3, dz = w / 3;  // row offsets within the halo (0..2)
    const unsigned int ntx = (unsigned int)g.nx / 16u;
    f16v acc[3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    float bs = 0.f;  // bias gradient of channel lr over the rows this wave adds up

    // this thread's staging items of a block: loaded while the block before multiplies
    constexpr int NI = (XI + DI + kGradThreads - 1) / kGradThreads;
    u4 v[NI][4];
    auto fetch = [&](unsigned int blk) {
        const int x0 = (int)(blk % ntx) * 16, y0 = (int)((blk / ntx) % nty) * 4, z0 = (int)(blk / (ntx * nty)) * 4;
#pragma unroll
        for (int m = 0; m < NI; ++m) {
            const int it = tid + m * kGradThreads;
            const bool isx = it < XI;
            const int u = isx ? it : it - XI;
            const int c = isx ? u % CH : u & 3, gq = isx ? u / CH : u >> 2;
            const int grp = isx ? gq % 5 : gq & 3, row = isx ? gq / 5 : gq >> 2;
            const int ly = isx ? row % 6 - 1 : row & 3, lz = isx ? row / 6 - 1 : row >> 2;
            // rows past the grid's edge carry no gradient: D is zero there, X any row
            const bool live = isx || (u < DI && y0 + ly < g.ny && z0 + lz < g.nz);
            const unsigned int line = ((unsigned int)wrapn(z0 + lz, g.nz) * (unsigned int)g.ny +
                                       (unsigned int)wrapn(y0 + ly, g.ny)) * (unsigned int)g.nx;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int xi = grp * 4 + j;
                v[m][j] = u4{0u, 0u, 0u, 0u};
                if (isx) {
                    if (xi < 18)
                        v[m][j] = *reinterpret_cast<const u4*>(
                            X + (size_t)(line + (unsigned int)wrap1(x0 + xi - 1, g.nx)) * CINP + c * 8);
                } else if (live) {
                    v[m][j] = *reinterpret_cast<const u4*>(D + (size_t)(line + (unsigned int)(x0 + xi)) * kNPad + c * 8);
                }
            }
        }
    };
    auto stage = [&]() {
#pragma unroll
        for (int m = 0; m < NI; ++m) {
            const int it = tid + m * kGradThreads;
            if (it >= XI + DI) continue;
            const bool isx = it < XI;
            const int u = isx ? it : it - XI;
            const int c = isx ? u % CH : u & 3, gq = isx ? u / CH : u >> 2;
            const int grp = isx ? gq % 5 : gq & 3, row = isx ? gq / 5 : gq >> 2;
            uint2 q[8];
            transpose_8x4(v[m], q);
            unsigned int* dst = isx ? sX + (c * 8) * kXStr + row * kXRow + grp * 2 : sD + (c * 8) * kDStr + row * 8 + grp * 2;
            const int str = isx ? kXStr : kDStr;
#pragma unroll
            for (int k = 0; k < 8; ++k) *reinterpret_cast<uint2*>(dst + k * str) = q[k];
        }
    };
    fetch(blockIdx.x);  // the grid has at most nblk workgroups
    for (unsigned int blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        __syncthreads();  // the block before is read
        stage();
        __syncthreads();
        if (blk + gridDim.x < nblk) fetch(blk + gridDim.x);
        const bool rows = CINP >= 32 || lr < CINP;
        const unsigned int* xa = sX + (rows ? lr : 0) * kXStr + lh * 4;
        const unsigned int* da = sD + lr * kDStr + lh * 4;
#pragma unroll 2
        for (int r = 0; r < 16; ++r) {
            const unsigned int* xr = xa + ((dz + (r >> 2)) * 6 + dy + (r & 3)) * kXRow;
            uint2 p0 = *reinterpret_cast<const uint2*>(xr), p1 = *reinterpret_cast<const uint2*>(xr + 2);
            unsigned int p2 = xr[4];
            if (!rows) p0 = p1 = uint2{0u, 0u}, p2 = 0u;
            const u4 b = *reinterpret_cast<const u4*>(da + r * 8);
            const u4 am = {p0.x, p0.y, p1.x, p1.y}, ap = {p0.y, p1.x, p1.y, p2};
            u4 a0;
#pragma unroll
            for (int j = 0; j < 4; ++j) a0[j] = __builtin_amdgcn_alignbit(ap[j], am[j], 16);
            if (r % kGradWaves == w) {
#pragma unroll
                for (int j = 0; j < 4; ++j) bs += __uint_as_float(b[j] << 16) + __uint_as_float(b[j] & 0xffff0000u);
            }
            const bf8 bb = __builtin_bit_cast(bf8, b);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, am), bb, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a0), bb, acc[1], 0, 0, 0);
            acc[2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, ap), bb, acc[2], 0, 0, 0);
        }
    }
    // the partial in the layout of the layer's parameters: W [27][cin][cout], b [cout];
    // accumulator element i of lane l: row (k) 8 (i / 4) + 4 (l / 32) + i % 4, column l % 32
    float* o = part + (size_t)blockIdx.x * ((size_t)27 * cin * cout + cout);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int k = (i >> 2) * 8 + lh * 4 + (i & 3);
            if (k < cin && lr < cout) o[((size_t)(w * 3 + t) * cin + k) * cout + lr] = acc[t][i];
        }
    // bias: the waves' and half-waves' sums of a channel through LDS
    __syncthreads();
    float* sb = reinterpret_cast<float*>(sD);  // [wave][half][channel]
    sb[tid] = bs;
    __syncthreads();
    if (tid < cout) {
        float t = 0.f;
        for (int q = 0; q < 2 * kGradWaves; ++q) t += sb[q * 32 + tid];
        o[(size_t)27 * cin * cout + tid] = t;
    }
}

// G[e] += sum over the np partials of part[.][e], in FP64 and in a fixed order: 64
// gradients per workgroup, the partials split over its four waves.
__global__ __launch_bounds__(kThreads) void k_grad_sum(const float* __restrict__ part, unsigned int ne, int np,
                                                       float* __restrict__ G)
{
    __shared__ double s[kThreads];
    const unsigned int e = blockIdx.x * 64 + (threadIdx.x & 63);
    double t = 0.0;
    if (e < ne) {
        const float* p = part + e;
#pragma unroll 8
        for (int q = (int)(threadIdx.x >> 6); q < np; q += 4) t += (double)p[(size_t)q * ne];
    }
    s[threadIdx.x] = t;
    __syncthreads();
    if (threadIdx.x < 64 && e < ne)
        G[e] += (float)((s[threadIdx.x] + s[threadIdx.x + 64]) + (s[threadIdx.x + 128] + s[threadIdx.x + 192]));
}

// The closure in flux and constrained-transport form: the corrected value of field q of
// cell c (q < 5: the cell field minus dt times the divergence of the face-flux
// corrections; q >= 5: the face field minus dt times the curl of the edge-EMF
// corrections).  Shared by the check and the update so that both see the same bits.
struct CorrIdx {
    unsigned int c, cp[3];  // the cell and its +x, +y, +z neighbours
};
__device__ __forceinline__ CorrIdx corr_idx(const Geo& g, unsigned int c)
{
    const int x = (int)(c % (unsigned int)g.nx), y = (int)((c / (unsigned int)g.nx) % (unsigned int)g.ny);
    const int z = (int)(c / ((unsigned int)g.nx * (unsigned int)g.ny));
    return CorrIdx{c, {tap_voxel(g, x, y, z, 14), tap_voxel(g, x, y, z, 16), tap_voxel(g, x, y, z, 22)}};
}
__device__ __forceinline__ double corrected(const Geo& g, const float* __restrict__ O, const float* __restrict__ sF,
                                            float sE, double dt, const double* __restrict__ U, const CorrIdx& k, int q)
{
    const unsigned int n = (unsigned int)g.n, c = k.c;
    if (q < 5) {
        double div = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float* o = O + (size_t)(3 * q + d) * n;
            div += (double)sF[q] * ((double)o[k.cp[d]] - (double)o[c]) * g.inv_dx[d];
        }
        return U[(size_t)q * n + c] - dt * div;
    }
    const float* Ex = O + (size_t)15 * n;
    const float* Ey = O + (size_t)16 * n;
    const float* Ez = O + (size_t)17 * n;
    auto dE = [&](const float* e, int d) { return (double)sE * ((double)e[k.cp[d]] - (double)e[c]) * g.inv_dx[d]; };
    const double curl = q == 5 ? dE(Ez, 1) - dE(Ey, 2) : (q == 6 ? dE(Ex, 2) - dE(Ez, 0) : dE(Ey, 0) - dE(Ex, 1));
    return U[(size_t)q * n + c] - dt * curl;
}

// The closure on a canonical FP64 state, in place (each thread writes only its own cell
// and faces; O is read-only).  With ok non-null nothing is written unless *ok > 0.
__global__ __launch_bounds__(kThreads) void k_closure_apply(Geo g, const float* __restrict__ O, const float* __restrict__ sF,
                                                            float sE, double dt, double* __restrict__ U,
                                                            const double* __restrict__ ok)
{
    const unsigned int c = blockIdx.x * kThreads + threadIdx.x;
    if (c >= (unsigned int)g.n) return;
    if (ok && !(ok[0] > 0.0)) return;
    const CorrIdx k = corr_idx(g, c);
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = corrected(g, O, sF, sE, dt, U, k, q);
#pragma unroll
    for (int q = 0; q < 8; ++q) U[(size_t)q * g.n + c] = v[q];
}

// Whether the closure would leave cell c valid: every corrected value finite, the density
// and the pressure (from the corrected total energy, momenta and the mean of the
// corrected bounding faces) at or above the floors.  One partial per workgroup: +inf if
// all its cells are valid, else -1.
__global__ __launch_bounds__(kThreads) void k_closure_check(Geo g, const float* __restrict__ O, const float* __restrict__ sF,
                                                            float sE, double dt, const double* __restrict__ U,
                                                            double gamma, double rho_floor, double p_floor,
                                                            double* __restrict__ partial)
{
    const unsigned int c = blockIdx.x * kThreads + threadIdx.x;
    bool good = true;
    if (c < (unsigned int)g.n) {
        const CorrIdx k = corr_idx(g, c);
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = corrected(g, O, sF, sE, dt, U, k, q);
        const double hi[3] = {corrected(g, O, sF, sE, dt, U, corr_idx(g, k.cp[0]), 5),
                              corrected(g, O, sF, sE, dt, U, corr_idx(g, k.cp[1]), 6),
                              corrected(g, O, sF, sE, dt, U, corr_idx(g, k.cp[2]), 7)};
        double bb = 0.0, mm = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double b = 0.5 * (v[5 + d] + hi[d]);
            bb += b * b;
            mm += v[1 + d] * v[1 + d];
        }
        const double p = (gamma - 1.0) * (v[4] - 0.5 * mm / v[0] - 0.5 * bb);
        for (int q = 0; q < 8; ++q) good = good && isfinite(v[q]);
        good = good && isfinite(hi[0]) && isfinite(hi[1]) && isfinite(hi[2]);
        good = good && v[0] >= rho_floor && p >= p_floor && isfinite(p);
    }
    __shared__ int bad;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    if (!good) atomicOr(&bad, 1);
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = bad ? -1.0 : INFINITY;
}

// With P the corrected value of the state U (k_closure_apply's, formed here instead of
// stored and read back): rw[f][c] = 2 w_f (P - T) / n and the loss partial
// sum_f w_f (P - T)^2 / n per block.
__global__ __launch_bounds__(kThreads) void k_residual(Geo g, const float* __restrict__ O, const float* __restrict__ sF,
                                                       float sE, double dt, const double* __restrict__ U,
                                                       const double* __restrict__ T, const float* __restrict__ w8,
                                                       float* __restrict__ RW, double* __restrict__ partial)
{
    __shared__ double s[kThreads / 64];
    const unsigned int c = blockIdx.x * kThreads + threadIdx.x;
    const unsigned int n = (unsigned int)g.n;
    double l = 0.0;
    if (c < n) {
        const CorrIdx k = corr_idx(g, c);
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            const double r = corrected(g, O, sF, sE, dt, U, k, f) - T[(size_t)f * n + c];
            RW[(size_t)f * n + c] = (float)(2.0 * w8[f] * r / (double)n);
            l += w8[f] * r * r / (double)n;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (s[0] + s[1]) + (s[2] + s[3]);
}

// d(loss)/d(output channel) through the adjoints of the closure, as BF16 [n][32].
__global__ __launch_bounds__(kThreads) void k_out_grad(Geo g, const float* __restrict__ RW, const float* __restrict__ sF,
                                                       float sE, double dt, bf16_t* __restrict__ D)
{
    const unsigned int c = blockIdx.x * kThreads + threadIdx.x;
    if (c >= (unsigned int)g.n) return;
    const unsigned int n = (unsigned int)g.n;
    const int x = (int)(c % (unsigned int)g.nx), y = (int)((c / (unsigned int)g.nx) % (unsigned int)g.ny);
    const int z = (int)(c / ((unsigned int)g.nx * (unsigned int)g.ny));
    // c - e_d
    const unsigned int cm[3] = {tap_voxel(g, x, y, z, 12), tap_voxel(g, x, y, z, 10), tap_voxel(g, x, y, z, 4)};
    // the voxel's 32 channels leave as four 16-byte stores
    bf16_t o[kNPad];
    // dF_fd[c] enters u_f[c] with +dt/dx_d and u_f[c - e_d] with -dt/dx_d
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        const float* r = RW + (size_t)f * n;
#pragma unroll
        for (int d = 0; d < 3; ++d)
            o[3 * f + d] = f2bf((float)((double)sF[f] * dt * g.inv_dx[d] * ((double)r[c] - (double)r[cm[d]])));
    }
    const float* gx = RW + (size_t)5 * n;
    const float* gy = RW + (size_t)6 * n;
    const float* gz = RW + (size_t)7 * n;
    auto dd = [&](const float* r, int d) { return dt * g.inv_dx[d] * ((double)r[c] - (double)r[cm[d]]); };
    o[15] = f2bf((float)(sE * (dd(gy, 2) - dd(gz, 1))));
    o[16] = f2bf((float)(sE * (dd(gz, 0) - dd(gx, 2))));
    o[17] = f2bf((float)(sE * (dd(gx, 1) - dd(gy, 0))));
#pragma unroll
    for (int q = 18; q < kNPad; ++q) o[q] = 0;
    uint4* d4 = reinterpret_cast<uint4*>(D + (size_t)c * kNPad);
#pragma unroll
    for (int q = 0; q < kNPad / 8; ++q) {
        const bf16_t* h = o + 8 * q;
        d4[q] = uint4{h[0] | (uint32_t)h[1] << 16, h[2] | (uint32_t)h[3] << 16, h[4] | (uint32_t)h[5] << 16,
                      h[6] | (uint32_t)h[7] << 16};
    }
}

// BF16 weight copies of layer l from the FP32 master: forward Wf[t][nn][k] = W[t][k][nn];
// backward Wb[t][nn=ci][k=co] = W[27-1-t][ci][co] (reflected tap).  Zero padded.
__global__ __launch_bounds__(kThreads) void k_pack_weights(const float* __restrict__ W, int cin, int cout, int cinp,
                                                           bf16_t* __restrict__ Wf, bf16_t* __restrict__ Wb)
{
    const unsigned int q = blockIdx.x * kThreads + threadIdx.x;
    if (q >= 27u * kNPad * (unsigned int)cinp) return;
    const int k = (int)(q % (unsigned int)cinp), nn = (int)((q / (unsigned int)cinp) % kNPad), t = (int)(q / ((unsigned int)cinp * kNPad));
    Wf[q] = (k < cin && nn < cout) ? f2bf(W[((size_t)t * cin + k) * cout + nn]) : (bf16_t)0;
    if (Wb) {
        // Wb[t][nn][k] with nn = ci (< cin), k = co (< cout); cinp == 32 == kNPad here
        const int ci = nn, co = k;
        Wb[q] = (ci < cin && co < cout) ? f2bf(W[((size_t)(26 - t) * cin + ci) * cout + co]) : (bf16_t)0;
    }
}

__global__ __launch_bounds__(kThreads) void k_adam(unsigned int np, float* __restrict__ P, const float* __restrict__ G,
                                                   float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                                   float b2, float eps, float c1, float c2, float gscale)
{
    const unsigned int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= np) return;
    const float gr = G[i] * gscale;
    const float mi = b1 * m[i] + (1.f - b1) * gr;
    const float vi = b2 * v[i] + (1.f - b2) * gr * gr;
    m[i] = mi;
    v[i] = vi;
    P[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// Box filter of a fine canonical state (r^3 cells, r^2 faces) onto the coarse grid.
__global__ __launch_bounds__(kThreads) void k_box_filter(Geo fine, Geo coarse, int r, const double* __restrict__ Fs,
                                                         double* __restrict__ Cs)
{
    const unsigned int c = blockIdx.x * kThreads + threadIdx.x;
    if (c >= (unsigned int)coarse.n) return;
    const unsigned int nf = (unsigned int)fine.n, nc = (unsigned int)coarse.n;
    const int X = (int)(c % (unsigned int)coarse.nx), Y = (int)((c / (unsigned int)coarse.nx) % (unsigned int)coarse.ny);
    const int Z = (int)(c / ((unsigned int)coarse.nx * (unsigned int)coarse.ny));
    auto fat = [&](int x, int y, int z) {
        return ((unsigned int)z * (unsigned int)fine.ny + (unsigned int)y) * (unsigned int)fine.nx + (unsigned int)x;
    };
    const double inv3 = 1.0 / (double)(r * r * r), inv2 = 1.0 / (double)(r * r);
    for (int f = 0; f < 5; ++f) {
        double s = 0.0;
        for (int k = 0; k < r; ++k)
            for (int j = 0; j < r; ++j)
                for (int i = 0; i < r; ++i) s += Fs[(size_t)f * nf + fat(X * r + i, Y * r + j, Z * r + k)];
        Cs[(size_t)f * nc + c] = s * inv3;
    }
    double sx = 0.0, sy = 0.0, sz = 0.0;
    for (int a = 0; a < r; ++a)
        for (int b = 0; b < r; ++b) {
            sx += Fs[(size_t)5 * nf + fat(X * r, Y * r + b, Z * r + a)];
            sy += Fs[(size_t)6 * nf + fat(X * r + b, Y * r, Z * r + a)];
            sz += Fs[(size_t)7 * nf + fat(X * r + b, Y * r + a, Z * r)];
        }
    Cs[(size_t)5 * nc + c] = sx * inv2;
    Cs[(size_t)6 * nc + c] = sy * inv2;
    Cs[(size_t)7 * nc + c] = sz * inv2;
}

}  // namespace mhd

// ----------------------------------------------------------------------------------
// host runtime
// ----------------------------------------------------------------------------------

struct mhd_cnn {
    Geo g;
    double gamma;
    hipStream_t stream;
    size_t np;
    float *P, *G, *M1, *M2;  // parameters, gradients, Adam moments (FP32, canonical order)
    bf16_t* Wf[kLayers];
    bf16_t* Wb[kLayers];     // layers 1..3
    bf16_t* A[kLayers];      // layer inputs: A[0] = X0 [n][16], A[l] [n][32]
    float* O;                // output channels [18][n]
    bf16_t *D0, *D1;         // backward gradients [n][32]
    float* RW;               // weighted residual [8][n]
    double* partial;
    float* gpart;            // gradient partials, one layer at a time
    float* scal;             // mu[8], sd[8], sF[5], w8[8]
    float sE;
    unsigned int nblk;
};

namespace {

size_t ca(size_t b) { return (b + 255) & ~size_t(255); }

struct CLayout {
    size_t params, wf[kLayers], wb[kLayers], a[kLayers], o, d, rw, partial, gpart, scal, total;
};

// Blocks of 16 x 4 x 4 voxels of the gradient kernel and the workgroups that share them.
unsigned int grad_blocks(int nx, int ny, int nz)
{
    return (unsigned int)(nx / 16) * (unsigned int)((ny + 3) / 4) * (unsigned int)((nz + 3) / 4);
}
unsigned int grad_groups(unsigned int nblk) { return nblk < (unsigned int)kGradGroups ? nblk : (unsigned int)kGradGroups; }

CLayout clayout(const mhd_grid* g)
{
    const size_t n = (size_t)g->nx * g->ny * g->nz;
    CLayout L;
    L.params = ca(total_params() * sizeof(float));
    for (int l = 0; l < kLayers; ++l) {
        L.wf[l] = ca((size_t)27 * kNPad * kCinPad[l] * sizeof(bf16_t));
        L.wb[l] = l > 0 ? ca((size_t)27 * kNPad * kNPad * sizeof(bf16_t)) : 0;
        L.a[l] = ca(n * (l == 0 ? 16 : kNPad) * sizeof(bf16_t));
    }
    L.o = ca(n * 18 * sizeof(float));
    L.d = ca(n * kNPad * sizeof(bf16_t));
    L.rw = ca(n * 8 * sizeof(float));
    L.partial = ca(((n + kThreads - 1) / kThreads + 1) * sizeof(double));  // + the closure's flag
    L.gpart = ca((size_t)grad_groups(grad_blocks(g->nx, g->ny, g->nz)) * layer_params(1) * sizeof(float));
    L.scal = ca(64 * sizeof(float));
    L.total = 4 * L.params + L.o + 2 * L.d + L.rw + L.partial + L.gpart + L.scal;
    for (int l = 0; l < kLayers; ++l) L.total += L.wf[l] + L.wb[l] + L.a[l];
    return L;
}

mhd_status cvalidate(const mhd_grid* g, const mhd_physics* p)
{
    if (!g || !p) return MHD_E_INVAL;
    if (g->nx < 16 || g->ny < 1 || g->nz < 1) return MHD_E_INVAL;
    if (g->nx % 16 != 0) return MHD_E_UNSUPPORTED;  // MFMA row blocks of 16 voxels along x
    for (int a = 0; a < 3; ++a)
        if (!(g->length[a] > 0.0) || !std::isfinite(g->length[a])) return MHD_E_INVAL;
    if ((long long)g->nx * g->ny * g->nz >= (1LL << 26)) return MHD_E_UNSUPPORTED;
    if (p->eos != MHD_EOS_ADIABATIC_MHD || !(p->gamma > 1.0)) return MHD_E_UNSUPPORTED;
    return MHD_OK;
}

mhd_status cdev(hipError_t e) { return e == hipSuccess ? MHD_OK : MHD_E_DEVICE; }

hipError_t pack_all(mhd_cnn* c)
{
    for (int l = 0; l < kLayers; ++l) {
        const unsigned int cnt = 27u * kNPad * kCinPad[l];
        hipLaunchKernelGGL(k_pack_weights, dim3((cnt + kThreads - 1) / kThreads), dim3(kThreads), 0, c->stream,
                           c->P + param_offset(l), kCin[l], kCout[l], kCinPad[l], c->Wf[l], l > 0 ? c->Wb[l] : nullptr);
    }
    return hipGetLastError();
}

// One convolution launch on blocks of WY GY rows x WZ GZ planes.
template <int CINP, int MODE, int WY, int WZ, int GY, int GZ>
void conv_blocks(const mhd_cnn* c, const bf16_t* X, const bf16_t* B, const float* bias, const bf16_t* M, bf16_t* Y,
                 float* O, int nstore)
{
    const unsigned int nty = (unsigned int)((c->g.ny + WY * GY - 1) / (WY * GY));
    const unsigned int nblk = (unsigned int)(c->g.nx / 16) * nty * (unsigned int)((c->g.nz + WZ * GZ - 1) / (WZ * GZ));
    const unsigned int grid = nblk < (unsigned int)kConvGroups ? nblk : (unsigned int)kConvGroups;
    hipLaunchKernelGGL((k_conv<CINP, MODE, WY, WZ, GY, GZ>), dim3(grid), dim3(kConvThreads), 0, c->stream, c->g, X, B,
                       bias, M, Y, O, nstore, nty, nblk);
}

// One convolution.  All block shapes give the same bits; a flat one, whose halo has 102 rows
// against 60, takes about 1.6 times as long, so it is chosen where it needs at most 5/8 of
// the rounds of workgroups.  The network's forward pass with 4 x 8 blocks only, with the
// flat ones, and with a wave per 64 voxels and no blocks (us): 512 x 512 x 1 362, 96, 174;
// 512 x 1 x 512 198, 94, 173; 512 x 512 x 3 354, 267, 463; 512 x 5 x 512 431, 350, 741;
// 64 x 64 x 2, a single round, 40, 49, 69.
template <int CINP, int MODE>
void conv(const mhd_cnn* c, const bf16_t* X, const bf16_t* B, const float* bias, const bf16_t* M, bf16_t* Y,
          float* O, int nstore)
{
    const long long ntx = c->g.nx / 16, ny = c->g.ny, nz = c->g.nz;
    auto rounds = [&](int ty, int tz) {
        return (ntx * ((ny + ty - 1) / ty) * ((nz + tz - 1) / tz) + kConvGroups - 1) / kConvGroups;
    };
    const long long tall = rounds(4, 8), row = rounds(32, 1), plane = rounds(1, 32);
    if (8 * row <= 5 * tall && row <= plane)
        conv_blocks<CINP, MODE, 8, 1, 4, 1>(c, X, B, bias, M, Y, O, nstore);
    else if (8 * plane <= 5 * tall)
        conv_blocks<CINP, MODE, 1, 8, 1, 4>(c, X, B, bias, M, Y, O, nstore);
    else
        conv_blocks<CINP, MODE, 4, 2, 1, 4>(c, X, B, bias, M, Y, O, nstore);
}

// forward pass from a canonical state; keeps every layer input for the backward pass
hipError_t forward(mhd_cnn* c, const double* U)
{
    hipLaunchKernelGGL(k_cnn_input, dim3(c->nblk), dim3(kThreads), 0, c->stream, c->g, c->gamma, U, c->scal,
                       c->scal + 8, c->A[0]);
    conv<16, 0>(c, c->A[0], c->Wf[0], c->P + param_offset(0) + layer_w(0), nullptr, c->A[1], nullptr, 0);
    conv<32, 0>(c, c->A[1], c->Wf[1], c->P + param_offset(1) + layer_w(1), nullptr, c->A[2], nullptr, 0);
    conv<32, 0>(c, c->A[2], c->Wf[2], c->P + param_offset(2) + layer_w(2), nullptr, c->A[3], nullptr, 0);
    conv<32, 1>(c, c->A[3], c->Wf[3], c->P + param_offset(3) + layer_w(3), nullptr, nullptr, c->O, 18);
    return hipGetLastError();
}

hipError_t apply(mhd_cnn* c, double dt, double* U, const double* ok = nullptr)
{
    hipLaunchKernelGGL(k_closure_apply, dim3(c->nblk), dim3(kThreads), 0, c->stream, c->g, c->O, c->scal + 16, c->sE,
                       dt, U, ok);
    return hipGetLastError();
}

// flag[0] = +inf if the closure leaves every cell of U valid, else -1 (partials in
// c->partial, the flag just after them).
hipError_t check(mhd_cnn* c, double dt, const double* U, const MhdParams& mp, double* flag)
{
    hipLaunchKernelGGL(k_closure_check, dim3(c->nblk), dim3(kThreads), 0, c->stream, c->g, c->O, c->scal + 16, c->sE,
                       dt, U, c->gamma, mp.rho_floor, mp.p_floor, c->partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_min_final(c->partial, c->nblk, 1.0, flag, c->stream);
}

}  // namespace

extern "C" {

mhd_status mhd_cnn_param_count(size_t* n)
{
    if (!n) return MHD_E_INVAL;
    *n = total_params();
    return MHD_OK;
}

mhd_status mhd_cnn_workspace_bytes(const mhd_grid* grid, const mhd_physics* phys, size_t* bytes)
{
    if (!bytes) return MHD_E_INVAL;
    const mhd_status st = cvalidate(grid, phys);
    if (st != MHD_OK) return st;
    *bytes = clayout(grid).total;
    return MHD_OK;
}

mhd_status mhd_cnn_create(const mhd_grid* grid, const mhd_physics* phys, void* workspace, size_t bytes,
                          void* hip_stream, mhd_cnn** out)
{
    if (!out) return MHD_E_INVAL;
    *out = nullptr;
    mhd_status st = cvalidate(grid, phys);
    if (st != MHD_OK) return st;
    if (!workspace || ((uintptr_t)workspace & 255u)) return MHD_E_INVAL;
    const CLayout L = clayout(grid);
    if (bytes < L.total) return MHD_E_NOMEM;
    mhd_cnn* c = new (std::nothrow) mhd_cnn();
    if (!c) return MHD_E_NOMEM;
    c->g.nx = grid->nx; c->g.ny = grid->ny; c->g.nz = grid->nz;
    c->g.n = (long long)grid->nx * grid->ny * grid->nz;
    const int ns[3] = {grid->nx, grid->ny, grid->nz};
    for (int a = 0; a < 3; ++a) {
        c->g.dx[a] = grid->length[a] / ns[a];
        c->g.inv_dx[a] = 1.0 / c->g.dx[a];
    }
    c->gamma = phys->gamma;
    c->stream = (hipStream_t)hip_stream;
    c->np = total_params();
    c->nblk = (unsigned int)((c->g.n + kThreads - 1) / kThreads);
    char* p = (char*)workspace;
    c->P = (float*)p; p += L.params;
    c->G = (float*)p; p += L.params;
    c->M1 = (float*)p; p += L.params;
    c->M2 = (float*)p; p += L.params;
    for (int l = 0; l < kLayers; ++l) {
        c->Wf[l] = (bf16_t*)p; p += L.wf[l];
        c->Wb[l] = L.wb[l] ? (bf16_t*)p : nullptr; p += L.wb[l];
        c->A[l] = (bf16_t*)p; p += L.a[l];
    }
    c->O = (float*)p; p += L.o;
    c->D0 = (bf16_t*)p; p += L.d;
    c->D1 = (bf16_t*)p; p += L.d;
    c->RW = (float*)p; p += L.rw;
    c->partial = (double*)p; p += L.partial;
    c->gpart = (float*)p; p += L.gpart;
    c->scal = (float*)p;
    c->sE = 1.0f;
    // zero parameters, moments and gradients; unit normalisation
    std::vector<float> zero(c->np, 0.f);
    float sc[64];
    for (int q = 0; q < 64; ++q) sc[q] = q < 8 ? 0.f : 1.f;
    hipError_t e = hipMemcpyAsync(c->P, zero.data(), c->np * sizeof(float), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(c->G, zero.data(), c->np * sizeof(float), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(c->M1, zero.data(), c->np * sizeof(float), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(c->M2, zero.data(), c->np * sizeof(float), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(c->scal, sc, sizeof(sc), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = pack_all(c);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        delete c;
        return MHD_E_DEVICE;
    }
    *out = c;
    return MHD_OK;
}

mhd_status mhd_cnn_set_params(mhd_cnn* c, const float* params)
{
    if (!c || !params) return MHD_E_INVAL;
    hipError_t e = hipMemcpyAsync(c->P, params, c->np * sizeof(float), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = pack_all(c);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    return cdev(e);
}

mhd_status mhd_cnn_get_params(mhd_cnn* c, float* params)
{
    if (!c || !params) return MHD_E_INVAL;
    hipError_t e = hipMemcpyAsync(params, c->P, c->np * sizeof(float), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    return cdev(e);
}

mhd_status mhd_cnn_get_grads(mhd_cnn* c, float* grads)
{
    if (!c || !grads) return MHD_E_INVAL;
    hipError_t e = hipMemcpyAsync(grads, c->G, c->np * sizeof(float), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    return cdev(e);
}

mhd_status mhd_cnn_set_scales(mhd_cnn* c, const float* mu, const float* sd, const float* sF, float sE,
                              const float* wU, float wB)
{
    if (!c || !mu || !sd || !sF || !wU) return MHD_E_INVAL;
    float sc[64] = {0};
    for (int q = 0; q < 8; ++q) {
        if (!(sd[q] > 0.f)) return MHD_E_INVAL;
        sc[q] = mu[q];
        sc[8 + q] = sd[q];
    }
    for (int q = 0; q < 5; ++q) sc[16 + q] = sF[q];
    for (int q = 0; q < 5; ++q) sc[24 + q] = wU[q];
    for (int q = 5; q < 8; ++q) sc[24 + q] = wB;
    c->sE = sE;
    hipError_t e = hipMemcpyAsync(c->scal, sc, sizeof(sc), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    return cdev(e);
}

mhd_status mhd_cnn_forward(mhd_cnn* c, const double* state)
{
    if (!c || !state) return MHD_E_INVAL;
    return cdev(forward(c, state));
}

mhd_status mhd_cnn_output(mhd_cnn* c, float* dst, int dst_is_device)
{
    if (!c || !dst) return MHD_E_INVAL;
    hipError_t e = hipMemcpyAsync(dst, c->O, (size_t)c->g.n * 18 * sizeof(float),
                                  dst_is_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess && !dst_is_device) e = hipStreamSynchronize(c->stream);
    return cdev(e);
}

mhd_status mhd_closure_apply(mhd_cnn* c, double dt, double* state)
{
    if (!c || !state || !(dt > 0.0) || !std::isfinite(dt)) return MHD_E_INVAL;
    return cdev(apply(c, dt, state));
}

mhd_status mhd_cnn_zero_grad(mhd_cnn* c)
{
    if (!c) return MHD_E_INVAL;
    return cdev(hipMemsetAsync(c->G, 0, c->np * sizeof(float), c->stream));
}

mhd_status mhd_cnn_accumulate(mhd_cnn* c, const double* state_t, const double* coarse_next, const double* target,
                              double dt, double* loss)
{
    if (!c || !state_t || !coarse_next || !target || !(dt > 0.0) || !std::isfinite(dt)) return MHD_E_INVAL;
    hipError_t e = forward(c, state_t);
    if (e == hipSuccess && !in_place(coarse_next, c->stream)) {
        // by way of the second gradient buffer, whose 32 BF16 channels a voxel are 8 doubles
        // (the backward pass writes it first after the residual is formed)
        static_assert(kNPad * sizeof(bf16_t) == 8 * sizeof(double), "a canonical state");
        e = hipMemcpyAsync(c->D1, coarse_next, (size_t)c->g.n * 8 * sizeof(double), hipMemcpyDeviceToDevice, c->stream);
        coarse_next = (const double*)c->D1;
    }
    if (e != hipSuccess) return MHD_E_DEVICE;
    hipLaunchKernelGGL(k_residual, dim3(c->nblk), dim3(kThreads), 0, c->stream, c->g, c->O, c->scal + 16, c->sE, dt,
                       coarse_next, target, c->scal + 24, c->RW, c->partial);
    hipLaunchKernelGGL(k_out_grad, dim3(c->nblk), dim3(kThreads), 0, c->stream, c->g, c->RW, c->scal + 16, c->sE, dt,
                       c->D0);
    // backward: layer l consumes D (its output gradient) and A[l] (its input)
    const dim3 bl(kThreads);
    const unsigned int gblk = grad_blocks(c->g.nx, c->g.ny, c->g.nz), ng = grad_groups(gblk);
    const unsigned int gty = (unsigned int)((c->g.ny + 3) / 4);
    bf16_t* D = c->D0;
    bf16_t* Dn = c->D1;
    for (int l = kLayers - 1; l >= 0 && e == hipSuccess; --l) {
        if (l == 0)
            hipLaunchKernelGGL((k_grad<16>), dim3(ng), dim3(kGradThreads), 0, c->stream, c->g, c->A[0], D, c->gpart,
                               kCin[l], kCout[l], gty, gblk);
        else
            hipLaunchKernelGGL((k_grad<32>), dim3(ng), dim3(kGradThreads), 0, c->stream, c->g, c->A[l], D, c->gpart,
                               kCin[l], kCout[l], gty, gblk);
        const unsigned int ne = (unsigned int)layer_params(l);
        hipLaunchKernelGGL(k_grad_sum, dim3((ne + 63) / 64), bl, 0, c->stream, c->gpart, ne, (int)ng,
                           c->G + param_offset(l));
        if (l > 0) {
            // gradient of layer l's input, through the ReLU of layer l-1 (mask = A[l] > 0)
            conv<32, 2>(c, D, c->Wb[l], nullptr, c->A[l], Dn, nullptr, 0);
            bf16_t* t = D;
            D = Dn;
            Dn = t;
        }
        e = hipGetLastError();
    }
    if (e != hipSuccess) return MHD_E_DEVICE;
    if (loss) {
        std::vector<double> part(c->nblk);
        e = hipMemcpyAsync(part.data(), c->partial, c->nblk * sizeof(double), hipMemcpyDeviceToHost, c->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return MHD_E_DEVICE;
        double s = 0.0;
        for (double v : part) s += v;
        *loss = s;
    }
    return MHD_OK;
}

mhd_status mhd_cnn_adam(mhd_cnn* c, float lr, float beta1, float beta2, float eps, int step, float grad_scale)
{
    if (!c || step < 1 || !(lr > 0.f)) return MHD_E_INVAL;
    const float c1 = 1.f / (1.f - std::pow(beta1, (float)step));
    const float c2 = 1.f / (1.f - std::pow(beta2, (float)step));
    hipLaunchKernelGGL(k_adam, dim3((unsigned int)((c->np + kThreads - 1) / kThreads)), dim3(kThreads), 0, c->stream,
                       (unsigned int)c->np, c->P, c->G, c->M1, c->M2, lr, beta1, beta2, eps, c1, c2, grad_scale);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = pack_all(c);
    return cdev(e);
}

mhd_status mhd_step_closure(mhd_ctx* ctx, mhd_cnn* c, double dt, int* applied)
{
    if (!ctx || !c || !(dt > 0.0) || !std::isfinite(dt)) return MHD_E_INVAL;
    CtxView v = ctx_view(ctx);
    if (!v.state) return MHD_E_UNSUPPORTED;  // FP64 adiabatic MHD contexts
    // the same grid (cells and spacing) and the same stream: the network's kernels and
    // the context's run in one order without events between them
    if (v.geo.nx != c->g.nx || v.geo.ny != c->g.ny || v.geo.nz != c->g.nz) return MHD_E_INVAL;
    for (int a = 0; a < 3; ++a)
        if (v.geo.dx[a] != c->g.dx[a]) return MHD_E_INVAL;
    if (v.stream != c->stream) return MHD_E_INVAL;
    double* flag = c->partial + c->nblk;
    // corrections from the state at the start of the step, read where it lives
    mhd_status st = cdev(forward(c, v.state));
    // the plain step, then the closure in place on the stepped state if it leaves every
    // cell finite and above the floors (else the plain step stands), and the time step
    // of the result
    if (st == MHD_OK) st = mhd_step(ctx, dt);
    if (st != MHD_OK) return st;
    v = ctx_view(ctx);
    hipError_t e = check(c, dt, v.state, v.mp, flag);
    if (e == hipSuccess) e = apply(c, dt, v.state, flag);
    if (e == hipSuccess) e = ctx_refresh_cfl(ctx);
    if (e == hipSuccess && applied) {
        double h = 0.0;
        e = hipMemcpyAsync(&h, flag, sizeof(double), hipMemcpyDeviceToHost, c->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
        *applied = h > 0.0 ? 1 : 0;
    }
    return cdev(e);
}

mhd_status mhd_box_filter(const mhd_grid* fine, int r, const double* fine_state, double* coarse_state, void* hip_stream)
{
    if (!fine || !fine_state || !coarse_state || r < 1) return MHD_E_INVAL;
    if (fine->nx % r || fine->ny % r || fine->nz % r) return MHD_E_INVAL;
    Geo f, c;
    f.nx = fine->nx; f.ny = fine->ny; f.nz = fine->nz;
    f.n = (long long)f.nx * f.ny * f.nz;
    c.nx = f.nx / r; c.ny = f.ny / r; c.nz = f.nz / r;
    c.n = (long long)c.nx * c.ny * c.nz;
    if (f.n >= (1LL << 29)) return MHD_E_UNSUPPORTED;
    hipLaunchKernelGGL(k_box_filter, dim3((unsigned int)((c.n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                       (hipStream_t)hip_stream, f, c, r, fine_state, coarse_state);
    return cdev(hipGetLastError());
}

void mhd_cnn_destroy(mhd_cnn* c) { delete c; }

}  // extern "C"
