// reduce.hip -- the time step of eq. (cfl) and the conservation diagnostics.
//
// Both are two-pass reductions with a fixed assignment of cells to lanes and of
// partials to the final pass, so the result is bitwise reproducible run to run.
// Within a wavefront the 64 lanes combine by butterfly shuffles.
#include <algorithm>

#include "launch.hpp"
#include "physics.hpp"

namespace mhd {

__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min_nan(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Block-wide minimum; the result is valid in thread 0.
__device__ __forceinline__ double block_min(double v)
{
    __shared__ double sm[kBlock / 64];
    v = wave_min(v);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = sm[0];
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) r = min_nan(r, sm[w]);
    }
    return r;
}

// Time step of eq. (cfl) of cell c of a grid of n cells; cx, cy, cz: the cells whose
// low faces are c's high faces.  The same arithmetic, rounded as written, as the time
// step the last stage of a step reduces (mhd_tiles.hpp), so a state gives the same bits
// whichever kernel takes its step.
__device__ __forceinline__ double cfl_cell(const Geo& g, const MhdParams& p, const double* __restrict__ U,
                                           long long n, long long c, long long cx, long long cy, long long cz)
{
#pragma clang fp contract(off)
    const double bx = 0.5 * (U[5 * n + c] + U[5 * n + cx]);
    const double by = 0.5 * (U[6 * n + c] + U[6 * n + cy]);
    const double bz = 0.5 * (U[7 * n + c] + U[7 * n + cz]);
    double d = U[c];
    if (d < p.rho_floor) d = p.rho_floor;
    const double id = rcp(d);
    const double v[3] = {U[n + c] * id, U[2 * n + c] * id, U[3 * n + c] * id};
    const double ke = 0.5 * d * ((v[0] * v[0] + v[1] * v[1]) + v[2] * v[2]);
    const double b2 = (bx * bx + by * by) + bz * bz;
    double pr = (p.gamma - 1.0) * ((U[4 * n + c] - ke) - 0.5 * b2);
    if (pr < p.p_floor) pr = p.p_floor;
    const double bd[3] = {bx, by, bz};
    double r = INFINITY;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double cf = fast_speed(p.gamma, d, pr, b2, bd[a]);
        r = min_nan(r, div_r(g.dx[a], fabs(v[a]) + cf));
    }
    return r;
}

__global__ __launch_bounds__(kBlock) void k_cfl_mhd(Geo g, MhdParams p, const double* __restrict__ U,
                                                    double* __restrict__ partial)
{
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    double r = INFINITY;
    if (c < g.n) {
        int i, j, k;
        cell_ijk(g, c, i, j, k);
        r = cfl_cell(g, p, U, g.n, c, shifted(g, i, j, k, 0, 1), shifted(g, i, j, k, 1, 1), shifted(g, i, j, k, 2, 1));
    }
    r = block_min(r);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

// The time step over the interior cells of nb equal padded blocks (grid pg each, g
// ghost layers, interior bx x by x bz; block b's register at reg + 8 off[b] doubles):
// ghost cells are left out (the outermost layer's high neighbours are not in the block).
__global__ __launch_bounds__(kBlock) void k_cfl_blocks(Geo pg, MhdParams p, const double* __restrict__ reg,
                                                       const unsigned long long* __restrict__ off, int nb, int gh,
                                                       int bx, int by, int bz, double* __restrict__ partial)
{
    const long long per = (long long)bx * by * bz;
    double r = INFINITY;
    // a fixed grid strides over the cells, so the final pass has few partials
    for (long long t = (long long)blockIdx.x * kBlock + threadIdx.x; t < per * nb;
         t += (long long)gridDim.x * kBlock) {
        const int b = (int)(t / per);
        const long long q = t - (long long)b * per;
        const int i = (int)(q % bx) + gh, j = (int)((q / bx) % by) + gh, k = (int)(q / ((long long)bx * by)) + gh;
        const long long c = ((long long)k * pg.ny + j) * pg.nx + i;
        r = min_nan(r, cfl_cell(pg, p, reg + off[b] * 8ULL, pg.n, c, c + 1, c + pg.nx, c + (long long)pg.nx * pg.ny));
    }
    r = block_min(r);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

// All blocks of a batch in one launch, `per` workgroups striding over the cells of each:
// bound by its bytes, where a copy, a reduction, its final pass and a conversion per block
// were bound by their launches (512 blocks, 26.8 M cells, FP32-bulk: 0.62 ms in
// and 0.56 ms back; the pair took 9.6 ms).
template <class R>
__device__ __forceinline__ double load_block(const BlockDesc& d, const MhdParams& p, const double* __restrict__ src,
                                             char* __restrict__ reg, int w, int per)
{
    const long long n = d.g.n;
    const double* U = src + 8ULL * d.at;
    const RegView<R> v = reg_view<R>(reg + d.off * (unsigned long long)register_bytes(1, sizeof(R) == 4), n);
    double r = INFINITY;
    for (long long c = (long long)w * kBlock + threadIdx.x; c < n; c += (long long)per * kBlock) {
        int i, j, k;
        cell_ijk(d.g, c, i, j, k);
        r = min_nan(r, cfl_cell(d.g, p, U, n, c, shifted(d.g, i, j, k, 0, 1), shifted(d.g, i, j, k, 1, 1),
                                shifted(d.g, i, j, k, 2, 1)));
        v.rho[c] = (R)U[c];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v.m[a][c] = (R)U[(1 + a) * n + c];
            v.b[a][c] = (R)U[(5 + a) * n + c];
        }
        v.E[c] = U[4 * n + c];
    }
    return block_min(r);
}

template <class R>
__global__ __launch_bounds__(kBlock) void k_batch_load(const BlockDesc* __restrict__ blk, int per, MhdParams p,
                                                       const double* __restrict__ src, char* __restrict__ reg,
                                                       double* __restrict__ partial)
{
    const double r = load_block<R>(blk[blockIdx.x / per], p, src, reg, (int)(blockIdx.x % per), per);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

// The state of one grid in one pass over it, where a copy or a conversion and the
// reduction each read it (256^3 FP64 426 + 228 -> 424 us, FP32-bulk 227 + 269 -> 339 us).
template <class R>
__global__ __launch_bounds__(kBlock) void k_state_load(Geo g, MhdParams p, const double* __restrict__ src,
                                                       char* __restrict__ reg, double* __restrict__ partial)
{
    const double r = load_block<R>(BlockDesc{g, 0, 0}, p, src, reg, (int)blockIdx.x, (int)gridDim.x);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

template <class R>
__global__ __launch_bounds__(kBlock) void k_batch_store(const BlockDesc* __restrict__ blk, int per,
                                                        const char* __restrict__ reg, double* __restrict__ dst)
{
    const BlockDesc d = blk[blockIdx.x / per];
    const long long n = d.g.n;
    double* U = dst + 8ULL * d.at;
    const RegView<R> v =
        reg_view<R>(const_cast<char*>(reg) + d.off * (unsigned long long)register_bytes(1, sizeof(R) == 4), n);
    for (long long c = (long long)(blockIdx.x % per) * kBlock + threadIdx.x; c < n; c += (long long)per * kBlock) {
        U[c] = v.rho[c];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            U[(1 + a) * n + c] = v.m[a][c];
            U[(5 + a) * n + c] = v.b[a][c];
        }
        U[4 * n + c] = v.E[c];
    }
}

// LOAD: the state also goes into the register reg on the way, FP32 forms rounded (192^3, 8
// species: FP64 795 + 362 -> 784 us, FP32 355 + 581 -> 600 us against a copy or a
// conversion of its own).
template <bool LOAD, class R>
__global__ __launch_bounds__(kBlock) void k_cfl_dust(Geo g, DustParams p, const double* __restrict__ U,
                                                     R* __restrict__ reg, double* __restrict__ partial)
{
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    double r = INFINITY;
    if (c < g.n) {
        const long long n = g.n;
        for (int s = 0; s <= p.nd; ++s) {
            const double* u = U + 4LL * s * n;
            double d = u[c];
            const double m[3] = {u[n + c], u[2 * n + c], u[3 * n + c]};
            if constexpr (LOAD) {
                R* w = reg + 4LL * s * n;
                w[c] = (R)d;
#pragma unroll
                for (int a = 0; a < 3; ++a) w[(1 + a) * n + c] = (R)m[a];
            }
            double v[3];
            if (s == 0) {
                if (d < p.rho_floor) d = p.rho_floor;
                v[0] = m[0] / d; v[1] = m[1] / d; v[2] = m[2] / d;
            } else if (d < p.dust_floor) {
                v[0] = v[1] = v[2] = 0.0;
            } else {
                v[0] = m[0] / d; v[1] = m[1] / d; v[2] = m[2] / d;
            }
            const double cs = s == 0 ? p.cs : 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a) r = min_nan(r, g.dx[a] / (fabs(v[a]) + cs));
        }
    }
    r = block_min(r);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

// out[b] = scale * min of the m partials of block b, a workgroup of T lanes each, eight
// independent loads in flight per lane: bound by the latency of its rounds of loads (27648
// partials, the dust step at 192^3: T = 1024, 46 -> 9 us with four waves and one load at a
// time before).
template <int T>
__global__ __launch_bounds__(T) void k_min_final(const double* __restrict__ partial, long long m, double scale,
                                                 double* __restrict__ out)
{
    __shared__ double sm[T / 64];
    partial += blockIdx.x * m;
    double r = INFINITY;
    for (long long q0 = 0; q0 < m; q0 += 8 * T) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const long long q = q0 + u * T + (int)threadIdx.x;
            v[u] = q < m ? partial[q] : INFINITY;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) r = min_nan(r, v[u]);
    }
    r = wave_min(r);
    if constexpr (T > 64) {
        if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = r;
        __syncthreads();
        if (threadIdx.x >= 64) return;
        r = wave_min(threadIdx.x < T / 64 ? sm[threadIdx.x] : INFINITY);
    }
    if (threadIdx.x == 0) out[blockIdx.x] = scale * r;
}

// nb blocks of m partials: as many lanes as one round of loads fills, within 64 and 1024 (up
// to 512 partials 1.6 us with 64 lanes, 2.6 with 1024; four waves and one load at a time 1.7).
static void min_final(const double* partial, long long m, int nb, double scale, double* out, hipStream_t s)
{
    if (m <= 8 * 64)
        hipLaunchKernelGGL(k_min_final<64>, dim3(nb), dim3(64), 0, s, partial, m, scale, out);
    else if (m <= 8 * 256)
        hipLaunchKernelGGL(k_min_final<256>, dim3(nb), dim3(256), 0, s, partial, m, scale, out);
    else
        hipLaunchKernelGGL(k_min_final<1024>, dim3(nb), dim3(1024), 0, s, partial, m, scale, out);
}

hipError_t launch_min_final(const double* partial, long long m, double scale, double* out,
                            hipStream_t s)
{
    min_final(partial, m, 1, scale, out, s);
    return hipGetLastError();
}

hipError_t launch_cfl_mhd(const Geo& g, const MhdParams& p, const double* U, double* partial,
                          double* dt_out, double scale, hipStream_t s)
{
    const unsigned int nb = blocks_for(g.n);
    hipLaunchKernelGGL(k_cfl_mhd, dim3(nb), dim3(kBlock), 0, s, g, p, U, partial);
    min_final(partial, (long long)nb, 1, scale, dt_out, s);
    return hipGetLastError();
}

hipError_t launch_state_load(const Geo& g, const MhdParams& p, bool fp32, const double* src, void* reg,
                             double* partial, double* dt, double scale, hipStream_t s)
{
    const unsigned int nb = std::min(blocks_for(g.n), 16384u);
    if (fp32)
        hipLaunchKernelGGL(k_state_load<float>, dim3(nb), dim3(kBlock), 0, s, g, p, src, (char*)reg, partial);
    else
        hipLaunchKernelGGL(k_state_load<double>, dim3(nb), dim3(kBlock), 0, s, g, p, src, (char*)reg, partial);
    min_final(partial, (long long)nb, 1, scale, dt, s);
    return hipGetLastError();
}

hipError_t launch_batch_load(const BlockDesc* blk, int nb, int per, const MhdParams& p, bool fp32, const double* src,
                             void* reg, double* partial, double* dt, double scale, hipStream_t s)
{
    const dim3 gr((unsigned int)nb * (unsigned int)per), bl(kBlock);
    if (fp32)
        hipLaunchKernelGGL(k_batch_load<float>, gr, bl, 0, s, blk, per, p, src, (char*)reg, partial);
    else
        hipLaunchKernelGGL(k_batch_load<double>, gr, bl, 0, s, blk, per, p, src, (char*)reg, partial);
    min_final(partial, per, nb, scale, dt, s);
    return hipGetLastError();
}

hipError_t launch_batch_store(const BlockDesc* blk, int nb, int per, bool fp32, const void* reg, double* dst,
                              hipStream_t s)
{
    const dim3 gr((unsigned int)nb * (unsigned int)per), bl(kBlock);
    if (fp32)
        hipLaunchKernelGGL(k_batch_store<float>, gr, bl, 0, s, blk, per, (const char*)reg, dst);
    else
        hipLaunchKernelGGL(k_batch_store<double>, gr, bl, 0, s, blk, per, (const char*)reg, dst);
    return hipGetLastError();
}

hipError_t launch_cfl_blocks(const Geo& pg, const MhdParams& p, const double* reg, const unsigned long long* off,
                             int nb, int ghost, int bx, int by, int bz, double* partial, double* dt_out,
                             double scale, hipStream_t s)
{
    const long long m = std::min<long long>(((long long)bx * by * bz * nb + kBlock - 1) / kBlock, 4096);
    hipLaunchKernelGGL(k_cfl_blocks, dim3((unsigned int)m), dim3(kBlock), 0, s, pg, p, reg, off, nb, ghost, bx, by, bz,
                       partial);
    min_final(partial, m, 1, scale, dt_out, s);
    return hipGetLastError();
}

hipError_t launch_cfl_dust(const Geo& g, const DustParams& p, const double* U, double* partial,
                           double* dt_out, double scale, hipStream_t s)
{
    const unsigned int nb = blocks_for(g.n);
    hipLaunchKernelGGL((k_cfl_dust<false, double>), dim3(nb), dim3(kBlock), 0, s, g, p, U, (double*)nullptr, partial);
    min_final(partial, (long long)nb, 1, scale, dt_out, s);
    return hipGetLastError();
}

hipError_t launch_dust_load(const Geo& g, const DustParams& p, bool fp32, const double* src, void* reg,
                            double* partial, double* dt, double scale, hipStream_t s)
{
    const unsigned int nb = blocks_for(g.n);
    if (fp32)
        hipLaunchKernelGGL((k_cfl_dust<true, float>), dim3(nb), dim3(kBlock), 0, s, g, p, src, (float*)reg, partial);
    else
        hipLaunchKernelGGL((k_cfl_dust<true, double>), dim3(nb), dim3(kBlock), 0, s, g, p, src, (double*)reg, partial);
    min_final(partial, (long long)nb, 1, scale, dt, s);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------
// diagnostics: out[0] gas mass, [1..3] gas momentum, [4] E, [5..7] face-field
// integrals, [8] max |div B|, [9..8+nd] dust masses, [9+nd..11+nd] total momentum
// ----------------------------------------------------------------------------------

int diag_count(int ndust) { return 12 + ndust; }

__global__ __launch_bounds__(kBlock) void k_diag_partial(Geo g, int mhd, int nd,
                                                         const double* __restrict__ U,
                                                         double* __restrict__ partial)
{
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    const int nq = 12 + nd;
    const long long n = g.n;
    __shared__ double sm[kBlock / 64][12 + kMaxDust];
    const bool live = c < n;
    double vals[12 + kMaxDust];
    for (int q = 0; q < nq; ++q) vals[q] = 0.0;
    if (live) {
        if (mhd) {
            for (int q = 0; q < 8; ++q) {
                const double x = U[q * n + c];
                if (q < 5) vals[q] = x; else vals[q] = x;
            }
            int i, j, k;
            cell_ijk(g, c, i, j, k);
            const double dv = (U[5 * n + shifted(g, i, j, k, 0, 1)] - U[5 * n + c]) * g.inv_dx[0] +
                              (U[6 * n + shifted(g, i, j, k, 1, 1)] - U[6 * n + c]) * g.inv_dx[1] +
                              (U[7 * n + shifted(g, i, j, k, 2, 1)] - U[7 * n + c]) * g.inv_dx[2];
            vals[8] = fabs(dv);
            for (int a = 0; a < 3; ++a) vals[9 + a] = U[(1 + a) * n + c];
        } else {
            for (int q = 0; q < 4; ++q) vals[q] = U[q * n + c];
            for (int a = 0; a < 3; ++a) vals[9 + nd + a] = U[(1 + a) * n + c];
            for (int s = 1; s <= nd; ++s) {
                vals[9 + s - 1] = U[4LL * s * n + c];
                for (int a = 0; a < 3; ++a) vals[9 + nd + a] += U[(4LL * s + 1 + a) * n + c];
            }
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int q = 0; q < nq; ++q) {
        const double r = (q == 8) ? wave_max(vals[q]) : wave_sum(vals[q]);
        if (lane == 0) sm[w][q] = r;
    }
    __syncthreads();
    if (threadIdx.x < nq) {
        const int q = threadIdx.x;
        double r = sm[0][q];
        for (int ww = 1; ww < kBlock / 64; ++ww) r = (q == 8) ? fmax(r, sm[ww][q]) : r + sm[ww][q];
        partial[(long long)blockIdx.x * nq + q] = r;
    }
}

// One workgroup per quantity; lanes stride over the partials in a fixed order.
__global__ __launch_bounds__(kBlock) void k_diag_final(const double* __restrict__ partial, long long m,
                                                       int nq, double dV, double* __restrict__ out)
{
    const int q = blockIdx.x;
    const bool mx = (q == 8);
    double r = 0.0;
    for (long long b = threadIdx.x; b < m; b += kBlock) {
        const double x = partial[b * nq + q];
        r = mx ? fmax(r, x) : r + x;
    }
    __shared__ double sm[kBlock / 64];
    r = mx ? wave_max(r) : wave_sum(r);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = sm[0];
        for (int w = 1; w < kBlock / 64; ++w) t = mx ? fmax(t, sm[w]) : t + sm[w];
        out[q] = mx ? t : t * dV;
    }
}

hipError_t launch_diag(const Geo& g, int mhd, int ndust, const double* U, double* partial,
                       double* out, hipStream_t s)
{
    const unsigned int nb = blocks_for(g.n);
    const int nq = diag_count(ndust);
    hipLaunchKernelGGL(k_diag_partial, dim3(nb), dim3(kBlock), 0, s, g, mhd, ndust, U, partial);
    const double dV = g.dx[0] * g.dx[1] * g.dx[2];
    hipLaunchKernelGGL(k_diag_final, dim3(nq), dim3(kBlock), 0, s, partial, (long long)nb, nq, dV, out);
    return hipGetLastError();
}

}  // namespace mhd
