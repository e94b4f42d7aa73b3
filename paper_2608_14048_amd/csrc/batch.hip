// batch.hip -- many self-periodic meshblocks of uneven sizes advanced together.
//
// The paper advances the meshblocks a rank owns in one launch, with the block index as
// one more launch dimension (Sec. "Mesh, Coordinates, and Boundary Conditions"); here
// the blocks are independent periodic
// boxes of any sizes, and each stage kernel is one persistent launch per tile shape in
// use (one launch for all blocks when they share a shape, three at most): a queue of
// (block, tile, z chunk) work items, longest first, that the workgroups of the launch
// drain through a device counter.  Tile shapes: 64x4 / 32x8 / 16x16 columns for the
// flux kernel, 64x8 / 32x16 / 16x32 for the CT/update kernel; the shape of each
// block-size class is picked by measurement (mhd_batch_tune).  A shape is a template
// argument rather than a runtime switch because the three inlined tile bodies of one
// kernel would not fit the register file together.  The tile bodies are the single-grid
// ones (mhd_tiles.hpp), so a block advanced in a batch is bitwise identical to the same
// block advanced alone.
//
// Work counter: a 64-bit device counter that only grows.  A launch over m items with g
// workgroups takes exactly m + g values (every workgroup stops at its first fetch past
// the end), so the host knows each launch's base without resetting anything.
//
// Each block advances by its own time step (the blocks are separate problems): the
// step reads dt[b] from device memory, either written from the caller's host array or
// left there by the CFL reduction of the previous step.
//
// Coupled blocks (mhd_batch_couple): equal blocks become one periodic domain, each
// block a slab of it padded by ghost layers; after every stage one kernel refills every
// ghost cell from the block that owns it, and every block takes the domain's one step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <numeric>
#include <vector>

#include "../../include/mhd950.h"
#include "mhd_tiles.hpp"

using namespace mhd;
using namespace mhd::tiles;

namespace {

constexpr int kShapes = 3;
constexpr int kFluxThreads = 256, kCtThreads = 512;
constexpr int kFluxTX[kShapes] = {64, 32, 16};
constexpr int kCtTX[kShapes] = {64, 32, 16};
constexpr int kAlignCells = 64;  // block offsets in cells: keeps every field 256-B aligned

struct WorkItem {
    int block, x0, y0, k0, k1, shape;
};

int flux_ty(int s) { return kFluxThreads / kFluxTX[s]; }
int ct_ty(int s) { return kCtThreads / kCtTX[s]; }

}  // namespace

namespace mhd {

// ----------------------------------------------------------------------------------
// persistent stage kernels
// ----------------------------------------------------------------------------------

__device__ __forceinline__ int next_item(unsigned long long* ctr, unsigned long long base, int* slot)
{
    if (threadIdx.x == 0) *slot = (int)(long long)(atomicAdd(ctr, 1ULL) - base);
    __syncthreads();
    const int it = *slot;
    __syncthreads();
    return it;
}

struct BatchCt {
    char* in;
    char* base;
    char* out;
    int reg_bpc;
    double g0, g1, beta;  // out = g0 in + g1 base + beta dt[b] L
    const double* dt;     // per block
    double* partial;      // per item (CFL)
};

// Waves per SIMD a batch flux kernel asks for: the single-grid request, or fewer where
// the tile shape's LDS leaves room for fewer workgroups per CU (one workgroup of four
// waves per CU is one wave per SIMD).
template <int RECON, int RS, class R, int SHAPE>
struct BatchFluxWaves {
    static constexpr int TX = SHAPE == 0 ? 64 : (SHAPE == 1 ? 32 : 16);
    static constexpr int lds_fit =
        (int)(160 * 1024 / (sizeof(typename FluxTile<RECON, RS, true, R, TX, kFluxThreads / TX>::Lds) + 64));
    static constexpr int min = lds_fit < FluxWaves<RECON, RS, R>::min ? lds_fit : FluxWaves<RECON, RS, R>::min;
};

template <int RECON, int RS, bool IN, class R, int SHAPE>
__global__ __launch_bounds__(kFluxThreads) __attribute__((amdgpu_waves_per_eu(BatchFluxWaves<RECON, RS, R, SHAPE>::min)))
void k_flux3_batch(const BlockDesc* __restrict__ blk,
                                                             const WorkItem* __restrict__ items, int nitems,
                                                             unsigned long long* ctr, unsigned long long base,
                                                             MhdParams P, BatchCt a, R* F, R* Rc, unsigned char* S)
{
    constexpr int TX = SHAPE == 0 ? 64 : (SHAPE == 1 ? 32 : 16);
    using Tile = FluxTile<RECON, RS, IN, R, TX, kFluxThreads / TX>;
    __shared__ typename Tile::Lds lds;
    __shared__ int slot;
    for (;;) {
        const int it = next_item(ctr, base, &slot);
        if (it < 0 || it >= nitems) break;
        const WorkItem w = items[it];
        const BlockDesc b = blk[w.block];
        const unsigned long long ob = b.off * (unsigned long long)a.reg_bpc;
        const StageArgs<R> s{reg_view<R>(a.in + ob, b.g.n), reg_view<R>(a.base + ob, b.g.n),
                             reg_view<R>(a.out + ob, b.g.n), F + b.off * (unsigned long long)NFACE,
                             Rc + b.off * 3ULL, S + b.off, StageCoef{a.g0, a.g1, a.beta * a.dt[w.block]}};
        Tile::run(b.g, P, s, w.x0, w.y0, w.k0, w.k1, lds);
        __syncthreads();  // the next item reuses the LDS
    }
}

// items: this launch's items, which start at item id `first` of the whole list (the
// CFL partial of item id q goes to partial[q]).
template <bool CFL, bool IN, class R, int SHAPE>
__global__ __launch_bounds__(kCtThreads) void k_ct_batch(const BlockDesc* __restrict__ blk,
                                                        const WorkItem* __restrict__ items, int nitems, int first,
                                                        unsigned long long* ctr, unsigned long long base,
                                                        MhdParams P, BatchCt a, const R* F, const R* Rc,
                                                        const unsigned char* S)
{
    constexpr int TX = SHAPE == 0 ? 64 : (SHAPE == 1 ? 32 : 16);
    using Tile = CtTile<CFL, IN, R, TX, kCtThreads / TX>;
    __shared__ typename Tile::Lds lds;
    __shared__ int slot;
    __shared__ double sMin[kCtThreads / 64];
    for (;;) {
        const int it = next_item(ctr, base, &slot);
        if (it < 0 || it >= nitems) break;
        const WorkItem w = items[it];
        const BlockDesc b = blk[w.block];
        const unsigned long long ob = b.off * (unsigned long long)a.reg_bpc;
        CtArgs<R> c{reg_view<R>(a.in + ob, b.g.n), reg_view<R>(a.base + ob, b.g.n), F + b.off * (unsigned long long)NFACE,
                    Rc + b.off * 3ULL, S + b.off, reg_view<R>(a.out + ob, b.g.n), nullptr,
                    StageCoef{a.g0, a.g1, a.beta * a.dt[w.block]}};
        double vmin = Tile::run(b.g, P, c, w.x0, w.y0, w.k0, w.k1, lds);
        if (CFL) {
            vmin = wave_min64(vmin);
            if ((threadIdx.x & 63) == 0) sMin[threadIdx.x >> 6] = vmin;
            __syncthreads();
            if (threadIdx.x == 0) {
                double r = sMin[0];
#pragma unroll
                for (int q = 1; q < kCtThreads / 64; ++q) r = min_nan(r, sMin[q]);
                a.partial[first + it] = r;
            }
        }
        __syncthreads();  // the next item reuses the LDS
    }
}

// dt[b] = scale * min of the CFL partials of block b's items (CSR lists).
__global__ __launch_bounds__(256) void k_block_min(const double* __restrict__ partial,
                                                   const int* __restrict__ start,
                                                   const int* __restrict__ list, double scale,
                                                   double* __restrict__ dt)
{
    __shared__ double sm[4];
    const int b = blockIdx.x;
    double r = INFINITY;
    for (int q = start[b] + (int)threadIdx.x; q < start[b + 1]; q += 256) r = min_nan(r, partial[list[q]]);
    r = wave_min64(r);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) dt[b] = scale * min_nan(min_nan(sm[0], sm[1]), min_nan(sm[2], sm[3]));
}

// ----------------------------------------------------------------------------------
// coupled blocks of one periodic domain
// ----------------------------------------------------------------------------------

// Block b = (bi, bj, bk), x fastest, holds the domain cells [bi bs0, (bi + 1) bs0) x ...
// as its interior, padded by g ghost cells on every side (padded extents pn).
struct DomainMap {
    int nb[3], bs[3], pn[3], dn[3];  // blocks, interior cells, padded cells, domain cells
    int g;
    long long pc;                    // cells of a padded block
    long long dcells;                // cells of the domain
};

// i taken periodically into [0, n) (couple() keeps n >= the ghost width, so one wrap
// suffices; the full modulo keeps every index in range regardless).
__device__ __forceinline__ int dwrap(int i, int n)
{
    const int r = i % n;
    return r < 0 ? r + n : r;
}

// Every block's ghost cells from the blocks that own those domain cells (all 8 fields;
// a face field travels with the cell on its high side); one thread per ghost cell: the
// shell of a padded block is enumerated as its two z slabs (whole planes), then the two
// y slabs of the interior planes, then the two x slabs of the interior rows.
__global__ __launch_bounds__(256) void k_ghost_fill(DomainMap m, const unsigned long long* __restrict__ off,
                                                    int nblocks, double* reg)
{
    const int g = m.g, p0 = m.pn[0], p1 = m.pn[1];
    const long long zs = 2LL * g * p1 * p0, ys = 2LL * g * m.bs[2] * p0, xs = 2LL * g * m.bs[2] * m.bs[1];
    const long long per = zs + ys + xs;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= per * nblocks) return;
    const int b = (int)(t / per);
    long long q = t - (long long)b * per;
    int i, j, k;
    if (q < zs) {
        const int pz = (int)(q / ((long long)p1 * p0));
        const long long r = q - (long long)pz * p1 * p0;
        k = pz < g ? pz : m.bs[2] + pz;
        j = (int)(r / p0);
        i = (int)(r - (long long)j * p0);
    } else if ((q -= zs) < ys) {
        const int kk = (int)(q / (2LL * g * p0));
        const long long r = q - (long long)kk * 2 * g * p0;
        const int jj = (int)(r / p0);
        k = g + kk;
        j = jj < g ? jj : m.bs[1] + jj;
        i = (int)(r - (long long)jj * p0);
    } else {
        q -= ys;
        const int kk = (int)(q / (2LL * g * m.bs[1]));
        const int r = (int)(q - (long long)kk * 2 * g * m.bs[1]);
        const int ii = r % (2 * g);
        k = g + kk;
        j = g + r / (2 * g);
        i = ii < g ? ii : m.bs[0] + ii;
    }
    const int bi = b % m.nb[0], bj = (b / m.nb[0]) % m.nb[1], bk = b / (m.nb[0] * m.nb[1]);
    const int I = dwrap(bi * m.bs[0] + i - g, m.dn[0]);
    const int J = dwrap(bj * m.bs[1] + j - g, m.dn[1]);
    const int K = dwrap(bk * m.bs[2] + k - g, m.dn[2]);
    const int oi = I / m.bs[0], oj = J / m.bs[1], ok = K / m.bs[2];
    const int ob = (ok * m.nb[1] + oj) * m.nb[0] + oi;
    const long long c = ((long long)k * p1 + j) * p0 + i;
    const long long oc = ((long long)(K - ok * m.bs[2] + g) * p1 + (J - oj * m.bs[1] + g)) * p0 + (I - oi * m.bs[0] + g);
    double* blk = reg + off[b] * 8ULL;
    const double* src = reg + off[ob] * 8ULL;
#pragma unroll
    for (int f = 0; f < 8; ++f) blk[f * m.pc + c] = src[f * m.pc + oc];
}

// MODE 0: every block's ghost cells from their owners (as k_ghost_fill, one thread per
// padded cell).  MODE 1: every padded cell from the domain state dom ([8][NZ][NY][NX]).
// MODE 2: the interior cells into dom.  reg: the FP64 register, block b's 8 fields of pc
// cells at reg + 8 off[b].
template <int MODE>
__global__ __launch_bounds__(256) void k_domain_copy(DomainMap m, const unsigned long long* __restrict__ off,
                                                     int nblocks, double* reg, double* dom)
{
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= m.pc * nblocks) return;
    const int b = (int)(t / m.pc);
    const long long c = t - (long long)b * m.pc;
    const int i = (int)(c % m.pn[0]), j = (int)((c / m.pn[0]) % m.pn[1]), k = (int)(c / ((long long)m.pn[0] * m.pn[1]));
    const bool interior = i >= m.g && i < m.g + m.bs[0] && j >= m.g && j < m.g + m.bs[1] && k >= m.g &&
                          k < m.g + m.bs[2];
    if (MODE == 0 && interior) return;
    if (MODE == 2 && !interior) return;
    const int bi = b % m.nb[0], bj = (b / m.nb[0]) % m.nb[1], bk = b / (m.nb[0] * m.nb[1]);
    // the domain cell (taken periodically)
    const int I = dwrap(bi * m.bs[0] + i - m.g, m.dn[0]);
    const int J = dwrap(bj * m.bs[1] + j - m.g, m.dn[1]);
    const int K = dwrap(bk * m.bs[2] + k - m.g, m.dn[2]);
    double* blk = reg + off[b] * 8ULL;
    if constexpr (MODE == 0) {
        const int oi = I / m.bs[0], oj = J / m.bs[1], ok = K / m.bs[2];
        const int ob = (ok * m.nb[1] + oj) * m.nb[0] + oi;
        const long long oc = ((long long)(K - ok * m.bs[2] + m.g) * m.pn[1] + (J - oj * m.bs[1] + m.g)) * m.pn[0] +
                             (I - oi * m.bs[0] + m.g);
        const double* src = reg + off[ob] * 8ULL;
#pragma unroll
        for (int f = 0; f < 8; ++f) blk[f * m.pc + c] = src[f * m.pc + oc];
    } else {
        const long long dc = ((long long)K * m.dn[1] + J) * m.dn[0] + I;
        if constexpr (MODE == 1) {
#pragma unroll
            for (int f = 0; f < 8; ++f) blk[f * m.pc + c] = dom[f * m.dcells + dc];
        } else {
#pragma unroll
            for (int f = 0; f < 8; ++f) dom[f * m.dcells + dc] = blk[f * m.pc + c];
        }
    }
}

// dt[1 .. n) = dt[0]: every block of a coupled domain takes the domain's step.
__global__ void k_dt_broadcast(double* dt, int n)
{
    for (int b = 1 + (int)threadIdx.x; b < n; b += (int)blockDim.x) dt[b] = dt[0];
}

}  // namespace mhd

// ----------------------------------------------------------------------------------
// host runtime
// ----------------------------------------------------------------------------------

struct mhd_batch {
    int nb;
    std::vector<Geo> geo;
    std::vector<unsigned long long> off;
    unsigned long long ncell;  // padded total
    mhd_physics phys;
    mhd_scheme scheme;
    MhdParams mp;
    bool fp32;
    int reg_bpc;  // register bytes per cell
    hipStream_t stream;
    int cus;
    // workspace views
    char* reg[3];
    void* F;   // face fluxes; also the canonical FP64 staging area of the FP32-bulk form
    void* Rc;
    double* partial;
    double* dt;            // per block
    unsigned long long* ctr;  // [0] flux queue, [1] CT queue
    BlockDesc* d_blk;
    WorkItem* d_fitems;
    WorkItem* d_citems;
    int* d_cstart;
    int* d_clist;
    int cap_f, cap_c;      // item capacities
    // host state
    std::vector<int> shape;  // per block
    int nf, nc;            // current item counts
    int fbeg[kShapes + 1], cbeg[kShapes + 1];  // item ranges of each tile shape
    unsigned long long base[2];
    int cur;
    double cfl_scale;
    // coupled blocks of one periodic domain (mhd_batch_couple)
    bool coupled = false;
    DomainMap dom;
    unsigned long long* d_off = nullptr;  // block offsets (cells) on the device
};

namespace {

size_t a256(size_t b) { return (b + 255) & ~size_t(255); }

struct BLayout {
    size_t reg, F, Rc, partial, dt, ctr, blk, offs, fitems, citems, cstart, clist, total;
    unsigned long long ncell;
    int cap_f, cap_c;
    std::vector<unsigned long long> off;
};

// z planes of an item: equal chunks of at most 24 (flux kernels) and 64 (CT).  A chunk
// costs the flux kernel about one plane more than its own, but few long ones leave the
// last round of workgroups part empty: 8 coupled blocks of 128^3, 3 workgroups per CU, with
// 64 64 2 planes 2046 + 2235 us, with 6 x 22 1943 + 2106 (12, 18 and 32 planes within 2 %
// of that).  512 uneven FP32 blocks, many items either way, do not care, and the CT kernels
// gain nothing (64 planes 680 + 761 us, 22 planes 704 + 780).
constexpr int kFluxPlanes = 24, kCtPlanes = 64;
int chunks_of(int nz, int most) { return (nz + most - 1) / most; }
int chunk_of(int nz, int most)
{
    const int n = chunks_of(nz, most);
    return (nz + n - 1) / n;
}

// The most items a block can have (a coupled block's range is shorter, never longer).
long long flux_items_of(const mhd_grid& g, int s)
{
    const int ty = flux_ty(s);
    return (long long)((g.nx + kFluxTX[s] - 1) / kFluxTX[s]) * ((g.ny + ty - 1) / ty) * chunks_of(g.nz, kFluxPlanes);
}
long long ct_items_of(const mhd_grid& g, int s)
{
    const int ty = ct_ty(s);
    return (long long)((g.nx + kCtTX[s] - 1) / kCtTX[s]) * ((g.ny + ty - 1) / ty) * chunks_of(g.nz, kCtPlanes);
}

mhd_status bvalidate(int nb, const mhd_grid* grids, const mhd_physics* p, const mhd_scheme* s)
{
    if (nb < 1 || !grids || !p || !s) return MHD_E_INVAL;
    if (p->eos != MHD_EOS_ADIABATIC_MHD || p->ndust != 0) return MHD_E_UNSUPPORTED;
    if (s->integ != MHD_INT_VL2 && s->integ != MHD_INT_RK2 && s->integ != MHD_INT_EULER1)
        return MHD_E_UNSUPPORTED;
    if (s->prec != MHD_PREC_FP64 && s->prec != MHD_PREC_FP32_BULK) return MHD_E_UNSUPPORTED;
    if (s->recon < MHD_RECON_DC || s->recon > MHD_RECON_PPM) return MHD_E_UNSUPPORTED;
    if (s->riemann != MHD_RS_HLLE && s->riemann != MHD_RS_HLLD) return MHD_E_UNSUPPORTED;
    if (!(s->courant > 0.0) || !std::isfinite(s->courant)) return MHD_E_INVAL;
    if (!(p->gamma > 1.0)) return MHD_E_INVAL;
    long long tot = 0;
    for (int b = 0; b < nb; ++b) {
        const mhd_grid& g = grids[b];
        if (g.nx < 1 || g.ny < 1 || g.nz < 1) return MHD_E_INVAL;
        for (int a = 0; a < 3; ++a)
            if (!(g.length[a] > 0.0) || !std::isfinite(g.length[a])) return MHD_E_INVAL;
        const long long n = (long long)g.nx * g.ny * g.nz;
        tot += (n + kAlignCells - 1) / kAlignCells * kAlignCells;
        // 32-bit offsets inside a block, and the whole batch below 2^29 cells
        if (n >= (1LL << 29) || tot >= (1LL << 29)) return MHD_E_UNSUPPORTED;
    }
    return MHD_OK;
}

BLayout blayout(int nb, const mhd_grid* grids, const mhd_scheme* s)
{
    BLayout L;
    const bool fp32 = s->prec == MHD_PREC_FP32_BULK;
    unsigned long long o = 0;
    long long cf = 0, cc = 0, maxblk = 1;
    for (int b = 0; b < nb; ++b) {
        const mhd_grid& g = grids[b];
        const long long n = (long long)g.nx * g.ny * g.nz;
        L.off.push_back(o);
        o += (unsigned long long)((n + kAlignCells - 1) / kAlignCells * kAlignCells);
        long long mf = 0, mc = 0;
        for (int sh = 0; sh < kShapes; ++sh) {
            mf = std::max(mf, flux_items_of(g, sh));
            mc = std::max(mc, ct_items_of(g, sh));
        }
        cf += mf;
        cc += mc;
        maxblk = std::max(maxblk, (long long)blocks_for(n));
    }
    L.ncell = o;
    L.cap_f = (int)cf;
    L.cap_c = (int)cc;
    L.reg = a256((size_t)o * register_bytes(1, fp32));
    L.F = a256((size_t)o * 8 * sizeof(double));  // 6 face fields, or a canonical FP64 state
    L.Rc = a256(edge_area_bytes((long long)o, fp32));
    // CFL partials: one per CT item, per workgroup of a block's own reduction, or per
    // workgroup of the reduction over all blocks' cells (a coupled domain)
    L.partial = a256((size_t)std::max({cc, maxblk, (long long)blocks_for((long long)o)}) * sizeof(double));
    L.dt = a256((size_t)nb * sizeof(double));
    L.ctr = a256(2 * sizeof(unsigned long long));
    L.blk = a256((size_t)nb * sizeof(BlockDesc));
    L.offs = a256((size_t)nb * sizeof(unsigned long long));
    L.fitems = a256((size_t)cf * sizeof(WorkItem));
    L.citems = a256((size_t)cc * sizeof(WorkItem));
    L.cstart = a256((size_t)(nb + 1) * sizeof(int));
    L.clist = a256((size_t)cc * sizeof(int));
    L.total = 3 * L.reg + L.F + L.Rc + L.partial + L.dt + L.ctr + L.blk + L.offs + L.fitems + L.citems +
              L.cstart + L.clist;
    return L;
}

mhd_status bdev(hipError_t e) { return e == hipSuccess ? MHD_OK : MHD_E_DEVICE; }

// Default tile shape of a block: the widest tile that wastes no more lanes along x
// than the narrower ones.
int default_shape(int nx)
{
    int best = 0;
    long long waste_best = -1;
    for (int s = 0; s < kShapes; ++s) {
        const long long waste = (long long)((nx + kFluxTX[s] - 1) / kFluxTX[s]) * kFluxTX[s] - nx;
        if (waste_best < 0 || waste < waste_best) {
            waste_best = waste;
            best = s;
        }
    }
    return best;
}

// Build both item lists (only blocks with include[b]), sorted by decreasing cost, and
// the per-block CSR lists of CT items; upload them.
mhd_status build_items(mhd_batch* c, const std::vector<char>& include)
{
    std::vector<WorkItem> fi, ci;
    for (int b = 0; b < c->nb; ++b) {
        if (!include[b]) continue;
        const Geo& g = c->geo[b];
        const int s = c->shape[b];
        // the cells whose face fields are advanced, and one more on every side, whose
        // fluxes and face values the edges around them take: all of a block on its own, the
        // interior of a coupled one (the exchange fills every ghost cell after the stage).
        // 8 blocks of 128^3 and 3 ghost layers: the CT kernels 936 + 1052 -> 680 + 761 us, the
        // flux kernels, whose 130 cells take as many 16-wide tiles as 134, 2112 + 2280 ->
        // 2046 + 2235 us.
        const int gh = c->coupled ? c->dom.g : 0, fh = gh > 0 ? gh - 1 : 0;
        const int kz = chunk_of(g.nz - 2 * fh, kFluxPlanes), kzc = chunk_of(g.nz - 2 * gh, kCtPlanes);
        for (int k0 = fh; k0 < g.nz - fh; k0 += kz)
            for (int y0 = fh; y0 < g.ny - fh; y0 += flux_ty(s))
                for (int x0 = fh; x0 < g.nx - fh; x0 += kFluxTX[s])
                    fi.push_back(WorkItem{b, x0, y0, k0, std::min(k0 + kz, g.nz - fh), s});
        for (int k0 = gh; k0 < g.nz - gh; k0 += kzc)
            for (int y0 = gh; y0 < g.ny - gh; y0 += ct_ty(s))
                for (int x0 = gh; x0 < g.nx - gh; x0 += kCtTX[s])
                    ci.push_back(WorkItem{b, x0, y0, k0, std::min(k0 + kzc, g.nz - gh), s});
    }
    // grouped by tile shape (one launch each), longest z chunks first within a shape
    auto order = [](const WorkItem& a, const WorkItem& b) {
        if (a.shape != b.shape) return a.shape < b.shape;
        return a.k1 - a.k0 > b.k1 - b.k0;
    };
    std::stable_sort(fi.begin(), fi.end(), order);
    std::stable_sort(ci.begin(), ci.end(), order);
    for (int sh = 0; sh <= kShapes; ++sh) {
        c->fbeg[sh] = (int)(std::lower_bound(fi.begin(), fi.end(), sh, [](const WorkItem& w, int v) { return w.shape < v; }) - fi.begin());
        c->cbeg[sh] = (int)(std::lower_bound(ci.begin(), ci.end(), sh, [](const WorkItem& w, int v) { return w.shape < v; }) - ci.begin());
    }
    if ((int)fi.size() > c->cap_f || (int)ci.size() > c->cap_c) return MHD_E_NOMEM;
    std::vector<int> start(c->nb + 1, 0), list(ci.size());
    for (const WorkItem& w : ci) ++start[w.block + 1];
    for (int b = 0; b < c->nb; ++b) start[b + 1] += start[b];
    std::vector<int> fill(start.begin(), start.end() - 1);
    for (int q = 0; q < (int)ci.size(); ++q) list[fill[ci[q].block]++] = q;
    hipError_t e = hipSuccess;
    if (!fi.empty()) e = hipMemcpyAsync(c->d_fitems, fi.data(), fi.size() * sizeof(WorkItem), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess && !ci.empty())
        e = hipMemcpyAsync(c->d_citems, ci.data(), ci.size() * sizeof(WorkItem), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(c->d_cstart, start.data(), start.size() * sizeof(int), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess && !list.empty())
        e = hipMemcpyAsync(c->d_clist, list.data(), list.size() * sizeof(int), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);  // the host vectors go out of scope
    c->nf = (int)fi.size();
    c->nc = (int)ci.size();
    return bdev(e);
}

mhd_status build_all(mhd_batch* c) { return build_items(c, std::vector<char>(c->nb, 1)); }

int persistent_grid(const mhd_batch* c, int nitems) { return std::max(1, std::min(nitems, 4 * c->cus)); }

template <int RECON, int RS, bool IN, class R, int SH>
void flux_launch(mhd_batch* c, const BatchCt& a)
{
    const int m = c->fbeg[SH + 1] - c->fbeg[SH];
    if (m == 0) return;
    const int grid = persistent_grid(c, m);
    hipLaunchKernelGGL((k_flux3_batch<RECON, RS, IN, R, SH>), dim3(grid), dim3(kFluxThreads), 0, c->stream,
                       c->d_blk, c->d_fitems + c->fbeg[SH], m, c->ctr, c->base[0], c->mp, a, (R*)c->F,
                       (R*)c->Rc, flow_area<R>(c->Rc, (long long)c->ncell));
    c->base[0] += (unsigned long long)m + grid;
}

template <int RECON, int RS, bool IN, class R>
void flux_shapes(mhd_batch* c, const BatchCt& a)
{
    flux_launch<RECON, RS, IN, R, 0>(c, a);
    flux_launch<RECON, RS, IN, R, 1>(c, a);
    flux_launch<RECON, RS, IN, R, 2>(c, a);
}

template <int RECON, int RS, class R>
void flux_in(mhd_batch* c, const BatchCt& a, bool use_in)
{
    if (use_in) flux_shapes<RECON, RS, true, R>(c, a);
    else flux_shapes<RECON, RS, false, R>(c, a);
}

template <class R>
void flux_any(mhd_batch* c, int recon, const BatchCt& a, bool use_in)
{
    if (c->scheme.riemann == MHD_RS_HLLD) {
        if (recon == 0) flux_in<0, 1, R>(c, a, use_in);
        else if (recon == 1) flux_in<1, 1, R>(c, a, use_in);
        else flux_in<2, 1, R>(c, a, use_in);
    } else {
        if (recon == 0) flux_in<0, 0, R>(c, a, use_in);
        else if (recon == 1) flux_in<1, 0, R>(c, a, use_in);
        else flux_in<2, 0, R>(c, a, use_in);
    }
}

template <bool CFL, bool IN, class R, int SH>
void ct_launch(mhd_batch* c, const BatchCt& a)
{
    const int m = c->cbeg[SH + 1] - c->cbeg[SH];
    if (m == 0) return;
    const int grid = persistent_grid(c, m);
    hipLaunchKernelGGL((k_ct_batch<CFL, IN, R, SH>), dim3(grid), dim3(kCtThreads), 0, c->stream, c->d_blk,
                       c->d_citems + c->cbeg[SH], m, c->cbeg[SH], c->ctr + 1, c->base[1], c->mp, a,
                       (const R*)c->F, (const R*)c->Rc, flow_area<R>(c->Rc, (long long)c->ncell));
    c->base[1] += (unsigned long long)m + grid;
}

template <bool CFL, bool IN, class R>
void ct_shapes(mhd_batch* c, const BatchCt& a)
{
    ct_launch<CFL, IN, R, 0>(c, a);
    ct_launch<CFL, IN, R, 1>(c, a);
    ct_launch<CFL, IN, R, 2>(c, a);
}

template <class R>
void ct_any(mhd_batch* c, const BatchCt& a, bool cfl, bool use_in)
{
    if (cfl) {
        if (use_in) ct_shapes<true, true, R>(c, a);
        else ct_shapes<true, false, R>(c, a);
    } else {
        if (use_in) ct_shapes<false, true, R>(c, a);
        else ct_shapes<false, false, R>(c, a);
    }
}

// One stage over every block: out = g0 in + g1 base + beta dt L: the cell fields with
// the fluxes of `in`, then the face fields from the edge EMFs (and, if last, the CFL
// step of out into dt[]).
mhd_status bstage(mhd_batch* c, int recon, char* in, char* base, char* out, double g0, double g1,
                  double beta, bool last)
{
    BatchCt a{in, base, out, c->reg_bpc, g0, g1, beta, c->dt, c->partial};
    const bool flux_in_reg = g0 != 0.0 || c->mp.gacc[0] != 0.0 || c->mp.gacc[1] != 0.0 || c->mp.gacc[2] != 0.0;
    if (c->fp32) flux_any<float>(c, recon, a, flux_in_reg);
    else flux_any<double>(c, recon, a, flux_in_reg);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return MHD_E_DEVICE;
    const bool use_in = g0 != 0.0;
    if (c->fp32) ct_any<float>(c, a, last, use_in);
    else ct_any<double>(c, a, last, use_in);
    e = hipGetLastError();
    if (e != hipSuccess) return MHD_E_DEVICE;
    if (last) {
        hipLaunchKernelGGL(k_block_min, dim3(c->nb), dim3(256), 0, c->stream, c->partial, c->d_cstart, c->d_clist,
                           c->cfl_scale, c->dt);
        e = hipGetLastError();
    }
    return bdev(e);
}

// The CFL step of a coupled domain (the minimum over every block's interior) into every
// dt[b].
hipError_t domain_cfl(mhd_batch* c, const char* reg)
{
    const DomainMap& m = c->dom;
    hipError_t e = launch_cfl_blocks(c->geo[0], c->mp, (const double*)reg, c->d_off, c->nb, m.g, m.bs[0], m.bs[1],
                                     m.bs[2], c->partial, c->dt, c->cfl_scale, c->stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dt_broadcast, dim3(1), dim3(256), 0, c->stream, c->dt, c->nb);
    return hipGetLastError();
}

// After a stage of a coupled domain: every block's ghost cells of the stage's output
// from their owners (one exchange per stage, Sec. "Mesh, Coordinates, and Boundary
// Conditions"); after the last stage also the domain's CFL step.
mhd_status domain_after_stage(mhd_batch* c, char* out, bool last)
{
    const DomainMap& m = c->dom;
    const long long per = 2LL * m.g * ((long long)m.pn[1] * m.pn[0] + (long long)m.bs[2] * m.pn[0] +
                                       (long long)m.bs[2] * m.bs[1]);
    const long long tot = per * c->nb;
    hipLaunchKernelGGL(k_ghost_fill, dim3((unsigned int)((tot + 255) / 256)), dim3(256), 0, c->stream, m, c->d_off,
                       c->nb, (double*)out);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && last) e = domain_cfl(c, out);
    return bdev(e);
}

mhd_status bstep(mhd_batch* c)
{
    const int s0 = c->cur, s1 = (c->cur + 1) % 3, s2 = (c->cur + 2) % 3;
    char* S = c->reg[s0];
    char* A = c->reg[s1];
    char* B = c->reg[s2];
    // a coupled domain takes its time step after the exchange, not from the blocks'
    // padded cells (their outer ghost layers are not updated correctly)
    const bool cp = c->coupled;
    mhd_status st;
    switch (c->scheme.integ) {
    case MHD_INT_VL2:
        st = bstage(c, MHD_RECON_DC, S, S, A, 0.0, 1.0, 0.5, false);
        if (st == MHD_OK && cp) st = domain_after_stage(c, A, false);
        if (st != MHD_OK) return st;
        st = bstage(c, c->scheme.recon, A, S, B, 0.0, 1.0, 1.0, !cp);
        if (st == MHD_OK && cp) st = domain_after_stage(c, B, true);
        c->cur = s2;
        return st;
    case MHD_INT_RK2:
        st = bstage(c, c->scheme.recon, S, S, A, 0.0, 1.0, 1.0, false);
        if (st == MHD_OK && cp) st = domain_after_stage(c, A, false);
        if (st != MHD_OK) return st;
        st = bstage(c, c->scheme.recon, A, S, B, 0.5, 0.5, 0.5, !cp);
        if (st == MHD_OK && cp) st = domain_after_stage(c, B, true);
        c->cur = s2;
        return st;
    default:
        st = bstage(c, c->scheme.recon, S, S, A, 0.0, 1.0, 1.0, !cp);
        if (st == MHD_OK && cp) st = domain_after_stage(c, A, true);
        c->cur = s1;
        return st;
    }
}

// Workgroups of a block in the launches that load and store all states: about 8192 in all,
// and never more CFL partials than a partial per 256 cells (the area holds at least those
// and one per block).
int state_grid(const mhd_batch* c)
{
    const long long cap = (long long)blocks_for((long long)c->ncell) / c->nb;
    return (int)std::max(1LL, std::min((8191LL + c->nb) / c->nb, cap));
}

// Whether the FP64 states leave by a copy per block: a single block, or blocks of a million
// cells (64 MB) and more in the mean.  A copy of a large block is up to 8 % faster than the
// kernel that stores all blocks but costs a call of its own (us, copies against the kernel):
// one block of 128^3 37.5 and 41.5, one of 256^3 412 and 448, two of 16 x 16 x 4096 39.0 and
// 40.2, three of 101^3 78.5 and 80.6; eight of 64 x 64 x 200 170 and 157, two of 64^3 12.0 and
// 10.8, 64 of 40 x 24 x 33 169 and 39.
bool copy_blocks(const mhd_batch* c) { return !c->fp32 && (c->nb == 1 || c->ncell / c->nb >= 1000000); }

size_t state_bytes(const mhd_batch* c)
{
    size_t t = 0;
    for (const Geo& g : c->geo) t += (size_t)g.n * 8 * sizeof(double);
    return t;
}

}  // namespace

extern "C" {

mhd_status mhd_batch_workspace_bytes(int nblocks, const mhd_grid* grids, const mhd_physics* phys,
                                     const mhd_scheme* scheme, size_t* bytes)
{
    if (!bytes) return MHD_E_INVAL;
    const mhd_status st = bvalidate(nblocks, grids, phys, scheme);
    if (st != MHD_OK) return st;
    *bytes = blayout(nblocks, grids, scheme).total;
    return MHD_OK;
}

mhd_status mhd_batch_create(int nblocks, const mhd_grid* grids, const mhd_physics* phys,
                            const mhd_scheme* scheme, void* workspace, size_t bytes, void* hip_stream,
                            mhd_batch** out)
{
    if (!out) return MHD_E_INVAL;
    *out = nullptr;
    mhd_status st = bvalidate(nblocks, grids, phys, scheme);
    if (st != MHD_OK) return st;
    if (!workspace || ((uintptr_t)workspace & 255u)) return MHD_E_INVAL;
    const BLayout L = blayout(nblocks, grids, scheme);
    if (bytes < L.total) return MHD_E_NOMEM;
    mhd_batch* c = new (std::nothrow) mhd_batch();
    if (!c) return MHD_E_NOMEM;
    c->nb = nblocks;
    c->phys = *phys;
    c->scheme = *scheme;
    c->fp32 = scheme->prec == MHD_PREC_FP32_BULK;
    c->reg_bpc = (int)register_bytes(1, c->fp32);
    c->stream = (hipStream_t)hip_stream;
    c->mp.gamma = phys->gamma;
    c->mp.gm1inv = 1.0 / (phys->gamma - 1.0);
    c->mp.rho_floor = phys->rho_floor;
    c->mp.p_floor = phys->p_floor;
    c->mp.hlld_eps = c->fp32 && scheme->hlld_eps < 1e-6 ? 1e-6 : scheme->hlld_eps;
    for (int a = 0; a < 3; ++a) c->mp.gacc[a] = phys->gas_accel[a];
    c->cfl_scale = scheme->courant;  // C_max = 1 for VL2, RK2 and EULER1
    c->off = L.off;
    c->ncell = L.ncell;
    c->cap_f = L.cap_f;
    c->cap_c = L.cap_c;
    std::vector<BlockDesc> desc(nblocks);
    unsigned long long at = 0;
    for (int b = 0; b < nblocks; ++b) {
        const mhd_grid& g = grids[b];
        Geo q;
        q.nx = g.nx; q.ny = g.ny; q.nz = g.nz;
        q.n = (long long)g.nx * g.ny * g.nz;
        const int ns[3] = {g.nx, g.ny, g.nz};
        for (int a = 0; a < 3; ++a) {
            q.dx[a] = g.length[a] / ns[a];
            q.inv_dx[a] = 1.0 / q.dx[a];
        }
        c->geo.push_back(q);
        desc[b] = BlockDesc{q, L.off[b], at};
        at += (unsigned long long)q.n;
        c->shape.push_back(default_shape(g.nx));
    }
    int dev = 0;
    c->cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) c->cus = v;
    }
    char* p = (char*)workspace;
    for (int r = 0; r < 3; ++r) {
        c->reg[r] = p;
        p += L.reg;
    }
    c->F = p; p += L.F;
    c->Rc = p; p += L.Rc;
    c->partial = (double*)p; p += L.partial;
    c->dt = (double*)p; p += L.dt;
    c->ctr = (unsigned long long*)p; p += L.ctr;
    c->d_blk = (BlockDesc*)p; p += L.blk;
    c->d_off = (unsigned long long*)p; p += L.offs;
    c->d_fitems = (WorkItem*)p; p += L.fitems;
    c->d_citems = (WorkItem*)p; p += L.citems;
    c->d_cstart = (int*)p; p += L.cstart;
    c->d_clist = (int*)p;
    c->base[0] = c->base[1] = 0;
    c->cur = 0;
    // counters start at zero; the block table and the default item lists go up once
    const unsigned long long zero[2] = {0, 0};
    hipError_t e = hipMemcpyAsync(c->ctr, zero, sizeof(zero), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(c->d_blk, desc.data(), desc.size() * sizeof(BlockDesc), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(c->d_off, L.off.data(), L.off.size() * sizeof(unsigned long long), hipMemcpyHostToDevice,
                           c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    st = e == hipSuccess ? build_all(c) : MHD_E_DEVICE;
    if (st != MHD_OK) {
        delete c;
        return st;
    }
    *out = c;
    return MHD_OK;
}

mhd_status mhd_batch_state_len(const mhd_batch* c, size_t* n)
{
    if (!c || !n) return MHD_E_INVAL;
    *n = state_bytes(c) / sizeof(double);
    return MHD_OK;
}

mhd_status mhd_batch_set_state(mhd_batch* c, const double* src, int src_is_device)
{
    if (!c || !src) return MHD_E_INVAL;
    hipError_t e = hipSuccess;
    const double* d = src;
    // what the kernel may not read where it lies goes by way of the face area, which holds
    // at least 8 doubles per cell
    if (!src_is_device || !in_place(src, c->stream)) {
        e = hipMemcpyAsync(c->F, src, state_bytes(c), src_is_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                           c->stream);
        d = (const double*)c->F;
    }
    if (e == hipSuccess)
        e = launch_batch_load(c->d_blk, c->nb, state_grid(c), c->mp, c->fp32, d, c->reg[c->cur], c->partial, c->dt,
                              c->cfl_scale, c->stream);
    if (e == hipSuccess && !src_is_device) e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess && c->coupled) return domain_after_stage(c, c->reg[c->cur], true);
    return bdev(e);
}

mhd_status mhd_batch_get_state(mhd_batch* c, double* dst, int dst_is_device)
{
    if (!c || !dst) return MHD_E_INVAL;
    if (copy_blocks(c)) {
        hipError_t e = hipSuccess;
        double* d = dst;
        for (int b = 0; b < c->nb && e == hipSuccess; ++b) {
            const size_t m = (size_t)c->geo[b].n * 8;
            e = hipMemcpyAsync(d, (const double*)c->reg[c->cur] + c->off[b] * 8ULL, m * sizeof(double),
                               dst_is_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, c->stream);
            d += m;
        }
        if (e == hipSuccess && !dst_is_device) e = hipStreamSynchronize(c->stream);
        return bdev(e);
    }
    const bool direct = dst_is_device && in_place(dst, c->stream);
    double* d = direct ? dst : (double*)c->F;
    hipError_t e = launch_batch_store(c->d_blk, c->nb, state_grid(c), c->fp32, c->reg[c->cur], d, c->stream);
    if (e == hipSuccess && !direct)
        e = hipMemcpyAsync(dst, d, state_bytes(c), dst_is_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                           c->stream);
    if (e == hipSuccess && !dst_is_device) e = hipStreamSynchronize(c->stream);
    return bdev(e);
}

mhd_status mhd_batch_step(mhd_batch* c, const double* dt)
{
    if (!c) return MHD_E_INVAL;
    if (dt) {
        for (int b = 0; b < c->nb; ++b) {
            if (!(dt[b] > 0.0) || !std::isfinite(dt[b])) return MHD_E_INVAL;
            if (c->coupled && dt[b] != dt[0]) return MHD_E_INVAL;  // one domain, one step
        }
        hipError_t e = hipMemcpyAsync(c->dt, dt, (size_t)c->nb * sizeof(double), hipMemcpyHostToDevice, c->stream);
        if (e != hipSuccess) return MHD_E_DEVICE;
    }
    return bstep(c);
}

mhd_status mhd_batch_dt_cfl(mhd_batch* c, double* dt)
{
    if (!c || !dt) return MHD_E_INVAL;
    hipError_t e = hipMemcpyAsync(dt, c->dt, (size_t)c->nb * sizeof(double), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return MHD_E_DEVICE;
    for (int b = 0; b < c->nb; ++b)
        if (!std::isfinite(dt[b]) || !(dt[b] > 0.0)) return MHD_E_NONFINITE;
    return MHD_OK;
}

mhd_status mhd_batch_set_shapes(mhd_batch* c, const int* shapes, int n)
{
    if (!c || !shapes || n != c->nb) return MHD_E_INVAL;
    for (int b = 0; b < n; ++b)
        if (shapes[b] < 0 || shapes[b] >= kShapes) return MHD_E_INVAL;
    for (int b = 0; b < n; ++b) c->shape[b] = shapes[b];
    return build_all(c);
}

mhd_status mhd_batch_get_shapes(const mhd_batch* c, int* shapes, int n)
{
    if (!c || !shapes || n != c->nb) return MHD_E_INVAL;
    for (int b = 0; b < n; ++b) shapes[b] = c->shape[b];
    return MHD_OK;
}

mhd_status mhd_batch_tune(mhd_batch* c, int reps, float* ms_out, int nout)
{
    if (!c || reps < 1) return MHD_E_INVAL;
    // classes: blocks of one x extent share a tile shape
    std::vector<int> xs;
    for (const Geo& g : c->geo) xs.push_back(g.nx);
    std::sort(xs.begin(), xs.end());
    xs.erase(std::unique(xs.begin(), xs.end()), xs.end());
    if (ms_out && nout < (int)xs.size() * kShapes) return MHD_E_INVAL;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return MHD_E_DEVICE;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return MHD_E_DEVICE;
    }
    const std::vector<int> saved = c->shape;
    std::vector<int> best(xs.size(), 0);
    mhd_status st = MHD_OK;
    const int s0 = c->cur, s1 = (c->cur + 1) % 3;
    for (size_t q = 0; q < xs.size() && st == MHD_OK; ++q) {
        std::vector<char> inc(c->nb);
        for (int b = 0; b < c->nb; ++b) inc[b] = c->geo[b].nx == xs[q];
        float tbest = 0.0f;
        for (int s = 0; s < kShapes && st == MHD_OK; ++s) {
            for (int b = 0; b < c->nb; ++b)
                if (inc[b]) c->shape[b] = s;
            st = build_items(c, inc);
            if (st != MHD_OK) break;
            // the configured-reconstruction stage into the scratch register (the state
            // itself is only read); one untimed pass, then reps timed
            float ms = 0.0f;
            for (int r = 0; r <= reps && st == MHD_OK; ++r) {
                if (r == 1 && hipEventRecord(e0, c->stream) != hipSuccess) st = MHD_E_DEVICE;
                if (st == MHD_OK)
                    st = bstage(c, c->scheme.recon, c->reg[s0], c->reg[s0], c->reg[s1], 0.0, 1.0, 1.0, false);
            }
            if (st == MHD_OK && hipEventRecord(e1, c->stream) != hipSuccess) st = MHD_E_DEVICE;
            if (st == MHD_OK && hipEventSynchronize(e1) != hipSuccess) st = MHD_E_DEVICE;
            if (st == MHD_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) st = MHD_E_DEVICE;
            if (st != MHD_OK) break;
            if (ms_out) ms_out[q * kShapes + s] = ms / reps;
            if (s == 0 || ms < tbest) {
                tbest = ms;
                best[q] = s;
            }
        }
    }
    // Classes share launches and the GPU, so the per-class optimum need not be the best
    // whole: time the full batch with it and with each uniform shape, keep the fastest.
    auto class_of = [&](int b) { return (int)(std::lower_bound(xs.begin(), xs.end(), c->geo[b].nx) - xs.begin()); };
    std::vector<std::vector<int>> cands;
    {
        std::vector<int> a(c->nb);
        for (int b = 0; b < c->nb; ++b) a[b] = best[class_of(b)];
        cands.push_back(a);
        for (int s = 0; s < kShapes; ++s) cands.push_back(std::vector<int>(c->nb, s));
    }
    int pick = 0;
    float tpick = 0.0f;
    for (size_t k = 0; k < cands.size() && st == MHD_OK; ++k) {
        c->shape = cands[k];
        st = build_all(c);
        if (st != MHD_OK) break;
        float ms = 0.0f;
        for (int r = 0; r <= reps && st == MHD_OK; ++r) {
            if (r == 1 && hipEventRecord(e0, c->stream) != hipSuccess) st = MHD_E_DEVICE;
            if (st == MHD_OK)
                st = bstage(c, c->scheme.recon, c->reg[s0], c->reg[s0], c->reg[s1], 0.0, 1.0, 1.0, false);
        }
        if (st == MHD_OK && hipEventRecord(e1, c->stream) != hipSuccess) st = MHD_E_DEVICE;
        if (st == MHD_OK && hipEventSynchronize(e1) != hipSuccess) st = MHD_E_DEVICE;
        if (st == MHD_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) st = MHD_E_DEVICE;
        if (st == MHD_OK && (k == 0 || ms < tpick)) {
            tpick = ms;
            pick = (int)k;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != MHD_OK) {
        c->shape = saved;
        (void)build_all(c);
        return st;
    }
    c->shape = cands[pick];
    return build_all(c);
}

mhd_status mhd_batch_couple(mhd_batch* c, const int nblocks_xyz[3], int ghost, const double length[3])
{
    if (!c || !nblocks_xyz || !length) return MHD_E_INVAL;
    if (c->fp32) return MHD_E_UNSUPPORTED;
    // the reconstruction's stencil plus the one cell the edge EMFs reach beyond it
    const int need = c->scheme.recon == MHD_RECON_PPM ? 4 : (c->scheme.recon == MHD_RECON_PLM ? 3 : 2);
    if (ghost < need || ghost > 64) return MHD_E_INVAL;
    long long nbt = 1;
    for (int a = 0; a < 3; ++a) {
        if (nblocks_xyz[a] < 1 || nblocks_xyz[a] > 4096) return MHD_E_INVAL;
        if (!(length[a] > 0.0) || !std::isfinite(length[a])) return MHD_E_INVAL;
        nbt *= nblocks_xyz[a];
    }
    if (nbt != c->nb) return MHD_E_INVAL;
    const Geo& g0 = c->geo[0];
    const int pn[3] = {g0.nx, g0.ny, g0.nz};
    for (int b = 1; b < c->nb; ++b)
        if (c->geo[b].nx != pn[0] || c->geo[b].ny != pn[1] || c->geo[b].nz != pn[2]) return MHD_E_INVAL;
    DomainMap m;
    m.g = ghost;
    for (int a = 0; a < 3; ++a) {
        m.nb[a] = nblocks_xyz[a];
        m.pn[a] = pn[a];
        m.bs[a] = pn[a] - 2 * ghost;
        if (m.bs[a] < 1) return MHD_E_INVAL;
        m.dn[a] = m.nb[a] * m.bs[a];
        if (m.dn[a] < ghost) return MHD_E_INVAL;  // a ghost layer must map onto distinct domain cells
    }
    m.pc = (long long)pn[0] * pn[1] * pn[2];
    m.dcells = (long long)m.dn[0] * m.dn[1] * m.dn[2];
    // every block takes the domain's spacing, as a single grid of the domain does
    std::vector<BlockDesc> desc(c->nb);
    for (int b = 0; b < c->nb; ++b) {
        for (int a = 0; a < 3; ++a) {
            c->geo[b].dx[a] = length[a] / m.dn[a];
            c->geo[b].inv_dx[a] = 1.0 / c->geo[b].dx[a];
        }
        desc[b] = BlockDesc{c->geo[b], c->off[b], (unsigned long long)b * (unsigned long long)m.pc};
    }
    hipError_t e = hipMemcpyAsync(c->d_blk, desc.data(), desc.size() * sizeof(BlockDesc), hipMemcpyHostToDevice,
                                  c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return MHD_E_DEVICE;
    c->dom = m;
    c->coupled = true;
    const mhd_status st = build_all(c);
    if (st != MHD_OK) return st;
    // the current state: ghosts from their owners, and the domain's step
    return domain_after_stage(c, c->reg[c->cur], true);
}

mhd_status mhd_batch_set_domain_state(mhd_batch* c, const double* src, int src_is_device)
{
    if (!c || !src || !c->coupled) return MHD_E_INVAL;
    const size_t nbytes = (size_t)c->dom.dcells * 8 * sizeof(double);
    const double* d = src;
    hipError_t e = hipSuccess;
    if (!src_is_device) {
        // staged through the face-flux area, which holds at least 8 doubles per cell
        e = hipMemcpyAsync(c->F, src, nbytes, hipMemcpyHostToDevice, c->stream);
        d = (const double*)c->F;
    }
    const long long tot = c->dom.pc * c->nb;
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_domain_copy<1>, dim3((unsigned int)((tot + 255) / 256)), dim3(256), 0, c->stream, c->dom,
                           c->d_off, c->nb, (double*)c->reg[c->cur], const_cast<double*>(d));
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = domain_cfl(c, c->reg[c->cur]);
    if (e == hipSuccess && !src_is_device) e = hipStreamSynchronize(c->stream);
    return bdev(e);
}

mhd_status mhd_batch_get_domain_state(mhd_batch* c, double* dst, int dst_is_device)
{
    if (!c || !dst || !c->coupled) return MHD_E_INVAL;
    const size_t nbytes = (size_t)c->dom.dcells * 8 * sizeof(double);
    double* d = dst_is_device ? dst : (double*)c->F;
    const long long tot = c->dom.pc * c->nb;
    hipLaunchKernelGGL(k_domain_copy<2>, dim3((unsigned int)((tot + 255) / 256)), dim3(256), 0, c->stream, c->dom,
                       c->d_off, c->nb, (double*)c->reg[c->cur], d);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && !dst_is_device) e = hipMemcpyAsync(dst, c->F, nbytes, hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess && !dst_is_device) e = hipStreamSynchronize(c->stream);
    return bdev(e);
}

void mhd_batch_destroy(mhd_batch* c) { delete c; }

}  // extern "C"
