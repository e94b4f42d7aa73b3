// dust_kernels.hip -- IMEX2P step of isothermal gas + N pressureless dust fluids.
//
// Explicit part F(u): minus the flux divergence (isothermal HLLE for the gas, the
// pressureless Rusanov flux for each species; Sec. "Multifluid Dust") plus the gas
// acceleration rho_g g as an unsplit source.  Implicit part G(u): the linear drag of
// eq. (dust_momentum) and its reaction on the gas.  The ARS(2,2,2) pair with the
// diagonal weight lam = 1 + 1/sqrt(2) (Sec. "Time Integration"):
//   U1    = S_h(u + lam dt F(u)),                                   h = lam dt
//   u_new = S_h(u + dt[delta F(u) + (1-delta) F(U1)] + (1-lam) dt G(U1))
// with delta = 1 - 1/(2 lam).  Stage 2 recovers dt F(u) from stage 1's own output,
// dt F(u) = (U1 - u)/lam - dt G(U1), so only the two registers u and U1 exist:
//   u_new = S_h((1 - delta/lam) u + (delta/lam) U1 + (1-delta) dt F(U1)
//               + (1 - lam - delta) dt G(U1)).
// S_h is the closed-form solve of the arrowhead drag system: with w_k = h/(t_k + h),
//   v_g' = (p_g + sum_k w_k p_k) / (rho_g + sum_k w_k rho_k),
//   p_k' = (t_k p_k + h rho_k v_g') / (t_k + h),   p_g' = rho_g v_g',
// exact, O(N) and momentum conserving.
//
// Each stage is two launches:
//   k_fluid_pass  one wave = one fluid on a tile of 64 columns x 1 or 2 rows marching a
//                 chunk of z planes; waves share nothing and there is no barrier.  A lane
//                 owns a column of each row: the z stencil is a register pipeline that
//                 carries the flux of the low z face, the y stencil the tile's rows (held
//                 by the pipelines) and the rows beside them, the x stencil the row in the
//                 wave's own LDS.  Every low x face is solved by one lane, which hands its
//                 flux to the lane on its left; the two faces at the tile's edge of all
//                 rows are solved together in one more pass.  A face is solved once per
//                 direction within a tile (x: 1 + 1/rows per cell, y: 1 + 1/rows, z: 1)
//                 and a cell's slope once (x twice on small grids, where a lane solves
//                 both faces of its cell), and each stage's explicit part is written:
//                   stage 1: X = u + h L(u);  stage 2: X = cu u + c1 U1 + cf L(U1).
//                 Densities are final after this pass (drag moves only momentum).
//   k_donor_pass  the same for the donor cell in FP64 on larger grids, a workgroup per
//                 64 x 4 columns of a fluid.
//   k_drag        pointwise: adds the stage-1 drag rates (stage 2), solves S_h for the
//                 momenta in place and, after stage 2, reduces the CFL step of the new
//                 state (one partial per workgroup).
//
// Precision: templated on the stored real type R.  R = double is the FP64 form; with
// R = float the state, the primitives, reconstruction, Riemann solves and explicit
// updates are FP32 while the drag solve (and the CFL step) stay FP64.
#include "launch.hpp"
#include "physics.hpp"

namespace mhd {

namespace {
constexpr double kLam = 1.7071067811865475244;     // 1 + 1/sqrt(2)
constexpr double kDelta = 0.70710678118654752440;  // 1 - 1/(2 lam) = 1/sqrt(2)

constexpr int DTX = 64;    // lanes along x
constexpr int DWAVES = 4;  // waves of a workgroup (independent of each other)

// Orders one wave's LDS writes before its other lanes' reads (and the reads before the
// next writes): LDS serves a wave's accesses in order, only the compiler has to keep it.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Blocks are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of work
// items so neighbouring tiles of one fluid share an L2.
__device__ __forceinline__ unsigned int xcd_item(unsigned int b, unsigned int nb)
{
    const unsigned int q = nb >> 3, rem = nb & 7u;
    const unsigned int x = b & 7u, r = b >> 3;
    return x * q + (x < rem ? x : rem) + r;
}

__device__ __forceinline__ int wrap_any(int i, int n)
{
    if (i >= 0 && i < n) return i;
    const int r = i % n;
    return r < 0 ? r + n : r;
}

template <class T>
__device__ __forceinline__ T ld(const T* __restrict__ base, unsigned int idx)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + idx * (unsigned int)sizeof(T));
}
template <class T>
__device__ __forceinline__ void st(T* base, unsigned int idx, T v)
{
    *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + idx * (unsigned int)sizeof(T)) = v;
}

// Halo (cells on each side) of the reconstruction when both faces of a cell are built.
template <int RECON>
struct Halo {
    static constexpr int H = RECON == 0 ? 1 : 2;
};

// Face flux along direction D from the global-frame states; returns global-frame
// components (mass, Mx, My, Mz).
template <int D, bool GAS, class R>
__device__ __forceinline__ void face_flux(R cs, const R L[4], const R Rs[4], R out[4])
{
    constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
    const Prim4<R> l{L[0], L[1 + D], L[1 + T1], L[1 + T2]};
    const Prim4<R> r{Rs[0], Rs[1 + D], Rs[1 + T1], Rs[1 + T2]};
    Flux4<R> f;
    if constexpr (GAS)
        riemann_iso_hlle(l, r, cs, f);
    else
        riemann_dust(l, r, f);
    out[0] = f.d;
    out[1 + D] = f.mn;
    out[1 + T1] = f.mt1;
    out[1 + T2] = f.mt2;
}

}  // namespace

// ----------------------------------------------------------------------------------
// explicit part of a stage, one fluid per wave (or per workgroup, donor cell in FP64)
// ----------------------------------------------------------------------------------

template <class R>
struct PassArgs {
    const R* src;   // state whose fluxes are taken (u in stage 1, U1 in stage 2)
    const R* base;  // stage 2: u (read at the own cell only); stage 1: unused
    R* out;         // stage 1: U1; stage 2: u (in place: each cell reads then writes itself)
    double h;       // stage 1: lam dt; stage 2: (1 - delta) dt
    double cu, c1;  // stage 2 weights of u and U1
};

// z reconstruction of one variable of one column as a pipeline over the planes the
// column visits: push(plane m + 1 + AHEAD) returns the two states on the face m + 1/2
// (one slope per plane for PLM).  Between the pushes of planes m + AHEAD and m + 1 + AHEAD
// here() is the value of plane m.
template <int RECON, class R>
struct ZLine;
template <class R>
struct ZLine<0, R> {
    static constexpr int AHEAD = 0, PRIME = 1;
    R prev;
    __device__ void prime(const R* a) { prev = a[0]; }
    __device__ R here() const { return prev; }
    __device__ void push(R a, R& aL, R& aR)
    {
        aL = prev;
        aR = a;
        prev = a;
    }
};
template <class R>
struct ZLine<1, R> {
    static constexpr int AHEAD = 1, PRIME = 3;
    R am, a0, apl;  // a(m-1), a(m), high-side state of cell m-1
    __device__ void prime(const R* a)
    {
        apl = a[1] + R(0.5) * slope_vl(a[0], a[1], a[2]);
        am = a[1];
        a0 = a[2];
    }
    __device__ R here() const { return am; }
    __device__ void push(R a, R& aL, R& aR)
    {
        const R d = slope_vl(am, a0, a);
        aL = apl;
        aR = a0 - R(0.5) * d;
        apl = a0 + R(0.5) * d;
        am = a0;
        a0 = a;
    }
};

// Value of the lane on the left / right of a wavefront (the first / last lane: `edge`).
__device__ __forceinline__ float lane_left(float v, float edge)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_right(float v, float edge)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ double lane_left(double v, double edge)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), 0x138, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), 0x138, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_right(double v, double edge)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), 0x130, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), 0x130, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// States of a cell on its low and high face from the cell and its two neighbours.
template <int RECON, class R>
__device__ __forceinline__ void cell_states(R am, R a0, R ap, R& lo, R& hi)
{
    if constexpr (RECON == 0) {
        lo = hi = a0;
    } else {
        const R s = slope_vl(am, a0, ap);
        lo = fma_r(R(-0.5), s, a0);
        hi = fma_r(R(0.5), s, a0);
    }
}

template <int RECON, class R, int NR>
struct PassLds {
    static constexpr int LX = DTX + 2 * Halo<RECON>::H;
    R row[NR][4][LX];  // primitives of the wave's rows with their x halo
    R edge[NR][2][4];  // (not SOLO) high-side state of column x0 - 1, flux through face x0 + 63 1/2
};

// One wave's tile of fluid s (GAS: the gas, else a dust species; a template argument so
// that the faces of a cell are one straight block).  Bound by its arithmetic and its
// latency at two (FP64) and three (FP32) waves per SIMD; 192^3, 8 species, PLM, stage 1 /
// stage 2: FP64 2.28 / 2.41 -> 1.65 / 1.76 ms, FP32 0.98 / 1.03 -> 0.83 / 0.87 ms against
// a workgroup of four waves on 64 x 4 columns that staged the tile with its halo in
// double-buffered LDS and solved both faces of every cell in x and y (five Riemann
// problems and seven slopes per variable and cell; here four and five).  Four rows need
// more registers than two waves per SIMD leave (FP64 spills: 3.7 ms; FP32 0.96 ms).
// SOLO (a single row): every lane solves both faces of its cell along x instead of the edge
// faces' own pass.  As many instructions, without the wait for a second exchange, but more
// registers (FP64 PLM 184 against 164, two waves per SIMD against three).
template <int RECON, int STAGE, class R, int NR, bool GAS, bool SOLO>
__device__ __forceinline__ void fluid_tile(const Geo& g, const DustParams& p, const PassArgs<R>& a, int s, int x0,
                                           int y0, int k0, int k1, PassLds<RECON, R, NR>& lds)
{
    // every rounding is written out: a cell's update does not depend on the tiling
#pragma clang fp contract(off)
    constexpr int H = Halo<RECON>::H, NX = NR * 2 * H;
    static_assert(NX <= 64, "one lane per cell of the x halo");
    using Z = ZLine<RECON, R>;
    const int lane = (int)threadIdx.x & 63;
    const int i = x0 + lane;
    const bool live = i < g.nx;
    // columns and rows past the grid's edge are the periodic ones
    const unsigned int col = (unsigned int)wrap_any(i, g.nx);
    const long long n = g.n;
    const unsigned int plane = (unsigned int)g.nx * (unsigned int)g.ny;
    auto rowoff = [&](int r) { return (unsigned int)wrap_any(y0 + r, g.ny) * (unsigned int)g.nx; };
    const R *f[4], *b[4];
    R* o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f[q] = a.src + (4LL * s + q) * n;
        b[q] = a.base + (4LL * s + q) * n;
        o[q] = a.out + (4LL * s + q) * n;
    }
    const R cs = R(p.cs);
    const R rho_floor = R(p.rho_floor), dust_floor = R(p.dust_floor);
    const R gx3[3] = {R(p.gacc[0]), R(p.gacc[1]), R(p.gacc[2])};
    const R hr = R(a.h), cur_ = R(a.cu), c1r = R(a.c1);
    const R idx[3] = {R(g.inv_dx[0]), R(g.inv_dx[1]), R(g.inv_dx[2])};

    // primitives from the raw state: the gas density is floored; a dust species below
    // its floor reads as the floor at rest
    auto prim_of = [&](const R raw[4], R w[4]) {
        const bool rest = !GAS && raw[0] < dust_floor;
        R d = raw[0];
        if (GAS && d < rho_floor) d = rho_floor;
        const R id = rcp(d);
        w[0] = rest ? dust_floor : d;
        w[1] = rest ? R(0) : raw[1] * id;
        w[2] = rest ? R(0) : raw[2] * id;
        w[3] = rest ? R(0) : raw[3] * id;
    };
    auto load_raw = [&](unsigned int c, R raw[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) raw[q] = ld(f[q], c);
    };
    // this lane's cell of the x halo: row xr, column xe of the staged row
    const int xr = lane / (2 * H), xc = lane % (2 * H), xe = xc < H ? xc : DTX + xc;
    const unsigned int xoff = lane < NX ? (unsigned int)wrap_any(y0 + xr, g.ny) * (unsigned int)g.nx +
                                              (unsigned int)wrap_any(x0 + xe - H, g.nx)
                                        : 0u;

    // z pipelines of the own columns, primed so that the first push yields face k0 - 1/2
    Z zl[NR][4];
    R fzlo[NR][4];  // z flux on the low face of the current cell
    R zraw[NR][4];  // raw state of the next plane the z pipeline takes
    R xraw[4];      // raw x halo of the current plane
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        R pre[4][Z::PRIME];
#pragma unroll
        for (int m = 0; m < Z::PRIME; ++m) {
            R r4[4], w[4];
            load_raw((unsigned int)wrap_any(k0 - Z::PRIME + Z::AHEAD + m, g.nz) * plane + rowoff(r) + col, r4);
            prim_of(r4, w);
#pragma unroll
            for (int v = 0; v < 4; ++v) pre[v][m] = w[v];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) zl[r][v].prime(pre[v]);
        load_raw((unsigned int)wrap_any(k0 + Z::AHEAD, g.nz) * plane + rowoff(r) + col, zraw[r]);
        R w[4], L[4], Rr[4];
        prim_of(zraw[r], w);
#pragma unroll
        for (int v = 0; v < 4; ++v) zl[r][v].push(w[v], L[v], Rr[v]);
        face_flux<2, GAS>(cs, L, Rr, fzlo[r]);
        load_raw((unsigned int)wrap_any(k0 + 1 + Z::AHEAD, g.nz) * plane + rowoff(r) + col, zraw[r]);
    }
    if (lane < NX) load_raw((unsigned int)k0 * plane + xoff, xraw);

    for (int k = k0; k < k1; ++k) {
        const bool more = k + 1 < k1;
        const unsigned int pb = (unsigned int)k * plane;
        wave_sync();  // the plane below is read
        R hraw[2 * H][4];  // the rows below and above the tile, needed after the edge faces
#pragma unroll
        for (int m = 0; m < 2 * H; ++m) load_raw(pb + rowoff(m < H ? m - H : NR + m - H) + col, hraw[m]);
        // ---- the rows of plane k with their x halo
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int v = 0; v < 4; ++v) lds.row[r][v][lane + H] = zl[r][v].here();
        if (lane < NX) {
            R w[4];
            prim_of(xraw, w);
#pragma unroll
            for (int v = 0; v < 4; ++v) lds.row[xr][v][xe] = w[v];
        }
        // the x halo of the next plane goes out first; it lands while this plane computes
        if (more && lane < NX) load_raw(pb + plane + xoff, xraw);
        wave_sync();
        // ---- the edge faces of all rows in one pass: lane 2 r + e the face at x0 + 64 e of row r
        if (!SOLO && lane < 2 * NR) {
            const int r = lane >> 1, e = lane & 1;
            R lo[4], hi[4], fx[4], dum;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const R* q = &lds.row[r][v][e * DTX];
                if constexpr (RECON == 0) {
                    hi[v] = q[0];
                    lo[v] = q[1];
                } else {
                    cell_states<RECON, R>(q[0], q[1], q[2], dum, hi[v]);
                    cell_states<RECON, R>(q[1], q[2], q[3], lo[v], dum);
                }
            }
            face_flux<0, GAS>(cs, hi, lo, fx);
#pragma unroll
            for (int v = 0; v < 4; ++v) lds.edge[r][e][v] = e ? fx[v] : hi[v];
        }
        if constexpr (!SOLO) wave_sync();

        R hv[2 * H][4];
#pragma unroll
        for (int m = 0; m < 2 * H; ++m) prim_of(hraw[m], hv[m]);
        // ---- y: flux through the low face of row 0, then one face per row
        R hy[4], fy[4];  // high-side state of the row below, flux through the face above it
        {
            R lo[4], dum, hm[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if constexpr (RECON == 0) {
                    hm[v] = hv[0][v];
                } else {
                    cell_states<RECON, R>(hv[0][v], hv[1][v], zl[0][v].here(), dum, hm[v]);
                }
                const R below = hv[H - 1][v], up = NR > 1 ? zl[NR > 1 ? 1 : 0][v].here() : hv[H][v];
                cell_states<RECON, R>(below, zl[0][v].here(), up, lo[v], hy[v]);
            }
            face_flux<1, GAS>(cs, hm, lo, fy);
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const unsigned int c = pb + rowoff(r) + col;
            R own[4], ub[4];
            load_raw(c, own);
            if constexpr (STAGE == 2) {
#pragma unroll
                for (int v = 0; v < 4; ++v) ub[v] = ld(b[v], c);
            }
            // acc = ((fx + fy) + fz): flux differences over the spacings, direction by direction
            R acc[4];
            if constexpr (SOLO) {
                R lo[4], hi[4], ot[4], fl[4], dum;  // own states, the one beside
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const R* q = &lds.row[r][v][lane + H];
                    const R a0 = zl[r][v].here();
                    cell_states<RECON, R>(q[-1], a0, q[1], lo[v], hi[v]);
                    cell_states<RECON, R>(q[-H], q[-1], a0, dum, ot[v]);
                }
                face_flux<0, GAS>(cs, ot, lo, fl);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const R* q = &lds.row[r][v][lane + H];
                    cell_states<RECON, R>(zl[r][v].here(), q[1], q[H], ot[v], dum);
                }
                face_flux<0, GAS>(cs, hi, ot, lo);
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] = lo[v] - fl[v];
            } else {
                R lo[4], hi[4], L[4], fl[4], ed[4];
                const R* e = &lds.edge[r][lane == 63][0];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    ed[v] = e[v];
                    const R* q = &lds.row[r][v][lane + H];
                    cell_states<RECON, R>(RECON == 0 ? R(0) : q[-1], zl[r][v].here(), RECON == 0 ? R(0) : q[1], lo[v], hi[v]);
                    L[v] = lane_left(hi[v], ed[v]);
                }
                face_flux<0, GAS>(cs, L, lo, fl);
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] = lane_right(fl[v], ed[v]) - fl[v];
            }
            {
                R lo[4], hn[4], fn[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    // the row above, between row r and the one after it
                    const R up0 = r + 1 < NR ? zl[r + 1 < NR ? r + 1 : 0][v].here() : hv[H][v];
                    const R up1 = RECON == 0 ? R(0)
                                  : r + 2 < NR ? zl[r + 2 < NR ? r + 2 : 0][v].here() : hv[H + (r + 2 - NR < H ? r + 2 - NR : 0)][v];
                    cell_states<RECON, R>(zl[r][v].here(), up0, up1, lo[v], hn[v]);
                }
                face_flux<1, GAS>(cs, hy, lo, fn);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    acc[v] = fma_r(acc[v], idx[0], (fn[v] - fy[v]) * idx[1]);
                    fy[v] = fn[v];
                    hy[v] = hn[v];
                }
            }
            {
                R zw[4], L[4], Rr[4], fh[4];
                prim_of(zraw[r], zw);
                if (more)
                    load_raw((unsigned int)wrap_any(k + 2 + Z::AHEAD, g.nz) * plane + rowoff(r) + col, zraw[r]);
#pragma unroll
                for (int v = 0; v < 4; ++v) zl[r][v].push(zw[v], L[v], Rr[v]);
                face_flux<2, GAS>(cs, L, Rr, fh);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    acc[v] = fma_r(fh[v] - fzlo[r][v], idx[2], acc[v]);
                    fzlo[r][v] = fh[v];
                }
            }
            if (live && y0 + r < g.ny) {
                // the step's input u passes the dust floor reset (a species below its floor
                // becomes the floor at rest) where it enters the combination, in both stages
                R* uin = STAGE == 1 ? own : ub;
                if (!GAS && uin[0] < dust_floor) {
                    uin[0] = dust_floor;
                    uin[1] = uin[2] = uin[3] = R(0);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    R L = -acc[v];
                    // the gas acceleration acts on the raw gas density
                    if (GAS && v > 0) L = fma_r(own[0], gx3[v - 1], L);
                    R X;
                    if constexpr (STAGE == 1)
                        X = fma_r(hr, L, own[v]);
                    else
                        X = fma_r(hr, L, fma_r(cur_, ub[v], c1r * own[v]));
                    st(o[v], c, X);
                }
            }
        }
    }
}

template <int RECON, int STAGE, class R, int NR, bool SOLO>
__global__ __launch_bounds__(64 * DWAVES) __attribute__((amdgpu_waves_per_eu(2))) void k_fluid_pass(
    Geo g, DustParams p, PassArgs<R> a, int kz, unsigned int ntx, unsigned int nty, unsigned int ntiles,
    unsigned int nitems, unsigned int nblk)
{
    __shared__ PassLds<RECON, R, NR> lds[DWAVES];
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const unsigned int item = xcd_item(blockIdx.x, nblk) * DWAVES + (unsigned int)wv;
    if (item >= nitems) return;  // (the waves of a workgroup share nothing)
    const int s = __builtin_amdgcn_readfirstlane((int)(item / ntiles));  // fluid: 0 gas, 1.. dust
    const unsigned int t = item - (unsigned int)s * ntiles;
    const int y0 = __builtin_amdgcn_readfirstlane((int)(t % nty) * NR);
    const int x0 = __builtin_amdgcn_readfirstlane((int)((t / nty) % ntx) * DTX);
    const int k0 = __builtin_amdgcn_readfirstlane((int)(t / (ntx * nty)) * kz);
    const int k1 = min(k0 + kz, g.nz);
    if (s == 0)
        fluid_tile<RECON, STAGE, R, NR, true, SOLO>(g, p, a, s, x0, y0, k0, k1, lds[wv]);
    else
        fluid_tile<RECON, STAGE, R, NR, false, SOLO>(g, p, a, s, x0, y0, k0, k1, lds[wv]);
}

// What a pass takes of its arguments, in its own real.
template <class R>
struct PassConst {
    R cs, rho_floor, dust_floor, gx[3], h, cu, c1, idx[3];
    __device__ PassConst(const Geo& g, const DustParams& p, const PassArgs<R>& a)
        : cs(R(p.cs)), rho_floor(R(p.rho_floor)), dust_floor(R(p.dust_floor)),
          gx{R(p.gacc[0]), R(p.gacc[1]), R(p.gacc[2])}, h(R(a.h)), cu(R(a.cu)), c1(R(a.c1)),
          idx{R(g.inv_dx[0]), R(g.inv_dx[1]), R(g.inv_dx[2])}
    {
    }
};

// Primitives from the raw state: the gas density is floored; a dust species below its floor
// reads as the floor at rest.
template <bool GAS, class R>
__device__ __forceinline__ void prim_of(const PassConst<R>& q, const R raw[4], R w[4])
{
#pragma clang fp contract(off)
    const bool rest = !GAS && raw[0] < q.dust_floor;
    R d = raw[0];
    if (GAS && d < q.rho_floor) d = q.rho_floor;
    const R id = rcp(d);
    w[0] = rest ? q.dust_floor : d;
    w[1] = rest ? R(0) : raw[1] * id;
    w[2] = rest ? R(0) : raw[2] * id;
    w[3] = rest ? R(0) : raw[3] * id;
}

// The stage's explicit part of cell c from its raw state own, the step's input (stage 2: ub)
// and the flux divergence acc.  The input passes the dust floor reset (a species below its
// floor becomes the floor at rest) where it enters the combination, in both stages.
template <int STAGE, bool GAS, class R>
__device__ __forceinline__ void stage_store(const PassConst<R>& q, R own[4], R ub[4], const R acc[4], R* const o[4],
                                            unsigned int c)
{
#pragma clang fp contract(off)
    R* uin = STAGE == 1 ? own : ub;
    if (!GAS && uin[0] < q.dust_floor) {
        uin[0] = q.dust_floor;
        uin[1] = uin[2] = uin[3] = R(0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        R L = -acc[v];
        // the gas acceleration acts on the raw gas density
        if (GAS && v > 0) L = fma_r(own[0], q.gx[v - 1], L);
        R X;
        if constexpr (STAGE == 1)
            X = fma_r(q.h, L, own[v]);
        else
            X = fma_r(q.h, L, fma_r(q.cu, ub[v], q.c1 * own[v]));
        st(o[v], c, X);
    }
}

// The donor cell in FP64 on larger grids: a workgroup of four waves on 64 x 4 columns of one
// fluid, a row each, that stage the primitives of a plane with its x/y halo in LDS (double
// buffered: the loads of plane k + 1 go out before plane k is computed).  Without slopes the
// passes are bound by their loads, and a halo row is read here once per four rows without
// the registers of four; every cell solves both of its x and y faces (no exchange).  A stage
// of 148 x 46 x 88 with 9 species 463 us a step against 480 to 490 with independent waves of
// 1 or 2 rows in chunks of any length, 120 x 174 x 210 with 4 1621 against 1675, 100^3 with 4
// 388 against 396; with 4 rows a wave 468, 1648, 392 at the best chunk, up to 8 % more at the
// next.  FP32 gains from independent waves (128^3 with 8 694 against 656).
constexpr int DTY = 4;

template <int STAGE, class R, bool GAS>
__device__ __forceinline__ void donor_block(const Geo& g, const DustParams& p, const PassArgs<R>& a, int s, int x0,
                                            int y0, int k0, int k1, R (&sw)[2][4][DTY + 2][DTX + 2])
{
    // every rounding as in fluid_tile: the two give the same bits
#pragma clang fp contract(off)
    constexpr int LX = DTX + 2, LY = DTY + 2, NT = DTX * DTY, NI = (LX * LY + NT - 1) / NT;
    const int lane = (int)threadIdx.x & 63, row = (int)threadIdx.x >> 6;
    const int i = x0 + lane, j = y0 + row;
    const bool live = i < g.nx && j < g.ny;
    const long long n = g.n;
    const unsigned int plane = (unsigned int)g.nx * (unsigned int)g.ny;
    const unsigned int col = live ? (unsigned int)j * (unsigned int)g.nx + (unsigned int)i : 0u;
    const R *f[4], *b[4];
    R* o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f[q] = a.src + (4LL * s + q) * n;
        b[q] = a.base + (4LL * s + q) * n;
        o[q] = a.out + (4LL * s + q) * n;
    }
    const PassConst<R> pc(g, p, a);
    auto load_raw = [&](unsigned int c, R raw[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) raw[q] = ld(f[q], c);
    };
    // this thread's staging items of a plane (tile and halo without corners; a thread
    // without one loads cell 0 of the plane)
    unsigned int soff[NI];
    int at[NI];
#pragma unroll
    for (int m = 0; m < NI; ++m) {
        const int q = (int)threadIdx.x + m * NT, sr = q / LX, sc = q - sr * LX;
        const bool xh = sc < 1 || sc > DTX, yh = sr < 1 || sr > DTY;
        const bool has = q < LX * LY && !(xh && yh);
        at[m] = has ? q : -1;
        soff[m] = has ? (unsigned int)wrap_any(y0 + sr - 1, g.ny) * (unsigned int)g.nx +
                            (unsigned int)wrap_any(x0 + sc - 1, g.nx)
                      : 0u;
    }
    R raw[NI][4];
    auto fetch_plane = [&](int kk) {
#pragma unroll
        for (int m = 0; m < NI; ++m) load_raw((unsigned int)kk * plane + soff[m], raw[m]);
    };
    auto store_plane = [&](int buf) {
#pragma unroll
        for (int m = 0; m < NI; ++m)
            if (at[m] >= 0) {
                R w[4];
                prim_of<GAS>(pc, raw[m], w);
#pragma unroll
                for (int v = 0; v < 4; ++v) (&sw[buf][v][0][0])[at[m]] = w[v];
            }
    };
    // the z faces of the own column: primitives below, flux through the low face
    R zb[4], fz[4], zraw[4];
    {
        R r4[4], w[4];
        load_raw((unsigned int)wrap_any(k0 - 1, g.nz) * plane + col, r4);
        load_raw((unsigned int)k0 * plane + col, zraw);
        prim_of<GAS>(pc, r4, w);
        prim_of<GAS>(pc, zraw, zb);
        face_flux<2, GAS>(pc.cs, w, zb, fz);
    }
    load_raw((unsigned int)wrap_any(k0 + 1, g.nz) * plane + col, zraw);
    fetch_plane(k0);
    store_plane(k0 & 1);
    __syncthreads();
    for (int k = k0; k < k1; ++k) {
        const bool more = k + 1 < k1;
        if (more) fetch_plane(k + 1);
        const unsigned int c = (unsigned int)k * plane + col;
        R own[4], ub[4], zw[4];
        load_raw(c, own);
        if constexpr (STAGE == 2) {
#pragma unroll
            for (int v = 0; v < 4; ++v) ub[v] = ld(b[v], c);
        }
        prim_of<GAS>(pc, zraw, zw);
        if (more) load_raw((unsigned int)wrap_any(k + 2, g.nz) * plane + col, zraw);
        R acc[4], L[4], C[4], Rr[4], fl[4], fh[4];
        const R(&w)[4][LY][LX] = sw[k & 1];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            L[v] = w[v][row + 1][lane];
            C[v] = w[v][row + 1][lane + 1];
            Rr[v] = w[v][row + 1][lane + 2];
        }
        face_flux<0, GAS>(pc.cs, L, C, fl);
        face_flux<0, GAS>(pc.cs, C, Rr, fh);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            acc[v] = fh[v] - fl[v];
            L[v] = w[v][row][lane + 1];
            Rr[v] = w[v][row + 2][lane + 1];
        }
        face_flux<1, GAS>(pc.cs, L, C, fl);
        face_flux<1, GAS>(pc.cs, C, Rr, fh);
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = fma_r(acc[v], pc.idx[0], (fh[v] - fl[v]) * pc.idx[1]);
        face_flux<2, GAS>(pc.cs, zb, zw, fh);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            acc[v] = fma_r(fh[v] - fz[v], pc.idx[2], acc[v]);
            fz[v] = fh[v];
            zb[v] = zw[v];
        }
        if (live) stage_store<STAGE, GAS>(pc, own, ub, acc, o, c);
        if (more) store_plane((k + 1) & 1);
        __syncthreads();
    }
}

template <int STAGE, class R>
__global__ __launch_bounds__(DTX* DTY) void k_donor_pass(Geo g, DustParams p, PassArgs<R> a, int kz, unsigned int ntx,
                                                         unsigned int nty, unsigned int ntiles, unsigned int nblk)
{
    __shared__ R sw[2][4][DTY + 2][DTX + 2];  // primitives of plane k, and of k + 1 being staged
    const unsigned int item = xcd_item(blockIdx.x, nblk);
    const int s = (int)(item / ntiles);  // fluid: 0 gas, 1.. dust
    const unsigned int t = item - (unsigned int)s * ntiles;
    const int x0 = (int)(t % ntx) * DTX, y0 = (int)((t / ntx) % nty) * DTY, k0 = (int)(t / (ntx * nty)) * kz;
    const int k1 = min(k0 + kz, g.nz);
    if (s == 0)
        donor_block<STAGE, R, true>(g, p, a, s, x0, y0, k0, k1, sw);
    else
        donor_block<STAGE, R, false>(g, p, a, s, x0, y0, k0, k1, sw);
}

// ----------------------------------------------------------------------------------
// drag solve (and the CFL step after stage 2), pointwise
// ----------------------------------------------------------------------------------

// Constants of one drag solve S_h, computed on the host per launch (h = lam dt):
// w_k = h/(t_k + h), a_k = t_k/(t_k + h) and 1/t_k, so that no cell divides by them.
struct DragCoef {
    double w[kMaxDust], a[kMaxDust], its[kMaxDust];
    double h, cg;  // cg: weight of the stage-1 drag rates (stage 2)
};

static DragCoef drag_coef(const DustParams& p, double h, double cg)
{
    DragCoef q{};
    for (int s = 0; s < p.nd; ++s) {
        q.w[s] = h / (p.ts[s] + h);
        q.a[s] = p.ts[s] / (p.ts[s] + h);
        q.its[s] = 1.0 / p.ts[s];
    }
    q.h = h;
    q.cg = cg;
    return q;
}

// Closed-form drag solve of one momentum component, in place on mom[0..ND]:
// v_g' = (p_g + sum w_k p_k)/(rho_g + sum w_k rho_k), p_k' = a_k p_k + w_k rho_k v_g'.
template <int ND>
__device__ __forceinline__ void drag_solve(const DragCoef& q, const double* rho, double* mom)
{
    double num = mom[0], den = rho[0];
#pragma unroll
    for (int s = 1; s <= ND; ++s) {
        num += q.w[s - 1] * mom[s];
        den += q.w[s - 1] * rho[s];
    }
    const double vg = num / den;
#pragma unroll
    for (int s = 1; s <= ND; ++s) mom[s] = q.a[s - 1] * mom[s] + q.w[s - 1] * (rho[s] * vg);
    mom[0] = rho[0] * vg;
}

// Reciprocal density of fluid s for its velocity: the gas density floored; a dust
// species below its floor is at rest (0).
__device__ __forceinline__ double inv_density(const DustParams& p, int s, double d)
{
    const double f = s == 0 ? p.rho_floor : p.dust_floor;
    const double iv = 1.0 / (d < f ? f : d);
    return s > 0 && d < f ? 0.0 : iv;
}

// NaN-propagating maximum of non-negative speeds
__device__ __forceinline__ double max_nan(double a, double b)
{
    const double m = a > b ? a : b;
    return (a != a) || (b != b) ? a + b : m;
}

__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min_nan(v, __shfl_xor(v, off, 64));
    return v;
}

// X: the explicit part (densities final); U1: stage-1 state (stage 2 only).  The number
// of dust species ND is a template parameter so the per-cell vectors live in registers.
// Loads are of the stored type R; the solve is FP64.
template <int STAGE, int ND, class R>
__global__ __launch_bounds__(kBlock) void k_drag(Geo g, DustParams p, DragCoef q, R* __restrict__ X,
                                                 const R* __restrict__ U1, double* __restrict__ partial)
{
    const long long cl = (long long)blockIdx.x * kBlock + threadIdx.x;
    const long long n = g.n;
    double r = INFINITY;
    if (cl < n) {
        const unsigned int c = (unsigned int)cl;
        double rho[ND + 1], r1[ND + 1], ivn[ND + 1], ivg1 = 0.0;
#pragma unroll
        for (int s = 0; s <= ND; ++s) rho[s] = (double)ld(X + 4LL * s * n, c);
        if constexpr (STAGE == 2) {
#pragma unroll
            for (int s = 0; s <= ND; ++s) {
                r1[s] = (double)ld(U1 + 4LL * s * n, c);
                ivn[s] = inv_density(p, s, rho[s]);
            }
            ivg1 = inv_density(p, 0, r1[0]);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double mom[ND + 1];
#pragma unroll
            for (int s = 0; s <= ND; ++s) mom[s] = (double)ld(X + (4LL * s + 1 + a) * n, c);
            if constexpr (STAGE == 2) {
                // + (1 - lam - delta) dt G(U1): drag rates of the stage-1 state in their
                // momentum form (rho_k v_g - p_k)/t_k, the map the stage-1 solve inverted
                const double vg = (double)ld(U1 + (1LL + a) * n, c) * ivg1;
                double gsum = 0.0;
#pragma unroll
                for (int s = 1; s <= ND; ++s) {
                    const double pk = (double)ld(U1 + (4LL * s + 1 + a) * n, c);
                    const double fk = (r1[s] * vg - pk) * q.its[s - 1];
                    mom[s] = mom[s] + q.cg * fk;
                    gsum -= fk;
                }
                mom[0] = mom[0] + q.cg * gsum;
            }
            drag_solve<ND>(q, rho, mom);
#pragma unroll
            for (int s = 0; s <= ND; ++s) {
                st(X + (4LL * s + 1 + a) * n, c, (R)mom[s]);
                mom[s] = (double)(R)mom[s];  // the CFL step sees the stored state
            }
            if constexpr (STAGE == 2) {
                // time step of the new state, as the standalone CFL kernel takes it:
                // min_s dx/(|v_s| + c_s) = dx / max_s(|v_s| + c_s) (division is monotone)
                double sp = fabs(mom[0] * ivn[0]) + p.cs;
#pragma unroll
                for (int s = 1; s <= ND; ++s) sp = max_nan(sp, fabs(mom[s] * ivn[s]));
                r = min_nan(r, g.dx[a] / sp);
            }
        }
    }
    if constexpr (STAGE == 2) {
        __shared__ double sm[kBlock / 64];
        r = wave_min(r);
        if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = r;
        __syncthreads();
        if (threadIdx.x == 0) {
            double m = sm[0];
#pragma unroll
            for (int w = 1; w < kBlock / 64; ++w) m = min_nan(m, sm[w]);
            partial[blockIdx.x] = m;
        }
    }
}

template <int STAGE, int ND, class R>
static void drag_launch(const Geo& g, const DustParams& p, const DragCoef& q, R* X, const R* U1,
                        double* partial, hipStream_t s)
{
    hipLaunchKernelGGL((k_drag<STAGE, ND, R>), dim3(blocks_for(g.n)), dim3(kBlock), 0, s, g, p, q, X, U1,
                       partial);
}

// Dispatch on the species count (1..kMaxDust) to the specialised kernel.
template <int STAGE, class R, int ND = 1>
static hipError_t drag_dispatch(const Geo& g, const DustParams& p, const DragCoef& q, R* X, const R* U1,
                                double* partial, hipStream_t s)
{
    if constexpr (ND > kMaxDust) {
        return hipErrorInvalidValue;
    } else {
        if (p.nd == ND) {
            drag_launch<STAGE, ND, R>(g, p, q, X, U1, partial, s);
            return hipGetLastError();
        }
        return drag_dispatch<STAGE, R, ND + 1>(g, p, q, X, U1, partial, s);
    }
}

// ----------------------------------------------------------------------------------

// Tile and planes per chunk.  Two rows share their y faces and halo rows, and a chunk primes
// its z pipeline once, but a small grid needs the waves: two rows where chunks of four planes
// still give 2048 waves (PLM: a round of what the GPU holds at two per SIMD; 48^3 with 8
// species FP64 135 -> 124 us a step, FP32 77 -> 72) or 4096 (FP32 donor cell), beyond about
// 16384 waves, whose last round costs little (192^3 with 8 by waves 8192 / 16384 / 32768: 1722
// / 1670 / 1700 us a stage).  Else one row and the chunk of 2 to 8 planes that takes the
// fewest plane times in rounds of 4096 waves, a chunk costing about 1.5 planes beside its own
// (two rounds of 2048: with one as the unit 70 grids of up to 4e6 cells x fluids take as long
// in FP64 and 1 % longer in FP32).  FP64 stage 1, us, one row and 2 planes / two rows and 4 at
// least: 24^3 with 2 species 13 / 25, 40^3 with 4 29 / 28, 64^3 with 8 89 / 80.
// The donor cell in FP64 has one row a wave, in chunks of four planes beyond 8192 waves (64^3
// with 16 species 284 -> 274 us a step, 256 x 256 x 4 with 8 163 -> 152), up to where two
// would give 12288 waves, and from there blocks of four, about 4096 of them.
// A single row whose waves all run at once (two per SIMD) is solo: 4096 x 1 x 1 with 2 species
// FP64 7.7 -> 7.0 us a stage; with more waves its registers cost more (48 x 30 x 102 with 1
// 57.9 -> 58.8 us a step).
DustGrid dust_grid(const Geo& g, int nfluids, int recon, bool fp32)
{
    DustGrid d;
    d.ntx = (unsigned int)((g.nx + DTX - 1) / DTX);
    const long long cols = (long long)d.ntx * nfluids;
    const bool donor = recon == 0 && !fp32;
    const long long pairs = cols * ((g.ny + 1) / 2) * ((g.nz + 3) / 4);
    const bool many = pairs >= (recon != 0 ? 2048 : fp32 ? 4096 : 12288);
    d.block = many && donor;
    d.rows = d.block ? DTY : many ? 2 : 1;
    d.nty = (unsigned int)((g.ny + d.rows - 1) / d.rows);
    const long long tiles = cols * d.nty;
    auto chunks = [&](int q) { return (long long)(g.nz + q - 1) / q; };
    int kz = 4;
    if (many) {
        const long long want = ((d.block ? 4096 : 16384) + tiles - 1) / tiles;
        const int least = d.block ? 8 : 4;
        kz = (int)((g.nz + want - 1) / want);
        if (kz < least) kz = least;
    } else if (!donor || tiles * chunks(4) <= 8192) {
        long long best = -1;
        for (int q = 2; q <= 8; ++q) {
            const long long cost = (tiles * chunks(q) + 4095) / 4096 * (2 * q + 3);
            if (best < 0 || cost < best) {
                best = cost;
                kz = q;
            }
        }
    }
    if (kz > g.nz) kz = g.nz;
    d.kz = kz;
    d.ntz = (unsigned int)((g.nz + kz - 1) / kz);
    d.ntiles = d.ntx * d.nty * d.ntz;
    d.nitems = d.ntiles * (unsigned int)nfluids;
    d.solo = d.rows == 1 && d.nitems <= 2048;
    d.nblk = d.block ? d.nitems : (d.nitems + DWAVES - 1) / DWAVES;
    return d;
}

template <int RECON, class R, int NR, bool SOLO>
static hipError_t pass_rows(const Geo& g, const DustParams& p, const DustGrid& d, int stage, const PassArgs<R>& a,
                            hipStream_t s)
{
    const dim3 gr(d.nblk), bl(64 * DWAVES);
    if (stage == 1)
        hipLaunchKernelGGL((k_fluid_pass<RECON, 1, R, NR, SOLO>), gr, bl, 0, s, g, p, a, d.kz, d.ntx, d.nty, d.ntiles,
                           d.nitems, d.nblk);
    else
        hipLaunchKernelGGL((k_fluid_pass<RECON, 2, R, NR, SOLO>), gr, bl, 0, s, g, p, a, d.kz, d.ntx, d.nty, d.ntiles,
                           d.nitems, d.nblk);
    return hipGetLastError();
}

template <int RECON, class R>
static hipError_t pass(const Geo& g, const DustParams& p, const DustGrid& d, int stage, const PassArgs<R>& a,
                       hipStream_t s)
{
    if constexpr (RECON == 0 && sizeof(R) == 8) {
        if (d.block) {
            const dim3 gr(d.nblk), bl(DTX * DTY);
            if (stage == 1)
                hipLaunchKernelGGL((k_donor_pass<1, R>), gr, bl, 0, s, g, p, a, d.kz, d.ntx, d.nty, d.ntiles, d.nblk);
            else
                hipLaunchKernelGGL((k_donor_pass<2, R>), gr, bl, 0, s, g, p, a, d.kz, d.ntx, d.nty, d.ntiles, d.nblk);
            return hipGetLastError();
        }
    } else if (d.rows == 2) {
        return pass_rows<RECON, R, 2, false>(g, p, d, stage, a, s);
    }
    if (d.solo) return pass_rows<RECON, R, 1, true>(g, p, d, stage, a, s);
    return pass_rows<RECON, R, 1, false>(g, p, d, stage, a, s);
}

template <class R>
static hipError_t pass1(const Geo& g, const DustParams& p, const DustGrid& d, int recon, const void* u, void* U1,
                        double dt, hipStream_t s)
{
    PassArgs<R> a{(const R*)u, nullptr, (R*)U1, kLam * dt, 0.0, 0.0};
    return recon == 0 ? pass<0, R>(g, p, d, 1, a, s) : pass<1, R>(g, p, d, 1, a, s);
}

template <class R>
static hipError_t pass2(const Geo& g, const DustParams& p, const DustGrid& d, int recon, void* u, const void* U1,
                        double dt, hipStream_t s)
{
    PassArgs<R> a{(const R*)U1, (const R*)u, (R*)u, (1.0 - kDelta) * dt, 1.0 - kDelta / kLam, kDelta / kLam};
    return recon == 0 ? pass<0, R>(g, p, d, 2, a, s) : pass<1, R>(g, p, d, 2, a, s);
}

hipError_t launch_fluid_pass1(const Geo& g, const DustParams& p, const DustGrid& d, bool fp32, int recon,
                              const void* u, void* U1, double dt, hipStream_t s)
{
    return fp32 ? pass1<float>(g, p, d, recon, u, U1, dt, s) : pass1<double>(g, p, d, recon, u, U1, dt, s);
}

hipError_t launch_fluid_pass2(const Geo& g, const DustParams& p, const DustGrid& d, bool fp32, int recon,
                              void* u, const void* U1, double dt, hipStream_t s)
{
    return fp32 ? pass2<float>(g, p, d, recon, u, U1, dt, s) : pass2<double>(g, p, d, recon, u, U1, dt, s);
}

hipError_t launch_drag1(const Geo& g, const DustParams& p, bool fp32, void* U1, double dt, hipStream_t s)
{
    const DragCoef q = drag_coef(p, kLam * dt, 0.0);
    if (fp32) return drag_dispatch<1, float>(g, p, q, (float*)U1, nullptr, nullptr, s);
    return drag_dispatch<1, double>(g, p, q, (double*)U1, nullptr, nullptr, s);
}

hipError_t launch_drag2_cfl(const Geo& g, const DustParams& p, bool fp32, void* u, const void* U1, double dt,
                            double* partial, double* dt_out, double cfl_scale, hipStream_t s)
{
    const DragCoef q = drag_coef(p, kLam * dt, (1.0 - kLam - kDelta) * dt);
    hipError_t e = fp32 ? drag_dispatch<2, float>(g, p, q, (float*)u, (const float*)U1, partial, s)
                        : drag_dispatch<2, double>(g, p, q, (double*)u, (const double*)U1, partial, s);
    if (e != hipSuccess) return e;
    return launch_min_final(partial, blocks_for(g.n), cfl_scale, dt_out, s);
}

// FP32 dust register <-> canonical FP64 state (nv fields)
__global__ __launch_bounds__(kBlock) void k_dust_pack(long long m, const double* __restrict__ canon,
                                                      float* __restrict__ reg)
{
    const long long q = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (q < m) reg[q] = (float)canon[q];
}
__global__ __launch_bounds__(kBlock) void k_dust_unpack(long long m, const float* __restrict__ reg,
                                                        double* __restrict__ canon)
{
    const long long q = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (q < m) canon[q] = reg[q];
}

hipError_t launch_dust_pack(long long m, const double* canon, void* reg, hipStream_t s)
{
    hipLaunchKernelGGL(k_dust_pack, dim3(blocks_for(m)), dim3(kBlock), 0, s, m, canon, (float*)reg);
    return hipGetLastError();
}

hipError_t launch_dust_unpack(long long m, const void* reg, double* canon, hipStream_t s)
{
    hipLaunchKernelGGL(k_dust_unpack, dim3(blocks_for(m)), dim3(kBlock), 0, s, m, (const float*)reg, canon);
    return hipGetLastError();
}

}  // namespace mhd
