// lhmm_sph.hip -- gfx950 kernels and runtime of the SPH macro side and of the
// coupled exchange interval (include/lhmm.h, lhmm_sph_* and
// lhmm_couple_step).
//
// The macro problem is small (10^3-10^4 particles) and double precision, so a
// step is bound by launches and by chains of dependent loads: few launches,
// every one over the whole chip.  Each particle I is summed by one wave; lane
// l takes candidates l, l + 64, ... of a fixed enumeration (the particles of
// the 3 x 3 cells of side >= h around I, cell by cell and by index inside a
// cell; every particle when the periodic box holds fewer than 3 cells per
// side) with the minimum image of the periodic box, and a fixed shuffle tree
// adds the 64 partial sums, so every sum has a fixed order.  A step is
//   k_tile -> k_force(drift) -> k_tile -> k_force(kick) -> k_gradient
// (velocity-Verlet, then the micro-domain gradients at the new state): k_tile
// sorts the particles into the cells and sums the densities, k_force sums the
// accelerations and moves the particles.  Without cells it is
//   k_density -> k_accel -> k_kick_drift -> k_density -> k_accel -> k_kick
//   -> k_gradL.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "lhmm.h"
#include "lhmm_internal.h"
#include "lhmm_grid.h"
#include "lhmm_stage.h"

namespace {

constexpr int TPB = 256;             // threads per block
constexpr int WPB = TPB / 64;        // particles (waves) per block

// Sum over the wave, the same in every lane: lanes 32, 16, 8, 4, 2, 1 apart in
// turn, in registers (six steps through ds_bpermute are 0.3 us of a chain
// that nothing else of the wave overlaps).
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_sum(double x) {
    auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
    auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
    x = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
    hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
    x = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    x += dpp<0x128>(x);  // rotate by 8 in rows of 16
    x += dpp<0x124>(x);  // by 4
    x += dpp<0x4E>(x);   // quads: 2, 3, 0, 1
    x += dpp<0xB1>(x);   // quads: 1, 0, 3, 2
    return x;
}

__device__ __forceinline__ double pow4(double x) {
    const double x2 = x * x;
    return x2 * x2;
}

struct SphCtx {
    int n, n_mobile, force_mode;  // particles n_mobile .. n-1 are frozen walls
    int kernel;                   // LHMM_KERNEL_QUINTIC or LHMM_KERNEL_LUCY
    int micro_dim;                // 3: micro-domains are 3-D boxes; 2: planar cells (no zz stress)
    int ncx, ncy;                 // cell columns and cells of a column (0: all pairs)
    int turned;                   // columns run along x instead of y
    int rows, tiles;              // cells of a column per tile, tiles per column (k_tile)
    int* cstart;                  // ncx * ncy + 1 cell offsets
    unsigned* key;                // each particle's cell, column << 16 | row
    // in cell order: particle indices, cells, positions, velocities, 1 / d of
    // the density d, and over d^2 the pressure p and the polymer stress (xx,
    // xy, yy; 0 for walls): what a neighbour brings to a force sum
    int* cidx;
    unsigned* cell;
    double2 *rs, *vs;
    double *ids, *p2s;
    double *s2s;  // x 3
    double qs, cW, cF;            // kernel constants (see kernel_W)
    double rho0, eta, zeta, c, theta, F, h, dt, mass, Lx, Ly, lambda_star, alpha;
    double* r;    // n x 2
    double* v;    // n x 2
    double* d;    // n
    double* p;    // n
    double* acc;  // n x 2
};

// The kernels take q = |dr| / h, resp. 3 |dr| / h, times S.qs (1 / h, 3 / h),
// and their constant factors from S.cW and S.cF; divisions by a constant are
// products with its reciprocal.

// quintic kernel of support radius h: W = cW w(q), cW = 63 / (478 pi h^2),
// F = -W'(r) / r = cF f(q) / r, cF = 3 cW / h
__device__ __forceinline__ double quintic_w(double q) {
    const double a = 3.0 - q, b = fmax(2.0 - q, 0.0), c = fmax(1.0 - q, 0.0);
    const double w = pow4(a) * a - 6.0 * (pow4(b) * b) + 15.0 * (pow4(c) * c);
    return q >= 3.0 ? 0.0 : w;
}

__device__ __forceinline__ double quintic_f(double q) {
    const double f = 5.0 * pow4(3.0 - q) - 30.0 * pow4(fmax(2.0 - q, 0.0)) + 75.0 * pow4(fmax(1.0 - q, 0.0));
    return q >= 3.0 ? 0.0 : f;
}

// 2-D Lucy kernel, Eq. (lucy_kernel): W = 5/(pi h^2) (1 + 3q)(1 - q)^3, whose
// F reduces to 60 (1 - q)^2 / (pi h^4)
__device__ __forceinline__ double lucy_w(double q) {
    const double u = 1.0 - q;
    return q >= 1.0 ? 0.0 : (1.0 + 3.0 * q) * (u * u * u);
}

__device__ __forceinline__ double lucy_f(double q) {
    const double u = 1.0 - q;
    return q >= 1.0 ? 0.0 : u * u;
}

// The kernel choice is one value per engine, so the branch is uniform.
// W at squared distance r2
__device__ __forceinline__ double kernel_W(const SphCtx& S, double r2) {
    const double q = r2 > 0.0 ? r2 * rsqrt(r2) * S.qs : r2;  // r2: 0, or NaN
    return S.cW * (S.kernel == LHMM_KERNEL_LUCY ? lucy_w(q) : quintic_w(q));
}

// F at distance rr = 1 / ir
__device__ __forceinline__ double kernel_F(const SphCtx& S, double rr, double ir) {
    const double q = rr * S.qs;
    return S.kernel == LHMM_KERNEL_LUCY ? S.cF * lucy_f(q) : S.cF * quintic_f(q) * ir;
}

// Positions lie in [0, L), so the nearest image is at most one box away (a
// separation of half a box is beyond every kernel's support: L > 2 h).
__device__ __forceinline__ double min_image(double dx, double L) {
    return dx > 0.5 * L ? dx - L : (dx < -0.5 * L ? dx + L : dx);
}
__device__ __forceinline__ void min_image(const SphCtx& S, double& dx, double& dy) {
    dx = min_image(dx, S.Lx);
    dy = min_image(dy, S.Ly);
}

__device__ __forceinline__ int cell_along(double x, int n, double L) {
    return min(max((int)(x * (double)n / L), 0), n - 1);
}
__device__ __forceinline__ unsigned cell_key(const SphCtx& S, double x, double y) {
    const unsigned ix = (unsigned)cell_along(x, S.turned ? S.ncy : S.ncx, S.Lx);
    const unsigned iy = (unsigned)cell_along(y, S.turned ? S.ncx : S.ncy, S.Ly);
    return S.turned ? (iy << 16) | ix : (ix << 16) | iy;
}

// Tait pressure of the number density d, with the background pressure
__device__ __forceinline__ double pressure(const SphCtx& S, double d) {
    const double B = S.c * S.c * S.rho0 / 7.0;
    const double x = S.mass * d / S.rho0, x2 = x * x;
    return B * (x2 * x2 * x2 * x - 1.0) + S.theta * B;
}

// All pairs: one wave per particle.
__global__ __launch_bounds__(TPB) void k_density(SphCtx S) {
    const int I = blockIdx.x * WPB + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (I >= S.n) return;  // wave-uniform
    const double xi = S.r[2 * I], yi = S.r[2 * I + 1];
    double s = 0.0;
    for (int J = lane; J < S.n; J += 64) {
        double dx = xi - S.r[2 * J], dy = yi - S.r[2 * J + 1];
        min_image(S, dx, dy);
        s += kernel_W(S, dx * dx + dy * dy);
    }
    s = wave_sum(s);
    if (lane == 0) {
        S.d[I] = s;
        S.p[I] = pressure(S, s);
    }
}

// polymer stress of particle I: alpha/lambda* x in-plane part of the
// deviatoric part of its micro-domain's mean stress (xx, yy, zz, xy, xz,
// yz).  A 3-D micro-domain loses its isotropic part tr/3; a planar one has
// no zz stress (its particles and forces lie in the plane), so its
// deviatoric part is taken in the plane, (xx + yy)/2 off the diagonal.
__device__ __forceinline__ void polymer_stress(const SphCtx& S, const double* sigma, int I, double& xx, double& xy,
                                               double& yy) {
    if (!sigma) {
        xx = xy = yy = 0.0;
        return;
    }
    const double* g = sigma + 6 * I;
    const double s = S.alpha / S.lambda_star;
    const double iso = S.micro_dim == 2 ? 0.5 * (g[0] + g[1]) : (g[0] + g[1] + g[2]) / 3.0;
    xx = s * (g[0] - iso);
    xy = s * g[3];
    yy = s * (g[1] - iso);
}

__device__ __forceinline__ double body_force(const SphCtx& S, double y) {
    return (S.force_mode == LHMM_FORCE_UNIFORM || y >= 0.5 * S.Ly) ? S.F : -S.F;
}

// What a particle brings to a force sum: position, velocity, 1 / d, pressure
// and polymer stress over d^2.
struct ForceRec {
    double2 r, v;
    double id, p2, xx, xy, yy;
};

// Pressure, viscous and polymer terms of Eq. (sph_continuity) on particle i
// from particle j, added to (fx, fy): one rsqrt and no division per pair (the
// formula as written has six divisions, 66 of 250 instructions).
__device__ __forceinline__ void add_force(const SphCtx& S, const ForceRec& i, const ForceRec& j, double av, double bv,
                                          double& fx, double& fy) {
    double dx = i.r.x - j.r.x, dy = i.r.y - j.r.y;
    min_image(S, dx, dy);
    const double r2 = dx * dx + dy * dy;
    if (r2 >= S.h * S.h || r2 == 0.0) return;
    const double ir = rsqrt(r2), F = kernel_F(S, r2 * ir, ir);
    const double ex = dx * ir, ey = dy * ir;
    const double ux = i.v.x - j.v.x, uy = i.v.y - j.v.y;
    const double pp = i.p2 + j.p2, ve = bv * (ux * ex + uy * ey), idd = i.id * j.id;
    const double sxx = i.xx + j.xx, sxy = i.xy + j.xy, syy = i.yy + j.yy;
    fx += F * (pp * dx - (av * ux + ve * ex) * idd - (sxx * dx + sxy * dy));
    fy += F * (pp * dy - (av * uy + ve * ey) * idd - (sxy * dx + syy * dy));
}

// velocity gradient sum of particle i: F/dj (ri - rj) (vi - vj)
__device__ __forceinline__ void add_gradient(const SphCtx& S, double2 ri, double2 rj, double2 vi, double2 vj,
                                             double idj, double (&g)[4]) {
    double dx = ri.x - rj.x, dy = ri.y - rj.y;
    min_image(S, dx, dy);
    const double r2 = dx * dx + dy * dy;
    if (r2 >= S.h * S.h || r2 == 0.0) return;
    const double ir = rsqrt(r2), F = kernel_F(S, r2 * ir, ir) * idj;
    const double ux = vi.x - vj.x, uy = vi.y - vj.y;
    dx *= F;
    dy *= F;
    g[0] += dx * ux;
    g[1] += dx * uy;
    g[2] += dy * ux;
    g[3] += dy * uy;
}

// record of particle J (index order), its position and velocity given
__device__ __forceinline__ ForceRec force_rec(const SphCtx& S, const double* sigma, int J, double2 r, double2 v,
                                              double d, double p) {
    ForceRec q;
    q.r = r;
    q.v = v;
    q.id = 1.0 / d;
    const double i2 = q.id * q.id;
    q.p2 = p * i2;
    q.xx = q.xy = q.yy = 0.0;
    if (J < S.n_mobile) polymer_stress(S, sigma, J, q.xx, q.xy, q.yy);
    q.xx *= i2;
    q.xy *= i2;
    q.yy *= i2;
    return q;
}

__device__ __forceinline__ double2 position(const SphCtx& S, int J) { return make_double2(S.r[2 * J], S.r[2 * J + 1]); }
__device__ __forceinline__ double2 velocity(const SphCtx& S, int J) { return make_double2(S.v[2 * J], S.v[2 * J + 1]); }

// Eq. (sph_continuity) divided by the mass, plus the body force
__global__ __launch_bounds__(TPB) void k_accel(SphCtx S, const double* __restrict__ sigma) {
    const int I = blockIdx.x * WPB + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (I >= S.n_mobile) return;  // wave-uniform
    const double av = 2.0 * S.eta - S.zeta, bv = 4.0 * S.zeta + 2.0 * S.eta;
    const ForceRec i = force_rec(S, sigma, I, position(S, I), velocity(S, I), S.d[I], S.p[I]);
    double fx = 0.0, fy = 0.0;
    for (int J = lane; J < S.n; J += 64)
        if (J != I)
            add_force(S, i, force_rec(S, sigma, J, position(S, J), velocity(S, J), S.d[J], S.p[J]), av, bv, fx, fy);
    fx = wave_sum(fx);
    fy = wave_sum(fy);
    if (lane == 0) {
        S.acc[2 * I] = fx / S.mass + body_force(S, i.r.y);
        S.acc[2 * I + 1] = fy / S.mass;
    }
}

__device__ __forceinline__ double wrap_len(double x, double L) {
    x -= L * floor(x / L);
    return x >= L ? 0.0 : x;
}

__global__ void k_kick_drift(SphCtx S) {
    const int I = blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= S.n_mobile) return;
    const double hdt = 0.5 * S.dt;
    const double vx = S.v[2 * I] + hdt * S.acc[2 * I], vy = S.v[2 * I + 1] + hdt * S.acc[2 * I + 1];
    S.v[2 * I] = vx;
    S.v[2 * I + 1] = vy;
    S.r[2 * I] = wrap_len(S.r[2 * I] + S.dt * vx, S.Lx);
    S.r[2 * I + 1] = wrap_len(S.r[2 * I + 1] + S.dt * vy, S.Ly);
}

__global__ void k_kick(SphCtx S) {
    const int I = blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= S.n_mobile) return;
    const double hdt = 0.5 * S.dt;
    S.v[2 * I] += hdt * S.acc[2 * I];
    S.v[2 * I + 1] += hdt * S.acc[2 * I + 1];
}

// Eq. (macro_micro) with 1/d_J: G_ab = d_a v_b; micro gradient
// L = lambda* x traceless part of G^T (u = L r), 3x3 row-major, zero z.
__device__ __forceinline__ void store_gradient(const SphCtx& S, double (&g)[4], int lane, double* o) {
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k] = wave_sum(g[k]);
    if (lane > 0) return;
    const double half_tr = 0.5 * (g[0] + g[3]);
    o[0] = S.lambda_star * (g[0] - half_tr);
    o[1] = S.lambda_star * g[2];
    o[2] = 0.0;
    o[3] = S.lambda_star * g[1];
    o[4] = S.lambda_star * (g[3] - half_tr);
    o[5] = 0.0;
    o[6] = 0.0;
    o[7] = 0.0;
    o[8] = 0.0;
}

__global__ __launch_bounds__(TPB) void k_gradL(SphCtx S, double* __restrict__ gradL) {
    const int I = blockIdx.x * WPB + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (I >= S.n) return;  // wave-uniform
    if (I >= S.n_mobile) {
        if (lane < 9) gradL[9 * I + lane] = 0.0;
        return;
    }
    const double2 ri = position(S, I), vi = velocity(S, I);
    double g[4] = {};
    for (int J = lane; J < S.n; J += 64)
        if (J != I) add_gradient(S, ri, position(S, J), vi, velocity(S, J), 1.0 / S.d[J], g);
    store_gradient(S, g, lane, gradL + 9 * I);
}

// With cells: one workgroup per tile of `rows` cells of a column (cell_tiles:
// about as many as the chip has CUs).  Every workgroup reads all particles'
// cells (4 bytes each), counting those before its tile and collecting those in
// the 3 x (rows + 2) cells around it, so it needs nothing from another one.
// It sorts what it collected by cell and index and sums the densities of its
// own particles, a wave per particle, from LDS; then writes their records in
// cell order.  It is bound by its chain of loads and barriers: 8.7 us for 4096
// particles, where a one-workgroup sort (12.5 us) and a density launch that
// waited for it (13 us) came before.  Steps on the way: positions loaded one
// by one as they are collected 10.4 us, the records written by each density
// wave 10.4 us, sums through ds_bpermute in place of wave_sum's 9.5 us.
constexpr int TILE_THREADS = 1024;
constexpr int TILE_POSITIONS = 512;  // collected positions, own densities held in LDS; beyond, read again

// dynamic LDS of k_tile: the collected particles grouped by cell (index << 16
// | slot, 4 bytes; all n at most), each slot's particle and the slots in cell
// order (2 bytes each), each slot's cell (1 byte)
constexpr int TILE_LDS = 9;  // per particle

__global__ __launch_bounds__(TILE_THREADS) void k_tile(SphCtx S, const double* __restrict__ sigma) {
    extern __shared__ unsigned grouped[];
    unsigned short *ent = (unsigned short*)(grouped + S.n), *list = ent + S.n;
    unsigned char* cell = (unsigned char*)(list + S.n);
    __shared__ double2 pos[TILE_POSITIONS];
    __shared__ double dens[TILE_POSITIONS];  // own particles' densities
    __shared__ int cnt[TILE_CELLS], start[TILE_CELLS + 1], before_sh, total_sh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int ax = blockIdx.y, ay = blockIdx.x * S.rows;
    const int rows = min(S.rows, S.ncy - ay), hy = rows + 2, ncell = 3 * hy;
    const unsigned first = ((unsigned)ax << 16) | (unsigned)ay;
    if (tid < TILE_CELLS) cnt[tid] = 0;
    if (tid == 0) before_sh = total_sh = 0;
    __syncthreads();
    int before = 0;
    for (int I0 = tid; I0 - tid < S.n; I0 += 4 * TILE_THREADS) {  // four keys in flight
        unsigned key[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) key[u] = S.key[min(I0 + u * TILE_THREADS, S.n - 1)];
        unsigned long long hit[4];
        int c[4], hits = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool on = I0 + u * TILE_THREADS < S.n;
            before += __popcll(__ballot(on && key[u] < first));
            // the particle's cell around the tile: column ax - 1 + lx, row ay - 1 + ly
            int lx = (int)(key[u] >> 16) - ax + 1, ly = (int)(key[u] & 0xFFFFu) - ay + 1;
            lx += lx < 0 ? S.ncx : (lx >= S.ncx ? -S.ncx : 0);
            ly += ly < 0 ? S.ncy : (ly >= S.ncy ? -S.ncy : 0);
            c[u] = on && lx < 3 && ly < hy ? lx * hy + ly : -1;
            hit[u] = __ballot(c[u] >= 0);
            hits += __popcll(hit[u]);
        }
        if (hits == 0) continue;  // wave-uniform
        int e0 = 0;
        if (lane == 0) e0 = atomicAdd(&total_sh, hits);
        e0 = __builtin_amdgcn_readfirstlane(e0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (c[u] >= 0) {
                const int e = e0 + __popcll(hit[u] & ((1ull << lane) - 1));
                atomicAdd(&cnt[c[u]], 1);
                ent[e] = (unsigned short)(I0 + u * TILE_THREADS);
                cell[e] = (unsigned char)c[u];
            }
            e0 += __popcll(hit[u]);
        }
    }
    if (lane == 0 && before) atomicAdd(&before_sh, before);
    __syncthreads();
    const int total = total_sh;
    double2 mine;  // on its way while wave 0 scans
    if (tid < min(total, TILE_POSITIONS)) mine = position(S, ent[tid]);
    if (tid < 64) {  // exclusive scan over at most 64 cells
        const int v = tid < ncell ? cnt[tid] : 0;
        int x = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        start[tid] = x - v;
        cnt[tid] = x - v;
        if (tid == 63) start[64] = x;
    }
    __syncthreads();
    for (int e = tid; e < total; e += TILE_THREADS)
        grouped[atomicAdd(&cnt[cell[e]], 1)] = ((unsigned)ent[e] << 16) | (unsigned)e;
    __syncthreads();
    for (int k = tid; k < total; k += TILE_THREADS) {  // by index inside each cell
        const unsigned x = grouped[k];
        const int c = cell[x & 0xFFFFu], q0 = start[c], q1 = start[c + 1];
        int to = q0;
        for (int q = q0; q < q1; ++q) to += grouped[q] < x ? 1 : 0;
        list[to] = (unsigned short)x;
    }
    if (tid < min(total, TILE_POSITIONS)) pos[tid] = mine;
    __syncthreads();
    auto slot_position = [&](int e) { return e < TILE_POSITIONS ? pos[e] : position(S, ent[e]); };
    // the tile's own cells are one run of the list, and of the cell order
    const int own0 = start[hy + 1], own1 = start[hy + 1 + rows], g0 = before_sh - own0;
    for (int k = tid; k < rows; k += TILE_THREADS) S.cstart[ax * S.ncy + ay + k] = g0 + start[hy + 1 + k];
    if (tid == 0 && ax == 0 && ay == 0) S.cstart[S.ncx * S.ncy] = S.n;
    // velocity and stress of the thread's first own particle, on their way
    // while the densities are summed
    double2 vi;
    double xx = 0.0, xy = 0.0, yy = 0.0;
    auto load = [&](int I) {
        vi = velocity(S, I);
        xx = xy = yy = 0.0;
        if (I < S.n_mobile) polymer_stress(S, sigma, I, xx, xy, yy);
    };
    if (own0 + tid < own1) load(ent[list[own0 + tid]]);
    for (int k = own0 + (tid >> 6); k < own1; k += TILE_THREADS / 64) {
        const int e = list[k], c = (int)cell[e] - hy - 1;  // c: first of its 3 cells in the left column
        const double2 ri = slot_position(e);
        const int a0 = start[c], a1 = start[c + hy], a2 = start[c + 2 * hy];
        const int p1 = start[c + 3] - a0, p2 = p1 + start[c + hy + 3] - a1, p3 = p2 + start[c + 2 * hy + 3] - a2;
        double s = 0.0;
        for (int t = lane; t < p3; t += 64) {
            const double2 rj = slot_position(list[t < p1 ? a0 + t : (t < p2 ? a1 + t - p1 : a2 + t - p2)]);
            double dx = ri.x - rj.x, dy = ri.y - rj.y;
            min_image(S, dx, dy);
            s += kernel_W(S, dx * dx + dy * dy);
        }
        s = wave_sum(s);
        if (lane == 0) {
            S.d[ent[e]] = s;
            if (k - own0 < TILE_POSITIONS) dens[k - own0] = s;
        }
    }
    __syncthreads();
    for (int k = own0 + tid; k < own1; k += TILE_THREADS) {
        const int e = list[k], I = ent[e], g = g0 + k;
        if (k != own0 + tid) load(I);
        const double s = k - own0 < TILE_POSITIONS ? dens[k - own0] : S.d[I], id = 1.0 / s, i2 = id * id;
        S.cidx[g] = I;
        S.cell[g] = ((unsigned)ax << 16) | (unsigned)(ay + (int)cell[e] - hy - 1);
        S.rs[g] = slot_position(e);
        S.vs[g] = vi;
        S.ids[g] = id;
        S.p2s[g] = pressure(S, s) * i2;
        S.s2s[3 * g] = xx * i2;
        S.s2s[3 * g + 1] = xy * i2;
        S.s2s[3 * g + 2] = yy * i2;
    }
}

// The candidates of one particle: the particles of the 3 x 3 cells around its
// cell lie in six runs of the cell order, two per column (the second empty
// unless the column wraps).  Candidate t lies at o_k + t in run k, which
// starts at candidate p_k.
struct Runs {
    int o0, o1, o2, o3, o4, o5, p1, p2, p3, p4, p5, n;
    __device__ __forceinline__ int at(int t) const {
        // all members read first: a choice among them would be one among
        // addresses, and keep them in memory
        const int a0 = o0, a1 = o1, a2 = o2, a3 = o3, a4 = o4, a5 = o5;
        int o = t >= p1 ? a1 : a0;
        o = t >= p2 ? a2 : o;
        o = t >= p3 ? a3 : o;
        o = t >= p4 ? a4 : o;
        o = t >= p5 ? a5 : o;
        return t + o;
    }
};

__device__ __forceinline__ Runs cell_runs(const SphCtx& S, unsigned cell, int lane) {
    const int cx = (int)(cell >> 16), cy = (int)(cell & 0xFFFFu);
    // lanes 4 k + m load the bounds of column cx - 1 + k in one go: m = 0, 1
    // of the run from row cy - 1, m = 2, 3 of its rest across the edge (row
    // cy - 1 comes first: at the lower edge it is the column's last cell, at
    // the upper edge the column's first cell comes last)
    int ax = cx + (lane >> 2) % 3 - 1;
    ax += ax < 0 ? S.ncx : (ax >= S.ncx ? -S.ncx : 0);
    const int lo = cy == 0 ? S.ncy - 1 : cy - 1, hi = cy == 0 ? S.ncy : min(cy + 2, S.ncy);
    const int wrap = cy == 0 ? 2 : (cy == S.ncy - 1 ? 1 : 0);
    const int m = lane & 3;
    const int b = S.cstart[ax * S.ncy + (m == 0 ? lo : (m == 1 ? hi : (m == 2 ? 0 : wrap)))];
    Runs q;
    int p = 0;
    auto run = [&](int k, int& o) {
        const int b0 = __builtin_amdgcn_readlane(b, 2 * k);
        o = b0 - p;
        p += __builtin_amdgcn_readlane(b, 2 * k + 1) - b0;
        return p;
    };
    q.p1 = run(0, q.o0);
    q.p2 = run(1, q.o1);
    q.p3 = run(2, q.o2);
    q.p4 = run(3, q.o3);
    q.p5 = run(4, q.o4);
    q.n = run(5, q.o5);
    return q;
}

// Accelerations (Eq. sph_continuity divided by the mass, plus the body force)
// and the particle's move: drift = 1 the first half kick and the drift, else
// the second half kick.  One wave per particle, in cell order: neighbours are
// read from runs of the sorted records, so index-ordered state can be updated
// in place.  A wave is a chain of three dependent loads (its record and cell,
// its cell runs, its candidates); two rounds of candidates (3 x 3 cells hold
// about 84) are loaded whole before any is tested, as there are but 3.5 waves
// per SIMD for 3572 particles.  6.1 us, gradients 5.4 us, for 3572 particles
// (27 us and 20 us, each candidate through its cell's index list, position
// and then the rest).
constexpr int FORCE_ROUNDS = 2;

__device__ __forceinline__ ForceRec sorted_rec(const SphCtx& S, int g) {
    return {S.rs[g], S.vs[g], S.ids[g], S.p2s[g], S.s2s[3 * g], S.s2s[3 * g + 1], S.s2s[3 * g + 2]};
}

__global__ __launch_bounds__(TPB, 3) void k_force(SphCtx S, int drift) {
    const int g = blockIdx.x * WPB + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    if (g >= S.n) return;
    const int I = S.cidx[g];
    const ForceRec i = sorted_rec(S, g);
    const Runs nb = cell_runs(S, S.cell[g], lane);
    if (I >= S.n_mobile) return;
    const double av = 2.0 * S.eta - S.zeta, bv = 4.0 * S.zeta + 2.0 * S.eta;
    double fx = 0.0, fy = 0.0;
    for (int t = lane; t - lane < nb.n; t += 64 * FORCE_ROUNDS) {
        ForceRec j[FORCE_ROUNDS];
        int q[FORCE_ROUNDS];
#pragma unroll
        for (int u = 0; u < FORCE_ROUNDS; ++u) {
            const int tu = t + 64 * u;
            q[u] = tu < nb.n ? nb.at(tu) : g;  // itself: skipped
            j[u] = sorted_rec(S, q[u]);
        }
#pragma unroll
        for (int u = 0; u < FORCE_ROUNDS; ++u)
            if (q[u] != g) add_force(S, i, j[u], av, bv, fx, fy);
    }
    fx = wave_sum(fx);
    fy = wave_sum(fy);
    if (lane == 0) {
        const double hdt = 0.5 * S.dt;
        const double vx = i.v.x + hdt * (fx / S.mass + body_force(S, i.r.y)), vy = i.v.y + hdt * (fy / S.mass);
        S.v[2 * I] = vx;
        S.v[2 * I + 1] = vy;
        if (drift) {
            const double x = wrap_len(i.r.x + S.dt * vx, S.Lx), y = wrap_len(i.r.y + S.dt * vy, S.Ly);
            S.r[2 * I] = x;
            S.r[2 * I + 1] = y;
            S.key[I] = cell_key(S, x, y);
        }
    }
}

// cells of the initial positions
__global__ __launch_bounds__(TPB) void k_keys(SphCtx S) {
    const int I = blockIdx.x * TPB + (int)threadIdx.x;
    if (I < S.n) S.key[I] = cell_key(S, S.r[2 * I], S.r[2 * I + 1]);
}

// k_gradL with cells (positions in cell order, velocities by index)
__global__ __launch_bounds__(TPB, 3) void k_gradient(SphCtx S, double* __restrict__ gradL) {
    const int g = blockIdx.x * WPB + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    if (g >= S.n) return;
    const int I = S.cidx[g];
    const Runs nb = cell_runs(S, S.cell[g], lane);
    const double2 ri = S.rs[g];
    if (I >= S.n_mobile) {
        if (lane < 9) gradL[9 * I + lane] = 0.0;
        return;
    }
    const double2 vi = velocity(S, I);
    double sum[4] = {};
    for (int t = lane; t - lane < nb.n; t += 64 * FORCE_ROUNDS) {
        double2 r[FORCE_ROUNDS], v[FORCE_ROUNDS];
        double id[FORCE_ROUNDS];
        int q[FORCE_ROUNDS], J[FORCE_ROUNDS];
#pragma unroll
        for (int u = 0; u < FORCE_ROUNDS; ++u) {
            const int tu = t + 64 * u;
            q[u] = tu < nb.n ? nb.at(tu) : g;
            J[u] = S.cidx[q[u]];
            r[u] = S.rs[q[u]];
            id[u] = S.ids[q[u]];
        }
#pragma unroll
        for (int u = 0; u < FORCE_ROUNDS; ++u) v[u] = velocity(S, J[u]);
#pragma unroll
        for (int u = 0; u < FORCE_ROUNDS; ++u)
            if (q[u] != g) add_gradient(S, ri, r[u], vi, v[u], id[u], sum);
    }
    store_gradient(S, sum, lane, gradL + 9 * I);
}

}  // namespace

struct lhmm_sph {
    SphCtx S{};
    hipStream_t stream = nullptr;
    double* d_sigma = nullptr;  // n x 6, micro stresses of the last interval (zero at start)
    double* d_gradL = nullptr;  // n x 9
    void* arena = nullptr;  // every device array
    HostStage stage;
};

namespace {

void sph_release(lhmm_sph* s) {
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    if (s->arena) (void)hipFree(s->arena);
    s->stage.release();
}

void launch_tile(lhmm_sph* s, const double* sigma) {
    const SphCtx& S = s->S;
    k_tile<<<dim3(S.tiles, S.ncx), TILE_THREADS, TILE_LDS * (size_t)S.n, s->stream>>>(S, sigma);
}

// densities at the current positions (and, with cells, the cell order)
void launch_density(lhmm_sph* s) {
    if (s->S.ncx > 0)
        launch_tile(s, nullptr);
    else
        k_density<<<(s->S.n + WPB - 1) / WPB, TPB, 0, s->stream>>>(s->S);
}

void launch_sph_step(lhmm_sph* s, const double* sigma, double* gradL) {
    const int gw = (s->S.n + WPB - 1) / WPB;  // wave per particle
    const int gt = (s->S.n + TPB - 1) / TPB;  // thread per particle
    hipStream_t st = s->stream;
    if (s->S.ncx > 0) {
        launch_tile(s, sigma);
        k_force<<<gw, TPB, 0, st>>>(s->S, 1);
        launch_tile(s, sigma);
        k_force<<<gw, TPB, 0, st>>>(s->S, 0);
        if (gradL) k_gradient<<<gw, TPB, 0, st>>>(s->S, gradL);
        return;
    }
    k_density<<<gw, TPB, 0, st>>>(s->S);
    k_accel<<<gw, TPB, 0, st>>>(s->S, sigma);
    k_kick_drift<<<gt, TPB, 0, st>>>(s->S);
    k_density<<<gw, TPB, 0, st>>>(s->S);
    k_accel<<<gw, TPB, 0, st>>>(s->S, sigma);
    k_kick<<<gt, TPB, 0, st>>>(s->S);
    if (gradL) k_gradL<<<gw, TPB, 0, st>>>(s->S, gradL);
}

}  // namespace

hipStream_t lhmm_sph_caller_stream(const lhmm_sph* s) { return s->stream; }

void lhmm_sph_counts(const lhmm_sph* s, int* n, int* n_mobile) {
    *n = s->S.n;
    *n_mobile = s->S.n_mobile;
}

extern "C" {

int lhmm_sph_create(const lhmm_sph_params* p, int32_t n, const double* r0, const double* v0, void* stream,
                    lhmm_sph** out) {
    lhmm_clear_error();
    if (!p || !r0 || !v0 || !out) return lhmm_fail(LHMM_ERR_ARG, "null argument");
    *out = nullptr;
    if (n <= 0) return lhmm_fail(LHMM_ERR_ARG, "n must be positive (got %d)", n);
    if (p->n_fixed < 0 || p->n_fixed >= n) return lhmm_fail(LHMM_ERR_ARG, "n_fixed must be in 0..n-1 (got %d)", p->n_fixed);
    if (p->force_mode != LHMM_FORCE_REVERSE && p->force_mode != LHMM_FORCE_UNIFORM)
        return lhmm_fail(LHMM_ERR_ARG, "unknown force_mode %d", p->force_mode);
    if (p->kernel != LHMM_KERNEL_QUINTIC && p->kernel != LHMM_KERNEL_LUCY)
        return lhmm_fail(LHMM_ERR_ARG, "unknown kernel %d", p->kernel);
    if (p->micro_dim != 0 && p->micro_dim != 2 && p->micro_dim != 3)
        return lhmm_fail(LHMM_ERR_ARG, "micro_dim must be 0, 2 or 3 (got %d)", p->micro_dim);
    const double vals[] = {p->rho0, p->eta, p->zeta, p->c, p->theta, p->F, p->h, p->dt, p->mass, p->Lx, p->Ly,
                           p->lambda_star, p->alpha};
    for (double x : vals)
        if (!std::isfinite(x)) return lhmm_fail(LHMM_ERR_ARG, "non-finite SPH parameter");
    if (!(p->rho0 > 0) || !(p->c > 0) || !(p->h > 0) || !(p->dt > 0) || !(p->mass > 0) || !(p->lambda_star > 0) ||
        p->eta < 0 || p->zeta < 0)
        return lhmm_fail(LHMM_ERR_ARG, "SPH parameters out of range");
    if (!(p->Lx > 2 * p->h) || !(p->Ly > 2 * p->h))
        return lhmm_fail(LHMM_ERR_ARG, "the periodic box must be wider than twice the kernel support");
    for (int k = 0; k < 2 * n; ++k) {
        if (!std::isfinite(r0[k]) || !std::isfinite(v0[k])) return lhmm_fail(LHMM_ERR_ARG, "non-finite state");
        const double L = (k % 2 == 0) ? p->Lx : p->Ly;
        if (!(r0[k] >= 0.0 && r0[k] < L)) return lhmm_fail(LHMM_ERR_ARG, "position %d outside the box", k / 2);
    }
    lhmm_sph* s = new (std::nothrow) lhmm_sph();
    if (!s) return lhmm_fail(LHMM_ERR_OOM, "host allocation failed");
    s->stream = (hipStream_t)stream;
    SphCtx& S = s->S;
    S.n = n;
    S.n_mobile = n - p->n_fixed;
    S.force_mode = p->force_mode;
    S.kernel = p->kernel;
    S.micro_dim = p->micro_dim == 2 ? 2 : 3;
    S.rho0 = p->rho0; S.eta = p->eta; S.zeta = p->zeta; S.c = p->c; S.theta = p->theta; S.F = p->F; S.h = p->h;
    S.dt = p->dt; S.mass = p->mass; S.Lx = p->Lx; S.Ly = p->Ly; S.lambda_star = p->lambda_star; S.alpha = p->alpha;
    S.qs = (S.kernel == LHMM_KERNEL_LUCY ? 1.0 : 3.0) / S.h;
    S.cW = S.kernel == LHMM_KERNEL_LUCY ? 5.0 / (M_PI * S.h * S.h) : 63.0 / (478.0 * M_PI * S.h * S.h);
    S.cF = S.kernel == LHMM_KERNEL_LUCY ? 60.0 / (M_PI * (S.h * S.h) * (S.h * S.h)) : 3.0 * S.cW / S.h;
    // cell grid of side >= h: at least 3 x 3 cells; k_tile holds
    // every particle's slot in LDS (TILE_LDS bytes each, 144 KiB at this bound)
    {
        const int gx = (int)std::floor(p->Lx / p->h), gy = (int)std::floor(p->Ly / p->h);
        const bool fits = gx >= 3 && gy >= 3 && (long long)gx * gy + n <= (65536 - 64) / 4;
        if (fits) {
            const CellTiles tiles = cell_tiles(gx, gy);
            S.turned = tiles.turned;
            S.ncx = tiles.ncol;
            S.ncy = tiles.nrow;
            S.rows = tiles.rows;
            S.tiles = tiles.tiles;
        }
    }
    // beyond 64 KiB with k_tile's static LDS (13 KiB)
    if (S.ncx > 0 && TILE_LDS * n > 48 * 1024 &&
        hipFuncSetAttribute((const void*)&k_tile, hipFuncAttributeMaxDynamicSharedMemorySize, TILE_LDS * 16384) != hipSuccess) {
        delete s;
        return lhmm_fail(LHMM_ERR_HIP, "cell tiles: LDS of 144 KiB refused");
    }
    const size_t m = (size_t)n;
    const size_t sizes[16] = {2 * m, 2 * m, m, m, 2 * m, 6 * m, 9 * m, (size_t)S.ncx * S.ncy + 1, m, m, 2 * m, 2 * m, m, m,
                              3 * m, m};
    // one allocation, its arrays on 256-byte boundaries
    size_t total = 0;
    for (size_t k : sizes) total += (k * sizeof(double) + 255) / 256 * 256;
    if (hipMalloc(&s->arena, total) != hipSuccess) {
        sph_release(s);
        delete s;
        return lhmm_fail(LHMM_ERR_OOM, "hipMalloc failed");
    }
    void* bufs[16];
    char* at = (char*)s->arena;
    for (int k = 0; k < 16; ++k) {
        bufs[k] = at;
        at += (sizes[k] * sizeof(double) + 255) / 256 * 256;
    }
    S.r = (double*)bufs[0];
    S.v = (double*)bufs[1];
    S.d = (double*)bufs[2];
    S.p = (double*)bufs[3];
    S.acc = (double*)bufs[4];
    s->d_sigma = (double*)bufs[5];
    s->d_gradL = (double*)bufs[6];
    S.cstart = (int*)bufs[7];
    S.cidx = (int*)bufs[8];
    S.key = (unsigned*)bufs[9];
    S.rs = (double2*)bufs[10];
    S.vs = (double2*)bufs[11];
    S.ids = (double*)bufs[12];
    S.p2s = (double*)bufs[13];
    S.s2s = (double*)bufs[14];
    S.cell = (unsigned*)bufs[15];
    auto init = [&]() -> int {
        LHMM_HIPCHK(s->stage.reserve(0));
        LHMM_HIPCHK(hipMemcpy(S.r, r0, 2 * (size_t)n * sizeof(double), hipMemcpyHostToDevice));
        LHMM_HIPCHK(hipMemcpy(S.v, v0, 2 * (size_t)n * sizeof(double), hipMemcpyHostToDevice));
        LHMM_HIPCHK(hipMemset(s->d_sigma, 0, 6 * (size_t)n * sizeof(double)));
        LHMM_HIPCHK(hipMemset(s->d_gradL, 0, 9 * (size_t)n * sizeof(double)));
        if (S.ncx > 0) {
            k_keys<<<(n + TPB - 1) / TPB, TPB, 0, s->stream>>>(S);
            LHMM_HIPCHK(hipGetLastError());
        }
        return LHMM_OK;
    };
    int rc = init();
    if (rc != LHMM_OK) {
        sph_release(s);
        delete s;
        return rc;
    }
    *out = s;
    return LHMM_OK;
}

int lhmm_sph_step(lhmm_sph* s, const double* sigma, double* gradL_out) {
    lhmm_clear_error();
    if (!s) return lhmm_fail(LHMM_ERR_ARG, "null engine");
    launch_sph_step(s, sigma, gradL_out);
    LHMM_HIPCHK(hipGetLastError());
    return LHMM_OK;
}

int lhmm_sph_get_state(lhmm_sph* s, double* r, double* v, double* d) {
    lhmm_clear_error();
    if (!s) return lhmm_fail(LHMM_ERR_ARG, "null engine");
    if (d) launch_density(s);  // at the current positions
    LHMM_HIPCHK(hipGetLastError());
    const size_t b = (size_t)s->S.n * sizeof(double);
    LHMM_HIPCHK(s->stage.copy(s->stream, {{s->S.r, 2 * b}, {s->S.v, 2 * b}, {s->S.d, b}}, {r, v, d}));
    return LHMM_OK;
}

int lhmm_sph_coupling_state(lhmm_sph* s, double* sigma, double* gradL) {
    lhmm_clear_error();
    if (!s) return lhmm_fail(LHMM_ERR_ARG, "null engine");
    const size_t b = (size_t)s->S.n * sizeof(double);
    LHMM_HIPCHK(s->stage.copy(s->stream, {{s->d_sigma, 6 * b}, {s->d_gradL, 9 * b}}, {sigma, gradL}));
    return LHMM_OK;
}

int lhmm_couple_step(lhmm_sph* s, lhmm_micro* m, int32_t m_bar, int32_t k_micro) {
    lhmm_clear_error();
    if (!s || !m) return lhmm_fail(LHMM_ERR_ARG, "null engine");
    if (m_bar <= 0) return lhmm_fail(LHMM_ERR_ARG, "m_bar must be positive (got %d)", m_bar);
    if (k_micro <= 0) return lhmm_fail(LHMM_ERR_ARG, "k_micro must be positive (got %d)", k_micro);
    int32_t nb = 0;
    int rc = lhmm_micro_sizes(m, nullptr, &nb);
    if (rc != LHMM_OK) return rc;
    if (nb != s->S.n_mobile)
        return lhmm_fail(LHMM_ERR_ARG, "micro engine holds %d boxes for %d mobile SPH particles", nb, s->S.n_mobile);
    if (lhmm_micro_caller_stream(m) != s->stream)
        return lhmm_fail(LHMM_ERR_ARG, "the SPH and micro engines must share one stream");
    // m_bar SPH steps under the stored micro stresses; the gradient of the
    // last one drives the micro-domains
    for (int k = 0; k < m_bar; ++k) launch_sph_step(s, s->d_sigma, k + 1 == m_bar ? s->d_gradL : nullptr);
    LHMM_HIPCHK(hipGetLastError());
    return lhmm_micro_step(m, s->d_gradL, k_micro, s->d_sigma);
}

int lhmm_sph_destroy(lhmm_sph* s) {
    lhmm_clear_error();
    if (!s) return LHMM_OK;
    sph_release(s);
    delete s;
    return LHMM_OK;
}

}  // extern "C"
