// lhmm_micro.hip -- gfx950 kernels and runtime of the batched micro-DPD
// engine behind include/lhmm.h.
//
// A step of every box (velocity-Verlet of the micro-scale equation of motion,
// Eq. motion, in a periodic cell deformed by the box's velocity gradient;
// Appendix "Detailed Coupling Protocol", Step 3) is two launches over a
// flattened index of all boxes:
//   k_bin          a counting sort of the particles by cell, a workgroup per
//                  slab of a box's cell columns, each cell in index order so
//                  every sum has a fixed order; beside it the next step's cell
//                  (FP64: mid-step cell inverse, deformation h <- exp(L dt) h,
//                  Lagrange-Gauss reduction of the in-plane basis, cell grid,
//                  width guard);
//   k_forces       per particle: conservative + dissipative + random pair
//                  forces (Eqs. conservative, dissipative, random) over the
//                  neighbour cells, FENE springs (Eq. fene_force), the
//                  second half kick with the final force, the block's virial
//                  and kinetic partial sums in FP64, and the next step's half
//                  kick c += dt/2 (F/m - L c) and drift of the fractional
//                  coordinates with the mid-step cell (remap by the reduction,
//                  wrap, cell index), written in cell order for the next
//                  binning.  k_forces_wide does the same with sixteen lanes
//                  per particle, for launches too small to fill the chip.
// Steps come in chunks (captured in HIP graphs): k_begin_chunk takes the
// particles from their arrays in index order through the first half kick and
// drift, the last step's force pass puts them back, and k_window_sums and
// k_flush reduce the window's partial sums to the boxes' stresses (Eqs. IKtotal, kinetic_stress,
// potential_stress with a uniform weight over the cell).
// A box may instead be a micro-domain with boundary regions (Sec.
// "Macro-to-Micro Coupling", Tab. 2): its cell stays fixed, the particles of
// the boundary-condition ring relax toward the imposed field v' = G r' of
// Eq. micro_bc after each half kick (an Ornstein-Uhlenbeck step with thermal
// noise), and its stress is the Irving-Kirkwood stress of the core (kinetic
// part over the core's particles relative to the imposed field, each pair's
// virial weighted by the fraction of its segment inside the core).
// The per-particle kernels run over work blocks of BS particles; a block
// never straddles two boxes, so per-box quantities are uniform in a block
// and reductions stay deterministic.  Particle state is single or double precision (template
// parameter); cells, gradients and stress sums are always double.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "lhmm.h"
#include "lhmm_internal.h"
#include "lhmm_grid.h"
#include "lhmm_stage.h"

namespace {

constexpr int BS = 256;                 // particles per work block
constexpr int SREC_PAD = 4;             // padding records per column of the search layout
constexpr int MAX_CELLS_PER_BOX = 17424;
constexpr int GRAPH_CHUNK = 50;         // default steps per captured graph
constexpr int MAX_GROUPS = 4;           // overlapped box groups of a captured step
// Default groups, by work blocks.  Below four blocks per CU the two launches
// of a group leave each other little to overlap and split the chip's tail:
// 166k particles with stress components 1290 us in one group, 1473 in two
// (plain forces 1264 and 1263); 311k plain 1530 and 1457.  Three pay from about
// 930k particles: 2984 us in two, 2836 in three (681k: 2360 and 2402).
constexpr int GROUP2_BLOCKS = 1024;
constexpr int GROUP3_BLOCKS = 3584;
constexpr int MAX_WINDOW = 50;          // steps whose partial sums are kept before a flush (at most 64)
constexpr size_t PART_BYTES = size_t(64) << 20;  // their memory, where more than one step would take more
constexpr int ACC = 36;                 // per-box stress sums: kinetic, pair, FENE, C, D, R (6 each)

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIPCHK(expr)                                                                       \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess) return fail(LHMM_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

struct BoxInfo {
    int off;       // first particle (global index)
    int n;         // particles
    int n_beads;   // n_chains * chain_len
    int cell_cap;  // cell capacity
    int gcell_off; // first slot in gcell_start (2 cap + 1 slots per box)
    long long srec_off;  // first record in srec
    int zsub;      // cells per cutoff along z (1 or 2): the z range of a stencil row is 2 zsub + 1 cells
    int blk_off;   // first work block
    int nblk;      // work blocks
    int slab_off;  // first slab of the binning
    int nslab;     // slabs
    unsigned rng_id;  // box word of the random-force counter
};

struct BoxDyn {  // per-box FP64 state, rewritten every step; two slots (see Step)
    double h[9];
    double L[9];
    double E[9];
    double Eh[9];
    double hmi[9];  // inverse of the mid-step cell
    double vol;
    int U[4];       // in-plane reduction of this step, h_new = h U
    int nc[3];      // cell grid of this step
    int changed;
    // boundary regions (hc > 0): core |x'|, |y'| < hc, ring hc <= max(|x'|, |y'|)
    // < hb, positions relative to the cell centre; G: the imposed in-plane
    // gradient (xx, xy, yx, yy), while the cell's own L stays zero
    double hc, hb;
    double G[4];
};

struct Ctx {
    int n_total, n_boxes, n_blocks, chain_len;
    const BoxInfo* box;
    BoxDyn* dyn;  // 2 x n_boxes: slot 0 holds the state between chunks
    unsigned* flags;
    const int* blk_box;
    const int* blk_first;
    const int* slab_box;
    // selection: when sel is set, per-box kernels run over the n_sel boxes
    // sel[0..n_sel), per-block kernels over the work blocks blk_list[..] (those
    // of sel[q] from blk0[q] on) and the binning over the slabs slab_list[..]
    const int* sel;
    const int* blk0;
    const int* blk_list;
    const int* slab_list;
    int n_sel;
    void* s;  // SoA: component k of particle i at [k * n_total + i]
    void* c;
    void* f;
    // inside a chunk: records (s, index) by index for the bonds (every
    // particle's at the first step, the beads' later) and in the last cell
    // order, two slots each (one read, one written by a force pass); (c, cell)
    // and the cell alone in the source order of the next binning; each
    // cell-order position's source position
    void* sid[2];
    void* sord[2];
    void* cord;
    int* key;
    int* perm;
    // per box, cell-sorted pairs of records: (x, y, z, local index), r = h s,
    // then (cx, cy, cz, local index), 2 x 4 reals per particle (one scattered
    // 32-byte store in the binning, one 32-byte segment per neighbour in the
    // force kernel's evaluation)
    void* cell_pv;
    // Search layout: per box (at 2 x its particle offset) every cell column
    // (m0, m1) as [images of its top zsub cells shifted by -h_z][its cells]
    // [images of its bottom zsub cells shifted by +h_z], so the z cells
    // k2 - zsub .. k2 + zsub around any cell are one contiguous range.
    // SREC_PAD records far away follow each column, so that a search may read
    // past a range's end; gcell_start holds the starts of a column's n2 + 2 zsub
    // cells and the end of the last.
    // srec: (x, y, z, cell-order position << 5 | 9 x z image: 0 none,
    // 1 below, 2 above), r = h s; padded by four records.
    int* gcell_start;
    void* srec;
    // partial sums of the window's steps: part_step per step, nv per work block
    // (or per sixteen particles: k_forces_wide) in the launch's order: pair
    // virial 6, FENE virial 6, ordered pairs, kinetic 6 (+ C, D, R virials)
    double* part;
    size_t part_step;
    int nv;             // 19, or 37 when the conservative, dissipative and random parts are kept
    double* sums;       // nv per box and step of the window: the partial sums reduced
    double* vol;        // n_boxes per step of the window
    double vir_scale;   // 1 when each pair is evaluated once, 1/2 when twice
    double* acc;        // n_boxes x ACC: kinetic, pair, FENE, C, D, R stress sums
    unsigned long long* acc_pairs;  // n_boxes
    unsigned long long* tot_pairs;  // n_boxes, every step since the engine was created
    unsigned long long* step;       // completed steps
    double a, gamma, sigma, rdt, dt, mass, inv_mass, rc, rc2, H, inv_R02;
    double ou_damp, ou_amp;  // ring relaxation over half a step: exp(-zeta dt/2), sqrt(kBT/m (1 - exp(-zeta dt)))
    unsigned key0, key1;
};

// One step's launches inside a chunk.  A step's cell is in dyn slot `slot`, the
// next one's in the other; its own positions come from sid[slot] (first) or
// sord[slot], its bond partners' from sid[slot].
struct Step {
    int slot;
    int first;  // first step of the chunk
    int more;   // another step of the chunk follows
    int kick;   // 0: forces only (no second half kick)
    int w;      // place in the window of partial sums
    int k;      // this step's random-force counter is *C.step + k
    int part0;  // first work block of the launch in the partial sums
};

// ---------------------------------------------------------------------------
// Counter-based random numbers: Philox4x32-10 (Salmon et al., SC'11) keyed
// by the seed, counter (min id, max id, step, box); a Box-Muller normal from
// the top 23 bits of the first two output words.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void philox4x32_10(unsigned& x0, unsigned& x1, unsigned& x2, unsigned& x3,
                                              unsigned k0, unsigned k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const unsigned long long p0 = (unsigned long long)0xD2511F53u * x0;
        const unsigned long long p1 = (unsigned long long)0xCD9E8D57u * x2;
        // three-input xors as one v_bitop3_b32 each (truth table 0x96)
        const unsigned y0 = __builtin_amdgcn_bitop3_b32((unsigned)(p1 >> 32), x1, k0, 0x96);
        const unsigned y2 = __builtin_amdgcn_bitop3_b32((unsigned)(p0 >> 32), x3, k1, 0x96);
        x1 = (unsigned)p1;
        x3 = (unsigned)p0;
        x0 = y0;
        x2 = y2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// The pair stream's generator: counter (x0, x1, step, box), where step,
// box and the key are the same for a whole workgroup.  In the first two
// rounds two of the three inputs of one or both xors are then uniform; the
// xors are grouped so that the scalar unit combines those two (one vector
// xor, where a v_bitop3_b32 would need one of them moved to a vector
// register first).  The output equals philox4x32_10's.
__device__ __forceinline__ void philox_pair(unsigned& x0, unsigned& x1, unsigned step, unsigned box, unsigned k0,
                                            unsigned k1) {
    // round 1: M1 step and key are uniform, and so are box and key
    unsigned long long p0 = (unsigned long long)0xD2511F53u * x0;
    unsigned long long p1 = (unsigned long long)0xCD9E8D57u * step;
    unsigned y0 = ((unsigned)(p1 >> 32) ^ k0) ^ x1;
    unsigned y2 = (box ^ k1) ^ (unsigned)(p0 >> 32);
    const unsigned u1 = (unsigned)p1;  // the second word is uniform after round 1
    unsigned x3 = (unsigned)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    // round 2: the second word and key are uniform
    p0 = (unsigned long long)0xD2511F53u * y0;
    p1 = (unsigned long long)0xCD9E8D57u * y2;
    x0 = (u1 ^ k0) ^ (unsigned)(p1 >> 32);
    unsigned x2 = __builtin_amdgcn_bitop3_b32((unsigned)(p0 >> 32), x3, k1, 0x96);
    x1 = (unsigned)p1;
    x3 = (unsigned)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        p0 = (unsigned long long)0xD2511F53u * x0;
        p1 = (unsigned long long)0xCD9E8D57u * x2;
        const unsigned z0 = __builtin_amdgcn_bitop3_b32((unsigned)(p1 >> 32), x1, k0, 0x96);
        const unsigned z2 = __builtin_amdgcn_bitop3_b32((unsigned)(p0 >> 32), x3, k1, 0x96);
        x1 = (unsigned)p1;
        x3 = (unsigned)p0;
        x0 = z0;
        x2 = z2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

template <typename real>
__device__ __forceinline__ real box_muller(unsigned w0, unsigned w1);

// (m + 1/2) 2^-23 for the top 23 bits m of w: the float 1 + m 2^-23 (exponent
// bits 0x7F above m, one funnel shift) less 1 - 2^-24, a subtraction without
// rounding since both lie in [1/2, 2)
__device__ __forceinline__ float unit_open(unsigned w) {
    return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, w, 9u)) - 0x1.fffffep-1f;
}

template <>
__device__ __forceinline__ float box_muller<float>(unsigned w0, unsigned w1) {
    const float u0 = unit_open(w0);
    const float u1 = unit_open(w1);
    // v_log_f32 is log2; v_cos_f32 takes its argument in revolutions
    // -2 ln u0 lies in [1e-7, 35]: the hardware square root (1 ulp) needs no range handling
    const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u0));  // -2 ln u0
    return r * __builtin_amdgcn_cosf(u1);
}

template <>
__device__ __forceinline__ double box_muller<double>(unsigned w0, unsigned w1) {
    const double u0 = ((double)(w0 >> 9) + 0.5) * 1.1920928955078125e-07;
    const double u1 = ((double)(w1 >> 9) + 0.5) * 1.1920928955078125e-07;
    return sqrt(-2.0 * log(u0)) * cos(2.0 * M_PI * u1);
}

// both Box-Muller normals (cosine and sine branches) of two output words
template <typename real>
__device__ __forceinline__ void box_muller2(unsigned w0, unsigned w1, real& x, real& y);

template <>
__device__ __forceinline__ void box_muller2<float>(unsigned w0, unsigned w1, float& x, float& y) {
    const float u0 = ((float)(w0 >> 9) + 0.5f) * 1.1920928955078125e-07f;
    const float u1 = ((float)(w1 >> 9) + 0.5f) * 1.1920928955078125e-07f;
    const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u0));
    x = r * __builtin_amdgcn_cosf(u1);
    y = r * __builtin_amdgcn_sinf(u1);
}

template <>
__device__ __forceinline__ void box_muller2<double>(unsigned w0, unsigned w1, double& x, double& y) {
    const double u0 = ((double)(w0 >> 9) + 0.5) * 1.1920928955078125e-07;
    const double u1 = ((double)(w1 >> 9) + 0.5) * 1.1920928955078125e-07;
    const double r = sqrt(-2.0 * log(u0));
    x = r * cos(2.0 * M_PI * u1);
    y = r * sin(2.0 * M_PI * u1);
}

template <typename real>
__device__ __forceinline__ real pair_theta(unsigned id_i, unsigned id_j, unsigned step, unsigned box,
                                           unsigned k0, unsigned k1) {
    unsigned x0 = min(id_i, id_j), x1 = max(id_i, id_j);
    philox_pair(x0, x1, step, box, k0, k1);
    return box_muller<real>(x0, x1);
}

// ---------------------------------------------------------------------------
// Cell-sorted particle records: (x, y, z, local index) in one 4-vector
// ---------------------------------------------------------------------------

template <typename real>
struct Rec;
template <>
struct Rec<float> {
    using T = float4;
    __device__ static T make(float x, float y, float z, int id) { return make_float4(x, y, z, __int_as_float(id)); }
    __device__ static int id(T v) { return __float_as_int(v.w); }
};
template <>
struct Rec<double> {
    using T = double4;
    __device__ static T make(double x, double y, double z, int id) { return make_double4(x, y, z, (double)id); }
    __device__ static int id(T v) { return (int)v.w; }
};

// Raw buffer view of a record array (stride 0, no range limit in practice):
// a float record is read by one 16-byte buffer load, which the compiler keeps
// whole, so the loads of a search step are issued together and none is
// deferred into the branch that queues a neighbour.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rec_rsrc(const char* base) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, 0x7fffffff, 0x00020000);
}

template <typename real>
__device__ __forceinline__ typename Rec<real>::T load_rec(__amdgpu_buffer_rsrc_t r, const char* base, unsigned off);

template <>
__device__ __forceinline__ float4 load_rec<float>(__amdgpu_buffer_rsrc_t r, const char*, unsigned off) {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    const u4 x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    return make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
}

template <>
__device__ __forceinline__ double4 load_rec<double>(__amdgpu_buffer_rsrc_t, const char* base, unsigned off) {
    return *(const double4*)(base + off);
}

// ---------------------------------------------------------------------------
// FP64 cell algebra (row-major 3x3; columns are lattice vectors)
// ---------------------------------------------------------------------------

__host__ __device__ inline void m3_mul(const double* A, const double* B, double* C) {
    double T[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j)
            T[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] + A[3 * i + 2] * B[6 + j];
    for (int k = 0; k < 9; ++k) C[k] = T[k];
}

__host__ __device__ inline void m3_inv(const double* A, double* B) {
    const double id = 1.0 / m3_det(A);
    double T[9];
    T[0] = (A[4] * A[8] - A[5] * A[7]) * id;
    T[1] = (A[2] * A[7] - A[1] * A[8]) * id;
    T[2] = (A[1] * A[5] - A[2] * A[4]) * id;
    T[3] = (A[5] * A[6] - A[3] * A[8]) * id;
    T[4] = (A[0] * A[8] - A[2] * A[6]) * id;
    T[5] = (A[2] * A[3] - A[0] * A[5]) * id;
    T[6] = (A[3] * A[7] - A[4] * A[6]) * id;
    T[7] = (A[1] * A[6] - A[0] * A[7]) * id;
    T[8] = (A[0] * A[4] - A[1] * A[3]) * id;
    for (int k = 0; k < 9; ++k) B[k] = T[k];
}

// Is L finite, in-plane and traceless?
__host__ __device__ inline bool gradient_ok(const double* L) {
    double scale = 1.0;
    for (int k = 0; k < 9; ++k) {
        if (!(fabs(L[k]) <= 1e300)) return false;
        scale += fabs(L[k]);
    }
    if (L[2] != 0.0 || L[5] != 0.0 || L[6] != 0.0 || L[7] != 0.0 || L[8] != 0.0) return false;
    return fabs(L[0] + L[4]) <= 1e-12 * scale;
}

// exp(L tau) for in-plane traceless L: in the plane L^2 = k^2 I, k^2 = a^2 + bc,
// so exp(L tau) = f0 I + f1 L with (cosh, sinh/k), (cos, sin/w) or (1, tau).
__host__ __device__ inline void expm_planar(const double* L, double tau, double* E) {
    const double a = 0.5 * (L[0] - L[4]), b = L[1], c = L[3];
    const double k2 = a * a + b * c;
    double f0, f1;
    if (k2 > 0.0) {
        const double k = sqrt(k2);
        f0 = cosh(k * tau);
        f1 = sinh(k * tau) / k;
    } else if (k2 < 0.0) {
        const double w = sqrt(-k2);
        f0 = cos(w * tau);
        f1 = sin(w * tau) / w;
    } else {
        f0 = 1.0;
        f1 = tau;
    }
    E[0] = f0 + f1 * a; E[1] = f1 * b;      E[2] = 0.0;
    E[3] = f1 * c;      E[4] = f0 - f1 * a; E[5] = 0.0;
    E[6] = 0.0;         E[7] = 0.0;         E[8] = 1.0;
}

// Lagrange-Gauss reduction of the in-plane basis (columns 0 and 1 of h);
// swaps as (b1, b2) -> (b2, -b1), size reductions b2 -= m b1 with
// m = floor(mu + 1/2).  U accumulates h_new = h U (det U = +1).
__host__ __device__ inline int reduce_planar(double* h, int* U) {
    double b1x = h[0], b1y = h[3], b2x = h[1], b2y = h[4];
    long long u00 = 1, u01 = 0, u10 = 0, u11 = 1;
    int changed = 0;
    for (int it = 0; it < 256; ++it) {
        const double n1 = b1x * b1x + b1y * b1y, n2 = b2x * b2x + b2y * b2y;
        if (n2 < n1) {
            const double tx = b1x, ty = b1y;
            b1x = b2x; b1y = b2y;
            b2x = -tx; b2y = -ty;
            const long long a0 = u01, a1 = -u00, c0 = u11, c1 = -u10;
            u00 = a0; u01 = a1; u10 = c0; u11 = c1;
            changed = 1;
            continue;
        }
        const long long m = (long long)floor((b1x * b2x + b1y * b2y) / n1 + 0.5);
        if (m == 0) break;
        b2x -= (double)m * b1x;
        b2y -= (double)m * b1y;
        u01 -= m * u00;
        u11 -= m * u10;
        changed = 1;
    }
    h[0] = b1x; h[3] = b1y; h[1] = b2x; h[4] = b2y;
    U[0] = (int)u00; U[1] = (int)u01; U[2] = (int)u10; U[3] = (int)u11;
    return changed;
}

// ---------------------------------------------------------------------------
// Reductions
// ---------------------------------------------------------------------------

// One level of a wave reduction of N values per lane: lanes o apart add, and
// each keeps half of the values (the lane with the bit set the upper half).
// idx and n follow which values a lane still holds.
template <int N>
__device__ __forceinline__ void halve(double (&v)[N], int o, bool up, int& idx, int& n, double (&out)[(N + 1) / 2]) {
    constexpr int M = (N + 1) / 2;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const double hi = k + M < N ? v[k + M] : 0.0;
        const double send = up ? v[k] : hi, keep = up ? hi : v[k];
        out[k] = keep + __shfl_xor(send, o, 64);
    }
    if (up) {
        idx += M;
        n -= M;
    } else {
        n = min(n, M);
    }
}

// Sums of NV doubles over the workgroup (BS threads) to out[0 .. NV).  Lanes
// 32, 16, .. 1 apart are added in that order and the waves after them in
// order; each level halves the values a lane carries on, which takes about
// 22 exchanges instead of 6 NV for the same sums.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* sh /* NV * (BS/64) */, double* out) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int idx = 0, n = NV;
    constexpr int N1 = (NV + 1) / 2, N2 = (N1 + 1) / 2, N3 = (N2 + 1) / 2, N4 = (N3 + 1) / 2, N5 = (N4 + 1) / 2,
                  N6 = (N5 + 1) / 2;
    double a1[N1], a2[N2], a3[N3], a4[N4], a5[N5], a6[N6];
    halve<NV>(v, 32, lane & 32, idx, n, a1);
    halve<N1>(a1, 16, lane & 16, idx, n, a2);
    halve<N2>(a2, 8, lane & 8, idx, n, a3);
    halve<N3>(a3, 4, lane & 4, idx, n, a4);
    halve<N4>(a4, 2, lane & 2, idx, n, a5);
    halve<N5>(a5, 1, lane & 1, idx, n, a6);
    static_assert(N6 == 1, "one value per lane at the end");
    if (n > 0) sh[wv * NV + idx] = a6[0];
    __syncthreads();
    if ((int)threadIdx.x < NV) {
        double t = 0.0;
        for (int w = 0; w < BS / 64; ++w) t += sh[w * NV + threadIdx.x];
        out[threadIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------

constexpr int N_XCD = 8;  // MI355X: workgroups are dealt to the 8 XCDs round robin

// Work item of workgroup b out of n, chosen so that each XCD (b mod 8) gets
// one contiguous run of work items: the blocks of a box then share one L2.
__device__ __forceinline__ int xcd_local_work(int b, int n) {
    const int x = b % N_XCD, l = b / N_XCD;
    const int per = n / N_XCD, rem = n % N_XCD;
    return x * per + min(x, rem) + l;
}

// Per call.  The first n_mean workgroups remove their box's mean peculiar
// velocity (every box, or every selected one): the pair forces cancel, so the
// mean obeys d<c>/dt = -L <c>; a flow that compresses the box amplifies it,
// and the rounding of the two-sided single-precision pair forces seeds it.
// The micro-domain moves with its macro particle, so its mean is zero.  The
// remaining workgroups, a thread per box, take the box's gradient (device
// array n_boxes x 9), validate it, form exp(L dt) and exp(L dt/2), and, where
// steps follow (clear), zero the call's sums: a force evaluation leaves the last
// step call's pair counts.  One launch: the two parts touch different data.
constexpr int CALL_THREADS = 1024;

template <typename real>
__global__ __launch_bounds__(CALL_THREADS) void k_begin_call(Ctx C, const double* __restrict__ gradL, int n_mean,
                                                             int clear) {
    if ((int)blockIdx.x >= n_mean) {
        const int b = (blockIdx.x - n_mean) * 64 + threadIdx.x / 16, sub = threadIdx.x % 16;
        if (b >= C.n_boxes) return;
        if (clear)
            for (int q = sub; q < ACC; q += 16) C.acc[ACC * (size_t)b + q] = 0.0;
        if (sub != 0) return;
        if (clear) C.acc_pairs[b] = 0ull;
        BoxDyn& D = C.dyn[b];
        double L[9];
        for (int k = 0; k < 9; ++k) L[k] = gradL[9 * (size_t)b + k];
        if (!gradient_ok(L)) {
            for (int k = 0; k < 9; ++k) L[k] = 0.0;
            C.flags[b] |= LHMM_FLAG_ARG;
        }
        if (D.hc > 0.0) {  // boundary regions: the gradient drives the ring, the cell stays fixed
            D.G[0] = L[0]; D.G[1] = L[1]; D.G[2] = L[3]; D.G[3] = L[4];
            for (int k = 0; k < 9; ++k) L[k] = 0.0;
        }
        for (int k = 0; k < 9; ++k) D.L[k] = L[k];
        expm_planar(L, C.dt, D.E);
        expm_planar(L, 0.5 * C.dt, D.Eh);
        return;
    }
    const int b = C.sel ? C.sel[blockIdx.x] : (int)blockIdx.x;
    const BoxInfo B = C.box[b];
    const int N = C.n_total;
    real* c = (real*)C.c + B.off;
    __shared__ double red[3][CALL_THREADS / 64];
    // thread t adds particles t, t + 1024, ... in that order, four particles'
    // loads in flight; then a fixed tree over the wave and the waves in order
    double acc[3] = {0.0, 0.0, 0.0};
    int i = threadIdx.x;
    for (; i + 3 * CALL_THREADS < B.n; i += 4 * CALL_THREADS) {
        real v[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < 3; ++k) v[u][k] = c[(long)k * N + i + u * CALL_THREADS];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < 3; ++k) acc[k] += (double)v[u][k];
    }
    for (; i < B.n; i += CALL_THREADS)
        for (int k = 0; k < 3; ++k) acc[k] += (double)c[(long)k * N + i];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o, 64);
        if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = acc[k];
    }
    __syncthreads();
    real mean[3];
    for (int k = 0; k < 3; ++k) {
        double t = 0.0;
        for (int w = 0; w < CALL_THREADS / 64; ++w) t += red[k][w];
        mean[k] = (real)(t / B.n);
    }
#pragma unroll 4
    for (int j = threadIdx.x; j < B.n; j += CALL_THREADS)
        for (int k = 0; k < 3; ++k) c[(long)k * N + j] -= mean[k];
}

// One box's cell from S to D (which may not alias).  advance = 1: mid-step
// inverse, deformation and reduction of a step; advance = 0: grid of the
// current cell only.  raise: the caller raises the box's cell flags (one
// caller per box and step).
__device__ void cell_step_box(const Ctx& C, int b, const BoxDyn& S, BoxDyn& D, int advance, bool raise) {
    D = S;
    double h[9];
    for (int k = 0; k < 9; ++k) h[k] = S.h[k];
    int U[4] = {1, 0, 0, 1};
    int changed = 0;
    if (advance) {
        double hm[9];
        m3_mul(S.Eh, h, hm);
        m3_inv(hm, D.hmi);
        m3_mul(S.E, h, h);
        changed = reduce_planar(h, U);
        for (int k = 0; k < 9; ++k) D.h[k] = h[k];
    }
    for (int k = 0; k < 4; ++k) D.U[k] = U[k];
    D.changed = changed;
    // the stress is averaged over the core of a boundary-region box
    D.vol = S.hc > 0.0 ? 4.0 * S.hc * S.hc * h[8] : fabs(m3_det(h));
    double w[3];
    m3_widths(h, w);
    int nc[3];
    const int zsub = C.box[b].zsub, zmin = 2 * zsub + 1;
    const bool narrow = cell_counts(w, C.rc, zsub, nc);
    const int cap = C.box[b].cell_cap;
    while ((long long)nc[0] * nc[1] * nc[2] > cap) {  // only reachable for a flagged (narrow) cell
        int a = nc[0] >= nc[1] ? 0 : 1;
        if (nc[a] <= 3) {
            if (nc[2] <= zmin) break;
            a = 2;
        }
        nc[a] -= 1;
    }
    if (raise) {
        if (narrow) C.flags[b] |= LHMM_FLAG_CELL;
        if (!(fmin(fmin(w[0], w[1]), w[2]) >= LHMM_THIN_WIDTH * C.rc)) C.flags[b] |= LHMM_FLAG_THIN;
    }
    D.nc[0] = nc[0]; D.nc[1] = nc[1]; D.nc[2] = nc[2];
}

template <typename real>
__device__ __forceinline__ void cell_coords(real s0, real s1, real s2, const int* nc, int& k0, int& k1, int& k2) {
    k0 = min(max((int)(s0 * (real)nc[0]), 0), nc[0] - 1);
    k1 = min(max((int)(s1 * (real)nc[1]), 0), nc[1] - 1);
    k2 = min(max((int)(s2 * (real)nc[2]), 0), nc[2] - 1);
}

template <typename real>
__device__ __forceinline__ int cell_of(real s0, real s1, real s2, const int* nc) {
    int k0, k1, k2;
    cell_coords(s0, s1, s2, nc, k0, k1, k2);
    return (k0 * nc[1] + k1) * nc[2] + k2;
}

// a / d for 0 <= a < 2^22 and d >= 1, given inv = 1.0f / d: single-precision
// rounding moves (a + 1/2) / d by less than the 1/(2d) it keeps from integers
__device__ __forceinline__ int div_small(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

template <typename real>
__device__ __forceinline__ real wrap01(real x) {
    x -= floor(x);
    return x >= (real)1 ? (real)0 : x;
}

// The ring of a boundary-region box (Eq. micro_bc): a particle at in-plane
// position (x, y) relative to the cell centre with hc <= max(|x|, |y|) < hb
// has its in-plane velocity relaxed toward the imposed field u = G r' over
// half a step, c <- u + (c - u) damp + amp xi, with the normal pair xi of
// Philox4x32-10 at counter (id, 0xFFFFFFF0 + half, step, box).
template <typename real>
__device__ __forceinline__ void ring_relax(real x, real y, real hc, real hb, const real (&G)[4], real damp, real amp,
                                           unsigned id, unsigned half, unsigned step, unsigned box, unsigned k0,
                                           unsigned k1, real& c0, real& c1) {
    const real mx = fmax(fabs(x), fabs(y));
    if (!(mx >= hc && mx < hb)) return;
    unsigned x0 = id, x1 = 0xFFFFFFF0u + half, x2 = step, x3 = box;
    philox4x32_10(x0, x1, x2, x3, k0, k1);
    real n0, n1;
    box_muller2<real>(x0, x1, n0, n1);
    const real u0 = fma(G[0], x, G[1] * y), u1 = fma(G[2], x, G[3] * y);
    c0 = fma(amp, n0, fma(c0 - u0, damp, u0));
    c1 = fma(amp, n1, fma(c1 - u1, damp, u1));
}

// A box's step constants for the half kick and drift, read once into
// registers (the per-particle stores could otherwise force reloads).
template <typename real>
struct KickDrift {
    real hdt, im, dt, L0, L1, L3, L4, M[9];
    int changed, U[4], nc[3];
    // boundary regions: half-widths, imposed gradient, the cell's in-plane
    // basis and random-stream words of the first half kick
    bool afbc;
    real hc, hb, G[4], h00, h01, h10, h11, damp, amp;
    unsigned step, box, k0, k1;
    __device__ explicit KickDrift(const Ctx& C, const BoxDyn& D, unsigned box_rng, unsigned step_made) {
        hdt = (real)(0.5 * C.dt);
        im = (real)C.inv_mass;
        dt = (real)C.dt;
        L0 = (real)D.L[0]; L1 = (real)D.L[1]; L3 = (real)D.L[3]; L4 = (real)D.L[4];
        for (int k = 0; k < 9; ++k) M[k] = (real)D.hmi[k];
        changed = D.changed;
        for (int k = 0; k < 4; ++k) U[k] = D.U[k];
        for (int k = 0; k < 3; ++k) nc[k] = D.nc[k];
        afbc = D.hc > 0.0;
        hc = (real)D.hc; hb = (real)D.hb;
        for (int k = 0; k < 4; ++k) G[k] = (real)D.G[k];
        h00 = (real)D.h[0]; h01 = (real)D.h[1]; h10 = (real)D.h[3]; h11 = (real)D.h[4];
        damp = (real)C.ou_damp; amp = (real)C.ou_amp;
        step = step_made;
        box = box_rng; k0 = C.key0; k1 = C.key1;
    }
};

// Half kick c += dt/2 (F/m - L c); in-plane L: (L c)_z = 0.
template <typename real>
__device__ __forceinline__ void half_kick(real hdt, real im, real L0, real L1, real L3, real L4, real f0, real f1,
                                          real f2, real& c0, real& c1, real& c2) {
    const real lc0 = fma(L0, c0, L1 * c1), lc1 = fma(L3, c0, L4 * c1);
    c0 = fma(hdt, fma(f0, im, -lc0), c0);
    c1 = fma(hdt, fma(f1, im, -lc1), c1);
    c2 = fma(hdt, f2 * im, c2);
}

// Half kick, drift of the fractional coordinate with
// the mid-step cell, remap after a reduction, wrap (in registers).  AF:
// the box may have boundary regions.  The integration's roundings are fixed by
// explicit fmas (here, in half_kick and in bond_forces): the launches that make
// a step, fused or not, then agree to the bit.
template <typename real, bool AF>
__device__ __forceinline__ void kick_drift(const KickDrift<real>& K, real (&sv)[3], real (&cv)[3], const real (&fv)[3],
                                           int id) {
    half_kick<real>(K.hdt, K.im, K.L0, K.L1, K.L3, K.L4, fv[0], fv[1], fv[2], cv[0], cv[1], cv[2]);
    if (AF && K.afbc) {
        const real x = fma(K.h00, sv[0] - (real)0.5, K.h01 * (sv[1] - (real)0.5));
        const real y = fma(K.h10, sv[0] - (real)0.5, K.h11 * (sv[1] - (real)0.5));
        ring_relax<real>(x, y, K.hc, K.hb, K.G, K.damp, K.amp, (unsigned)id, 0u, K.step, K.box, K.k0, K.k1, cv[0], cv[1]);
    }
    real s0 = fma(K.dt, fma(K.M[2], cv[2], fma(K.M[1], cv[1], K.M[0] * cv[0])), sv[0]);
    real s1 = fma(K.dt, fma(K.M[5], cv[2], fma(K.M[4], cv[1], K.M[3] * cv[0])), sv[1]);
    const real s2 = fma(K.dt, fma(K.M[8], cv[2], fma(K.M[7], cv[1], K.M[6] * cv[0])), sv[2]);
    if (K.changed) {  // s <- U^{-1} s in the plane, U^{-1} = [[u11, -u01], [-u10, u00]]
        const real x = s0, y = s1;
        s0 = fma((real)K.U[3], x, -((real)K.U[1] * y));
        s1 = fma((real)K.U[0], y, -((real)K.U[2] * x));
    }
    sv[0] = wrap01(s0); sv[1] = wrap01(s1); sv[2] = wrap01(s2);
}

// Position r = h s of a fractional coordinate in the in-plane cell, with a
// fixed rounding sequence (the binning and the force kernel must agree to
// the bit: a particle finds itself at distance exactly zero).
template <typename real>
__device__ __forceinline__ void cell_position(real s0, real s1, real s2, real h00, real h01, real h10, real h11,
                                              real h22, real& x, real& y, real& z) {
    x = fma(h01, s1, h00 * s0);
    y = fma(h11, s1, h10 * s0);
    z = h22 * s2;
}

// First launch of a chunk of steps, per work block: the box's cell step from
// slot 0 to slot 1 (by the block's first thread; the box's first block stores
// it), then, from the arrays in index order, the first step's half kick and
// drift (advance = 1) and every particle's records by index: (s, index) in
// sid[1], (c, cell) in cord, and its cell in key.
template <typename real>
__global__ __launch_bounds__(BS) void k_begin_chunk(Ctx C, int koff, int advance) {
    using R = Rec<real>;
    __shared__ BoxDyn D;
    const int blk = C.blk_list ? C.blk_list[blockIdx.x] : (int)blockIdx.x;
    const int b = C.blk_box[blk];
    const BoxInfo B = C.box[b];
    const bool first = blk == B.blk_off;
    const int i = C.blk_first[blk] + (int)threadIdx.x, N = C.n_total;
    const bool act = i < B.off + B.n;
    const real* s = (const real*)C.s;
    const real* c = (const real*)C.c;
    const real* f = (const real*)C.f;
    real sv[3] = {0, 0, 0}, cv[3] = {0, 0, 0}, fv[3] = {0, 0, 0};
    if (act)
        for (int a = 0; a < 3; ++a) {
            sv[a] = s[(size_t)a * N + i];
            cv[a] = c[(size_t)a * N + i];
            fv[a] = f[(size_t)a * N + i];
        }
    if (threadIdx.x == 0) cell_step_box(C, b, C.dyn[b], D, advance, first);
    __syncthreads();
    if (first)
        for (int q = threadIdx.x; q < (int)(sizeof(BoxDyn) / sizeof(int)); q += BS)
            ((int*)&C.dyn[(size_t)C.n_boxes + b])[q] = ((const int*)&D)[q];
    if (!act) return;
    const int local = i - B.off;
    if (advance) {
        const KickDrift<real> K(C, D, B.rng_id, (unsigned)(*C.step + (unsigned long long)koff + 1ull));
        kick_drift<real, true>(K, sv, cv, fv, local);
    }
    const int cell = cell_of(sv[0], sv[1], sv[2], D.nc);
    ((typename R::T*)C.sid[1])[i] = R::make(sv[0], sv[1], sv[2], local);
    ((typename R::T*)C.cord)[i] = R::make(cv[0], cv[1], cv[2], cell);
    C.key[i] = cell;
}

// Inclusive scans in registers over rows of 16 lanes and over the wave (six
// steps through LDS permutes, and wave totals read one by one, cost the
// binning 1 us a launch).
__device__ __forceinline__ int row_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // from 1, 2, 4 and 8 lanes below in the row
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
    return x;
}

// lane L of each row of 16, in all its lanes
template <int L>
__device__ __forceinline__ int row_lane(int x) {
    return __builtin_amdgcn_update_dpp(0, x, 0x150 + L, 0xF, 0xF, false);
}
template <int L>
__device__ __forceinline__ float row_lane(float x) {
    return __int_as_float(row_lane<L>(__float_as_int(x)));
}
template <int L>
__device__ __forceinline__ double row_lane(double x) {
    return __hiloint2double(row_lane<L>(__double2hiint(x)), row_lane<L>(__double2loint(x)));
}

__device__ __forceinline__ int wave_scan(int x) {
    x = row_scan(x);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // lane 15 of a row to rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // lane 31 to rows 2 and 3
    return x;
}

// Exclusive scan over k in [0, n) of val(k) by a workgroup of BT threads:
// each thread sums a run of consecutive k, the run totals are scanned
// (in the wave, then the wave totals), and each thread walks its run
// again calling out(k, sum of val(0 .. k-1)); out(n, total) once.  val(k)
// is read before out(k) is called, by the same thread.
template <int BT, class Val, class Out>
__device__ __forceinline__ void block_scan(int n, int* wsum /* BT / 64 */, Val val, Out out) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int per = (n + BT - 1) / BT;
    const int k0 = min((int)threadIdx.x * per, n), k1 = min(k0 + per, n);
    int run = 0;
    for (int k = k0; k < k1; ++k) run += val(k);
    const int x = wave_scan(run);
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    // the wave totals (16 at most), scanned by every wave
    const int sums = row_scan(lane < BT / 64 ? wsum[lane] : 0), w = __builtin_amdgcn_readfirstlane(wv);
    const int total = __builtin_amdgcn_readlane(sums, BT / 64 - 1);
    int excl = x - run + (w > 0 ? __builtin_amdgcn_readlane(sums, w - 1) : 0);
    __syncthreads();
    for (int k = k0; k < k1; ++k) {
        const int v = val(k);
        out(k, excl);
        excl += v;
    }
    if (threadIdx.x == 0) out(n, total);
}

// Binning: a counting sort of every box's particles by cell, each cell in
// index order so that all later sums have a fixed order.  A box is cut into
// slabs of consecutive cell columns (about SLAB_TARGET particles each), one
// workgroup per slab and no exchange between them: every workgroup reads the
// cells of all its box's particles (4 bytes each), counting those in earlier
// slabs (its base position, and the z images stored before it in the search
// layout) and, per cell, those in its own; then it ranks and moves its own
// particles only.  The source records are in the last step's cell order (in
// index order at a chunk's first step), so a wave's loads and stores fall on
// neighbouring records; they are loaded as soon as the slab's particles are
// known and arrive during the scans.  Written per particle: (x, y, z, index), (c, index) in
// cell order, the source position in perm, and (x, y, z, cell-order position)
// in the search layout, once more for the images of the bottom and top cells.
//
// One workgroup per box (the earlier form) took 19 us for 3000 particles,
// 67 us for a batch with boxes of 1.5k to 12k and 160 us for eight of 23k,
// which did not fit its LDS; the largest box set the time.  Now 8, 32 and
// 19 us: one chain of loads, scans and barriers for small launches, and for
// large boxes the reading of all keys by every slab.
//
// A slab holding more than SLAB_CAP particles (a very uneven density) orders
// its cells in global memory instead; the result is the same.
//
// The first n_cell workgroups, a thread per box, make the next step's cell
// (slot of this step -> the other slot) and note this step's volume.
// a coordinate beyond the cutoff of every particle of the cell
template <typename real>
__device__ __forceinline__ real far_away(const Ctx& C, const BoxDyn& D) {
    return (real)(1.0e6 * (C.rc + fabs(D.h[0]) + fabs(D.h[1]) + fabs(D.h[3]) + fabs(D.h[4]) + D.h[8]));
}

constexpr int SLAB_TARGET = 1024;  // particles per slab
constexpr int SLAB_CAP = 2048;     // particles a slab can order in LDS
constexpr int SLAB_CELLS = 4096;   // a box has at least cells / SLAB_CELLS slabs

template <typename real, int T>
__global__ __launch_bounds__(T) void k_bin(Ctx C, Step A, int n_cell, int lds_cells, int lds_cols) {
    using R = Rec<real>;
    using V4 = typename R::T;
    constexpr int PER = SLAB_CAP / T;
    extern __shared__ int lds[];
    __shared__ int wsum[T / 64];
    __shared__ int base[4];  // particles and images before the slab, images in it, its particles
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < n_cell) {
        const int q = blockIdx.x * T + tid;
        if (q >= (C.sel ? C.n_sel : C.n_boxes)) return;
        const int b = C.sel ? C.sel[q] : q;
        const BoxDyn& S = C.dyn[(size_t)A.slot * C.n_boxes + b];
        C.vol[(size_t)A.w * C.n_boxes + b] = S.vol;
        if (A.more) cell_step_box(C, b, S, C.dyn[(size_t)(A.slot ^ 1) * C.n_boxes + b], 1, true);
        return;
    }
    int* cnt = lds;                  // counts, starts, then ends of the slab's cells
    int* col_off = cnt + lds_cells;  // offsets from cell order to the search layout: the column's cells,
    int* lo_off = col_off + lds_cols;  // the image of its top cells below it,
    int* hi_off = lo_off + lds_cols;   // the image of its bottom cells above it
    int* own = hi_off + lds_cols;    // SLAB_CAP: source positions of the slab's particles, as found
    int* lid = own + SLAB_CAP;       // SLAB_CAP: particle indices by cell
    int slab = xcd_local_work(blockIdx.x - n_cell, gridDim.x - n_cell);
    if (C.slab_list) slab = C.slab_list[slab];
    const int b = C.slab_box[slab];
    const BoxInfo B = C.box[b];
    const BoxDyn& D = C.dyn[(size_t)A.slot * C.n_boxes + b];
    const int n2 = D.nc[2], zs = B.zsub, gs = n2 + 2 * zs + 1, ncol = D.nc[0] * D.nc[1];
    const int q = slab - B.slab_off;
    const int c0 = (int)((long long)q * ncol / B.nslab), c1 = (int)((long long)(q + 1) * ncol / B.nslab);
    const int nc = c1 - c0, s0 = c0 * n2, s1 = c1 * n2, ncell = nc * n2;
    if (nc == 0) return;  // fewer columns than slabs
    for (int k = tid; k < ncell; k += T) cnt[k] = 0;
    if (tid < 4) base[tid] = 0;
    __syncthreads();
    const float inv_n2 = 1.0f / (float)n2;
    const int* key = C.key + B.off;
    int before = 0, img = 0;
    int next[4];  // the keys after the four at hand
#pragma unroll
    for (int u = 0; u < 4; ++u) next[u] = key[min(tid + u * T, B.n - 1)];
    for (int k0 = tid; k0 - tid < B.n; k0 += 4 * T) {
        int cell[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            cell[u] = k0 + u * T < B.n ? next[u] : s1;
            next[u] = key[min(k0 + (4 + u) * T, B.n - 1)];
        }
        unsigned long long mine[4];
        int found = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned long long early = __ballot(cell[u] < s0);
            if (early) {  // the keys are nearly sorted: most waves have none, or only these
                const int z = cell[u] - div_small(cell[u], inv_n2) * n2;
                before += __popcll(early);
                img += __popcll(early & __ballot(z < zs)) + __popcll(early & __ballot(z >= n2 - zs));
            }
            mine[u] = __ballot(cell[u] < s1) & ~early;
            found += __popcll(mine[u]);
        }
        if (found == 0) continue;  // wave-uniform
        int e = 0;
        if ((tid & 63) == 0) e = atomicAdd(&base[3], found);
        e = __builtin_amdgcn_readfirstlane(e);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (mine[u] >> (tid & 63) & 1) {
                const int slot = e + __popcll(mine[u] & ((1ull << (tid & 63)) - 1));
                atomicAdd(&cnt[cell[u] - s0], 1);
                if (slot < SLAB_CAP) own[slot] = k0 + u * T;
            }
            e += __popcll(mine[u]);
        }
    }
    if ((tid & 63) == 0) {
        atomicAdd(&base[0], before);
        atomicAdd(&base[1], img);
    }
    __syncthreads();
    before = base[0];
    img = base[1];
    const int total = base[3];
    const bool fits = total <= SLAB_CAP;
    const V4* srcS = (const V4*)(A.first ? C.sid[A.slot] : C.sord[A.slot]) + B.off;
    const V4* srcC = (const V4*)C.cord + B.off;
    // the records of the slab's particles, on their way during the scans
    V4 S[PER], V[PER];
    int src[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = tid + u * T;
        src[u] = fits && e < total ? own[e] : -1;
        if (src[u] >= 0) {
            S[u] = srcS[src[u]];
            V[u] = srcC[src[u]];
        }
    }
    block_scan<T>(ncell, wsum, [&](int k) { return cnt[k]; }, [&](int k, int excl) { cnt[k] = excl; });
    __syncthreads();
    // images before each column (its top and bottom zsub cells' particles
    // appear once more), scanned over the slab's columns
    block_scan<T>(
        nc, wsum,
        [&](int col) {
            const int k = col * n2;
            return (cnt[k + n2] - cnt[k + n2 - zs]) + (cnt[k + zs] - cnt[k]);
        },
        [&](int col, int excl) {
            if (col == nc) {
                base[2] = excl;
                return;
            }
            const int k = col * n2;
            const int first = cnt[k] + img + excl + SREC_PAD * (c0 + col), top = cnt[k + n2] - cnt[k + n2 - zs];
            lo_off[col] = first - cnt[k + n2 - zs];
            col_off[col] = first + top - cnt[k];
            hi_off[col] = first + top + (cnt[k + n2] - cnt[k]) - cnt[k];
        });
    __syncthreads();
    // starts of the search-layout cells, a segment's offset plus the start of
    // the cell it repeats, and the columns' ends; padding after each end
    int* gstart = C.gcell_start + B.gcell_off + c0 * gs;
    const float inv_gs = 1.0f / (float)gs;
    V4* srec = (V4*)C.srec + B.srec_off;
    const real far = far_away<real>(C, D);
    for (int g = tid; g < nc * gs; g += T) {
        const int col = div_small(g, inv_gs), zg = g - col * gs, k = col * n2;
        gstart[g] = before + (zg < zs ? lo_off[col] + cnt[k + n2 - zs + zg]
                                      : (zg < zs + n2 ? col_off[col] + cnt[k + zg - zs] : hi_off[col] + cnt[k + zg - zs - n2]));
    }
    for (int g = tid; g < nc * SREC_PAD; g += T) {
        const int col = g / SREC_PAD;
        srec[before + hi_off[col] + cnt[col * n2 + zs] + g % SREC_PAD] = R::make(far, far, far, 0);
    }
    __syncthreads();
    int* perm = C.perm + B.off;
    // from here on cnt[k] counts up to the end of cell k
    if (fits) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (src[u] >= 0) lid[atomicAdd(&cnt[R::id(V[u]) - s0], 1)] = R::id(S[u]);
    } else {
        for (int k = tid; k < B.n; k += T) {
            const int cell = key[k];
            if (cell >= s0 && cell < s1) perm[before + atomicAdd(&cnt[cell - s0], 1)] = k;
        }
        __threadfence_block();
    }
    __syncthreads();
    V4* pv = (V4*)C.cell_pv + 2 * (size_t)B.off;
    const real h00 = (real)D.h[0], h01 = (real)D.h[1], h10 = (real)D.h[3], h11 = (real)D.h[4];
    const real h22 = (real)D.h[8];
    // particle `src` (records S, V) to cell-order position p (local to the slab)
    auto store = [&](int p, int src, const V4& S, const V4& V, int cell) {
        real x, y, z;
        cell_position<real>(S.x, S.y, S.z, h00, h01, h10, h11, h22, x, y, z);
        const int id = R::id(S), g = before + p;
        pv[2 * g] = R::make(x, y, z, id);
        pv[2 * g + 1] = R::make(V.x, V.y, V.z, id);
        perm[g] = src;
        const int col = div_small(cell, inv_n2), zc = cell - col * n2;
        V4* o = srec + before;
        o[p + col_off[col]] = R::make(x, y, z, g << 5);
        if (zc >= n2 - zs) o[p + lo_off[col]] = R::make(x, y, z - h22, (g << 5) | 9);
        if (zc < zs) o[p + hi_off[col]] = R::make(x, y, z + h22, (g << 5) | 18);
    };
    if (fits) {
        // a particle's position is its cell's start plus the number of its
        // cell's entries with a smaller index (a few each)
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (src[u] < 0) continue;
            const int cell = R::id(V[u]) - s0, id = R::id(S[u]);
            const int p0 = cell == 0 ? 0 : cnt[cell - 1], p1 = cnt[cell];
            int rank = 0;
            for (int p = p0; p < p1; ++p) rank += lid[p] < id;
            store(p0 + rank, src[u], S[u], V[u], cell);
        }
        return;
    }
    for (int k = tid; k < ncell; k += T) {
        const int p0 = before + (k == 0 ? 0 : cnt[k - 1]), p1 = before + cnt[k];
        for (int p = p0 + 1; p < p1; ++p) {  // insertion sort by index
            const int v = perm[p], id = R::id(srcS[v]);
            int r = p - 1;
            while (r >= p0 && R::id(srcS[perm[r]]) > id) {
                perm[r + 1] = perm[r];
                --r;
            }
            perm[r + 1] = v;
        }
    }
    __threadfence_block();
    __syncthreads();
    for (int p = tid; p < total; p += T) {
        const int src = perm[before + p];
        const V4 V = srcC[src];
        store(p, src, srcS[src], V, R::id(V) - s0);
    }
}

// In-plane image shift sh0 a + sh1 b of the cell's lattice vectors for the
// code ic = 3 (sh0 + 1) + (sh1 + 1) (0 .. 8), with a fixed rounding sequence:
// the search and the evaluation of a pair form the same separation.
template <typename real>
__device__ __forceinline__ void image_shift(int ic, real h00, real h01, real h10, real h11, real& sx, real& sy) {
    const int c0 = (ic * 11) >> 5;  // ic / 3 for 0 <= ic <= 8
    const real a = (real)(c0 - 1), b = (real)(ic - 3 * c0 - 1);
    sx = fma(h01, b, h00 * a);
    sy = fma(h11, b, h10 * a);
}

template <typename real>
__device__ __forceinline__ real inv_sqrt(real x);
template <>
__device__ __forceinline__ float inv_sqrt<float>(float x) { return __builtin_amdgcn_rsqf(x); }
template <>
__device__ __forceinline__ double inv_sqrt<double>(double x) { return 1.0 / sqrt(x); }

// Pair forces (Eqs. conservative, dissipative, random) and FENE bonds (Eq.
// fene_force).  Each lane owns one particle in cell order and sums that
// particle's force in registers, so every ordered pair is evaluated by its
// first particle's lane: no atomics, and a fixed summation order.
//   Search: the wave walks the nine stencil rows in step (z cells
//   k2 - zsub .. k2 + zsub of a row, periodic images included, are one
//   contiguous range of the search layout; with two cells per cutoff along z
//   the rows hold ~20% fewer candidates); each lane scans its own row range
//   SU records at a time (lanes of one home cell read the same records) and
//   appends each accepted neighbour (0 < r < rc; the particle itself has
//   r = 0) to its own LDS queue of QD four-byte entries: the neighbour's
//   cell-order position and its image code.  QD, `drain` and `busy` are
//   tuning parameters; none changes the order in which a lane evaluates its
//   neighbours, so results do not depend on them.
//   Evaluation: a round pops one queued neighbour per lane, reloads its
//   position and velocity records, re-forms the separation with the same
//   rounding as the search, and evaluates the pair (relative velocity
//   including the streaming difference L d, Philox normal, force, virial).
//   Rounds run when a queue could overflow, until every queue holds at most
//   `drain` entries (and while `busy` or more lanes have work), and the
//   queues are drained at the end.  Deep queues let most lanes hold work in
//   every round.
//   What bounds it (256 relaxed boxes, 1.5M particles, 164 us): a wave makes
//   ~5300 accesses to the vector cache, one per cycle and CU (28 for a search
//   step's 16-byte load, 64 for each of a round's two gathers), and issues 4235
//   vector instructions, both near the limit of the CU, so that what helped last
//   was waves to overlap them (64 registers, eight waves per SIMD, took 173 us
//   when six took 181): 6% fewer instructions, with the tests of a search step
//   scheduled apart, are no faster.  Evaluating a round without its branch (idle
//   lanes on a zero force) cost 2 us, loading only for lanes with records left
//   gained nothing.
// records tested per lane and search iteration for a queue of depth QD
__host__ __device__ constexpr int scan_unroll(int qd) { return qd >= 8 ? 4 : (qd >= 4 ? 2 : 1); }

// Fraction of the in-plane segment a + t e, t in [0, 1], inside the square
// |x|, |y| <= hc (the bond function of a weight uniform over a
// boundary-region box's core, times the core's volume).
template <typename real>
__device__ __forceinline__ real core_fraction(real ax, real ay, real ex, real ey, real hc) {
    real t0 = (real)0, t1 = (real)1;
    const real a[2] = {ax, ay}, e[2] = {ex, ey};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (e[k] == (real)0) {
            if (a[k] < -hc || a[k] > hc) return (real)0;
            continue;
        }
        real ta = (-hc - a[k]) / e[k], tb = (hc - a[k]) / e[k];
        if (ta > tb) {
            const real x = ta;
            ta = tb;
            tb = x;
        }
        t0 = fmax(t0, ta);
        t1 = fmin(t1, tb);
    }
    return t1 > t0 ? t1 - t0 : (real)0;
}

// PRUNE selects the stencil-pruning variant.  COMP keeps the virials of the
// conservative, dissipative and random forces apart as well (their sum is
// accumulated as in the default variant), at the cost of 18 more registers.
// AF handles boxes with boundary regions: each pair's and bond's virial is
// weighted by the fraction of its segment inside the core, and the second
// half kick relaxes the ring toward the imposed field; the core's kinetic
// sums use the velocity relative to that field.

// One ordered pair: separation d, unit vector e, magnitude of the force on i
// along e, force g; wR, ev, th are its factors.
template <typename real>
struct PairOut {
    real ex, ey, ez, mag, gx, gy, gz, wR, ev, th;
};

// The part of pair_force below the separation (dx, dy, dz): v the relative
// velocity without the streaming difference L d.
template <typename real>
struct PairConst {
    real a, gam, sig, irc, L00, L01, L10, L11;
    unsigned step, box, k0, k1;
};

template <typename real>
__device__ __forceinline__ PairOut<real> pair_force(const PairConst<real>& P, real dx, real dy, real dz, real ci0,
                                                    real ci1, real ci2, real cj0, real cj1, real cj2, unsigned id_i,
                                                    unsigned id_j) {
    PairOut<real> o;
    const real r2 = fma(dz, dz, fma(dx, dx, dy * dy));  // fixed association
    const real ir = inv_sqrt(r2);
    const real r = r2 * ir;
    o.ex = dx * ir; o.ey = dy * ir; o.ez = dz * ir;
    o.wR = (real)1 - r * P.irc;
    const real vx = ci0 - cj0 + P.L00 * dx + P.L01 * dy;
    const real vy = ci1 - cj1 + P.L10 * dx + P.L11 * dy;
    const real vz = ci2 - cj2;
    o.ev = o.ex * vx + o.ey * vy + o.ez * vz;
    o.th = pair_theta<real>(id_i, id_j, P.step, P.box, P.k0, P.k1);
    o.mag = o.wR * (P.a - P.gam * o.wR * o.ev + P.sig * o.th);
    o.gx = o.mag * o.ex; o.gy = o.mag * o.ey; o.gz = o.mag * o.ez;
    return o;
}

// FENE springs of a bead to its chain neighbours: their forces added to f,
// each bond's virial once (by its lower bead) to wf; S: (s, index) by index of
// the box.  wgt(dx, dy): weight of a bond's virial.
template <typename real, class Wgt>
__device__ __forceinline__ void bond_forces(const Ctx& C, int b, int id, const typename Rec<real>::T* S, real h00,
                                            real h01, real h10, real h11, real h22, real& fx, real& fy, real& fz,
                                            real (&wf)[6], Wgt wgt) {
    const typename Rec<real>::T si = S[id];
    const int bead = id % C.chain_len;
    const real Hf = (real)C.H, iR02 = (real)C.inv_R02;
    for (int side = 0; side < 2; ++side) {
        if (side == 0 && bead == 0) continue;
        if (side == 1 && bead == C.chain_len - 1) continue;
        const typename Rec<real>::T sj = S[side == 0 ? id - 1 : id + 1];
        real ds0 = si.x - sj.x, ds1 = si.y - sj.y, ds2 = si.z - sj.z;
        ds0 -= rint(ds0); ds1 -= rint(ds1); ds2 -= rint(ds2);
        const real dx = fma(h00, ds0, h01 * ds1), dy = fma(h10, ds0, h11 * ds1), dz = h22 * ds2;
        real den = fma(-fma(dz, dz, fma(dx, dx, dy * dy)), iR02, (real)1);
        if (den <= (real)0) atomicOr(&C.flags[b], LHMM_FLAG_BOND);
        if (den < (real)0.01) den = (real)0.01;
        const real k = -Hf / den;
        fx = fma(k, dx, fx); fy = fma(k, dy, fy); fz = fma(k, dz, fz);
        if (side == 1) {
            const real gx = k * dx, gy = k * dy, gz = k * dz;
            const real w = wgt(dx, dy);
            const real dxw = dx * w, dyw = dy * w, dzw = dz * w;
            wf[0] = fma(dxw, gx, wf[0]); wf[1] = fma(dyw, gy, wf[1]); wf[2] = fma(dzw, gz, wf[2]);
            wf[3] = fma(dxw, gy, wf[3]); wf[4] = fma(dxw, gz, wf[4]); wf[5] = fma(dyw, gz, wf[5]);
        }
    }
}

// The end of a particle's step: second half kick of the velocity-Verlet step,
// c += dt/2 (F/m - L c), with its final force; the kinetic sums m c c in
// kin; then either the next step's half kick and drift with that step's cell
// Dn, written at its cell-order position (and by index for a bead), or, after
// the chunk's last step, position, velocity and force in index order.
template <typename real, bool AF>
__device__ __forceinline__ void end_step(const Ctx& C, const Step& A, const BoxInfo& B, const BoxDyn& D,
                                         const BoxDyn& Dn, int pos, int id, real s0, real s1, real s2, real c0,
                                         real c1, real c2, real fx, real fy, real fz, real L00, real L01, real L10,
                                         real L11, unsigned stepc, bool store, double (&kin)[6]) {
    using R = Rec<real>;
    using V4 = typename R::T;
    const bool afbc = AF && D.hc > 0.0;
    const int N = C.n_total, i = B.off + id;
    const real hdt = (real)(0.5 * C.dt), im = (real)C.inv_mass;
    half_kick<real>(hdt, im, L00, L01, L10, L11, fx, fy, fz, c0, c1, c2);
    bool in_core = true;
    real u0 = (real)0, u1 = (real)0;  // imposed field at the particle (boundary regions)
    if (afbc) {
        const real h00 = (real)D.h[0], h01 = (real)D.h[1], h10 = (real)D.h[3], h11 = (real)D.h[4], hcr = (real)D.hc;
        const real x = fma(h00, s0 - (real)0.5, h01 * (s1 - (real)0.5));
        const real y = fma(h10, s0 - (real)0.5, h11 * (s1 - (real)0.5));
        const real G[4] = {(real)D.G[0], (real)D.G[1], (real)D.G[2], (real)D.G[3]};
        ring_relax<real>(x, y, hcr, (real)D.hb, G, (real)C.ou_damp, (real)C.ou_amp, (unsigned)id, 1u, stepc, B.rng_id,
                         C.key0, C.key1, c0, c1);
        in_core = fmax(fabs(x), fabs(y)) < hcr;
        u0 = fma(G[0], x, G[1] * y);
        u1 = fma(G[2], x, G[3] * y);
    }
    if (in_core) {
        const double mm = C.mass, x = (double)(c0 - u0), y = (double)(c1 - u1), z = (double)c2;
        kin[0] = mm * x * x; kin[1] = mm * y * y; kin[2] = mm * z * z;
        kin[3] = mm * x * y; kin[4] = mm * x * z; kin[5] = mm * y * z;
    }
    if (!store) return;
    if (!A.more) {
        real* s = (real*)C.s;
        real* c = (real*)C.c;
        real* f = (real*)C.f;
        s[i] = s0; s[(size_t)N + i] = s1; s[2 * (size_t)N + i] = s2;
        c[i] = c0; c[(size_t)N + i] = c1; c[2 * (size_t)N + i] = c2;
        f[i] = fx; f[(size_t)N + i] = fy; f[2 * (size_t)N + i] = fz;
        return;
    }
    real sv[3] = {s0, s1, s2}, cv[3] = {c0, c1, c2};
    const real fv[3] = {fx, fy, fz};
    const KickDrift<real> K(C, Dn, B.rng_id, stepc + 1u);
    kick_drift<real, AF>(K, sv, cv, fv, id);
    const int cell = cell_of(sv[0], sv[1], sv[2], K.nc), ns = A.slot ^ 1;
    const V4 rec = R::make(sv[0], sv[1], sv[2], id);
    ((V4*)C.sord[ns])[B.off + pos] = rec;
    ((V4*)C.cord)[B.off + pos] = R::make(cv[0], cv[1], cv[2], cell);
    C.key[B.off + pos] = cell;
    if (id < B.n_beads) ((V4*)C.sid[ns])[i] = rec;
}

// FLAT: some box may be too flat for its stencil (see the scan state).
template <typename real, int QD, bool PRUNE, bool COMP = false, bool AF = false, bool FLAT = false>
__global__ __launch_bounds__(BS, sizeof(real) == 4 ? (QD >= 32 || (COMP && AF) ? 4 : (COMP || AF || PRUNE || FLAT ? 5 : 8)) : 1) void k_forces(
    Ctx C, Step A, int drain, int busy) {
    constexpr bool prune = PRUNE;
    constexpr int NV = COMP ? 37 : 19;  // block partial sums
    using R = Rec<real>;
    using V4 = typename R::T;
    constexpr int NW = BS / 64;
    constexpr int SU = scan_unroll(QD);
    // queue entry: cell-order position of j << 5 | image code, the code
    // 9 x z image (0 none, 1 below, 2 above) + in-plane image code (0 .. 8)
    __shared__ int qbuf[QD][NW][64];
    __shared__ double red[NV * NW];
    // per image code (0 .. 26) the shift of the block's box: in-plane
    // image_shift, and 0, -h22 or +h22 along z
    __shared__ real shift_tab[32][4];

    const int work = xcd_local_work(blockIdx.x, gridDim.x);
    const int blk = C.blk_list ? C.blk_list[work] : work;
    const int b = C.blk_box[blk];
    const BoxInfo B = C.box[b];
    const BoxDyn& D = C.dyn[(size_t)A.slot * C.n_boxes + b];
    const int t = threadIdx.x, wv = t >> 6, lane = t & 63;
    const int p0 = C.blk_first[blk] - B.off;  // first cell-order position of the block
    const int pos = p0 + t;
    const bool act = pos < B.n;
    const V4* pv = (const V4*)C.cell_pv + 2 * (size_t)B.off;
    const char* sbase = (const char*)((const V4*)C.srec + B.srec_off);
    const __amdgpu_buffer_rsrc_t srsrc = rec_rsrc(sbase);
    const V4* srcS = (const V4*)(A.first ? C.sid[A.slot] : C.sord[A.slot]) + B.off;

    // in-plane cell and gradient
    const real h00 = (real)D.h[0], h01 = (real)D.h[1], h10 = (real)D.h[3], h11 = (real)D.h[4];
    const real h22 = (real)D.h[8];
    if (t < 27) {
        image_shift<real>(t % 9, h00, h01, h10, h11, shift_tab[t][0], shift_tab[t][1]);
        shift_tab[t][2] = t < 9 ? (real)0 : (t < 18 ? -h22 : h22);
    }
    __syncthreads();
    real ri0 = 0, ri1 = 0, ri2 = 0, ci0 = 0, ci1 = 0, ci2 = 0;
    real own_s0 = 0, own_s1 = 0, own_s2 = 0;
    int own_id = 0, src = 0;
    if (act) {
        const V4 u = pv[2 * pos + 1];
        ci0 = u.x; ci1 = u.y; ci2 = u.z;
        own_id = R::id(u);
        src = C.perm[B.off + pos];
        const V4 S = srcS[src];
        own_s0 = S.x; own_s1 = S.y; own_s2 = S.z;
        cell_position<real>(own_s0, own_s1, own_s2, h00, h01, h10, h11, h22, ri0, ri1, ri2);
    }
    const real L00 = (real)D.L[0], L01 = (real)D.L[1], L10 = (real)D.L[3], L11 = (real)D.L[4];
    // boundary regions: core half-width, the cell centre (r' = r - centre)
    const bool afbc = AF && D.hc > 0.0;
    const real hcr = AF ? (real)D.hc : (real)0;
    const real cx = AF ? (real)(0.5 * (D.h[0] + D.h[1])) : (real)0, cy = AF ? (real)(0.5 * (D.h[3] + D.h[4])) : (real)0;
    const int n0 = D.nc[0], n1 = D.nc[1], n2 = D.nc[2], zs = B.zsub;
    const real dzc = h22 / (real)n2;  // cell height
    auto sqr = [](real x) { return x * x; };
    const unsigned stepc = (unsigned)(*C.step + (unsigned long long)A.k);
    const PairConst<real> P{(real)C.a, (real)C.gamma, (real)(C.sigma * C.rdt), (real)(1.0 / C.rc), L00, L01, L10, L11,
                            stepc, B.rng_id, C.key0, C.key1};
    const real rc2 = (real)C.rc2;
    const int* gstart = C.gcell_start + B.gcell_off;

    int k0 = 0, k1 = 0, k2 = 0;
    if (act) cell_coords(own_s0, own_s1, own_s2, D.nc, k0, k1, k2);  // as the binning found it
    // Stencil pruning: distances from the particle to the planes bounding
    // its cell (fractional gap x perpendicular width of the cell); any point
    // of a neighbour cell across such a plane is at least that far away.  A
    // row (d0, d1) is skipped when its in-plane lower bound g reaches the
    // cutoff, and its cells below / above the particle's z cell are scanned
    // only if they may hold a point within sqrt(rc^2 - g^2).  Bounds are
    // compared with a 0.1% larger cutoff, so no pair within rc is dropped
    // and the scan order of the kept candidates is unchanged.
    real gl0 = 0, gh0 = 0, gl1 = 0, gh1 = 0, zl = 0, zh = 0;
    const real rcp2 = prune ? (real)(1.002 * C.rc2) : (real)0;
    if (act && prune) {
        const real s0 = own_s0, s1 = own_s1, s2 = own_s2;
        const real area = fabs(h00 * h11 - h01 * h10);
        const real w0 = area / sqrt(h01 * h01 + h11 * h11), w1 = area / sqrt(h00 * h00 + h10 * h10);
        const real f0 = s0 * (real)n0 - (real)k0, f1 = s1 * (real)n1 - (real)k1, f2 = s2 * (real)n2 - (real)k2;
        gl0 = fmax(f0, (real)0) * w0 / (real)n0;
        gh0 = fmax((real)1 - f0, (real)0) * w0 / (real)n0;
        gl1 = fmax(f1, (real)0) * w1 / (real)n1;
        gh1 = fmax((real)1 - f1, (real)0) * w1 / (real)n1;
        zl = fmax(f2, (real)0) * h22 / (real)n2;
        zh = fmax((real)1 - f2, (real)0) * h22 / (real)n2;
    }
    // this lane's queue: entries popped and pushed, counted in queue rows
    // (NW x 64 ints) so that an entry's LDS byte address is one and-or of the
    // count with the lane's offset
    constexpr unsigned QROW = NW * 64 * sizeof(int), QMASK = (QD - 1) * QROW;
    const unsigned qlane = (unsigned)t * sizeof(int);
    char* const qbase = (char*)&qbuf[0][0][0];
    unsigned qh = 0, qt = 0;
    real fx = 0, fy = 0, fz = 0;
    real w[6] = {0, 0, 0, 0, 0, 0};
    real wc[COMP ? 6 : 1] = {}, wd[COMP ? 6 : 1] = {}, wr[COMP ? 6 : 1] = {};  // C, D, R parts

    int ic = 4;  // in-plane image code of the row being scanned
    // one evaluation round: each lane with a queued neighbour takes the oldest
    auto round = [&]() {
        if (qt > qh) {
            const int e = *(const int*)(qbase + ((qh & QMASK) | qlane));
            qh += QROW;
            // one 32-bit byte offset from the box's records (scalar base)
            const unsigned po = ((unsigned)e >> 5) * (unsigned)(2 * sizeof(V4));
            const V4 pj = *(const V4*)((const char*)pv + po);
            const V4 cj = *(const V4*)((const char*)pv + po + sizeof(V4));
            const int code = e & 31;
            const real sx = shift_tab[code][0], sy = shift_tab[code][1];
            // the z image: one rounding of z + (0, -h22, +h22), the same as the
            // binning's z - h22, z + h22
            const real zj = pj.z + shift_tab[code][2];
            const real dx = (ri0 - sx) - pj.x, dy = (ri1 - sy) - pj.y, dz = ri2 - zj;
            const PairOut<real> o = pair_force<real>(P, dx, dy, dz, ci0, ci1, ci2, cj.x, cj.y, cj.z, (unsigned)own_id,
                                                     (unsigned)R::id(cj));
            const real ex = o.ex, ey = o.ey, ez = o.ez, gx = o.gx, gy = o.gy, gz = o.gz;
            fx = fma(o.mag, ex, fx); fy = fma(o.mag, ey, fy); fz = fma(o.mag, ez, fz);
            // a boundary-region box weighs the pair by its segment's share of the core
            const real wgt = afbc ? core_fraction<real>(ri0 - cx, ri1 - cy, -dx, -dy, hcr) : (real)1;
            const real dxw = AF ? dx * wgt : dx, dyw = AF ? dy * wgt : dy, dzw = AF ? dz * wgt : dz;
            w[0] = fma(dxw, gx, w[0]); w[1] = fma(dyw, gy, w[1]); w[2] = fma(dzw, gz, w[2]);
            w[3] = fma(dxw, gy, w[3]); w[4] = fma(dxw, gz, w[4]); w[5] = fma(dyw, gz, w[5]);
            if constexpr (COMP) {
                // d (x) e times each force's magnitude
                const real mc = o.wR * P.a, md = -(o.wR * P.gam * o.wR * o.ev), mr = o.wR * P.sig * o.th;
                const real de[6] = {dxw * ex, dyw * ey, dzw * ez, dxw * ey, dxw * ez, dyw * ez};
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    wc[k] = fma(mc, de[k], wc[k]);
                    wd[k] = fma(md, de[k], wd[k]);
                    wr[k] = fma(mr, de[k], wr[k]);
                }
            }
        }
    };
    // test one candidate record v against (bx, by, ri2), the lane's position
    // minus the image shift of the range scanned; queue it if accepted
    real bx = 0, by = 0;
    auto push = [&](const V4& v) {
        const real dx = bx - v.x, dy = by - v.y, dz = ri2 - v.z;
        // the acceptance test's rounding is fixed by explicit fmas, whatever the
        // surrounding code lets the compiler contract
        const real r2 = fma(dz, dz, fma(dy, dy, dx * dx));
        // one branch per candidate: the tests combined without short-circuit
        if ((r2 < rc2) & (r2 > (real)0)) {
            const unsigned at = (qt & QMASK) | qlane;
            asm volatile("" : "+v"(qt) : "v"(at));  // the address first, so the count advances in place
            *(int*)(qbase + at) = R::id(v) + ic;
            qt += QROW;
        }
    };

    // Scan state: the wave is at stencil row `row` (d0, d1); each lane scans
    // the search-layout records from byte q to byte qe (z cells k2 - zsub ..
    // k2 + zsub of the row's column, the periodic images included).
    // Up to SREC_PAD records past a range's end are the column's next z cells, at
    // least the cutoff away along z where zsub cells span it, or the column's
    // padding: they need no test of their own, and a lane whose range has ended
    // stays at its end.  In a box too flat for that (flagged) they may lie within
    // it: one record per iteration, none at the end of the range (it would be
    // queued again for as long as another lane of the wave scans).  A variant of
    // its own: in the common kernel, whose 64 registers are all taken, most forms
    // of that branch spilled and cost the batch 4 to 9%.  A lane that scans
    // nothing (no particle, a pruned row) tests from far away.
    int row = 0;
    unsigned q = 0, qe = 0;
    const bool spans = !FLAT || z_cells_span(D.h[8], zs, n2, C.rc);
    const real far = far_away<real>(C, D);
    auto set_range = [&]() {
        const int d0 = row / 3 - 1, d1 = row % 3 - 1;
        int m0 = k0 + d0, m1 = k1 + d1;
        const int i0 = m0 < 0 ? 0 : (m0 >= n0 ? 6 : 3), i1 = m1 < 0 ? 0 : (m1 >= n1 ? 2 : 1);
        m0 += m0 < 0 ? n0 : (m0 >= n0 ? -n0 : 0);
        m1 += m1 < 0 ? n1 : (m1 >= n1 ? -n1 : 0);
        // cells and columns are below 2^24 (MAX_CELLS_PER_BOX)
        const int gb = __mul24(__mul24(m0, n1) + m1, n2 + 2 * zs + 1) + k2;
        ic = i0 + i1;
        bx = ri0 - shift_tab[ic][0];
        by = ri1 - shift_tab[ic][1];
        int lo = 0, hi = 2 * zs + 1;
        bool live = act;
        if (act && prune) {
            const real ga = d0 < 0 ? gl0 : (d0 > 0 ? gh0 : (real)0);
            const real gb2 = d1 < 0 ? gl1 : (d1 > 0 ? gh1 : (real)0);
            const real g = fmax(ga, gb2);
            const real zmax2 = rcp2 - g * g;
            live = zmax2 > (real)0;
            // z cells below (above) the particle's, farthest first
            for (int j = zs; j >= 1 && !(sqr(zl + (real)(j - 1) * dzc) < zmax2); --j) ++lo;
            for (int j = zs; j >= 1 && !(sqr(zh + (real)(j - 1) * dzc) < zmax2); --j) --hi;
        }
        if constexpr (prune) {
            q = qe = 0u;
            if (!live) bx = far;
            if (live) {
                q = (unsigned)gstart[gb + lo] * (unsigned)sizeof(V4);
                qe = (unsigned)gstart[gb + hi] * (unsigned)sizeof(V4);
            }
        } else {
            q = (unsigned)gstart[(unsigned)gb] * (unsigned)sizeof(V4);
            qe = (unsigned)gstart[(unsigned)(gb + 2 * zs + 1)] * (unsigned)sizeof(V4);
        }
    };
    if (!act) ri0 = far;
    set_range();
    unsigned qfull = (QD - SU) * QROW;  // pushed entries beyond which the queue may not take SU more
    bool scanning = true;               // wave-uniform
    while (true) {
        // search until the stencil is done or some queue might not take SU more
        while (scanning) {
            if (__ballot(q < qe) == 0ull) {
                if (++row == 9) {
                    scanning = false;
                    break;
                }
                set_range();
                continue;
            }
            // SU records per lane per iteration, all loads issued before the
            // first test, addressed by one 32-bit byte offset from the box's
            // records
            if (spans) {
                V4 cand[SU];
#pragma unroll
                for (int u = 0; u < SU; ++u) cand[u] = load_rec<real>(srsrc, sbase, q + u * (unsigned)sizeof(V4));
#pragma unroll
                for (int u = 0; u < SU; ++u) push(cand[u]);
                q = min(q + SU * (unsigned)sizeof(V4), qe);
            } else if (q < qe) {
                push(load_rec<real>(srsrc, sbase, q));
                q += (unsigned)sizeof(V4);
            }
            // evaluate when a queue may not take SU more, or when enough
            // lanes hold a neighbour for a well-filled round
            if (__ballot(qt > qfull) != 0ull) break;
            if (busy <= 64 && __popcll(__ballot(qt > qh)) >= busy) break;
        }
        // evaluate until every queue holds at most `drain` entries (none once
        // the stencil is done) and fewer than `busy` lanes hold one
        const unsigned keep = scanning ? (unsigned)drain * QROW : 0u;
        do {
            round();
        } while (__ballot(qt - qh > keep) != 0ull || (busy <= 64 && __popcll(__ballot(qt > qh)) >= busy));
        if (!scanning) break;
        qfull = qh + (QD - SU) * QROW;
    }
    if (!act) ri0 = 0;

    real wf[6] = {0, 0, 0, 0, 0, 0};
    if (act && own_id < B.n_beads)
        bond_forces<real>(C, b, own_id, (const V4*)C.sid[A.slot] + B.off, h00, h01, h10, h11, h22, fx, fy, fz, wf,
                          [&](real dx, real dy) { return afbc ? core_fraction<real>(ri0 - cx, ri1 - cy, -dx, -dy, hcr) : (real)1; });
    double v[NV];
    for (int k = 0; k < 6; ++k) {
        v[k] = (double)w[k];
        v[6 + k] = (double)wf[k];
        v[13 + k] = 0.0;
        if constexpr (COMP) {
            v[19 + k] = (double)wc[k];
            v[25 + k] = (double)wd[k];
            v[31 + k] = (double)wr[k];
        }
    }
    v[12] = (double)(qt / QROW);  // every queued neighbour was evaluated once
    if (act && A.kick) {
        const V4 S = srcS[src];  // read again rather than held through the search
        double kin[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        end_step<real, AF>(C, A, B, D, C.dyn[(size_t)(A.slot ^ 1) * C.n_boxes + b], pos, own_id, S.x, S.y, S.z, ci0, ci1,
                           ci2, fx, fy, fz, L00, L01, L10, L11, stepc, true, kin);
        for (int k = 0; k < 6; ++k) v[13 + k] = kin[k];
    } else if (act) {
        real* f = (real*)C.f;
        const int i = B.off + own_id, N = C.n_total;
        f[i] = fx; f[(size_t)N + i] = fy; f[2 * (size_t)N + i] = fz;
    }
    block_sum<NV>(v, red, C.part + (size_t)A.w * C.part_step + (size_t)(A.part0 + work) * NV);
}

// The force pass for launches too small to fill the chip, where the lone
// waves of k_forces wait for their ~37 dependent search loads and ~20 serial
// evaluation rounds (32 us however few particles).  Sixteen lanes own one
// particle: nine of them search a stencil row each, then all evaluate one
// neighbour each, and one lane per component adds the results in the order
// k_forces adds them (row by row, in cell order), so the sums are the same to
// the bit.  A workgroup takes the sixteen particles l = r + 4 j of a wave's 64
// (r = 0 .. 3): their partial sums are a subtree of k_forces's wave sum.
// Slower per particle (four particles per wave), so only for at most
// WIDE_BLOCKS work blocks.  FP32 boxes of 3072 particles, us a step with the
// wide kernel and with k_forces: 12 blocks 18.9 and 41.3, 96 blocks 25.9 and
// 36.3, 192 blocks 35.7 and 37.1, 252 blocks 41.5 and 40.8, 312 blocks 46.9
// and 43.1.
constexpr int WIDE_UNITS = 16;    // workgroups per work block
constexpr int WIDE_BLOCKS = 256;  // largest launch, in work blocks
constexpr int WIDE_ROW = 12;      // accepted neighbours per row that LDS holds

// Make a wave's LDS writes visible to its other lanes: one wave's LDS
// operations execute in order, so only the compiler has to keep it.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename real, bool COMP>
__global__ __launch_bounds__(BS) void k_forces_wide(Ctx C, Step A) {
    using R = Rec<real>;
    using V4 = typename R::T;
    constexpr int NV = COMP ? 37 : 19;
    constexpr int NF = COMP ? 19 : 10;   // values per evaluated pair
    constexpr int NA = COMP ? 27 : 9;    // summed components
    constexpr int PS = 20;               // stride of a value's 16 entries (16-byte reads)
    __shared__ real shift_tab[32][4];
    __shared__ int rowq[16][9][WIDE_ROW];
    __shared__ int list[16][9 * WIDE_ROW];
    __shared__ __align__(16) real res[16][NF][PS];
    __shared__ double vals[16][NV];

    const int unit = xcd_local_work(blockIdx.x, gridDim.x), work = unit / WIDE_UNITS, sub = unit % WIDE_UNITS;
    const int blk = C.blk_list ? C.blk_list[work] : work;
    const int b = C.blk_box[blk];
    const BoxInfo B = C.box[b];
    const BoxDyn& D = C.dyn[(size_t)A.slot * C.n_boxes + b];
    const int t = threadIdx.x, a = t & 15, p = t >> 4;  // lane of the particle, particle of the workgroup
    const int gbase = (t & 63) & ~15;                   // first lane of the particle in its wave
    const int pos = C.blk_first[blk] - B.off + 64 * (sub >> 2) + (sub & 3) + 4 * p;
    const bool act = pos < B.n;
    const V4* pv = (const V4*)C.cell_pv + 2 * (size_t)B.off;
    const char* sbase = (const char*)((const V4*)C.srec + B.srec_off);
    const __amdgpu_buffer_rsrc_t srsrc = rec_rsrc(sbase);
    const V4* srcS = (const V4*)(A.first ? C.sid[A.slot] : C.sord[A.slot]) + B.off;
    const real h00 = (real)D.h[0], h01 = (real)D.h[1], h10 = (real)D.h[3], h11 = (real)D.h[4];
    const real h22 = (real)D.h[8];
    if (t < 27) {
        image_shift<real>(t % 9, h00, h01, h10, h11, shift_tab[t][0], shift_tab[t][1]);
        shift_tab[t][2] = t < 9 ? (real)0 : (t < 18 ? -h22 : h22);
    }
    __syncthreads();
    real ri0 = 0, ri1 = 0, ri2 = 0, ci0 = 0, ci1 = 0, ci2 = 0, s0 = 0, s1 = 0, s2 = 0;
    int own_id = 0;
    if (act) {
        const V4 u = pv[2 * pos + 1];
        ci0 = u.x; ci1 = u.y; ci2 = u.z;
        own_id = R::id(u);
        const V4 S = srcS[C.perm[B.off + pos]];
        s0 = S.x; s1 = S.y; s2 = S.z;
        cell_position<real>(s0, s1, s2, h00, h01, h10, h11, h22, ri0, ri1, ri2);
    }
    const real L00 = (real)D.L[0], L01 = (real)D.L[1], L10 = (real)D.L[3], L11 = (real)D.L[4];
    const int n0 = D.nc[0], n1 = D.nc[1], n2 = D.nc[2], zs = B.zsub;
    const unsigned stepc = (unsigned)(*C.step + (unsigned long long)A.k);
    const PairConst<real> P{(real)C.a, (real)C.gamma, (real)(C.sigma * C.rdt), (real)(1.0 / C.rc), L00, L01, L10, L11,
                            stepc, B.rng_id, C.key0, C.key1};
    const real rc2 = (real)C.rc2;
    const int* gstart = C.gcell_start + B.gcell_off;
    int k0 = 0, k1 = 0, k2 = 0;
    if (act) cell_coords(s0, s1, s2, D.nc, k0, k1, k2);
    // the search-layout range of stencil row `row`, its image code, and the
    // particle's position less the row's in-plane image shift
    auto row_range = [&](int row, int& q, int& qe, int& ic, real& bx, real& by) {
        const int d0 = row / 3 - 1, d1 = row % 3 - 1;
        int m0 = k0 + d0, m1 = k1 + d1;
        const int sh0 = m0 < 0 ? -1 : (m0 >= n0 ? 1 : 0);
        const int sh1 = m1 < 0 ? -1 : (m1 >= n1 ? 1 : 0);
        m0 -= sh0 * n0;
        m1 -= sh1 * n1;
        const int gb = (m0 * n1 + m1) * (n2 + 2 * zs + 1) + k2;
        ic = 3 * (sh0 + 1) + (sh1 + 1);
        bx = ri0 - shift_tab[ic][0];
        by = ri1 - shift_tab[ic][1];
        q = gstart[gb];
        qe = gstart[gb + 2 * zs + 1];
    };
    auto accepted = [&](const V4& v, real bx, real by) {
        const real dx = bx - v.x, dy = by - v.y, dz = ri2 - v.z;
        const real r2 = fma(dz, dz, fma(dy, dy, dx * dx));
        return (r2 < rc2) & (r2 > (real)0);
    };
    // summed components: force 3, virial 6 (C, D, R virials 6 each) as sums of
    // products of two of an entry's values: mag e, d g (and mc, md, mr with d e)
    auto factors = [](int c, int& fa, int& fb) {
        if (c < 3) {
            fa = 0;
            fb = 1 + c;
            return;
        }
        const int k = (c - 3) % 6, part = (c - 3) / 6;
        const int ia = k < 3 ? k : (k == 5 ? 1 : 0), ib = k < 3 ? k : (k == 3 ? 1 : 2);
        fa = part == 0 ? 4 + ia : 9 + part;
        fb = part == 0 ? 7 + ib : 13 + k;
    };
    int fa0, fb0, fa1, fb1;
    factors(min(a, NA - 1), fa0, fb0);
    factors(min(a + 16, NA - 1), fa1, fb1);
    real acc0 = 0, acc1 = 0;
    // evaluate entry e of the particle's m (one per lane, m <= 16), then add
    // the results in entry order; entries past m contribute exact zeros
    auto evaluate = [&](int m, int e) {
        real o[NF];
#pragma unroll
        for (int k = 0; k < NF; ++k) o[k] = (real)0;
        if (a < m) {
            const unsigned po = ((unsigned)e >> 5) * (unsigned)(2 * sizeof(V4));
            const V4 pj = *(const V4*)((const char*)pv + po);
            const V4 cj = *(const V4*)((const char*)pv + po + sizeof(V4));
            const int code = e & 31;
            const real sx = shift_tab[code][0], sy = shift_tab[code][1];
            const real zj = pj.z + shift_tab[code][2];
            const real dx = (ri0 - sx) - pj.x, dy = (ri1 - sy) - pj.y, dz = ri2 - zj;
            const PairOut<real> w = pair_force<real>(P, dx, dy, dz, ci0, ci1, ci2, cj.x, cj.y, cj.z, (unsigned)own_id,
                                                     (unsigned)R::id(cj));
            o[0] = w.mag; o[1] = w.ex; o[2] = w.ey; o[3] = w.ez;
            o[4] = dx; o[5] = dy; o[6] = dz;
            o[7] = w.gx; o[8] = w.gy; o[9] = w.gz;
            if constexpr (COMP) {
                o[10] = w.wR * P.a;
                o[11] = -(w.wR * P.gam * w.wR * w.ev);
                o[12] = w.wR * P.sig * w.th;
                o[13] = dx * w.ex; o[14] = dy * w.ey; o[15] = dz * w.ez;
                o[16] = dx * w.ey; o[17] = dx * w.ez; o[18] = dy * w.ez;
            }
        }
#pragma unroll
        for (int k = 0; k < NF; ++k) res[p][k][a] = o[k];
        wave_lds_sync();
        const real* xa = res[p][fa0];
        const real* xb = res[p][fb0];
#pragma unroll
        for (int k = 0; k < 16; ++k) acc0 = fma(xa[k], xb[k], acc0);
        if constexpr (COMP) {
            const real* ya = res[p][fa1];
            const real* yb = res[p][fb1];
#pragma unroll
            for (int k = 0; k < 16; ++k) acc1 = fma(ya[k], yb[k], acc1);
        }
        wave_lds_sync();
    };

    // search: lane a < 9 scans row a
    int q = 0, qe = 0, ic = 4, found = 0;
    real bx = 0, by = 0;
    if (act && a < 9) row_range(a, q, qe, ic, bx, by);
    while (__ballot(q < qe) != 0ull) {
        V4 cand[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) cand[u] = load_rec<real>(srsrc, sbase, (unsigned)(q + u) * (unsigned)sizeof(V4));
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((q + u < qe) & accepted(cand[u], bx, by)) {
                if (found < WIDE_ROW) rowq[p][a][found] = R::id(cand[u]) + ic;
                ++found;
            }
        q = min(q + 4, qe);
    }
    const int incl = row_scan(found);  // accepted in this row and the ones before it
    const int total = row_lane<15>(incl);
    const unsigned over = (unsigned)(__ballot(found > WIDE_ROW) >> gbase) & 0xFFFFu;
    if (over == 0u)
        for (int k = 0; k < found; ++k) list[p][incl - found + k] = rowq[p][a][k];
    wave_lds_sync();
    const int fast = over == 0u ? total : 0;
    for (int e0 = 0; __ballot(e0 < fast) != 0ull; e0 += 16)
        evaluate(min(fast - e0, 16), e0 + a < fast ? list[p][e0 + a] : 0);
    // a row holds more than WIDE_ROW neighbours (a very dense spot): row by
    // row, sixteen candidates at a time, in the same order
    if (__ballot(over != 0u) != 0ull) {
        for (int row = 0; row < 9; ++row) {
            int rq = 0, re = 0, rc = 4;
            real rx = 0, ry = 0;
            if (act && over != 0u) row_range(row, rq, re, rc, rx, ry);
            while (__ballot(rq < re) != 0ull) {
                const V4 v = load_rec<real>(srsrc, sbase, (unsigned)min(rq + a, max(re - 1, 0)) * (unsigned)sizeof(V4));
                const bool ok = (rq + a < re) & accepted(v, rx, ry);
                const unsigned mask = (unsigned)(__ballot(ok) >> gbase) & 0xFFFFu;
                if (ok) list[p][__popc(mask & ((1u << a) - 1u))] = R::id(v) + rc;
                wave_lds_sync();
                const int m = __popc(mask);
                evaluate(m, a < m ? list[p][a] : 0);
                rq = min(rq + 16, re);
            }
        }
    }
    real fx = row_lane<0>(acc0), fy = row_lane<1>(acc0), fz = row_lane<2>(acc0);
    real wf[6] = {0, 0, 0, 0, 0, 0};
    if (act && own_id < B.n_beads)
        bond_forces<real>(C, b, own_id, (const V4*)C.sid[A.slot] + B.off, h00, h01, h10, h11, h22, fx, fy,
                          fz, wf, [](real, real) { return (real)1; });
    double kin[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (act && A.kick) {
        end_step<real, false>(C, A, B, D, C.dyn[(size_t)(A.slot ^ 1) * C.n_boxes + b], pos, own_id, s0, s1, s2, ci0,
                              ci1, ci2, fx, fy, fz, L00, L01, L10, L11, stepc, a == 0, kin);
    } else if (act && a == 0) {
        real* f = (real*)C.f;
        const int i = B.off + own_id, N = C.n_total;
        f[i] = fx; f[(size_t)N + i] = fy; f[2 * (size_t)N + i] = fz;
    }
    if (a >= 3 && a < 9) vals[p][a - 3] = act ? (double)acc0 : 0.0;
    if constexpr (COMP) {
        if (a >= 9) vals[p][19 + a - 9] = (double)acc0;
        if (a + 16 < NA) vals[p][19 + a + 7] = (double)acc1;
    }
    if (a == 0) {
        for (int k = 0; k < 6; ++k) {
            vals[p][6 + k] = (double)wf[k];
            vals[p][13 + k] = kin[k];
        }
        vals[p][12] = act ? (double)total : 0.0;
    }
    __syncthreads();
    // the subtree over j (lanes 32, 16, 8, 4 apart)
    if (t < NV) {
        double x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = vals[j][t];
#pragma unroll
        for (int o = 8; o > 0; o >>= 1)
#pragma unroll
            for (int j = 0; j < o; ++j) x[j] += x[j + o];
        C.part[(size_t)A.w * C.part_step + ((size_t)work * WIDE_UNITS + sub) * NV + t] = x[0];
    }
}

// One step's partial sums of one box, a workgroup per (box, step of the
// window): column l of LDS takes blocks l, l + 64, ... in order, then a fixed
// tree (lanes 32, 16, .. 1 apart; missing blocks are zero).
constexpr int SUM_THREADS = 256;

template <int NV>
__global__ __launch_bounds__(SUM_THREADS) void k_window_sums(Ctx C, int nbox, int part0, int wide) {
    __shared__ double x[64][NV];
    const int q = blockIdx.x % nbox, w = blockIdx.x / nbox, b = C.sel ? C.sel[q] : q;
    const BoxInfo B = C.box[b];
    const int first = C.sel ? C.blk0[q] : B.blk_off, cols = min(B.nblk, 64);
    const double* part = C.part + (size_t)w * C.part_step + (size_t)(part0 + first) * NV * (wide ? WIDE_UNITS : 1);
    for (int i = threadIdx.x; i < cols * NV; i += SUM_THREADS) {
        const int l = i / NV, r = i - l * NV;
        double s = 0.0;
        for (int k = l; k < B.nblk; k += 64) {
            if (wide) {  // per wave of 64 particles the residues two and one apart, then the waves in order
                const double* p = part + (size_t)k * NV * WIDE_UNITS + r;
                double y[WIDE_UNITS];
#pragma unroll
                for (int u = 0; u < WIDE_UNITS; ++u) y[u] = p[(size_t)u * NV];
                double z = 0.0;
#pragma unroll
                for (int v = 0; v < WIDE_UNITS; v += 4) z += (y[v] + y[v + 2]) + (y[v + 1] + y[v + 3]);
                s += z;
            } else {
                s += part[(size_t)k * NV + r];
            }
        }
        x[l][r] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < NV) {
        const int r = threadIdx.x;
        int o = 32;
        while (o >= cols) o >>= 1;  // upper halves that hold no block
        for (; o > 0; o >>= 1)
            for (int l = 0; l < o && l + o < cols; ++l) x[l][r] += x[l + o][r];
        C.sums[((size_t)w * C.n_boxes + b) * NV + r] = x[0][r];
    }
}

// The stresses of a window of nw steps, one wave per box: sigma = -(K + W)/V
// by part and step, the steps added in order.  After a chunk's last window
// the box's cell returns to slot 0 and, when this launch covers all of the
// chunk's boxes, the step counter advances by `add`.
template <int NV>
__global__ __launch_bounds__(64) void k_flush(Ctx C, int nw, int copy_dyn, int add) {
    const int b = C.sel ? C.sel[blockIdx.x] : (int)blockIdx.x;
    // the window's sums and inverse volumes, all on their way at once (read
    // step by step, 50 steps took 17 us)
    __shared__ double sum[MAX_WINDOW][NV], ivol[MAX_WINDOW];
    const double* sums = C.sums + (size_t)b * NV;
    double* acc = C.acc + (size_t)ACC * b;
    const int r = threadIdx.x;
#pragma unroll 8
    for (int i = r; i < nw * NV; i += 64) sum[i / NV][i % NV] = sums[(size_t)(i / NV) * C.n_boxes * NV + i % NV];
    if (r < nw) ivol[r] = 1.0 / C.vol[(size_t)r * C.n_boxes + b];
    __syncthreads();
    if (r < 6) {
        double a0 = acc[r], a1 = acc[6 + r], a2 = acc[12 + r];
        bool finite = true;
#pragma unroll 4
        for (int w = 0; w < nw; ++w) {
            const double iv = ivol[w];
            const double sk = -sum[w][13 + r] * iv, sp = -C.vir_scale * sum[w][r] * iv, sf = -sum[w][6 + r] * iv;
            a0 += sk;
            a1 += sp;
            a2 += sf;
            if (!(fabs(sk + sp + sf) <= 1e300)) finite = false;
        }
        acc[r] = a0;
        acc[6 + r] = a1;
        acc[12 + r] = a2;
        if (!finite) atomicOr(&C.flags[b], LHMM_FLAG_NONFINITE);
    } else if (r == 6) {
        unsigned long long up = 0ull;
#pragma unroll 4
        for (int w = 0; w < nw; ++w) {
            const unsigned long long np = (unsigned long long)sum[w][12];
            up += C.vir_scale < 1.0 ? np / 2 : np;
        }
        C.acc_pairs[b] += up;
        C.tot_pairs[b] += up;
        if (add && blockIdx.x == 0) *C.step += (unsigned long long)add;
    } else if (NV > 19 && r >= 18 && r < 36) {
        double a = acc[r];
#pragma unroll 4
        for (int w = 0; w < nw; ++w) a += -C.vir_scale * sum[w][r + 1] * ivol[w];
        acc[r] = a;
    }
    if (copy_dyn)
        for (int k = r; k < (int)(sizeof(BoxDyn) / sizeof(int)); k += 64)
            ((int*)&C.dyn[b])[k] = ((const int*)&C.dyn[(size_t)C.n_boxes + b])[k];
}

__global__ void k_step_add(unsigned long long* __restrict__ step, int add) { *step += (unsigned long long)add; }

// Copy the snapshot state of the selected boxes back (one workgroup per box)
// and clear their flags.
template <typename real>
__global__ __launch_bounds__(256) void k_restore(Ctx C, const real* __restrict__ ss, const real* __restrict__ sc,
                                                 const real* __restrict__ sf, const BoxDyn* __restrict__ sdyn) {
    const int b = C.sel[blockIdx.x];
    const BoxInfo B = C.box[b];
    const int N = C.n_total;
    real* s = (real*)C.s;
    real* c = (real*)C.c;
    real* f = (real*)C.f;
    for (int k = 0; k < 3; ++k)
        for (int i = threadIdx.x; i < B.n; i += blockDim.x) {
            const long q = (long)k * N + B.off + i;
            s[q] = ss[q];
            c[q] = sc[q];
            f[q] = sf[q];
        }
    if (threadIdx.x == 0) {
        C.dyn[b] = sdyn[b];
        C.flags[b] = 0u;
    }
}

__global__ void k_finalize(Ctx C, double* __restrict__ stress_out, double* __restrict__ parts_out,
                           double inv_steps) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= C.n_boxes) return;
    const double* acc = C.acc + ACC * b;
    for (int q = 0; q < 6; ++q) stress_out[6 * b + q] = (acc[q] + acc[6 + q] + acc[12 + q]) * inv_steps;
    for (int q = 0; q < ACC; ++q) parts_out[ACC * b + q] = acc[q] * inv_steps;
}

}  // namespace

// ---------------------------------------------------------------------------
// Engine
// ---------------------------------------------------------------------------

struct lhmm_micro {
    lhmm_params p{};
    HostStage stage;  // read-backs
    lhmm_micro_config cfg{};
    int lds_cells = 0, lds_cols = 0;  // dynamic LDS of the binning (ints)
    int n_slabs = 0, window = 1;      // slabs of all boxes; steps whose partial sums are kept
    std::vector<double> hz;           // largest z extent each box has had (bounds its cells per column)
    int n_boxes = 0, n_blocks = 0, precision = LHMM_FP32;
    long long n_total = 0;
    size_t real_size = 4;
    std::vector<BoxInfo> box;
    std::vector<int> blk_box, blk_first, slab_box;
    hipStream_t user_stream = nullptr, stream = nullptr;
    hipEvent_t ev_in = nullptr, ev_out = nullptr;
    // device buffers
    BoxInfo* d_box = nullptr;
    BoxDyn* d_dyn = nullptr;
    unsigned* d_flags = nullptr;
    int *d_blk_box = nullptr, *d_blk_first = nullptr, *d_slab_box = nullptr;
    void *d_s = nullptr, *d_c = nullptr, *d_f = nullptr;
    int *d_key = nullptr, *d_perm = nullptr, *d_gcell_start = nullptr;
    void *d_sid[2] = {}, *d_sord[2] = {}, *d_cord = nullptr;
    void* d_cell_pv = nullptr;
    void* d_srec = nullptr;
    double *d_part = nullptr, *d_sums = nullptr, *d_vol = nullptr;
    double *d_acc = nullptr, *d_parts = nullptr, *d_gradL = nullptr;
    unsigned long long *d_acc_pairs = nullptr, *d_tot_pairs = nullptr, *d_step = nullptr;
    // selection lists (device) and their pinned staging, reused once ev_sel completes
    int *d_sel = nullptr, *h_sel = nullptr;
    size_t sel_cap = 0;
    hipEvent_t ev_sel = nullptr;
    // snapshot of the particle state and per-box cells
    void *d_snap_s = nullptr, *d_snap_c = nullptr, *d_snap_f = nullptr;
    BoxDyn* d_snap_dyn = nullptr;
    bool have_snapshot = false;
    bool have_state = false, forces_valid = false;
    bool afbc = false;  // some box has boundary regions (lhmm_micro_set_afbc)
    bool flat = false;  // some box has been too flat for its stencil
    std::map<int, hipGraphExec_t> graphs;
    // graphs of subset steps, keyed by (boxes, blocks, slabs, steps): a shape is
    // captured the second time it is asked for (history replays repeat it)
    std::map<std::tuple<int, int, int, int>, hipGraphExec_t> sub_graphs;
    std::map<std::tuple<int, int, int, int>, int> sub_seen;
    // overlapped groups of boxes (cfg.groups > 1): boxes by particle count,
    // smallest first; inside a captured chunk of steps each group runs all
    // its steps on its own stream, and the groups join at the chunk's end
    struct Group {
        int* d_lists = nullptr;  // sel, blk0, blk_list, slab_list in one allocation
        int n_sel = 0, nblk = 0, nslab = 0, part0 = 0;
    };
    std::vector<Group> groups;
    hipStream_t aux[MAX_GROUPS - 1] = {};
    hipEvent_t ev_fork = nullptr, ev_join[MAX_GROUPS - 1] = {};
    Ctx ctx{};
};

namespace {

// Column capacity of a box's cell grid: n0 n1 n2 <= cell_cap with
// n2 >= 2 zsub + 1, or n0, n1 <= 3 when the grid had to be clipped.
int box_cols(const BoxInfo& B) { return std::max(B.cell_cap / (2 * B.zsub + 1), 9) + 1; }

// What a launch covers: all boxes (C without lists), or the lists in C.
struct Launch {
    Ctx C;
    int nbox, nblk, nslab, part0;
    bool wide;  // sixteen lanes per particle (its partial sums take WIDE_UNITS places per block, from 0)
    hipStream_t st;
};

// Sixteen lanes per particle where one lane each would leave the chip idle:
// below 256 work blocks of 256 particles (a wave per SIMD) k_forces's time is
// that of one wave's dependent loads and rounds.  The wide kernel has no
// variant for boundary regions or pruning.
bool use_wide(const lhmm_micro* m, int nblk) { return nblk <= WIDE_BLOCKS && !m->afbc && !m->cfg.prune; }

Launch all_boxes(lhmm_micro* m) {
    return Launch{m->ctx, m->n_boxes, m->n_blocks, m->n_slabs, 0, use_wide(m, m->n_blocks), m->stream};
}

template <typename real>
void launch_bin(lhmm_micro* m, const Launch& L, const Step& A) {
    // where the slabs do not fill the chip a workgroup's latency counts: 1024
    // threads (5 boxes of 4000: 1393 us per 50 steps against 1469 with 512; the
    // batch of 256, 1.5k slabs: 5046 per 20 steps with 512, 5666 with 1024)
    const int T = L.nslab <= 256 ? 1024 : m->cfg.bin_threads, nc = (L.nbox + T - 1) / T;
    const size_t bytes = sizeof(int) * ((size_t)m->lds_cells + 3 * (size_t)m->lds_cols + 2 * (size_t)SLAB_CAP);
    const int grid = nc + L.nslab;
    switch (T) {
        case 256: k_bin<real, 256><<<grid, 256, bytes, L.st>>>(L.C, A, nc, m->lds_cells, m->lds_cols); break;
        case 512: k_bin<real, 512><<<grid, 512, bytes, L.st>>>(L.C, A, nc, m->lds_cells, m->lds_cols); break;
        default: k_bin<real, 1024><<<grid, 1024, bytes, L.st>>>(L.C, A, nc, m->lds_cells, m->lds_cols); break;
    }
}

template <typename real>
void launch_forces(lhmm_micro* m, const Launch& L, const Step& A) {
    int drain = m->cfg.drain;
    const int busy = m->cfg.busy_lanes;
    const Ctx& C = L.C;
    const bool comp = C.nv > 19;
    if (L.wide) {
        if (comp)
            k_forces_wide<real, true><<<L.nblk * WIDE_UNITS, BS, 0, L.st>>>(C, A);
        else
            k_forces_wide<real, false><<<L.nblk * WIDE_UNITS, BS, 0, L.st>>>(C, A);
        return;
    }
#define LHMM_FORCES(QD, FLAT)                                                                     \
    do {                                                                                          \
        if (m->afbc && comp)                                                                      \
            k_forces<real, QD, false, true, true, FLAT><<<L.nblk, BS, 0, L.st>>>(C, A, drain, busy);  \
        else if (m->afbc)                                                                         \
            k_forces<real, QD, false, false, true, FLAT><<<L.nblk, BS, 0, L.st>>>(C, A, drain, busy); \
        else if (comp)                                                                            \
            k_forces<real, QD, false, true, false, FLAT><<<L.nblk, BS, 0, L.st>>>(C, A, drain, busy); \
        else if (m->cfg.prune)                                                                    \
            k_forces<real, QD, true, false, false, FLAT><<<L.nblk, BS, 0, L.st>>>(C, A, drain, busy); \
        else                                                                                      \
            k_forces<real, QD, false, false, false, FLAT><<<L.nblk, BS, 0, L.st>>>(C, A, drain, busy); \
    } while (0)
    if (m->flat) {  // rare, in one queue depth (it changes no result)
        drain = std::min(drain, 16 - scan_unroll(16));
        LHMM_FORCES(16, true);
        return;
    }
    switch (m->cfg.queue_depth) {
        case 2: LHMM_FORCES(2, false); break;
        case 4: LHMM_FORCES(4, false); break;
        case 8: LHMM_FORCES(8, false); break;
        case 32: LHMM_FORCES(32, false); break;
        default: LHMM_FORCES(16, false); break;
    }
#undef LHMM_FORCES
}

void launch_flush(lhmm_micro* m, const Launch& L, int nw, bool copy_dyn, int add) {
    const int wide = L.wide ? 1 : 0;
    if (L.C.nv > 19) {
        k_window_sums<37><<<L.nbox * nw, SUM_THREADS, 0, L.st>>>(L.C, L.nbox, L.part0, wide);
        k_flush<37><<<L.nbox, 64, 0, L.st>>>(L.C, nw, copy_dyn ? 1 : 0, add);
    } else {
        k_window_sums<19><<<L.nbox * nw, SUM_THREADS, 0, L.st>>>(L.C, L.nbox, L.part0, wide);
        k_flush<19><<<L.nbox, 64, 0, L.st>>>(L.C, nw, copy_dyn ? 1 : 0, add);
    }
}

// n steps of the boxes L covers, the random-force counters *C.step + k0 + 1
// .. k0 + n; add: advance *C.step by that much at the end.  between(q, i):
// called around the launches (q: the kernel, i = 0 before, 1 after).
template <typename real, class Between>
void launch_chunk(lhmm_micro* m, const Launch& L, int k0, int n, int add, Between between) {
    between(LHMM_K_KICK_DRIFT, 0);
    k_begin_chunk<real><<<L.nblk, BS, 0, L.st>>>(L.C, k0, 1);
    between(LHMM_K_KICK_DRIFT, 1);
    for (int k = 1; k <= n; ++k) {
        Step A{};
        A.slot = k & 1;
        A.first = k == 1;
        A.more = k < n;
        A.kick = 1;
        A.w = (k - 1) % m->window;
        A.k = k0 + k;
        A.part0 = L.part0;
        between(LHMM_K_BIN, 0);
        launch_bin<real>(m, L, A);
        between(LHMM_K_BIN, 1);
        between(LHMM_K_FORCES, 0);
        launch_forces<real>(m, L, A);
        between(LHMM_K_FORCES, 1);
        if (A.w == m->window - 1 || k == n) {
            between(LHMM_K_STRESS, 0);
            launch_flush(m, L, A.w + 1, k == n && (n & 1), k == n ? add : 0);
            between(LHMM_K_STRESS, 1);
        }
    }
}

// With fuse_bin off every step takes the particles from and back to index
// order: the half kick and drift run as their own launch.
template <typename real, class Between>
void launch_steps(lhmm_micro* m, const Launch& L, int n, bool add, Between between) {
    if (m->cfg.fuse_bin) {
        launch_chunk<real>(m, L, 0, n, add ? n : 0, between);
        return;
    }
    for (int k = 0; k < n; ++k) launch_chunk<real>(m, L, k, 1, add && k + 1 == n ? n : 0, between);
}

void launch_steps(lhmm_micro* m, const Launch& L, int n, bool add = true) {
    auto nothing = [](int, int) {};
    if (m->precision == LHMM_FP64)
        launch_steps<double>(m, L, n, add, nothing);
    else
        launch_steps<float>(m, L, n, add, nothing);
}

// A captured chunk of nsteps steps with the boxes in overlapped groups.  The
// boxes of one group never read another group's data, so each group runs its
// whole chunk on its own stream; the step counter advances once they joined.
void launch_chunk_grouped(lhmm_micro* m, int nsteps) {
    const int G = (int)m->groups.size();
    (void)hipEventRecord(m->ev_fork, m->stream);
    for (int g = 1; g < G; ++g) (void)hipStreamWaitEvent(m->aux[g - 1], m->ev_fork, 0);
    for (int g = 0; g < G; ++g) {
        const lhmm_micro::Group& gr = m->groups[g];
        Launch L{m->ctx, gr.n_sel, gr.nblk, gr.nslab, gr.part0, false, g == 0 ? m->stream : m->aux[g - 1]};
        L.C.sel = gr.d_lists;
        L.C.blk0 = gr.d_lists + gr.n_sel;
        L.C.blk_list = gr.d_lists + 2 * gr.n_sel;
        L.C.slab_list = gr.d_lists + 2 * gr.n_sel + gr.nblk;
        L.C.n_sel = gr.n_sel;
        launch_steps(m, L, nsteps, false);
    }
    for (int g = 1; g < G; ++g) {
        (void)hipEventRecord(m->ev_join[g - 1], m->aux[g - 1]);
        (void)hipStreamWaitEvent(m->stream, m->ev_join[g - 1], 0);
    }
    k_step_add<<<1, 1, 0, m->stream>>>(m->d_step, nsteps);
}

// Set-up of a call: gradients and cleared sums of every box, zero mean
// velocity of the boxes L covers; the forces if none are carried.
template <typename real>
void launch_force_eval_t(lhmm_micro* m) {
    const Launch L = all_boxes(m);
    Step A{};
    A.slot = 1;
    A.first = 1;
    k_begin_chunk<real><<<L.nblk, BS, 0, L.st>>>(L.C, 0, 0);
    launch_bin<real>(m, L, A);
    launch_forces<real>(m, L, A);
}

void launch_force_eval(lhmm_micro* m) {
    if (m->precision == LHMM_FP64)
        launch_force_eval_t<double>(m);
    else
        launch_force_eval_t<float>(m);
}

void launch_begin_call(lhmm_micro* m, const Ctx& C, int n_mean, const double* gradL, int clear = 1) {
    const int grid = n_mean + (m->n_boxes + 63) / 64;
    if (m->precision == LHMM_FP64)
        k_begin_call<double><<<grid, CALL_THREADS, 0, m->stream>>>(C, gradL, n_mean, clear);
    else
        k_begin_call<float><<<grid, CALL_THREADS, 0, m->stream>>>(C, gradL, n_mean, clear);
}

int get_graph(lhmm_micro* m, int nsteps, hipGraphExec_t* out) {
    auto it = m->graphs.find(nsteps);
    if (it != m->graphs.end()) {
        *out = it->second;
        return LHMM_OK;
    }
    hipGraph_t g = nullptr;
    // launches that use the wide force kernel do not fill the chip: one stream
    const bool grouped = m->groups.size() > 1 && m->cfg.fuse_bin && !use_wide(m, m->n_blocks);
    HIPCHK(hipStreamBeginCapture(m->stream, hipStreamCaptureModeThreadLocal));
    if (grouped)
        launch_chunk_grouped(m, nsteps);
    else
        launch_steps(m, all_boxes(m), nsteps);
    HIPCHK(hipStreamEndCapture(m->stream, &g));
    hipGraphExec_t ex = nullptr;
    hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) return fail(LHMM_ERR_HIP, "hipGraphInstantiate: %s", hipGetErrorString(e));
    m->graphs[nsteps] = ex;
    *out = ex;
    return LHMM_OK;
}

bool cell_ok(const double* h) {
    for (int k = 0; k < 9; ++k)
        if (!std::isfinite(h[k])) return false;
    if (h[2] != 0.0 || h[5] != 0.0 || h[6] != 0.0 || h[7] != 0.0) return false;
    if (!(h[8] > 0.0)) return false;
    return m3_det(h) > 0.0;
}

template <typename T>
int dalloc(T** p, size_t count) {
    if (count == 0) count = 1;
    hipError_t e = hipMalloc((void**)p, count * sizeof(T));
    if (e != hipSuccess) return fail(LHMM_ERR_OOM, "hipMalloc(%zu bytes): %s", count * sizeof(T), hipGetErrorString(e));
    return LHMM_OK;
}

void drop_groups(lhmm_micro* m) {
    for (auto& gr : m->groups)
        if (gr.d_lists) (void)hipFree(gr.d_lists);
    m->groups.clear();
}

void release(lhmm_micro* m) {
    if (m->stream) (void)hipStreamSynchronize(m->stream);
    for (auto& kv : m->graphs) (void)hipGraphExecDestroy(kv.second);
    m->graphs.clear();
    for (auto& kv : m->sub_graphs) (void)hipGraphExecDestroy(kv.second);
    m->sub_graphs.clear();
    void* bufs[] = {m->d_box, m->d_dyn, m->d_flags, m->d_blk_box, m->d_blk_first, m->d_slab_box, m->d_s, m->d_c, m->d_f,
                    m->d_key, m->d_perm, m->d_gcell_start, m->d_sid[0], m->d_sid[1], m->d_sord[0], m->d_sord[1],
                    m->d_cord, m->d_cell_pv, m->d_srec, m->d_part, m->d_sums, m->d_vol, m->d_acc, m->d_parts, m->d_gradL,
                    m->d_acc_pairs, m->d_tot_pairs, m->d_step, m->d_sel, m->d_snap_s, m->d_snap_c, m->d_snap_f,
                    m->d_snap_dyn};
    for (void* b : bufs)
        if (b) (void)hipFree(b);
    m->stage.release();
    drop_groups(m);
    for (int g = 0; g < MAX_GROUPS - 1; ++g) {
        if (m->aux[g]) (void)hipStreamDestroy(m->aux[g]);
        if (m->ev_join[g]) (void)hipEventDestroy(m->ev_join[g]);
    }
    if (m->ev_fork) (void)hipEventDestroy(m->ev_fork);
    if (m->h_sel) (void)hipHostFree(m->h_sel);
    if (m->ev_sel) (void)hipEventDestroy(m->ev_sel);
    if (m->ev_in) (void)hipEventDestroy(m->ev_in);
    if (m->ev_out) (void)hipEventDestroy(m->ev_out);
    if (m->stream) (void)hipStreamDestroy(m->stream);
}

int sync_engine(lhmm_micro* m) {
    HIPCHK(hipStreamSynchronize(m->stream));
    HIPCHK(hipGetLastError());
    return LHMM_OK;
}

// device memory of the engine -> host, after the work on its stream
int read_back(lhmm_micro* m, void* dst, const void* src, size_t bytes) {
    HIPCHK(m->stage.copy(m->stream, {{src, bytes}}, {dst}));
    HIPCHK(hipGetLastError());
    return LHMM_OK;
}

// elements [e0, e0 + n) of a 3 x N array -> rows of an N x 3 one
template <typename real>
void to_rows(double* dst, size_t N, size_t e0, const real* x, size_t n) {
    while (n > 0) {
        const size_t k = e0 / N, i = e0 % N, len = std::min(n, N - i);
        for (size_t j = 0; j < len; ++j) dst[3 * (i + j) + k] = (double)x[j];
        e0 += len;
        x += len;
        n -= len;
    }
}

constexpr size_t MAX_SUB_GRAPHS = 64;

// len steps of the selected boxes: a captured graph for a shape seen before,
// else eager launches.  The graph reads the selection lists from the fixed
// device buffer, whose layout goes by the shape, so any selection of the same
// shape can replay it.
int launch_subset_steps(lhmm_micro* m, const Launch& L, int len) {
    const auto key = std::make_tuple(L.nbox, L.nblk, L.nslab, len);
    auto it = m->sub_graphs.find(key);
    if (it == m->sub_graphs.end() && ++m->sub_seen[key] >= 2) {
        if (m->sub_graphs.size() >= MAX_SUB_GRAPHS) {
            for (auto& kv : m->sub_graphs) (void)hipGraphExecDestroy(kv.second);
            m->sub_graphs.clear();
        }
        hipGraph_t g = nullptr;
        HIPCHK(hipStreamBeginCapture(m->stream, hipStreamCaptureModeThreadLocal));
        launch_steps(m, L, len);
        HIPCHK(hipStreamEndCapture(m->stream, &g));
        hipGraphExec_t ex = nullptr;
        hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) return fail(LHMM_ERR_HIP, "hipGraphInstantiate: %s", hipGetErrorString(e));
        it = m->sub_graphs.emplace(key, ex).first;
    }
    if (it != m->sub_graphs.end()) {
        HIPCHK(hipGraphLaunch(it->second, m->stream));
    } else {
        launch_steps(m, L, len);
    }
    return LHMM_OK;
}

// A box of z extent hz is too flat for its stencil where the smallest number of
// cells does not span the cutoff (more cells come only with more extent).
bool is_flat(const lhmm_micro* m, int b, double hz) {
    return !z_cells_span(hz, m->box[b].zsub, 2 * m->box[b].zsub + 1, m->p.rc);
}

// LDS of the binning for the boxes' present z extents.  The cells of a
// column are at most those of the largest z extent the box has had.
void bin_lds(lhmm_micro* m) {
    m->lds_cells = m->lds_cols = 0;
    for (int b = 0; b < m->n_boxes; ++b) {
        const BoxInfo& B = m->box[b];
        const long long nz = (long long)std::floor(B.zsub * m->hz[b] / m->p.rc * (1.0 + 1e-9));
        // the grid is clipped to cell_cap cells with at least 9 columns
        const int n2 = (int)std::min<long long>(std::max<long long>(nz, 2 * B.zsub + 1), std::max(B.cell_cap / 9, 2 * B.zsub + 1));
        const int cols = box_cols(B);
        m->lds_cells = std::max(m->lds_cells, std::min(B.cell_cap, B.cell_cap / B.nslab + n2) + 1);
        m->lds_cols = std::max(m->lds_cols, std::min(cols, cols / B.nslab + 2));
    }
}

// Cut the boxes into slabs for the binning: about SLAB_TARGET particles (or
// bin_split, where that is smaller) and at most SLAB_CELLS cells each.  Where
// the allocation fails the slabs stay as they were.
int build_slabs(lhmm_micro* m, int bin_split) {
    const int target = bin_split > 0 ? std::min(bin_split, SLAB_TARGET) : SLAB_TARGET;
    std::vector<BoxInfo> box = m->box;
    std::vector<int> slab_box;
    for (int b = 0; b < m->n_boxes; ++b) {
        BoxInfo& B = box[b];
        B.slab_off = (int)slab_box.size();
        // every column belongs to one slab, so more slabs than columns (9 at least) would only idle
        B.nslab = std::max((B.n + target - 1) / target, (B.cell_cap + SLAB_CELLS - 1) / SLAB_CELLS);
        B.nslab = std::min(B.nslab, box_cols(B));
        for (int q = 0; q < B.nslab; ++q) slab_box.push_back(b);
    }
    int* d = nullptr;
    int rc = dalloc(&d, slab_box.size());
    if (rc != LHMM_OK) return rc;
    std::swap(d, m->d_slab_box);
    if (d) (void)hipFree(d);
    m->ctx.slab_box = m->d_slab_box;
    m->n_slabs = (int)slab_box.size();
    m->slab_box.swap(slab_box);
    m->box.swap(box);
    bin_lds(m);
    HIPCHK(hipMemcpy(m->d_slab_box, m->slab_box.data(), m->n_slabs * sizeof(int), hipMemcpyHostToDevice));
    HIPCHK(hipMemcpy(m->d_box, m->box.data(), m->n_boxes * sizeof(BoxInfo), hipMemcpyHostToDevice));
    return LHMM_OK;
}

// Drop every captured graph (they hold launch shapes and contexts).
void drop_graphs(lhmm_micro* m) {
    for (auto& kv : m->graphs) (void)hipGraphExecDestroy(kv.second);
    m->graphs.clear();
    for (auto& kv : m->sub_graphs) (void)hipGraphExecDestroy(kv.second);
    m->sub_graphs.clear();
    m->sub_seen.clear();
}

// Lists of a selection in one host array: the boxes, each one's first work
// block in the block list, the work blocks, the slabs.
struct Lists {
    int nblk = 0, nslab = 0;
};

Lists fill_lists(const lhmm_micro* m, const int* boxes, int n_sel, int* out) {
    Lists L;
    int *sel = out, *blk0 = out + n_sel, *blk = out + 2 * n_sel;
    for (int q = 0; q < n_sel; ++q) {
        const BoxInfo& B = m->box[boxes[q]];
        sel[q] = boxes[q];
        blk0[q] = L.nblk;
        for (int k = 0; k < B.nblk; ++k) blk[L.nblk++] = B.blk_off + k;
    }
    int* slab = blk + L.nblk;
    for (int q = 0; q < n_sel; ++q) {
        const BoxInfo& B = m->box[boxes[q]];
        for (int k = 0; k < B.nslab; ++k) slab[L.nslab++] = B.slab_off + k;
    }
    return L;
}

// Partition the boxes into G groups of about equal particle counts and mixed
// sizes (largest first, each to the least loaded group), with their lists:
// groups that take equally long overlap to the chunk's end (with the largest
// boxes, two thirds of the particles, in one group, that one ran alone after
// the other: batch of 256, 20 steps, 5046 us against 4800).
int make_groups(lhmm_micro* m, int G) {
    HIPCHK(hipStreamSynchronize(m->stream));
    drop_groups(m);
    if (G <= 1) return LHMM_OK;
    if (!m->ev_fork) {
        HIPCHK(hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming));
        for (int g = 0; g < MAX_GROUPS - 1; ++g) {
            HIPCHK(hipStreamCreateWithFlags(&m->aux[g], hipStreamNonBlocking));
            HIPCHK(hipEventCreateWithFlags(&m->ev_join[g], hipEventDisableTiming));
        }
    }
    std::vector<int> order(m->n_boxes);
    for (int b = 0; b < m->n_boxes; ++b) order[b] = b;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return m->box[a].n < m->box[b].n; });
    std::vector<std::vector<int>> members(G);
    std::vector<long long> load(G, 0);
    for (auto it = order.rbegin(); it != order.rend(); ++it) {
        const int g = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        members[g].push_back(*it);
        load[g] += m->box[*it].n;
    }
    int part0 = 0;
    std::vector<int> lists(2 * (size_t)m->n_boxes + m->n_blocks + m->n_slabs);
    for (int g = 0; g < G; ++g) {
        if (members[g].empty()) continue;
        std::sort(members[g].begin(), members[g].end());
        lhmm_micro::Group gr;
        gr.n_sel = (int)members[g].size();
        const Lists L = fill_lists(m, members[g].data(), gr.n_sel, lists.data());
        gr.nblk = L.nblk;
        gr.nslab = L.nslab;
        gr.part0 = part0;
        part0 += L.nblk;
        const size_t n = 2 * (size_t)gr.n_sel + L.nblk + L.nslab;
        int rc = dalloc(&gr.d_lists, n);
        if (rc != LHMM_OK) return rc;
        m->groups.push_back(gr);
        HIPCHK(hipMemcpy(gr.d_lists, lists.data(), sizeof(int) * n, hipMemcpyHostToDevice));
    }
    return LHMM_OK;
}

// Groups that could not all be made would leave boxes out: then there are none.
int prepare_groups(lhmm_micro* m, int G) {
    const int rc = make_groups(m, G);
    if (rc != LHMM_OK) drop_groups(m);
    return rc;
}

// Validate a host list of boxes (strictly increasing, in range), upload it
// with its lists on the engine stream, and return a launch that covers them.
int select_boxes(lhmm_micro* m, const int32_t* boxes, int32_t n_sel, Launch* out) {
    if (!boxes || n_sel < 1 || n_sel > m->n_boxes) return fail(LHMM_ERR_ARG, "need 1..%d boxes (got %d)", m->n_boxes, n_sel);
    for (int q = 0; q < n_sel; ++q) {
        if (boxes[q] < 0 || boxes[q] >= m->n_boxes) return fail(LHMM_ERR_ARG, "box %d out of range", boxes[q]);
        if (q && boxes[q] <= boxes[q - 1]) return fail(LHMM_ERR_ARG, "boxes must be strictly increasing");
    }
    const size_t cap = 2 * (size_t)m->n_boxes + m->n_blocks + m->n_slabs;
    if (m->sel_cap < cap) {  // first use, or more slabs than before (set_config waited and dropped the graphs)
        if (m->d_sel) HIPCHK(hipFree(m->d_sel));
        m->d_sel = nullptr;
        if (m->h_sel) HIPCHK(hipHostFree(m->h_sel));
        m->h_sel = nullptr;
        m->sel_cap = 0;
        int rc = dalloc(&m->d_sel, cap);
        if (rc != LHMM_OK) return rc;
        HIPCHK(hipHostMalloc((void**)&m->h_sel, sizeof(int) * cap));
        if (!m->ev_sel) HIPCHK(hipEventCreateWithFlags(&m->ev_sel, hipEventDisableTiming));
        m->sel_cap = cap;
    } else {
        HIPCHK(hipEventSynchronize(m->ev_sel));  // the previous upload has left the staging buffer
    }
    const Lists L = fill_lists(m, boxes, n_sel, m->h_sel);
    const size_t n = 2 * (size_t)n_sel + L.nblk + L.nslab;
    HIPCHK(hipMemcpyAsync(m->d_sel, m->h_sel, sizeof(int) * n, hipMemcpyHostToDevice, m->stream));
    HIPCHK(hipEventRecord(m->ev_sel, m->stream));
    *out = Launch{m->ctx, n_sel, L.nblk, L.nslab, 0, use_wide(m, L.nblk), m->stream};
    out->C.sel = m->d_sel;
    out->C.blk0 = m->d_sel + n_sel;
    out->C.blk_list = m->d_sel + 2 * n_sel;
    out->C.slab_list = m->d_sel + 2 * n_sel + L.nblk;
    out->C.n_sel = n_sel;
    return LHMM_OK;
}

}  // namespace

int lhmm_fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

void lhmm_clear_error() { g_err.clear(); }

hipStream_t lhmm_micro_caller_stream(const lhmm_micro* m) { return m->user_stream; }

extern "C" {

const char* lhmm_last_error(void) { return g_err.c_str(); }

int lhmm_micro_create(const lhmm_params* p, const lhmm_box* boxes, int32_t n_boxes, void* stream,
                      lhmm_micro** out) {
    g_err.clear();
    if (!p || !boxes || !out) return fail(LHMM_ERR_ARG, "null argument");
    *out = nullptr;
    if (n_boxes <= 0) return fail(LHMM_ERR_ARG, "n_boxes must be positive (got %d)", n_boxes);
    const double vals[9] = {p->a, p->gamma, p->sigma, p->kBT, p->mass, p->rc, p->dt, p->H, p->R0};
    for (double v : vals)
        if (!std::isfinite(v)) return fail(LHMM_ERR_ARG, "non-finite parameter");
    if (!(p->dt > 0) || !(p->rc > 0) || !(p->mass > 0) || !(p->R0 > 0) || p->gamma < 0 || p->sigma < 0 || p->H < 0)
        return fail(LHMM_ERR_ARG, "parameters out of range (dt, rc, mass, R0 > 0; gamma, sigma, H >= 0)");
    if (p->chain_len < 2) return fail(LHMM_ERR_ARG, "chain_len must be >= 2");
    if (p->precision != LHMM_FP32 && p->precision != LHMM_FP64) return fail(LHMM_ERR_ARG, "bad precision");

    lhmm_micro* m = new (std::nothrow) lhmm_micro();
    if (!m) return fail(LHMM_ERR_OOM, "host allocation failed");
    m->p = *p;
    m->n_boxes = n_boxes;
    m->precision = p->precision;
    m->cfg.queue_depth = 16;
    m->cfg.drain = 12;
    m->cfg.busy_lanes = 65;
    m->cfg.bin_threads = 512;
    m->cfg.graph_chunk = GRAPH_CHUNK;
    m->cfg.prune = 0;
    m->cfg.fuse_bin = 1;
    m->cfg.groups = 1;  // by size, below
    m->cfg.bin_split = 0;
    m->real_size = p->precision == LHMM_FP64 ? sizeof(double) : sizeof(float);
    m->user_stream = (hipStream_t)stream;

    long long off = 0, srec_off = 0;
    int gcell_off = 0, blk_off = 0;
    m->box.resize(n_boxes);
    for (int b = 0; b < n_boxes; ++b) {
        const lhmm_box& in = boxes[b];
        if (in.n_particles < 2 || in.n_particles > (1 << 25) || in.n_chains < 0 ||
            (long long)in.n_chains * p->chain_len > in.n_particles) {
            delete m;
            return fail(LHMM_ERR_ARG, "box %d: bad particle/chain counts", b);
        }
        if (in.reserved != 0) {
            delete m;
            return fail(LHMM_ERR_ARG, "box %d: reserved field must be 0", b);
        }
        if (!cell_ok(in.h0)) {
            delete m;
            return fail(LHMM_ERR_ARG, "box %d: cell must be finite, in-plane, with det > 0", b);
        }
        // n0 n1 <= w0 w1 <= area and n2 = floor(zsub z extent / rc): the grid
        // never needs more; two cells per cutoff along z unless that exceeds
        // the cell limit
        const double area = fabs(in.h0[0] * in.h0[4] - in.h0[1] * in.h0[3]);
        const long long inplane = (long long)std::floor(area / (p->rc * p->rc) * (1.0 + 1e-9));
        long long cap = 0;
        int zsub = 2;
        for (; zsub >= 1; --zsub) {
            const long long nz = (long long)std::floor(zsub * in.h0[8] / p->rc * (1.0 + 1e-9));
            cap = std::max(9LL * (2 * zsub + 1), std::max(inplane, 9LL) * std::max(nz, 2LL * zsub + 1));
            if (cap <= MAX_CELLS_PER_BOX) break;
        }
        if (cap > MAX_CELLS_PER_BOX) {
            delete m;
            return fail(LHMM_ERR_ARG, "box %d: needs %lld cells, more than %d", b, cap, MAX_CELLS_PER_BOX);
        }
        BoxInfo& B = m->box[b];
        B.off = (int)off;
        B.n = in.n_particles;
        B.n_beads = in.n_chains * p->chain_len;
        B.cell_cap = (int)cap;
        B.gcell_off = gcell_off;
        B.zsub = zsub;
        B.blk_off = blk_off;
        B.nblk = (in.n_particles + BS - 1) / BS;
        B.rng_id = in.rng_id;
        for (int k = 0; k < B.nblk; ++k) {
            m->blk_box.push_back(b);
            m->blk_first.push_back(B.off + k * BS);
        }
        off += in.n_particles;
        B.srec_off = srec_off;
        srec_off += 2 * (long long)in.n_particles + SREC_PAD * (long long)box_cols(B);
        gcell_off += 2 * (int)cap + 1;  // n0 n1 (n2 + 2 zsub + 1) starts and ends, n2 >= 2 zsub + 1
        blk_off += B.nblk;
        if (off > (1LL << 30)) {
            delete m;
            return fail(LHMM_ERR_ARG, "too many particles");
        }
    }
    m->n_total = off;
    m->n_blocks = blk_off;
    m->hz.resize(n_boxes);
    for (int b = 0; b < n_boxes; ++b) {
        m->hz[b] = boxes[b].h0[8];
        m->flat = m->flat || is_flat(m, b, boxes[b].h0[8]);
    }
    const size_t N = (size_t)m->n_total;
    int rc = LHMM_OK;
#define ALLOC(ptr, cnt)                     \
    if (rc == LHMM_OK) rc = dalloc(&(ptr), (cnt));
    ALLOC(m->d_box, (size_t)n_boxes);
    ALLOC(m->d_dyn, 2 * (size_t)n_boxes);
    ALLOC(m->d_flags, (size_t)n_boxes);
    ALLOC(m->d_blk_box, (size_t)m->n_blocks);
    ALLOC(m->d_blk_first, (size_t)m->n_blocks);
    ALLOC(m->d_key, N);
    ALLOC(m->d_perm, N);
    ALLOC(m->d_gcell_start, (size_t)gcell_off);
    const int nv = (p->flags & LHMM_OPT_COMPONENTS) ? 37 : 19;
    const size_t part_step = nv * std::max((size_t)m->n_blocks, (size_t)WIDE_UNITS * std::min(m->n_blocks, WIDE_BLOCKS));
    m->window = (int)std::min<size_t>(MAX_WINDOW, std::max<size_t>(1, PART_BYTES / (part_step * sizeof(double))));
    ALLOC(m->d_part, part_step * m->window);
    ALLOC(m->d_sums, (size_t)n_boxes * m->window * nv);
    ALLOC(m->d_vol, (size_t)n_boxes * m->window);
    ALLOC(m->d_acc, (size_t)n_boxes * ACC);
    ALLOC(m->d_parts, (size_t)n_boxes * ACC);
    ALLOC(m->d_gradL, (size_t)n_boxes * 9);
    ALLOC(m->d_acc_pairs, (size_t)n_boxes);
    ALLOC(m->d_tot_pairs, (size_t)n_boxes);
    ALLOC(m->d_step, (size_t)1);
#undef ALLOC
    if (rc == LHMM_OK) {
        const size_t bytes = 3 * N * m->real_size;
        if (m->stage.reserve(2 * bytes + n_boxes * sizeof(BoxDyn) + 64) != hipSuccess)
            rc = fail(LHMM_ERR_OOM, "pinned allocation failed");
        // search layout: each particle at most twice (its cell, and the
        // image of a bottom or top cell; n2 >= 3)
        for (void** pp : {&m->d_s, &m->d_c, &m->d_f, &m->d_sid[0], &m->d_sid[1], &m->d_sord[0], &m->d_sord[1], &m->d_cord,
                          &m->d_cell_pv, &m->d_srec}) {
            const size_t nb = pp == &m->d_cell_pv ? 8 * N * m->real_size
                              : pp == &m->d_srec ? 4 * (size_t)srec_off * m->real_size
                              : pp == &m->d_s || pp == &m->d_c || pp == &m->d_f ? bytes : 4 * N * m->real_size;
            if (hipMalloc(pp, nb ? nb : 1) != hipSuccess) {
                rc = fail(LHMM_ERR_OOM, "hipMalloc of particle arrays failed");
                break;
            }
        }
    }
    if (rc != LHMM_OK) {
        release(m);
        delete m;
        return rc;
    }
    auto setup = [&]() -> int {
        HIPCHK(hipStreamCreateWithFlags(&m->stream, hipStreamNonBlocking));
        HIPCHK(hipEventCreateWithFlags(&m->ev_in, hipEventDisableTiming));
        HIPCHK(hipEventCreateWithFlags(&m->ev_out, hipEventDisableTiming));
        HIPCHK(hipMemcpy(m->d_blk_box, m->blk_box.data(), m->n_blocks * sizeof(int), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(m->d_blk_first, m->blk_first.data(), m->n_blocks * sizeof(int), hipMemcpyHostToDevice));
        std::vector<BoxDyn> dyn(n_boxes);
        for (int b = 0; b < n_boxes; ++b) {
            memset(&dyn[b], 0, sizeof(BoxDyn));
            for (int k = 0; k < 9; ++k) dyn[b].h[k] = boxes[b].h0[k];
        }
        for (int slot = 0; slot < 2; ++slot)
            HIPCHK(hipMemcpy(m->d_dyn + (size_t)slot * n_boxes, dyn.data(), n_boxes * sizeof(BoxDyn), hipMemcpyHostToDevice));
        HIPCHK(hipMemset(m->d_flags, 0, n_boxes * sizeof(unsigned)));
        HIPCHK(hipMemset(m->d_acc, 0, n_boxes * ACC * sizeof(double)));
        HIPCHK(hipMemset(m->d_parts, 0, n_boxes * ACC * sizeof(double)));
        HIPCHK(hipMemset(m->d_acc_pairs, 0, n_boxes * sizeof(unsigned long long)));
        HIPCHK(hipMemset(m->d_tot_pairs, 0, n_boxes * sizeof(unsigned long long)));
        HIPCHK(hipMemset(m->d_step, 0, sizeof(unsigned long long)));
        if (N) HIPCHK(hipMemset(m->d_f, 0, 3 * N * m->real_size));
        return LHMM_OK;
    };
    rc = setup();
    if (rc != LHMM_OK) {
        release(m);
        delete m;
        return rc;
    }
    Ctx& C = m->ctx;
    C.n_total = (int)m->n_total;
    C.n_boxes = n_boxes;
    C.n_blocks = m->n_blocks;
    C.chain_len = p->chain_len;
    C.box = m->d_box;
    C.dyn = m->d_dyn;
    C.flags = m->d_flags;
    C.blk_box = m->d_blk_box;
    C.blk_first = m->d_blk_first;
    C.s = m->d_s;
    C.c = m->d_c;
    C.f = m->d_f;
    for (int k = 0; k < 2; ++k) {
        C.sid[k] = m->d_sid[k];
        C.sord[k] = m->d_sord[k];
    }
    C.cord = m->d_cord;
    C.key = m->d_key;
    C.perm = m->d_perm;
    C.gcell_start = m->d_gcell_start;
    C.cell_pv = m->d_cell_pv;
    C.srec = m->d_srec;
    C.vir_scale = 0.5;  // every unordered pair is evaluated from both ends
    C.part = m->d_part;
    C.part_step = part_step;
    C.nv = nv;
    C.sums = m->d_sums;
    C.vol = m->d_vol;
    C.acc = m->d_acc;
    C.acc_pairs = m->d_acc_pairs;
    C.tot_pairs = m->d_tot_pairs;
    C.step = m->d_step;
    C.a = p->a;
    C.gamma = p->gamma;
    C.sigma = p->sigma;
    C.rdt = 1.0 / std::sqrt(p->dt);
    C.dt = p->dt;
    C.mass = p->mass;
    C.inv_mass = 1.0 / p->mass;
    C.rc = p->rc;
    C.rc2 = p->rc * p->rc;
    C.H = p->H;
    C.inv_R02 = 1.0 / (p->R0 * p->R0);
    C.key0 = (unsigned)(p->seed & 0xFFFFFFFFull);
    C.key1 = (unsigned)(p->seed >> 32);
    m->cfg.groups = m->n_blocks < GROUP2_BLOCKS ? 1 : (m->n_blocks < GROUP3_BLOCKS ? 2 : 3);
    rc = build_slabs(m, m->cfg.bin_split);
    if (rc == LHMM_OK) rc = prepare_groups(m, m->cfg.groups);
    if (rc != LHMM_OK) {
        release(m);
        delete m;
        return rc;
    }
    *out = m;
    return LHMM_OK;
}

int lhmm_micro_set_state(lhmm_micro* m, const double* s, const double* c, const double* f, const double* h,
                         uint64_t step) {
    g_err.clear();
    if (!m || !s || !c) return fail(LHMM_ERR_ARG, "null argument");
    const size_t N = (size_t)m->n_total;
    for (size_t k = 0; k < 3 * N; ++k) {
        if (!(s[k] >= 0.0 && s[k] < 1.0)) return fail(LHMM_ERR_ARG, "s[%zu] = %g outside [0, 1)", k, s[k]);
        if (!std::isfinite(c[k])) return fail(LHMM_ERR_ARG, "c[%zu] is not finite", k);
        if (f && !std::isfinite(f[k])) return fail(LHMM_ERR_ARG, "f[%zu] is not finite", k);
    }
    if (h)
        for (int b = 0; b < m->n_boxes; ++b)
            if (!cell_ok(h + 9 * b)) return fail(LHMM_ERR_ARG, "box %d: bad cell", b);
    HIPCHK(hipStreamSynchronize(m->stream));
    // AoS double -> SoA real
    std::vector<char> buf(3 * N * m->real_size + 1);
    const double* srcs[3] = {s, c, f};
    void* dsts[3] = {m->d_s, m->d_c, m->d_f};
    for (int which = 0; which < 3; ++which) {
        const double* src = srcs[which];
        if (!src) continue;
        for (size_t i = 0; i < N; ++i)
            for (int k = 0; k < 3; ++k) {
                const double v = src[3 * i + k];
                if (m->precision == LHMM_FP64) {
                    ((double*)buf.data())[k * N + i] = v;
                } else {
                    float x = (float)v;
                    if (which == 0 && x >= 1.0f) x = 0.0f;
                    ((float*)buf.data())[k * N + i] = x;
                }
            }
        HIPCHK(hipMemcpy(dsts[which], buf.data(), 3 * N * m->real_size, hipMemcpyHostToDevice));
    }
    if (h) {
        std::vector<BoxDyn> dyn(m->n_boxes);
        HIPCHK(hipMemcpy(dyn.data(), m->d_dyn, m->n_boxes * sizeof(BoxDyn), hipMemcpyDeviceToHost));
        for (int b = 0; b < m->n_boxes; ++b)
            for (int k = 0; k < 9; ++k) dyn[b].h[k] = h[9 * b + k];
        HIPCHK(hipMemcpy(m->d_dyn, dyn.data(), m->n_boxes * sizeof(BoxDyn), hipMemcpyHostToDevice));
        // captured launches hold the binning's LDS size and the force kernel's
        // variant; a restored snapshot has extents that were set before
        bool taller = false, flat = m->flat;
        for (int b = 0; b < m->n_boxes; ++b) {
            if (h[9 * b + 8] > m->hz[b]) {
                m->hz[b] = h[9 * b + 8];
                taller = true;
            }
            flat = flat || is_flat(m, b, h[9 * b + 8]);
        }
        if (taller) bin_lds(m);
        if (taller || flat != m->flat) drop_graphs(m);
        m->flat = flat;
    }
    unsigned long long st = step;
    HIPCHK(hipMemcpy(m->d_step, &st, sizeof st, hipMemcpyHostToDevice));
    m->have_state = true;
    m->forces_valid = f != nullptr;
    return LHMM_OK;
}

int lhmm_micro_get_state(lhmm_micro* m, double* s, double* c, double* f, double* h, uint64_t* step) {
    g_err.clear();
    if (!m) return fail(LHMM_ERR_ARG, "null engine");
    const size_t N = (size_t)m->n_total, bytes = 3 * N * m->real_size;
    double* const dsts[3] = {s, c, f};
    const void* const srcs[3] = {m->d_s, m->d_c, m->d_f};
    HostStage::Part parts[5];
    int kind[5], n = 0;
    for (int k = 0; k < 3; ++k)
        if (dsts[k]) {
            kind[n] = k;
            parts[n++] = {srcs[k], bytes};
        }
    std::vector<BoxDyn> dyn(h ? m->n_boxes : 0);
    if (h) {
        kind[n] = 3;
        parts[n++] = {m->d_dyn, m->n_boxes * sizeof(BoxDyn)};
    }
    unsigned long long st = 0;
    if (step) {
        kind[n] = 4;
        parts[n++] = {m->d_step, sizeof st};
    }
    HIPCHK(m->stage.read(m->stream, parts, n, [&](int k, size_t at, size_t len, const char* x) {
        if (kind[k] >= 3) {
            memcpy((kind[k] == 3 ? (char*)dyn.data() : (char*)&st) + at, x, len);
        } else if (m->precision == LHMM_FP64) {
            to_rows(dsts[kind[k]], N, at / sizeof(double), (const double*)x, len / sizeof(double));
        } else {
            to_rows(dsts[kind[k]], N, at / sizeof(float), (const float*)x, len / sizeof(float));
        }
    }));
    HIPCHK(hipGetLastError());
    for (size_t b = 0; b < dyn.size(); ++b)
        for (int k = 0; k < 9; ++k) h[9 * b + k] = dyn[b].h[k];
    if (step) *step = st;
    return LHMM_OK;
}

int lhmm_micro_step(lhmm_micro* m, const double* gradL, int32_t n_steps, double* stress_out) {
    g_err.clear();
    if (!m || !gradL || !stress_out) return fail(LHMM_ERR_ARG, "null argument");
    if (n_steps <= 0) return fail(LHMM_ERR_ARG, "n_steps must be positive (got %d)", n_steps);
    if (!m->have_state) return fail(LHMM_ERR_STATE, "no particle state loaded");
    const int bt = 256, bg = (m->n_boxes + bt - 1) / bt;
    HIPCHK(hipEventRecord(m->ev_in, m->user_stream));
    HIPCHK(hipStreamWaitEvent(m->stream, m->ev_in, 0));
    launch_begin_call(m, m->ctx, m->n_boxes, gradL);
    if (!m->forces_valid) {
        launch_force_eval(m);
        m->forces_valid = true;
    }
    HIPCHK(hipGetLastError());
    if (m->p.flags & LHMM_OPT_NO_GRAPH) {
        for (int k = 0; k < n_steps; k += m->cfg.graph_chunk)
            launch_steps(m, all_boxes(m), std::min(m->cfg.graph_chunk, n_steps - k));
    } else {
        const int chunk = n_steps < m->cfg.graph_chunk ? n_steps : m->cfg.graph_chunk;
        const int full = n_steps / chunk, rest = n_steps % chunk;
        hipGraphExec_t g = nullptr;
        int rc = get_graph(m, chunk, &g);
        if (rc != LHMM_OK) return rc;
        for (int k = 0; k < full; ++k) HIPCHK(hipGraphLaunch(g, m->stream));
        if (rest) {
            rc = get_graph(m, rest, &g);
            if (rc != LHMM_OK) return rc;
            HIPCHK(hipGraphLaunch(g, m->stream));
        }
    }
    k_finalize<<<bg, bt, 0, m->stream>>>(m->ctx, stress_out, m->d_parts, 1.0 / n_steps);
    HIPCHK(hipGetLastError());
    HIPCHK(hipEventRecord(m->ev_out, m->stream));
    HIPCHK(hipStreamWaitEvent(m->user_stream, m->ev_out, 0));
    return LHMM_OK;
}

int lhmm_micro_set_config(lhmm_micro* m, const lhmm_micro_config* cfg) {
    g_err.clear();
    if (!m || !cfg) return fail(LHMM_ERR_ARG, "null argument");
    const int qd = cfg->queue_depth;
    const bool qd_ok = qd == 2 || qd == 4 || qd == 8 || qd == 16 || qd == 32;
    if (!qd_ok) return fail(LHMM_ERR_ARG, "queue_depth must be 2, 4, 8, 16 or 32");
    // a search iteration pushes up to scan_unroll(qd) neighbours per lane
    // before it checks the queues, so a lane may hold at most qd - that many
    // when the search resumes
    const int dmax = qd - scan_unroll(qd);
    if (cfg->drain < 0 || cfg->drain > dmax) return fail(LHMM_ERR_ARG, "drain must be in 0..%d", dmax);
    if (cfg->busy_lanes < 1 || cfg->busy_lanes > 65) return fail(LHMM_ERR_ARG, "busy_lanes must be in 1..65");
    if (cfg->bin_threads != 256 && cfg->bin_threads != 512 && cfg->bin_threads != 1024)
        return fail(LHMM_ERR_ARG, "bin_threads must be 256, 512 or 1024");
    if (cfg->graph_chunk < 1 || cfg->graph_chunk > 1000) return fail(LHMM_ERR_ARG, "graph_chunk must be 1..1000");
    if (cfg->prune != 0 && cfg->prune != 1) return fail(LHMM_ERR_ARG, "prune must be 0 or 1");
    if (cfg->fuse_bin != 0 && cfg->fuse_bin != 1) return fail(LHMM_ERR_ARG, "fuse_bin must be 0 or 1");
    if (cfg->groups < 1 || cfg->groups > MAX_GROUPS) return fail(LHMM_ERR_ARG, "groups must be 1..%d", MAX_GROUPS);
    if (cfg->bin_split != 0 && (cfg->bin_split < 256 || cfg->bin_split > 4096))
        return fail(LHMM_ERR_ARG, "bin_split must be 0 or 256..4096");
    HIPCHK(hipStreamSynchronize(m->stream));
    drop_graphs(m);
    const bool reslab = cfg->bin_split != m->cfg.bin_split, regroup = cfg->groups != m->cfg.groups || reslab;
    int rc = reslab ? build_slabs(m, cfg->bin_split) : LHMM_OK;
    if (rc != LHMM_OK) return rc;
    m->cfg = *cfg;
    if (regroup) rc = prepare_groups(m, cfg->groups);
    if (rc != LHMM_OK) m->cfg.groups = 1;
    return rc;
}

int lhmm_micro_set_afbc(lhmm_micro* m, const double* regions, double zeta) {
    g_err.clear();
    if (!m || !regions) return fail(LHMM_ERR_ARG, "null argument");
    if (!(zeta >= 0.0) || !std::isfinite(zeta)) return fail(LHMM_ERR_ARG, "zeta must be finite and >= 0");
    HIPCHK(hipStreamSynchronize(m->stream));
    std::vector<BoxDyn> dyn(m->n_boxes);
    HIPCHK(hipMemcpy(dyn.data(), m->d_dyn, m->n_boxes * sizeof(BoxDyn), hipMemcpyDeviceToHost));
    bool any = false;
    for (int b = 0; b < m->n_boxes; ++b) {
        const double hc = regions[2 * b], hb = regions[2 * b + 1];
        if (hc == 0.0 && hb == 0.0) continue;
        double w[3];
        m3_widths(dyn[b].h, w);
        if (!(hc > 0.0) || !(hb >= hc) || !(hb <= 0.5 * std::min(w[0], w[1])) || !std::isfinite(hb))
            return fail(LHMM_ERR_ARG, "box %d: need 0 < hc <= hb <= half the cell's in-plane width (%g)", b,
                        0.5 * std::min(w[0], w[1]));
        any = true;
    }
    for (int b = 0; b < m->n_boxes; ++b) {
        dyn[b].hc = regions[2 * b];
        dyn[b].hb = regions[2 * b + 1];
        if (dyn[b].hc == 0.0)
            for (int k = 0; k < 4; ++k) dyn[b].G[k] = 0.0;
    }
    HIPCHK(hipMemcpy(m->d_dyn, dyn.data(), m->n_boxes * sizeof(BoxDyn), hipMemcpyHostToDevice));
    m->afbc = any;
    const double dt = m->p.dt;
    m->ctx.ou_damp = std::exp(-0.5 * zeta * dt);
    m->ctx.ou_amp = std::sqrt(m->p.kBT / m->p.mass * (1.0 - std::exp(-zeta * dt)));
    // captured graphs hold the kernel variant and the context
    drop_graphs(m);
    return LHMM_OK;
}

int lhmm_micro_get_config(lhmm_micro* m, lhmm_micro_config* cfg) {
    g_err.clear();
    if (!m || !cfg) return fail(LHMM_ERR_ARG, "null argument");
    *cfg = m->cfg;
    return LHMM_OK;
}

int lhmm_micro_autotune(lhmm_micro* m, const double* gradL, int32_t trial_steps, lhmm_micro_config* best,
                        double* best_ms) {
    g_err.clear();
    if (!m || !gradL) return fail(LHMM_ERR_ARG, "null argument");
    if (trial_steps < 1) return fail(LHMM_ERR_ARG, "trial_steps must be positive");
    if (!m->have_state) return fail(LHMM_ERR_STATE, "no particle state loaded");
    // keep the state (particles, cells, counter, flags) to put it back after every trial
    const size_t bytes = 3 * (size_t)m->n_total * m->real_size;
    void *ss = nullptr, *sc = nullptr, *sf = nullptr, *sdyn = nullptr, *sflags = nullptr, *sout = nullptr;
    unsigned long long step0 = 0;
    int rc = dalloc((char**)&ss, bytes);
    if (rc == LHMM_OK) rc = dalloc((char**)&sc, bytes);
    if (rc == LHMM_OK) rc = dalloc((char**)&sf, bytes);
    if (rc == LHMM_OK) rc = dalloc((char**)&sdyn, sizeof(BoxDyn) * m->n_boxes);
    if (rc == LHMM_OK) rc = dalloc((char**)&sflags, sizeof(unsigned) * m->n_boxes);
    if (rc == LHMM_OK) rc = dalloc((char**)&sout, sizeof(double) * 6 * m->n_boxes);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto done = [&](int code) {
        (void)hipStreamSynchronize(m->stream);
        for (void* q : {ss, sc, sf, sdyn, sflags, sout})
            if (q) (void)hipFree(q);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        return code;
    };
    if (rc != LHMM_OK) return done(rc);
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return done(fail(LHMM_ERR_HIP, "hipEventCreate failed"));
    if (hipStreamSynchronize(m->user_stream) != hipSuccess || sync_engine(m) != LHMM_OK)
        return done(fail(LHMM_ERR_HIP, "synchronisation failed"));
    const bool fv = m->forces_valid;
    auto save = [&]() -> hipError_t {
        hipError_t e = hipMemcpy(ss, m->d_s, bytes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(sc, m->d_c, bytes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(sf, m->d_f, bytes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(sdyn, m->d_dyn, sizeof(BoxDyn) * m->n_boxes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(sflags, m->d_flags, sizeof(unsigned) * m->n_boxes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(&step0, m->d_step, sizeof step0, hipMemcpyDeviceToHost);
        return e;
    };
    auto load = [&]() -> hipError_t {
        hipError_t e = hipStreamSynchronize(m->stream);
        if (e == hipSuccess) e = hipMemcpy(m->d_s, ss, bytes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(m->d_c, sc, bytes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(m->d_f, sf, bytes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(m->d_dyn, sdyn, sizeof(BoxDyn) * m->n_boxes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(m->d_flags, sflags, sizeof(unsigned) * m->n_boxes, hipMemcpyDeviceToDevice);
        if (e == hipSuccess) e = hipMemcpy(m->d_step, &step0, sizeof step0, hipMemcpyHostToDevice);
        m->forces_valid = fv;
        return e;
    };
    if (save() != hipSuccess) return done(fail(LHMM_ERR_HIP, "state copy failed"));
    // mean ms per step of one configuration (one warm-up call, then one timed call)
    auto trial = [&](const lhmm_micro_config& c, double* ms) -> int {
        int r = lhmm_micro_set_config(m, &c);
        if (r != LHMM_OK) return r;
        r = lhmm_micro_step(m, gradL, trial_steps, (double*)sout);
        if (r != LHMM_OK) return r;
        HIPCHK(hipEventRecord(e0, m->user_stream));
        r = lhmm_micro_step(m, gradL, trial_steps, (double*)sout);
        if (r != LHMM_OK) return r;
        HIPCHK(hipEventRecord(e1, m->user_stream));
        HIPCHK(hipEventSynchronize(e1));
        float el = 0.0f;
        HIPCHK(hipEventElapsedTime(&el, e0, e1));
        *ms = el / trial_steps;
        return load() == hipSuccess ? LHMM_OK : fail(LHMM_ERR_HIP, "state restore failed");
    };
    // coordinate search: force-kernel queue, binning workgroup, pruning, graph chunk
    lhmm_micro_config cur = m->cfg;
    double cur_ms = 0.0;
    rc = trial(cur, &cur_ms);
    const int qds[] = {8, 16, 32};
    for (int iq = 0; rc == LHMM_OK && iq < 3; ++iq) {
        const int qd = qds[iq];
        // (drain, busy): full drain range / no busy rule, or rounds driven by busy lanes
        const int dmax = qd - scan_unroll(qd);
        const int cand[4][2] = {{dmax, 65}, {qd / 2 <= dmax ? qd / 2 : dmax, 65}, {dmax, 56}, {0, 65}};
        for (const auto& dc : cand) {
            lhmm_micro_config c = cur;
            c.queue_depth = qd;
            c.drain = dc[0];
            c.busy_lanes = dc[1];
            if (c.queue_depth == cur.queue_depth && c.drain == cur.drain && c.busy_lanes == cur.busy_lanes) continue;
            double ms = 0.0;
            rc = trial(c, &ms);
            if (rc != LHMM_OK) break;
            if (ms < cur_ms) {
                cur = c;
                cur_ms = ms;
            }
        }
    }
    for (int bt : {256, 512, 1024}) {
        if (rc != LHMM_OK || bt == cur.bin_threads) continue;
        lhmm_micro_config c = cur;
        c.bin_threads = bt;
        double ms = 0.0;
        rc = trial(c, &ms);
        if (rc == LHMM_OK && ms < cur_ms) {
            cur = c;
            cur_ms = ms;
        }
    }
    for (int fb : {0, 1}) {
        if (rc != LHMM_OK || fb == cur.fuse_bin) continue;
        lhmm_micro_config c = cur;
        c.fuse_bin = fb;
        double ms = 0.0;
        rc = trial(c, &ms);
        if (rc == LHMM_OK && ms < cur_ms) {
            cur = c;
            cur_ms = ms;
        }
    }
    for (int pr : {0, 1}) {
        if (rc != LHMM_OK || pr == cur.prune) continue;
        lhmm_micro_config c = cur;
        c.prune = pr;
        double ms = 0.0;
        rc = trial(c, &ms);
        if (rc == LHMM_OK && ms < cur_ms) {
            cur = c;
            cur_ms = ms;
        }
    }
    for (int gr : {1, 2, 3}) {
        if (rc != LHMM_OK || gr == cur.groups) continue;
        lhmm_micro_config c = cur;
        c.groups = gr;
        double ms = 0.0;
        rc = trial(c, &ms);
        if (rc == LHMM_OK && ms < cur_ms) {
            cur = c;
            cur_ms = ms;
        }
    }
    for (int ch : {25, 50, 100}) {
        if (rc != LHMM_OK || ch == cur.graph_chunk) continue;
        lhmm_micro_config c = cur;
        c.graph_chunk = ch;
        double ms = 0.0;
        rc = trial(c, &ms);
        if (rc == LHMM_OK && ms < cur_ms) {
            cur = c;
            cur_ms = ms;
        }
    }
    if (rc != LHMM_OK) {
        (void)load();
        return done(rc);
    }
    rc = lhmm_micro_set_config(m, &cur);
    if (rc == LHMM_OK) {
        if (best) *best = cur;
        if (best_ms) *best_ms = cur_ms;
    }
    return done(rc);
}

int lhmm_micro_step_subset(lhmm_micro* m, const double* gradL, int32_t n_steps, double* stress_out,
                           const int32_t* boxes, int32_t n_sel) {
    g_err.clear();
    if (!m || !gradL || !stress_out) return fail(LHMM_ERR_ARG, "null argument");
    if (n_steps <= 0) return fail(LHMM_ERR_ARG, "n_steps must be positive (got %d)", n_steps);
    if (!m->have_state) return fail(LHMM_ERR_STATE, "no particle state loaded");
    const int bt = 256, bg = (m->n_boxes + bt - 1) / bt;
    HIPCHK(hipEventRecord(m->ev_in, m->user_stream));
    HIPCHK(hipStreamWaitEvent(m->stream, m->ev_in, 0));
    Launch L{};
    int rc = select_boxes(m, boxes, n_sel, &L);
    if (rc != LHMM_OK) return rc;
    launch_begin_call(m, L.C, n_sel, gradL);
    if (!m->forces_valid) {
        launch_force_eval(m);
        m->forces_valid = true;
    }
    if (m->p.flags & LHMM_OPT_NO_GRAPH) {
        for (int k = 0; k < n_steps; k += m->cfg.graph_chunk)
            launch_steps(m, L, std::min(m->cfg.graph_chunk, n_steps - k));
    } else {
        const int chunk = n_steps < m->cfg.graph_chunk ? n_steps : m->cfg.graph_chunk;
        int done = 0;
        while (done < n_steps) {
            const int len = n_steps - done >= chunk ? chunk : n_steps - done;
            rc = launch_subset_steps(m, L, len);
            if (rc != LHMM_OK) return rc;
            done += len;
        }
    }
    k_finalize<<<bg, bt, 0, m->stream>>>(m->ctx, stress_out, m->d_parts, 1.0 / n_steps);
    HIPCHK(hipGetLastError());
    HIPCHK(hipEventRecord(m->ev_out, m->stream));
    HIPCHK(hipStreamWaitEvent(m->user_stream, m->ev_out, 0));
    return LHMM_OK;
}

int lhmm_micro_snapshot(lhmm_micro* m) {
    g_err.clear();
    if (!m) return fail(LHMM_ERR_ARG, "null argument");
    if (!m->have_state) return fail(LHMM_ERR_STATE, "no particle state loaded");
    const size_t bytes = 3 * (size_t)m->n_total * m->real_size;
    if (!m->d_snap_s) {
        int rc = dalloc((char**)&m->d_snap_s, bytes);
        if (rc == LHMM_OK) rc = dalloc((char**)&m->d_snap_c, bytes);
        if (rc == LHMM_OK) rc = dalloc((char**)&m->d_snap_f, bytes);
        if (rc == LHMM_OK) rc = dalloc(&m->d_snap_dyn, m->n_boxes);
        if (rc != LHMM_OK) return rc;
    }
    HIPCHK(hipEventRecord(m->ev_in, m->user_stream));
    HIPCHK(hipStreamWaitEvent(m->stream, m->ev_in, 0));
    if (!m->forces_valid) {
        launch_force_eval(m);
        m->forces_valid = true;
    }
    HIPCHK(hipMemcpyAsync(m->d_snap_s, m->d_s, bytes, hipMemcpyDeviceToDevice, m->stream));
    HIPCHK(hipMemcpyAsync(m->d_snap_c, m->d_c, bytes, hipMemcpyDeviceToDevice, m->stream));
    HIPCHK(hipMemcpyAsync(m->d_snap_f, m->d_f, bytes, hipMemcpyDeviceToDevice, m->stream));
    HIPCHK(hipMemcpyAsync(m->d_snap_dyn, m->d_dyn, sizeof(BoxDyn) * m->n_boxes, hipMemcpyDeviceToDevice, m->stream));
    HIPCHK(hipEventRecord(m->ev_out, m->stream));
    HIPCHK(hipStreamWaitEvent(m->user_stream, m->ev_out, 0));
    m->have_snapshot = true;
    return LHMM_OK;
}

int lhmm_micro_restore(lhmm_micro* m, const int32_t* boxes, int32_t n_sel) {
    g_err.clear();
    if (!m) return fail(LHMM_ERR_ARG, "null argument");
    if (!m->have_snapshot) return fail(LHMM_ERR_STATE, "no snapshot taken");
    HIPCHK(hipEventRecord(m->ev_in, m->user_stream));
    HIPCHK(hipStreamWaitEvent(m->stream, m->ev_in, 0));
    Launch L{};
    int rc = select_boxes(m, boxes, n_sel, &L);
    if (rc != LHMM_OK) return rc;
    const Ctx& C = L.C;
    if (m->precision == LHMM_FP64)
        k_restore<double><<<n_sel, 256, 0, m->stream>>>(C, (const double*)m->d_snap_s, (const double*)m->d_snap_c,
                                                        (const double*)m->d_snap_f, m->d_snap_dyn);
    else
        k_restore<float><<<n_sel, 256, 0, m->stream>>>(C, (const float*)m->d_snap_s, (const float*)m->d_snap_c,
                                                       (const float*)m->d_snap_f, m->d_snap_dyn);
    HIPCHK(hipGetLastError());
    HIPCHK(hipEventRecord(m->ev_out, m->stream));
    HIPCHK(hipStreamWaitEvent(m->user_stream, m->ev_out, 0));
    return LHMM_OK;
}

int lhmm_micro_forces(lhmm_micro* m, const double* gradL, double* f_out, double* virial_out) {
    g_err.clear();
    if (!m || !gradL || !f_out) return fail(LHMM_ERR_ARG, "null argument");
    if (!m->have_state) return fail(LHMM_ERR_STATE, "no particle state loaded");
    for (int k = 0; k < 9 * m->n_boxes; ++k)
        if (!std::isfinite(gradL[k])) return fail(LHMM_ERR_ARG, "gradient not finite");
    int rc = sync_engine(m);
    if (rc != LHMM_OK) return rc;
    HIPCHK(hipMemcpy(m->d_gradL, gradL, 9 * m->n_boxes * sizeof(double), hipMemcpyHostToDevice));
    launch_begin_call(m, m->ctx, 0, m->d_gradL, 0);  // gradients only: velocities keep their mean, sums stay
    launch_force_eval(m);
    HIPCHK(hipGetLastError());
    rc = sync_engine(m);
    if (rc != LHMM_OK) return rc;
    m->forces_valid = false;  // the next step recomputes forces with its own gradient
    const size_t N = (size_t)m->n_total;
    std::vector<char> buf(3 * N * m->real_size + 1);
    HIPCHK(hipMemcpy(buf.data(), m->d_f, 3 * N * m->real_size, hipMemcpyDeviceToHost));
    for (size_t i = 0; i < N; ++i)
        for (int k = 0; k < 3; ++k)
            f_out[3 * i + k] = m->precision == LHMM_FP64 ? ((double*)buf.data())[k * N + i]
                                                         : (double)((float*)buf.data())[k * N + i];
    if (virial_out) {
        const size_t nv = (size_t)m->ctx.nv;
        const bool wide = use_wide(m, m->n_blocks);
        std::vector<double> pv((size_t)m->n_blocks * nv * (wide ? WIDE_UNITS : 1));
        HIPCHK(hipMemcpy(pv.data(), m->d_part, pv.size() * sizeof(double), hipMemcpyDeviceToHost));
        for (int b = 0; b < m->n_boxes; ++b) {
            double* o = virial_out + 12 * b;
            for (int q = 0; q < 12; ++q) o[q] = 0.0;
            for (int k = 0; k < m->box[b].nblk; ++k) {
                const size_t blk = (size_t)(m->box[b].blk_off + k);
                for (int q = 0; q < 12; ++q) {
                    double x = 0.0;
                    if (wide) {  // as k_window_sums adds them
                        for (int w = 0; w < 4; ++w) {
                            const double* y = &pv[(blk * WIDE_UNITS + 4 * w) * nv + q];
                            x += (y[0] + y[2 * nv]) + (y[nv] + y[3 * nv]);
                        }
                    } else {
                        x = pv[blk * nv + q];
                    }
                    o[q] += x;
                }
            }
            for (int q = 0; q < 6; ++q) o[q] *= m->ctx.vir_scale;  // ordered pairs count each pair twice
        }
    }
    return LHMM_OK;
}

int lhmm_micro_time(lhmm_micro* m, const double* gradL, int32_t n_steps, double* avg_ms, double* stress_out) {
    g_err.clear();
    if (!m || !gradL || !avg_ms) return fail(LHMM_ERR_ARG, "null argument");
    if (n_steps <= 0) return fail(LHMM_ERR_ARG, "n_steps must be positive (got %d)", n_steps);
    if (!m->have_state) return fail(LHMM_ERR_STATE, "no particle state loaded");
    const int bt = 256, bg = (m->n_boxes + bt - 1) / bt;
    hipEvent_t ev[2 * LHMM_N_KERNELS];
    for (auto& e : ev) HIPCHK(hipEventCreate(&e));
    HIPCHK(hipEventRecord(m->ev_in, m->user_stream));
    HIPCHK(hipStreamWaitEvent(m->stream, m->ev_in, 0));
    launch_begin_call(m, m->ctx, m->n_boxes, gradL);
    if (!m->forces_valid) {
        launch_force_eval(m);
        m->forces_valid = true;
    }
    double sum[LHMM_N_KERNELS] = {0, 0, 0, 0, 0, 0};
    int rc = LHMM_OK;
    auto around = [&](int q, int after) {
        (void)hipEventRecord(ev[2 * q + after], m->stream);
        if (!after || rc != LHMM_OK) return;
        float ms = 0.f;
        if (hipEventSynchronize(ev[2 * q + 1]) != hipSuccess || hipEventElapsedTime(&ms, ev[2 * q], ev[2 * q + 1]) != hipSuccess)
            rc = fail(LHMM_ERR_HIP, "timing of a kernel failed");
        sum[q] += ms;
    };
    for (int k = 0; k < n_steps && rc == LHMM_OK; k += m->cfg.graph_chunk) {
        const int n = std::min(m->cfg.graph_chunk, n_steps - k);
        if (m->precision == LHMM_FP64)
            launch_steps<double>(m, all_boxes(m), n, true, around);
        else
            launch_steps<float>(m, all_boxes(m), n, true, around);
    }
    if (rc == LHMM_OK) {
        for (int q = 0; q < LHMM_N_KERNELS; ++q) avg_ms[q] = sum[q] / n_steps;
        if (stress_out) k_finalize<<<bg, bt, 0, m->stream>>>(m->ctx, stress_out, m->d_parts, 1.0 / n_steps);
        hipError_t e = hipStreamSynchronize(m->stream);
        if (e != hipSuccess) rc = fail(LHMM_ERR_HIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
    }
    for (auto& e : ev) (void)hipEventDestroy(e);
    return rc;
}

int lhmm_micro_stress_parts(lhmm_micro* m, double* parts_out) {
    g_err.clear();
    if (!m || !parts_out) return fail(LHMM_ERR_ARG, "null argument");
    std::vector<double> v((size_t)ACC * m->n_boxes);
    int rc = read_back(m, v.data(), m->d_parts, v.size() * sizeof(double));
    if (rc != LHMM_OK) return rc;
    for (int b = 0; b < m->n_boxes; ++b)
        for (int q = 0; q < 18; ++q) parts_out[18 * (size_t)b + q] = v[(size_t)ACC * b + q];
    return LHMM_OK;
}

int lhmm_micro_components(lhmm_micro* m, double* out) {
    g_err.clear();
    if (!m || !out) return fail(LHMM_ERR_ARG, "null argument");
    if (!(m->p.flags & LHMM_OPT_COMPONENTS))
        return fail(LHMM_ERR_STATE, "the engine was created without LHMM_OPT_COMPONENTS");
    std::vector<double> v((size_t)ACC * m->n_boxes);
    int rc = read_back(m, v.data(), m->d_parts, v.size() * sizeof(double));
    if (rc != LHMM_OK) return rc;
    // sums: kinetic 0, pair 6, FENE 12, C 18, D 24, R 30 -> kin, C, D, R, FENE
    const int src[5] = {0, 18, 24, 30, 12};
    for (int b = 0; b < m->n_boxes; ++b)
        for (int part = 0; part < 5; ++part)
            for (int q = 0; q < 6; ++q) out[30 * (size_t)b + 6 * part + q] = v[(size_t)ACC * b + src[part] + q];
    return LHMM_OK;
}

int lhmm_micro_pair_total(lhmm_micro* m, uint64_t* pairs_out) {
    g_err.clear();
    if (!m || !pairs_out) return fail(LHMM_ERR_ARG, "null argument");
    std::vector<unsigned long long> v(m->n_boxes);
    int rc = read_back(m, v.data(), m->d_tot_pairs, m->n_boxes * sizeof(unsigned long long));
    if (rc != LHMM_OK) return rc;
    for (int b = 0; b < m->n_boxes; ++b) pairs_out[b] = v[b];
    return LHMM_OK;
}

int lhmm_micro_prepare(lhmm_micro* m, int32_t n_steps) {
    g_err.clear();
    if (!m) return fail(LHMM_ERR_ARG, "null engine");
    if (n_steps <= 0) return fail(LHMM_ERR_ARG, "n_steps must be positive (got %d)", n_steps);
    if (m->p.flags & LHMM_OPT_NO_GRAPH) return LHMM_OK;
    const int chunk = n_steps < m->cfg.graph_chunk ? n_steps : m->cfg.graph_chunk;
    hipGraphExec_t g = nullptr;
    int rc = get_graph(m, chunk, &g);
    if (rc == LHMM_OK && n_steps % chunk) rc = get_graph(m, n_steps % chunk, &g);
    return rc;
}

int lhmm_micro_pair_counts(lhmm_micro* m, uint64_t* pairs_out) {
    g_err.clear();
    if (!m || !pairs_out) return fail(LHMM_ERR_ARG, "null argument");
    std::vector<unsigned long long> v(m->n_boxes);
    int rc = read_back(m, v.data(), m->d_acc_pairs, m->n_boxes * sizeof(unsigned long long));
    if (rc != LHMM_OK) return rc;
    for (int b = 0; b < m->n_boxes; ++b) pairs_out[b] = v[b];
    return LHMM_OK;
}

int lhmm_micro_flags(lhmm_micro* m, uint32_t* flags_out, int32_t clear) {
    g_err.clear();
    if (!m || !flags_out) return fail(LHMM_ERR_ARG, "null argument");
    int rc = read_back(m, flags_out, m->d_flags, m->n_boxes * sizeof(unsigned));
    if (rc != LHMM_OK) return rc;
    if (clear) HIPCHK(hipMemsetAsync(m->d_flags, 0, m->n_boxes * sizeof(unsigned), m->stream));
    return LHMM_OK;
}

int lhmm_micro_sizes(const lhmm_micro* m, int64_t* n_total, int32_t* n_boxes) {
    g_err.clear();
    if (!m) return fail(LHMM_ERR_ARG, "null engine");
    if (n_total) *n_total = m->n_total;
    if (n_boxes) *n_boxes = m->n_boxes;
    return LHMM_OK;
}

int lhmm_micro_destroy(lhmm_micro* m) {
    g_err.clear();
    if (!m) return LHMM_OK;
    release(m);
    delete m;
    return LHMM_OK;
}

}  // extern "C"
