// lhmm_mlp.h -- fused kernels of the stress surrogate (lhmm_sur.hip): the
// forward pass of a tile of rows in one launch, and a training step in three.
//
// Shapes of the ensemble are small (5 x 129-256-256-3 in this framework), so
// what a layer-by-layer pass waits for is launches, latency and the traffic
// of activations, not the matrix cores.  Here one workgroup takes 32 rows of
// one member through every layer with the activations in LDS:
//   k_mlp_rows<train = false>  X -> Y;
//   k_mlp_rows<train = true>   X -> Y -> dY -> dZ2 -> dZ1, GELU's derivative
//                              kept in registers from the forward half;
//   k_mlp_dw                   the three weight gradients' partial products
//                              and the bias gradients' partial sums;
//   k_mlp_update               partials summed in order, Adam, BF16 copies
//                              and the loss.
// Each product runs the same matrix instruction over the reduction index in
// the same order as the layer-wise pass does, and the sums over rows keep its
// order too: losses, gradients and weights are the same to the bit.
//
// Operands are kept packed by matrix fragment: element (row, k) of an
// operand with reduction index k sits at
//   ((row / 32) (K / 16) + k / 16) 512 + lane 8 + k % 8,
//   lane = row % 32 + 32 ((k % 16) / 8),
// so that a wave reads the 1 KiB of one 32 x 16 fragment contiguously.
#ifndef LHMM_MLP_H
#define LHMM_MLP_H

#include <hip/hip_runtime.h>

namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// Waves of a k_mlp_rows workgroup, one 32-column tile each at a time.  In layers
// of one or two tiles the others only load: two waves do there, from more
// workgroups than the chip takes at once with eight (four a CU), 5 x 30000 rows
// of 129-32-32-32 64 us with eight waves and 46 with two (layer by layer 59),
// their training step 317 and 198; 5 x 700 rows 12.0 and 13.5.  Training
// transposes the features as well, with eight waves where they are many (3000
// rows of 1700-32-32-3: 153 us and 208).
constexpr int MLP_WAVES = 8, MLP_NARROW_WAVES = 2;
inline bool mlp_few_waves(bool train, int workgroups, int nin_p) { return workgroups > 1024 && (!train || nin_p <= 320); }
constexpr int MLP_MAX_NH = 64 * MLP_WAVES;  // two tiles per wave
constexpr int MLP_PAD = 8;      // bf16 of padding per LDS row (16-byte reads of 32 rows spread over the banks)
constexpr size_t MLP_LDS_MAX = 150 * 1024;

struct MlpArgs {
    const float* X;  // B x nin
    const float* T;  // B x nout (training)
    float* Y;        // E x B x nout (inference)
    int B, Bp, nin, nin_p, nh, nout;
    // packed weights, member after member: forward operands [out x in], and
    // for backward W2, W3 as [in x out]
    const bf16 *W1f, *W2f, *W3f, *W2r, *W3r;
    const float *b1, *b2, *b3;
    // training outputs, packed as operands of the weight gradients (reduction over rows)
    bf16 *Xt, *H1t, *H2t, *dYt, *dZ2t, *dZ1t;
    float *dYf, *dZ2f, *dZ1f;  // FP32, row-major, for the bias gradients
    float* ploss;              // E x Bp / 8: squared errors of eight rows
};

// features in LDS at a time: xcols
inline size_t mlp_lds_bytes(int xcols, int nh) {
    return sizeof(bf16) * 32 * ((size_t)(xcols + MLP_PAD) + 2 * (size_t)(nh + MLP_PAD) + 32 + MLP_PAD);
}

// Weight fragments in flight per wave, so that a product of 16 k-steps does
// not wait for L2 at every step.  Inference: 4 (14.3 us for 217 rows, 8 take
// 15.5: the registers hold fewer waves).  Training keeps GELU' in registers
// and has two workgroups per CU either way: 8 (64 us for 5 x 4096 rows, 4 took
// 67); so does a wide forward pass.
constexpr int mlp_pf(bool train, bool wide) { return train || wide ? 8 : 4; }

template <int PF>
__device__ __forceinline__ void mlp_preload(bf16x8 (&b)[PF], const bf16* w, int KS, int l) {
    const bf16x8* p = (const bf16x8*)w + l;
#pragma unroll
    for (int i = 0; i < PF; ++i) b[i] = p[min(i, KS - 1) * 64];
}

// acc += A W^T for one 32-column tile: A rows in LDS (row stride lda), the
// tile's packed fragments at w, the first PF of them in b already.
template <int PF>
__device__ __forceinline__ void mlp_tile(floatx16& acc, bf16x8 (&b)[PF], const bf16* As, int lda, const bf16* w,
                                         int KS, int l) {
    const bf16x8* p = (const bf16x8*)w + l;
    const bf16* a = As + (l & 31) * lda + 8 * (l >> 5);
    for (int k0 = 0; k0 < KS; k0 += PF) {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            if (k0 + i < KS) {
                const bf16x8 av = *(const bf16x8*)(a + 16 * (k0 + i));
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, b[i], acc, 0, 0, 0);
                if (k0 + PF + i < KS) b[i] = p[(k0 + PF + i) * 64];
            }
        }
    }
}

// The tile's four consecutive rows vg of lane l's column, stored into the
// packed operand whose reduction index is the row of the batch.
__device__ __forceinline__ void mlp_store_t(bf16* base, int t, int KSB, int R0, int vg, int l, bf16x4 q) {
    *(bf16x4*)(base + ((size_t)t * KSB + R0 / 16 + (vg >> 1)) * 512 + ((l & 31) + 32 * (vg & 1)) * 8 + 4 * (l >> 5)) = q;
}

// One workgroup per (32 rows, member), 32 the smallest tile of the matrix
// instruction.  NTW: 32-column tiles per wave and hidden layer.  Measured (5
// members 129-256-256-3): inference of 3572 rows 21.4 us against 57.7 layer by
// layer, 217 rows 13.4 against 37.6 (22.6 and 14.3 with features loaded one
// by one); the rows of a 4096-row training step 58 us against 200.  Bound by the
// GELU: 52 vector instructions per hidden value and wave, all others included,
// fill 12 of the 21 us, on the 2 or 3 workgroups that share a CU; in training
// (33 of 58 us) by 85 MB of transposed operands and FP32 dZ written as well.  GELU' parked in
// memory instead of registers (three workgroups per CU) took 73 us.
//
// WIDE (inference, more than mlp_xcols features): they pass through LDS that many
// at a time, the next ones on their way while these are multiplied, in
// the same order.  With all of them in LDS a CU held one workgroup, whose loads
// waited for one another: 5 x 12000 rows of 1250-128-128-3 193 us layer by
// layer, 390 with all features in LDS, 113 in pieces; 1700-32-32-3 113, 490 and
// 92; 400-32-32-3 44, 47 and 36.
constexpr int mlp_xcols(int waves) { return waves == MLP_NARROW_WAVES ? 192 : 320; }

template <bool TRAIN, int NTW, bool WIDE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_mlp_rows(MlpArgs g) {
    static_assert(!(TRAIN && WIDE), "training reads all features again");
    constexpr int XC = mlp_xcols(WAVES), RW = 32 / WAVES;  // features loaded at a time; rows of a wave
    extern __shared__ __align__(16) unsigned char mlp_lds[];
    const int ldx = (WIDE ? XC : g.nin_p) + MLP_PAD, ldh = g.nh + MLP_PAD, ldy = 32 + MLP_PAD;
    bf16* Xs = (bf16*)mlp_lds;
    bf16* Ha = Xs + 32 * ldx;
    bf16* Hb = Ha + 32 * ldh;
    bf16* Ys = Hb + 32 * ldh;
    const int e = blockIdx.y, R0 = blockIdx.x * 32;
    const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;
    const int nt = g.nh / 32, KS1 = g.nin_p / 16, KSH = g.nh / 16, KSB = g.Bp / 16;
    const bf16* W1 = g.W1f + (size_t)e * g.nin_p * g.nh;
    const bf16* W2 = g.W2f + (size_t)e * g.nh * g.nh;
    const bf16* W3 = g.W3f + (size_t)e * 32 * g.nh;
    bf16x8 b[mlp_pf(TRAIN, WIDE)];
    // the rows, rounded to BF16, XC features in flight; rows and columns of the
    // padding are zero
    float x[RW][XC / 64];  // rows wv, wv + WAVES, ..
    auto load = [&](int c0) {
#pragma unroll
        for (int k = 0; k < XC / 64; ++k)
            if (c0 + 64 * k < g.nin_p)
#pragma unroll
                for (int q = 0; q < RW; ++q) {
                    const int r = wv + WAVES * q, c = c0 + 64 * k + l;
                    x[q][k] = (R0 + r < g.B && c < g.nin) ? g.X[(size_t)(R0 + r) * g.nin + c] : 0.0f;
                }
    };
    auto keep = [&](int c0, int at) {  // features c0 .. to column at of the LDS rows
#pragma unroll
        for (int k = 0; k < XC / 64; ++k)
            if (c0 + 64 * k + l < g.nin_p)
#pragma unroll
                for (int q = 0; q < RW; ++q) Xs[(wv + WAVES * q) * ldx + at + 64 * k + l] = (bf16)x[q][k];
    };
    floatx16 acc1[NTW] = {};  // WIDE: the first layer's products
    load(0);
    if constexpr (WIDE) {
        auto ksteps = [&](int c0) { return min(XC, g.nin_p - c0) / 16; };
        auto weights = [&](int j, int c0) { return W1 + ((size_t)(wv + WAVES * j) * KS1 + c0 / 16) * 512; };
        if (wv < nt) mlp_preload(b, weights(0, 0), ksteps(0), l);
        for (int c0 = 0; c0 < g.nin_p; c0 += XC) {
            if (c0 > 0) __syncthreads();
            keep(c0, 0);
            __syncthreads();
            if (c0 + XC < g.nin_p) load(c0 + XC);
#pragma unroll
            for (int j = 0; j < NTW; ++j)
                if (wv + WAVES * j < nt) {
                    if (j > 0) mlp_preload(b, weights(j, c0), ksteps(c0), l);
                    mlp_tile(acc1[j], b, Xs, ldx, weights(j, c0), ksteps(c0), l);
                }
            if (wv < nt && c0 + XC < g.nin_p) mlp_preload(b, weights(0, c0 + XC), ksteps(c0 + XC), l);
        }
    } else {
        if (wv < nt) mlp_preload(b, W1 + (size_t)wv * KS1 * 512, KS1, l);
        for (int c0 = 0; c0 < g.nin_p; c0 += XC) {
            if (c0 > 0) load(c0);
            keep(c0, c0);
        }
        __syncthreads();
    }
    if (TRAIN && e == 0) {  // X as the weight gradient reads it, once for all members
        for (int q = tid; q < 4 * g.nin_p; q += 64 * WAVES) {
            const int c = q >> 2, s = q & 3;  // feature, group of eight rows
            bf16x8 v;
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = Xs[(8 * s + u) * ldx + c];
            *(bf16x8*)(g.Xt + ((size_t)(c / 32) * KSB + R0 / 16 + (s >> 1)) * 512 + ((c & 31) + 32 * (s & 1)) * 8) = v;
        }
    }
    floatx16 d1[TRAIN ? NTW : 1], d2[TRAIN ? NTW : 1];  // GELU'(Z1), GELU'(Z2) of the wave's tiles
    // one hidden layer: As -> Hs (and, training, its transpose and derivative);
    // done: its products, where they are there already
    auto hidden = [&](const bf16* As, int lda, const bf16* W, int KS, const float* bias, bf16* Hs, bf16* Ht,
                      floatx16* d, const bf16* Wnext, int KSn, int ntn, const floatx16* done) {
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
            const int t = wv + WAVES * j;
            if (t < nt) {
                floatx16 acc{};
                if (done) {
                    acc = done[j];
                } else {
                    if (j > 0) mlp_preload(b, W + (size_t)t * KS * 512, KS, l);
                    mlp_tile(acc, b, As, lda, W + (size_t)t * KS * 512, KS, l);
                }
                // the next product's first fragments travel during the GELU
                if (j + 1 == NTW || t + WAVES >= nt)
                    if (wv < ntn) mlp_preload(b, Wnext + (size_t)wv * KSn * 512, KSn, l);
                const int col = 32 * t + (l & 31);
                const float bv = bias[(size_t)e * g.nh + col];
#pragma unroll
                for (int vg = 0; vg < 4; ++vg) {
                    const int r0 = 8 * vg + 4 * (l >> 5);
                    bf16x4 q;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float z = acc[4 * vg + u] + bv;
                        const bf16 h = (bf16)gelu_f(z);
                        Hs[(r0 + u) * ldh + col] = h;
                        if (TRAIN) {
                            q[u] = h;
                            d[j][4 * vg + u] = gelu_grad_f(z);
                        }
                    }
                    if (TRAIN) mlp_store_t(Ht + (size_t)e * g.nh * g.Bp, t, KSB, R0, vg, l, q);
                }
            }
        }
        __syncthreads();
    };
    hidden(Xs, ldx, W1, KS1, g.b1, Ha, g.H1t, d1, W2, KSH, nt, WIDE ? acc1 : nullptr);
    hidden(Ha, ldh, W2, KSH, g.b2, Hb, g.H2t, d2, W3, KSH, 1, nullptr);
    if (wv == 0) {
        floatx16 acc{};
        mlp_tile(acc, b, Hb, ldh, W3, KSH, l);
        const int col = l & 31;
        const float bv = g.b3[(size_t)e * 32 + col];
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
            bf16x4 q;
            float sq[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int r = 8 * vg + 4 * (l >> 5) + u, row = R0 + r;
                const float y = acc[4 * vg + u] + bv;
                const bool real = row < g.B && col < g.nout;
                if (!TRAIN) {
                    if (real) g.Y[((size_t)e * g.B + row) * g.nout + col] = y;
                } else {
                    // mean squared error: dY = 2 (Y - T) / (B n_out), 0 on padding
                    float d = 0.0f;
                    sq[u] = 0.0f;
                    if (real) {
                        const float diff = y - g.T[(size_t)row * g.nout + col];
                        sq[u] = __fmul_rn(diff, diff);
                        d = 2.0f * diff / (float)(g.B * g.nout);
                    }
                    g.dYf[((size_t)e * g.Bp + row) * 32 + col] = d;
                    q[u] = (bf16)d;
                    Ys[r * ldy + col] = q[u];
                }
            }
            if (TRAIN) {
                mlp_store_t(g.dYt + (size_t)e * 32 * g.Bp, 0, KSB, R0, vg, l, q);
                // eight rows by 32 columns: rows four, two and one apart, then the columns
#pragma unroll
                for (int u = 0; u < 4; ++u) sq[u] += __shfl_xor(sq[u], 32, 64);
                float x = (sq[0] + sq[2]) + (sq[1] + sq[3]);
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
                if (l == 0) g.ploss[(size_t)e * (g.Bp / 8) + R0 / 8 + vg] = x;
            }
        }
    }
    if (!TRAIN) return;
    // backward of a hidden layer: dZ = (dOut W^T) GELU'(Z); dOut in LDS
    auto back = [&](const bf16* As, int lda, const bf16* W, int KS, const floatx16* d, bf16* Zs, bf16* Zt, float* Zf) {
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
            const int t = wv + WAVES * j;
            if (t < nt) {
                floatx16 acc{};
                if (j > 0) mlp_preload(b, W + (size_t)t * KS * 512, KS, l);
                mlp_tile(acc, b, As, lda, W + (size_t)t * KS * 512, KS, l);
                const int col = 32 * t + (l & 31);
#pragma unroll
                for (int vg = 0; vg < 4; ++vg) {
                    bf16x4 q;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int r = 8 * vg + 4 * (l >> 5) + u;
                        const float dz = acc[4 * vg + u] * d[j][4 * vg + u];
                        Zf[((size_t)e * g.Bp + R0 + r) * g.nh + col] = dz;
                        q[u] = (bf16)dz;
                        if (Zs) Zs[r * ldh + col] = q[u];
                    }
                    mlp_store_t(Zt + (size_t)e * g.nh * g.Bp, t, KSB, R0, vg, l, q);
                }
            }
        }
    };
    const bf16* W3r = g.W3r + (size_t)e * 32 * g.nh;
    const bf16* W2r = g.W2r + (size_t)e * g.nh * g.nh;
    if (wv < nt) mlp_preload(b, W3r + (size_t)wv * 2 * 512, 2, l);
    __syncthreads();
    back(Ys, ldy, W3r, 2, d2, Ha, g.dZ2t, g.dZ2f);
    if (wv < nt) mlp_preload(b, W2r + (size_t)wv * KSH * 512, KSH, l);
    __syncthreads();
    back(Ha, ldh, W2r, KSH, d1, nullptr, g.dZ1t, g.dZ1f);
}

// Partial products of the three weight gradients dW = A B^T over chunks of
// the batch, one wave per 2 x 2 tiles and chunk.  A: inputs (shared by the
// members), H1, H2; B: dZ1, dZ2, dY, all packed; the partials are row-major
// per member and chunk.  Units are numbered matrix after matrix, chunk after
// chunk; after them come the bias gradients, a wave per 64 columns and row
// slice: rows y, y + 16, ... of the slice are added in order for each y, then
// the 16 partials in order, sixteen independent loads in flight.
constexpr int COLSUM_SLICES = 16;

struct DwVec {
    const float* x;  // E x Bp x n, row-major
    float* part;     // E x COLSUM_SLICES x n
    int n, u0;
};
struct DwMat {
    const bf16 *A, *B;
    long sA, sB;    // member strides
    int mt, ntl;    // tiles
    int u0;         // first unit
    float* part;    // E x chunks x (32 mt) x (32 ntl)
};
struct DwArgs {
    DwMat m[3];
    DwVec b[3];
    int units, chunks, KSB, kschunk;
};

__global__ __launch_bounds__(64) void k_mlp_dw(DwArgs g) {
    const int e = blockIdx.y, l = threadIdx.x;
    const int n_mat = g.units * g.chunks;
    if ((int)blockIdx.x >= n_mat) {
        const int w = blockIdx.x - n_mat;
        const DwVec& V = w >= g.b[2].u0 ? g.b[2] : (w >= g.b[1].u0 ? g.b[1] : g.b[0]);
        const int z = (w - V.u0) % COLSUM_SLICES, col = 64 * ((w - V.u0) / COLSUM_SLICES) + l;
        const int rows = 16 * g.KSB, len = (rows + COLSUM_SLICES - 1) / COLSUM_SLICES;
        const int r0 = z * len, r1 = min(rows, r0 + len);
        if (col >= V.n) return;
        const float* x = V.x + (size_t)e * rows * V.n + col;
        float s[16];
#pragma unroll
        for (int y = 0; y < 16; ++y) s[y] = 0.0f;
        int r = r0;
        for (; r + 16 <= r1; r += 16)
#pragma unroll
            for (int y = 0; y < 16; ++y) s[y] += x[(size_t)(r + y) * V.n];
#pragma unroll
        for (int y = 0; y < 16; ++y)
            if (r + y < r1) s[y] += x[(size_t)(r + y) * V.n];
        float t = 0.0f;
#pragma unroll
        for (int y = 0; y < 16; ++y) t += s[y];
        V.part[((size_t)e * COLSUM_SLICES + z) * V.n + col] = t;
        return;
    }
    const int u = blockIdx.x / g.chunks, c = blockIdx.x % g.chunks;
    const DwMat& M = u >= g.m[2].u0 ? g.m[2] : (u >= g.m[1].u0 ? g.m[1] : g.m[0]);
    const int v = u - M.u0, nn = (M.ntl + 1) / 2;
    const int tm = 2 * (v / nn), tn = 2 * (v % nn);
    // an odd last tile is computed twice and stored once
    const int tm1 = min(tm + 1, M.mt - 1), tn1 = min(tn + 1, M.ntl - 1);
    const int k0 = c * g.kschunk, k1 = min(k0 + g.kschunk, g.KSB);
    const bf16x8* a0 = (const bf16x8*)(M.A + e * M.sA + (size_t)tm * g.KSB * 512) + l;
    const bf16x8* a1 = (const bf16x8*)(M.A + e * M.sA + (size_t)tm1 * g.KSB * 512) + l;
    const bf16x8* b0 = (const bf16x8*)(M.B + e * M.sB + (size_t)tn * g.KSB * 512) + l;
    const bf16x8* b1 = (const bf16x8*)(M.B + e * M.sB + (size_t)tn1 * g.KSB * 512) + l;
    constexpr int PF = 4;
    bf16x8 f[PF][4];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        const int k = min(k0 + i, k1 - 1) * 64;
        f[i][0] = a0[k]; f[i][1] = a1[k]; f[i][2] = b0[k]; f[i][3] = b1[k];
    }
    floatx16 acc[4] = {floatx16{}, floatx16{}, floatx16{}, floatx16{}};
    for (int kb = k0; kb < k1; kb += PF) {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            if (kb + i < k1) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i][q >> 1], f[i][2 + (q & 1)], acc[q], 0, 0, 0);
                const int k = min(kb + PF + i, k1 - 1) * 64;
                f[i][0] = a0[k]; f[i][1] = a1[k]; f[i][2] = b0[k]; f[i][3] = b1[k];
            }
        }
    }
    const int N = 32 * M.ntl;
    float* out = M.part + ((size_t)e * g.chunks + c) * 32 * M.mt * N;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if ((q >> 1) && tm + 1 >= M.mt) continue;
        if ((q & 1) && tn + 1 >= M.ntl) continue;
        float* o = out + (size_t)(32 * (tm + (q >> 1)) + 4 * (l >> 5)) * N + 32 * (tn + (q & 1)) + (l & 31);
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) o[(size_t)(8 * (vv >> 2) + (vv & 3)) * N] = acc[q][vv];
    }
}

// Gradients from their partials (chunks added in order), one Adam step on
// the FP32 masters, and the packed BF16 copies.  The first blocks take the
// weights, a thread eight consecutive rows (the reduction index of the
// forward operand) of one column, so the forward copy is one 16-byte store;
// then come the biases (a thread per column) and one block per member for
// the loss.
struct UpMat {
    float *w, *g, *m, *v;
    const float* part;
    bf16 *f, *r;   // packed copies: forward operand [cols x rows], backward operand [rows x cols] (may be null)
    int rows, cols;
    int blk0;      // first block
};
struct UpVec {
    float *w, *g, *m, *v;
    const float* part;  // E x COLSUM_SLICES x n
    int n, blk0;
};
struct UpArgs {
    UpMat m[3];
    UpVec b[3];
    int loss0;  // first loss block
    int E, chunks, nparts, B, nout;  // nparts: loss partials per member (0: no gradients, as in chunks)
    float lr, c1, c2;
    const float* ploss;
    float* loss;  // may be null
};

__device__ __forceinline__ float adam_step(float w, float g, float& m, float& v, float lr, float c1, float c2) {
    m = 0.9f * m + 0.1f * g;
    v = 0.999f * v + 0.001f * g * g;
    return w - lr * (m / c1) / (sqrtf(v / c2) + 1e-8f);
}

__global__ __launch_bounds__(256) void k_mlp_update(UpArgs g) {
    __shared__ double sh[256];
    const int blk = blockIdx.x, tid = threadIdx.x;
    if (blk < g.b[0].blk0) {
        const UpMat& M = blk >= g.m[2].blk0 ? g.m[2] : (blk >= g.m[1].blk0 ? g.m[1] : g.m[0]);
        const long per = (long)(M.rows / 8) * M.cols;
        const long t = (long)(blk - M.blk0) * 256 + tid;
        if (t >= per * g.E) return;
        const int e = (int)(t / per);
        const int q = (int)(t - e * per);
        const int r0 = 8 * (q / M.cols), c = q % M.cols;
        const size_t RC = (size_t)M.rows * M.cols, base = e * RC + (size_t)r0 * M.cols + c;
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (g.chunks > 0) {
            const float* p = M.part + (size_t)e * g.chunks * RC + (size_t)r0 * M.cols + c;
            for (int k = 0; k < g.chunks; ++k)
#pragma unroll
                for (int u = 0; u < 8; ++u) s[u] += p[(size_t)k * RC + (size_t)u * M.cols];
        }
        bf16x8 h;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const size_t i = base + (size_t)u * M.cols;
            float m = M.m[i], v = M.v[i];
            const float w = adam_step(M.w[i], s[u], m, v, g.lr, g.c1, g.c2);
            M.g[i] = s[u];
            M.m[i] = m;
            M.v[i] = v;
            M.w[i] = w;
            h[u] = (bf16)w;
            if (M.r) {
                const int r = r0 + u;
                M.r[e * RC + ((size_t)(r / 32) * (M.cols / 16) + c / 16) * 512 + (r % 32 + 32 * ((c % 16) / 8)) * 8 + c % 8] = h[u];
            }
        }
        *(bf16x8*)(M.f + e * RC + ((size_t)(c / 32) * (M.rows / 16) + r0 / 16) * 512 + (c % 32 + 32 * ((r0 % 16) / 8)) * 8) = h;
        return;
    }
    if (blk < g.loss0) {
        const UpVec& V = blk >= g.b[2].blk0 ? g.b[2] : (blk >= g.b[1].blk0 ? g.b[1] : g.b[0]);
        const long i = (long)(blk - V.blk0) * 256 + tid;
        if (i >= (long)g.E * V.n) return;
        const int e = (int)(i / V.n), c = (int)(i % V.n);
        float s = 0.0f;
        if (g.chunks > 0)
#pragma unroll
            for (int z = 0; z < COLSUM_SLICES; ++z) s += V.part[((size_t)e * COLSUM_SLICES + z) * V.n + c];
        float m = V.m[i], v = V.v[i];
        V.w[i] = adam_step(V.w[i], s, m, v, g.lr, g.c1, g.c2);
        V.g[i] = s;
        V.m[i] = m;
        V.v[i] = v;
        return;
    }
    const int e = blk - g.loss0;
    double s = 0.0;
    for (int t = tid; t < g.nparts; t += 256) s += (double)g.ploss[(size_t)e * g.nparts + t];
    sh[tid] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) sh[tid] += sh[tid + o];
        __syncthreads();
    }
    if (tid == 0 && g.loss) g.loss[e] = (float)(sh[0] / (double)(g.B * g.nout));
}

}  // namespace

#endif  // LHMM_MLP_H
